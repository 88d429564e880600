"""The decoding calls whose speed is tracked, and how their inputs are made.

Every case goes through the public binding (`paper_2510_09085_amd.binding`): a one-shot
`decode` of a batch whose workspace the caller keeps, or a live `Stream` session that is fed
chunk by chunk.  `listed()` names a dozen of them, from one short utterance to batches that
fill the chip; `draw(rng)` gives one more of the same ranges:

    batch      1 .. 4096 utterances of 20 .. 1500 frames (20 ms each), equal or ragged lengths
    vocabulary 24 .. 4096 tokens (characters to sub-words), multiples of four and odd sizes
    beam       4 .. 1000 entries (streams: up to 512)
    threshold  R = 0.1 .. 0.001, or 0 (every token is kept)
    options    static top-N, score window, bigram table (in LDS or gathered), n-best, traces
    streams    1 .. 64 live streams, chunks of 5 .. 50 frames

Emissions follow the recipe of `synth.py` (sharply peaked log-softmax rows, 65% blank frames, a
share of frames with a second strong token), drawn on the GPU in fp64 and rounded once to fp32.
"""
from __future__ import annotations

import math

import torch

from paper_2510_09085_amd import binding, synth

TRANSCRIPT_LEN = 60
MOST_EMISSION_BYTES = 4 * 4096 * 500 * 32  # of the largest listed batch
MOST_TRIE_BYTES = 1 << 30                  # what that batch's beam needs of the workspace
MOST_SECONDS = 0.025                       # estimate for a drawn case (the longest listed: 0.04)


def _decode(name, B, T, V, beam, r, **more):
    case = {"name": name, "kind": "decode", "B": B, "T": T, "V": V, "beam": beam, "r": r,
            "hard_rate": 0.10, "zipf": 0.0, "ragged": False, "top_n": 0, "window": 0.0,
            "lm": False, "nbest": False, "traces": False}
    case.update(more)
    return case


def _stream(name, B, chunk, chunks, V, beam, r, **more):
    case = {"name": name, "kind": "stream", "B": B, "T": chunk * chunks, "chunk": chunk, "V": V,
            "beam": beam, "r": r, "hard_rate": 0.10, "zipf": 0.0, "top_n": 0, "window": 0.0,
            "lm": False}
    case.update(more)
    return case


def listed():
    return [
        # one person dictating: half-second chunks, a partial transcript after each
        _stream("live_stream", 1, 25, 4, 32, 32, 0.01),
        # one short utterance on request (4 s of audio, small beam): latency of a single call
        _decode("single", 1, 200, 32, 8, 0.01),
        # a server's ordinary batch of characters, pruned and with every token kept
        _decode("batch64", 64, 500, 32, 32, 0.01),
        _decode("batch64_unpruned", 64, 500, 32, 32, 0.0),
        # a corpus batch with utterances of 5 to 30 s, noisier emissions and a wider beam
        _decode("varlen256", 256, 1500, 32, 100, 0.01, hard_rate=0.25, ragged=True),
        # sub-word vocabulary, pruned and with every token kept
        _decode("subword128", 128, 400, 1024, 64, 0.01, zipf=1.1),
        _decode("subword_unpruned", 128, 400, 1024, 64, 0.0, zipf=1.1),
        # a bigram table of characters (4 KB) and one of sub-words (4 MB)
        _decode("bigram128", 128, 500, 32, 64, 0.01, lm=True),
        _decode("subword_bigram128", 128, 400, 1024, 64, 0.01, zipf=1.1, lm=True),
        # offline transcription of an archive: as many utterances per call as the chip takes
        _decode("bulk4096", 4096, 500, 32, 32, 0.01),
        # the setting of a decoder tuned for accuracy: a beam of 1000, Top-4, score window 25
        _decode("beam1000", 64, 500, 32, 1000, 0.007, top_n=4, window=25.0),
        # rescoring: the whole final beam and its traces, of a ragged batch of an odd size
        _decode("nbest_ragged", 37, 613, 29, 200, 0.003, ragged=True, nbest=True, traces=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _seconds(c):
    """A generous estimate of a decode's time: its serial frames times a frame's cost."""
    kept = c["V"] if c["r"] == 0.0 else 2 + c["V"] * min(1.0, 0.03 * (0.01 / c["r"]) ** 0.5)
    if c["top_n"] > 0:
        kept = min(kept, c["top_n"])
    frame = 3e-6 + 1.6e-9 * c["beam"] * kept
    return c["T"] * frame * max(1.0, c["B"] / (256.0 if c["V"] > 64 or c["beam"] > 128 else 512.0))


def draw(rng):
    while True:
        V = rng.choice((29, 32, 32, 32, _log_int(rng, 24, 256), _log_int(rng, 256, 4096)))
        if rng.random() < 0.15:
            chunk = rng.choice((5, 10, 25, 40, 50, _log_int(rng, 5, 50)))
            c = _stream("", _log_int(rng, 1, 64), chunk, rng.randint(2, 8), V,
                        _log_int(rng, 4, 256), rng.choice((0.1, 0.01, 0.01, 0.003)))
        else:
            c = _decode("", _log_int(rng, 1, 4096), _log_int(rng, 20, 1500), V,
                        _log_int(rng, 4, 1000) if rng.random() < 0.4 else _log_int(rng, 8, 128),
                        rng.choice((0.1, 0.01, 0.01, 0.007, 0.001, 0.0)),
                        ragged=rng.random() < 0.5)
            c["nbest"] = c["B"] * c["beam"] * c["T"] <= 1 << 23 and rng.random() < 0.2
            c["traces"] = rng.random() < 0.2
        c["hard_rate"] = rng.choice((0.10, 0.10, 0.25))
        c["zipf"] = 1.1 if V > 256 else 0.0
        c["lm"] = V <= 1024 and rng.random() < 0.25
        c["top_n"] = rng.choice((4, 8, 16)) if rng.random() < 0.15 else 0
        c["window"] = rng.choice((10.0, 25.0)) if rng.random() < 0.2 else 0.0
        del c["name"]
        if c["beam"] > 512 and V > binding.MAX_VOCAB_WIDE_BEAM:
            continue
        if 4 * c["B"] * c["T"] * V > MOST_EMISSION_BYTES:
            continue
        if 16 * c["B"] * c["T"] * c["beam"] > MOST_TRIE_BYTES or _seconds(c) > MOST_SECONDS:
            continue
        return c


def _emissions(c, gen, dev):
    """fp32 [B, T, V] log-softmax rows of `synth.utterance_emissions`' recipe, on the GPU."""
    B, T, V = c["B"], c["T"], c["V"]
    uniform = lambda lo, hi: lo + (hi - lo) * torch.rand(  # noqa: E731
        (B, T), generator=gen, device=dev, dtype=torch.float64)
    transcript = torch.randint(1, V, (B, TRANSCRIPT_LEN), generator=gen, device=dev)
    x = torch.randn((B, T, V), generator=gen, device=dev, dtype=torch.float64)
    if c["zipf"] > 0.0:
        x[:, :, 1:] -= c["zipf"] * torch.log(
            torch.arange(1, V, device=dev, dtype=torch.float64))
    blank = uniform(0.0, 1.0) < 0.65
    read = ((~blank).cumsum(1) - 1).clamp_min(0) % TRANSCRIPT_LEN
    primary = torch.where(blank, torch.zeros_like(read), transcript.gather(1, read))
    boost = uniform(6.0, 12.0)
    x.scatter_add_(2, primary.unsqueeze(2), boost.unsqueeze(2))
    other = torch.randint(0, V - 1, (B, T), generator=gen, device=dev)
    other = other + (other >= primary)
    second = torch.where(uniform(0.0, 1.0) < c["hard_rate"], uniform(4.0, 8.0),
                         torch.zeros_like(boost))
    x.scatter_add_(2, other.unsqueeze(2), second.unsqueeze(2))
    return torch.log_softmax(x, dim=2).to(torch.float32).contiguous()


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    c = case
    lp = _emissions(c, gen, dev)
    lm = None
    if c["lm"]:
        lm = torch.from_numpy(synth.make_bigram_lm(c["V"], seed=synth.LM_SEED + int(seed))).to(dev)
    weights = {"lm_table": lm, "lm_weight": 0.5, "insertion_bonus": 1.0} if c["lm"] else {}
    options = {"top_n": c["top_n"], "beam_threshold": c["window"], **weights}
    if c["kind"] == "stream":
        live = binding.Stream(c["B"], c["T"], c["chunk"], c["V"], c["beam"], c["r"], dev, **options)
        full = torch.full((c["B"],), c["chunk"], dtype=torch.int32, device=dev)
        pieces = [lp[:, t:t + c["chunk"]].contiguous() for t in range(0, c["T"], c["chunk"])]
        return {"case": c, "live": live, "pieces": pieces, "full": full, "lm": lm}
    if c["ragged"]:
        lengths = torch.randint(max(1, c["T"] // 6), c["T"] + 1, (c["B"],), generator=gen,
                                device=dev).to(torch.int32)
    else:
        lengths = torch.full((c["B"],), c["T"], dtype=torch.int32, device=dev)
    workspace = binding.alloc_workspace(c["B"], c["T"], c["V"], c["beam"], dev)
    return {"case": c, "lp": lp, "lengths": lengths, "workspace": workspace, "options": options}


def run(state):
    c = state["case"]
    if c["kind"] == "stream":  # one session: every chunk as it comes in
        live = state["live"]
        live.begin()
        for piece in state["pieces"]:
            live.feed(piece, state["full"])
        return {"tokens": live.tokens, "lengths": live.lengths, "scores": live.scores}
    out = binding.decode(state["lp"], state["lengths"], c["beam"], c["r"],
                         workspace=state["workspace"], want_nbest=c["nbest"],
                         want_traces=c["traces"], **state["options"])
    del out["workspace"]  # the caller's own
    return out


def work(case):
    """Emissions (and table) read once, results written once; per frame a maximum and a threshold
    test of every token, and for every beam entry one merge (a log-sum-exp of two masses: 50
    operations).  Ragged batches are counted at their mean length."""
    c = case
    frames = c["B"] * c["T"]
    rows = c["B"] * (c["T"] + 2)  # tokens, lengths, scores
    if c.get("traces"):
        rows += 2 * frames
    if c.get("nbest"):
        rows += c["B"] * c["beam"] * (c["T"] + 5)
    if c.get("ragged"):
        frames *= 7.0 / 12.0
    table = 4 * c["V"] * c["V"] if c["lm"] else 0
    return {"bytes": 4.0 * c["V"] * frames + 4.0 * rows + table,
            "flops": frames * (2.0 * c["V"] + 50.0 * c["beam"])}


def tolerance(case):
    """Tokens, lengths and frames are whole numbers decided by fp64 scores: the same for every
    correct implementation.  Scores are fp64 sums, rounded once to fp32."""
    return {"rel": 1e-6, "max": 1e-6, "differ": 0.0}
