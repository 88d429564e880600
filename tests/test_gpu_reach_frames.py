"""Frames that go through the tokens that can reach the beam only: small vocabularies whose frames keep more than
the six survivors of a header (256 threads where R > 0, 512 where every token is kept), and vocabularies above 64 tokens
(512).  Against the oracle, statistics included: at the beams where the blocks of extensions change size, with lists of one
token, of more than one round and of more than are taken, with frames that no token changes, crowds at the cut, masked
rows and tokens, tables with and without gaps, windows, streams cut anywhere, and records that did not fit."""
import numpy as np
import pytest
import torch

from paper_2510_09085_amd import binding, synth

pytestmark = pytest.mark.gpu


def frames(seed, B, T, V, zipf=0.0):
    """fp32 [B, T, V] of the workloads' kind, whose competitors come close in every third frame or so."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((B, T, V))
    if zipf:
        x[:, :, 1:] -= zipf * np.log(np.arange(1, V))
    for b in range(B):
        for t in range(T):
            top = 0 if rng.random() < 0.6 else int(rng.integers(1, min(V, 12)))
            x[b, t, top] += rng.choice((2.0, 7.0, 11.0))
            if rng.random() < 0.3:  # a burst of tokens that compete
                n = int(rng.integers(1, min(V, 30)))
                x[b, t, rng.permutation(V)[:n]] += rng.uniform(2.0, 8.0)
    m = x.max(axis=2, keepdims=True)
    return (x - m - np.log(np.exp(x - m).sum(axis=2, keepdims=True))).astype(np.float32)


def check(oracle_lib, lp, beam, label, r, window=0.0, top_n=0, **more):
    from test_gpu_ties import check_case
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B, T, _ = lp.shape
    ln = np.full(B, T, dtype=np.int32)
    ln[B // 2] = T - T // 3
    return check_case(torch.device("cuda:0"), oracle_lib, lp, ln, beam, r, top_n, window, label, **more)


@pytest.mark.parametrize("options", ["plain", "window", "lm"])
@pytest.mark.parametrize("beam", [1, 2, 15, 16, 17, 32, 33, 64, 65, 100, 128])
def test_small_vocabularies_that_keep_every_token(oracle_lib, beam, options):
    """(With a table, and at beams above 64, other builds: those without these frames.)"""
    lp = frames(beam, 3, 75, 29)
    lm = synth.make_bigram_lm(29, seed=beam) if options == "lm" else None
    check(oracle_lib, lp, beam, f"beam{beam} {options}", 0.0, window=5.0 if options == "window" else 0.0,
          lm=lm, lm_weight=0.7, insertion_bonus=0.3)


@pytest.mark.parametrize("window", [0.0, 5.0])
@pytest.mark.parametrize("beam", [1, 2, 16, 17, 33, 64, 65, 86, 100, 127, 128])
def test_small_vocabularies_at_small_thresholds(oracle_lib, beam, window):
    """256 threads, above beam 64 two wavefronts with the stays and one block of extensions."""
    check(oracle_lib, frames(50 + beam, 3, 75, 29), beam, f"beam{beam} window{window}", 0.0005, window=window)


@pytest.mark.parametrize("beam, V", [(16, 32), (24, 29), (64, 12), (64, 32), (40, 64)])
def test_more_utterances_than_compute_units_that_keep_every_token(oracle_lib, beam, V):
    """Two workgroups of 256 threads per CU for few candidates a frame, 512 threads from 2048 on at beams above 32."""
    B = torch.cuda.get_device_properties(0).multi_processor_count + 5
    lp = np.tile(frames(60 + beam, 5, 40, V), (B // 5 + 1, 1, 1))[:B]
    check(oracle_lib, np.ascontiguousarray(lp), beam, f"B{B} beam{beam} V{V}", 0.0)


@pytest.mark.parametrize("r, top_n", [(0.01, 0), (0.0005, 0), (0.0, 20), (0.0, 64)])
@pytest.mark.parametrize("V, beam", [(65, 1), (65, 64), (100, 65), (257, 31), (1024, 64), (1024, 128), (2048, 64),
                                     (2048, 128)])
def test_large_vocabularies(oracle_lib, V, beam, r, top_n):
    check(oracle_lib, frames(V + beam, 3, 40, V, zipf=1.1), beam, f"V{V} beam{beam} r{r} N{top_n}", r, top_n=top_n)


@pytest.mark.parametrize("window, table", [(4.0, False), (0.0, True), (4.0, True)])
@pytest.mark.parametrize("V, beam, r", [(65, 30, 0.01), (128, 128, 0.003), (200, 64, 0.01), (1024, 32, 0.01),
                                        (1024, 64, 0.01)])
def test_large_vocabularies_with_tables_and_windows(oracle_lib, V, beam, r, window, table):
    """A table without gaps: tokens are left out, with the statistics asked for."""
    lm = synth.make_bigram_lm(V, seed=beam) if table else None
    check(oracle_lib, frames(V + beam + 1, 3, 40, V, zipf=1.1), beam, f"V{V} beam{beam} window{window} table{table}", r,
          window=window, lm=lm, lm_weight=0.7, insertion_bonus=0.3)


@pytest.mark.parametrize("V, r", [(29, 0.0), (70, 0.003)])
def test_masked_tokens_and_gaps_in_the_table(oracle_lib, V, r):
    """Tokens and pairs without mass: never listed, and not counted by the statistics."""
    lp = frames(7, 4, 60, V)
    lp[:, ::3, 3::4] = -np.inf
    lm = synth.make_bigram_lm(V, seed=3)
    lm[2::5, 1::3] = -np.inf
    for table in (None, lm):
        check(oracle_lib, lp, 40, f"V{V} table{table is not None}", r, lm=table, lm_weight=0.7, insertion_bonus=0.3)


def check_beams(oracle_lib, lp, beam, r, top_n=0, **more):
    """Transcripts, and the whole final beam, of every utterance."""
    dev = torch.device("cuda:0")
    B, T, _ = lp.shape
    ln = np.full(B, T, dtype=np.int32)
    out = binding.decode(torch.from_numpy(lp).to(dev), torch.from_numpy(ln).to(dev), beam, r, top_n=top_n,
                         want_nbest=True, **more)
    got = {k: out[k].cpu().numpy() for k in ("tokens", "lengths", "nbest_count", "nbest_tokens", "nbest_lengths")}
    want, _, _ = oracle_lib.decode(lp, ln, beam, r, n_threads=8, top_n=top_n)
    for b in range(B):
        assert got["tokens"][b, :got["lengths"][b]].tolist() == want[b], b
        final = oracle_lib.decode_beam(lp[b], beam, r, max_entries=beam, top_n=top_n)
        mine = [tuple(got["nbest_tokens"][b, i, :got["nbest_lengths"][b, i]]) for i in range(got["nbest_count"][b])]
        assert sorted(mine) == sorted(tuple(e[0]) for e in final), b


@pytest.mark.parametrize("row", [-1e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("V, beam, r, top_n", [(16, 8, 0.0, 0), (16, 16, 0.0, 0), (20, 40, 0.0, 0), (100, 8, 0.0, 20),
                                               (100, 70, 0.0, 20)])
def test_nothing_is_left_out_behind_a_row_of_masked_tokens(oracle_lib, V, beam, r, top_n, row):
    """All tokens of a frame masked: from there on the scores are so large that what a frame adds is lost, every
    candidate scores the same and the hashes decide.  The frame itself is one of a run, not its end."""
    lp = frames(21, 40, 24, V)
    lp[:, 9] = row
    check_beams(oracle_lib, lp, beam, r, top_n=top_n)


@pytest.mark.parametrize("V, beam, r, top_n", [(24, 10, 0.0, 0), (24, 40, 0.0, 0), (31, 16, 0.0, 0), (300, 10, 0.0, 60),
                                               (300, 40, 0.0, 60)])
def test_entries_farther_below_than_the_bins_are_wide(oracle_lib, V, beam, r, top_n):
    """Every token but the blank masked, by sizes from 1e31 to the lowest fp32: a full beam whose worst entry lies
    farther below the best than any spread that bins are made for, and extensions that come in between."""
    rng = np.random.default_rng(beam)
    lp = -10.0 ** rng.uniform(31.0, 38.5, (30, 40, V))
    lp[:, ::3, 1:] = -10.0 ** rng.uniform(37.5, 38.5, lp[:, ::3, 1:].shape)
    lp[:, :, 0] = -0.1 - rng.random((30, 40))
    check_beams(oracle_lib, lp.astype(np.float32), beam, r, top_n=top_n)


@pytest.mark.parametrize("V, r", [(32, 0.0), (90, 0.002)])
@pytest.mark.parametrize("cut", [1, 3, 7, 32, 50])
def test_streams_give_what_the_whole_utterance_gives(V, r, cut):
    dev = torch.device("cuda:0")
    lp = torch.from_numpy(frames(11, 3, 100, V)).to(dev)
    want = binding.decode(lp, torch.full((3,), 100, dtype=torch.int32, device=dev), 24, r)
    live = binding.Stream(3, 100, cut, V, 24, r, dev)
    for t in range(0, 100, cut):
        n = min(cut, 100 - t)
        live.feed(lp[:, t:t + n].contiguous(), torch.full((3,), n, dtype=torch.int32, device=dev))
    assert torch.equal(live.lengths, want["lengths"]) and torch.equal(live.scores, want["scores"])
    for b in range(3):
        n = int(want["lengths"][b])
        assert torch.equal(live.tokens[b, :n], want["tokens"][b, :n])


@pytest.mark.parametrize("V, r", [(32, 0.0), (29, 0.0005), (90, 0.002)])
def test_streams_whose_calls_take_different_builds(V, r):
    """Calls of one or two frames take builds without these frames, the others theirs: what is carried between them
    holds whichever wrote it."""
    dev, sizes = torch.device("cuda:0"), [1, 30, 2, 2, 17, 1, 33, 2, 12]
    T = sum(sizes)
    lp = torch.from_numpy(frames(13, 3, T, V)).to(dev)
    want = binding.decode(lp, torch.full((3,), T, dtype=torch.int32, device=dev), 24, r)
    live, t = binding.Stream(3, T, max(sizes), V, 24, r, dev), 0
    for n in sizes:
        live.feed(lp[:, t:t + n].contiguous(), torch.full((3,), n, dtype=torch.int32, device=dev))
        t += n
    assert torch.equal(live.lengths, want["lengths"]) and torch.equal(live.scores, want["scores"])
    for b in range(3):
        n = int(want["lengths"][b])
        assert torch.equal(live.tokens[b, :n], want["tokens"][b, :n])


def test_records_that_did_not_fit_are_not_asked_for():
    """Survivors of the next full frame are read ahead of its turn: not those of a frame without records."""
    dev = torch.device("cuda:0")
    B, T, V, beam = 6, 80, 32, 16
    lp = torch.from_numpy(frames(5, B, T, V)).to(dev)
    ln = torch.full((B,), T, dtype=torch.int32, device=dev)
    small = binding.alloc_workspace(B, T, V, beam, dev, max_records=0)
    assert int(binding.decode(lp, ln, beam, 0.0005, workspace=small)["lengths"].min()) == -1


def flat(seed, B, T, V, spread):
    """fp32 [B, T, V] rows without a peak: every token competes in every frame."""
    x = spread * np.random.default_rng(seed).standard_normal((B, T, V))
    return (x - np.log(np.exp(x).sum(axis=2, keepdims=True))).astype(np.float32)


@pytest.mark.parametrize("V, beam, r", [(16, 64, 0.0), (24, 16, 0.0), (29, 64, 0.001)])
def test_crowds_at_the_cut_take_a_bounded_time(V, beam, r):
    """All tokens equal in every frame: hundreds of candidates of one score at the cut.  (Ranked one by one they took 24
    times as long as candidates whose scores differ; handed to the general path 1.1 to 3 times.)"""
    from test_gpu_light_frames import fastest_ms
    equal, apart = (fastest_ms(flat(1, 64, 100, V, spread), beam, r) for spread in (0.0, 0.3))
    assert equal < 6.0 * apart, (equal, apart)


@pytest.mark.parametrize("r, beam", [(0.0, 8), (0.0, 24), (0.0, 64), (0.001, 40), (0.001, 128)])
@pytest.mark.parametrize("step", [0.0, 0.5])
def test_crowds_at_the_cut_are_ordered_as_the_general_path_does(r, beam, step):
    """Tokens that are all equal, or in steps: whole generations of candidates tie at the cut, more and fewer than are ranked
    one by one.  Bit for bit with a build that has no such frames (which a vocabulary above 2048 tokens takes: the same
    emissions with tokens that have no mass)."""
    dev = torch.device("cuda:0")
    lp = flat(beam, 4, 120, 29, 1.0 if step else 0.0)
    if step:
        lp = (np.round(lp / step) * step).astype(np.float32)
    lp[:, 40:70] = frames(beam, 4, 30, 29)
    ln = torch.full((4,), 120, dtype=torch.int32, device=dev)
    got, want = (binding.decode(torch.from_numpy(np.ascontiguousarray(x)).to(dev), ln, beam, r, want_nbest=True)
                 for x in (lp, np.pad(lp, ((0, 0), (0, 0), (0, 2040)), constant_values=-np.inf)))
    for key in ("tokens", "lengths", "scores", "nbest_count", "nbest_tokens", "nbest_pb", "nbest_pnb"):
        assert torch.equal(got[key], want[key]), key


def extremes(g, lp):
    """Some tokens masked by a finite value, whole rows of one, rows far below the others, tokens without mass."""
    if g.random() < 0.3:
        lp[g.random(lp.shape) < 0.3] = g.choice([-1e4, -1e9, -1e30, -3e38])
        lp[:, :, 0] = np.maximum(lp[:, :, 0], -8.0)
    if g.random() < 0.3:
        lp[:, g.integers(0, lp.shape[1], 2)] = g.choice([-1e4, -2e4, -1e12, -1e30, -3e38])
    if g.random() < 0.2:
        lp[:, int(g.integers(0, lp.shape[1]))] -= g.choice([1e4, 1e6, 1e8])
    if g.random() < 0.2:
        lp[g.random(lp.shape) < 0.2] = -np.inf
    return lp


@pytest.mark.parametrize("group", range(12))
def test_random_calls_as_the_general_path_decodes_them(group):
    """25 calls each, bit for bit with a build that has no such frames (a vocabulary above 2048 tokens: the same
    emissions and table with tokens that have no mass), final beams included.  (Of 4600 such calls 130 differed while
    bounds were asked once a run.)"""
    dev, wide = torch.device("cuda:0"), 2060
    for seed in range(1000 + 25 * group, 1025 + 25 * group):
        g = np.random.default_rng(seed)
        V = int(g.choice([6, 9, 16, 24, 29, 32, 64, 65, 90, 128, 300]))
        B, T = int(g.choice([1, 3, 5])), int(g.integers(5, 120))
        beam = int(g.choice([1, 2, 5, 8, 16, 17, 32, 33, 57, 64, 65, 80, 100, 128]))
        r = float(g.choice([0.0, 0.0, 0.0005, 0.001, 0.003] if V <= 64 else [0.001, 0.003, 0.01, 0.1]))
        more = {"top_n": int(g.choice([0, 0, 8, 20])) if V > 22 else 0, "beam_threshold": float(g.choice([0.0, 0.0, 5.0]))}
        lp = frames(seed, B, T, V) if g.random() < 0.6 else flat(seed, B, T, V, float(g.choice([0.0, 0.3, 2.0])))
        if g.random() < 0.2:
            lp = np.round(lp * 2) / 2
        lp = extremes(g, lp).astype(np.float32)
        tables = [{}, {}]
        if g.random() < 0.3:
            lm = synth.make_bigram_lm(V, seed=seed)
            if g.random() < 0.4:
                lm[g.random(lm.shape) < 0.3] = g.choice([-np.inf, -1e4, -1e30])
            padded = np.pad(lm, (0, wide - V), constant_values=-5.0)
            tables = [{"lm_table": torch.from_numpy(x).to(dev), "lm_weight": 0.5, "insertion_bonus": 1.0}
                      for x in (lm, padded)]
        ln = torch.from_numpy(g.integers(max(1, T // 2), T + 1, B).astype(np.int32)).to(dev)
        emissions = (lp, np.pad(lp, ((0, 0), (0, 0), (0, wide - V)), constant_values=-np.inf))
        got, want = (binding.decode(torch.from_numpy(np.ascontiguousarray(x)).to(dev), ln, beam, r, want_nbest=True,
                                    **more, **table) for x, table in zip(emissions, tables))
        for key in ("tokens", "lengths", "scores", "nbest_count", "nbest_tokens", "nbest_pb", "nbest_pnb"):
            same = torch.equal(got[key].nan_to_num(7.0), want[key].nan_to_num(7.0))
            assert same, f"seed {seed}: V{V} B{B} T{T} beam{beam} r{r} {more} table{bool(tables[0])}: {key}"


def test_frames_whose_tokens_all_compete_take_little_longer():
    """R = 0, no frame of which few tokens can change: about as fast as in the build that does not ask (which calls
    with a table have; here one of zeros, of weight zero)."""
    from test_gpu_light_frames import fastest_ms
    zeros = torch.zeros((64, 64), dtype=torch.float32, device="cuda:0")
    lp = flat(2, 64, 100, 64, 0.3)
    asks, does_not = fastest_ms(lp, 64, 0.0), fastest_ms(lp, 64, 0.0, lm_table=zeros)
    assert asks < 1.6 * does_not, (asks, does_not)  # (measured: 1.1; with 256 threads and every frame tried 2.2)


@pytest.mark.parametrize("chunk", [1, 2, 3])
def test_streams_of_short_chunks_take_little_longer(chunk):
    """The same of streams that keep every token, whose calls have few frames to make up for what the first costs."""
    dev, zeros = torch.device("cuda:0"), torch.zeros((64, 64), dtype=torch.float32, device="cuda:0")
    n, B, V = 6 * chunk, 64, 64
    lp = torch.from_numpy(frames(3, B, n, V)).to(dev)
    pieces = [lp[:, t:t + chunk].contiguous() for t in range(0, n, chunk)]
    full = torch.full((B,), chunk, dtype=torch.int32, device=dev)
    took = []
    for more in ({}, {"lm_table": zeros}):
        live, times = binding.Stream(B, n, chunk, V, 64, 0.0, dev, **more), []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            live.begin()
            for piece in pieces:
                live.feed(piece, full)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        took.append(min(times))
    assert took[0] < 1.6 * took[1], took  # (measured: 1.0 to 1.1; 2.1 to 3.9 before)
