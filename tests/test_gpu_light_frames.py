"""Frames whose survivors fit their header, in the builds with 256 and 128 threads (one thread per
candidate, or a few candidates per thread): at the beams where the blocks of extensions change size
(powers of two and their neighbours), for every number of survivors with and without the blank, mixed
with longer frames and with runs of blank-only ones.  Against the oracle, statistics included."""
import numpy as np
import pytest
import torch

from paper_2510_09085_amd import binding, synth

pytestmark = pytest.mark.gpu


def frames(seed, B, T, V, step=0.0, blank_runs=True):
    """fp32 [B, T, V]: one to eight tokens per frame within 4 nats of each other, the others at -30."""
    rng = np.random.default_rng(seed)
    lp = np.full((B, T, V), -30.0, dtype=np.float64)
    for b in range(B):
        for t in range(T):
            if blank_runs and rng.random() < 0.4:
                lp[b, t, 0] = -0.1 * rng.random()
                continue
            K = min(V, int(rng.integers(1, 9)))
            # few tokens, so that entries repeat their last one and extend into one another
            pool = rng.permutation(min(V, 9))
            if rng.random() < 0.5:
                pool = np.concatenate(([0], pool[pool != 0]))
            lp[b, t, pool[:K]] = -4.0 * rng.random(min(K, len(pool)))
    if step:
        lp = np.round(lp / step) * step
    return lp.astype(np.float32)


def check(oracle_lib, lp, beam, label, r=0.01, window=0.0, **more):
    from test_gpu_ties import check_case
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B, T, _ = lp.shape
    ln = np.full(B, T, dtype=np.int32)
    ln[B // 2] = T - T // 3
    return check_case(torch.device("cuda:0"), oracle_lib, lp, ln, beam, r, 0, window, label, **more)


@pytest.mark.parametrize("options", ["plain", "window", "lm"])
@pytest.mark.parametrize("beam", [1, 2, 7, 16, 17, 32, 33, 63, 64, 65, 85, 86, 127, 128])
def test_every_block_size(oracle_lib, beam, options):
    lp = frames(beam, 4, 70, 33)
    lm = synth.make_bigram_lm(33, seed=beam) if options == "lm" else None
    check(oracle_lib, lp, beam, f"beam{beam} {options}", window=6.0 if options == "window" else 0.0,
          lm=lm, lm_weight=0.7, insertion_bonus=0.3)


@pytest.mark.parametrize("window", [0.0, 5.0])
@pytest.mark.parametrize("beam", [1, 15, 32, 33, 64])
def test_more_utterances_than_the_chip_holds(oracle_lib, beam, window):
    """The build with 128 threads: two wavefronts, up to three extensions per thread."""
    B = 2 * torch.cuda.get_device_properties(0).multi_processor_count + 6
    lp = np.tile(frames(100 + beam, 6, 40, 29), (B // 6 + 1, 1, 1))[:B]
    check(oracle_lib, np.ascontiguousarray(lp), beam, f"B{B} beam{beam}", window=window)


@pytest.mark.parametrize("B", [3, 520])
@pytest.mark.parametrize("beam", [8, 32, 64])
def test_equal_scores_are_ordered_by_hash(oracle_lib, beam, B):
    """Emissions in steps of 1/2: several candidates of one score at the cut, stays and extensions."""
    lp = np.tile(frames(200 + beam, 3, 40, 12, step=0.5), (B // 3 + 1, 1, 1))[:B]
    tied, _ = check(oracle_lib, np.ascontiguousarray(lp), beam, f"steps B{B} beam{beam}")
    assert tied > 0


@pytest.mark.parametrize("beam", [3, 20, 50])
def test_survivors_without_mass_and_far_apart(oracle_lib, beam):
    """R = 0 on a vocabulary of six: every token survives, also those of log-prob -inf, which are no
    candidates; some frames lie a million nats below the others, some tokens a thousand below the
    rest of their frame, so scores leave the bins on either side."""
    rng = np.random.default_rng(beam)
    lp = synth.random_emissions(beam, 3, 60, 6, flat=2.0)
    lp[rng.random(lp.shape) < 0.25] = -np.inf
    lp[:, :, 0] = np.where(np.isinf(lp).all(axis=2), -0.5, lp[:, :, 0])
    lp[rng.random(lp.shape) < 0.1] -= 1000.0
    lp[:, 20] -= 1e6
    check(oracle_lib, lp.astype(np.float32), beam, f"-inf beam{beam}", r=0.0)


@pytest.mark.parametrize("chunk", [1, 7, 32, 33])
def test_streams_leave_and_enter_light_frames_at_any_chunk(oracle_lib, chunk):
    """Parents' places and children lists are carried from call to call whichever kind of frame the
    call ended on."""
    dev = torch.device("cuda:0")
    B, T, V, beam = 3, 66, 29, 40
    lp = frames(300, B, T, V)
    want_tok, want_sc, _ = oracle_lib.decode(lp, np.full(B, T, dtype=np.int32), beam, 0.01, n_threads=4)
    live = binding.Stream(B, T, chunk, V, beam, 0.01, dev)
    live.begin()
    for t in range(0, T, chunk):
        n = min(chunk, T - t)
        piece = np.zeros((B, chunk, V), dtype=np.float32)
        piece[:, :n] = lp[:, t:t + n]
        live.feed(torch.from_numpy(piece).to(dev), torch.full((B,), n, dtype=torch.int32, device=dev))
    torch.cuda.synchronize()
    lens = live.lengths.cpu().numpy()
    toks = live.tokens.cpu().numpy()
    for b in range(B):
        assert toks[b, :lens[b]].tolist() == want_tok[b], (chunk, b)
    np.testing.assert_allclose(live.scores.cpu().numpy(), np.asarray(want_sc, dtype=np.float32), atol=1e-4)


@pytest.mark.parametrize("blank", [-1e30, -5e4])
def test_blank_only_frames_of_masked_rows(oracle_lib, blank):
    """Rows whose blank has a mask's value and the rest none: in fp32 their sum over a chunk of headers loses
    what the other frames add, which must not get into the bounds of the scores."""
    lp = frames(500, 4, 70, 29)
    for t in (3, 4, 21, 40, 41):
        lp[:, t] = -np.inf
        lp[:, t, 0] = blank
    check(oracle_lib, lp, 40, f"masked {blank}")


@pytest.mark.parametrize("mask", [-1e30, -3e38])
@pytest.mark.parametrize("beam", [40, 64])
def test_masked_tokens_that_stay_in_the_beam(oracle_lib, beam, mask):
    """R = 0 on five tokens, three of them masked in every frame: entries lie 1e30 to 1e40 nats below the
    best for hundreds of light frames, the cut in their last bin."""
    rng = np.random.default_rng(beam)
    lp = np.full((3, 90, 5), mask, dtype=np.float32)
    lp[:, :, 0] = -0.1 - rng.random((3, 90))
    lp[:, :, 1] = -0.5 - rng.random((3, 90))
    lp = np.tile(lp, (1, 3, 1))
    check(oracle_lib, np.ascontiguousarray(lp), beam, f"kept {mask} beam{beam}", r=0.0)


@pytest.mark.parametrize("mask", [-1e4, -1e30, -1e36])
def test_a_table_with_masked_pairs(oracle_lib, mask):
    """Most pairs of the table masked: prefixes that hold one stay in the beam for want of better ones, in
    light frames and in longer ones."""
    lp = frames(600, 3, 90, 12)
    lm = synth.make_bigram_lm(12, seed=6)
    lm[np.random.default_rng(7).random(lm.shape) < 0.7] = mask
    check(oracle_lib, lp, 64, f"table {mask}", lm=lm, lm_weight=0.5, insertion_bonus=1.0)


@pytest.mark.parametrize("B", [3, 520])
@pytest.mark.parametrize("beam, tokens", [(8, 6), (16, 3), (32, 5), (64, 6), (64, 4), (100, 3), (128, 3)])
def test_equal_scores_at_the_cut_few_and_many(beam, tokens, B):
    """Every token of a frame has the same log-prob, so whole generations of candidates tie at the cut, up to 64
    of them (which are listed) and more.  The last bit of a log-sum-exp decides there, so it is compared, bit
    for bit, with a build that has no light frames of either kind (which a vocabulary above 2048 tokens takes: the
    same emissions with tokens that never survive)."""
    dev = torch.device("cuda:0")
    lp = np.full((3, 150, 12), -30.0, dtype=np.float32)
    lp[:, :, :tokens] = -1.5
    lp[:, 60:100] = frames(beam, 3, 40, 12)
    lp[1, 20:] = frames(beam + 1, 1, 130, 12)[0]

    def decoded(x, **more):
        ln = torch.full((len(x),), 150, dtype=torch.int32, device=dev)
        ln[1] = 140
        return binding.decode(torch.from_numpy(np.ascontiguousarray(x)).to(dev), ln, beam, 0.01, **more)

    want = decoded(np.pad(lp, ((0, 0), (0, 0), (0, 2040)), constant_values=-60.0), want_nbest=True)
    got = decoded(np.tile(lp, (B // 3 + 1, 1, 1))[:B], want_nbest=B == 3)
    for b in range(3):
        if b == 1 and B > 3:
            continue  # (only the first one of its kind is shorter)
        for key in ("tokens", "lengths", "scores") + (("nbest_count", "nbest_tokens", "nbest_pb", "nbest_pnb")
                                                      if B == 3 else ()):
            assert torch.equal(got[key][b], want[key][b]), (key, b)
    assert torch.equal(got["tokens"][3:B:3], got["tokens"][0].expand_as(got["tokens"][3:B:3]))


def fastest_ms(lp, beam, r, **more):
    """of six decodes of host emissions, the workspace kept"""
    dev = torch.device("cuda:0")
    B, T, V = lp.shape
    x, took = torch.from_numpy(lp).to(dev), []
    ln = torch.full((B,), T, dtype=torch.int32, device=dev)
    workspace = binding.alloc_workspace(B, T, V, beam, dev)
    for _ in range(6):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        binding.decode(x, ln, beam, r, workspace=workspace, **more)
        end.record()
        end.synchronize()
        took.append(start.elapsed_time(end))
    return min(took)


def test_equal_scores_take_a_bounded_time():
    """Six equal tokens, beam 64, a cut among hundreds of equal scores: ranked one by one among all candidates
    that took 25 times as long as frames whose scores differ (12.3 ms for 64 x 200 frames)."""
    equal = np.full((64, 200, 12), -30.0, dtype=np.float32)
    equal[:, :, :6] = -1.5
    apart = equal.copy()
    apart[:, :, :6] -= np.random.default_rng(0).random((64, 200, 6)).astype(np.float32)
    took = [fastest_ms(lp, 64, 0.01) for lp in (equal, apart)]
    assert took[0] < 12.0 * took[1], took  # (measured: 5)


def test_six_utterances_with_a_table_fit_a_compute_unit():
    """V = 32 and its table in LDS, beam 64: six workgroups per CU, as many as registers allow, so six
    utterances per CU take little longer than five.  (With five resident they took 1.5 times as long.)"""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    lp = np.tile(synth.random_emissions(3, 8, 60, 32, flat=3.0), (6 * n_cu // 8 + 1, 1, 1)).astype(np.float32)
    table = {"lm_table": torch.from_numpy(synth.make_bigram_lm(32)).to("cuda:0"), "lm_weight": 0.5}
    took = [fastest_ms(np.ascontiguousarray(lp[:per_cu * n_cu]), 64, 0.001, **table) for per_cu in (6, 5)]
    assert took[0] < 1.25 * took[1], took  # (measured: 1.03)
