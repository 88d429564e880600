"""Frames with many candidates per thread (long survivor lists), at the sizes where the search
changes its way of going through them: the number of candidates per thread from which a frame
gets a score floor, batches of four with a remainder, more than 64 and more than 128 numbers per
thread, and each beam capacity.  Against the oracle, statistics included."""
import numpy as np
import pytest
import torch

from paper_2510_09085_amd import binding, synth

pytestmark = pytest.mark.gpu

# 512 threads: beam 32 -> 16 threads per entry, so V - 1 = 48 / 49 / 64 / 65 / 1024 / 1025 / 2049
# non-blank tokens are 3 / 4 / 4 / 5 / 64 / 65 / 129 candidates per thread
SIZES = [(49, 32, 24), (50, 32, 24), (65, 32, 24), (66, 32, 24), (1025, 32, 8), (1026, 32, 8),
         (2050, 32, 6), (97, 64, 20), (1024, 128, 5), (40, 129, 24), (37, 300, 20),
         (33, 600, 20), (300, 1000, 4)]


@pytest.mark.parametrize("options", ["plain", "window", "lm", "top_n"])
@pytest.mark.parametrize("V,beam,T", SIZES)
def test_long_survivor_lists(oracle_lib, V, beam, T, options):
    from test_gpu_ties import check_case
    assert torch.cuda.is_available(), "these tests need the MI355X"
    w = synth.Workload("long", B=2, T=T, V=V, beam=beam, rel_thresholds=(0.0,), seed=V + beam,
                       hard_rate=0.25)
    lp, ln = synth.make_emissions(w)
    lm = synth.make_bigram_lm(V, seed=beam) if options == "lm" else None
    check_case(torch.device("cuda:0"), oracle_lib, lp, ln, beam, 0.0,
               V - 3 if options == "top_n" else 0, 12.0 if options == "window" else 0.0,
               f"V{V} beam{beam} {options}", lm=lm, lm_weight=0.7, insertion_bonus=0.3)


def _decode_and_compare(oracle_lib, lp, beam, label, **more):
    from test_gpu_ties import check_case
    ln = np.full(lp.shape[0], lp.shape[1], dtype=np.int32)
    return check_case(torch.device("cuda:0"), oracle_lib, lp, ln, beam, 0.0, 0, 0.0, label, **more)


@pytest.mark.parametrize("with_lm", [False, True])
@pytest.mark.parametrize("V,beam", [(100, 32), (1030, 32), (40, 300), (300, 600)])
def test_tokens_without_mass_in_a_long_list(oracle_lib, V, beam, with_lm):
    """R = 0 keeps tokens of log-prob -inf too; they are no candidates and are not counted.  A
    third of all tokens, a frame's top token included where it is the blank, and whole columns;
    the table has pairs of log-prob -inf as well."""
    rng = np.random.default_rng(V + beam)
    B, T = 2, 14
    lp = synth.random_emissions(V, B, T, V, flat=1.0)
    lp[rng.random(lp.shape) < 0.33] = -np.inf
    lp[:, 5, 1:] = -np.inf          # only the blank has mass
    lp[:, 9, 0] = -np.inf           # the blank has none
    lp[:, :, 3] = -np.inf
    lp[:, 5, 0] = -0.25
    more = {}
    if with_lm:
        lm = synth.make_bigram_lm(V, seed=beam)
        lm[rng.random(lm.shape) < 0.2] = -np.inf
        more = dict(lm=lm, lm_weight=0.7, insertion_bonus=0.3)
    _decode_and_compare(oracle_lib, lp, beam, f"V{V} beam{beam} -inf", **more)


@pytest.mark.parametrize("V,beam,T,with_lm", [(1026, 32, 4, False), (64, 128, 6, True),
                                              (64, 128, 6, False), (300, 64, 4, True)])
def test_more_utterances_than_compute_units(oracle_lib, V, beam, T, with_lm):
    """One to two utterances per compute unit: a build whose distance cache has a single row, so
    nearly every candidate is evaluated again by the later passes (table in LDS and in memory)."""
    B = torch.cuda.get_device_properties(0).multi_processor_count + 8
    lp = synth.random_emissions(V, B, T, V, flat=1.5)
    lm = synth.make_bigram_lm(V, seed=beam) if with_lm else None
    _decode_and_compare(oracle_lib, lp, beam, f"V{V} beam{beam} B{B}", lm=lm, lm_weight=0.7,
                        insertion_bonus=0.3)


@pytest.mark.parametrize("B", [2, 264])
def test_ties_beyond_64_candidates_per_thread(oracle_lib, B):
    """Emissions in steps of 1/2: many candidates of one score at the cut, so the selection goes
    on by hash, with candidate numbers taken in groups of two."""
    T = 4 if B == 2 else 3
    lp = (np.round(synth.random_emissions(7, B, T, 1030, flat=1.0) * 2) / 2).astype(np.float32)
    tied, _ = _decode_and_compare(oracle_lib, lp, 32, f"quantised B{B}")
    assert tied > 0


# (V, beam, top_n, the threshold at which the launcher goes over to another build): 512 threads with
# 128 entries, with 512 entries, 1024 threads, and from lists of a static top-N to short ones
SWITCHES = [(1024, 32, 0, 0.01829), (32, 200, 0, 0.00605), (40, 600, 0, 0.01259),
            (1024, 64, 16, 0.07676)]


@pytest.mark.parametrize("with_lm", [False, True])
@pytest.mark.parametrize("side", [0.99, 1.01])
@pytest.mark.parametrize("V,beam,top_n,r", SWITCHES)
def test_thresholds_at_which_the_build_changes(oracle_lib, V, beam, top_n, r, side, with_lm):
    """Frames of every length meet either build: some led by one token, some with many alike."""
    from test_gpu_ties import check_case
    rng = np.random.default_rng(V + beam)
    B, T = 3, 24
    x = rng.standard_normal((B, T, V)) * rng.choice([0.5, 2.0], size=(B, T, 1))
    lead = rng.random((B, T)) < 0.4
    x[..., 0][lead] += 9.0
    lp = synth._log_softmax64(x).astype(np.float32)
    ln = np.array([T, T - 5, T], dtype=np.int32)
    lm = synth.make_bigram_lm(V, seed=beam) if with_lm else None
    check_case(torch.device("cuda:0"), oracle_lib, lp, ln, beam, float(np.float32(r * side)), top_n,
               0.0, f"V{V} beam{beam} r{r * side:.5f}", lm=lm, lm_weight=0.6, insertion_bonus=0.2)


@pytest.mark.parametrize("options", ["plain", "lm", "lm with gaps", "window"])
@pytest.mark.parametrize("beam", [20, 128, 200, 600])
@pytest.mark.parametrize("near", [1, 300, 511, 512, 513, 1023])
def test_tokens_that_can_reach_the_floor(oracle_lib, near, beam, options):
    """`near` tokens lie within a nat of a frame's best, the others 40 nats below: the tokens that can
    reach the floor are listed up to 512 of them, beyond that the whole list is gone through, and also
    where the statistics are asked for and pairs of the table have no mass.  The blank is among either,
    and a column has no mass."""
    rng = np.random.default_rng(near + beam)
    B, T, V = 2, 5, 1026
    lp = -40.0 - rng.random((B, T, V))
    for b in range(B):
        for t in range(T):
            lp[b, t, rng.permutation(V)[:near]] = -rng.random(near)
    lp[:, :, 7] = -np.inf
    more = {}
    if options.startswith("lm"):
        lm = synth.make_bigram_lm(V, seed=beam)
        if options == "lm with gaps":
            lm[rng.random(lm.shape) < 0.1] = -np.inf
        more = dict(lm=lm, lm_weight=0.7, insertion_bonus=0.3)
    from test_gpu_ties import check_case
    check_case(torch.device("cuda:0"), oracle_lib, lp.astype(np.float32), np.full(B, T, dtype=np.int32),
               beam, 0.0, 0, 9.0 if options == "window" else 0.0, f"near{near} beam{beam} {options}", **more)
    if options == "lm with gaps":  # the same without statistics, which lists tokens here too
        x, ln = torch.from_numpy(lp.astype(np.float32)).to("cuda:0"), torch.full((B,), T, dtype=torch.int32).to("cuda:0")
        kw = dict(lm_table=torch.from_numpy(lm).to("cuda:0"), lm_weight=0.7, insertion_bonus=0.3, want_nbest=True)
        with_stats, without = (binding.decode(x, ln, beam, 0.0, want_stats=asked, **kw) for asked in (True, False))
        for key in ("tokens", "lengths", "scores", "nbest_count", "nbest_tokens", "nbest_pb", "nbest_pnb"):
            assert torch.equal(with_stats[key], without[key]), key


def test_statistics_cost_little_with_a_table(oracle_lib):
    """Tokens that cannot reach the floor are counted, not scored, for the statistics as well: scored for them,
    pair by pair, an unpruned search with a table took up to twice as long."""
    from test_gpu_light_frames import fastest_ms
    lp = np.tile(synth.random_emissions(5, 4, 30, 1024, flat=3.0), (16, 1, 1)).astype(np.float32)
    lp[:, :, 1:4] += 4.0
    table = {"lm_table": torch.from_numpy(synth.make_bigram_lm(1024)).to("cuda:0"), "lm_weight": 0.5}
    took = [fastest_ms(lp, 64, 0.0, want_stats=asked, **table) for asked in (True, False)]
    assert took[0] < 1.15 * took[1], took  # (measured: 1.01; scored pair by pair 1.32)
