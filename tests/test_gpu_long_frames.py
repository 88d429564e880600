"""Frames with many candidates per thread (long survivor lists), at the sizes where the search
changes its way of going through them: the number of candidates per thread from which a frame
gets a score floor, batches of four with a remainder, more than 64 and more than 128 numbers per
thread, and each beam capacity.  Against the oracle, statistics included."""
import pytest
import torch

from paper_2510_09085_amd import synth

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
