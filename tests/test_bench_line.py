"""The line bench.py prints: the fields its readers need, and short enough to be found whole at the
end of the output (a reader that keeps the last 8 KB lost the 20 KB line)."""
import json

import bench


def a_record():
    cfg = {"workload": "cfg4_subword1024", "B": 128, "T": 400, "V": 1024, "beam": 64,
           "rel_threshold": 0.001, "lm": False, "frames": 51200, "steps": 20,
           "ms_per_step": 11.2234, "frames_per_s": 4561904.6, "notes": "x" * 900,
           "cpu_oracle": {"all_cores": {"frames_per_s": 600.25}, "one_thread": {"frames_per_s": 50.1}}}
    rec = {"metric": "decoded frames/sec (1 GPU)", "value": 103367954.3, "unit": "frames/s",
           "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 2.1228, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
           "config": {"workload": "cfg3_varlen256"}, "roofline": {"kernel": "y" * 600},
           "roofline_emission_read": {"kernel": "y" * 500}, "cpu_baseline": {"sample": "z" * 400},
           "per_config": [dict(cfg) for _ in range(11)]}
    rec.update({k: ["w" * 7000] for k in bench.RECORD_ONLY})
    return rec


def test_printed_line_is_short_and_complete():
    rec = a_record()
    line = json.dumps(bench.headline(rec))
    assert len(line) < 6000 and "\n" not in line
    got = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
                "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config", "roofline",
                "cpu_baseline"):
        assert got[key] == rec[key]
    assert [c["ms_per_step"] for c in got["per_config"]] == [11.2234] * 11
    assert got["per_config"][0]["oracle_k_frames_per_s"] == 0.6
    assert "notes" in rec["per_config"][0], "the record itself is left alone"


def test_printed_line_without_the_optional_parts():
    rec = {k: v for k, v in a_record().items() if k != "per_config" and k not in bench.RECORD_ONLY}
    assert bench.headline(rec) == rec
