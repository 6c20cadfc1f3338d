"""The benchmark's printed line: one line of JSON that whoever keeps the end of
the output gets whole, with the headline fields and the roofline unchanged."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

HEAD = {"metric": bench.METRIC, "value": 51399.3214, "unit": "sources/s", "n_gpus": 1, "steps": 10, "warmup": 2,
        "ms_per_step": 19.4555, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
        "data": "synthetic", "config": {"workload": "1000 sources", "n_vis": 9266880, "precision": "fp64"},
        "stage_ms": {"model_vis": 3.9537, "extract": 8.7404, "fit": 6.7226},
        "roofline": {"kernel": "k_extract", "bound": "alu", "frac": 0.7075, "basis": "b" * 200, "slots_per_unit": {"x": 1}}}


def _result(rows):
    detail = {"kernel": "k" * 80, "basis": "b" * 160, "frac": 0.123456789, "loss_per_epoch": [-5.0] * 96}
    return dict(HEAD, kernel_rooflines={k: detail for k in ("extract", "fit", "model")},
                batched_and_surrogate={"training": [detail] * 4, "surrogate": [{"fit_ms": 1.0 / 3.0}] * rows},
                facet_size_scan={"rows": [{"K": 20, "m1": -0.1, "m1_err": 0.01}] * rows})


def test_line_has_the_headline_whole_and_is_short():
    line = bench.printed_line(_result(8))
    got = json.loads(line)
    assert len(line) <= bench.LINE_LIMIT < 16000 and "\n" not in line
    for k, v in HEAD.items():
        assert got[k] == v, k
    assert got["kernel_rooflines"]["fit"] == {"frac": 0.123457}
    assert got["facet_size_scan"]["rows"][0] == {"K": 20, "m1": -0.1}


def test_a_line_that_would_still_be_long_loses_its_last_blocks():
    line = bench.printed_line(_result(2000))
    got = json.loads(line)
    assert len(line) <= bench.LINE_LIMIT
    for k, v in HEAD.items():
        assert got[k] == v, k
    assert got["kernel_rooflines"]["fit"] == {"frac": 0.123457}


def test_the_whole_result_goes_to_the_detail_file(tmp_path, capsys):
    res = _result(8)
    bench.finish(res, str(tmp_path / "detail.json"))
    assert json.loads((tmp_path / "detail.json").read_text()) == res
    assert capsys.readouterr().out.count("\n") == 1
