"""The benchmark's stored counter figures, without a GPU."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench


def test_a_stored_figure_holds_for_its_schedule_and_code_only():
    (workload, f), meas = next(iter(bench.MEASURED_TRAFFIC.items()))
    code = bench.MEASURED_ON_CODE
    assert bench.stored_traffic(workload, f, meas["schedule"], code) == (meas, None)
    assert bench.stored_traffic(workload, f + 1, meas["schedule"], code) == (None, None)
    got, why = bench.stored_traffic(workload, f, meas["schedule"] + "x", code)
    assert got is None and "schedule" in why
    got, why = bench.stored_traffic(workload, f, meas["schedule"], "0" * 16)
    assert got is None and "code" in why


def test_the_code_digest_follows_the_code_and_not_its_comments(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2005_03300_amd" / "csrc"
    csrc.mkdir(parents=True)
    (csrc / "schedules.hip").write_text("int g();\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))

    def digest(text):
        (csrc / "spmm.hip").write_text(text)
        return bench.sparse_code_digest()
    first = digest("int f(int a) { return a; }\n")
    assert digest("// words\nint f(int a) {\n  /* more\n words */ return a;  // and more\n}\n") == first
    assert digest("int f(int a) { return a + 1; }\n") != first


def test_every_stored_figure_is_the_one_of_its_profile():
    for meas in bench.MEASURED_TRAFFIC.values():
        with open(os.path.join(ROOT, meas["profile"])) as fh:
            text = fh.read()
        assert meas["schedule"] in text
        assert re.search(r"per product \((\d+) bytes\)", text).group(1) == str(meas["bytes"])
