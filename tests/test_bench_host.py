"""What the bench reports of a build's kernels, without a GPU."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
bench = pytest.importorskip("bench")


def test_radix_passes_are_the_traced_ones():
    T, NO, R = 1000, 5000, 40_000
    b = bench.survey_bytes(T, NO, R, 3)
    assert b == 80 * T + 64 * NO + 8 * R
    # sorted as pairs: three passes of ten builds, and the model's bytes are the build's
    f = bench.survey_fields(b, 3, {"count_scan": (10, 0.2), "onesweep": (30, 0.5), "ranges": (10, 0.1)}, 10, 1e-3)
    assert f["radix_passes"] == 3 and not f["by_records"]
    assert f["frac_survey_model"] == f["pair_sort_equivalent"] == round(b / 1e-6 / 1e9 / bench.HBM_PEAK_GBS, 4)
    # by records: two passes, and no fraction of a roofline from bytes that were not moved
    f = bench.survey_fields(b, 3, {"records": (10, 0.2), "onesweep": (20, 0.3), "finish": (10, 0.2)}, 10, 1e-3)
    assert f["radix_passes"] == 2 and f["by_records"] and f["survey_model_passes"] == 3
    assert f["frac_survey_model"] is None and f["pair_sort_equivalent"] > 0
    # a batch's last pass has a name of its own
    assert bench.survey_fields(b, 3, {"onesweep": (2, 0.3), "onesweep_grids": (1, 0.2)}, 1, 1.0)["radix_passes"] == 3
