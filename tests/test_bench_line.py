"""The bench line: what stands beside the headline is rounded, so that the line
stays under the 20,000 characters that a reader may take, and every coupling's
roofline names the kernel that runs."""
import json

import bench


def test_short_rounds_floats_only():
    x = {"a": 123456.789012345, "b": [1, 0.1 + 0.2, "s", None, True], "c": {"d": -1.23456789e-12}}
    assert bench._short(x) == {"a": 123457.0, "b": [1, 0.3, "s", None, True], "c": {"d": -1.23457e-12}}
    assert len(json.dumps(bench._short([1.0 / 3.0] * 100))) < 100 * 11


def test_every_coupling_has_its_kernel():
    want = {1: "k_sweep", 2: "k_sweep", 3: "k_sweep", 4: "k_sweep_t", 5: "k_sweep_lw", 6: "k_sweep_ch",
            7: "k_sweep_ch", 8: "k_sweep_ch", 9: "k_sweep_rc", 10: "k_sweep_rc"}
    assert {c: bench.SWEEP_KERNELS.get(c, "k_sweep") for c in bench.COUPLINGS} == want
