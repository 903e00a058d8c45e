"""The large workload's line (no GPU): the bytes, label and shares follow from
the steps that the library says its two-step passes took, whatever the
parameters would suggest."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(__file__), ".."))
import bench  # noqa: E402


def library(passes):
    """A stand-in whose passes of two steps take passes(t) of the steps from t."""
    class Lat:
        def __init__(self, p, stream=None):
            self.t, self.passed = 0, 0

        def step(self, n):
            for _ in range(n):
                self.passed += passes(self.t)
                self.t += 1

        def pass_steps(self):
            return self.passed

        def kernel_time(self):
            return 20.0, 20  # 1 ms a step

        def get_launch(self):
            return {}

        def autotune(self, reps):
            return []

        def fourier_mode(self, *a):
            return 0j

        def nothing(self, *a):
            pass

        set_fields = sync = profile = close = set_launch = nothing

    class F:
        FP32_SHIFTED, FP64, INIT_FIELDS = 1, 0, 2
        BASIS_FNORM_LOCAL, BASIS_HERMITE, BASIS_FNORM_LUT = 0, 1, 2
        Lattice = Lat

        @staticmethod
        def make_params(*a, **k):
            return type("P", (), dict(precision=k["precision"], block_steps=0))

        @staticmethod
        def copy_probe(*a, **k):
            return 300.0  # one settling step

        stream_copy_probe = copy_probe

    class torch:
        class cuda:
            @staticmethod
            def current_stream():
                return None

            @staticmethod
            def synchronize():
                pass

    return F, torch


@pytest.mark.parametrize("passes,kw,share,label", [
    (lambda t: 1, dict(), 1.0, "step_march_kernel<fnorm_local>"),
    # the second buffer was refused, or the flow is too fast for FP32 collisions
    (lambda t: 0, dict(), 0.0, "step_kernel<float,float,fnorm_local>"),
    (lambda t: 0, dict(ux0=0.3), 0.0, "step_kernel<float,double,fnorm_local>"),
    # eight of ten steps between samples
    (lambda t: t % 10 >= 2, dict(sample_every=10), 0.8,
     "step_march_kernel<fnorm_local> and step_kernel<float,float,fnorm_local> "
     "(correlator-sampling variant every 10 steps)"),
])
def test_bytes_follow_the_steps_taken(passes, kw, share, label):
    F, torch = library(passes)
    r = bench.run_large(F, torch, 20, 10, nx=128, every=0, **kw)
    out = bench.large_rooflines(r)
    rf = out["roofline"]
    moved = 72 * (1 - share / 2)
    assert rf["pass_steps"] == 20 * share and rf["bytes_per_site"] == pytest.approx(moved)
    assert rf["kernel"] == label
    gbps = moved * 128 * 128 / 1e-3 / 1e9
    assert rf["bound"] == "hbm" and rf["unit"] == "GB/s" and rf["peak"] == 8000.0
    assert rf["achieved"] == pytest.approx(gbps, abs=0.06)
    assert out["pct_hbm_roofline"] == pytest.approx(
        out["pct_of_one_pass_rate"] * (1 - share / 2), abs=0.02)
    assert ("valu_issue" in out) == (share > 0 and "sample_every" not in kw)
    assert rf["traffic"] is None or share > 0
