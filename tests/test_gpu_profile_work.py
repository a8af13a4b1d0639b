"""Work credited by the per-launch profile of a mixed solve: one FP32 operator pass per solve and inner iteration, and
none after the last solve has converged."""
import math

import pytest

pytestmark = pytest.mark.gpu


def test_profiled_mixed_solve_credits_its_iterations(tiny_system):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import STERN_MIXED, System
    t = tiny_system
    s = System(t["spec"].L, t["spec"].ecut, t["gs"]["pos"])
    s.set_occupied(t["gs"]["psi"], t["eps"])
    plain = s.apply_chi0(t["dv"][:3], tol=1e-10, precision=STERN_MIXED)[1]
    info = s.apply_chi0(t["dv"][:3], tol=1e-10, precision=STERN_MIXED, profile=True)[1]
    N, nm = s.fft_n, int(math.sqrt(t["spec"].ecut) * t["spec"].L / (2.0 * math.pi))
    s.close()
    assert info["n_converged"] == 48 and info["n_fallback"] == 0
    assert info["total_iters"] == plain["total_iters"]
    nza = 2 * nm + 1
    per_row = N * ((2.0 * nza + 2.0 * N) * 5.0 * N * math.log2(N) + 2.0 * N * N)
    k = info["kernels"]["plane_h32"]
    # every solve of a pass that is still counted makes one iteration in it
    assert k["flops"] == pytest.approx(info["total_iters"] * per_row, rel=1e-12)
    # the x pencils of each pass: two launches
    assert info["kernels"]["x32"]["launches"] == 2 * k["launches"]
