"""Host rules of the kernel launches, through the library's own functions (no GPU): the LDS that the yz kernels are gated
by."""
import ctypes
import os

import pytest

stern = pytest.importorskip("paper_2607_14025_amd.stern")


def rule(name, res, *args):
    if not os.path.exists(stern.LIB_PATH):
        pytest.skip("libstern.so not built")
    f = getattr(stern.lib(), name)
    f.restype, f.argtypes = res, list(args)
    return f


@pytest.mark.parametrize("N,fp64,vectors", [(24, True, 8), (48, True, 4), (72, True, 2), (72, False, 2), (96, False, 2), (96, True, 1),
                                            (108, True, 1), (128, True, 1), (128, False, 1)])
def test_plane_gate_covers_the_kernel_with_lines_in_registers(N, fp64, vectors):
    """Its lines [vectors][active lines][N, padded to 2 mod 4], two twiddle tables and two column tables."""
    lds = rule("_ZN5stern12plane_hw_ldsEiib", ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_bool)
    rhs = rule("_ZN5stern14plane_fp64_ldsEii", ctypes.c_size_t, ctypes.c_int, ctypes.c_int)
    k = (N - 1) // 4
    nza, qld, tw, elem = 2 * k + 1, N + (6 - N % 4) % 4, (k + 1) | 1, 16 if fp64 else 8
    lines = vectors * nza * qld * elem
    need = lines + 2 * tw * (elem + 4)
    assert need <= lds(N, nza, fp64) and need <= 160 * 1024
    if fp64 and N != 96:  # there the right-hand sides take the full plane
        assert rhs(N, nza) >= lines
