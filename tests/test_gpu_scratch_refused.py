"""Scratch that the library can do without: where its allocation fails (the caller's allocator tried hipMalloc, which
leaves the runtime's last error set, and returns NULL) the call still runs and gives the same result, and leaves no error
behind."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def refusing(monkeypatch):
    """Sizes for which the allocator fails; what it refused is kept in `seen`."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd.stern import lib
    real = torch.cuda.caching_allocator_alloc
    state = dict(sizes=lambda n: False, seen=[])
    hip_malloc = lib().hipMalloc  # of the runtime that the library runs on
    hip_malloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]

    def alloc(size, device=None, stream=None):
        if state["sizes"](size):
            state["seen"].append(size)
            p = C.c_void_p()
            assert hip_malloc(C.byref(p), 1 << 50) != 0
            raise RuntimeError("refused")
        return real(size, device, stream)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
    return state


def test_density_response_without_segment_scratch(tiny_system, refusing):
    from paper_2607_14025_amd import System
    from paper_2607_14025_amd.stern import lib
    t = tiny_system
    dv, N = t["dv"][:3], t["cell"].N
    out, error = [], lib().stern_last_error()
    for refuse in (False, True):
        s = System(t["spec"].L, t["spec"].ecut, t["gs"]["pos"], torch_allocator=True)
        s.set_occupied(t["gs"]["psi"], t["eps"])
        assert s.n_occ == 16  # two segments of 8 bands: a grid per segment and field
        refusing["sizes"] = lambda n: refuse and n == 2 * 3 * N ** 3 * 8
        dn, info = s.apply_chi0(dv, tol=1e-10)
        assert info["n_converged"] == 48
        out.append(dn)
        assert lib().stern_last_error() == error
        s.close()
    assert len(refusing["seen"]) == 1
    assert abs(out[0] - out[1]).max() <= 1e-14 * abs(out[0]).max()  # 16 products summed in another grouping


def test_transition_densities_without_segment_scratch(tiny_system, refusing):
    import numpy as np
    from paper_2607_14025_amd import System
    t = tiny_system
    N = t["cell"].N
    rng = np.random.default_rng(4)
    out = []
    for refuse in (False, True):
        s = System(t["spec"].L, t["spec"].ecut, t["gs"]["pos"], torch_allocator=True)
        s.set_occupied(t["gs"]["psi"], t["eps"])
        if not refuse:
            a = rng.standard_normal((3, 16, s.n_pw)) + 1j * rng.standard_normal((3, 16, s.n_pw))
        refusing["sizes"] = lambda n: refuse and n == 2 * 3 * N ** 3 * 16
        out.append(s.liouville_apply(a))
        s.close()
    assert len(refusing["seen"]) == 1
    assert abs(out[0] - out[1]).max() <= 1e-13 * abs(out[0]).max()
