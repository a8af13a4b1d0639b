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


@pytest.mark.parametrize("limit", [1, 2, 3])
def test_direct_term_in_smaller_blocks(refusing, limit):
    """The pairs' potentials of `limit` bands at most fit: the direct term takes fewer bands at a time."""
    import numpy as np
    from oracle import OracleCell
    from oracle.liouville import liouville_apply
    from paper_2607_14025_amd import System
    from synth.cells import CellSpec, place_atoms
    L, ecut, nocc, n_scr = 8.0, 6.0, 9, 5
    pos = place_atoms(CellSpec("exchange_blocks", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos)
    rng = np.random.default_rng(3)
    psi = np.ascontiguousarray(np.linalg.qr(rng.standard_normal((cell.npw, nocc)) +
                                            1j * rng.standard_normal((cell.npw, nocc)))[0].T)
    eps = np.linspace(-0.8, -0.1, nocc)
    screen = (rng.standard_normal((n_scr, cell.N, cell.N, cell.N)), rng.uniform(-0.8, 0.2, n_scr))
    a = rng.standard_normal((1, nocc, cell.npw)) + 1j * rng.standard_normal((1, nocc, cell.npw))
    s = System(L, ecut, pos, torch_allocator=True)
    mil = s.miller()
    s.set_occupied(cell.give(psi, mil), eps)
    s.liouville_set_kernel(1.0)
    s.liouville_set_screening(*screen)
    refusing["sizes"] = lambda n: limit * nocc * cell.N ** 3 * 16 < n <= 4 * nocc * cell.N ** 3 * 16
    out = s.liouville_apply(cell.give(a.reshape(-1, cell.npw), mil).reshape(a.shape))
    s.close()
    assert refusing["seen"]
    out = cell.take(out.reshape(-1, cell.npw), mil).reshape(a.shape)
    ref = liouville_apply(cell, psi, eps, a, 1.0, screen)
    assert np.abs(out - ref).max() <= 1e-12 * np.abs(ref).max()
