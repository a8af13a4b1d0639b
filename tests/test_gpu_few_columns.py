"""Rows in and out and the FP64 projector GEMMs at the row counts where the kernels change (one block of 16
columns, two, three, the 64-column tile) and at band and atom counts that leave a block incomplete: P_c and H
on complex128 rows on the device against numpy and the oracle, and the same rows from host memory, from
a device pointer that only 8-byte loads may use, and through the allocation-free entry point."""
import ctypes as C

import numpy as np
import pytest

from oracle import OracleCell
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(10.0, 10.0, 3, 5), (12.5, 20.0, 17, 65), (9.0, 15.0, 64, 24)])
def system(request):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    L, ecut, natoms, nocc = request.param
    pos = place_atoms(CellSpec(f"few_{L}", 7, L, ecut, natoms, nocc, 1)) if natoms < 64 else \
        np.random.default_rng(4).uniform(0.0, L, (natoms, 3))
    cell = OracleCell(L, ecut, pos)
    s = System(L, ecut, pos)
    rng = np.random.default_rng(11)
    psi = np.linalg.qr(rng.standard_normal((cell.npw, nocc)) + 1j * rng.standard_normal((cell.npw, nocc)))[0].T
    s.set_occupied(np.ascontiguousarray(psi), np.linspace(-1.0, 0.0, nocc))
    yield s, cell, psi
    s.close()


def worst(a, b):
    return (np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)).max()


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 97])
def test_rows_on_the_device(system, rows):
    import torch
    s, cell, psi = system
    rng = np.random.default_rng(rows)
    c = rng.standard_normal((rows, cell.npw)) + 1j * rng.standard_normal((rows, cell.npw))
    d = torch.from_numpy(c).cuda()
    ref_p = c - (c @ psi.conj().T) @ psi
    assert worst(s.apply_pc(d).cpu().numpy(), ref_p) < 1e-13
    assert worst(s.apply_pc(c), ref_p) < 1e-13
    assert torch.equal(s.apply_pc_noalloc(d), s.apply_pc(d))
    shift = rng.standard_normal(rows)
    ref_h = cell.h_apply(c) - shift[:, None] * c
    assert worst(s.apply_h(d, torch.from_numpy(shift).cuda()).cpu().numpy(), ref_h) < 1e-13
    assert worst(s.apply_h(c, shift), ref_h) < 1e-13
    assert worst(s.apply_h(d).cpu().numpy(), cell.h_apply(c)) < 1e-13


def test_rows_at_an_odd_address_and_in_place(system):
    """Device rows that start 8 bytes off a 16-byte boundary, and output over the input."""
    import torch
    from paper_2607_14025_amd import stern
    s, cell, psi = system
    rng = np.random.default_rng(2)
    c = rng.standard_normal((5, cell.npw)) + 1j * rng.standard_normal((5, cell.npw))
    ref = c - (c @ psi.conj().T) @ psi
    flat = torch.zeros(2 * c.size + 1, dtype=torch.float64, device="cuda")
    flat[1:] = torch.from_numpy(c.view(np.float64).reshape(-1)).cuda()
    torch.cuda.synchronize()
    p = C.c_void_p(flat.data_ptr() + 8)
    assert stern.lib().stern_apply_pc(s._h, 5, p, p, stern.STERN_MEM_DEVICE) == 0
    out = flat[1:].cpu().numpy().view(np.complex128).reshape(5, -1)
    assert float(flat[0]) == 0.0 and worst(out, ref) < 1e-13
