"""The yz kernels of the products and band sums with whole lines in registers: the right-hand sides, the density
response and the Liouville apply on even grids of every kind (four lanes to a line only where the grid is a
multiple of four, explicit grids far above the cutoff, where neither runs), with band and field counts that
leave their groups incomplete, against the oracle. A field's response to a few bands takes both kernels."""
import numpy as np
import pytest

from oracle import OracleCell, apply_chi0
from oracle.liouville import liouville_apply
from oracle.sternheimer import rel_l2
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu

# (L, ecut, fft_n or 0, grid, bands, fields)
CASES = [(7.0, 4.0, 0, 12, 3, 2), (8.0, 6.0, 0, 16, 5, 9), (8.0, 8.0, 0, 18, 4, 3), (10.0, 10.0, 0, 24, 9, 17),
         (9.0, 7.0, 32, 32, 5, 5), (10.0, 10.0, 36, 36, 5, 3), (7.0, 4.0, 48, 48, 3, 1), (10.0, 10.0, 54, 54, 2, 3)]


def system(L, ecut, fft_n, grid, nocc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    pos = place_atoms(CellSpec(f"products_{grid}", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos, N=grid)
    e, U = np.linalg.eigh(cell.h_dense())
    s = System(L, ecut, pos, fft_n=fft_n)
    assert s.fft_n == grid
    mil = s.miller()
    psi = np.ascontiguousarray(U.T[:nocc])
    s.set_occupied(cell.give(psi, mil), e[:nocc])
    return s, cell, psi, e[:nocc], mil


@pytest.mark.parametrize("L,ecut,fft_n,grid,nocc,nf", CASES)
def test_response_matches_oracle(L, ecut, fft_n, grid, nocc, nf):
    s, cell, psi, eps, _ = system(L, ecut, fft_n, grid, nocc)
    dv = np.random.default_rng(grid).standard_normal((nf, grid, grid, grid))
    ref = apply_chi0(cell, psi, eps, dv, tol=1e-12)["dn"]
    dn, info = s.apply_chi0(dv, tol=1e-11)
    assert info["n_converged"] == nocc * nf and rel_l2(dn, ref).max() < 1e-9
    s.close()


@pytest.mark.parametrize("L,ecut,fft_n,grid,nocc,nf", CASES)
def test_liouville_apply_matches_oracle(L, ecut, fft_n, grid, nocc, nf):
    s, cell, psi, eps, mil = system(L, ecut, fft_n, grid, nocc)
    rng = np.random.default_rng(grid + 1)
    a = rng.standard_normal((nf, nocc, cell.npw)) + 1j * rng.standard_normal((nf, nocc, cell.npw))
    out = s.liouville_apply(cell.give(a.reshape(-1, cell.npw), mil).reshape(a.shape))
    out = cell.take(out.reshape(-1, cell.npw), mil).reshape(a.shape)
    ref = liouville_apply(cell, psi, eps, a)
    assert np.abs(out - ref).max() <= 1e-12 * np.abs(ref).max()
    s.close()
