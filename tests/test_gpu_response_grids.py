"""The density response on grids at both sides of the rules that choose the kernels of its right-hand sides (54^3 and 96^3
with the full plane in LDS, 48^3 and 64^3 with lines in registers) and of its band sums (72^3 with the full plane), in
the geometry of a default grid, against the oracle. The bands are random orthonormal rows and their energies lie below
the spectrum, so that the systems are positive definite; 17 bands are two segments of the band sums."""
import numpy as np
import pytest

from oracle import OracleCell, apply_chi0
from oracle.sternheimer import rel_l2
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ecut,grid,nocc,nf", [(15.3, 20.0, 48, 17, 2), (17.0, 20.0, 54, 3, 3), (18.0, 25.0, 64, 17, 1),
                                                 (20.0, 25.0, 72, 3, 2), (22.0, 36.0, 96, 2, 2)])
def test_response_matches_oracle(L, ecut, grid, nocc, nf):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    pos = place_atoms(CellSpec(f"response_{grid}", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos)
    s = System(L, ecut, pos)
    assert s.fft_n == cell.N == grid
    rng = np.random.default_rng(grid)
    psi = rng.standard_normal((cell.npw, nocc)) + 1j * rng.standard_normal((cell.npw, nocc))
    psi = np.ascontiguousarray(np.linalg.qr(psi / (1.0 + cell.g2)[:, None])[0].T)
    eps = np.linspace(-9.0, -8.0, nocc)
    s.set_occupied(cell.give(psi, s.miller()), eps)
    dv = rng.standard_normal((nf, grid, grid, grid))
    print(f"case: {grid}^3, {nocc} bands x {nf} fields", flush=True)
    dn, info = s.apply_chi0(dv, tol=1e-11)
    s.close()
    assert info["n_converged"] == nocc * nf
    # both solve to 1e-11 of systems whose smallest eigenvalue is above a tenth of the largest preconditioned one
    assert rel_l2(dn, apply_chi0(cell, psi, eps, dv, tol=1e-12)["dn"]).max() < 1e-9
