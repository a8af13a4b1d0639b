"""The Liouville apply on grids whose 4 Ecut sphere has more active z lines than the forward y stage takes in one
round of items (72^3 from 65 lines on, 81^3 from 57, 96^3 from 65): the Hartree term alone and with the pairs'
potentials, against the oracle's grid route. Lines at the most that a default grid has (72: 69, 96: 93) and that any
has (81: 81)."""
import numpy as np
import pytest

from oracle import OracleCell
from oracle.liouville import liouville_apply
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ecut,fft_n,grid,lines", [(21.5, 25.0, 0, 72, 69), (20.0, 41.0, 81, 81, 81), (22.5, 42.0, 0, 96, 93)])
@pytest.mark.parametrize("alpha", [0.0, 0.5])
def test_density_sphere_lines(L, ecut, fft_n, grid, lines, alpha):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    pos = place_atoms(CellSpec(f"density_{grid}", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos, N=grid)
    assert 2 * int(2.0 * np.sqrt(ecut) * L / (2.0 * np.pi)) + 1 == lines
    s = System(L, ecut, pos, fft_n=fft_n)
    assert s.fft_n == grid and s.n_pw == cell.npw
    mil = s.miller()
    rng = np.random.default_rng(grid)
    nocc, n_exc = 2, 2
    psi = np.ascontiguousarray(np.linalg.qr(rng.standard_normal((cell.npw, nocc)) +
                                            1j * rng.standard_normal((cell.npw, nocc)))[0].T)
    eps = np.linspace(-0.8, -0.1, nocc)
    s.set_occupied(cell.give(psi, mil), eps)
    s.liouville_set_kernel(alpha)
    a = rng.standard_normal((n_exc, nocc, cell.npw)) + 1j * rng.standard_normal((n_exc, nocc, cell.npw))
    print(f"case: {grid}^3, {lines} lines, alpha {alpha}", flush=True)
    out = s.liouville_apply(cell.give(a.reshape(-1, cell.npw), mil).reshape(a.shape))
    # the potential part alone: H on rows of this norm would hide an error in it
    pa = s.apply_pc(cell.give(a.reshape(-1, cell.npw), mil))
    d = s.apply_pc(s.apply_h(pa, np.tile(eps, n_exc)))
    s.close()
    out = cell.take((out.reshape(-1, cell.npw) - d), mil).reshape(a.shape)
    ref = liouville_apply(cell, psi, eps, a, alpha)
    ap = (a.reshape(-1, cell.npw) - (a.reshape(-1, cell.npw) @ psi.conj().T) @ psi)
    hd = cell.h_apply(ap) - np.tile(eps, n_exc)[:, None] * ap
    hd = hd - (hd @ psi.conj().T) @ psi
    ref = ref - hd.reshape(a.shape)
    # differences of the whole apply round at 1e-16 of its largest entries, about a hundred times the potential's
    scale = np.abs(hd).max()
    assert np.abs(out - ref).max() <= 1e-12 * np.abs(ref).max() + 1e-14 * scale
