"""The direct term's pair potentials, formed for w <= v only and for up to four bands at a time, against the
oracle's grid route at band counts around the block (one band, an incomplete block, whole blocks, a
remainder), excitation counts around the four that one pass holds, and potential counts around the
sixteen that it adds in registers and the eight of a projection tile."""
import numpy as np
import pytest

from oracle import OracleCell
from oracle.liouville import liouville_apply
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nocc,n_exc,n_scr,alpha", [(1, 1, 0, 1.0), (3, 2, 5, 0.25), (4, 4, 8, 1.0), (5, 5, 9, 1.0),
                                                    (8, 3, 16, 0.0), (9, 9, 17, 1.0), (9, 1, 3, 0.5)])
def test_direct_term_matches_oracle(nocc, n_exc, n_scr, alpha):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    L, ecut = 8.0, 6.0
    pos = place_atoms(CellSpec("exchange_blocks", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos)
    s = System(L, ecut, pos)
    mil = s.miller()
    rng = np.random.default_rng(nocc * 100 + n_exc)
    psi = np.ascontiguousarray(np.linalg.qr(rng.standard_normal((cell.npw, nocc)) +
                                            1j * rng.standard_normal((cell.npw, nocc)))[0].T)
    eps = np.linspace(-0.8, -0.1, nocc)
    s.set_occupied(cell.give(psi, mil), eps)
    s.liouville_set_kernel(alpha)
    screen = None
    if n_scr:
        screen = (rng.standard_normal((n_scr, cell.N, cell.N, cell.N)), rng.uniform(-0.8, 0.2, n_scr))
        s.liouville_set_screening(*screen)
    a = rng.standard_normal((n_exc, nocc, cell.npw)) + 1j * rng.standard_normal((n_exc, nocc, cell.npw))
    out = s.liouville_apply(cell.give(a.reshape(-1, cell.npw), mil).reshape(a.shape))
    out = cell.take(out.reshape(-1, cell.npw), mil).reshape(a.shape)
    ref = liouville_apply(cell, psi, eps, a, alpha, screen)
    assert np.abs(out - ref).max() <= 1e-12 * np.abs(ref).max()
    s.close()
