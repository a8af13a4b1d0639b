"""The yz pass with whole lines in registers (even grids): the FP64 H apply against the oracle on every
even grid the basis builds by default, with row counts that leave its groups of vectors incomplete, on
grids whose sphere reaches the last index the kernel takes, and on explicit grids far above the cutoff
(too few active lines for it: the two-stage kernel runs). Both precisions through the variants of the
chi0 apply are covered by test_gpu_autotune.py."""
import numpy as np
import pytest

from oracle import OracleCell
from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu

# (L, ecut, fft_n or 0, grid): default grids, then K = (N - 1) / 4 reached, then fft_n >> needed
CASES = [(7.0, 4.0, 0, 12), (8.0, 6.0, 0, 16), (8.0, 8.0, 0, 18), (10.0, 10.0, 0, 24),
         (12.9, 12.0, 0, 32), (12.5, 15.0, 0, 36), (15.3, 20.0, 0, 48), (17.0, 20.0, 0, 54), (18.0, 25.0, 0, 64),
         (20.0, 25.0, 0, 72), (22.0, 36.0, 0, 96), (5.0, 2.0, 8, 8), (10.0, 12.0, 24, 24), (6.0, 3.0, 32, 32),
         (6.0, 3.0, 72, 72)]


def residuals(L, ecut, fft_n, grid, rows):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    pos = place_atoms(CellSpec(f"half_{grid}", 7, L, ecut, 3, 4, 1))
    cell = OracleCell(L, ecut, pos, N=grid)
    s = System(L, ecut, pos, fft_n=fft_n)
    assert s.fft_n == grid and s.n_pw == cell.npw
    rng = np.random.default_rng(grid + rows)
    c = rng.standard_normal((rows, cell.npw)) + 1j * rng.standard_normal((rows, cell.npw))
    shift = rng.standard_normal(rows)
    ref = cell.h_apply(c) - shift[:, None] * c
    out = s.apply_h(c, shift)
    s.close()
    return np.linalg.norm(out - ref, axis=1) / np.linalg.norm(ref, axis=1)


@pytest.mark.parametrize("rows", [1, 5, 19])
@pytest.mark.parametrize("L,ecut,fft_n,grid", CASES)
def test_h_apply_matches_oracle(L, ecut, fft_n, grid, rows):
    assert residuals(L, ecut, fft_n, grid, rows).max() < 1e-13


def test_groups_of_vectors():
    """Enough rows for whole groups (the number of vectors to a workgroup grows with the batch) and a
    remainder; every row equals the same row applied alone (to the order of the projectors' split sums)."""
    import torch
    from paper_2607_14025_amd import System
    pos = place_atoms(CellSpec("half_groups", 7, 12.5, 15.0, 3, 4, 1))
    s = System(12.5, 15.0, pos)
    gen = torch.Generator(device="cuda").manual_seed(3)
    c = torch.randn(131, s.n_pw, dtype=torch.complex128, device="cuda", generator=gen)
    out = s.apply_h(c)
    for k in (0, 63, 128, 130):
        one = s.apply_h(c[k:k + 1].contiguous())[0]
        assert float(torch.linalg.vector_norm(out[k] - one) / torch.linalg.vector_norm(one)) < 1e-14, k
    s.close()
