"""The Liouville apply of many excitations of few bands: the densities and their potentials go in chunks of about 2 GB, as the
full grids do, and the excitations on both sides of a chunk's end are those of an apply of their own."""
import numpy as np
import pytest

from synth.cells import CellSpec, place_atoms

pytestmark = pytest.mark.gpu


def test_chunks_of_excitations(monkeypatch):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    real, sizes = torch.cuda.caching_allocator_alloc, []

    def alloc(size, device=None, stream=None):
        sizes.append(size)
        return real(size, device, stream)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
    n_exc, L, ecut = 9000, 10.0, 10.0
    s = System(L, ecut, place_atoms(CellSpec("many_exc", 7, L, ecut, 3, 4, 1)), torch_allocator=True)
    rng = np.random.default_rng(5)
    psi = rng.standard_normal((1, s.n_pw)) + 1j * rng.standard_normal((1, s.n_pw))
    s.set_occupied(psi / np.linalg.norm(psi), np.array([-1.0]))
    gen = torch.Generator(device="cuda").manual_seed(1)
    a = torch.randn(n_exc, 1, s.n_pw, dtype=torch.complex128, device="cuda", generator=gen)
    out = s.liouville_apply(a)
    grid = s.fft_n ** 3 * 16  # one density; with the pencils and coefficients of its sphere less than twice that
    assert 1 << 30 < n_exc * grid and max(sizes) <= 5 << 28
    per = [k for k in range(0, n_exc, 499)] + [n_exc - 1]
    for k in per:
        one = s.liouville_apply(a[k:k + 1].contiguous())[0]
        assert float((out[k] - one).abs().max()) <= 1e-13 * float(one.abs().max()), k
    s.close()
