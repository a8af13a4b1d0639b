"""The autotuner's cache across kernel versions: choices that an older library stored under the same sizes were made between
other kernels and are not taken; those of this library are."""
import re

import pytest

pytestmark = pytest.mark.gpu


def test_choices_of_another_version_are_found_anew(tiny_system, tmp_path):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_14025_amd import System
    t = tiny_system
    s = System(t["spec"].L, t["spec"].ecut, t["gs"]["pos"])
    s.set_occupied(t["gs"]["psi"], t["eps"])
    first = tmp_path / "first.txt"
    n, chosen = s.autotune(n_vec=32, cache_path=str(first))
    old = re.sub(r" kernels=\d+", "", first.read_text())  # the lines that carried no version
    old = re.sub(r"(tune=[01] value=)\d", r"\g<1>2", old)
    cache = tmp_path / "old.txt"
    cache.write_text(old)
    n2, _ = s.autotune(n_vec=32, cache_path=str(cache))
    assert n > 0 and n2 == n
    lines = cache.read_text().splitlines()
    assert lines[:5] == old.splitlines() and len(lines) == 10  # appended; what was there stays
    assert s.autotune(n_vec=32, cache_path=str(cache))[0] == 0
    s.close()
