"""Host rules of the kernel launches, through the library's own functions (no GPU): the LDS that the yz kernels are gated
by, and the split factors of the reduces."""
import ctypes
import math
import os

import pytest

stern = pytest.importorskip("paper_2607_14025_amd.stern")


def rule(name, res, *args):
    if not os.path.exists(stern.LIB_PATH):
        pytest.skip("libstern.so not built")
    f = getattr(stern.lib(), name)
    f.restype, f.argtypes = res, list(args)
    return f


@pytest.mark.parametrize("N,fp64,vectors", [(24, True, 8), (48, True, 4), (72, True, 2), (72, False, 2), (96, False, 2), (96, True, 1),
                                            (108, True, 1), (128, True, 1), (128, False, 1)])
def test_plane_gate_covers_the_kernel_with_lines_in_registers(N, fp64, vectors):
    """Its lines [vectors][active lines][N, padded to 2 mod 4], two twiddle tables and two column tables."""
    lds = rule("_ZN5stern12plane_hw_ldsEiib", ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_bool)
    rhs = rule("_ZN5stern14plane_fp64_ldsEii", ctypes.c_size_t, ctypes.c_int, ctypes.c_int)
    k = (N - 1) // 4
    nza, qld, tw, elem = 2 * k + 1, N + (6 - N % 4) % 4, (k + 1) | 1, 16 if fp64 else 8
    lines = vectors * nza * qld * elem
    need = lines + 2 * tw * (elem + 4)
    assert need <= lds(N, nza, fp64) and need <= 160 * 1024
    if fp64 and N != 96:  # there the right-hand sides take the full plane
        assert rhs(N, nza) >= lines


def choose_nsplit(*args, n_cu=256):
    return rule("_ZN5stern13choose_nsplitEiiiii", ctypes.c_int, *[ctypes.c_int] * 5)(*args, n_cu)


@pytest.mark.parametrize("target", [256, 1024, 2048, 4096])
@pytest.mark.parametrize("M,K", [(64, 576), (128, 16896), (1024, 91072)])
def test_tuned_reduces_keep_the_rules(M, K, target):
    """A workgroup target fills its last round as the default does, and few columns keep a count of their own."""
    bound = rule("_ZN5stern12nsplit_boundEiiii", ctypes.c_int, *[ctypes.c_int] * 4)

    def fill(ncols, ns):
        rounds = (M // 64) * math.ceil(ncols / 64) * ns / 1024
        return rounds / math.ceil(rounds)

    for n in (1, 16, 17, 48):
        assert choose_nsplit(M, n, K, target) == choose_nsplit(M, n, K, 0)
    for n in (49, 64, 200, 517, 1000, 4096):
        b, ns = bound(M, n, K, target), choose_nsplit(M, n, K, target)
        assert b // 2 <= ns <= b and ns >= 1
        assert fill(n, ns) >= max(fill(n, k) for k in range(b, b // 2, -1)) - 0.02 * (b - b // 2)
        assert fill(n, ns) >= fill(n, b)
        assert target != 2048 or ns == choose_nsplit(M, n, K, 0)  # the default's target, by name


@pytest.mark.parametrize("n_cu", [32, 64, 128])
def test_rounds_are_those_of_the_device(n_cu):
    """A device of fewer CUs (a partition) runs fewer workgroups at once: the split fills the last round there."""
    M, K = 1024, 91072
    for n in (64, 200, 517, 1000):
        base = (M // 64) * math.ceil(n / 64)
        fill = lambda ns: base * ns / (4 * n_cu) / math.ceil(base * ns / (4 * n_cu))
        assert fill(choose_nsplit(M, n, K, 0, n_cu=n_cu)) >= fill(choose_nsplit(M, n, K, 0)) - 0.02
    stretches = rule("_ZN5stern18scr_proj_stretchesEiiimi", ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_size_t,
                     ctypes.c_int)
    assert stretches(0, 1, 8, 48 ** 3, n_cu) == max(1, min(4 * n_cu, 48 ** 3 // 1024))


@pytest.mark.parametrize("n_cu", [256, 64])
def test_bf16_reduces_add_no_round(n_cu):
    """Chunks finer than 256 k, 128 k at the finest, only where they run in the rounds over the CUs that chunks of 256 k
    take, and never more workgroups than the target."""
    nsplit = rule("_ZN5stern18choose_nsplit_bf16Eiiiii", ctypes.c_int, *[ctypes.c_int] * 5)
    finer = 0
    for M in (64, 128, 256, 1024):
        for K in (64, 576, 5504, 7488, 12352, 16896, 27136, 38912, 91072):
            for n in (1, 96, 128, 129, 240, 512, 640, 864, 1024, 4096):
                base, ns = math.ceil(M / 128) * math.ceil(n / 128), nsplit(M, n, K, 0, n_cu)
                coarse = max(1, K // 256)
                assert 1 <= ns <= max(1, 512 // base) and ns <= max(1, K // 128)
                if base * coarse <= 512:
                    assert math.ceil(base * ns / n_cu) <= math.ceil(base * coarse / n_cu)
                    assert ns >= min(coarse, 512 // base)
                finer += ns > coarse
    assert finer > 0
