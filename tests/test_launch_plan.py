"""The launch plan of a greedy batch (host code, no GPU): every diagram fits
the LDS budget of its launch, whatever the batch's sizes and count."""
import ctypes as C
import random
import re

import numpy as np
import pytest

N_CU = 256


@pytest.fixture(scope="module")
def lib():
    from paper_2604_01059_amd import zx
    return zx.load()


def plan(lib, sizes, begin=0):
    a = np.ascontiguousarray(sizes, dtype=np.int32)
    out = [(C.c_int32 * 8)() for _ in range(3)]
    k = lib.zx_plan_launches(a.ctypes.data_as(C.c_void_p), len(a), begin, N_CU, *out)
    return [tuple(o[i] for o in out) for i in range(k)]


def budget(lib, variant):
    """LDS bytes of a variant, from its name (by-size itself is never a launch)."""
    lib.zx_simplify_variant_name.restype = C.c_char_p
    return int(re.match(r"bs\d+-lds(\d+)k$", lib.zx_simplify_variant_name(variant).decode()).group(1)) * 1024


def aux_bytes(n):
    """Phases and increments (n bytes each), partners and the selected list
    (2 n each), rounded up to words, and eight masks of ceil(n / 64) words."""
    return 2 * ((n + 7) // 8 * 8) + 2 * ((2 * n + 7) // 8 * 8) + 64 * ((n + 63) // 64)


def check(lib, sizes, begin=0):
    at = begin
    for variant, first, count in plan(lib, sizes, begin):
        assert first == at and count > 0
        at += count
        n, cap = sizes[first], budget(lib, variant)
        assert aux_bytes(n) <= cap, (len(sizes), n, cap)
    assert at == len(sizes)


@pytest.mark.parametrize("n", [1, 64, 65, 128, 500, 1024, 1472, 1857, 2048, 2920, 2922, 4096, 4672, 4681, 4700, 5000, 5900,
                               6014, 6428, 8000, 8192])
def test_equal_sizes_fit(lib, n):
    for count in [1, 2, 255, 256, 257, 511, 512, 513, 700, 760, 1024, 1025, 4096, 20000]:
        check(lib, [n] * count)


def test_uneven_sizes_fit(lib):
    rng = random.Random(7)
    check(lib, [4700] * 64 + [1400] * 40000)
    check(lib, sorted((16 + 6000 * i // 4096 for i in range(4096)), reverse=True))
    for _ in range(300):
        hi = int(2 ** rng.uniform(4, 13))
        count = int(2 ** rng.uniform(0, 13))
        sizes = sorted((int(2 ** rng.uniform(0, np.log2(hi))) for _ in range(count)), reverse=True)
        sizes += [rng.randint(1, 64)] * rng.choice([0, 0, 3000])
        sizes.sort(reverse=True)
        begin = rng.choice([0, 0, 1, min(8, len(sizes)), len(sizes)])
        check(lib, sizes, begin)


@pytest.mark.parametrize("n", [1153, 1472, 2048, 3000, 4600, 6500, 8192])
@pytest.mark.parametrize("count", [257, 300, 512, 600, 1024, 4096])
def test_rows_that_no_budget_holds(lib, n, count):
    """Diagrams whose rows no budget holds, more of them than CUs: two on a CU
    (64 KiB) take less time than one (152 KiB) or four with half the threads."""
    assert [budget(lib, v) for v, _, _ in plan(lib, [n] * count)] == [64 * 1024]
