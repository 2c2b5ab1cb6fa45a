"""Batched parities on the matrix cores (zx_gf2_matmul) and the phase-pair
product (zx_phase_pair_product) against the oracle.

Parities are bits: compared exactly.  The phase-pair product is fp32 complex
against the oracle's fp64; the tolerance is derived from the arithmetic:
each factor h has four terms of magnitude <= 1 summed with three fp32
roundings (<= 12u per component) plus the fp32 rounding of sqrt(1/2) in the
table (< 1.1u), i.e. an absolute error < 18.6u, which is a relative error
< 17.2u since every non-zero h has |h| >= 1.0824; each complex product adds
< 3u; the constant sqrt(2) and table value add < 2u.  Relative tolerance
(21 m + 4) u, u = 2^-24, m terms.  Zero factors (h = 0 exactly) are exact
zeros on both sides.
"""
import numpy as np
import pytest

import oracle
from oracle import phase as oph
from workloads import parity_problem
from workloads.generators import pack_rows

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (3, 70, 64), (257, 300, 200), (513, 1000, 130),
                                   (40, 600, 2000), (300, 257, 63),
                                   # beyond 2048 bits: the chunked 256 x 256 kernel, ragged rows and K
                                   (300, 700, 3000), (1100, 530, 2100), (5, 2049, 4100)])
def test_gf2_matmul_matches_oracle(zx, m, n, k):
    import torch
    print("gf2_matmul case", m, n, k, flush=True)
    rng = np.random.default_rng(m + 7 * n + 13 * k)
    U = pack_rows((rng.random((m, k)) < 0.5).astype(np.uint8))
    F = pack_rows((rng.random((n, k)) < 0.3).astype(np.uint8))
    Ug, Fg = U.copy(), F.copy()
    if k % 64:  # junk beyond k_bits must be ignored
        junk = np.uint64(~((1 << (k % 64)) - 1) & (2 ** 64 - 1))
        Ug[:, -1] |= junk
        Fg[:, -1] |= junk
    C = zx.gf2_matmul(zx.to_device_words(Ug), zx.to_device_words(Fg), k)
    torch.cuda.synchronize()
    assert np.array_equal(zx.to_host_words(C), oracle.gf2_matmul(U, F, k))


def test_gf2_matmul_full_size_sampled(zx):
    """The benchmark contraction (4096 terms x 65536 settings x 1024
    parameters): sampled term rows against the oracle, all settings."""
    import torch
    P = parity_problem(61, 4096, 65536, 1024)
    C = zx.gf2_matmul(zx.to_device_words(P.U), zx.to_device_words(P.F), P.n_params)
    torch.cuda.synchronize()
    Ch = zx.to_host_words(C)
    for r in (0, 255, 256, 4095):
        assert np.array_equal(Ch[r:r + 1], oracle.gf2_matmul(P.U[r:r + 1], P.F, P.n_params)), r


def _compare(mg, eg, mo, eo, m):
    tol = (21 * m + 4) * U32
    zg = mg[:, 0].astype(np.float64) + 1j * mg[:, 1].astype(np.float64)
    for l in range(len(mo)):
        if mo[l] == 0:
            assert zg[l] == 0, l
            continue
        d = abs(zg[l] * 2.0 ** float(int(eg[l]) - int(eo[l])) - mo[l])
        assert d <= tol * abs(mo[l]), (l, d, tol)


@pytest.mark.parametrize("seed,m,n", [(0, 0, 5), (1, 1, 64), (2, 37, 300), (3, 300, 200), (4, 1000, 65)])
def test_phase_pair_product_matches_oracle(zx, seed, m, n):
    import torch
    print("phase_pair case", seed, m, n, flush=True)
    rng = np.random.default_rng(500 + seed)
    ka = rng.integers(0, 8, m).astype(np.int8)
    kb = rng.integers(0, 8, m).astype(np.int8)
    if seed == 2:
        ka[::3], kb[::3] = 2, 6   # zero factors where a = b = 0
    A = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8)) if m else np.zeros((0, 1), np.uint64)
    B = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8)) if m else np.zeros((0, 1), np.uint64)
    phase8, pw = int(rng.integers(0, 8)), int(rng.integers(-9, 10))
    mo, eo = oph.phase_pair_product(A, B, ka, kb, n, phase8, pw)
    dev = "cuda"
    tA = zx.to_device_words(A) if m else None
    tB = zx.to_device_words(B) if m else None
    mg, eg = zx.phase_pair_product(tA, tB, torch.from_numpy(ka).to(dev), torch.from_numpy(kb).to(dev), n,
                                   phase8, pw)
    torch.cuda.synchronize()
    _compare(mg.cpu().numpy(), eg.cpu().numpy(), mo, eo, m)


@pytest.mark.parametrize("m,n", [(1, 1), (2, 63), (63, 64), (64, 65), (65, 255), (129, 256), (257, 257), (600, 2050)])
@pytest.mark.parametrize("last", ["unit", "any"])
def test_phase_pair_unit_terms(zx, m, n, last):
    """Terms whose factors are all 2 i^s (even codes, one of them 0 or 4) are
    counted and not multiplied: edges of the 64-term slices and of the
    256-setting blocks, either code first, both parities present.  The
    product is then exact but for the constant (tolerance of no factor at
    all).  With one other term at the end the whole product is multiplied
    out (tolerance of m factors)."""
    import torch
    print("phase_pair unit case", m, n, last, flush=True)
    rng = np.random.default_rng(900 + 31 * m + n)
    ka = 4 * rng.integers(0, 2, m)
    kb = 2 * rng.integers(0, 4, m)
    swap = rng.random(m) < 0.5
    ka, kb = np.where(swap, kb, ka).astype(np.int8), np.where(swap, ka, kb).astype(np.int8)
    if last == "any":
        ka[-1] = 3
    A = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8))
    B = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8))
    phase8, pw = int(rng.integers(0, 8)), int(rng.integers(-9, 10))
    mo, eo = oph.phase_pair_product(A, B, ka, kb, n, phase8, pw)
    mg, eg = zx.phase_pair_product(zx.to_device_words(A), zx.to_device_words(B), torch.from_numpy(ka).cuda(),
                                   torch.from_numpy(kb).cuda(), n, phase8, pw)
    torch.cuda.synchronize()
    _compare(mg.cpu().numpy(), eg.cpu().numpy(), mo, eo, 0 if last == "unit" else m)


@pytest.mark.parametrize("m,n,k", [(2500, 7000, 700), (1030, 16500, 70), (255, 257, 256), (129, 128, 257),
                                   (2049, 8200, 520)])
def test_gf2_matmul_tiles(zx, m, n, k):
    """Both tile sizes: rows of tiles off the band height of four, ragged
    rows, columns and words, odd row lengths, junk beyond the last bit."""
    import torch
    print("gf2_matmul tiles case", m, n, k, flush=True)
    rng = np.random.default_rng(m + 3 * n + 5 * k)
    kw = (k + 63) // 64
    U = rng.integers(0, 2 ** 64, (m, kw), dtype=np.uint64)
    F = rng.integers(0, 2 ** 64, (n, kw), dtype=np.uint64)
    C = zx.gf2_matmul(zx.to_device_words(U), zx.to_device_words(F), k)
    torch.cuda.synchronize()
    if k % 64:
        U[:, -1] &= np.uint64((1 << (k % 64)) - 1)
        F[:, -1] &= np.uint64((1 << (k % 64)) - 1)
    rows = sorted({0, 1, 63, 64, 127, 128, m // 2, m - 2, m - 1})
    Ch = zx.to_host_words(C)
    for r in (r for r in rows if r < m):
        assert np.array_equal(Ch[r:r + 1], oracle.gf2_matmul(U[r:r + 1], F, k)), r
    # every row: the parity of a row of C is that of its A row against the XOR of all B rows
    tot = np.bitwise_xor.reduce(F, axis=0)
    want = (np.bitwise_count(U & tot).sum(axis=1) & 1)
    assert np.array_equal(np.bitwise_count(Ch).sum(axis=1) & 1, want)


@pytest.mark.parametrize("m,n,k", [(2, 3, (1 << 23) + 1), (3, 2, (1 << 24) + 77), (130, 5, (1 << 22) + 65),
                                   (3, 140, (1 << 22) - 1)])
def test_gf2_matmul_long_rows(zx, m, n, k):
    """Rows whose counts leave the exact range of the fp32 accumulators, with
    all-ones rows (the largest count) beside random ones."""
    import torch
    print("gf2_matmul long case", m, n, k, flush=True)
    rng = np.random.default_rng(m + n)
    kw = (k + 63) // 64
    U = rng.integers(0, 2 ** 64, (m, kw), dtype=np.uint64)
    F = rng.integers(0, 2 ** 64, (n, kw), dtype=np.uint64)
    U[0] = F[0] = np.uint64(2 ** 64 - 1)
    C = zx.gf2_matmul(zx.to_device_words(U), zx.to_device_words(F), k)
    torch.cuda.synchronize()
    if k % 64:
        U[:, -1] &= np.uint64((1 << (k % 64)) - 1)
    want = np.zeros((m, (n + 63) // 64), np.uint64)
    for i in range(m):
        for j in range(n):
            bit = int(np.bitwise_count(np.bitwise_xor.reduce(U[i] & F[j]))) & 1
            want[i, j // 64] |= np.uint64(bit << (j % 64))
    assert np.array_equal(zx.to_host_words(C), want)


@pytest.mark.parametrize("phase8", range(8))
def test_phase_pair_unit_terms_have_positive_zeros(zx, phase8):
    """A product of unit terms has no negative zero: the angle of a negative
    real one is pi, as that of a single factor -2 is."""
    import torch
    m, n = 5, 130
    rng = np.random.default_rng(40 + phase8)
    ka, kb = np.array([0, 4, 0, 4, 0], np.int8), np.array([2, 2, 6, 4, 0], np.int8)
    A = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8))
    B = pack_rows((rng.random((m, n)) < 0.5).astype(np.uint8))
    print("phase_pair zeros", phase8, flush=True)
    mo, eo = oph.phase_pair_product(A, B, ka, kb, n, phase8, 0)
    mg, eg = zx.phase_pair_product(zx.to_device_words(A), zx.to_device_words(B), torch.from_numpy(ka).cuda(),
                                   torch.from_numpy(kb).cuda(), n, phase8, 0)
    torch.cuda.synchronize()
    z = mg.cpu().numpy()
    _compare(z, eg.cpu().numpy(), mo, eo, 0)
    assert not np.signbit(z[z == 0]).any()
    zero = z == 0
    assert zero.any() == (phase8 % 2 == 0)


@pytest.mark.parametrize("m,n,k", [(8320, 1, 64), (33000, 130, 200), (20001, 300, 70), (70000, 40, 130)])
def test_gf2_matmul_tall(zx, m, n, k):
    """Few columns of tiles: bands of more than four rows of tiles, the last
    one short."""
    import torch
    print("gf2_matmul tall case", m, n, k, flush=True)
    rng = np.random.default_rng(m + n)
    kw = (k + 63) // 64
    U = rng.integers(0, 2 ** 64, (m, kw), dtype=np.uint64)
    F = rng.integers(0, 2 ** 64, (n, kw), dtype=np.uint64)
    C = zx.gf2_matmul(zx.to_device_words(U), zx.to_device_words(F), k)
    torch.cuda.synchronize()
    if k % 64:
        U[:, -1] &= np.uint64((1 << (k % 64)) - 1)
    assert np.array_equal(zx.to_host_words(C), oracle.gf2_matmul(U, F, k))
