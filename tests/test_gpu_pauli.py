"""GPU symplectic commutation table (zx_pauli_commute) vs the CPU oracle."""
import numpy as np
import pytest

import oracle
from workloads import pauli_strings

pytestmark = pytest.mark.gpu


VARIANTS = ["valu", "mfma"]


def _flags(zx, variant):
    return zx.ZX_PAULI_FORCE_VALU if variant == "valu" else zx.ZX_PAULI_FORCE_MFMA


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("n,q", [(1, 1), (2, 3), (63, 64), (64, 65), (65, 100), (200, 130),
                                 (300, 1024), (1000, 17), (129, 2000), (257, 64), (600, 300)])
def test_full_table(zx, n, q, variant):
    import torch
    print("pauli case", n, q, variant, flush=True)
    X, Z = pauli_strings(100 + n, n, q)
    Cg = zx.pauli_commute(zx.to_device_words(X), zx.to_device_words(Z), q, flags=_flags(zx, variant))
    torch.cuda.synchronize()
    Co = oracle.pauli_commute(X, Z)
    assert np.array_equal(zx.to_host_words(Cg), Co)


@pytest.mark.parametrize("variant", VARIANTS)
def test_bits_beyond_qubits_ignored(zx, variant):
    """Set bits at or beyond n_qubits in the last word change nothing."""
    import torch
    n, q = 700, 100
    X, Z = pauli_strings(7, n, q)
    Xg, Zg = X.copy(), Z.copy()
    junk = np.uint64(~((1 << (q % 64)) - 1) & (2 ** 64 - 1))
    Xg[:, -1] |= junk
    Zg[:, -1] |= junk
    Cg = zx.pauli_commute(zx.to_device_words(Xg), zx.to_device_words(Zg), q, flags=_flags(zx, variant))
    torch.cuda.synchronize()
    assert np.array_equal(zx.to_host_words(Cg), oracle.pauli_commute(X, Z))


def test_variants_equal_at_full_size(zx):
    """65536 strings on 1024 qubits (seed 22): the matrix-core table equals
    the vector-unit table bit for bit (both are compared with the oracle on
    sampled rows below)."""
    import torch
    n, q = 65536, 1024
    X, Z = pauli_strings(22, n, q)
    dX, dZ = zx.to_device_words(X), zx.to_device_words(Z)
    C1 = zx.pauli_commute(dX, dZ, q, flags=zx.ZX_PAULI_FORCE_VALU)
    C2 = zx.pauli_commute(dX, dZ, q, flags=zx.ZX_PAULI_FORCE_MFMA)
    torch.cuda.synchronize()
    assert torch.equal(C1, C2)


@pytest.mark.parametrize("variant", VARIANTS)
def test_full_size_sampled_rows(zx, variant):
    """65536 strings on 1024 qubits (seed 22): rows from several tiles,
    including the first, the last and rows straddling tile borders."""
    import torch
    n, q = 65536, 1024
    X, Z = pauli_strings(22, n, q)
    Cg = zx.pauli_commute(zx.to_device_words(X), zx.to_device_words(Z), q, flags=_flags(zx, variant))
    torch.cuda.synchronize()
    rows = [0, 1, 63, 64, 65, 255, 256, 4095, 30000, 32767, 32768, 65471, 65472, 65535]
    Ch = Cg.cpu()
    for r in rows:
        Co = oracle.pauli_commute(X, Z, rows=(r, r + 1))
        assert np.array_equal(Ch[r].numpy().view(np.uint64), Co[0]), r
    # symmetry and zero diagonal on a sampled block
    blk = Ch[:256, :4].numpy().view(np.uint64)
    bits = np.unpackbits(blk.view(np.uint8), axis=1, bitorder="little")[:, :256]
    assert np.array_equal(bits, bits.T)
    assert not bits.diagonal().any()


@pytest.mark.parametrize("n,q", [(16500, 130), (16384, 64), (5000, 257), (2049, 1000)])
def test_tile_orders(zx, n, q):
    """The matrix-core table in bands of four rows of tiles (from 64 rows of
    tiles up, the last band short) and row by row, against the vector-unit
    table."""
    import torch
    print("pauli tile order case", n, q, flush=True)
    X, Z = pauli_strings(300 + q, n, q)
    dX, dZ = zx.to_device_words(X), zx.to_device_words(Z)
    C1 = zx.pauli_commute(dX, dZ, q, flags=zx.ZX_PAULI_FORCE_VALU)
    C2 = zx.pauli_commute(dX, dZ, q, flags=zx.ZX_PAULI_FORCE_MFMA)
    torch.cuda.synchronize()
    assert torch.equal(C1, C2)


@pytest.mark.parametrize("n,q", [(5, (1 << 22) + 3), (3, (1 << 23) + 64), (200, (1 << 21) + 5)])
def test_long_strings(zx, n, q):
    """Strings whose counts (up to 2 q) leave the exact range of the fp32
    accumulators: both variants and the default, Y on every qubit (the largest counts) and X
    on every qubit among them."""
    import torch
    rng = np.random.default_rng(n)
    qw = (q + 63) // 64
    X = rng.integers(0, 2 ** 64, (n, qw), dtype=np.uint64)
    Z = rng.integers(0, 2 ** 64, (n, qw), dtype=np.uint64)
    full, last = np.uint64(2 ** 64 - 1), np.uint64((1 << (q % 64 or 64)) - 1)
    X[0] = Z[0] = X[1] = Z[1] = X[2] = full
    Z[2] = 0
    Z[1, 0] -= np.uint64(1)  # an odd count
    X[:, -1] &= last
    Z[:, -1] &= last
    want = np.zeros((n, (n + 63) // 64), np.uint64)
    pick = range(n) if n < 10 else (0, 1, 2, 64, 130, n - 1)
    for i in pick:
        for j in range(n):
            bit = int(np.bitwise_count(np.bitwise_xor.reduce((X[i] & Z[j]) ^ (Z[i] & X[j])))) & 1
            want[i, j // 64] |= np.uint64(bit << (j % 64))
    for variant in VARIANTS + ["auto"]:
        print("pauli long case", n, q, variant, flush=True)
        flags = zx.ZX_PAULI_AUTO if variant == "auto" else _flags(zx, variant)
        C = zx.pauli_commute(zx.to_device_words(X), zx.to_device_words(Z), q, flags=flags)
        torch.cuda.synchronize()
        Ch = zx.to_host_words(C)
        for i in pick:
            assert np.array_equal(Ch[i], want[i]), (variant, i)
        assert np.array_equal(np.stack([(Ch[:, j // 64] >> np.uint64(j % 64)) & np.uint64(1) for j in pick]),
                              np.stack([[(int(Ch[j, i // 64]) >> (i % 64)) & 1 for i in range(n)] for j in pick]))
