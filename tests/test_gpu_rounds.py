"""Round updates with the adjacency in LDS against the oracle: row widths on
both sides of the table threshold, diagrams that leave no room for the
tables, rounds of more than 8 and of more than 64 rewrites, rounds of pivots
only, through the variants whose LDS budgets put the same diagram in LDS or
in the arena."""
import numpy as np
import pytest

import oracle
from workloads import make_diagram
from workloads.generators import Diagram

pytestmark = pytest.mark.gpu

# (spiders, qubits, density): 128/129 words edge, 6/7 words (tables from 7),
# 1060..1088 spiders fill the 152 KiB budget up to the last table's place,
# sparse ones have rounds of many rewrites
SIZES = [(65, 4, 0.2), (129, 6, 0.02), (384, 8, 0.3), (385, 8, 0.3), (447, 9, 0.004), (700, 12, 0.005),
         (1024, 16, 0.1), (1060, 16, 0.2), (1075, 16, 0.2), (1088, 16, 0.3)]


def diagram(seed, n, q, p, pauli):
    d = make_diagram(seed, n, q, n, p)
    if pauli:  # every phase 0 or pi: the first round is a pivot round
        d = Diagram(n=n, adj=d.adj, phase=(d.phase & 4).astype(np.int8), inputs=d.inputs, outputs=d.outputs,
                    bnd_is_h=d.bnd_is_h)
    return d


@pytest.mark.parametrize("pauli", [False, True])
@pytest.mark.parametrize("n,q,p", SIZES)
def test_round_updates(zx, n, q, p, pauli):
    d = diagram(71, n, q, p, pauli)
    og = oracle.Graph.from_diagram(d)
    assert og.simplify() == oracle.OK
    M, fp, rank, ops = og.frontier()
    names = zx.simplify_variants()
    for v, name in enumerate(names):
        if name.startswith("bs64") and n > 400:
            continue  # one wavefront: minutes of rounds add nothing
        g = zx.Graph.from_diagram(d)
        print("round updates", n, p, pauli, name, flush=True)
        try:
            zx.simplify([g], tune_id=v)
        except zx.ZxError as e:
            assert e.code == zx.ZX_ECAPACITY
            continue
        adj, ph, al, info = g.read()
        assert info.status == 0
        assert np.array_equal(al, og.alive) and np.array_equal(ph, og.k) and np.array_equal(adj, og.adj), name
        assert info.pow_sqrt2 == og.scalar.pow_sqrt2 and info.phase8 == og.scalar.phase8 % 8
        assert info.fill_in == og.scalar.fill_in and info.rank == rank and info.rowops == ops
        np.testing.assert_array_equal(g.trace(), og.trace)
        assert np.array_equal(g.frontier()[0], M)


@pytest.mark.parametrize("count,q_hi", [(1, 64), (257, 24), (1200, 64), (900, 72)])
def test_by_size_equals_one_variant(zx, count, q_hi):
    """Uneven batches in one to three launches by size (the default, its own
    variant) leave every arena as one 64 KiB launch for all does."""
    import torch
    from workloads import batch_diagram
    ds = [batch_diagram(81, i, q_hi=q_hi) for i in range(count)]
    arenas = []
    by_size = zx.simplify_variants().index("by-size")
    for tune in (-1, by_size, zx.simplify_variants().index("bs512-lds64k")):
        sizes = [(zx.Graph.bytes_for(d.n, d.qubits, d.qubits) + 255) // 256 * 256 for d in ds]
        pool = torch.zeros(sum(sizes), dtype=torch.uint8, device="cuda")
        offs = np.concatenate([[0], np.cumsum(sizes)])
        gs = [zx.Graph.from_diagram(d, arena=pool[offs[i]:offs[i + 1]]) for i, d in enumerate(ds)]
        print("by size", count, q_hi, tune, flush=True)
        b = zx.Batch(gs)
        b.run(tune_id=tune)
        b.run(tune_id=tune)
        assert b.status() == zx.ZX_OK
        arenas.append(pool)
    assert torch.equal(arenas[0], arenas[2]) and torch.equal(arenas[1], arenas[2])


@pytest.mark.parametrize("n,q,p", [(1153, 8, 0.002), (1280, 16, 0.1), (1409, 22, 0.003), (1472, 23, 0.02)])
@pytest.mark.parametrize("pauli", [False, True])
def test_arena_updates(zx, n, q, p, pauli):
    """Rows that no LDS budget holds, of odd and even numbers of words, with
    contribution tables of two and of four groups and one and several passes."""
    d = diagram(72, n, q, p, pauli)
    og = oracle.Graph.from_diagram(d)
    assert og.simplify() == oracle.OK
    for name in ("bs256-lds32k", "bs512-lds152k"):
        print("arena updates", n, p, pauli, name, flush=True)
        g = zx.Graph.from_diagram(d)
        zx.simplify([g], tune_id=zx.simplify_variants().index(name))
        adj, ph, al, info = g.read()
        assert np.array_equal(al, og.alive) and np.array_equal(ph, og.k) and np.array_equal(adj, og.adj), name
        assert info.fill_in == og.scalar.fill_in and info.phase8 == og.scalar.phase8 % 8
        np.testing.assert_array_equal(g.trace(), og.trace)


def test_many_large_diagrams(zx):
    """More large diagrams than a CU holds workgroups for, of a size whose
    auxiliary arrays exceed the smallest LDS budget: the default plan runs
    every one (a budget they do not fit leaves them as they were)."""
    import torch
    n, count = 4700, 800
    d = make_diagram(83, n, 4, n, 0.0008)
    one = zx.Graph.from_diagram(d)
    pool = one.arena[None, :].repeat(count, 1)
    gs = [zx.Graph.attach(pool[i]) for i in range(count)]
    print("many large", n, count, flush=True)
    zx.simplify([one], tune_id=zx.simplify_variants().index("bs512-lds152k"), max_rounds=3, extract=False)
    assert one.info().n_trace > 0
    b = zx.Batch(gs)
    b.run(max_rounds=3, extract=False)
    assert b.status() == zx.ZX_OK
    assert bool((pool == one.arena[None, :]).all())


@pytest.mark.parametrize("n,q,p", [(2048, 8, 0.003), (2049, 8, 0.05), (2177, 16, 0.0015), (3009, 8, 0.001)])
@pytest.mark.parametrize("pauli", [False, True])
def test_arena_updates_of_wide_rows(zx, n, q, p, pauli):
    """Rows on both sides of 32 words, beyond which rows without a hit are not
    written: sparse rounds of one and of several passes of tables, in which
    most rows have none, and dense ones."""
    d = diagram(73, n, q, p, pauli)
    og = oracle.Graph.from_diagram(d)
    assert og.simplify() == oracle.OK
    for name in ("bs256-lds32k", "bs512-lds64k", "bs512-lds152k"):
        print("arena wide", n, p, pauli, name, flush=True)
        g = [zx.Graph.from_diagram(d)]
        g += [g[0].snapshot() for _ in range(11)]  # so many that no team takes them
        zx.simplify(g, tune_id=zx.simplify_variants().index(name))
        for x in (g[0], g[11]):
            adj, ph, al, info = x.read()
            assert np.array_equal(al, og.alive) and np.array_equal(ph, og.k) and np.array_equal(adj, og.adj), name
            assert info.fill_in == og.scalar.fill_in and info.phase8 == og.scalar.phase8 % 8
            np.testing.assert_array_equal(x.trace(), og.trace)
