"""GPU parity at the edges of the scoring and comparison paths that are chosen by size:
small inputs in one or two launches, member rows, staged segments (Section II-A, II-B).
Integers, pair tables and contingency tables match the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from cqgen.smallgraphs import csr_from_edges
from tests.gpu_util import check_compare, check_per_community, check_score, note, sort_rows, table_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cq():
    from paper_1507_05492_amd import cq as mod

    return mod


@pytest.fixture(scope="module")
def ctx(cq):
    c = cq.Context(0)
    yield c
    c.close()


def hub_graph(n, m, seed, hubs=2):
    """m random edges, two hubs joined to every eighth node, every sixteenth node isolated."""
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n, (m, 2))
    if n > 64:
        star = [np.stack([np.full(len(range(h, n, 8)), h), np.arange(h, n, 8)], axis=1) for h in range(1, 1 + hubs)]
        e = np.concatenate([e] + star)
        e = e[(e % 16 != 15).all(axis=1)]
    return csr_from_edges(n, np.concatenate([e, [[0, 1]]]))  # never without an edge


def run_score(cq, ctx, rp, ci, lab, L, what, reorder=False):
    note(what)
    o = oracle.score(rp, ci, lab, L)
    G = cq.Graph(ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), reorder=reorder)
    cap = max(1, int(o.result["num_pairs"]))
    r, pc, pt = cq.score_partition(G, torch.as_tensor(lab).cuda(), L, per_community=True, pairs_capacity=cap)
    check_score(r, o.result, what)
    check_per_community(pc, o, int(o.result["m"]))
    assert table_equal(pt, o.pairs, L), what
    r2, _, _ = cq.score_partition(G, torch.as_tensor(lab).cuda(), L)
    assert r2 == r, f"{what}: a second call differs"
    if cap > 1:
        r3, _, _ = cq.score_partition(G, torch.as_tensor(lab).cuda(), L, pairs_capacity=cap - 1, allow=(cq.CQ_E_CAPACITY,))
        assert r3["status"] == cq.CQ_E_CAPACITY and r3["num_pairs"] == r["num_pairs"] and r3["Q"] == r["Q"], what
    bad = lab.copy()
    bad[len(bad) // 2] = L
    with pytest.raises(cq.CQError) as e:
        cq.score_partition(G, torch.as_tensor(bad).cuda(), L)
    assert e.value.status == cq.CQ_E_LABEL_RANGE, what
    G.close()
    return r


# 160 and 161 label ids, 16,384 and 16,385 nodes and 400,000 entries part the two-launch path
# from member rows; 512, 1,024, 4,096 and 16,384 ids their workgroup sizes; 16,385 ids and
# 2^21 nodes member rows from staged segments
@pytest.mark.parametrize("n,m,L", [
    (2, 1, 1), (3, 2, 160), (1_000, 7_000, 20), (16_384, 60_000, 160), (16_384, 60_000, 161), (16_385, 60_000, 160),
    (9_000, 196_000, 100), (9_000, 240_000, 100), (700, 3_000, 3), (20_000, 100_000, 1), (30_000, 100_000, 512),
    (30_000, 100_000, 1_025), (60_000, 200_000, 2_049), (60_000, 200_000, 4_096), (60_000, 200_000, 4_097),
    (100_000, 300_000, 16_384), (100_000, 300_000, 16_385), (5_000, 100, 3_000),
])
def test_score_size_edges(cq, ctx, n, m, L):
    rp, ci = hub_graph(n, m, n + m + L)
    rng = np.random.default_rng(L)
    near = (np.arange(n) * L // n).astype(np.int32)  # stored by community
    lab = np.where(rng.random(n) < 0.3, rng.integers(0, L, n), near).astype(np.int32)
    a = run_score(cq, ctx, rp, ci, lab, L, f"n={n} m={m} L={L}")
    assert run_score(cq, ctx, rp, ci, lab, L, f"n={n} m={m} L={L}, renumbered", reorder=True) == a


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1])
def test_score_rows_node_limit(cq, ctx, n):
    rp, ci = hub_graph(n, 2 * n, 7)
    lab = np.random.default_rng(3).integers(0, 700, n).astype(np.int32)
    run_score(cq, ctx, rp, ci, lab, 700, f"n={n}")


# one-launch comparison: 28,672 cells, 1,024 ids per side and 32,768 nodes are its limits
@pytest.mark.parametrize("n,La,Lb", [
    (2, 1, 1), (1_000, 22, 22), (32_768, 169, 169), (32_769, 169, 169), (5_000, 1_024, 28), (5_000, 28, 1_024),
    (5_000, 1_025, 3), (5_000, 169, 170), (8_193, 1, 1_024), (63, 64, 65),
])
@pytest.mark.parametrize("kind", ["close", "random"])
def test_compare_size_edges(cq, ctx, n, La, Lb, kind):
    rng = np.random.default_rng(n + La)
    a = np.sort(rng.integers(0, La, n)).astype(np.int32)
    b = (np.where(rng.random(n) < 0.2, rng.integers(0, Lb, n), a % Lb) if kind == "close" else rng.integers(0, Lb, n)).astype(np.int32)
    what = f"compare n={n} La={La} Lb={Lb} {kind}"
    note(what)
    o = oracle.compare(a, La, b, Lb, want_cells=True)
    ta, tb = torch.as_tensor(a).cuda(), torch.as_tensor(b).cuda()
    r, ct = cq.compare_partitions(ctx, ta, La, tb, Lb, cells_capacity=int(o.result["nnz"]))
    check_compare(r, o.result, what)
    assert np.array_equal(sort_rows(ct), o.cells), what
    r2, _ = cq.compare_partitions(ctx, ta, La, tb, Lb)
    assert r2 == r
    for t, L in ((ta, La), (tb, Lb)):
        keep = int(t[n // 2])
        t[n // 2] = L
        with pytest.raises(cq.CQError) as e:
            cq.compare_partitions(ctx, ta, La, tb, Lb)
        assert e.value.status == cq.CQ_E_LABEL_RANGE
        t[n // 2] = keep
