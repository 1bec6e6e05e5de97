"""GPU parity of the tiled edge pass (Section II-B; Eqs. (8), (9)) at the edges of its tiles:
blocks of 1,024 rows, windows of 8,192 ids, tiles of 24,576 entries, slices of 2^15 ids (2^16
beyond 2^24 nodes).  Integers and pair tables match the oracle bit for bit; weighted sums and
measures within the tolerance of gpu_util."""
import numpy as np
import pytest
import torch

import oracle
from cqgen import edge_weights
from cqgen.smallgraphs import csr_from_edges
from tests.gpu_util import check_per_community, check_score, note, sort_rows, table_equal
from tests.test_gpu_weighted import check_weighted, open_weighted

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


def near_far_graph(n, seed, near, far, hub=0, empty=0):
    """`near` edges to an id within 50, `far` edges to any id, a hub joined to `hub` nodes, and
    the last `empty` nodes without an edge."""
    rng = np.random.default_rng(seed)
    k = n - empty
    u = rng.integers(0, k, near)
    e = [np.stack([u, np.clip(u + rng.integers(-50, 51, near), 0, k - 1)], axis=1), rng.integers(0, k, (far, 2))]
    if hub:
        e.append(np.stack([np.full(hub, k // 2), rng.choice(k, hub, replace=False)], axis=1))
    return csr_from_edges(n, np.concatenate(e + [[[0, 1]]]))


GRAPHS = {
    # rows of the last block: one less than full, full, one more
    "n1023": (1023, 4000, 1000), "n1024": (1024, 4000, 1000), "n1025": (1025, 4000, 1000),
    # one slice less an id, whole, one more; far entries on both sides of the window
    "n32767": (32767, 150000, 60000), "n32768": (32768, 150000, 60000), "n32769": (32769, 150000, 60000),
    # blocks of more than 24,576 entries (several tiles), and of more than 16,384 far ones each
    "dense": (12000, 100000, 250000), "far": (60000, 100, 900000),
    # a row of more than a tile's entries, and rows without entries
    "hub": (60000, 100000, 20000, 50000, 3000),
    "sparse": (20000, 300, 50, 0, 9000),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("width", [1, 60, 70000])
def test_tiles(cq, ctx, name, width):
    """Runs of labels along the ids, random ones, and (70,000 label ids) 32-bit labels, staged
    by runs and by rows."""
    n = GRAPHS[name][0]
    rp, ci = near_far_graph(n, 5, *GRAPHS[name][1:])
    rng = np.random.default_rng(width)
    runs = (np.arange(n) // 97 * 31) % width
    G = cq.Graph(ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), reorder=True, blocks=True)
    assert G.stats["reordered"] == cq.CQ_GRAPH_REORDER
    for what, lab in (("runs", runs), ("random", rng.integers(0, width, n))):
        lab = lab.astype(np.int32)
        o = oracle.score(rp, ci, lab, width)
        cap = max(1, int(o.result["num_pairs"]))
        for frac in (2.0, -1.0):
            note(f"tiles: {name}, {width} ids, {what}, row staging from {frac}")
            cq.cq_context_set_row_staging(ctx.handle, frac)
            try:
                r, pc, pt = cq.score_partition(G, torch.as_tensor(lab).cuda(), width, per_community=True, pairs_capacity=cap)
            finally:
                cq.cq_context_set_row_staging(ctx.handle, 1 / 16)
            check_score(r, o.result, f"{name} {what}")
            check_per_community(pc, o, int(o.result["m"]))
            assert table_equal(pt, o.pairs, width), (name, what)
    bad = runs.astype(np.int32)
    bad[n // 2] = width
    with pytest.raises(cq.CQError) as e:
        cq.score_partition(G, torch.as_tensor(bad).cuda(), width)
    assert e.value.status == cq.CQ_E_LABEL_RANGE
    G.close()


@pytest.mark.parametrize("name", ["n1025", "n32769", "dense", "far", "hub", "sparse"])
@pytest.mark.parametrize("width", [7, 9000])
def test_tiles_weighted(cq, ctx, name, width):
    n = GRAPHS[name][0]
    rp, ci = near_far_graph(n, 6, *GRAPHS[name][1:])
    w = edge_weights(rp, ci, seed=3).numpy()
    lab = ((np.arange(n) // 23 * 31) % width).astype(np.int32)
    note(f"weighted tiles: {name}, {width} ids")
    o = oracle.score_w(rp, ci, w, lab, width)
    g = open_weighted(cq, ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), torch.as_tensor(w).cuda(), "blocked")
    r, _, pt = cq.score_partition(g, torch.as_tensor(lab).cuda(), width, pairs_capacity=max(1, int(o.result["num_pairs"])))
    check_weighted(r, o, f"{name} weighted")
    assert np.array_equal(sort_rows(pt), o.pairs)
    g.close()


def test_tiles_beyond_2_24_nodes(cq, ctx):
    """17M nodes with four neighbours each: larger slices, label moves through LDS, staging by
    rows.  The result has the bits of the input storage's, whatever the storage."""
    n, L = (1 << 24) + 70001, 20011
    u = torch.arange(n, device="cuda")
    ci = torch.stack([(u + d) % n for d in (1, -1, 5000011, -5000011)], dim=1)
    ci = torch.sort(ci, dim=1).values.reshape(-1).to(torch.int32)
    rp = (4 * torch.arange(n + 1, device="cuda")).to(torch.int32)
    lab = ((u // 613 * 7) % L).to(torch.int32)
    lab[::11] = (lab[::11] + 5) % L
    results = []
    for reorder in (False, True):
        note(f"17M nodes, reorder={reorder}")
        g = cq.Graph(ctx, rp, ci, reorder=reorder)
        results.append(cq.score_partition(g, lab, L)[0])
        g.close()
    assert results[0] == results[1]
    c = lab.long()
    own = sum(int((c == c.roll(-d)).sum()) for d in (1, -1, 5000011, -5000011))
    assert results[0]["sum_ein"] == own // 2


def test_workspace_without_room_for_far_labels(cq, ctx):
    """A workspace that lacks room for the far entries' labels alone is scored through the
    row-major copy, to the same bits; a smaller one is refused."""
    n, L = 40000, 300
    rp, ci = near_far_graph(n, 7, 150000, 60000)
    lab = torch.as_tensor((np.arange(n) // 97 * 31 % L).astype(np.int32)).cuda()
    G = cq.Graph(ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), reorder=True, blocks=True)
    full = G.workspace_size(L)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    want, _, _ = cq.score_partition(G, lab, L, workspace=ws)

    def accepted(size):
        try:
            r, _, _ = cq.score_partition(G, lab, L, workspace=ws[:size])
        except cq.CQError as e:
            assert e.status == cq.CQ_E_WORKSPACE
            return False
        assert r == want, size
        return True

    lo, hi = 0, full  # refused, accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        note(f"workspace of {mid} bytes")
        lo, hi = (lo, mid) if accepted(mid) else (mid, hi)
    assert hi < full and not accepted(hi - 1) and accepted(full - 1)
    G.close()
