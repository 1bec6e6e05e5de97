"""Scoring tiled graphs with the least workspace that a call takes (Section II-B; Eqs. (8), (9)):
without room for all far labels small graphs are scored by member rows, and on others the far
labels take turns, staged as with that room."""
import numpy as np
import pytest
import torch

import oracle
from cqgen import edge_weights
from tests.gpu_util import check_per_community, check_score, note, sort_rows, table_equal
from tests.test_gpu_tiles import GRAPHS, cq, ctx, near_far_graph  # noqa: F401  (fixtures)
from tests.test_gpu_weighted import check_weighted, open_weighted

pytestmark = pytest.mark.gpu


def least_workspace(cq, G, lab, width):  # noqa: F811
    """A workspace of the smallest accepted size (one byte less is refused)."""
    hi = G.workspace_size(width)
    ws = torch.empty(hi, dtype=torch.uint8, device="cuda")
    lo = 0
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            cq.score_partition(G, lab, width, workspace=ws[:mid])
            hi = mid
        except cq.CQError as e:
            assert e.status == cq.CQ_E_WORKSPACE
            lo = mid
    return ws[:hi]


@pytest.mark.parametrize("name", ["n32767", "n32768", "n32769", "dense", "far", "hub", "sparse"])
@pytest.mark.parametrize("width", [60, 12000, 20000, 70000])
def test_least_workspace(cq, ctx, name, width):  # noqa: F811
    """60 label ids: member rows.  More: the far labels in turns (16- and 32-bit labels, one chunk
    and several)."""
    n = GRAPHS[name][0]
    rp, ci = near_far_graph(n, 8, *GRAPHS[name][1:])
    lab_h = ((np.arange(n) // 97 * 31) % width).astype(np.int32)
    G = cq.Graph(ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), reorder=True, blocks=True)
    lab = torch.as_tensor(lab_h).cuda()
    o = oracle.score(rp, ci, lab_h, width)
    cap = max(1, int(o.result["num_pairs"]))
    ws = least_workspace(cq, G, lab, width)
    assert name == "sparse" or ws.numel() < G.workspace_size(width)
    for frac in (2.0, -1.0):
        note(f"{name}, {width} ids, {ws.numel()} bytes, row staging from {frac}")
        cq.cq_context_set_row_staging(ctx.handle, frac)
        try:
            want, _, _ = cq.score_partition(G, lab, width)
            staging = G.last_staging
            r, pc, pt = cq.score_partition(G, lab, width, workspace=ws, per_community=True, pairs_capacity=cap)
            if width > 60 and name != "sparse":
                assert G.last_staging == staging != 0
            bad = lab.clone()
            bad[n // 2] = width
            with pytest.raises(cq.CQError) as e:
                cq.score_partition(G, bad, width, workspace=ws)
            assert e.value.status == cq.CQ_E_LABEL_RANGE
        finally:
            cq.cq_context_set_row_staging(ctx.handle, 1 / 16)
        assert r == want
        check_score(r, o.result, name)
        check_per_community(pc, o, int(o.result["m"]))
        assert table_equal(pt, o.pairs, width)
    G.close()


@pytest.mark.parametrize("name", ["n32769", "far", "hub"])
@pytest.mark.parametrize("width", [7, 20000])
def test_least_workspace_weighted(cq, ctx, name, width):  # noqa: F811
    n = GRAPHS[name][0]
    rp, ci = near_far_graph(n, 9, *GRAPHS[name][1:])
    w = edge_weights(rp, ci, seed=4).numpy()
    lab_h = ((np.arange(n) // 23 * 31) % width).astype(np.int32)
    lab = torch.as_tensor(lab_h).cuda()
    note(f"weighted {name}, {width} ids")
    o = oracle.score_w(rp, ci, w, lab_h, width)
    g = open_weighted(cq, ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), torch.as_tensor(w).cuda(), "blocked")
    ws = least_workspace(cq, g, lab, width)
    assert ws.numel() < g.workspace_size(width)
    r, _, pt = cq.score_partition(g, lab, width, workspace=ws, pairs_capacity=max(1, int(o.result["num_pairs"])))
    assert g.last_staging == 1
    check_weighted(r, o, f"{name} weighted")
    assert np.array_equal(sort_rows(pt), o.pairs)
    g.close()
