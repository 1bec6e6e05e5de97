"""Which path a call of a given size takes (told by the stages that it times), and parity on both
sides of the line (Section II-A, II-B)."""
import numpy as np
import pytest
import torch

from cqgen.smallgraphs import csr_from_edges
from tests.test_gpu_paths import cq, ctx, run_score  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def stages_of(cq, ctx, call):  # noqa: F811
    cq.cq_context_enable_timing(ctx.handle, True)
    before = cq.cq_context_stage_times(ctx.handle)
    call()
    after = cq.cq_context_stage_times(ctx.handle)
    cq.cq_context_enable_timing(ctx.handle, False)
    return {k for k, v in after.items() if v[1] > before.get(k, (0, 0))[1]}


def route(cq, ctx, rp, ci, lab, L):  # noqa: F811
    g = cq.Graph(ctx, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda())
    t = torch.as_tensor(lab).cuda()
    st = stages_of(cq, ctx, lambda: cq.score_partition(g, t, L))
    g.close()
    return "staged" if "edge_gather" in st else "rows" if "group_count" in st else "small"


@pytest.mark.parametrize("n,m,L,path", [
    (20000, 50000, 12000, "staged"),  # communities of one or two nodes under a wide table
    (20000, 50000, 16384, "staged"),
    (20000, 50000, 8192, "rows"),
    (60000, 600000, 8193, "staged"),  # 146 entries a community
    (60000, 700000, 8193, "rows"),    # 170
])
def test_tiny_communities(cq, ctx, n, m, L, path):  # noqa: F811
    rng = np.random.default_rng(m)
    rp, ci = csr_from_edges(n, rng.integers(0, n, (m, 2)))
    lab = rng.integers(0, L, n).astype(np.int32)
    run_score(cq, ctx, rp, ci, lab, L, f"{n} nodes, {m} edges, {L} ids")
    assert route(cq, ctx, rp, ci, lab, L) == path


@pytest.mark.parametrize("n,m,L,path", [
    (1000, 7000, 48, "small"), (1000, 7000, 49, "rows"),
    (16384, 190000, 48, "small"), (16384, 190000, 49, "rows"), (16384, 190000, 160, "rows"),
    (16385, 190000, 48, "rows"), (16000, 210000, 48, "rows"),  # a node, or 20,000 entries, too many
])
def test_small_graphs(cq, ctx, n, m, L, path):  # noqa: F811
    rng = np.random.default_rng(m)
    rp, ci = csr_from_edges(n, rng.integers(0, n, (m, 2)))
    lab = rng.integers(0, L, n).astype(np.int32)
    run_score(cq, ctx, rp, ci, lab, L, f"{n} nodes, {m} edges, {L} ids")
    assert route(cq, ctx, rp, ci, lab, L) == path
