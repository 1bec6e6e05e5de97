"""Scoring a graph of more than 2^24 nodes (Section II-B; Eqs. (8), (9)): tiles with the larger
slices, staged by rows, and labels put in place in LDS by super-buckets of 65,536 ids.  The label
move takes that path when the workspace's staged labels (2 bytes an entry) hold 8 bytes an id of
all super-buckets, so from five entries a node on; fewer take the bucket plan."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import check_per_community, check_score, note
from tests.test_gpu_paths import cq, ctx  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def graph(n, dists, hub, empty):
    """Nodes joined to those `dists` further on (around the first n - empty), a hub, empty rows."""
    k = n - empty
    u = torch.arange(k, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    a = [u] * len(dists) + [torch.full((hub,), 7, device="cuda")]
    b = [(u + d) % k for d in dists] + [100 + torch.randperm(k - 100, generator=g, device="cuda")[:hub]]
    a, b = torch.cat(a), torch.cat(b)
    key = torch.unique(torch.cat([a * n + b, b * n + a]))
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.bincount(key // n, minlength=n).cumsum(0)
    return rp.to(torch.int32), (key % n).to(torch.int32)


@pytest.mark.parametrize("dists", [(1, 331, 5000011), (1, 5000011)])
def test_beyond_2_24_nodes(cq, ctx, dists):  # noqa: F811
    n, L = (1 << 24) + 70001, 20011  # the last super-bucket and the last group of 8 ids are partly filled
    rp, ci = graph(n, dists, 100000, 5000)
    buckets = (n + 65535) // 65536
    fits = 2 * ci.numel() >= 8 * buckets * 65536 + 4096
    assert fits == (len(dists) == 3) and buckets >= torch.cuda.get_device_properties(0).multi_processor_count
    u = torch.arange(n, device="cuda")
    lab = ((u // 613 * 7) % L).to(torch.int32)
    lab[::11] = (lab[::11] + 5) % L
    note(f"{n} nodes, {ci.numel()} entries")
    o = oracle.score(rp.cpu().numpy(), ci.cpu().numpy(), lab.cpu().numpy(), L, want_pairs=False)
    g = cq.Graph(ctx, rp, ci, reorder=True)
    assert g.stats["reordered"] == cq.CQ_GRAPH_REORDER | cq.CQ_GRAPH_NO_BLOCKS
    for _ in range(2):
        r, pc, _ = cq.score_partition(g, lab, L, per_community=True)
        check_score(r, o.result)
        check_per_community(pc, o, int(o.result["m"]))
    for at in (0, n - 1):
        bad = lab.clone()
        bad[at] = L
        with pytest.raises(cq.CQError) as e:
            cq.score_partition(g, bad, L)
        assert e.value.status == cq.CQ_E_LABEL_RANGE
    g.close()
