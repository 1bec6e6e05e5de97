"""Scoring by member rows where one community or one row holds much of the graph (Section II-B):
communities are cut into parts from two node chunks on (chunks of 1,024 nodes up to 2^18 nodes),
parts hold half a chunk, and rows of 4,096 entries are walked by a whole workgroup.  Integers
and pair tables match the oracle bit for bit."""
import time

import numpy as np
import pytest
import torch

from cqgen.smallgraphs import csr_from_edges
from tests.test_gpu_paths import cq, ctx, run_score  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def labels_of(n, sizes, L, seed):
    """Random node order: communities of the given sizes, the other nodes spread over the rest."""
    lab = np.repeat(np.arange(len(sizes)), sizes)
    rest = len(sizes) + np.arange(n - len(lab)) % (L - len(sizes)) if n > len(lab) else np.zeros(0, int)
    return np.random.default_rng(seed).permutation(np.concatenate([lab, rest])).astype(np.int32)


@pytest.mark.parametrize("n,sizes,L", [
    (20000, [20000], 1),  # one community: 40 parts, the last one short
    (17000, [8500, 8500], 2),
    # one node less than the cut, the cut, one more; whole parts and one more node
    (20000, [2047, 2048, 2049, 2560, 2561, 6000], 170),
    (20000, [2047, 2048, 2049, 2560, 2561, 6000], 9001),
    (40000, [30000], 16384),
    # chunks of 2,048 nodes
    ((1 << 18) + 3, [4095, 4096, 4097, 100000], 1000),
])
def test_large_communities(cq, ctx, n, sizes, L):  # noqa: F811
    rng = np.random.default_rng(n)
    rp, ci = csr_from_edges(n, rng.integers(0, n, (4 * n, 2)))
    run_score(cq, ctx, rp, ci, labels_of(n, sizes, L, L), L, f"{n} nodes, communities of {sizes}, {L} ids")


@pytest.mark.parametrize("degrees,sizes", [
    ([4095, 4096, 4097, 12288, 16999], [500]),
    ([4096] * 70, [3000]),  # more hubs in a part than it lists
])
def test_hub_rows(cq, ctx, degrees, sizes):  # noqa: F811
    """Hubs (the first nodes, all in community 0) joined to that many nodes each."""
    n, L = 17000, 170
    rng = np.random.default_rng(len(degrees))
    k = len(degrees)
    lab = labels_of(n, sizes, L, 1)
    at = np.flatnonzero(lab == 0)[:k]
    lab[at], lab[:k] = lab[:k].copy(), 0
    # the hubs' other ends lie past the hubs, so the degrees are exact (but for node k itself)
    e = [np.stack([np.full(d, h), k + rng.choice(n - k, min(d, n - k), replace=False)], axis=1) for h, d in enumerate(degrees)
         if d <= n - k]
    e += [np.stack([np.full(n - k, h), np.arange(k, n)], axis=1) for h, d in enumerate(degrees) if d > n - k]
    rp, ci = csr_from_edges(n, np.concatenate(e + [k + rng.integers(0, n - k, (2 * n, 2))]))
    assert (np.diff(rp)[:k] == np.minimum(degrees, n - k)).all()
    run_score(cq, ctx, rp, ci, lab, L, f"hubs of {degrees[:5]}")


def test_cost_of_one_community(cq, ctx):  # noqa: F811
    """The chip shares a community: 400,000 nodes in one community cost about what they cost in
    1,000 (33 times as much when one workgroup walked all rows)."""
    n = 400_000
    u = torch.arange(n, device="cuda")
    ds = [d * s for d in (1, 7, 113, 1009, 10007, 50021, 100003, 150001) for s in (1, -1)]
    ci = torch.sort(torch.stack([(u + d) % n for d in ds], dim=1), dim=1).values.reshape(-1).to(torch.int32)
    g = cq.Graph(ctx, (16 * torch.arange(n + 1, device="cuda")).to(torch.int32), ci)

    def cost(L):
        lab = (u * L // n).to(torch.int32)
        best = np.inf
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            cq.score_partition(g, lab, L)
            best = min(best, time.perf_counter() - t)
        return best

    many, one = cost(1000), cost(1)
    print(f"1,000 communities {1e6 * many:.0f} us, one {1e6 * one:.0f} us", flush=True)
    assert one < 5 * many
    g.close()
