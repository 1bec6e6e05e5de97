"""Comparisons where one community holds much of the nodes (Section II-A), label spaces beyond 16
bits: bins of 65,536 nodes and more are counted by slices of 32,768 nodes and their cells by 2
to 16 workgroups.  Integers and contingency tables match the oracle bit for bit."""
import time

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import check_compare, note, table_equal
from tests.test_gpu_paths import cq, ctx  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def skewed(n, giants, L, seed):
    """Communities of the given sizes first, the other nodes spread over the rest, in random order."""
    lab = np.concatenate([np.repeat(np.arange(len(giants)), giants),
                          len(giants) + np.arange(n - sum(giants)) % (L - len(giants))])
    return np.random.default_rng(seed).permutation(lab).astype(np.int32)


@pytest.mark.parametrize("n,giants,La,Lb", [
    # a node less than a large bin, one, one more; two and four classes
    (200_000, [65_535 - 1], 70_000, 1000), (200_000, [65_536], 70_000, 1000), (200_000, [131_072], 70_000, 1000),
    (400_000, [300_000], 66_000, 20_000),  # more cells than a table: classes split further
    (700_000, [540_000, 3_000], 100_000, 70_000),  # 16 classes; both sides beyond 16 bits
    (300_000, [150_000], 1000, 900),  # 16-bit labels: one workgroup per band
])
@pytest.mark.parametrize("swap", [False, True])
def test_giant_community(cq, ctx, n, giants, La, Lb, swap):  # noqa: F811
    a = skewed(n, giants, La, 1)
    b = np.random.default_rng(2).integers(0, Lb, n).astype(np.int32)
    if swap:
        a, b, La, Lb = b, a, Lb, La
    note(f"{n} nodes, {giants}, {La} x {Lb}")
    o = oracle.compare(a, La, b, Lb)
    ta, tb = torch.as_tensor(a).cuda(), torch.as_tensor(b).cuda()
    r, t = cq.compare_partitions(ctx, ta, La, tb, Lb, cells_capacity=int(o.result["nnz"]))
    check_compare(r, o.result)
    assert table_equal(t, o.cells, Lb)
    assert cq.compare_partitions(ctx, ta, La, tb, Lb)[0] == r
    tb[n // 2] = Lb
    with pytest.raises(cq.CQError) as e:
        cq.compare_partitions(ctx, ta, La, tb, Lb)
    assert e.value.status == cq.CQ_E_LABEL_RANGE


@pytest.mark.parametrize("La", [70_000, 1000])
def test_cost_of_a_giant_community(cq, ctx, La):  # noqa: F811
    """Half of a million nodes in one community against 5,000 unrelated ones cost no more than ten
    times what they cost spread evenly (100 times before)."""
    n, Lb = 1_000_000, 5000
    b = torch.as_tensor(np.random.default_rng(2).integers(0, Lb, n).astype(np.int32)).cuda()

    def cost(giants):
        a = torch.as_tensor(skewed(n, giants, La, 1)).cuda()
        best = np.inf
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            cq.compare_partitions(ctx, a, La, b, Lb)
            best = min(best, time.perf_counter() - t)
        return best

    even, giant = cost([]), cost([n // 2])
    print(f"{La} ground-truth ids: even {1e6 * even:.0f} us, a giant {1e6 * giant:.0f} us", flush=True)
    assert giant < 10 * even
