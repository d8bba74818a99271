"""The sort-based plan path at the edges of its classes of panel size: format and counts equal the
oracle's bit for bit, and invalid columns are refused in every class."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import INT_KEYS, assert_format_equal, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

# the last size of one number of keys a lane and the first of the next; 8192 is the largest
SIZES = (1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192)


def panels_of(sizes, K, seed):
    """A panel of each size; half of its entries in columns that its rows share."""
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    for p, n in enumerate(sizes):
        shared = rng.choice(K, size=max(1, n // 8), replace=False)
        shared[0] = K - 1                                       # the largest key of the panel
        cells = set()
        while len(cells) < n:
            c = int(shared[rng.integers(len(shared))]) if rng.random() < 0.5 else int(rng.integers(K))
            cells.add((16 * p + int(rng.integers(16)), c))
        rows += [r for r, _ in cells]
        cols += [c for _, c in cells]
    return W.csr_from_coo(16 * len(sizes), K, np.asarray(rows), np.asarray(cols),
                          rng.uniform(-1, 1, len(rows)).astype(np.float32))


# 2^19 columns and 2^21 are the first that the 32-bit keys of the largest and the other panels refuse
@pytest.mark.parametrize("K", [(1 << 19) - 1, 1 << 19, (1 << 21) - 1, 1 << 21, 3_000_000])
@pytest.mark.parametrize("sizes", [SIZES, SIZES[:10], SIZES[:14] + (0, 0), (8193, 5), (600,) * 255 + (2100,),
                                   (600,) * 256 + (2100,)],
                         ids=["all", "small", "mid", "beyond", "one_round", "above_a_round"])
def test_class_edges(gpu, K, sizes):  # noqa: F811
    A = panels_of(sizes, K, seed=len(sizes))
    print(f"panel sizes {sizes} K={K}", flush=True)
    plan = make_plan(gpu, A)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    assert_format_equal(gpu.spmm_plan_export(plan), ref)
    got, exp = gpu.spmm_synergy(plan, 8), oracle.synergy(A.M, A.K, 8, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])


@pytest.mark.parametrize("n", [40, 300, 1500, 5000])
@pytest.mark.parametrize("fault", ["swapped", "duplicate", "beyond", "negative"])
def test_invalid_columns_in_every_class(gpu, n, fault):  # noqa: F811
    import torch
    A = panels_of((3, n, 600), 1_500_000, seed=n)
    ci = A.colind.copy()
    lengths = np.diff(A.rowptr[16:33])
    row = 16 + int(np.argmax(lengths >= 2))                     # a row of the middle panel
    at = int(A.rowptr[row])
    assert A.rowptr[row + 1] - at >= 2
    if fault == "swapped":
        ci[at], ci[at + 1] = ci[at + 1], ci[at]
    elif fault == "duplicate":
        ci[at + 1] = ci[at]
    elif fault == "beyond":
        ci[int(A.rowptr[row + 1]) - 1] = A.K
    else:
        ci[at] = -1
    with pytest.raises(gpu.SpmmError) as e:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(ci).cuda(),
                      torch.from_numpy(A.vals).cuda())
    assert e.value.code == gpu.SPMM_EFORMAT


def test_bitmap_beyond_the_default_lds_limit(gpu):  # noqa: F811
    """One panel of more entries than a workgroup sorts, over a span of 700,000 columns."""
    rng = np.random.default_rng(3)
    cols = np.sort(rng.choice(700_000, size=1100, replace=False))
    cols[0], cols[-1] = 0, 699_999
    A = W.csr_from_coo(16, 700_000, np.repeat(np.arange(16), 1100), np.tile(cols, 16),
                       rng.uniform(-1, 1, 16 * 1100).astype(np.float32))
    assert_format_equal(gpu.spmm_plan_export(make_plan(gpu, A)),
                        oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals))


# with 2048 words of bitmap: the last count of bricks with a rank for every word, the first without, the
# last that fits, and the first that the search-based kernels take
@pytest.mark.parametrize("bricks", [11434, 11435, 12031, 12032])
def test_bitmap_build_at_its_limits_of_bricks(gpu, bricks):  # noqa: F811
    rng = np.random.default_rng(bricks)
    cols = rng.choice(65534, size=4 * bricks - 2, replace=False) + 1
    cols = np.concatenate([[0, 65535], cols])                   # the whole span of 2048 words
    again = rng.choice(cols, size=3000, replace=False)          # columns of two rows
    rows = rng.integers(0, 15, size=len(cols))
    A = W.csr_from_coo(16, 65536, np.concatenate([rows, np.full(len(again), 15)]), np.concatenate([cols, again]),
                       rng.uniform(-1, 1, len(cols) + len(again)).astype(np.float32))
    plan = make_plan(gpu, A)
    assert gpu.spmm_plan_sizes(plan)["n_bricks"] == bricks
    assert_format_equal(gpu.spmm_plan_export(plan), oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals))
