"""The first pass over a matrix at the edges of its rounds of 256 entries, of which two are fetched ahead, and of
what it clears on the way: the counts that follow are right for the next matrix in the same memory, too."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import INT_KEYS, assert_format_equal, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = (0, 1, 3, 4, 5, 255, 256, 257, 511, 512, 513, 767, 768, 769, 1024, 1025, 1300)


def band_of(sizes, rows_last=16):
    """A panel of each size within 200 columns of the diagonal; empty rows among them."""
    rng = np.random.default_rng(len(sizes) + rows_last)
    K = 16 * len(sizes) + 200
    r, c = [], []
    for p, n in enumerate(sizes):
        height = rows_last if p == len(sizes) - 1 else 16
        rows = rng.choice(height, size=max(1, height - p % 5), replace=False)
        cells = rng.choice(len(rows) * 200, size=min(n, len(rows) * 200), replace=False)
        r.append(16 * p + rows[cells // 200])
        c.append(16 * p + cells % 200)
    return W.csr_from_coo(16 * (len(sizes) - 1) + rows_last, K, np.concatenate(r), np.concatenate(c),
                          rng.uniform(-1, 1, sum(len(x) for x in r)).astype(np.float32))


def same(gpu, A):  # noqa: F811
    plan = make_plan(gpu, A)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    assert_format_equal(gpu.spmm_plan_export(plan), ref)
    got, exp = gpu.spmm_synergy(plan, 8), oracle.synergy(A.M, A.K, 8, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])


@pytest.mark.parametrize("times", [1, 3, 40])
@pytest.mark.parametrize("rows_last", [1, 5, 16])
def test_rounds(gpu, times, rows_last):  # noqa: F811
    A = band_of(SIZES * times, rows_last)
    same(gpu, A)
    same(gpu, band_of(SIZES[::-1] * times, rows_last))      # in memory that the plan before let go


@pytest.mark.parametrize("K", [100, 70_000, 5_000_000])     # the last: too much to clear for one workgroup
def test_few_rows_of_many_columns(gpu, K):  # noqa: F811
    for seed in (1, 2):
        same(gpu, W.uniform_random(20, K, min(0.5, 300 / K), seed))


@pytest.mark.parametrize("size", [200, 300, 700])
@pytest.mark.parametrize("fault", ["swapped", "duplicate", "beyond", "negative", "rowptr back", "rowptr end"])
def test_faults_in_every_round(gpu, size, fault):  # noqa: F811
    import torch
    A = band_of((20, size, 20))
    rp, ci = A.rowptr.copy(), A.colind.copy()
    row = 16 + int(np.argmax(np.cumsum(np.diff(A.rowptr[16:33])) > size - 10))   # in the panel's last round
    at, end = int(A.rowptr[row]), int(A.rowptr[row + 1])
    assert end - at >= 2
    if fault == "swapped":
        ci[at], ci[at + 1] = ci[at + 1], ci[at]
    elif fault == "duplicate":
        ci[at + 1] = ci[at]
    elif fault == "beyond":
        ci[end - 1] = A.K
    elif fault == "negative":
        ci[at] = -5
    elif fault == "rowptr back":
        rp[row] = rp[row + 1] + 3
    else:
        rp[-1] -= 1
    with pytest.raises(gpu.SpmmError) as e:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), torch.from_numpy(A.vals).cuda())
    assert e.value.code == gpu.SPMM_EFORMAT
