"""A few heavy panels among many light, scattered ones: ranked by a bitmap of all columns, up to the number of
columns and the mean of entries where that ends, and panel_ptr by one launch or two."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import INT_KEYS, assert_format_equal, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu

HEAVY = (513, 600, 1024, 2048, 2049, 4097, 8191, 8192)


def matrix(P, K, light, heavy, seed):
    """P panels of `light` entries each but for the heavy ones, far apart; a last panel of five rows."""
    rng = np.random.default_rng(seed)
    sizes = np.full(P, light)
    sizes[np.linspace(0, P - 2, len(heavy)).astype(int)] = heavy
    panel = np.repeat(np.arange(P), sizes)
    row = np.minimum(16 * panel + rng.integers(0, 16, len(panel)), 16 * P - 12)
    col = rng.integers(0, K, len(panel))
    # half of a panel's entries in columns that its rows share; its ends reached, so that the span is wide
    col = np.where(rng.random(len(panel)) < 0.5, (panel * 977 + rng.integers(0, 40, len(panel)) * (K // 41)) % K, col)
    edge = np.r_[True, panel[1:] != panel[:-1]]
    col[edge] = K - 1
    col[np.r_[False, edge[:-1]]] = 0
    return W.csr_from_coo(16 * P - 11, K, row, col, rng.uniform(-1, 1, len(panel)).astype(np.float32))


def same_as_the_oracle(gpu, A):  # noqa: F811
    plan = make_plan(gpu, A)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    assert_format_equal(gpu.spmm_plan_export(plan), ref)
    got, exp = gpu.spmm_synergy(plan, 8), oracle.synergy(A.M, A.K, 8, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])


# 2^19 columns are the last that the bitmap takes; more light panels than one workgroup of the scan
@pytest.mark.parametrize("K", [50_001, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("P", [300, 4097])
@pytest.mark.parametrize("heavy", [HEAVY, (513,), (2049,) * 3, (700,) * 40])
def test_heavy_panels_among_light_ones(gpu, K, P, heavy):  # noqa: F811
    same_as_the_oracle(gpu, matrix(P, K, 20, heavy, seed=P + len(heavy)))


@pytest.mark.parametrize("light", [126, 140])      # a mean below and above 128
def test_mean_of_entries(gpu, light):  # noqa: F811
    same_as_the_oracle(gpu, matrix(400, 300_000, light, (600, 700), seed=light))


@pytest.mark.parametrize("P", [1 << 16, (1 << 16) + 1])
def test_panels_of_one_scan_launch(gpu, P):  # noqa: F811
    same_as_the_oracle(gpu, matrix(P, 400_000, 6, (600, 3000), seed=7))


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("fault", ["swapped", "duplicate", "beyond", "negative"])
def test_invalid_columns_in_heavy_panels(gpu, n, fault):  # noqa: F811
    import torch
    A = matrix(300, 90_000, 20, (600, n, 600), seed=n)
    panel = int(np.argmax(np.diff(A.rowptr[::16]) == np.diff(A.rowptr[::16])[1:-1].max()))
    lengths = np.diff(A.rowptr)
    row = 16 * panel + int(np.argmax(lengths[16 * panel:16 * panel + 16] >= 3))
    ci, at, end = A.colind.copy(), int(A.rowptr[row]), int(A.rowptr[row + 1])
    assert end - at >= 3
    if fault == "swapped":
        ci[at], ci[at + 1] = ci[at + 1], ci[at]
    elif fault == "duplicate":
        ci[at + 1] = ci[at]
    elif fault == "beyond":
        ci[end - 1] = A.K
    else:
        ci[at] = -1
    with pytest.raises(gpu.SpmmError) as e:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(ci).cuda(),
                      torch.from_numpy(A.vals).cuda())
    assert e.value.code == gpu.SPMM_EFORMAT
