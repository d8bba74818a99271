"""The first pass of a plan, which counts the active columns of band-like panels: format and counts equal the
oracle's bit for bit around its limits (16,384 columns of span, bitmap words against entries, rounds of 256
entries in runs of four, ragged ends), and invalid arrays are refused wherever they are."""
import numpy as np
import pytest

import oracle
from paper_2504_06443_amd import workloads as W
from test_gpu_parity import INT_KEYS, assert_format_equal, gpu, make_plan  # noqa: F401

pytestmark = pytest.mark.gpu


def band(M, K, per_panel, span, seed, first=0):
    """Panel p holds per_panel[p % len] entries over exactly span[p % len] columns (one entry: any span)."""
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    for p in range((M + 15) // 16):
        n, w = per_panel[p % len(per_panel)], span[p % len(span)]
        here = min(16, M - 16 * p)
        n = min(n, here * w)
        if n == 0:
            continue
        c0 = int(rng.integers(first, K - w + 1))
        cells = {0, min(n, 2) - 1 and (here * w - 1)}            # (row, column) as row * w + column: both ends
        while len(cells) < n:
            cells.add(int(rng.integers(here * w)))
        cells = np.fromiter(cells, np.int64)
        rows.append(16 * p + cells // w)
        cols.append(c0 + cells % w)
    r = np.concatenate(rows) if rows else np.zeros(0, np.int64)
    c = np.concatenate(cols) if cols else np.zeros(0, np.int64)
    return W.csr_from_coo(M, K, r, c, rng.uniform(-1, 1, len(r)).astype(np.float32))


def check(gpu, A):  # noqa: F811
    plan = make_plan(gpu, A)
    ref = oracle.build_bricks(A.M, A.rowptr, A.colind, A.vals)
    assert_format_equal(gpu.spmm_plan_export(plan), ref)
    got, exp = gpu.spmm_synergy(plan, 8), oracle.synergy(A.M, A.K, 8, A.rowptr, A.colind, ref)
    for k in INT_KEYS:
        assert got[k] == exp[k], (k, got[k], exp[k])


@pytest.mark.parametrize("M", [1, 16, 17, 31, 16 * 8, 16 * 8 + 1, 16 * 6145 - 3])
@pytest.mark.parametrize("per_panel", [(1, 2, 3, 0, 5), (255, 256, 257, 260), (511, 512, 4, 513, 769)])
def test_ragged_panels_and_rounds_of_entries(gpu, M, per_panel):  # noqa: F811
    if M > 9000 and per_panel[0] > 1:
        per_panel = tuple(n // 8 for n in per_panel)
    check(gpu, band(M, 40000, per_panel, (90, 33, 32, 1, 700), seed=M))


@pytest.mark.parametrize("span", [16383, 16384, 16385, 16416, 16417])
@pytest.mark.parametrize("n", [96, 112, 113, 4000])
def test_span_and_words_at_their_limits(gpu, span, n):  # noqa: F811
    """512 words are 16,384 columns; 4 * 112 + 64 = 512.  Panels of one column beside them."""
    check(gpu, band(16 * 20, 60000, (n,), (span,), seed=n))
    check(gpu, band(16 * 20 + 9, 60000, (n, 16, 500), (span, 1, 300), seed=n))


def test_last_columns_of_the_matrix(gpu):  # noqa: F811
    check(gpu, band(400, 2000, (300,), (500,), seed=3, first=1500))
    check(gpu, band(400, 7, (30, 7, 0), (7, 7, 7), seed=4))


@pytest.mark.parametrize("lengths", [(64,) * 16, (0, 64, 0, 0, 128, 1, 63, 0), (0,) * 15 + (65,), (1,) * 16,
                                     (63, 1, 0, 0, 64, 0, 65), (128,) * 16, (128,) * 15 + (129,), (200,) * 16,
                                     (3, 0, 61, 0, 0, 0, 0, 192)])
def test_rows_that_begin_around_blocks_of_entries(gpu, lengths):  # noqa: F811
    """Rows that begin at, before and behind multiples of 64 entries, empty ones between, and panels of 2048
    entries, of one more and of many more, which are not staged; a panel of one row follows."""
    rng = np.random.default_rng(sum(lengths))
    r = np.repeat(np.arange(len(lengths)), lengths)
    c = np.concatenate([np.sort(rng.choice(330, n, replace=False)) for n in lengths])
    r, c = np.concatenate([r, np.full(7, 16)]), np.concatenate([c, np.arange(7) * 2])
    check(gpu, W.csr_from_coo(17, 400, r, c, rng.uniform(-1, 1, len(r)).astype(np.float32)))


@pytest.mark.parametrize("at", [0, 1, 3, 4, 7, 8, 255, 256, 257, 300])
@pytest.mark.parametrize("fault", ["swapped", "duplicate", "beyond", "negative", "rowptr"])
def test_faults_inside_a_counted_panel(gpu, at, fault):  # noqa: F811
    """One faulty entry pair at entry `at` of a panel whose first row holds them all."""
    import torch
    cols = np.arange(310, dtype=np.int64) * 3
    r = np.concatenate([np.repeat([0, 40], 5), np.full(310, 16), [17, 18]])
    c = np.concatenate([np.tile(np.arange(5), 2), cols, [4, 930]])
    A = W.csr_from_coo(60, 1000, r, c, np.ones(len(r), np.float32))
    rp, ci = A.rowptr.copy(), A.colind.copy()
    e = int(rp[16]) + at
    if fault == "swapped":
        ci[e], ci[e + 1] = ci[e + 1], ci[e]
    elif fault == "duplicate":
        ci[e + 1] = ci[e]
    elif fault == "beyond":
        ci[e] = A.K
    elif fault == "negative":
        ci[e] = -1
    else:
        rp[17 + at % 40] = (-1, A.nnz + 1)[at % 2]
    with pytest.raises(gpu.SpmmError) as err:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(),
                      torch.from_numpy(A.vals).cuda())
    assert err.value.code == gpu.SPMM_EFORMAT
    check(gpu, A)                                             # and the next plan is as ever


@pytest.mark.parametrize("ends", [(-2**31, 2**31 - 1), (-2**31 + 5, 2**31 - 1), (-2**31, 2**31 - 32), (-1, 2**31 - 1),
                                  (-2**31, 5), (0, 2**31 - 1), (-2, 900)])
def test_columns_far_outside_the_matrix(gpu, ends):  # noqa: F811
    """Spans that wrap around in 32 bits, or come to few bitmap words so, beside panels that are counted at the
    same time: refused, and no column is taken for a place in a bitmap."""
    import torch
    M, lo, hi = 16 * 24, *ends
    inner = np.unique(np.clip(lo + 32 * np.arange(1, 9000, 7, dtype=np.int64), lo + 1, hi - 1))[:1200]
    r = np.concatenate([np.repeat(np.arange(M), 6), np.full(len(inner), 37)])
    c = np.concatenate([np.tile(np.arange(6) * 5, M), 100 + np.arange(len(inner))])
    A = W.csr_from_coo(M, 2000, r, c, np.ones(len(r), np.float32))
    ci = A.colind.copy()
    b, e = int(A.rowptr[37]), int(A.rowptr[38])
    ci[b:e] = np.resize(inner, e - b)
    ci[b], ci[e - 1] = lo, hi
    with pytest.raises(gpu.SpmmError) as err:
        gpu.spmm_plan(A.M, A.K, torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(ci).cuda(),
                      torch.from_numpy(A.vals).cuda())
    assert err.value.code == gpu.SPMM_EFORMAT
    check(gpu, A)
