"""Performance cases of the sparse-dense product C = A.B.

A user of this library holds a sparse matrix as CSR arrays on the GPU, makes a plan for it, and
multiplies dense matrices with the plan, many times (iterative solvers, graph networks: "exec"), once
("oneshot": plan, product and destruction of the plan are all on the clock), or once per set of new
values of one pattern (a matrix re-assembled every time step: "update").  "noalloc" is the entry
point for serving loops that must not allocate.

The sparsity patterns are those of the benchmark's configurations, drawn with torch on the GPU
(making 41 million entries takes milliseconds there): a narrow band, dense 3x3 blocks scattered
within a wider band (structural and FEM matrices), a power-law graph, and 16x4 cells at random
places filled to a given fraction.  The arithmetic is the default one, float32; the reduced-precision
modes and 32-row panels are experiments that nothing selects by itself and are left out.
"""
import math

import torch

from paper_2504_06443_amd import binding as spmm

BLOCK = 3              # rows and columns of a dense block of the "blocks" pattern
ZIPF, DEGREE_CAP = 2.1, 3000
GRAPH_NNZ_PER_ROW = 929849 / 325760
CELL_ROWS, CELL_COLS = 16, 4


def listed():
    return [
        # smallest call: a banded 4096-row operator in a serving loop; latency and launches
        {"name": "band_4k_n32_noalloc", "mode": "noalloc", "pattern": "band", "M": 4096, "N": 32,
         "per_row": 10, "half_width": 64},
        # structural matrix of ordinary size, N = 128: the paper's main width
        {"name": "blocks_262k_n128", "mode": "exec", "pattern": "blocks", "M": 262144, "N": 128,
         "per_row": 10.0, "half_width": 256},
        # web graph: scattered columns, heavy rows beside empty ones (message passing in a graph network)
        {"name": "graph_326k_n128", "mode": "exec", "pattern": "graph", "M": 325760, "N": 128},
        # the largest single-GPU configuration, at both of its widths
        {"name": "blocks_923k_n128", "mode": "exec", "pattern": "blocks", "M": 923136, "N": 128,
         "per_row": 14.8, "half_width": 1024},
        {"name": "blocks_923k_n32", "mode": "exec", "pattern": "blocks", "M": 923136, "N": 32,
         "per_row": 14.8, "half_width": 1024},
        # scattered, thinly filled cells at a narrow width
        {"name": "cells_65k_f10_n64", "mode": "exec", "pattern": "cells", "M": 65536, "N": 64,
         "fill": 0.1, "nnz": 2000000},
        # well filled cells at the widest width (hidden features of a network)
        {"name": "cells_65k_f80_n512", "mode": "exec", "pattern": "cells", "M": 65536, "N": 512,
         "fill": 0.8, "nnz": 2000000},
        # well filled cells over a B of half a gigabyte: nothing stays in a cache
        {"name": "cells_1m_f80_n128", "mode": "exec", "pattern": "cells", "M": 1048576, "N": 128,
         "fill": 0.8, "nnz": 32000000},
        # ragged sizes: rows not a multiple of a panel, an odd number of right-hand sides
        {"name": "blocks_100003_n77", "mode": "exec", "pattern": "blocks", "M": 100003, "N": 77,
         "per_row": 10.0, "half_width": 256},
        # new pattern for every product: pre-processing is on the clock
        {"name": "blocks_262k_n128_oneshot", "mode": "oneshot", "pattern": "blocks", "M": 262144,
         "N": 128, "per_row": 10.0, "half_width": 256},
        {"name": "graph_326k_n64_oneshot", "mode": "oneshot", "pattern": "graph", "M": 325760,
         "N": 64},
        # a matrix re-assembled every time step: new values, then a product with a few vectors
        {"name": "blocks_262k_n16_update", "mode": "update", "pattern": "blocks", "M": 262144,
         "N": 16, "per_row": 10.0, "half_width": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case from the ranges of the listed ones."""
    while True:
        case = {"mode": rng.choice(["exec", "exec", "exec", "noalloc", "oneshot", "update"]),
                "pattern": rng.choice(["band", "blocks", "blocks", "graph", "cells"])}
        case["M"] = _log_int(rng, 4096, 1048576)
        n = _log_int(rng, 8, 512)
        # widths are multiples of 16 as often as not; the others are whatever comes, odd ones too
        case["N"] = max(16, n // 16 * 16) if rng.random() < 0.5 else n
        if case["pattern"] == "band":
            case["per_row"] = rng.randint(3, 20)
            case["half_width"] = _log_int(rng, 16, 512)
        elif case["pattern"] == "blocks":
            case["per_row"] = round(rng.uniform(4.0, 15.0), 1)
            case["half_width"] = _log_int(rng, 128, 1024)
        elif case["pattern"] == "cells":
            case["M"] = max(4096, case["M"] // 16 * 16)
            case["fill"] = round(math.exp(rng.uniform(math.log(0.05), math.log(0.8))), 3)
            case["nnz"] = case["M"] * rng.randint(8, 40)
        # no more than the largest listed cases, in products as in bytes of B and C
        if _nnz(case) * case["N"] <= 5.2e9 and case["M"] * case["N"] <= 1.35e8:
            return case


# ------------------------------------------------------------------------------- inputs
def _csr(M, K, keys):
    """Sorted, duplicate-free CSR of the (row * K + column) keys."""
    keys = torch.unique(keys)
    rows = torch.div(keys, K, rounding_mode="floor")
    rowptr = torch.zeros(M + 1, dtype=torch.int64, device=keys.device)
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=M), 0)
    return rowptr.to(torch.int32), (keys - rows * K).to(torch.int32)


def _band(case, gen, dev):
    M = case["M"]
    hw = case["half_width"]
    off = torch.randint(-hw, hw + 1, (M, case["per_row"]), generator=gen, device=dev)
    rows = torch.arange(M, device=dev)[:, None]
    return _csr(M, M, (rows * M + (rows + off).clamp_(0, M - 1)).flatten())


def _blocks(case, gen, dev, chunk=65536):
    M, per_row = case["M"], case["per_row"]
    n_rows = -(-M // BLOCK)
    hw = case["half_width"] // BLOCK
    base = int(per_row)
    at_most = min(base + 1, 2 * hw + 1)
    inner = torch.arange(BLOCK, device=dev)
    keys = []
    for r0 in range(0, n_rows, chunk):
        r = torch.arange(r0, min(n_rows, r0 + chunk), device=dev)
        weight = torch.rand((len(r), 2 * hw + 1), generator=gen, device=dev)
        pick = torch.topk(weight, at_most, dim=1).indices          # distinct block columns
        count = base + (torch.rand(len(r), generator=gen, device=dev) < per_row - base).long()
        col = r[:, None] - hw + pick
        keep = (torch.arange(at_most, device=dev)[None, :] < count[:, None]) & (col >= 0) & (col < n_rows)
        row = r[:, None].expand_as(col)[keep] * BLOCK
        col = col[keep] * BLOCK
        rr = (row[:, None, None] + inner[None, :, None]).expand(-1, BLOCK, BLOCK)
        cc = (col[:, None, None] + inner[None, None, :]).expand(-1, BLOCK, BLOCK)
        inside = (rr < M) & (cc < M)
        keys.append(rr[inside] * M + cc[inside])
    return _csr(M, M, torch.cat(keys))


def _graph(case, gen, dev):
    M = case["M"]
    p = torch.arange(1, DEGREE_CAP + 1, dtype=torch.float64, device=dev) ** -ZIPF
    zeta = p.sum() + (DEGREE_CAP + 0.5) ** (1.0 - ZIPF) / (ZIPF - 1.0)
    u = torch.rand(M, generator=gen, device=dev, dtype=torch.float64)
    degree = torch.searchsorted(torch.cumsum(p / zeta, 0), u).clamp_(max=DEGREE_CAP)
    rows = torch.repeat_interleave(torch.arange(M, device=dev), degree)
    keys = torch.unique(rows * M + torch.randint(0, M, rows.shape, generator=gen, device=dev))
    want = int(M * GRAPH_NNZ_PER_ROW)
    if keys.numel() > want:
        keys = keys[torch.randperm(keys.numel(), generator=gen, device=dev)[:want]]
    return _csr(M, M, keys)


def _cells(case, gen, dev, chunk=1 << 20):
    M = case["M"]
    per = max(1, round(CELL_ROWS * CELL_COLS * case["fill"]))
    n_cells = max(1, round(case["nnz"] / per))
    keys = []
    for c0 in range(0, n_cells, chunk):
        n = min(chunk, n_cells - c0)
        row = torch.randint(0, M // CELL_ROWS, (n, 1), generator=gen, device=dev) * CELL_ROWS
        col = torch.randint(0, M // CELL_COLS, (n, 1), generator=gen, device=dev) * CELL_COLS
        weight = torch.rand((n, CELL_ROWS * CELL_COLS), generator=gen, device=dev)
        pick = torch.topk(weight, per, dim=1).indices
        keys.append(((row + pick // CELL_COLS) * M + col + pick % CELL_COLS).flatten())
    return _csr(M, M, torch.cat(keys))


_PATTERNS = {"band": _band, "blocks": _blocks, "graph": _graph, "cells": _cells}


def _inputs(case, seed):
    """CSR arrays, B, and for "update" the next time step's values (else the same values)."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    M, N = case["M"], case["N"]
    rowptr, colind = _PATTERNS[case["pattern"]](case, gen, dev)
    nnz = colind.numel()
    if case["pattern"] == "graph":
        vals = torch.ones(nnz, device=dev)                          # adjacency
    else:
        vals = torch.rand(nnz, generator=gen, device=dev) * 2 - 1
    B = torch.randn((M, N), generator=gen, device=dev)
    new_vals = vals
    if case["mode"] == "update":
        new_vals = torch.rand(nnz, generator=gen, device=dev) * 2 - 1
    return rowptr, colind, vals, B, new_vals


def prepare(case, seed):
    M, N = case["M"], case["N"]
    rowptr, colind, vals, B, new_vals = _inputs(case, seed)
    state = {"mode": case["mode"], "M": M, "rowptr": rowptr, "colind": colind, "vals": new_vals,
             "B": B, "C": torch.empty((M, N), device=B.device)}
    if case["mode"] != "oneshot":
        state["plan"] = spmm.spmm_plan(M, M, rowptr, colind, vals)
    return state


def exact(case, seed, chunk=1 << 27):
    """The same product in 64 bits, a range of entries (about `chunk` products) at a time."""
    M, N = case["M"], case["N"]
    rowptr, colind, _, B, vals = _inputs(case, seed)
    rows = torch.repeat_interleave(torch.arange(M, device=B.device), rowptr.diff().long())
    C = torch.zeros((M, N), dtype=torch.float64, device=B.device)
    step = max(1, chunk // N)
    for e in range(0, rows.numel(), step):
        part = B[colind[e:e + step].long()].double() * vals[e:e + step, None].double()
        C.index_add_(0, rows[e:e + step], part)
    return C


def run(state):
    mode = state["mode"]
    if mode == "exec":
        return spmm.spmm_exec(state["plan"], state["B"], state["C"])
    if mode == "noalloc":
        return spmm.spmm_exec_noalloc(state["plan"], state["B"], state["C"])
    if mode == "update":
        spmm.spmm_plan_update_values(state["plan"], state["vals"])
        return spmm.spmm_exec(state["plan"], state["B"], state["C"])
    plan = spmm.spmm_plan(state["M"], state["M"], state["rowptr"], state["colind"], state["vals"])
    C = spmm.spmm_exec(plan, state["B"], state["C"])
    spmm.spmm_plan_destroy(plan)
    return C


# ------------------------------------------------------------------------------- model
def _nnz(case):
    M = case["M"]
    if case["pattern"] == "band":
        width = 2 * case["half_width"] + 1
        return int(M * width * (1.0 - (1.0 - 1.0 / width) ** case["per_row"]))
    if case["pattern"] == "blocks":
        return int(M * BLOCK * min(case["per_row"], 2 * (case["half_width"] // BLOCK) + 1))
    if case["pattern"] == "graph":
        return int(M * GRAPH_NNZ_PER_ROW)
    return case["nnz"]


def work(case):
    """The entries' values with a byte each for their places (what the brick format spends on
    them; the CSR arrays themselves where they are the input), the rows of B that occur, and C."""
    M, N, nnz = case["M"], case["N"], _nnz(case)
    used = M
    if case["pattern"] == "graph":
        used = M * (1.0 - math.exp(-GRAPH_NNZ_PER_ROW))
    elif case["pattern"] == "cells":
        cells = nnz / (CELL_ROWS * CELL_COLS * case["fill"])
        used = M * (1.0 - math.exp(-cells / (M / CELL_COLS)))
    a_bytes = 8 * nnz + 4 * (M + 1) if case["mode"] == "oneshot" else 5 * nnz
    if case["mode"] == "update":
        a_bytes += 4 * nnz                                          # the new values
    return {"bytes": a_bytes + 4.0 * N * (used + M), "flops": 2.0 * nnz * N}


def tolerance(case):
    # float32 products and sums.  Against the same product in float64 the library shows at most
    # 1.2e-7 (rel) and 1.4e-6 (max) for rows of up to a few dozen entries, 2.0e-7 and 2.6e-5 where
    # rows of the graph sum thousands; four times that.
    if case["pattern"] == "graph":
        return {"rel": 8e-7, "max": 1e-4}
    return {"rel": 5e-7, "max": 6e-6}
