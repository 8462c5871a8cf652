"""What users of this library run, as measurable cases: sparse matrix-vector products, the
COO -> CSR conversion, sparse matrix addition and the two 3rd-order tensor kernels.

The inputs follow the recipes of workloads.py (uniform, banded, bounded rows, power law, skewed
3rd-order tensors), drawn on the GPU so that any size is ready at once. A state holds what a
program keeps between calls: the descriptor of the operands, the dense vectors or factors, the
workspace and the output buffers. `run` is one call through the package's entry points.
"""
from __future__ import annotations

import math

import torch

import paper_1804_10112_amd as spt
from paper_1804_10112_amd.binding import SptTensor

DEV = "cuda:0"
DENSE, COMPRESSED, SINGLETON, RANGE, OFFSET = range(5)
DTYPES = {"f32": torch.float32, "f64": torch.float64}
ZIPF_ROWS, ZIPF_SLICES = 1.8, 1.5  # exponents of the power-law row lengths and of the skewed first tensor dimension


def listed():
    return [
        # a small matrix inside an outer loop (a solver, a time step): the call itself is the cost
        {"name": "spmv_csr_small", "op": "spmv", "format": "csr", "pattern": "uniform", "dtype": "f64",
         "rows": 4096, "nnz": 40_960},
        # a matrix with seven far-apart diagonals (7-point stencil), the usual CSR operand of a solver
        {"name": "spmv_csr_banded", "op": "spmv", "format": "csr", "pattern": "banded", "dtype": "f64",
         "rows": 2_000_000, "nnz": 14_000_000},
        # the same kind of matrix stored by diagonals, with a row count that no vector width divides
        {"name": "spmv_dia_odd", "op": "spmv", "format": "dia", "pattern": "banded", "dtype": "f64",
         "rows": 1_500_001, "nnz": 10_500_007},
        # a mesh-like matrix with 8 to 32 entries per row and columns anywhere, in ELL
        {"name": "spmv_ell", "op": "spmv", "format": "ell", "pattern": "bounded", "dtype": "f32",
         "rows": 1_000_000, "nnz": 19_000_000},
        # a web-like matrix as it is collected: entries in no order, multiplied without conversion
        {"name": "spmv_coo_unordered", "op": "spmv", "format": "coo_unordered", "pattern": "powerlaw",
         "dtype": "f32", "rows": 700_001, "nnz": 10_000_000},
        # the largest matrix: power-law rows (the longest of about 100 000 entries) in CSR
        {"name": "spmv_csr_powerlaw", "op": "spmv", "format": "csr", "pattern": "powerlaw", "dtype": "f64",
         "rows": 4_000_000, "nnz": 60_000_000},
        # assembling a small and the largest matrix from unordered triples
        {"name": "coo_to_csr_small", "op": "coo_to_csr", "pattern": "uniform", "dtype": "f64",
         "rows": 5003, "nnz": 50_021},
        {"name": "coo_to_csr_powerlaw", "op": "coo_to_csr", "pattern": "powerlaw", "dtype": "f64",
         "rows": 4_000_000, "nnz": 60_000_000},
        # A = B + C of two CSR matrices that share part of their structure
        {"name": "add_csr", "op": "add", "format": "csr", "pattern": "uniform", "dtype": "f64",
         "rows": 1_000_003, "nnz": 20_000_000, "nnz_c": 10_000_000},
        # tensor times vector on the largest tensor, a knowledge-base-like one with a skewed first dimension
        {"name": "ttv_coo", "op": "ttv", "format": "coo", "dtype": "f32", "i": 100_000, "j": 80_000, "k": 50_000,
         "nnz": 50_000_000, "skewed": True},
        # the inner step of a CP decomposition on an ordinary tensor (the size of a social network's) ...
        {"name": "mttkrp_csf", "op": "mttkrp", "format": "csf", "dtype": "f64", "i": 1600, "j": 64_000, "k": 64_000,
         "nnz": 737_934, "skewed": True, "rank": 16},
        # ... and on the largest
        {"name": "mttkrp_coo", "op": "mttkrp", "format": "coo", "dtype": "f32", "i": 100_000, "j": 80_000,
         "k": 50_000, "nnz": 50_000_000, "skewed": True, "rank": 32},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["spmv", "spmv", "spmv", "coo_to_csr", "add", "ttv", "mttkrp"])
    case = {"op": op, "dtype": rng.choice(["f32", "f64"])}
    if op in ("ttv", "mttkrp"):
        nnz = _log_uniform(rng, 50_000, 40_000_000 if case["dtype"] == "f32" else 20_000_000)
        case.update(format=rng.choice(["coo", "csf"]), skewed=rng.random() < 0.7)
        case.update(i=_log_uniform(rng, 1000, 100_000), j=_log_uniform(rng, 2000, 100_000),
                    k=_log_uniform(rng, 2000, 100_000))
        case["nnz"] = nnz = min(nnz, case["j"] * case["k"] // 4)  # the first slice holds up to 0.4 of a skewed tensor
        if op == "mttkrp":
            case["rank"] = rng.choice([8, 16, 16, 32, 32, 33, 64]) if nnz < 10_000_000 else rng.choice([8, 16, 32])
        return case
    nnz = _log_uniform(rng, 20_000, 40_000_000)
    if op == "spmv":
        case["format"] = rng.choice(["csr", "csr", "coo", "coo_unordered", "dia", "ell"])
    elif op == "add":
        nnz = min(nnz, 20_000_000)
        case.update(format=rng.choice(["csr", "coo"]), nnz_c=max(1000, int(nnz * rng.uniform(0.1, 1.0))))
    form = case.get("format")
    pattern = {"dia": "banded", "ell": "bounded"}.get(form)
    if pattern is None:
        pattern = rng.choice(["uniform", "bounded", "powerlaw"] + (["banded"] if op == "spmv" else []))
    mean = {"banded": 7, "bounded": 19, "powerlaw": 15}.get(pattern) or rng.uniform(4, 24)
    rows = max(2000, int(nnz / mean))
    nnz = 7 * rows if pattern == "banded" else 19 * rows if pattern == "bounded" else nnz
    case.update(pattern=pattern, rows=rows, nnz=nnz)
    return case


# ---------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _rand(n, g, dtype=torch.float64):
    return torch.rand(n, generator=g, device=DEV, dtype=dtype)


def _values(n, dtype, g):
    """U(-1, 1)."""
    return torch.rand(n, generator=g, device=DEV, dtype=dtype) * 2 - 1


def _exactly(n, draw_some, g):
    """n distinct keys, ascending: what draw_some() gives, more of it if needed, less what is too many."""
    keys = torch.unique(draw_some())
    while len(keys) < n:
        keys = torch.unique(torch.cat([keys, draw_some()]))
    if len(keys) > n:
        keep = torch.ones(len(keys), dtype=torch.bool, device=DEV)
        keep[torch.randperm(len(keys), generator=g, device=DEV)[: len(keys) - n]] = False
        keys = keys[keep]
    return keys


def _draw_keys(pattern, N, nnz, g):
    """nnz ascending distinct row * N + column of a square matrix."""

    def uniform():
        return torch.randint(0, N * N, (int(nnz * 1.05) + 64,), generator=g, device=DEV)

    def in_rows(length):
        row = torch.repeat_interleave(torch.arange(N, device=DEV), length)
        if len(row) > 1.02 * nnz:  # thinned
            row = row[_rand(len(row), g, torch.float32) < 1.02 * nnz / len(row)]
        return row * N + torch.randint(0, N, (len(row),), generator=g, device=DEV)

    def bounded():
        return in_rows(torch.randint(8, 33, (N,), generator=g, device=DEV))

    def powerlaw():  # the longest possible row N / 20 (at least 1000), thinned to about nnz entries
        longest = min(N, max(1000, N // 20))
        cdf = torch.arange(1, longest + 1, device=DEV, dtype=torch.float64).pow(-ZIPF_ROWS).cumsum(0)
        return in_rows((torch.searchsorted(cdf, _rand(N, g) * cdf[-1]) + 1).clamp_(max=longest))

    return _exactly(nnz, {"uniform": uniform, "bounded": bounded, "powerlaw": powerlaw}[pattern], g)


def _banded(N, g, dtype):
    """Offsets {0, +-1, +-sqrt(N), +-N/2}, their cells (diagonal-major), and which lie in the matrix."""
    a = max(2, math.isqrt(N))
    b = max(a + 1, N // 2)
    off = torch.tensor([-b, -a, -1, 0, 1, a, b], device=DEV)
    cells = _values(7 * N, dtype, g).view(7, N)
    col = torch.arange(N, device=DEV)[None, :] + off[:, None]
    inside = (col >= 0) & (col < N)
    return off, torch.where(inside, cells, torch.zeros((), dtype=dtype, device=DEV)), col, inside


def _matrix_entries(case, g):
    """(row, col, values), ordered by row and then column."""
    N, dtype = case["rows"], DTYPES[case["dtype"]]
    if case["pattern"] == "banded":
        _, cells, col, inside = _banded(N, g, dtype)
        inside = inside.t()
        row = torch.arange(N, device=DEV)[:, None].expand(N, 7)[inside]
        return row.int(), col.t()[inside].int(), cells.t()[inside].contiguous()
    keys = _draw_keys(case["pattern"], N, case["nnz"], g)
    return (keys // N).int(), (keys % N).int(), _values(len(keys), dtype, g)


def _starts(ids, n):
    """pos of the segments 0 .. n-1 of an ascending list of segment numbers."""
    return torch.searchsorted(ids.long(), torch.arange(n + 1, device=DEV)).int()


# ---------------------------------------------------------------------------- descriptors

def _tensor(order, vals, levels):
    """spt_tensor over arrays that live on the GPU; `levels` in storage order."""
    t = SptTensor()
    t.order, t.nlevels = order, len(levels)
    t.dtype = spt.SPT_F64 if vals.dtype == torch.float64 else spt.SPT_F32
    t.vals, t.nvals = vals.data_ptr(), vals.numel()
    keep = [vals]
    for k, lv in enumerate(levels):
        out = t.level[k]
        out.kind, out.mode, out.N, out.M = lv["kind"], lv["mode"], lv["N"], lv.get("M", 0)
        out.flags = (spt.SPT_ORDERED if lv.get("ordered", True) else 0) | (spt.SPT_UNIQUE if lv.get("unique", True) else 0)
        out.crd_stride = 1
        for name in ("pos", "crd", "offset"):
            if name in lv:
                setattr(out, name, lv[name].data_ptr())
                keep.append(lv[name])
    return t, keep


def _coo(N, row, col, vals, ordered=True):
    pos = torch.tensor([0, len(vals)], dtype=torch.int32, device=DEV)
    return _tensor(2, vals, [
        {"kind": COMPRESSED, "mode": 0, "N": N, "M": 1, "pos": pos, "crd": row, "ordered": ordered, "unique": False},
        {"kind": SINGLETON, "mode": 1, "N": N, "crd": col, "ordered": ordered}])


def _csr(N, row, col, vals):
    return _tensor(2, vals, [
        {"kind": DENSE, "mode": 0, "N": N},
        {"kind": COMPRESSED, "mode": 1, "N": N, "M": N, "pos": _starts(row, N), "crd": col}])


def _dia(N, off, cells):
    off = off.int()
    return _tensor(2, cells.reshape(-1), [
        {"kind": DENSE, "mode": -1, "N": len(off)},
        {"kind": RANGE, "mode": 0, "N": N, "M": N, "offset": off},
        {"kind": OFFSET, "mode": 1, "N": N, "offset": off}])


def _ell(N, row, col, vals):
    pos = _starts(row, N).long()
    width = int((pos[1:] - pos[:-1]).max())
    cell = (torch.arange(len(row), device=DEV) - pos[row.long()]) * N + row
    crd = torch.full((width * N,), -1, dtype=torch.int32, device=DEV)
    v = torch.zeros(width * N, dtype=vals.dtype, device=DEV)
    crd[cell], v[cell] = col, vals
    return _tensor(2, v, [
        {"kind": DENSE, "mode": -1, "N": width},
        {"kind": DENSE, "mode": 0, "N": N},
        {"kind": SINGLETON, "mode": 1, "N": N, "crd": crd, "ordered": False}])


def _tensor3(case, g):
    """The tensor in its format."""
    dims, dtype = (case["i"], case["j"], case["k"]), DTYPES[case["dtype"]]
    rest = dims[1] * dims[2]

    def some():
        n = int(case["nnz"] * 1.02) + 64
        if case["skewed"]:
            cdf = torch.arange(1, dims[0] + 1, device=DEV, dtype=torch.float64).pow(-ZIPF_SLICES).cumsum(0)
            i = torch.searchsorted(cdf, _rand(n, g) * cdf[-1]).clamp_(max=dims[0] - 1)
        else:
            i = torch.randint(0, dims[0], (n,), generator=g, device=DEV)
        return i * rest + torch.randint(0, rest, (n,), generator=g, device=DEV)

    keys = _exactly(case["nnz"], some, g)
    vals = torch.rand(len(keys), generator=g, device=DEV, dtype=dtype)
    fibre_keys, fibre_len = torch.unique_consecutive(keys // dims[2], return_counts=True)
    crd2 = (keys % dims[2]).int()
    nfib = len(fibre_keys)
    if case["format"] == "coo":
        pos = torch.tensor([0, len(keys)], dtype=torch.int32, device=DEV)
        return _tensor(3, vals, [
            {"kind": COMPRESSED, "mode": 0, "N": dims[0], "M": 1, "pos": pos, "crd": (keys // rest).int(), "unique": False},
            {"kind": SINGLETON, "mode": 1, "N": dims[1], "crd": (keys // dims[2] % dims[1]).int(), "unique": False},
            {"kind": SINGLETON, "mode": 2, "N": dims[2], "crd": crd2}])
    crd0, slice_len = torch.unique_consecutive(fibre_keys // dims[1], return_counts=True)
    zero = torch.zeros(1, dtype=torch.int32, device=DEV)
    ends = [torch.cat([zero, n.cumsum(0).int()]) for n in (slice_len, fibre_len)]
    pos0 = torch.tensor([0, len(crd0)], dtype=torch.int32, device=DEV)
    return _tensor(3, vals, [
        {"kind": COMPRESSED, "mode": 0, "N": dims[0], "M": 1, "pos": pos0, "crd": crd0.int()},
        {"kind": COMPRESSED, "mode": 1, "N": dims[1], "M": len(crd0), "pos": ends[0], "crd": (fibre_keys % dims[1]).int()},
        {"kind": COMPRESSED, "mode": 2, "N": dims[2], "M": nfib, "pos": ends[1], "crd": crd2}])


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV)


def _ints(n):
    return torch.zeros(n, dtype=torch.int32, device=DEV)


# ---------------------------------------------------------------------------- the four functions of a case

def prepare(case, seed):
    g, op, dtype = _gen(seed), case["op"], DTYPES[case["dtype"]]
    if op == "spmv":
        N = case["rows"]
        if case["format"] == "dia":
            off, cells, _, _ = _banded(N, g, dtype)
            A, keep = _dia(N, off, cells)
        else:
            row, col, vals = _matrix_entries(case, g)
            if case["format"] == "coo_unordered":
                p = torch.randperm(len(row), generator=g, device=DEV)
                A, keep = _coo(N, row[p], col[p], vals[p], ordered=False)
            else:
                A, keep = {"csr": _csr, "coo": _coo, "ell": _ell}[case["format"]](N, row, col, vals)
        return {"op": op, "A": A, "keep": keep, "x": _values(N, dtype, g),
                "y": torch.zeros(N, dtype=dtype, device=DEV),
                "ws": _workspace(spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A))}
    if op == "coo_to_csr":
        N = case["rows"]
        row, col, vals = _matrix_entries(case, g)
        p = torch.randperm(len(row), generator=g, device=DEV)
        A, keep = _coo(N, row[p], col[p], vals[p], ordered=False)
        return {"op": op, "A": A, "keep": keep, "pos": _ints(N + 1), "crd": _ints(len(vals)),
                "vals": torch.zeros_like(vals), "ws": _workspace(spt.spt_workspace_bytes(spt.SPT_OP_COO_TO_CSR, A))}
    if op == "add":
        # C takes about half of its entries from B's structure and draws the others afresh
        N, build = case["rows"], _csr if case["format"] == "csr" else _coo
        kb = _draw_keys(case["pattern"], N, case["nnz"], g)
        shared = kb[torch.randperm(len(kb), generator=g, device=DEV)[: case["nnz_c"] // 2]]
        fresh = _draw_keys("uniform", N, case["nnz_c"] - len(shared), g)
        kc = _exactly(case["nnz_c"], lambda: torch.cat([shared, fresh, torch.randint(0, N * N, (case["nnz_c"] // 50 + 64,), generator=g, device=DEV)]), g)
        B, keep_b = build(N, (kb // N).int(), (kb % N).int(), _values(len(kb), dtype, g))
        C, keep_c = build(N, (kc // N).int(), (kc % N).int(), _values(len(kc), dtype, g))
        cap = len(kb) + len(kc)
        csr = case["format"] == "csr"
        return {"op": op, "B": B, "C": C, "keep": keep_b + keep_c, "count": torch.zeros(1, dtype=torch.int64, device=DEV),
                "pos": _ints(N + 1) if csr else None, "crd0": None if csr else _ints(cap), "crd1": _ints(cap),
                "vals": torch.zeros(cap, dtype=dtype, device=DEV), "ws": _workspace(spt.spt_add_workspace_bytes(B, C))}
    B, keep = _tensor3(case, g)
    state = {"op": op, "B": B, "keep": keep}
    if op == "ttv":
        coo = case["format"] == "coo"
        cap = B.nvals
        state.update(c=_rand(case["k"], g, dtype), crd0=_ints(cap) if coo else None, crd1=_ints(cap) if coo else None,
                     vals=torch.zeros(cap, dtype=dtype, device=DEV), count=torch.zeros(1, dtype=torch.int64, device=DEV),
                     ws=_workspace(spt.spt_workspace_bytes(spt.SPT_OP_TTV, B)))
    else:
        J = case["rank"]
        state.update(J=J, C=_rand(case["j"] * J, g, dtype), D=_rand(case["k"] * J, g, dtype),
                     A=torch.zeros(case["i"], J, dtype=dtype, device=DEV),
                     ws=_workspace(spt.spt_workspace_bytes(spt.SPT_OP_MTTKRP, B, J)))
    return state


def run(state):
    s, op = state, state["op"]
    if op == "spmv":
        spt.spt_spmv(s["A"], s["x"], s["y"], s["ws"])
        return s["y"]
    if op == "coo_to_csr":
        spt.spt_coo_to_csr(s["A"], spt.SPT_ORDER_ROW_COL, s["pos"], s["crd"], s["vals"], s["ws"])
        return {"pos": s["pos"], "crd": s["crd"], "vals": s["vals"]}
    if op == "mttkrp":
        spt.spt_mttkrp(s["B"], s["C"], s["D"], s["J"], s["A"], s["ws"])
        return s["A"]
    # the entries of the result (their number comes in count) are followed by what the buffers held: zeros
    if op == "add":
        spt.spt_add(s["B"], s["C"], s["pos"], s["crd0"], s["crd1"], None, s["vals"], s["count"], s["ws"])
        return {"first": s["pos"] if s["crd0"] is None else s["crd0"], "crd1": s["crd1"], "vals": s["vals"], "count": s["count"]}
    spt.spt_ttv(s["B"], s["c"], s["crd0"], s["crd1"], s["vals"], s["count"], s["ws"])
    if s["crd0"] is None:
        return {"vals": s["vals"], "count": s["count"]}
    return {"crd0": s["crd0"], "crd1": s["crd1"], "vals": s["vals"], "count": s["count"]}


def work(case):
    op, nnz, v = case["op"], case["nnz"], 8 if case["dtype"] == "f64" else 4
    if op == "mttkrp":
        dense = (case["i"] + case["j"] + case["k"]) * case["rank"] * v
        return {"bytes": (12 + v if case["format"] == "coo" else 4 + v) * nnz + dense, "flops": 3 * case["rank"] * nnz}
    if op == "ttv":
        fibres = case["i"] * case["j"] * -math.expm1(-nnz / (case["i"] * case["j"]))  # if spread evenly
        if case["skewed"]:
            fibres = _skewed_fibres(case["i"], case["j"], nnz)
        if case["format"] == "coo":
            return {"bytes": (12 + v) * nnz + (8 + v) * fibres + v * case["k"], "flops": 2 * nnz}
        return {"bytes": (4 + v) * nnz + (4 + v) * fibres + v * case["k"], "flops": 2 * nnz}
    N = case["rows"]
    if op == "coo_to_csr":
        return {"bytes": (8 + v) * nnz + (4 + v) * nnz + 4 * (N + 1), "flops": 0}
    if op == "add":
        both = nnz + case["nnz_c"] + (nnz + case["nnz_c"] - case["nnz_c"] // 2)  # operands and result
        return {"bytes": both * (4 + v) + 12 * (N + 1) if case["format"] == "csr" else both * (8 + v), "flops": case["nnz_c"] // 2}
    if case["pattern"] == "banded":
        nnz = 7 * N - 2 - 2 * math.isqrt(N) - 2 * (N // 2)  # cells inside the matrix
    if case["format"] == "dia":
        return {"bytes": v * nnz + 2 * v * N, "flops": 2 * nnz}
    if case["format"] == "ell":
        return {"bytes": (4 + v) * 32 * N + 2 * v * N, "flops": 2 * nnz}
    entry = 4 + v if case["format"] == "csr" else 8 + v
    return {"bytes": entry * nnz + 2 * v * N + (4 * (N + 1) if case["format"] == "csr" else 0), "flops": 2 * nnz}


def _skewed_fibres(I, J, nnz):
    """Expected number of (i, j) pairs that hold an entry, slice i drawn with weight (i + 1)^-ZIPF_SLICES."""
    w = torch.arange(1, I + 1, dtype=torch.float64).pow(-ZIPF_SLICES)
    return float((J * -torch.expm1(-nnz * w / w.sum() / J)).sum())


def tolerance(case):
    # copied integers and values, and single rounded sums
    if case["op"] in ("coo_to_csr", "add"):
        return "exact"
    # sums in the operands' precision, taken in some order
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-13}
