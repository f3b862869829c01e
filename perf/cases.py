"""Timed workloads of the library: inputs, one call each, an fp64 reference.

A case names a public entry point, a matrix structure and the dense widths.
listed() holds the workloads of the benchmark at their own sizes beside the
shapes that a caller with other data brings (widths off the powers of two,
row counts off them, small and mid-size matrices); draw() gives further ones
of the same ranges.  All inputs are made on the GPU from the seed.

Structures (N rows = N columns in all of them):
  uniform   every row has `deg` uniformly drawn columns, sorted
  rmat      2^levels vertices, deg * 2^levels R-MAT edges drawn with
            (.57, .19, .19, .05), duplicates merged
  stencil   27-point stencil on an n^3 grid, boundary rows truncated
  power     Pareto row lengths (30% empty rows, mean about deg), columns
            drawn towards the low indices, as in a graph with popular vertices
"""
import torch

import paper_2205_11622_amd as slnr

RMAT_KEPT = 0.957  # share of the drawn R-MAT edges left after merging (at 2^20 x 16, 2^22 x 32)

FUSED = ("fused", "fused_noalloc", "fused_dt", "unfused")
EPILOGUE = ("fused_gemm", "spmm_gemm", "spmmh_gemm")


def listed():
    return [
        # one layer on a citation-network sized graph: launch and latency bound
        dict(name="fused_small_32", op="fused", kind="uniform", n=2048, deg=10, K=32, L=32),
        # a mid-size matrix at the usual width
        dict(name="fused_mid_64", op="fused", kind="uniform", n=65536, deg=16, K=64, L=64),
        # a web-scale graph at the usual hidden width: the benchmark's headline
        dict(name="fused_rmat20_128", op="fused", kind="rmat", levels=20, deg=16, K=128, L=128),
        # the largest graph
        dict(name="fused_rmat22_64", op="fused", kind="rmat", levels=22, deg=32, K=64, L=64),
        # a finite-element matrix with narrow features against a wide right side
        dict(name="fused_stencil_16x256", op="fused", kind="stencil", n=128, K=16, L=256),
        # feature and class counts as data sets have them: no power of two, rows off 16 bytes
        dict(name="fused_power_100x47", op="fused", kind="power", n=100003, deg=25, K=100, L=47),
        # the two separate passes, with the nonzero values as an output of their own
        dict(name="unfused_power_128", op="unfused", kind="power", n=700001, deg=20, K=128, L=128),
        # propagation alone, a width that is a multiple of 4 only
        dict(name="spmm_power_96", op="spmm", kind="power", n=300007, deg=20, K=0, L=96),
        # D as it comes out of a transposed projection
        dict(name="dt_uniform_64", op="fused_dt", kind="uniform", n=150000, deg=24, K=64, L=64),
        # the products with a dense matrix behind them, at the benchmark's sizes
        dict(name="fused_gemm_rmat20_64", op="fused_gemm", kind="rmat", levels=20, deg=16, K=64, L=64, out=64),
        dict(name="spmm_gemm_rmat20_128x64", op="spmm_gemm", kind="rmat", levels=20, deg=16, K=0, L=128, out=64),
        dict(name="spmmh_gemm_rmat20_128", op="spmmh_gemm", kind="rmat", levels=20, deg=16, K=0, L=128, out=128),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _width(rng):
    """Powers of two as often as other widths, up to 512."""
    if rng.random() < 0.5:
        return rng.choice([16, 32, 64, 128, 256, 512])
    w = _log_uniform(rng, 5, 400)
    return w - w % 4 + 4 if rng.random() < 0.4 else w


def draw(rng):
    while True:
        op = rng.choice(["fused", "fused", "fused", "fused", "fused_noalloc", "fused_dt", "unfused", "sddmm", "spmm",
                         "fused_gemm", "spmm_gemm", "spmmh_gemm"])
        kind = rng.choice(["uniform", "rmat", "power", "stencil"])
        if kind == "rmat" and op in ("unfused", "sddmm"):
            continue  # nnz outputs: structures whose nnz does not depend on the seed
        c = dict(op=op, kind=kind)
        if kind == "rmat":
            c.update(levels=rng.randint(11, 21), deg=rng.randint(4, 40))
        elif kind == "stencil":
            c.update(n=_log_uniform(rng, 12, 128))
        else:
            c.update(n=_log_uniform(rng, 1500, 2000000), deg=_log_uniform(rng, 3, 60))
        if op in EPILOGUE:
            L = rng.choice([16, 32, 64, 64, 128, 128, 256])
            c.update(K=L if op == "fused_gemm" else 0, L=L, out=rng.choice([16, 32, 64, 128, _log_uniform(rng, 7, 300)]))
        else:
            L = 0 if op == "sddmm" else _width(rng)
            K = 0 if op == "spmm" else L if L and rng.random() < 0.4 else _width(rng)
            c.update(K=K, L=L)
        # about as much gathered as the largest listed graph at most, and operands of at most 2 GB each
        if 4 * _nnz(c) * (c["K"] + c["L"]) < 6e10 and 4 * _rows(c) * max(c["K"], c["L"], c.get("out", 0)) < 2 << 30:
            return c


def _rows(c):
    if c["kind"] == "rmat":
        return 1 << c["levels"]
    return c["n"] ** 3 if c["kind"] == "stencil" else c["n"]


def _nnz(c):
    """Nonzeros (of the random structures: about)."""
    if c["kind"] == "rmat":
        return int(RMAT_KEPT * c["deg"] * _rows(c))
    return (3 * c["n"] - 2) ** 3 if c["kind"] == "stencil" else c["deg"] * c["n"]


# ------------------------------------------------------------- inputs


def _rmat(g, levels, deg):
    """Row-major sorted distinct edges (row << levels | column)."""
    total, part = deg << levels, 1 << 24
    keys = torch.empty(total, dtype=torch.int64, device="cuda")
    for a in range(0, total, part):
        k = keys[a:a + part]
        k.zero_()
        for _ in range(levels):
            r = torch.rand(k.numel(), device="cuda", generator=g)
            down = r >= 0.76
            right = ((r >= 0.57) & ~down) | (r >= 0.95)
            # one more bit of the row (above bit `levels`) and of the column
            k.mul_(2).add_(down.to(torch.int64) << levels).add_(right)
    return torch.unique(keys)


def _csr(c, g):
    N, kind = _rows(c), c["kind"]
    if kind == "uniform":
        col = torch.randint(0, N, (N, c["deg"]), device="cuda", generator=g).sort(dim=1).values.reshape(-1)
        ptr = torch.arange(N + 1, device="cuda") * c["deg"]
    elif kind == "rmat":
        key = _rmat(g, c["levels"], c["deg"])
        col = key & (N - 1)
        ptr = torch.searchsorted(key, torch.arange(N + 1, device="cuda") << c["levels"])
    elif kind == "stencil":
        n = c["n"]
        x = torch.arange(n, device="cuda")
        t = torch.tensor([-1, 0, 1], device="cuda")
        ok1 = ((x[:, None] + t >= 0) & (x[:, None] + t < n))  # n x 3
        ok = (ok1[:, None, None, :, None, None] & ok1[None, :, None, None, :, None]
              & ok1[None, None, :, None, None, :]).reshape(N, 27)
        off = (t[:, None, None] * n * n + t[None, :, None] * n + t[None, None, :]).reshape(27)
        col = (torch.arange(N, device="cuda")[:, None] + off)[ok]
        ptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), ok.sum(dim=1).cumsum(0)])
    else:
        u = torch.rand(N, device="cuda", generator=g, dtype=torch.float64)
        w = (1 - u) ** (-1 / 1.1) - 1
        w = torch.where(torch.rand(N, device="cuda", generator=g) < 0.3, torch.zeros_like(w), w.clamp(max=2000.0))
        ends = (w.cumsum(0) * (c["deg"] * N / float(w.sum()))).round().to(torch.int64)
        ends[-1] = c["deg"] * N
        ptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), ends])
        row = torch.repeat_interleave(torch.arange(N, device="cuda"), ptr.diff())
        col = (torch.rand(c["deg"] * N, device="cuda", generator=g, dtype=torch.float64) ** 2 * N).to(torch.int64).clamp(max=N - 1)
        col = (row * N + col).sort().values - row * N
    return ptr.to(torch.int32), col.to(torch.int32).contiguous()


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    op, N, K, L = case["op"], _rows(case), case["K"], case["L"]
    graph = case["kind"] == "rmat"

    def dense(rows, cols):
        if graph:
            return torch.randn(rows, cols, device="cuda", generator=g)
        return torch.rand(rows, cols, device="cuda", generator=g).mul_(2).sub_(1)

    ptr, col = _csr(case, g)
    vals = torch.rand(col.numel(), device="cuda", generator=g)
    s = dict(op=op, ptr=ptr, col=col, vals=vals if graph else vals.mul_(2).sub_(1))
    if K:
        s.update(C=dense(N, K), D=dense(K, N) if op == "fused_dt" else dense(N, K))
    if L:
        s["E"] = dense(N, L)
    if op == "spmmh_gemm":
        s["H"] = dense(N, L)
    if op in EPILOGUE:
        s["W"] = dense(L, case["out"])
    if op == "fused_noalloc":
        s["A"] = torch.empty(N, L, device="cuda")
    return s


def run(s):
    op, B = s["op"], (s["ptr"], s["col"], s["vals"])
    if op == "fused":
        return slnr.sparselnr_fused_sddmm_spmm(*B, s["C"], s["D"], s["E"])
    if op == "fused_noalloc":
        return slnr.sparselnr_fused_sddmm_spmm_noalloc(*B, s["C"], s["D"], s["E"], s["A"])
    if op == "fused_dt":
        return slnr.sparselnr_fused_sddmm_spmm_dt(*B, s["C"], s["D"], s["E"])
    if op == "unfused":
        return slnr.sparselnr_unfused_sddmm_spmm(*B, s["C"], s["D"], s["E"])
    if op == "sddmm":
        return slnr.sparselnr_sddmm(*B, s["C"], s["D"])
    if op == "spmm":
        return slnr.sparselnr_spmm(*B, s["E"])
    if op == "fused_gemm":
        return slnr.sparselnr_fused_sddmm_spmm_gemm(*B, s["C"], s["D"], s["E"], s["W"])
    if op == "spmm_gemm":
        return slnr.sparselnr_spmm_gemm(*B, s["E"], s["W"])
    return slnr.sparselnr_spmmh_gemm(*B, s["E"], s["H"], s["W"])


# ---------------------------------------------------- work and reference


def work(case):
    """Every array once, and the multiplications and additions of the result."""
    op, N, nnz, K, L, out = case["op"], _rows(case), _nnz(case), case["K"], case["L"], case.get("out", 0)
    words = N + 1 + 2 * nnz + 2 * N * K + N * L  # CSR; C, D; E
    flops = 2 * nnz * (K + L)
    if op == "sddmm":
        words += nnz
    elif op in EPILOGUE:
        words += L * out + N * out + (N * L if op == "spmmh_gemm" else 0)
        flops += 2 * N * L * out + (N * L if op == "spmmh_gemm" else 0)
    else:
        words += N * L + (nnz if op == "unfused" else 0)
    return {"bytes": 4 * words, "flops": flops}


def tolerance(case):
    """fp32 sums in another order, over rows of up to about 10^5 terms.  Measured over the listed cases and 14 drawn ones:
    up to 6e-7 (largest 1.1e-4) off the fp64 values, and up to 7.3e-7 (2.4e-4) between two splits of the long rows; the
    largest differences are in hub rows, whose terms cancel.  Four times that is allowed."""
    return {"rel": 3e-6, "max": 1e-3}


def exact(case, seed):
    """The same values in fp64, nonzeros in parts."""
    s = prepare(case, seed)
    op, ptr, col = s["op"], s["ptr"].long(), s["col"].long()
    N, nnz, K, L = _rows(case), s["col"].numel(), case["K"], case["L"]
    wide = lambda k: s[k].double() if k in s else None  # noqa: E731
    C, D, E, vals = wide("C"), wide("D"), wide("E"), s["vals"].double()
    if op == "fused_dt":
        D = D.t().contiguous()
    if op == "spmmh_gemm":
        E = E * wide("H")
    T = torch.zeros(N, L, dtype=torch.float64, device="cuda") if L else None
    Y = torch.empty(nnz, dtype=torch.float64, device="cuda") if K else None
    row = torch.repeat_interleave(torch.arange(N, device="cuda"), ptr.diff())
    part = max(1, (1 << 28) // max(K, L))
    for a in range(0, nnz, part):
        r, j, y = row[a:a + part], col[a:a + part], vals[a:a + part]
        if K:
            y = y * (C[r] * D[j]).sum(dim=1)
            Y[a:a + part] = y
        if L:
            T.index_add_(0, r, y[:, None] * E[j])
    if op == "sddmm":
        return Y
    if op == "unfused":
        return Y, T
    return T @ wide("W") if op in EPILOGUE else T
