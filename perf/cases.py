"""The work that users of this framework have it do, case by case: the matrix
multiplication query forward and with its adjoint (FP64 and residue forms),
group-by aggregates over relations with duplicate cells, the paper's Q1 and
Q3 queries with their dictionaries, the three-way join Q2, and the
matrix-to-table conversion.  Each case goes through the functions of
paper_2112_07552_amd.ops as a program calls them, on tables that are already
on the GPU.

  listed()            the fixed cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) the tables in GPU memory
  run(state)          one pass; its outputs
  work(case)          bytes and floating-point operations a pass cannot do without
  exact(case, seed)   the same outputs from plain torch in 64 bits
"""
import math

import torch

from paper_2112_07552_amd import ops
from paper_2112_07552_amd import workloads as wl


def _mm(name, M, K, N, values="uniform", dtype="f64", precision="fp64", step=False,
        checkpoint=False):
    return {"name": name, "kind": "mm", "M": M, "K": K, "N": N, "values": values, "dtype": dtype,
            "precision": precision, "step": step, "checkpoint": checkpoint}


def listed():
    return [
        # one interactive query over small tables: launches and host time
        _mm("fwd_2pow14", 128, 128, 128),
        # an ordinary query: 2^20 records per table
        _mm("fwd_2pow20", 1024, 1024, 1024),
        # a differentiable layer on 2^24-record tables, FP64
        _mm("step_2pow24", 4096, 4096, 4096, step=True),
        # the same in the residue form, values over eight decades
        _mm("step_crt_2pow24", 4096, 4096, 4096, values="loguniform", precision="crt_i8",
            step=True),
        # the largest: 2^28 FP32 records per table, encodings rebuilt in backward
        _mm("step_crt_2pow28", 16384, 16384, 16384, values="mixture", dtype="f32",
            precision="crt_i8", step=True, checkpoint=True),
        # SUM and COUNT per group pair over tables with repeated (group, key)
        # cells, no extent a multiple of anything
        {"name": "groupby_duplicates", "kind": "groupby", "n": 2_000_003, "M": 1500, "K": 2051,
         "N": 2777, "dtype": "f32", "count": True},
        # Q1, the natural join of two ID columns with few distinct values ...
        {"name": "q1_32_ids", "kind": "q1", "n": 16384, "ids": 32},
        # ... and with about one partner per tuple
        {"name": "q1_2pow20_ids", "kind": "q1", "n": 16384, "ids": 1 << 20},
        # Q3, an aggregate over a join grouped by a value column: long tables
        # with few keys, and shorter ones with many
        {"name": "q3_2pow24", "kind": "q3", "n": 1 << 24, "ids": 32, "groups": 32},
        {"name": "q3_many_ids", "kind": "q3", "n": 1_000_000, "ids": 100_000, "groups": 500},
        # Q2, the three-way join
        {"name": "join3_4096", "kind": "join3", "n": 4096, "ids": 512},
        # the table of a sparse result matrix
        {"name": "nonzero_8192", "kind": "nonzero", "rows": 8192, "cols": 8192, "density": 0.01},
    ]


def _between(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["fwd", "step", "step_crt", "groupby", "q1", "q3", "join3", "nonzero"])
    if kind in ("fwd", "step"):
        lo = 64 if kind == "fwd" else 256
        c = _mm("", *(_between(rng, lo, 4096) for _ in range(3)),
                values=rng.choice(["uniform", "loguniform", "mixture"]),
                dtype=rng.choice(["f64", "f32"]), step=kind == "step",
                checkpoint=kind == "step" and rng.random() < 0.3)
    elif kind == "step_crt":
        c = _mm("", *(_between(rng, 1024, 12288) for _ in range(3)),
                values=rng.choice(["uniform", "loguniform", "mixture"]),
                dtype=rng.choice(["f64", "f32"]), precision="crt_i8", step=True,
                checkpoint=rng.random() < 0.5)
    elif kind == "groupby":
        c = {"kind": kind, "n": _between(rng, 10_000, 4_000_000), "M": _between(rng, 100, 4000),
             "K": _between(rng, 100, 4000), "N": _between(rng, 100, 4000),
             "dtype": rng.choice(["f64", "f32"]), "count": rng.random() < 0.5}
    elif kind == "q1":
        c = {"kind": kind, "n": _between(rng, 1000, 16384), "ids": _between(rng, 16, 1 << 20)}
    elif kind == "q3":
        c = {"kind": kind, "n": _between(rng, 4096, 1 << 24), "ids": _between(rng, 16, 200_000),
             "groups": _between(rng, 1, 1000)}
    elif kind == "join3":
        n = _between(rng, 500, 4096)
        c = {"kind": kind, "n": n, "ids": _between(rng, max(1, n // 8), n)}
    else:
        c = {"kind": kind, "rows": _between(rng, 300, 9000), "cols": _between(rng, 300, 9000),
             "density": round(math.exp(rng.uniform(math.log(1e-3), math.log(0.2))), 6)}
    c.pop("name", None)
    return c


_DTYPE = {"f64": torch.float64, "f32": torch.float32}


def prepare(case, seed):
    dev = torch.device("cuda:0")
    kind = case["kind"]
    s = {"case": case}
    if kind == "mm":
        M, K, N = case["M"], case["K"], case["N"]
        A, B = wl.mm_query(M, K, N, seed, values=case["values"], device=dev,
                           dtype=_DTYPE[case["dtype"]])
        s["A"], s["B"] = A, B
        if case["step"]:
            s["W"] = wl.draw_values("uniform", M * N, seed + 1000, 0, device=dev).reshape(M, N)
            s["av"] = A.val.requires_grad_(True)
            s["bv"] = B.val.requires_grad_(True)
    elif kind == "groupby":
        dt = _DTYPE[case["dtype"]]
        s["A"] = wl.random_relation(case["n"], case["M"], case["K"], seed, 1, device=dev, dtype=dt)
        s["B"] = wl.random_relation(case["n"], case["N"], case["K"], seed, 2, device=dev, dtype=dt)
    elif kind in ("q1", "q3"):
        n = case["n"]
        s["ida"] = wl.id_column(n, case["ids"], seed, 1, device=dev)
        s["idb"] = wl.id_column(n, case["ids"], seed, 2, device=dev)
        if kind == "q1":
            s["tuples"] = torch.arange(n, dtype=torch.int32, device=dev)
        else:
            s["bval"] = wl.id_column(n, case["groups"], seed + 1, 7, device=dev)
            s["av"] = wl.draw_values("uniform", n, seed, 3, device=dev)
            s["none"] = s["ida"][:0]
    elif kind == "join3":
        # every ID the same number of times (give or take one), in random
        # order, so that all tables of one case join to as many tuples
        n, ids = case["n"], case["ids"]
        pool = wl.hash_counter(wl.stream_key(seed, 0), torch.arange(ids, device=dev))
        for tag, col in enumerate(("a1", "b1", "b2", "c2"), 1):
            if col == "b2":
                # spread over each ID of b1 alike
                at = torch.arange(n, device=dev) // ids + torch.arange(n, device=dev)
                order = wl.feistel_permute(torch.arange(n, device=dev), n, seed, 2)
                s[col] = pool[at[order] % ids]
            else:
                s[col] = pool[wl.feistel_permute(torch.arange(n, device=dev), n, seed, tag) % ids]
    else:
        # a fixed number of nonzero cells at random places
        rows, cols = case["rows"], case["cols"]
        count = max(1, int(rows * cols * case["density"]))
        v = wl.draw_values("uniform", count, seed, 5, device=dev)
        v[v == 0] = 1.0
        Z = torch.zeros(rows * cols, dtype=torch.float64, device=dev)
        Z[wl.feistel_permute(torch.arange(count, device=dev), rows * cols, seed, 1)] = v
        s["Z"] = Z.reshape(rows, cols)
        s["map"] = (torch.arange(cols, dtype=torch.int32, device=dev) * 7 + seed) % 1009
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mm":
        A, B = s["A"], s["B"]
        M, K, N = case["M"], case["K"], case["N"]
        tol = 1e-12 if case["precision"] != "fp64" else 0.0
        if not case["step"]:
            C, _, _ = ops.join_agg_fwd(A.group, A.key, A.val, B.key, B.group, B.val, M, K, N,
                                       case["precision"], tol, unique=True)
            return C
        C = ops.join_agg(A.group, A.key, s["av"], B.key, B.group, s["bv"], M, K, N,
                         case["precision"], tol, unique=True, checkpoint=case["checkpoint"])
        dA, dB = torch.autograd.grad(C, (s["av"], s["bv"]), s["W"])
        return C, dA, dB
    if kind == "groupby":
        A, B = s["A"], s["B"]
        C, count, _ = ops.join_agg_fwd(A.group, A.key, A.val, B.key, B.group, B.val, case["M"],
                                       case["K"], case["N"], with_count=case["count"])
        return (C, count) if case["count"] else C
    if kind == "q1":
        t, n = s["tuples"], case["n"]
        d, ka, kb = ops.dict_encode(s["ida"], s["idb"])
        C, _ = ops.join_agg_auto(t, ka, None, kb, t, None, n, d.numel(), n, unique=True)
        return C
    if kind == "q3":
        d, ka, kb = ops.dict_encode(s["ida"], s["idb"])
        gd, g, _ = ops.dict_encode(s["bval"], s["none"])
        c, count, _ = ops.join_agg_row(ka, s["av"], kb, g, None, d.numel(), gd.numel(),
                                       with_count=True)
        return gd, c, count, d, ka, kb
    if kind == "join3":
        return ops.join3(s["a1"], s["b1"], s["b2"], s["c2"])
    return ops.nonzero(s["Z"], col_map=s["map"])


def work(case):
    kind = case["kind"]
    if kind == "mm":
        M, K, N = case["M"], case["K"], case["N"]
        v = 8 if case["dtype"] == "f64" else 4
        b = (M * K + K * N) * (8 + v) + 8 * M * N
        f = 2 * M * K * N
        if case["step"]:
            # W in, one gradient per record out; the two products of the adjoint
            b += 8 * M * N + (M * K + K * N) * v
            f *= 3
        return {"bytes": b, "flops": f}
    if kind == "groupby":
        M, K, N = case["M"], case["K"], case["N"]
        v = 8 if case["dtype"] == "f64" else 4
        return {"bytes": 2 * case["n"] * (8 + v) + M * N * (12 if case["count"] else 8),
                "flops": 2 * M * K * N * (2 if case["count"] else 1)}
    n = case.get("n", 0)
    if kind == "q1":
        return {"bytes": 16 * n + 8 * n * n, "flops": 0}
    if kind == "q3":
        # three 8-byte columns and the values in, two code columns out
        return {"bytes": 4 * 8 * n + 2 * 4 * n, "flops": 2 * n}
    if kind == "join3":
        pairs = n * n / case["ids"]
        return {"bytes": 32 * n + 8 * pairs * n + 8 * pairs, "flops": 0}
    cells = case["rows"] * case["cols"]
    return {"bytes": 8 * cells + 12 * cells * case["density"], "flops": 0}


# ------------------------------------------------------------ 64-bit results


def _cut(Z, dim, bits):
    """Z = scale * (q0 2^-bits + q1 2^-2bits + q2 2^-3bits), q integers."""
    _, e = torch.frexp(Z.abs().amax(dim, keepdim=True))
    r = torch.ldexp(Z, -e)
    q = []
    for _ in range(3):
        r = r * 2.0 ** bits
        q.append(torch.round(r))
        r = r - q[-1]
    return q, e


def _matmul(X, Y):
    """X @ Y in FP64 with exact partial products: both operands are cut into
    integers short enough that every sum of a product stays below 2^53."""
    bits = (52 - math.ceil(math.log2(max(2, X.shape[1])))) // 2
    (xs, ex), (ys, ey) = _cut(X, 1, bits), _cut(Y, 0, bits)
    total = None
    for d in (2, 1, 0):  # the smallest products first
        part = sum(torch.matmul(xs[i], ys[d - i]) for i in range(d + 1))
        part = part * 2.0 ** (-bits * (d + 2))
        total = part if total is None else total + part
    return torch.ldexp(torch.ldexp(total, ex), ey)


def _dense(row, col, val, rows, cols):
    at = row.long() * cols + col.long()
    Z = torch.zeros(rows * cols, dtype=torch.float64, device=row.device)
    v = torch.ones(at.numel(), dtype=torch.float64, device=row.device) if val is None else \
        val.detach().double()
    return Z.index_add_(0, at, v).reshape(rows, cols)


def _by_group(values, group, groups):
    """Sums of `values` per group, each by torch's pairwise summation."""
    order = torch.argsort(group, stable=True)
    sizes = torch.bincount(group, minlength=groups).tolist()
    return torch.stack([p.sum() for p in torch.split(values[order], sizes)])


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    with torch.no_grad():
        if kind == "mm":
            M, K, N = case["M"], case["K"], case["N"]
            A, B = s["A"], s["B"]
            X = _dense(A.group, A.key, A.val, M, K)
            Y = _dense(B.key, B.group, B.val, K, N)
            C = _matmul(X, Y)
            if not case["step"]:
                return C
            dX = _matmul(s["W"], Y.t().contiguous())
            dA = dX.reshape(-1)[A.group.long() * K + A.key.long()]
            del dX
            dY = _matmul(X.t().contiguous(), s["W"])
            dB = dY.reshape(-1)[B.key.long() * N + B.group.long()]
            return C, dA, dB
        if kind == "groupby":
            M, K, N = case["M"], case["K"], case["N"]
            A, B = s["A"], s["B"]
            C = _matmul(_dense(A.group, A.key, A.val, M, K), _dense(B.key, B.group, B.val, K, N))
            if not case["count"]:
                return C
            count = torch.matmul(_dense(A.group, A.key, None, M, K),
                                 _dense(B.key, B.group, None, K, N))
            return C, count.to(torch.int32)
        if kind == "q1":
            return (s["ida"][:, None] == s["idb"][None, :]).double()
        if kind == "q3":
            d, codes = torch.unique(torch.cat([s["ida"], s["idb"]]), return_inverse=True)
            ka, kb = codes[:case["n"]], codes[case["n"]:]
            gd, g = torch.unique(s["bval"], return_inverse=True)
            hist = torch.zeros(d.numel(), dtype=torch.float64, device=ka.device)
            hist = _by_group(s["av"], ka, d.numel()) if d.numel() <= 4096 else \
                hist.index_add_(0, ka, s["av"])
            c = _by_group(hist[kb], g, gd.numel())
            count = torch.zeros(gd.numel(), dtype=torch.int64, device=ka.device)
            count.index_add_(0, g, torch.bincount(ka, minlength=d.numel())[kb])
            return gd, c, count, d, ka.int(), kb.int()
        if kind == "join3":
            pa, pb = torch.nonzero(s["a1"][:, None] == s["b1"][None, :], as_tuple=True)
            C3 = (s["b2"][pb][:, None] == s["c2"][None, :]).double()
            return pa.int(), pb.int(), C3
        r, c = torch.nonzero(s["Z"], as_tuple=True)
        return r.int(), c.int(), s["map"][c]
