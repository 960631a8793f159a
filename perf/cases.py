"""What this library is timed on: calls of its public entry points, as a program makes them.

A case is a dict of plain values.  ``listed()`` names the standing ones, ``draw`` makes more of the
same ranges; ``prepare`` builds what a program holds before the call (the sketch handle and the
data), ``run`` is one pass, ``exact`` the same result in 64 bits by plain torch.

Keys of a case: ``op`` ("cols": S A for A d x n, "rows": G S^T for G n x d, "gather": the block-row
sampling sketch, "gauss": the dense Gaussian sketch), ``dtype``, ``d``, ``n``, ``k``; for the block
sketches ``Bc``, ``Br``, ``kappa``, ``s``; ``data`` (distribution of the input); ``pad`` (elements
between the end of a row and the next row); ``chunk`` (> 0: the columns are applied in chunks of
this width into one output, as a gradient-compression pipeline hands them over).
"""
from __future__ import annotations

import math

import torch

from paper_2602_06071_amd import binding as fs
from paper_2602_06071_amd.blocks import suggest_blocks

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ELT = {"f32": 4, "bf16": 2, "f16": 2}
KINDS = {"cols": fs.KIND_BLOCKPERM, "rows": fs.KIND_BLOCKPERM, "gather": fs.KIND_BLOCKROW,
         "gauss": fs.KIND_GAUSS_DENSE}


def _case(op, dtype, d, n, k, Bc=0, Br=0, kappa=0, s=0, data="gaussian", pad=0, chunk=0, name=None):
    c = {"op": op, "dtype": dtype, "d": d, "n": n, "k": k, "Bc": Bc, "Br": Br, "kappa": kappa, "s": s,
         "data": data, "pad": pad, "chunk": chunk}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest configuration: a few thousand rows, one sketch in a loop of small problems.
        # Launches and latency.
        _case("cols", "f32", 4096, 512, 256, 512, 32, 2, 4, name="tiny"),
        # The right-hand side of sketch-and-solve: the same sketch applied to one vector.
        _case("cols", "f32", 262144, 1, 4096, 2048, 32, 4, 4, name="rhs_one_vector"),
        # The problem the quality sweep runs on: low-rank matrix plus noise, least squares.
        _case("cols", "f32", 65536, 1024, 4096, 512, 32, 4, 2, data="lowrank", name="least_squares"),
        # A tall coherent matrix (decaying spectrum, a few rows of high leverage).
        _case("cols", "f32", 262144, 256, 4096, 2048, 32, 4, 4, data="coherent", name="tall"),
        # The synthetic Gaussian matrix of the randomized-linear-algebra sweeps.
        _case("cols", "f32", 16384, 16384, 1024, 1024, 64, 4, 8, name="mid"),
        # Stacked weight matrices, heavy tails.
        _case("cols", "bf16", 65536, 8192, 4096, 2048, 128, 4, 8, data="student", name="wide"),
        # A slice of the same with an odd number of columns, as torch packs it: no row is aligned.
        _case("cols", "f16", 65536, 1531, 4096, 1024, 64, 2, 4, data="student", name="odd_columns"),
        # Per-example gradients as columns, handed over in chunks of 256 (the flagship workload).
        _case("cols", "bf16", 4194304, 1024, 8192, 4096, 8, 8, 2, data="gradient", chunk=256, name="gradient_columns"),
        # The same kind of data held examples-as-rows with a padded row stride: one batch.
        _case("rows", "bf16", 4194304, 256, 8192, 4096, 8, 8, 2, data="gradient", pad=64, name="gradient_rows"),
        # A handful of gradients of a small model, rows packed at an odd length.
        _case("rows", "f32", 1000003, 24, 2048, 3907, 8, 8, 2, data="gradient", name="few_odd_rows"),
        # The gather-only block-row sketch on the least-squares problem.
        _case("gather", "f32", 65536, 1024, 4096, 512, 32, 4, 2, data="lowrank", name="block_row"),
        # The dense Gaussian sketch on the least-squares problem.
        _case("gauss", "f32", 65536, 1024, 4096, data="lowrank", name="dense_gaussian"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choices(["cols", "rows", "gather", "gauss"], [8, 5, 1, 1])[0]
    dtype = rng.choice(["f32", "bf16", "f16"])
    elt = ELT[dtype]
    if op == "gauss":  # whole 64-row and 128-row tiles, columns a multiple of 4: what this kind takes
        d = 64 * _log_int(rng, 64, 1024)
        k = 128 * _log_int(rng, 2, 32)
        n = 4 * _log_int(rng, 8, 256)
        return _case(op, dtype, d, n, k, data="gaussian")
    while True:
        if op == "rows":
            d, n = _log_int(rng, 4096, 4194304), _log_int(rng, 1, 1024)
        else:
            d, n = _log_int(rng, 4096, 4194304), _log_int(rng, 1, 16384)
        if rng.random() < 0.6:  # round sizes, else whatever came out, odd ones among them
            d -= d % 64
            n = n if n < 8 else n - n % 8
        kappa, s = rng.choice([1, 2, 4, 8]), rng.choice([2, 4, 8])
        k = rng.choice([256, 512, 1024, 2048, 4096, 8192])
        if not (4096 <= d and 4 * k <= d <= 1024 * k and 16384 <= d * n * elt <= (4 << 30)):
            continue
        try:
            if rng.random() < 0.7:  # block sizes as the library proposes them
                Bc, Br, _ = suggest_blocks(d, k, kappa, s)
            else:                   # hand-picked larger blocks, as in the "mid" and "wide" configurations
                Br = rng.choice([32, 64, 128])
                M = k // Br
                Bc = -(-d // M)
                if kappa > M or -(-d // Bc) != M:
                    continue
        except ValueError:
            continue
        # no costlier than the listed ones, also as the dense product a matrix core would make of it
        if 2.0 * kappa * Br * d * n * (3 if dtype == "f32" else 1) > 5e11:
            continue
        data = rng.choice(["gaussian", "student", "gradient"])
        pad = rng.choice([0, 0, 0, 64]) if op == "rows" else 0
        return _case(op, dtype, d, n, k, Bc, Br, kappa, s, data, pad)


# ---- inputs -----------------------------------------------------------------------------------
def _values(data, rows, cols, g, dev):
    if data == "student":  # t with 3 degrees of freedom, unit variance
        z = torch.randn((rows, cols), generator=g, device=dev)
        q = torch.zeros((rows, cols), device=dev)
        for _ in range(3):
            q.add_(torch.randn((rows, cols), generator=g, device=dev).square_())
        return z / q.sqrt_()
    if data == "gradient":  # Laplace entries of unit variance
        u = torch.rand((rows, cols), generator=g, device=dev) - 0.5
        return torch.sign(u) * torch.log1p(u.abs_().mul_(-2.0)).clamp_(min=-80.0) * (-1.0 / math.sqrt(2.0))
    return torch.randn((rows, cols), generator=g, device=dev)


def _input(case, seed):
    """The matrix a program would hold (2-D view, unit column stride), from the seed alone."""
    dev, dt = "cuda", DTYPES[case["dtype"]]
    g = torch.Generator(device=dev).manual_seed(seed)
    d, n, data = case["d"], case["n"], case["data"]
    if data == "lowrank":  # rank 32 plus 1 % noise
        r = min(32, n)
        A = torch.randn((d, r), generator=g, device=dev) @ torch.randn((r, n), generator=g, device=dev)
        return (A / r ** 0.5 + 0.01 * torch.randn((d, n), generator=g, device=dev)).to(dt)
    if data == "coherent":  # singular values from 1 to 1e-6, sixteen rows a thousand times larger
        h = torch.Generator().manual_seed(seed)
        V = torch.linalg.qr(torch.randn((n, n), generator=h, dtype=torch.float64)).Q
        sigma = torch.pow(10.0, -6.0 * torch.arange(n, dtype=torch.float64) / max(n - 1, 1))
        W = (sigma[:, None] * V.T / math.sqrt(d)).to(dev, torch.float32)
        A = torch.randn((d, n), generator=g, device=dev) @ W
        A[torch.randperm(d, generator=h)[:16].to(dev)] *= 1.0e3
        return A.to(dt)
    rows, cols = (n, d) if case["op"] == "rows" else (d, n)
    ld = cols + case["pad"]
    buf = torch.empty((rows, ld), dtype=dt, device=dev)
    if case["pad"]:
        buf[:, cols:].zero_()
    scale = torch.ones((), device=dev)
    if data == "gradient":  # every vector with a norm of its own
        norms = torch.exp(torch.randn(n, generator=g, device=dev)) / math.sqrt(d)
        scale = norms[:, None] if case["op"] == "rows" else norms[None, :]
    step = max(1, (1 << 26) // cols)
    for r in range(0, rows, step):
        e = min(rows, r + step)
        sc = scale[r:e] if scale.dim() == 2 and scale.shape[0] == rows and rows > 1 else scale
        buf[r:e, :cols] = (_values(data, e - r, cols, g, dev) * sc).to(dt)
    return buf[:, :cols]


def prepare(case, seed):
    sketch = fs.Sketch(case["d"], case["k"], case["Bc"] or case["d"], case["Br"] or case["k"], case["kappa"] or 1,
                       case["s"] or 1, seed=seed, kind=KINDS[case["op"]])
    sketch.prepare()
    A = _input(case, seed)
    state = {"sketch": sketch, "A": A, "op": case["op"], "chunk": case["chunk"]}
    if case["chunk"]:
        state["out"] = torch.empty((case["k"], case["n"]), dtype=A.dtype, device=A.device)
    return state


def run(state):
    sketch, A, chunk = state["sketch"], state["A"], state["chunk"]
    if state["op"] == "rows":
        return sketch.apply_rows(A)
    if not chunk:
        return sketch.apply(A)
    out = state["out"]
    for j in range(0, A.shape[1], chunk):
        sketch.apply(A[:, j:j + chunk], out[:, j:j + chunk])
    return out


# ---- accounting -------------------------------------------------------------------------------
def work(case):
    d, n, k, elt = case["d"], case["n"], case["k"], ELT[case["dtype"]]
    out = k * n * elt
    if case["op"] == "gauss":  # the matrix is read too
        return {"bytes": d * n * elt + k * d * elt + out, "flops": 2.0 * k * d * n}
    nnz_row = case["kappa"] * case["s"]
    if case["op"] == "gather":  # the input rows that some output row samples
        seen = d * -math.expm1(-k * nnz_row / d)
        return {"bytes": int(seen) * n * elt + out, "flops": float(k) * nnz_row * n}
    return {"bytes": d * n * elt + out, "flops": float(d) * nnz_row * n}


def tolerance(case):
    # Measured against the 64-bit result, in 2-norm: 32-bit sums of some hundred to some thousand
    # terms 1e-7 to 5e-7, the dense sketch's sums over all d rows up to 6e-6; the 16-bit types round
    # the result once (bf16 1.7e-3, half 2.1e-4).
    if case["dtype"] == "f32":
        return {"rel": 2.5e-5 if case["op"] == "gauss" else 2e-6}
    return {"rel": {"bf16": 7e-3, "f16": 9e-4}[case["dtype"]]}


# ---- the same in 64 bits ------------------------------------------------------------------------
_MASK = 0xFFFFFFFF
_C1, _C2, _C3 = 0x6A09E667, 0xBB67AE85, 0x3C6EF373


def _mul32(x, c):
    return ((x * (c & 0xFFFF)) + (((x * (c >> 16)) & 0xFFFF) << 16)) & _MASK


def _mix(x):
    """The 32-bit mixing hash on int64 tensors (or Python integers) that hold 32-bit words."""
    x = x ^ (x >> 16)
    x = _mul32(x, _C1)
    x = x ^ (x >> 15)
    x = _mul32(x, _C2)
    x = x ^ (x >> 16)
    x = _mul32(x, _C3)
    return x ^ (x >> 15)


def _keys(seed):
    k0 = _mix((seed & _MASK) ^ _C1)
    return k0, _mix(((seed >> 32) & _MASK) ^ k0 ^ _C2)


def _wiring(M, key1):
    if M == 1:
        return 0, 0
    L, m, q = 1, M, 2
    while m > 1:
        if m % q == 0:
            L *= q
            while m % q == 0:
                m //= q
        q += 1
    if M % 4 == 0:
        L = math.lcm(L, 4)
    a = (1 + L * (_mix(key1 ^ 1) % (M // L))) % M
    b = _mix(key1 ^ 2) % M
    while math.gcd(b, M) != 1:
        b = (b + 1) % M
    return a, b


def _blocks64(case, A, rows, count):
    """The rows `rows` (count blocks of Bc input coordinates) of the input as count x Bc x n doubles."""
    d, Bc = case["d"], case["Bc"]
    idx = rows.clamp(max=d - 1)
    if case["op"] == "rows":
        X = A.index_select(1, idx).double().t().contiguous()
    else:
        X = A.index_select(0, idx).double()
    if int(rows[-1]) >= d or bool((rows >= d).any()):
        X[rows >= d] = 0.0
    return X.view(count, Bc, -1)


def exact(case, seed):
    A = _input(case, seed)
    dev, d, n, k = A.device, case["d"], case["n"], case["k"]
    _, key1 = _keys(seed)
    if case["op"] == "gauss":
        out = torch.empty((k, n), dtype=torch.float64, device=dev)
        A64 = A.double()
        step = max(1, (1 << 26) // d)
        for r in range(0, k, step):
            e = min(k, r + step)
            idx = torch.arange(r * d, e * d, device=dev, dtype=torch.int64)
            c = _mix((idx & _MASK) ^ _mix((idx >> 32) ^ key1 ^ _C1))
            u1 = ((_mix(c ^ 0x9E3779B9) >> 8) + 1).double() / 16777216.0
            u2 = (_mix(c ^ 0x85EBCA6B) >> 8).double() / 16777216.0
            S = torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2) / math.sqrt(k)
            out[r:e] = S.float().to(A.dtype).double().view(e - r, d) @ A64  # the matrix as its type holds it
        return out
    Bc, Br, kappa, s = case["Bc"], case["Br"], case["kappa"], case["s"]
    M = k // Br
    a, b = _wiring(M, key1)
    out = torch.zeros((M, Br, n), dtype=torch.float64, device=dev)
    unit = torch.tensor([next((c + j) % Br for j in range(Br) if math.gcd((c + j) % Br, Br) == 1) if Br > 1 else 0
                         for c in range(Br)], device=dev, dtype=torch.int64)
    u = torch.arange(Bc, device=dev, dtype=torch.int64)
    G = max(1, min(M, (1 << 27) // (Bc * max(n, Br))))  # blocks at a time: about 1 GiB of doubles
    h_all = torch.arange(M, device=dev, dtype=torch.int64)
    for _ in range(kappa):
        h_all = (a * h_all + b) % M
        for g0 in range(0, M, G):
            h = h_all[g0:g0 + G]
            cnt = h.numel()
            g = torch.arange(g0, g0 + cnt, device=dev, dtype=torch.int64)
            key = _mix(key1 ^ _mix((g * M + h + _C3) & _MASK))
            phi = torch.zeros((cnt, Br, Bc), dtype=torch.float64, device=dev)
            if case["op"] == "gather":
                r = torch.arange(Br, device=dev, dtype=torch.int64)
                for t in range(s):
                    w = _mix(key[:, None] ^ _C1 ^ (r * 32 + t)[None, :])
                    sign = 1.0 - 2.0 * (_mix(w ^ _C2) & 1).double()
                    phi.scatter_add_(2, (w % Bc)[:, :, None], sign[:, :, None])
            else:
                h1 = _mix(key[:, None] ^ u[None, :])
                h2 = _mix(h1 ^ _C2)
                shift, stride = (h1 & 0xFFFF) % Br, unit[(h1 >> 16) % Br]
                for i in range(s):
                    row = (shift + i * stride) % Br
                    sign = 1.0 - 2.0 * ((h2 >> i) & 1).double()
                    phi.scatter_(1, row[:, None, :], sign[:, None, :])
            rows = (h[:, None] * Bc + u[None, :]).reshape(-1)
            out[g0:g0 + cnt] += torch.bmm(phi, _blocks64(case, A, rows, cnt))
    scale = 1.0 / math.sqrt(kappa * s)
    if case["op"] == "gather":
        scale *= math.sqrt(d / k)
    out = (out * scale).view(k, n)
    return out.t().contiguous() if case["op"] == "rows" else out
