"""Timed cases of the framework: products, their consumers and their gradients, each through its public entry points.

A case is a dict of plain values; ``kind`` names the program it stands for:

  oneshot        spgemm(A, B): workspaces, symbolic pass, plan, product, concatenation, all in the call
  product        a kept Engine: symbolic pass, batch plan, product (in layers or semirings), rows sorted
  topk           a kept Engine whose batches are pruned as they are formed (Markov clustering's expansion step)
  aat            C = A A^T: transpose, then the product (overlap and similarity detection)
  train          SpGEMMFn forward, loss 0.5 ||C||^2, backward through torch.autograd
  grad           a kept Backward: dA and dB for a given dC on a fixed pattern
  batched        a captured forward of many small products, rows sorted
  batched_train  a captured forward and fused backward of many products, dC = C
  prune          threshold and top-k pruning of a matrix at hand

The hash kernels write the rows of a column in table order, so programs that hand a matrix on ask for sorted rows;
``topk`` sorts only the few entries that it keeps.
"""
from __future__ import annotations

import json
import math

import torch

import paper_2010_08526_amd as S
import paper_2010_08526_amd.batched as Bt

DTYPE = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # the smallest call: one product of two small matrices, everything formed in the call
        {"name": "oneshot_512", "kind": "oneshot", "m": 512, "k": 512, "n": 512, "da": 4, "db": 4, "dtype": "f32"},
        # Erdos-Renyi 4096, 8 per column, float64, on a kept engine
        {"name": "er4096_f64", "kind": "product", "graph": "er", "n": 4096, "d": 8, "layers": 1, "batches": 1,
         "semiring": "plus_times", "dtype": "f64"},
        # one step of all-pairs shortest paths on a scale-free graph
        {"name": "rmat13_minplus", "kind": "product", "graph": "rmat", "scale": 13, "ef": 16, "layers": 1,
         "batches": 1, "semiring": "min_plus", "dtype": "f64"},
        # squaring a scale-free graph, sorted rows, one layer
        {"name": "rmat16_sorted", "kind": "product", "graph": "rmat", "scale": 16, "ef": 16, "layers": 1,
         "batches": 1, "semiring": "plus_times", "dtype": "f32"},
        # protein-similarity-like power law in inner-dimension layers, merged, in memory-bounded batches
        {"name": "protein60k_layers", "kind": "product", "graph": "protein", "n": 60000, "mean": 50, "layers": 8,
         "batches": 3, "semiring": "plus_times", "dtype": "f32"},
        # the expansion step of Markov clustering: four batches, each pruned to 100 entries per column
        {"name": "rmat18_topk", "kind": "topk", "graph": "rmat", "scale": 18, "ef": 16, "batches": 4, "keep": 100,
         "dtype": "f32"},
        # k-mer-like overlap detection: many inner columns of two entries
        {"name": "aat_100k", "kind": "aat", "m": 100003, "k": 5000000, "d": 2, "dtype": "f32"},
        # a training step with both operands learned
        {"name": "train_er262k", "kind": "train", "m": 262144, "k": 262144, "n": 262144, "da": 16, "db": 16,
         "dtype": "f32"},
        # gradients on a fixed pattern, rectangular operands of odd sizes, float64
        {"name": "grad_rect_f64", "kind": "grad", "m": 50021, "k": 30011, "n": 70001, "da": 20, "db": 12,
         "dtype": "f64"},
        # serving many small products by one graph replay: latency and launches
        {"name": "batched_64", "kind": "batched", "count": 64, "nmin": 64, "nmax": 1024, "dmin": 4, "dmax": 16,
         "dtype": "f32"},
        # a training step over uneven products by one graph replay
        {"name": "batched_train_256", "kind": "batched_train", "count": 256, "nmin": 256, "nmax": 65536, "dmin": 4,
         "dmax": 32, "dtype": "f32"},
        # pruning a matrix at hand, columns from empty to a few hundred thousand entries
        {"name": "prune_200m", "kind": "prune", "m": 1000003, "n": 20011, "mean": 10000, "keep": 100,
         "threshold": 0.25, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["oneshot", "product", "product", "product", "topk", "aat", "train", "grad", "batched",
                       "batched_train", "prune"])
    dt = rng.choice(["f32", "f32", "f64"])
    if kind == "oneshot":
        return {"kind": kind, "m": _log(rng, 64, 4096), "k": _log(rng, 64, 4096), "n": _log(rng, 64, 4096),
                "da": rng.randint(2, 8), "db": rng.randint(2, 8), "dtype": dt}
    if kind == "product":
        sr = rng.choice(["plus_times", "plus_times", "min_plus", "or_and"])
        graph = rng.choice(["er", "rmat", "protein"])
        layers = rng.choice([1, 1, rng.randint(2, 16)])
        c = {"kind": kind, "graph": graph, "layers": layers, "batches": rng.randint(1, 4), "semiring": sr, "dtype": dt}
        if graph == "er":
            c.update(n=_log(rng, 1000, 262144), d=rng.randint(4, 32))
        elif graph == "rmat":
            c.update(scale=rng.randint(11, 15), ef=rng.randint(4, 16))
        else:
            c.update(n=_log(rng, 3000, 50000), mean=rng.randint(15, 50))
        return c
    if kind == "topk":
        return {"kind": kind, "graph": "rmat", "scale": rng.randint(12, 17), "ef": rng.randint(6, 16),
                "batches": rng.randint(1, 8), "keep": _log(rng, 10, 1000), "dtype": dt}
    if kind == "aat":
        k = _log(rng, 20000, 5000000)
        return {"kind": kind, "m": _log(rng, max(1000, k // 60), max(20000, 2 * k)), "k": k, "d": 2, "dtype": dt}
    if kind in ("train", "grad"):
        big = 262144 if kind == "train" else 100000
        return {"kind": kind, "m": _log(rng, 2000, big), "k": _log(rng, 2000, big), "n": _log(rng, 2000, big),
                "da": rng.randint(4, 24), "db": rng.randint(4, 16), "dtype": dt}
    if kind == "batched":
        return {"kind": kind, "count": _log(rng, 8, 256), "nmin": 32, "nmax": _log(rng, 128, 2048), "dmin": 2,
                "dmax": rng.randint(4, 16), "dtype": dt}
    if kind == "batched_train":
        return {"kind": kind, "count": _log(rng, 16, 200), "nmin": 256, "nmax": _log(rng, 2048, 65536), "dmin": 4,
                "dmax": rng.randint(8, 32), "dtype": dt}
    return {"kind": kind, "m": _log(rng, 2000, 2000000), "n": _log(rng, 500, 40000), "mean": _log(rng, 50, 5000),
            "keep": _log(rng, 1, 1000), "threshold": rng.choice([0.0, 0.25, 0.9]), "dtype": dt}


# ------------------------------------------------------------------ inputs
# A case's structure up to numbering is its own (drawn from PATTERN); the seed gives the numbering of rows, columns and
# inner indices (rotated by random offsets, so that hubs stay neighbours) and the values.
PATTERN = 201008526


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _turns(g, *sizes):
    """A random rotation for each index range."""
    return [int(torch.randint(0, s, (1,), generator=g, device="cuda")) for s in sizes]


def _rand(n, g):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _values(n, dtype, g, dist="uniform"):
    if dist == "normal":
        return torch.randn(n, generator=g, device="cuda", dtype=torch.float64).to(dtype)
    return (1.0 - _rand(n, g)).to(dtype)


def _from_keys(keys, m, n, dtype, g, dist="uniform"):
    """CSC of the distinct column-major keys col * m + row, with new values."""
    keys = torch.unique(keys)
    col = keys // m
    cp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    cp[1:] = torch.cumsum(torch.bincount(col, minlength=n), 0)
    return S.CSC(m, n, cp, (keys - col * m).to(torch.int32), _values(keys.numel(), dtype, g, dist))


def _er(m, n, d, dtype, g, turns, dist="uniform", tag=0):
    """About d distinct uniform rows in each of n columns; rows and columns turned."""
    d = min(d, m)
    row = torch.randint(0, m, (n * d,), generator=_gen(PATTERN + tag), device="cuda")
    col = torch.arange(n, device="cuda").repeat_interleave(d)
    return _from_keys((col + turns[1]) % n * m + (row + turns[0]) % m, m, n, dtype, g, dist)


def _rmat(scale, ef, dtype, g):
    """Symmetrized R-MAT graph, quadrant probabilities .57, .19, .19."""
    n, gp = 1 << scale, _gen(PATTERN)
    r = torch.zeros(ef * n, dtype=torch.int64, device="cuda")
    c = torch.zeros_like(r)
    for _ in range(scale):
        u = _rand(r.numel(), gp)
        r = 2 * r + (u >= 0.76)
        c = 2 * c + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    t = _turns(g, n)[0]
    r, c = (r + t) % n, (c + t) % n
    return _from_keys(torch.cat([c * n + r, r * n + c]), n, n, dtype, g)


def _protein(n, mean, dtype, g):
    """Symmetric Chung-Lu graph, degrees from a power law x^-2.1 capped at 5000, columns of sum one."""
    lo, hi, cap = 1e-6, float(mean), 5000.0
    for _ in range(60):  # the cut-off that gives the mean degree
        x = 0.5 * (lo + hi)
        got = 11.0 * (x ** -0.1 - cap ** -0.1) / (x ** -1.1 - cap ** -1.1)
        lo, hi = (x, hi) if got < mean else (lo, x)
    gp = _gen(PATTERN)
    w = (lo ** -1.1 - _rand(n, gp) * (lo ** -1.1 - cap ** -1.1)) ** (-1 / 1.1)
    cdf = torch.cumsum(w, 0) / w.sum()
    ne, t = n * mean // 2, _turns(g, n)[0]
    i = torch.searchsorted(cdf, _rand(ne, gp)).clamp_(max=n - 1)
    j = torch.searchsorted(cdf, _rand(ne, gp)).clamp_(max=n - 1)
    i, j = (i[i != j] + t) % n, (j[i != j] + t) % n
    A = _from_keys(torch.cat([i * n + j, j * n + i]), n, n, torch.float64, g)
    col = torch.arange(n, device="cuda").repeat_interleave(A.colptr[1:] - A.colptr[:-1])
    s = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, col, A.values)
    return S.CSC(n, n, A.colptr, A.rowidx, (A.values / s[col]).to(dtype))


def _graph(case, g):
    dt = DTYPE[case["dtype"]]
    if case["graph"] == "er":
        return _er(case["n"], case["n"], case["d"], dt, g, _turns(g, case["n"]) * 2)
    if case["graph"] == "rmat":
        return _rmat(case["scale"], case["ef"], dt, g)
    return _protein(case["n"], case["mean"], dt, g)


def _batch(case, g):
    """Two packed block-diagonal operands of uneven square instances, and the instances' sizes."""
    q, dt = case["count"], DTYPE[case["dtype"]]
    gp = _gen(PATTERN)
    a, b = math.log(case["nmin"]), math.log(case["nmax"])
    ns = torch.exp(a + (b - a) * _rand(q, gp)).round().to(torch.int64)
    off = torch.cumsum(ns, 0) - ns
    m = int(ns.sum())
    tm, tk, tn = ((_rand(q, g) * ns).to(torch.int64) for _ in range(3))
    mats = []
    for tr, tc in ((tm, tk), (tk, tn)):
        d = torch.randint(case["dmin"], case["dmax"] + 1, (q,), generator=gp, device="cuda")
        per = torch.repeat_interleave(d, ns)
        inst = torch.repeat_interleave(torch.arange(q, device="cuda"), ns).repeat_interleave(per)
        col = torch.repeat_interleave(torch.arange(m, device="cuda"), per) - off[inst]
        row = (_rand(col.numel(), gp) * ns[inst]).to(torch.int64)
        col = off[inst] + (col + tc[inst]) % ns[inst]
        row = off[inst] + (row + tr[inst]) % ns[inst]
        mats.append(_from_keys(col * m + row, m, m, dt, g))
    return mats[0], mats[1], ns.tolist()


def _operands(case, g):
    """(A, B) of the product kinds."""
    dt, kind = DTYPE[case["dtype"]], case["kind"]
    if kind in ("product", "topk"):
        A = _graph(case, g)
        return A, A
    if kind in ("batched", "batched_train"):
        return _batch(case, g)[:2]
    if kind == "aat":
        A = _left(case, g)
        return A, S.transpose(A, perm=False)[0]
    dist = "normal" if kind in ("train", "grad") else "uniform"
    tm, tk, tn = _turns(g, case["m"], case["k"], case["n"])
    return (_er(case["m"], case["k"], case["da"], dt, g, (tm, tk), dist),
            _er(case["k"], case["n"], case["db"], dt, g, (tk, tn), dist, 1))


def _left(case, g):
    """A of A A^T."""
    return _er(case["m"], case["k"], case["d"], DTYPE[case["dtype"]], g, _turns(g, case["m"], case["k"]))


def _prune_input(case, g):
    """Columns of exponentially distributed length, distinct rows in scattered order, values in steps (so with ties):
    a column of a given length holds the same values whatever the seed, in another order."""
    m, n = case["m"], case["n"]
    lens = (-case["mean"] * torch.log(1.0 - _rand(n, _gen(PATTERN)))).to(torch.int64).clamp_(max=m)
    lens = torch.roll(lens, _turns(g, n)[0])
    cp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    cp[1:] = torch.cumsum(lens, 0)
    nnz = int(cp[-1])
    # distinct rows: position p of column j holds (start_j + p * step) mod m, step coprime to m
    step = next(s for s in range(int(0.618 * m) | 1, 2 * m, 2) if math.gcd(s, m) == 1)
    start = torch.randint(0, m, (n,), generator=g, device="cuda")
    col = torch.repeat_interleave(torch.arange(n, device="cuda"), lens)
    p = torch.arange(nnz, device="cuda") - cp[col]
    row = ((start[col] + p * step) % m).to(torch.int32)
    turn = torch.randint(0, 1 << 40, (n,), generator=g, device="cuda")
    rank = (p * 1000003 + turn[col]) % lens[col]  # a prime above every length: each rank once
    v = torch.round(((rank + 0.5) / lens[col]) ** 4 * 65536) / 65536
    return S.CSC(m, n, cp, row, v.to(DTYPE[case["dtype"]]))


def _set_batches(eng, plan, case):
    """An HBM budget that splits the product into about the wanted number of batches."""
    if case["batches"] <= 1:
        return
    r = 4 + eng.vbytes
    u = plan.nnz_host[-1].sum() * (2 if eng.sorted_output else 1)
    part = plan.nnz_host[:-1].sum() if eng.L > 1 else 0
    per_col = 8 * (eng.L + 1) if eng.L > 1 else 8
    total = int(r * (u + part)) + per_col * eng.B.ncols
    largest = int((r * (plan.nnz_host[-1] * (2 if eng.sorted_output else 1) +
                        (plan.nnz_host[:-1].sum(0) if eng.L > 1 else 0)) + per_col).max())
    eng.budget_bytes = eng.input_bytes + eng.reserve_bytes + max(int(1.02 * total / case["batches"]), largest) + 4096


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "prune":
        C = _prune_input(case, g)
        return {"case": case, "C": C, "ws": S.alloc_workspace(S.workspace_size(S.OP_PRUNE, C))}
    if kind == "aat":
        return {"case": case, "A": _left(case, g)}
    A, B = _operands(case, g)
    st = {"case": case, "A": A, "B": B}
    if kind == "product":
        st["eng"] = S.Engine(A, B, case["layers"], semiring=case["semiring"], sorted_output=True)
        _set_batches(st["eng"], st["eng"].plan(), case)
    elif kind == "topk":
        st["eng"] = S.Engine(A, B)
        _set_batches(st["eng"], st["eng"].plan(), case)
        st["ws"] = None
    elif kind == "train":
        st["a"] = A.values.clone().requires_grad_(True)
        st["b"] = B.values.clone().requires_grad_(True)
    elif kind == "grad":
        C = S.spgemm(A, B, sorted_output=True)
        st["dC"] = _values(C.nnz, C.values.dtype, g, "normal")
        st["bw"] = S.Backward(A, B, C)
    elif kind == "batched":
        eng = Bt.BatchedEngine(A, B)
        eng.forward()
        C = eng.C
        out = (torch.empty_like(C.rowidx), torch.empty_like(C.values))
        ws = S.alloc_workspace(S.workspace_size(S.OP_SORT, C))
        eng.capture(lambda: (eng.forward(), S.sort_columns(eng.C, out[0], out[1], ws)))
        st.update(eng=eng, out=out, ws=ws)
    elif kind == "batched_train":
        eng = Bt.BatchedEngine(A, B, backward=True)
        eng.capture(lambda: (eng.forward(), eng.backward(eng.values[:eng.nnz_c])))
        st["eng"] = eng
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    kind = st["case"]["kind"]
    if kind == "oneshot":
        C = S.spgemm(st["A"], st["B"], sorted_output=True)
        return C.colptr, C.rowidx, C.values
    if kind == "product":
        C, _ = st["eng"].run()
        return C.colptr, C.rowidx, C.values
    if kind == "topk":
        kept = []

        def consume(c0, c1, Cb):
            need = S.workspace_size(S.OP_PRUNE, Cb)
            if st["ws"] is None or st["ws"].numel() < need:
                st["ws"] = S.alloc_workspace(need)
            P = S.prune_topk(Cb, 0.0, st["case"]["keep"], ws=st["ws"])
            kept.append(S.sort_columns(P))

        st["eng"].run(consume)
        return (torch.cat([P.colptr[1:] - P.colptr[:-1] for P in kept]), torch.cat([P.rowidx for P in kept]),
                torch.cat([P.values for P in kept]))
    if kind == "aat":
        A = st["A"]
        T, _ = S.transpose(A, perm=False)
        C = S.spgemm(A, T, sorted_output=True)
        return C.colptr, C.rowidx, C.values
    if kind == "train":
        st["a"].grad = None
        st["b"].grad = None
        c, _, _ = S.SpGEMMFn.apply(st["a"], st["b"], st["A"], st["B"])
        loss = 0.5 * c.square().sum()
        loss.backward()
        return loss.detach(), st["a"].grad, st["b"].grad
    if kind == "grad":
        return st["bw"](st["dC"])
    if kind == "batched":
        eng = st["eng"]
        eng.replay()
        return eng.colptr, st["out"][0], st["out"][1]
    if kind == "batched_train":
        eng = st["eng"]
        eng.replay()
        return eng.colptr, eng.dA, eng.dB
    P = S.prune_topk(st["C"], st["case"]["threshold"], st["case"]["keep"], ws=st["ws"])
    return P.colptr, P.rowidx, P.values


# ------------------------------------------------------------------ the least a pass moves and computes
_COUNTS = {}


def _counts(case):
    """(nnz(A), nnz(B), multiplications, counts of C's columns) for one seed."""
    key = json.dumps({k: v for k, v in case.items() if k != "name"}, sort_keys=True)
    if key not in _COUNTS:
        A, B = _operands(case, _gen(0))
        plan = S.Engine(A, B).plan()
        _COUNTS[key] = (A, B, plan.total_flops, plan.nnz_host[0])
        _COUNTS[key] = (A.nnz, A.ncols, B.nnz, B.ncols, plan.total_flops, plan.nnz_host[0].copy())
    return _COUNTS[key]


def work(case):
    vb = 4 if case["dtype"] == "f32" else 8
    r, kind = 4 + vb, case["kind"]
    if kind == "prune":
        n, nnz = case["n"], case["n"] * min(case["mean"], case["m"])
        return {"bytes": vb * nnz + 16 * n + r * min(nnz, n * case["keep"]), "flops": nnz}
    na, ka, nb, n, mult, cols = _counts(case)
    nc = int(cols.sum())
    same = kind in ("product", "topk")  # B is A
    inputs = r * (na + (0 if same or kind == "aat" else nb)) + 8 * (ka + (0 if same or kind == "aat" else n))
    if kind == "topk":
        return {"bytes": inputs + r * int(cols.clip(max=case["keep"]).sum()) + 8 * n, "flops": 2 * mult}
    if kind == "train":  # C is written for the caller, dC read, gradients written
        return {"bytes": inputs + r * nc + 8 * n + vb * nc + vb * (na + nb), "flops": 6 * mult}
    if kind == "grad":
        return {"bytes": inputs + r * nc + 8 * n + vb * (na + nb), "flops": 4 * mult}
    if kind == "batched_train":
        return {"bytes": inputs + r * nc + 8 * n + vb * (na + nb), "flops": 6 * mult}
    return {"bytes": inputs + r * nc + 8 * n, "flops": 2 * mult}


# ------------------------------------------------------------------ the same in 64 bits, with torch alone
def _exact_columns(Acp, Ari, Av, Bcp, Bri, Bv, m, semiring, row0=0, dense=1 << 28, terms=1 << 27, grad=None,
                   keep=None):
    """C = A B by column chunks on a dense float64 array of the rows [row0, row0 + m): (counts per column, rows,
    values).  A's and B's rows index rows and A's columns from 0.  With ``grad`` ((dA, dB), both added to), the
    gradients of 0.5 ||C||^2 as well; with ``keep``, only the largest entries of each column."""
    n = Bcp.numel() - 1
    deg = Acp[1:] - Acp[:-1]
    cum = torch.zeros(Bri.numel() + 1, dtype=torch.int64, device="cuda")
    cum[1:] = torch.cumsum(deg[Bri.long()], 0)
    colterms = cum[Bcp].tolist()
    counts, rows, vals = [], [], []
    c0, wmax = 0, max(1, dense // m)
    while c0 < n:
        c1 = c0 + 1
        while c1 < n and c1 - c0 < wmax and colterms[c1 + 1] - colterms[c0] <= terms:
            c1 += 1
        e0, e1 = int(Bcp[c0]), int(Bcp[c1])
        k = Bri[e0:e1].long()
        ecol = torch.repeat_interleave(torch.arange(c1 - c0, device="cuda"), Bcp[c0 + 1:c1 + 1] - Bcp[c0:c1])
        total = colterms[c1] - colterms[c0]
        e = torch.repeat_interleave(torch.arange(e1 - e0, device="cuda"), deg[k], output_size=total)
        p = torch.arange(total, device="cuda") - (cum[e0:e1] - cum[e0])[e] + Acp[k][e]
        at = ecol[e] * m + Ari[p].long()
        a, b = Av[p].double(), Bv[e0:e1].double()[e]
        size = (c1 - c0) * m
        if semiring == "min_plus":
            acc = torch.full((size,), math.inf, dtype=torch.float64, device="cuda")
            acc.scatter_reduce_(0, at, a + b, "amin")
        else:
            acc = torch.zeros(size, dtype=torch.float64, device="cuda")
            if semiring == "or_and":
                acc[at] = 1.0
            else:
                acc.index_add_(0, at, a * b)
        if grad is not None:
            dc = acc[at]
            grad[0].index_add_(0, p, b * dc)
            grad[1][e0:e1].index_add_(0, e, a * dc)
        hit = torch.zeros(size, dtype=torch.bool, device="cuda")
        hit[at] = True
        nz = hit.nonzero().squeeze(1)
        cnt, r, v = hit.view(c1 - c0, m).sum(1), (nz % m + row0).to(torch.int32), acc[nz]
        if keep is not None:  # ranked as the product stores them
            cp, r, v = _exact_prune(_pointers(cnt), r, v, v.to(Av.dtype), 0.0, keep)
            cnt = cp[1:] - cp[:-1]
        rows.append(r)
        vals.append(v)
        counts.append(cnt)
        c0 = c1
    cat = lambda x, dt: torch.cat(x) if x else torch.zeros(0, dtype=dt, device="cuda")  # noqa: E731
    return cat(counts, torch.int64), cat(rows, torch.int32), cat(vals, torch.float64)


def _pointers(counts):
    cp = torch.zeros(counts.numel() + 1, dtype=torch.int64, device="cuda")
    cp[1:] = torch.cumsum(counts, 0)
    return cp


def _exact_prune(cp, ri, v64, v, threshold, keep):
    """The kept entries of a matrix with values v (ranked as stored) in input order; v64 in their place."""
    n = cp.numel() - 1
    col = torch.repeat_interleave(torch.arange(n, device="cuda"), cp[1:] - cp[:-1])
    idx = torch.nonzero(v.double() >= threshold).squeeze(1)
    idx = idx[torch.argsort(ri[idx], stable=True)]
    idx = idx[torch.argsort(v[idx], descending=True, stable=True)]
    idx = idx[torch.argsort(col[idx], stable=True)]
    c = col[idx]
    first = _pointers(torch.bincount(c, minlength=n))
    idx = idx[torch.arange(idx.numel(), device="cuda") - first[c] < keep]
    idx = torch.sort(idx)[0]
    return _pointers(torch.bincount(col[idx], minlength=n)), ri[idx], v64[idx]


def exact(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "prune":
        C = _prune_input(case, g)
        return _exact_prune(C.colptr, C.rowidx, C.values.double(), C.values, case["threshold"], case["keep"])
    dt = DTYPE[case["dtype"]]
    if kind in ("batched", "batched_train"):
        A, B, ns = _batch(case, g)
        dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
        dB = torch.zeros(B.nnz, dtype=torch.float64, device="cuda")
        parts, o = [], 0
        for q in ns:
            a0, a1, b0, b1 = (int(x) for x in (A.colptr[o], A.colptr[o + q], B.colptr[o], B.colptr[o + q]))
            parts.append(_exact_columns(A.colptr[o:o + q + 1] - a0, A.rowidx[a0:a1] - o, A.values[a0:a1],
                                        B.colptr[o:o + q + 1] - b0, B.rowidx[b0:b1] - o, B.values[b0:b1], q,
                                        "plus_times", o, grad=(dA[a0:a1], dB[b0:b1]) if kind != "batched" else None))
            if kind != "batched":
                parts[-1] = (parts[-1][0], None, None)
            o += q
        cp = _pointers(torch.cat([x[0] for x in parts]))
        if kind == "batched_train":
            return cp, dA, dB
        return cp, torch.cat([x[1] for x in parts]), torch.cat([x[2] for x in parts])
    if kind == "aat":
        A = _left(case, g)
        col = torch.repeat_interleave(torch.arange(A.ncols, device="cuda"), A.colptr[1:] - A.colptr[:-1])
        order = torch.argsort(A.rowidx, stable=True)
        B = S.CSC(A.ncols, A.nrows, _pointers(torch.bincount(A.rowidx.long(), minlength=A.nrows)),
                  col[order].to(torch.int32), A.values[order])
    else:
        A, B = _operands(case, g)
    m, sr = A.nrows, case.get("semiring", "plus_times")
    args = (A.colptr, A.rowidx, A.values, B.colptr, B.rowidx, B.values, m, sr)
    if kind == "train":
        dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
        dB = torch.zeros(B.nnz, dtype=torch.float64, device="cuda")
        _, _, v = _exact_columns(*args, grad=(dA, dB))
        return 0.5 * v.square().sum(), dA, dB
    if kind == "grad":
        counts, ri, v = _exact_columns(*args)
        dC = _values(v.numel(), dt, g, "normal").double()  # the draw that prepare makes after the operands
        return _exact_grad(A, B, _pointers(counts), ri, dC)
    counts, ri, v = _exact_columns(*args, keep=case["keep"] if kind == "topk" else None)
    return (counts if kind == "topk" else _pointers(counts)), ri, v


def _exact_grad(A, B, cp, ri, dC, chunk=1 << 26):
    """dA and dB on the patterns of A and B for dC on the pattern (cp, ri) of the product, rows ascending."""
    m = A.nrows
    keys = torch.repeat_interleave(torch.arange(cp.numel() - 1, device="cuda"), cp[1:] - cp[:-1]) * m + ri.long()
    deg = A.colptr[1:] - A.colptr[:-1]
    bcol = torch.repeat_interleave(torch.arange(B.ncols, device="cuda"), B.colptr[1:] - B.colptr[:-1])
    dA = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
    dB = torch.zeros(B.nnz, dtype=torch.float64, device="cuda")
    step = max(1, chunk // max(1, int(deg.max())))
    for e0 in range(0, B.nnz, step):
        k = B.rowidx[e0:e0 + step].long()
        e = torch.repeat_interleave(torch.arange(k.numel(), device="cuda"), deg[k])
        first = torch.cumsum(deg[k], 0) - deg[k]
        p = torch.arange(e.numel(), device="cuda") - first[e] + A.colptr[k][e]
        dc = dC[torch.searchsorted(keys, bcol[e0:e0 + step][e] * m + A.rowidx[p].long())]
        dA.index_add_(0, p, B.values[e0:e0 + step].double()[e] * dc)
        dB[e0:e0 + step].index_add_(0, e, A.values[p].double() * dc)
    return dA, dB
