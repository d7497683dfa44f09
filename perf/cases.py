"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values: the call it makes (`call`), the pattern its inputs
are drawn from (`pattern`), and the sizes.  prepare(case, seed) draws the inputs on
the GPU, run(state) makes one pass through the public entry points, work(case) states
the bytes and additions a pass cannot do without, and exact(case, seed) sums the same
inputs in 64 bits with plain torch.

Patterns:
  er    every column of every input holds about Poisson(d) distinct uniform rows
  tall  every column of every input holds d distinct uniform rows of a long column
  rmat  independent skewed R-MAT matrices (a=.57, b=c=.19), duplicates removed
Calls:
  sum    spkadd(): plan, symbolic and numeric of new inputs
  refill spkadd_numeric() on a kept plan: new values on known patterns
  batch  one batched run over many independent requests, and the one-request path
         for the requests it reports as too large

The number of entries of the inputs and of the sum follow from the case alone, so that
the inputs of every seed are equally much work: a case's patterns are drawn once, and a
seed turns them (rows and columns rotated by distances of its own, the inputs in an
order of its own) and draws the values.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2112_10223_amd import binding

DEV = "cuda:0"
SEED = 211210223  # of the patterns
RMAT = (0.57, 0.19, 0.19, 0.05)
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def _sum(name, pattern, m, n, k, d, dtype="f32", option=""):
    return {"name": name, "call": "sum", "pattern": pattern, "m": m, "n": n, "k": k, "d": d, "dtype": dtype,
            "option": option}


def listed():
    return [
        # the smallest call: a handful of small matrices, where launches and waits are all there is
        _sum("small_er_f32", "er", 1000, 1000, 4, 8.0),
        # the benchmark's ordinary call: 32 square matrices, about 500 entries per column
        _sum("er_f32", "er", 65536, 65536, 32, 16.0),
        # the same in double precision
        _sum("er_f64", "er", 65536, 65536, 32, 16.0, "f64"),
        # a plan kept over several numeric passes (an assembly loop with fixed patterns), odd sizes
        dict(_sum("refill_er_f32", "er", 50021, 70001, 31, 12.5), call="refill"),
        # few entries per column of very tall matrices (graphs without a skew), odd sizes
        _sum("sparse_er_f32", "er", 1000003, 150001, 16, 12.0),
        # many inputs at once, each nearly empty per column (partial results of many workers)
        _sum("many_er_f32", "er", 65536, 16384, 128, 6.0),
        # the benchmark's largest call: skewed graphs, from empty columns to very long ones
        _sum("rmat_f32", "rmat", 1 << 20, 1 << 20, 64, 16.0),
        # a smaller skewed sum in double precision
        _sum("rmat_f64", "rmat", 1 << 16, 1 << 16, 32, 16.0, "f64"),
        # every column far too long for on-chip memory: the sliding method throughout
        _sum("tall_f32", "tall", 1 << 24, 1024, 128, 4096.0),
        # reproducible sums: every value added in input order, odd sizes
        _sum("ordered_er_f32", "er", 40009, 30011, 24, 20.0, option="ordered"),
        # inputs whose columns come in any row order (products that were never sorted)
        _sum("unsorted_rmat_f32", "rmat", 1 << 17, 1 << 17, 32, 16.0, option="unsorted_in"),
        # sixteen requests of a service in one run: each with shapes and densities of its own
        {"name": "batch_f32", "call": "batch", "spec_seed": 211210228, "nreq": 16, "k_most": 64, "mn_most": 65536,
         "nnz_most": 1 << 23, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["er", "er", "er", "er_refill", "er_ordered", "er_many", "rmat", "rmat_unsorted", "tall",
                       "batch"])
    dtype = rng.choice(["f32", "f32", "f64"])
    if kind.startswith("er"):
        k = _log(rng, 65, 128) if kind == "er_many" else _log(rng, 2, 64)
        d = round(math.exp(rng.uniform(math.log(2.0), math.log(40.0))), 2)
        m = _log(rng, 600, 1 << 20)
        most = (1 << 25) / (k * d)  # input entries of a pass at most
        n = _log(rng, 500, min(150000.0, most))
        c = _sum("", "er", m, n, k, min(d, m / 64.0), dtype, "ordered" if kind == "er_ordered" else "")
        if kind == "er_refill":
            c["call"] = "refill"
    elif kind.startswith("rmat"):
        scale = rng.randint(12, 17)
        c = _sum("", "rmat", 1 << scale, 1 << scale, _log(rng, 4, 64), float(rng.randint(4, 16)), dtype,
                 "unsorted_in" if kind == "rmat_unsorted" else "")
    elif kind == "tall":
        k = _log(rng, 8, 128)
        c = _sum("", "tall", _log(rng, 1 << 18, 1 << 24), _log(rng, 16, 512), k, float(_log(rng, 500, 4096)), dtype)
    else:
        c = {"name": "", "call": "batch", "spec_seed": rng.randrange(1 << 30), "nreq": rng.randint(4, 20),
             "k_most": 64, "mn_most": _log(rng, 2048, 65536), "nnz_most": _log(rng, 1 << 17, 1 << 23),
             "dtype": dtype}
    del c["name"]
    return c


# ---- inputs ----

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed & 0x7FFFFFFFFFFFFFFF)
    return g


def _csc(key, m, n):
    """colptr and rowidx of the sorted distinct keys col * m + row."""
    bounds = torch.arange(n + 1, device=DEV, dtype=torch.int64) * m
    colptr = torch.searchsorted(key, bounds).to(torch.int32)
    return colptr, (key % m).to(torch.int32)


def _distinct(key):
    key = key.sort().values
    keep = torch.ones(key.numel(), dtype=torch.bool, device=DEV)
    if key.numel() > 1:
        keep[1:] = key[1:] != key[:-1]
    return key[keep]


def _values(g, nnz, pattern, dtype):
    dt = DTYPES[dtype]
    if pattern == "rmat":
        return torch.randn(nnz, generator=g, device=DEV, dtype=dt)
    return torch.rand(nnz, generator=g, device=DEV, dtype=dt) * 2 - 1


def _turned_key(col, row, m, n, turn):
    """Keys of the entries with columns and rows rotated (col and row are overwritten)."""
    col.add_(turn[0]).remainder_(n).mul_(m)
    return col.add_(row.add_(turn[1]).remainder_(m))


def _er(g, m, n, d, poisson, turn):
    if poisson:
        cnt = torch.poisson(torch.full((n,), d, device=DEV), generator=g).clamp_(max=m).to(torch.int64)
    else:
        cnt = torch.full((n,), int(round(d)), device=DEV, dtype=torch.int64)
    col = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int64), cnt)
    row = torch.randint(0, m, (col.numel(),), generator=g, device=DEV)
    return _csc(_distinct(_turned_key(col, row, m, n, turn)), m, n)


def _rmat(g, m, n, d, turn):
    scale = m.bit_length() - 1
    edges = int(d * n)
    a, b, c, _ = RMAT
    row = torch.zeros(edges, device=DEV, dtype=torch.int64)
    col = torch.zeros(edges, device=DEV, dtype=torch.int64)
    for _ in range(scale):
        q = torch.rand(edges, generator=g, device=DEV)
        lower = q >= a + b
        right = (q >= a) & ~(lower & (q < a + b + c))
        row.mul_(2).add_(lower)
        col.mul_(2).add_(right)
    return _csc(_distinct(_turned_key(col, row, m, n, turn)), m, n)


def _shuffle_columns(g, colptr, rowidx, n):
    """The same columns with their rows in random order."""
    col = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int64), (colptr[1:] - colptr[:-1]).long())
    key = col.mul_(1 << 31).add_(torch.randint(0, 1 << 31, (col.numel(),), generator=g, device=DEV))
    return rowidx[key.argsort()]


def _inputs(pattern_seed, pattern, m, n, means, dtype, option, rng, g):
    """(colptrs, rowidxs, values) of one sum.  The patterns come from pattern_seed; rng
    and g (the seed's) turn and order them and draw the values."""
    turn = (rng.randrange(n), rng.randrange(m))
    order = list(range(len(means)))
    rng.shuffle(order)
    cps, ris, vas = [], [], []
    for i in order:
        gp = _gen(pattern_seed * 1009 + i)
        if pattern == "rmat":
            c, r = _rmat(gp, m, n, means[i], turn)
        else:
            c, r = _er(gp, m, n, means[i], pattern == "er", turn)
        if option == "unsorted_in":
            r = _shuffle_columns(g, c, r, n)
        cps.append(c)
        ris.append(r)
        vas.append(_values(g, r.numel(), pattern, dtype))
    return cps, ris, vas


def _matrices(case, seed):
    return _inputs(SEED, case["pattern"], case["m"], case["n"], [case["d"]] * case["k"], case["dtype"],
                   case["option"], random.Random(seed), _gen(seed))


def _requests(case):
    """Shapes of the requests of a batched run: 2..k_most inputs, m and n log-uniform in
    [256, mn_most], each input's density log-uniform in [1e-4, 1e-2]; requests above
    nnz_most expected entries are drawn again."""
    rng = random.Random(case["spec_seed"])
    out = []
    while len(out) < case["nreq"]:
        k = rng.randint(2, case["k_most"])
        m, n = _log(rng, 256, case["mn_most"]), _log(rng, 256, case["mn_most"])
        dens = [math.exp(rng.uniform(math.log(1e-4), math.log(1e-2))) for _ in range(k)]
        if sum(dens) * m * n <= case["nnz_most"]:
            out.append((m, n, dens))
    return out


def _request_matrices(case, seed):
    rng, g = random.Random(seed), _gen(seed)
    return [(m, n, *_inputs(case["spec_seed"] + 7919 * t, "er", m, n, [x * m for x in dens], case["dtype"], "", rng,
                            g))
            for t, (m, n, dens) in enumerate(_requests(case))]


# ---- the passes ----

def _opts(case):
    flags = {"ordered": binding.SPKADD_FLAG_ORDERED, "unsorted_in": binding.SPKADD_FLAG_UNSORTED_IN}
    option = case.get("option", "")
    return binding.make_opts(flags=flags[option]) if option else None


def prepare(case, seed):
    dtype = binding.SPKADD_F64 if case["dtype"] == "f64" else binding.SPKADD_F32
    if case["call"] == "batch":
        reqs = []
        for m, n, cps, ris, vas in _request_matrices(case, seed):
            cap = max(1, sum(r.numel() for r in ris))
            reqs.append({"m": m, "colptrs": cps, "rowidxs": ris, "values": vas, "cap_c": cap,
                         "colptr_c": torch.empty(n + 1, dtype=torch.int32, device=DEV),
                         "rowidx_c": torch.empty(cap, dtype=torch.int32, device=DEV),
                         "values_c": torch.empty(cap, dtype=DTYPES[case["dtype"]], device=DEV)})
        cols = sum(q["colptr_c"].numel() - 1 for q in reqs)
        handle = binding.Batch(dtype, len(reqs), cols, sum(len(q["colptrs"]) for q in reqs))
        return {"call": "batch", "requests": reqs, "handle": handle}
    cps, ris, vas = _matrices(case, seed)
    s = {"call": case["call"], "m": case["m"], "cps": cps, "ris": ris, "vas": vas, "opts": _opts(case)}
    if case["call"] == "refill":
        s["plan"] = binding.spkadd_plan(case["m"], case["n"], cps, ris, dtype, s["opts"])
        s["colptr_c"] = torch.empty(case["n"] + 1, dtype=torch.int32, device=DEV)
        nnz = binding.spkadd_symbolic(s["plan"], s["colptr_c"])
        s["rowidx_c"] = torch.empty(nnz, dtype=torch.int32, device=DEV)
        s["values_c"] = torch.empty(nnz, dtype=DTYPES[case["dtype"]], device=DEV)
        s["values"] = binding.PtrArray(vas, non_null=True)
    return s


def run(state):
    if state["call"] == "sum":
        return binding.spkadd(state["m"], state["cps"], state["ris"], state["vas"], state["opts"])
    if state["call"] == "refill":
        binding.spkadd_numeric(state["plan"], state["values"], state["rowidx_c"], state["values_c"])
        return state["colptr_c"], state["rowidx_c"], state["values_c"]
    reqs = state["requests"]
    state["handle"].run(reqs)
    nnz, status = state["handle"].results()
    out = []
    for q, z, st in zip(reqs, nnz, status):
        if st == binding.SPKADD_REQ_TOO_LARGE:
            out.append(binding.spkadd(q["m"], q["colptrs"], q["rowidxs"], q["values"]))
        else:
            out.append((q["colptr_c"], q["rowidx_c"][:z], q["values_c"][:z]))
    return out


# ---- what a pass cannot do without ----

def _rmat_distinct(scale, edges):
    """Expected distinct cells of `edges` draws of a 2^scale R-MAT matrix: the cells with
    i, j, l and the other levels in each quadrant share one probability."""
    a, b, c, d = RMAT
    total = 0.0
    for i in range(scale + 1):
        for j in range(scale + 1 - i):
            for l in range(scale + 1 - i - j):
                r = scale - i - j - l
                cells = math.factorial(scale) // (math.factorial(i) * math.factorial(j) * math.factorial(l) *
                                                  math.factorial(r))
                p = a ** i * b ** j * c ** l * d ** r
                total += cells * -math.expm1(edges * math.log1p(-p))
    return total


def _counts(m, n, pattern, means):
    """Expected input and output entries."""
    if pattern == "rmat":
        scale = m.bit_length() - 1
        return len(means) * _rmat_distinct(scale, means[0] * n), _rmat_distinct(scale, len(means) * means[0] * n)
    if pattern == "er":  # draws of a Poisson count: a row is missed with probability exp(-mean / m)
        miss = [math.exp(-x / m) for x in means]
    else:
        miss = [(1.0 - 1.0 / m) ** x for x in means]
    nin = sum(m * (1.0 - x) for x in miss) * n
    nout = m * (1.0 - math.prod(miss)) * n
    return nin, nout


def work(case):
    v = 8 if case["dtype"] == "f64" else 4
    if case["call"] == "batch":
        shapes = [(m, n, "er", [x * m for x in dens]) for m, n, dens in _requests(case)]
    else:
        shapes = [(case["m"], case["n"], case["pattern"], [case["d"]] * case["k"])]
    total = adds = 0.0
    for m, n, pattern, means in shapes:
        nin, nout = _counts(m, n, pattern, means)
        total += (4 + v) * (nin + nout) + 4.0 * (len(means) + 1) * (n + 1)
        adds += max(nin - nout, 0.0)
    return {"bytes": total, "flops": adds + 1.0}


# ---- the same sums in 64 bits ----

EXACT_PART = 1 << 26  # input entries sorted at a time


def _exact_sum(m, n, cps, ris, vas):
    counts = sum((c[1:] - c[:-1]).long() for c in cps)
    upto = torch.cumsum(counts, 0)
    colptr = [torch.zeros(1, dtype=torch.int64, device=DEV)]
    rows, vals = [], []
    at, c0, base = 0, 0, 0
    ends = upto.cpu()
    ptr = [c.cpu() for c in cps]
    while c0 < n:
        c1 = int(torch.searchsorted(ends, at + EXACT_PART))
        c1 = min(n, max(c1, c0 + 1))
        keys, vs = [], []
        for c, r, v, p in zip(cps, ris, vas, ptr):
            s, e = int(p[c0]), int(p[c1])
            col = torch.repeat_interleave(torch.arange(c1 - c0, device=DEV), (c[c0 + 1:c1 + 1] - c[c0:c1]).long())
            keys.append(col * m + r[s:e].long())
            vs.append(v[s:e].double())
        key, order = torch.cat(keys).sort(stable=True)
        v = torch.cat(vs)[order]
        first = torch.ones(key.numel(), dtype=torch.bool, device=DEV)
        if key.numel() > 1:
            first[1:] = key[1:] != key[:-1]
        place = torch.cumsum(first, 0) - 1
        key = key[first]
        vals.append(torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, place, v))
        rows.append((key % m).to(torch.int32))
        bounds = torch.arange(1, c1 - c0 + 1, device=DEV, dtype=torch.int64) * m
        colptr.append(torch.searchsorted(key, bounds) + base)
        base += key.numel()
        at, c0 = int(ends[c1 - 1]), c1
    empty = torch.zeros(0, dtype=torch.int32, device=DEV)
    return (torch.cat(colptr).to(torch.int32), torch.cat(rows) if rows else empty,
            torch.cat(vals) if vals else empty.double())


def exact(case, seed):
    if case["call"] == "batch":
        return [_exact_sum(m, n, cps, ris, vas) for m, n, cps, ris, vas in _request_matrices(case, seed)]
    cps, ris, vas = _matrices(case, seed)
    return _exact_sum(case["m"], case["n"], cps, ris, vas)
