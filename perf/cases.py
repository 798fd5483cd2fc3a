"""Timed workloads of the local SpGEMM library, through its Python entry points.

Every input is drawn on the GPU from a seed: the matrices of `synth.py`'s
recipes (uniform rows, ragged rows, bands, aggregation operators, R-MAT,
Markov-clustering matrices), with torch's generator so that large inputs take
milliseconds.  A case is a dict of plain values; "kind" picks the entry point:

  product   Plan.symbolic, then Plan.numeric into the program's own buffers
  permute   binding.permute(A, p, p, out): symmetric permutation
  stages    StageGraph.replay(): block products summed into one C, one graph
  train     autograd: numeric pass forward, both gradients backward
  mcl       binding.mcl_iteration(X, out): one Markov-clustering iteration

A program that multiplies again and again keeps its output buffers: they are
sized from the case alone (_capacity), start at zero and are returned whole, so
outputs have one shape for every seed.  Training works at fixed sparsity: there
the pattern goes with the case and the values with the seed.
"""
import math

import torch

from paper_2603_21444_amd import autograd, binding
from paper_2603_21444_amd.graph import StageGraph

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # The smallest call: launches, read-backs and host work count.
        dict(name="product_4096_f64", kind="product", a="uniform", m=4096, k=4096, n=4096,
             lo=8, hi=8, b="same", dtype="f64"),
        # The headline benchmark: one GPU's block share of an unstructured product.
        dict(name="product_2p20_f32", kind="product", a="uniform", m=1 << 20, k=1 << 20,
             n=1 << 20, lo=16, hi=16, b="uniform", dtype="f32"),
        # Ragged rows and odd sizes in double precision: many bins at once.
        dict(name="product_ragged_f64", kind="product", a="uniform", m=100003, k=80021, n=120011,
             lo=1, hi=40, b="uniform", dtype="f64"),
        # Algebraic-multigrid restriction A R: one entry per row of R, few products per row.
        dict(name="restriction_2p20_f32", kind="product", a="uniform", m=1 << 20, k=1 << 20,
             n=1 << 17, lo=16, hi=16, b="aggregation", dtype="f32"),
        # A^2 of a structured matrix in its own order: columns cluster in bands.
        dict(name="banded_2p20_f32", kind="product", a="banded", m=1 << 20, k=1 << 20, n=1 << 20,
             lo=16, hi=16, b="same", dtype="f32"),
        # The random symmetric permutation applied to such a matrix beforehand.
        dict(name="permute_2p20_f32", kind="permute", a="banded", m=1 << 20, lo=16, hi=16,
             dtype="f32"),
        # The rounds of the distributed product on one GPU: 8 uneven blocks into one C.
        dict(name="stages_uniform_f32", kind="stages", a="uniform", m=1 << 18, n=1 << 20, K=8,
             kmin=1 << 18, kmax=1 << 20, lo=4, hi=32, dtype="f32"),
        # The same rounds with a power-law left operand: hub rows beside short ones.
        dict(name="stages_rmat_f32", kind="stages", a="rmat", m=1 << 20, n=1 << 20, K=8,
             kmin=1 << 16, kmax=1 << 18, lo=4, hi=32, dtype="f32"),
        # A training step at fixed sparsity (float dB).
        dict(name="train_2p18_f32", kind="train", m=1 << 18, k=1 << 18, n=1 << 18, lo=16, hi=16,
             deterministic=False, dtype="f32"),
        # The reproducible training step, double precision, odd sizes and ragged rows.
        dict(name="train_det_f64", kind="train", m=50021, k=60013, n=40009, lo=4, hi=24,
             deterministic=True, dtype="f64"),
        # The heaviest iterations of clustering: hundreds of entries per row, no clusters yet.
        dict(name="mcl_unstructured", kind="mcl", a="mixed", n=1 << 17, d=400, prune=1e-4,
             topk=1000, order="workload"),
        # Later iterations: clusters have formed, weak links between them are pruned.
        dict(name="mcl_clusters", kind="mcl", a="clusters", n=1 << 16, d=64, prune=1e-4,
             topk=1000, order="workload"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; sizes mostly odd."""
    kind = rng.choice(["product", "product", "product", "restriction", "banded", "permute",
                       "stages", "rmat", "train", "mcl_mixed", "mcl_clusters"])
    dtype = rng.choice(["f32", "f32", "f64"])
    if kind in ("product", "train"):
        hi = _log(rng, 4, 40)
        lo = rng.choice([hi, max(1, hi // 2), 1])
        top = min(1 << 20 if kind == "product" else 1 << 18, int(2.4e8 / hi ** 2))
        m, k, n = (max(4096, _log(rng, top / 16, top)) for _ in range(3))
        if kind == "train":
            return dict(kind="train", m=m, k=k, n=n, lo=lo, hi=hi,
                        deterministic=rng.random() < 0.5, dtype=dtype)
        return dict(kind="product", a="uniform", m=m, k=k, n=n, lo=lo, hi=hi, b="uniform",
                    dtype=dtype)
    if kind == "restriction":
        m = _log(rng, 1 << 14, 1 << 20)
        return dict(kind="product", a="uniform", m=m, k=m, n=max(64, m // rng.randint(3, 27)),
                    lo=rng.choice([5, 7]), hi=rng.choice([7, 16, 27]), b="aggregation",
                    dtype=dtype)
    if kind in ("banded", "permute"):
        m = _log(rng, 1 << 14, 1 << 20)
        hi = rng.randint(3, 16)
        lo = rng.choice([hi, max(1, hi // 2)])
        if kind == "permute":
            return dict(kind="permute", a=rng.choice(["banded", "uniform"]), m=m, lo=lo, hi=hi,
                        dtype=dtype)
        return dict(kind="product", a="banded", m=m, k=m, n=m, lo=lo, hi=hi, b="same",
                    dtype=dtype)
    if kind == "stages":
        m = _log(rng, 1 << 13, 1 << 17)
        kmax = _log(rng, 1 << 14, 1 << 18)
        return dict(kind="stages", a="uniform", m=m, n=_log(rng, 1 << 15, 1 << 20),
                    K=rng.randint(2, 8), kmin=kmax // 4, kmax=kmax, lo=4, hi=_log(rng, 8, 32),
                    dtype="f32")
    if kind == "rmat":
        m = 1 << rng.randint(14, 19)
        return dict(kind="stages", a="rmat", m=m, n=_log(rng, m // 2, m), K=rng.randint(2, 8),
                    kmin=m // 16, kmax=m // 4, lo=4, hi=_log(rng, 8, 32), dtype="f32")
    if kind == "mcl_mixed":
        return dict(kind="mcl", a="mixed", n=_log(rng, 1 << 14, 1 << 17), d=_log(rng, 130, 400),
                    prune=1e-4, topk=1000, order="workload")
    order = rng.choice(["workload", "paper"])
    return dict(kind="mcl", a="clusters", n=_log(rng, 1 << 13, 1 << 17), d=_log(rng, 8, 64),
                prune=1e-4 if order == "workload" else 2e-3,
                topk=1000 if order == "workload" else 500, order=order)


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((int(seed) + 1) * 1000 + stream)


def _pack(m, n, cols, vals):
    """CSR of sorted columns [m, d] (n or more: no entry) and values [m, d]."""
    keep = cols < n
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(keep.sum(1), 0, out=rp[1:])
    return binding.DeviceCSR((m, n), rp.int(), cols[keep].int(), vals[keep])


def _distinct(m, n, lo, hi, g):
    """Sorted columns [m, hi]; row i holds U{lo..hi} distinct ones, then n."""
    cols = torch.randint(0, n, (m, hi), generator=g, device="cuda")
    if lo < hi:
        lens = torch.randint(lo, hi + 1, (m, 1), generator=g, device="cuda")
        cols[torch.arange(hi, device="cuda")[None, :] >= lens] = n
    cols = cols.sort(1).values
    while True:  # redraw the repeats
        dup = torch.zeros_like(cols, dtype=torch.bool)
        dup[:, 1:] = (cols[:, 1:] == cols[:, :-1]) & (cols[:, 1:] < n)
        c = int(dup.sum())
        if c == 0:
            return cols
        cols[dup] = torch.randint(0, n, (c,), generator=g, device="cuda")
        cols = cols.sort(1).values


def _values(shape, kind, dtype, g):
    v = torch.empty(shape, dtype=torch.float64, device="cuda")
    if kind == "u01":
        v.uniform_(generator=g)
        v = 1.0 - v
    else:
        v.normal_(generator=g)
    return v.to(dtype)


def _uniform(m, n, lo, hi, kind, dtype, g):
    hi = min(hi, max(1, n // 4))
    cols = _distinct(m, n, min(lo, hi), hi, g)
    return _pack(m, n, cols, _values(cols.shape, kind, dtype, g))


def _banded(n, lo, hi, dtype, g):
    """Rows on three diagonal bands (offsets 0, +-n/8, half-width 256)."""
    half = min(256, max(8, n // 64))
    w = 2 * half + 1
    slots = _distinct(n, 3 * w, lo, hi, g)
    off = torch.tensor([0, n // 8, -(n // 8), 0], device="cuda")
    cols = torch.arange(n, device="cuda")[:, None] + off[slots // w] + slots % w - half
    cols = torch.where(cols < 0, -cols - 1, cols)
    cols = torch.where(cols >= n, 2 * n - 1 - cols, cols)
    cols = torch.where(slots < 3 * w, cols, n).sort(1).values
    dup = torch.zeros_like(cols, dtype=torch.bool)
    dup[:, 1:] = cols[:, 1:] == cols[:, :-1]
    cols[dup] = n
    cols = cols.sort(1).values
    return _pack(n, n, cols, _values(cols.shape, "u01", dtype, g))


def _aggregation(n, nc, dtype, g):
    agg = torch.randperm(n, generator=g, device="cuda") % nc
    return _pack(n, nc, agg[:, None], _values((n, 1), "u01", dtype, g))


def _rmat(n, dtype, g):
    """R-MAT(0.57, 0.19, 0.19, 0.05), 16 n draws, repeats collapsed."""
    row = torch.zeros(16 * n, dtype=torch.int64, device="cuda")
    col = torch.zeros_like(row)
    for _ in range(n.bit_length() - 1):
        r = torch.rand(row.numel(), generator=g, device="cuda")
        row = (row << 1) | (r >= 0.76)
        col = (col << 1) | (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    key = torch.unique(row * n + col)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(key // n, minlength=n), 0, out=rp[1:])
    return binding.DeviceCSR((n, n), rp.int(), (key % n).int(),
                             _values((key.numel(),), "normal", dtype, g))


def _rows_of(M):
    lens = (M.row_ptr[1:] - M.row_ptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(M.shape[0], device="cuda"), lens)


def _pairs(case, seed):
    """The block pairs (A_k, B_k) of a stage sequence."""
    dt, g = DTYPES[case["dtype"]], _gen(seed, 0)
    m, n, K, lo, hi = case["m"], case["n"], case["K"], case["lo"], case["hi"]
    w = torch.randint(case["kmin"], case["kmax"] + 1, (K,), generator=g, device="cuda").double()
    if case["a"] == "uniform":
        return [(_uniform(m, int(k), lo, hi, "normal", dt, g),
                 _uniform(int(k), n, lo, hi, "normal", dt, g)) for k in w.tolist()]
    A = _rmat(m, dt, g)
    bounds = [0] + (w.cumsum(0) / w.sum() * m).floor().long().tolist()
    bounds[-1] = m
    rows, pairs = _rows_of(A), []
    for lo_k, hi_k in zip(bounds[:-1], bounds[1:]):
        sel = (A.col_idx >= lo_k) & (A.col_idx < hi_k)
        rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(torch.bincount(rows[sel], minlength=m), 0, out=rp[1:])
        Ak = binding.DeviceCSR((m, hi_k - lo_k), rp.int(), (A.col_idx[sel] - lo_k).contiguous(),
                               A.vals[sel].contiguous())
        pairs.append((Ak, _uniform(hi_k - lo_k, n, lo, hi, "normal", dt, g)))
    return pairs


def _operands(case, seed):
    dt, g = DTYPES[case["dtype"]], _gen(seed, 0)
    m, lo, hi = case["m"], case["lo"], case["hi"]
    if case["kind"] == "train":
        pat = _gen(0, 1)
        A = _uniform(m, case["k"], lo, hi, "normal", dt, pat)
        B = _uniform(case["k"], case["n"], lo, hi, "normal", dt, pat)
        A.vals, B.vals = (_values((M.nnz,), "normal", dt, g) for M in (A, B))
        return A, B
    if case["a"] == "banded":
        A = _banded(m, lo, hi, dt, g)
    else:
        A = _uniform(m, case.get("k", m), min(lo, hi), hi, "u01", dt, g)
    if case["kind"] == "permute":
        return A, torch.randperm(m, generator=g, device="cuda").int()
    if case["b"] == "same":
        return A, A
    if case["b"] == "aggregation":
        return A, _aggregation(case["k"], case["n"], dt, g)
    return A, _uniform(case["k"], case["n"], lo, hi, "u01", dt, g)


def _mcl_input(case, seed):
    """Row-stochastic X.  mixed: d uniform columns per row with squared
    uniform weights.  clusters: clusters of d vertices under random labels,
    full inside, and two links of a ten-thousandth of the weight per vertex."""
    n, d, g = case["n"], case["d"], _gen(seed, 0)
    if case["a"] == "mixed":
        cols = _distinct(n, n, d, d, g)
        w = _values(cols.shape, "u01", torch.float64, g).square()
    else:
        label = torch.randperm(n, generator=g, device="cuda")
        at = torch.empty_like(label)
        at[label] = torch.arange(n, device="cuda")
        base = at // d * d
        cols = base[:, None] + torch.arange(d, device="cuda")[None, :]
        far = (at[:, None] + d + torch.randint(0, n // 2 - 2 * d, (n, 2), generator=g,
                                               device="cuda") + torch.tensor([0, n // 2 - d],
                                                                             device="cuda")) % n
        inside = cols < n
        cols = torch.where(inside, label[cols.clamp(max=n - 1)], n)
        cols = torch.cat([cols, label[far]], 1)
        w = _values(cols.shape, "u01", torch.float64, g) * 0.5 + 0.5
        w[:, d:] *= 1e-4
        cols, order = cols.sort(1)
        dup = torch.zeros_like(cols, dtype=torch.bool)
        dup[:, 1:] = cols[:, 1:] == cols[:, :-1]
        cols[dup] = n
        w = w.gather(1, order)
        w = torch.where(cols < n, w, 0.0)
        cols, order = cols.sort(1)
        w = w.gather(1, order)
    w = (w / w.sum(1, keepdim=True)).float()
    return _pack(n, n, cols, w)


def _capacity(case):
    """Entries of the output buffers: the scalar products (a fifth more than
    their expected number where row lengths are drawn), which bound nnz."""
    if case["kind"] == "mcl":
        return case["n"] * min(case["topk"], case["n"])
    lo, hi, m = case["lo"], case["hi"], case["m"]
    if case["kind"] == "permute":
        return m * hi
    slack = 1.0 if lo == hi else 1.2
    mean = (lo + hi) / 2.0
    if case["kind"] == "stages":
        return int(slack * mean * (16 * m if case["a"] == "rmat" else case["K"] * m * mean))
    return int(slack * m * mean * (1 if case["b"] == "aggregation" else mean))


def _out(rows, cap, dtype):
    return (torch.zeros(rows + 1, dtype=torch.int32, device="cuda"),
            torch.zeros(cap, dtype=torch.int32, device="cuda"),
            torch.zeros(cap, dtype=dtype, device="cuda"))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mcl":
        return dict(kind=kind, X=_mcl_input(case, seed), plan=binding.Plan(),
                    prune=case["prune"], topk=case["topk"], order=case["order"],
                    out=_out(case["n"], _capacity(case), torch.float32))
    if kind == "stages":
        graph = StageGraph(_pairs(case, seed), capacity=_capacity(case))
        graph.col.zero_()
        graph.vals.zero_()
        return dict(kind=kind, graph=graph)
    if kind == "permute":
        A, p = _operands(case, seed)
        return dict(kind=kind, A=A, p=p, plan=binding.Plan(),
                    out=_out(case["m"], _capacity(case), A.vals.dtype))
    A, B = _operands(case, seed)
    if kind == "product":
        return dict(kind=kind, A=A, B=B, plan=binding.Plan(),
                    out=_out(case["m"], _capacity(case), A.vals.dtype))
    pat = autograd.SpGEMMPattern(A, B, deterministic=case["deterministic"])
    return dict(kind=kind, A=A, B=B, pat=pat, a=A.vals.clone().requires_grad_(),
                b=B.vals.clone().requires_grad_(),
                w=_values((pat.nnz,), "normal", A.vals.dtype, _gen(seed, 9)))


def run(state):
    kind = state["kind"]
    if kind == "product":
        A, B, plan = state["A"], state["B"], state["plan"]
        rp, col, vals = state["out"]
        _, nnz = plan.symbolic([A], [B], rp=rp)
        if nnz > col.numel():
            raise ValueError("output buffers too small")
        plan.numeric([A], [B], rp, nnz, col=col, vals=vals)
        return rp, col, vals
    if kind == "permute":
        binding.permute(state["A"], state["p"], state["p"], plan=state["plan"],
                        out=state["out"])
        return state["out"]
    if kind == "stages":
        g = state["graph"]
        g.replay()
        return g.row_ptr, g.col, g.vals
    if kind == "train":
        state["a"].grad = state["b"].grad = None
        c = autograd.spgemm_values(state["a"], state["b"], state["A"], state["B"], state["pat"])
        c.backward(state["w"])
        return c.detach(), state["a"].grad, state["b"].grad
    binding.mcl_iteration(state["X"], 2, state["prune"], state["topk"], plan=state["plan"],
                          out=state["out"], order=state["order"])
    return state["out"]


# ---------------------------------------------------------------- work

def work(case):
    """Each operand read once, each result written once (the expected number
    of distinct columns where the pattern is random)."""
    kind = case["kind"]
    if kind == "mcl":
        n, d = case["n"], case["d"]
        out = n * (min(case["topk"], 0.04 * n) if case["a"] == "mixed" else d)
        return dict(bytes=8.0 * (n * d + out) + 8.0 * n, flops=2.0 * n * d * d)
    vb = 8 if case["dtype"] == "f64" else 4
    ent = 4 + vb
    m, mean = case["m"], (case["lo"] + case["hi"]) / 2.0
    if kind == "permute":
        return dict(bytes=2 * (4.0 * m + ent * m * mean) + 8.0 * m, flops=0.0)
    n = case["n"]
    if kind == "stages":
        k = case["K"] * (case["kmin"] + case["kmax"]) / 2.0
        a_nnz = 15.7 * m if case["a"] == "rmat" else case["K"] * m * mean
        if case["a"] == "rmat":
            k = m
    else:
        a_nnz, k = m * mean, case["k"]
    b_mean = mean
    if kind == "product" and case["b"] == "aggregation":
        b_mean = 1.0
    p = a_nnz * b_mean
    out = m * n * -math.expm1(-p / (float(m) * n)) if p < 50.0 * m * n else float(m) * n
    b_nnz = 0.0 if kind == "product" and case["b"] == "same" else k * b_mean
    total = 4.0 * (2 * m + k) + ent * (a_nnz + b_nnz + out)
    if kind == "train":  # W read, C's columns read; both gradients written
        return dict(bytes=2 * total, flops=6.0 * p)
    return dict(bytes=total, flops=2.0 * p)


# ---------------------------------------------------------------- exact

def _products(A, B, r0, r1):
    """Every scalar product of rows [r0, r1) of A B: (row, column, position in
    A, position in B)."""
    s, e = int(A.row_ptr[r0]), int(A.row_ptr[r1])
    ac = A.col_idx[s:e].long()
    bs = B.row_ptr.long()
    lens = bs[ac + 1] - bs[ac]
    rows = torch.repeat_interleave(
        torch.arange(r0, r1, device="cuda"),
        (A.row_ptr[r0 + 1:r1 + 1] - A.row_ptr[r0:r1]).long())
    pa = torch.repeat_interleave(torch.arange(s, e, device="cuda"), lens)
    first = torch.cumsum(lens, 0) - lens
    pb = torch.arange(pa.numel(), device="cuda") - first[pa - s] + bs[ac][pa - s]
    return rows[pa - s], B.col_idx[pb].long(), pa, pb


def _sum_of_products(pairs, m, n):
    """Row counts, columns and 64-bit values of sum_k A_k B_k."""
    p = sum(float(A.nnz) * B.nnz / max(1, B.shape[0]) for A, B in pairs)
    step = max(1, int(m / max(1.0, p / 6e7)))
    counts = torch.zeros(m, dtype=torch.int64, device="cuda")
    cols, vals = [], []
    for r0 in range(0, m, step):
        keys, prod = [], []
        for A, B in pairs:
            r, c, pa, pb = _products(A, B, r0, min(m, r0 + step))
            keys.append(r * n + c)
            prod.append(A.vals[pa].double() * B.vals[pb].double())
            del r, c, pa, pb
        u, inv = torch.unique(torch.cat(keys), return_inverse=True)
        del keys
        v = torch.zeros(u.numel(), dtype=torch.float64, device="cuda")
        v.index_add_(0, inv, torch.cat(prod))
        counts += torch.bincount(u // n, minlength=m)
        cols.append((u % n).int())
        vals.append(v)
    return counts, torch.cat(cols), torch.cat(vals)


def _filled(case, counts, col, vals):
    """Row pointer, columns and values as the output buffers hold them."""
    rp, c, v = _out(counts.numel(), _capacity(case), torch.float64)
    rp[1:] = torch.cumsum(counts, 0)
    c[:col.numel()] = col
    v[:vals.numel()] = vals
    return rp, c, v


def exact(case, seed):
    kind = case["kind"]
    if kind == "product":
        A, B = _operands(case, seed)
        return _filled(case, *_sum_of_products([(A, B)], A.shape[0], B.shape[1]))
    if kind == "stages":
        return _filled(case, *_sum_of_products(_pairs(case, seed), case["m"], case["n"]))
    if kind == "permute":
        A, p = _operands(case, seed)
        p = p.long()
        key, order = (p[_rows_of(A)] * A.shape[1] + p[A.col_idx.long()]).sort()
        return _filled(case, torch.bincount(key // A.shape[1], minlength=A.shape[0]),
                       (key % A.shape[1]).int(), A.vals[order].double())
    if kind == "train":
        A, B = _operands(case, seed)
        r, c, pa, pb = _products(A, B, 0, A.shape[0])
        u, inv = torch.unique(r * B.shape[1] + c, return_inverse=True)
        del r, c
        w = _values((u.numel(),), "normal", A.vals.dtype, _gen(seed, 9)).double()[inv]
        a, b = A.vals.double()[pa], B.vals.double()[pb]
        out = [torch.zeros(k, dtype=torch.float64, device="cuda")
               for k in (u.numel(), A.nnz, B.nnz)]
        out[0].index_add_(0, inv, a * b)
        out[1].index_add_(0, pa, w * b)
        out[2].index_add_(0, pb, w * a)
        return out
    if case["a"] == "mixed":  # entries at the thresholds may fall either way in 32 bits
        return None
    # no entry is near the threshold: clusters are kept, links between them dropped
    n, X = case["n"], _mcl_input(case, seed)
    counts, col, v = _sum_of_products([(X, X)], n, n)
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), counts)
    if case["order"] == "workload":
        v = v * v

    def by_row_sum(rows, v):
        return v / torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, v)[rows]

    v = by_row_sum(rows, v)
    keep = v >= case["prune"]
    rows, col, v = rows[keep], col[keep], v[keep]
    v = by_row_sum(rows, v) if case["order"] == "workload" else v * v
    return _filled(case, torch.bincount(rows, minlength=n), col, v)
