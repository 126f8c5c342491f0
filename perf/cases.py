"""Timed cases of the library's public calls, over the range it is used for.

A case is one call that a program makes on matrices it already holds on the
GPU: the lower triangle tril(A A^T), an off-diagonal block or half of one, the
mirror of a stored lower part, the product with a stored lower part, one
accumulated stage, or the execution of a plan for new values.  The matrices
have the shapes of the repository's workloads (uniform rows, k-mer overlap
patterns, R-MAT graphs), drawn on the GPU: the case gives the pattern, the seed
its row and column labels and every value.
"""
import math

import numpy as np
import torch

import paper_2608_09713_amd as sp

DEV = "cuda:0"
MAX_COL = 50    # k-mer shape: columns with more entries are dropped
ZIPF = 0.9      # k-mer shape: exponent of the column ranks' law
FLOAT = {"f64": torch.float64, "f32": torch.float32}
OUT = {"f64": torch.float64, "f32": torch.float32, "count": torch.int32, "jaccard": torch.float32}
OUT_BYTES = {"f64": 8, "f32": 4, "count": 4, "jaccard": 4}
IN_BYTES = {"f64": 8, "f32": 4, "count": 0, "jaccard": 0}


def listed():
    return [
        # the smallest diagonal block: launches and host waits are the whole cost
        dict(name="lower_f64_tiny", op="lower", shape="uniform", semiring="f64", m=4096, n=16384, d=8),
        # a diagonal block of a process grid, rows of 0 to 48 entries, sizes that divide by nothing
        dict(name="lower_f64_ragged", op="lower", shape="ragged", semiring="f64", m=400_009, n=12_000_017, d=24),
        # k-mer overlap counts of a read set
        dict(name="lower_count_kmer", op="lower", shape="kmer", semiring="count", m=1 << 20, n=1 << 26, d=32),
        # Jaccard similarities of a large sample set: the benchmark's default
        dict(name="lower_jaccard_large", op="lower", shape="kmer", semiring="jaccard", m=1 << 23, n=1 << 28, d=16),
        # A A^T of a power-law graph: hub columns, rows of millions of products, gigabytes of output
        dict(name="lower_f32_rmat", op="lower", shape="rmat", semiring="f32", scale=19),
        # the off-diagonal block of two processes' rows
        dict(name="offdiag_f64", op="offdiag", shape="uniform", semiring="f64", m=1 << 19, n=1 << 24, d=24),
        # the full matrix from the lower part: long rows (a graph)
        dict(name="mirror_f32_rmat", op="mirror", shape="rmat", semiring="f32", scale=17),
        # the full matrix from the lower part: short rows (k-mer overlaps)
        dict(name="mirror_count_kmer", op="mirror", shape="kmer", semiring="count", m=1 << 20, n=1 << 26, d=32),
        # one product of an iteration that changes values on a fixed pattern
        dict(name="execute_f64", op="execute", shape="uniform", semiring="f64", m=1 << 19, n=1 << 24, d=24),
        # the second stage of a sum over column blocks
        dict(name="accumulate_count_kmer", op="accumulate", shape="kmer", semiring="count", m=1 << 20, n=1 << 25, d=16),
        # C x from a large similarity matrix's lower part, one vector
        dict(name="symm_jaccard_k1", op="symm", shape="kmer", semiring="jaccard", m=1 << 23, n=1 << 28, d=16, k=1),
        # C X from a block's lower part, a panel of vectors
        dict(name="symm_f64_k8", op="symm", shape="uniform", semiring="f64", m=1 << 19, n=1 << 24, d=24, k=8),
    ]


def draw(rng):
    """One more case: a call, a shape that it is used with, a value type, and
    sizes spread over their logarithm, odd ones among them."""
    op = rng.choice(["lower", "lower", "lower", "offdiag", "half_top", "half_right", "mirror", "execute",
                     "accumulate", "symm"])
    two = op in ("offdiag", "half_top", "half_right")
    shape = rng.choice(["uniform", "ragged", "kmer"] if two else ["uniform", "ragged", "kmer", "rmat"])
    if shape == "rmat":
        semiring = rng.choice(["f32", "f64"])
        case = dict(op=op, shape=shape, semiring=semiring, scale=rng.randint(11, 16 if op in ("symm", "accumulate") else 17))
    else:
        if shape == "kmer":
            semiring = rng.choice(["count", "jaccard"]) if op not in ("accumulate", "execute") else rng.choice(["count", "f32"])
            d = rng.randint(12, 32)
        else:
            semiring = rng.choice(["f64", "f64", "f32", "count"])
            d = rng.randint(6, 32)
        m = int(2 ** rng.uniform(11, 21))
        n = int(m * 2 ** rng.uniform(2, 6))
        if rng.random() < 0.7:
            m, n = m | 1, n | 1
        case = dict(op=op, shape=shape, semiring=semiring, m=m, n=n, d=d)
    if op == "symm":
        case["k"] = rng.choice([1, 1, 2, 5, 8, 16])
    return case


# ---- inputs

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _values(nnz, dtype, g):
    """Uniform in (0, 1]."""
    return 1.0 - torch.rand(nnz, dtype=dtype, device=DEV, generator=g)


def _relabel(case, seed, m, n):
    """Row and column labels of the seed.  Other labels give other inputs and
    other results, while the number of row pairs that share a column (and with
    it the sizes of tril(A A^T), of a block and of its halves) stays: the rows
    are permuted within each half, the columns all over."""
    g = _gen(seed, 30)
    half = m // 2
    rows = torch.cat([torch.randperm(half, device=DEV, generator=g),
                      half + torch.randperm(m - half, device=DEV, generator=g)])
    if case["shape"] == "rmat":  # one label per vertex
        return rows, lambda c: rows[c]
    a = (int(seed) * 2654435761 + 40503) % n | 1
    while math.gcd(a, n) != 1:
        a = (a + 2) % n or 1
    return rows, lambda c: c.mul(a).add_(int(seed) * 7919 % n).remainder_(n)


def _pattern(case, seed, stream):
    """row_ptr and col_idx of one matrix of the case's shape, labelled by the seed."""
    g = _gen(0, stream)
    if case["shape"] == "rmat":
        s = case["scale"]
        m = n = 1 << s
        ne = 16 << s
        rows = torch.zeros(ne, dtype=torch.int64, device=DEV)
        cols = torch.zeros(ne, dtype=torch.int64, device=DEV)
        for _ in range(s):
            u = torch.rand(ne, device=DEV, generator=g)
            rows = (rows << 1) | (u >= 0.76).long()
            cols = (cols << 1) | (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).long()
        mix = torch.randperm(n, device=DEV, generator=g)  # (hubs anywhere)
        key = torch.unique((mix[rows] << s | mix[cols])[rows != cols])
        rows, cols = key >> s, key & (n - 1)
    else:
        m, n, d = case["m"], case["n"], case["d"]
        width = 2 * d if case["shape"] == "ragged" else d
        u = torch.rand((m, width), dtype=torch.float64, device=DEV, generator=g)
        if case["shape"] == "kmer":
            # bounded Zipf by inverting the integral of x^-s over [1, n + 1)
            q = 1.0 - ZIPF
            cols = (u.mul_((n + 1.0) ** q - 1.0).add_(1.0)).pow_(1.0 / q).long().sub_(1).clamp_(0, n - 1)
        else:
            cols = u.mul_(n).long().clamp_(0, n - 1)
        if case["shape"] == "ragged":
            lens = torch.randint(0, width + 1, (m, 1), device=DEV, generator=g)
            cols[torch.arange(width, device=DEV)[None, :] >= lens] = n
        cols = cols.sort(dim=1).values
        keep = cols < n
        keep[:, 1:] &= cols[:, 1:] != cols[:, :-1]
        if case["shape"] == "kmer":
            count = torch.bincount(cols[keep], minlength=n)
            keep &= count[cols] <= MAX_COL
            del count
        rows = torch.repeat_interleave(torch.arange(m, device=DEV), keep.sum(1))
        cols = cols[keep]
    label, relabel = _relabel(case, seed, m, n)
    key = (label[rows] * n + relabel(cols)).sort().values
    rows = torch.div(key, n, rounding_mode="floor")
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.bincount(rows, minlength=m).cumsum(0)
    return row_ptr, (key - rows * n).int()


def _ncols(case):
    return 1 << case["scale"] if case["shape"] == "rmat" else case["n"]


def _matrix(case, seed, stream):
    row_ptr, cols = _pattern(case, seed, stream)
    dtype = FLOAT.get(case["semiring"])
    values = _values(cols.numel(), dtype, _gen(seed, stream + 1)) if dtype else None
    return sp.DeviceCSR(row_ptr.numel() - 1, _ncols(case), row_ptr, cols, values, cols.numel())


def _vectors(case, seed, m):
    dtype = torch.float64 if case["semiring"] in ("f64", "count") else torch.float32
    return _values(m * case["k"], dtype, _gen(seed, 20)).view(m, case["k"])


def prepare(case, seed):
    op, sr = case["op"], case["semiring"]
    A = _matrix(case, seed, 1)
    state = dict(op=op, semiring=sr)
    if op == "lower":
        state["A"] = A
    elif op in ("offdiag", "half_top", "half_right"):
        state.update(A=A, B=_matrix(case, seed, 3))
    elif op == "mirror":
        state["C"] = sp.lower(A, sr)
    elif op == "execute":
        plan, _ = sp.lower_plan(A, sr)
        state.update(plan=plan, values=None if sr == "count" else _values(A.nnz, FLOAT[sr], _gen(seed, 10)))
    elif op == "accumulate":
        state.update(C=sp.lower(A, sr), A=_matrix(case, seed, 5))
    else:
        state.update(C=sp.lower(A, sr), X=_vectors(case, seed, A.nrows))
    return state


def run(state):
    op, sr = state["op"], state["semiring"]
    if op == "lower":
        C = sp.lower(state["A"], sr)
    elif op == "offdiag":
        C = sp.offdiag(state["A"], state["B"], sr)
    elif op in ("half_top", "half_right"):
        C = sp.offdiag_half(state["A"], state["B"], op[5:], sr)
    elif op == "mirror":
        C = sp.mirror(state["C"], sr)
    elif op == "execute":
        C = state["plan"].execute(state["values"])
    elif op == "accumulate":
        C = sp.lower_accumulate(state["C"], state["A"], sr)
    else:
        return dict(Y=sp.symm(state["C"], state["X"], sr))
    return dict(row_ptr=C.row_ptr, col_idx=C.col_idx, values=C.values)


# ---- what a call cannot do without

# entries of A, lower multiply-adds and entries of tril(A A^T) of the R-MAT
# graph of scale 11 to 20 (edge factor 16), in units of 2^scale, counted
_RMAT = {11: (12.446, 577.6, 196.6), 12: (13.026, 825.5, 293.9), 13: (13.508, 1164.2, 425.9),
         14: (13.931, 1625.0, 616.6), 15: (14.286, 2241.6, 880.4), 16: (14.578, 3075.9, 1247.7),
         17: (14.821, 4158.8, 1750.5), 18: (15.025, 5602.7, 2434.6), 19: (15.197, 7501.6, 3370.1),
         20: (15.341, 9988.2, 4625.7)}


def _sizes(case):
    """(nnz of one operand, partner pairs in one operand, pairs between two
    operands), expected values for the case's shape."""
    if case["shape"] == "rmat":
        v = 1 << case["scale"]
        e, f, _ = _RMAT[case["scale"]]
        return v * e, v * (f - e), v * (2 * f - e)
    m, n, d = case["m"], case["n"], case["d"]
    if case["shape"] != "kmer":
        nnz = float(m) * d
        return nnz, nnz * nnz / (2.0 * n), nnz * nnz / n
    # entries per column: Poisson about m d p(rank), dropped above MAX_COL
    q = 1.0 - ZIPF
    edge = np.unique(np.concatenate([np.arange(1, 64), np.geomspace(64, n + 1, 1500)]))
    width, mid = np.diff(edge), np.sqrt(edge[1:] * edge[:-1])
    lam = m * d * q * mid ** -ZIPF / ((n + 1.0) ** q - 1.0)
    k = np.arange(MAX_COL + 1)[:, None]
    logk = np.array([math.lgamma(x + 1.0) for x in range(MAX_COL + 1)])[:, None]
    p = np.exp(k * np.log(lam) - lam - logk)
    one = (p * k).sum(0)
    return float((one * width).sum()), float((p * k * (k - 1) / 2 * width).sum()), float((one * one * width).sum())


def work(case):
    """Every input read once, every output written once; two operations per
    multiply-add (per stored value of the product for C X)."""
    op, sr = case["op"], case["semiring"]
    m = 1 << case["scale"] if case["shape"] == "rmat" else case["m"]
    nnz, pairs, between = _sizes(case)
    a = 8.0 * (m + 1) + nnz * (4 + IN_BYTES[sr])
    low = m * _RMAT[case["scale"]][2] if case["shape"] == "rmat" else pairs + m
    c = 8.0 * (m + 1) + low * (4 + OUT_BYTES[sr])
    flops = 2.0 * (pairs + nnz)
    if op == "lower":
        return dict(bytes=a + c, flops=flops)
    if op in ("offdiag", "half_top", "half_right"):
        part = 1.0 if op == "offdiag" else 0.5
        out = 8.0 * (m + 1) + part * between * (4 + OUT_BYTES[sr])
        return dict(bytes=(1.0 + part) * a + out, flops=2.0 * part * between)
    if op == "mirror":
        return dict(bytes=c + 8.0 * (m + 1) + 2.0 * low * (4 + OUT_BYTES[sr]), flops=0.0)
    if op == "execute":
        return dict(bytes=a + c, flops=flops)
    if op == "accumulate":
        both = low if case["shape"] == "rmat" else 2.0 * low - m
        return dict(bytes=a + c + 8.0 * (m + 1) + both * (4 + OUT_BYTES[sr]), flops=flops + low)
    x = 8 if sr in ("f64", "count") else 4
    return dict(bytes=c + 2.0 * m * case["k"] * x, flops=4.0 * low * case["k"])


def tolerance(case):
    """Counts, Jaccard values (one correctly rounded division of exact counts)
    and copies are the same bits in any order.  Plus-times products and sums
    are formed in 64 bits: f64 results differ by the order of positive terms,
    f32 results by that and one rounding to 24 bits; so does C X."""
    op, sr = case["op"], case["semiring"]
    if op == "mirror" or (op != "symm" and sr in ("count", "jaccard")):
        return "exact"
    if sr in ("f64", "count"):
        return dict(rel=1e-14, max=1e-13)
    return dict(rel=1e-7, max=1e-6)


# ---- the same results in plain torch, 64 bits

def _exact_product(rpa, cia, va, rpb, cib, vb, lower, jaccard):
    """A B^T (or its lower triangle, B = A) as sorted (row, column, value):
    every product expanded, sorted by (row, column) and summed, in blocks of
    rows.  Values are counts where va is None."""
    ma, mb = rpa.numel() - 1, rpb.numel() - 1
    lena, lenb = rpa.diff(), rpb.diff()
    rowa = torch.repeat_interleave(torch.arange(ma, device=DEV), lena)
    rowb = torch.repeat_interleave(torch.arange(mb, device=DEV), lenb)
    n = int(max(cia.max(), cib.max())) + 1 if cia.numel() and cib.numel() else 1
    order = torch.sort(cib.long(), stable=True).indices
    start = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    start[1:] = torch.bincount(cib, minlength=n).cumsum(0)
    first = start[cia.long()]
    if lower:  # the entries of the column with a row up to the entry's own
        place = torch.empty_like(order)
        place[order] = torch.arange(order.numel(), device=DEV)
        count = place - first + 1
    else:
        count = start[cia.long() + 1] - first
    del start
    total = torch.zeros(count.numel() + 1, dtype=torch.int64, device=DEV)
    total[1:] = count.cumsum(0)
    at = total[rpa].cpu().numpy()  # products before every row
    rows, cols, vals = [], [], []
    r = 0
    while r < ma:
        end = max(r + 1, int(np.searchsorted(at, at[r] + (1 << 28), side="right")) - 1)
        e0, e1 = int(rpa[r]), int(rpa[end])
        c = count[e0:e1]
        e = torch.repeat_interleave(torch.arange(e0, e1, device=DEV), c)
        t = torch.arange(e.numel(), device=DEV) + int(at[r])
        p = order[first[e] + (t - total[e])]
        del t
        key = rowa[e] * mb + rowb[p]
        v = va[e].double() * vb[p].double() if va is not None else None
        del e, p
        key, by = torch.sort(key)
        key, group, times = torch.unique_consecutive(key, return_inverse=True, return_counts=True)
        if va is not None:
            v = torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, group, v[by])
        else:
            v = times.double()
        del group, by, times
        i, j = key // mb, key % mb
        if jaccard:
            v = v / (lena[i] + lenb[j] - v)
        rows.append(i.int())
        cols.append(j.int())
        vals.append(v)
        r = end
    return torch.cat(rows), torch.cat(cols), torch.cat(vals)


def _csr(m, rows, cols, vals, sr):
    rp = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.bincount(rows, minlength=m).cumsum(0)
    return dict(row_ptr=rp, col_idx=cols, values=vals.round().int() if sr == "count" else vals)


def exact(case, seed):
    op, sr = case["op"], case["semiring"]
    A = _matrix(case, seed, 1)
    m, jac = A.nrows, sr == "jaccard"
    if op in ("offdiag", "half_top", "half_right"):
        B = _matrix(case, seed, 3)
        i, j, v = _exact_product(A.row_ptr, A.col_idx, A.values, B.row_ptr, B.col_idx, B.values, False, jac)
        if op == "half_top":
            keep = i < m // 2
            return _csr(m // 2, i[keep], j[keep], v[keep], sr)
        if op == "half_right":
            keep = j >= B.nrows // 2
            i, j, v = i[keep], j[keep], v[keep]
        return _csr(m, i, j, v, sr)
    val = A.values if op != "execute" or sr == "count" else _values(A.nnz, FLOAT[sr], _gen(seed, 10))
    i, j, v = _exact_product(A.row_ptr, A.col_idx, val, A.row_ptr, A.col_idx, val, True, jac)
    if op in ("lower", "execute"):
        return _csr(m, i, j, v, sr)
    v = v.to(OUT[sr]).double()  # (the later calls start from a stored C_L)
    if op == "accumulate":
        B = _matrix(case, seed, 5)
        i2, j2, v2 = _exact_product(B.row_ptr, B.col_idx, B.values, B.row_ptr, B.col_idx, B.values, True, jac)
        key, by = torch.sort(torch.cat([i.long() * m + j, i2.long() * m + j2]))
        key, group = torch.unique_consecutive(key, return_inverse=True)
        v = torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, group, torch.cat([v, v2])[by])
        return _csr(m, key // m, (key % m).int(), v, sr)
    off = i != j
    if op == "mirror":
        key, by = torch.sort(torch.cat([i.long() * m + j, j[off].long() * m + i[off]]))
        return _csr(m, key // m, (key % m).int(), torch.cat([v, v[off]])[by], sr)
    X = _vectors(case, seed, m).double()
    Y = torch.zeros_like(X)
    i, j = i.long(), j.long()
    for c in range(case["k"]):
        Y[:, c].index_add_(0, i, v * X[j, c])
        Y[:, c].index_add_(0, j[off], v[off] * X[i[off], c])
    return dict(Y=Y)
