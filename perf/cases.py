"""The work that this library is used for, as cases that can be timed and compared.

Every case goes through the package's public entry points as a user's program
calls them.  Graphs are symmetric R-MAT(.57,.19,.19,.05) with self-loops and
the normalised values 1/sqrt(d_i d_j); sparse features have every entry
present with probability rho and U[-1, 1) values: the inputs of the bench and
of the tests, built here with torch on the device so that they are quick to
make.  Kinds of work:

  aggregate  C = A X: plan and product in one pass (what a program does for
             every new feature matrix), A's values given or derived (sym_norm)
  twohop     C = A A: plan and product
  serve      the allocation-free product with a plan and output arrays kept
  combine    Y = relu(C W): the layer's weights on aggregated sparse features
  propagate  Y = A H with dense H: a deeper layer forward, and the backward
             pass (A is symmetric)
  stream     C = A X with A and X in pinned host memory, C returned there,
             under a device budget
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2507_02006_amd as aires

ABC = (0.57, 0.19, 0.19)
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def listed():
    return [
        # one sampled subgraph or a small citation graph: latency and launches
        dict(name="aggregate-tiny", kind="aggregate", n=4096, deg=16, f=256, rho=0.10, values="given", rp64=False),
        # derived values and 64-bit row pointers on ragged sizes
        dict(name="aggregate-derived", kind="aggregate", n=100003, deg=20, f=200, rho=0.08, values="sym_norm", rp64=True),
        # the mid-sized aggregation of the bench
        dict(name="aggregate-mid", kind="aggregate", n=262144, deg=32, f=512, rho=0.05, values="given", rp64=False),
        # bag-of-words features: thousands of columns, one in a hundred present
        dict(name="aggregate-words", kind="aggregate", n=60013, deg=12, f=6001, rho=0.01, values="given", rp64=False),
        # a graph of millions of nodes, resident in HBM
        dict(name="aggregate-large", kind="aggregate", n=8388608, deg=24, f=128, rho=0.10, values="given", rp64=False),
        # two-hop adjacency of a small and of a large graph
        dict(name="twohop-small", kind="twohop", n=12000, deg=10, rp64=False),
        dict(name="twohop-large", kind="twohop", n=524288, deg=16, rp64=False),
        # inference on a fixed graph without allocation
        dict(name="serve-noalloc", kind="serve", n=16384, deg=16, f=64, rho=0.10, rp64=False),
        # the layer's weights and activation on aggregated features
        dict(name="combine-mid", kind="combine", n=262144, deg=32, f=512, rho=0.05, fout=256, rp64=True),
        # dense hidden features, wide, and an output layer with an odd number of classes
        dict(name="propagate-wide", kind="propagate", n=1048576, deg=16, fout=256, rp64=False),
        dict(name="propagate-classes", kind="propagate", n=150001, deg=14, fout=41, rp64=False),
        # out of core: tiles from pinned host memory and back
        dict(name="stream-host", kind="stream", n=2000000, deg=22, f=64, rho=0.10, budget_mb=2048, rp64=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["aggregate", "aggregate", "aggregate", "twohop", "serve", "combine", "propagate", "propagate",
                       "stream"])
    rp64 = rng.random() < 0.4
    deg = rng.randint(8, 32)
    if kind == "aggregate":
        values = rng.choice(["given", "given", "sym_norm"])
        if rng.random() < 0.25:  # bag of words
            n, f = _log(rng, 2000, 120000), rng.randint(2049, 12000)
            rho = round(min(rng.uniform(0.002, 0.02), 80.0 / f), 4)
        else:
            f = _log(rng, 16, 2048)
            rho = round(min(rng.uniform(0.01, 0.15), 100.0 / f), 4)
            # no more products than the largest listed case
            most = min(4.0e6, 1.6e9 / (deg * max(1.0, f * rho)), 8.0e8 / f)
            n = _log(rng, 2000, max(4000, most))
        return dict(kind=kind, n=n, deg=deg, f=f, rho=rho, values=values, rp64=rp64)
    if kind == "twohop":
        return dict(kind=kind, n=_log(rng, 2000, 250000), deg=rng.randint(6, 16), rp64=rp64)
    if kind == "serve":
        f = _log(rng, 16, 512)
        return dict(kind=kind, n=_log(rng, 1000, 100000), deg=deg, f=f, rho=round(rng.uniform(0.02, 0.12), 4), rp64=rp64)
    if kind == "combine":
        return dict(kind=kind, n=_log(rng, 4000, 262144), deg=deg, f=rng.randint(64, 512),
                    rho=round(rng.uniform(0.003, 0.1), 4), fout=_log(rng, 7, 512), rp64=rp64)
    if kind == "propagate":
        return dict(kind=kind, n=_log(rng, 2000, 700000), deg=rng.randint(8, 20), fout=_log(rng, 7, 512), rp64=rp64)
    return dict(kind=kind, n=_log(rng, 50000, 2000000), deg=rng.randint(8, 22), f=_log(rng, 16, 64),
                rho=round(rng.uniform(0.03, 0.1), 4), budget_mb=rng.choice([1536, 2048, 4096]), rp64=rp64)


# ----------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rmat(n, deg, g):
    """Distinct edges u * n + v of a symmetric R-MAT graph with self-loops."""
    want, levels = n * deg // 2, max(1, (n - 1).bit_length())
    a, b, c = ABC
    us, vs, have = [], [], 0
    while have < want:
        s = min(want - have, 1 << 25)
        s += s // 4 + 64
        u = torch.zeros(s, dtype=torch.int32, device=DEV)
        v = torch.zeros(s, dtype=torch.int32, device=DEV)
        for _ in range(levels):
            r = torch.rand(s, generator=g, device=DEV)
            u = 2 * u + (r >= a + b)
            v = 2 * v + (((r >= a) & (r < a + b)) | (r >= a + b + c))
        ok = ((u < n) & (v < n)).nonzero().squeeze(1)[: want - have]
        us.append(u[ok])
        vs.append(v[ok])
        have += ok.numel()
    u, v, d = torch.cat(us).long(), torch.cat(vs).long(), torch.arange(n, device=DEV)
    del us, vs
    return torch.unique(torch.cat([u * n + v, v * n + u, d * n + d]))


def _row_ptr(lens, rp64):
    rp = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    rp[1:] = lens.cumsum(0)
    return rp if rp64 else rp.to(torch.int32)


def _graph(n, key, perm, rp64):
    """The graph with its vertices renumbered, values 1/sqrt(d_i d_j)."""
    key = torch.sort(perm[key // n] * n + perm[key % n])[0]
    row, col = key // n, (key % n).to(torch.int32)
    rp = _row_ptr(torch.bincount(row, minlength=n), rp64)
    inv = (rp[1:] - rp[:-1]).double().rsqrt()
    return n, n, rp, col, (inv[row] * inv[col.long()]).float()


def _sparse(n, f, p, base, perm, g, scaled=False, rp64=False):
    """CSR (n x f): entry present with probability p (a number, or one per
    vertex), vertices and columns renumbered, U[-1, 1) values (over
    sqrt(f p) of the row when scaled)."""
    step = max(1, (1 << 27) // f)
    mask = torch.empty((n, f), dtype=torch.bool, device=DEV)
    for r0 in range(0, n, step):
        q = p if isinstance(p, float) else p[r0:r0 + step, None]
        torch.lt(torch.rand(mask[r0:r0 + step].shape, generator=base, device=DEV), q, out=mask[r0:r0 + step])
    old = torch.empty_like(perm)
    old[perm] = torch.arange(n, device=DEV)
    order = torch.randperm(f, generator=g, device=DEV)
    cols, vals, lens = [], [], []
    for r0 in range(0, n, step):
        at = mask[old[r0:r0 + step]][:, order].nonzero()
        lens.append(torch.bincount(at[:, 0], minlength=min(n, r0 + step) - r0))
        cols.append(at[:, 1].to(torch.int32))
        v = torch.rand(at.shape[0], generator=g, device=DEV) * 2 - 1
        vals.append(v * (f * p[old[r0 + at[:, 0]]]).rsqrt() if scaled else v)
        del at
    return n, f, _row_ptr(torch.cat(lens), rp64), torch.cat(cols), torch.cat(vals)


def _inputs(case, seed):
    """One graph (and pattern of features) per case, so that C has as many
    entries for every seed; the seed renumbers vertices and columns, which
    moves every entry, and draws the values."""
    kind, n = case["kind"], case["n"]
    base, g = _gen(4711), _gen(seed)
    key = _rmat(n, case["deg"], base)
    perm = torch.randperm(n, generator=g, device=DEV)
    if kind == "combine":
        # an aggregate of d_i rows of density rho: an entry is present with
        # probability 1 - (1 - rho)^d_i
        p = 1 - (1 - case["rho"]) ** torch.bincount(key // n, minlength=n).float()
        C = _sparse(n, case["f"], p, base, perm, g, scaled=True, rp64=case["rp64"])
        return C, (torch.rand((case["f"], case["fout"]), generator=g, device=DEV) - 0.5)
    A = _graph(n, key, perm, case["rp64"])
    if kind == "twohop":
        return A, A
    if kind == "propagate":
        return A, torch.rand((n, case["fout"]), generator=g, device=DEV) * 2 - 1
    return A, _sparse(n, case["f"], case["rho"], base, perm, g)


def prepare(case, seed):
    A, B = _inputs(case, seed)
    kind = case["kind"]
    if kind == "aggregate" and case["values"] == "sym_norm":
        A = A[:4] + (None,)
    if kind == "serve":
        n = case["n"]
        most = n * case["f"]
        return dict(kind=kind, plan=aires.tile_plan(A, B), rp=torch.empty(n + 1, dtype=torch.int64, device=DEV),
                    col=torch.empty(most, dtype=torch.int32, device=DEV),
                    val=torch.empty(most, dtype=torch.float32, device=DEV))
    if kind == "stream":
        A, B = ((M[0], M[1]) + tuple(x.cpu().pin_memory() for x in M[2:]) for M in (A, B))
        return dict(kind=kind, A=A, B=B, budget=case["budget_mb"] << 20)
    s = dict(kind=kind, A=A, B=B)
    if kind == "aggregate":
        s["values"] = case["values"]
    return s


class _Held(np.ndarray):
    """A view of pinned memory that keeps the library's output alive."""


def _held(C, x):
    v = x.view(_Held)
    v.owner = C
    return v


def run(s):
    kind = s["kind"]
    if kind in ("aggregate", "twohop"):
        with aires.tile_plan(s["A"], s["B"], a_values=s.get("values", "given")) as plan:
            C = aires.spgemm(plan)
        return [C.rp, C.col, C.val]
    if kind == "serve":
        nnz = aires.spgemm_noalloc(s["plan"], s["rp"], s["col"], s["val"])
        return [s["rp"], s["col"][:nnz], s["val"][:nnz]]
    if kind == "combine":
        return aires.spmm(s["A"], s["B"], relu=True)
    if kind == "propagate":
        return aires.spmm(s["A"], s["B"])
    with aires.tile_plan(s["A"], s["B"], s["budget"], c_on_host=True) as plan:
        C = aires.spgemm(plan)
    return [_held(C, x) for x in (C.rp, C.col, C.val)]


# --------------------------------------------------------- work and exact

def _unions(A, B, want_values):
    """C = A B in 64 bits by row blocks: yields (row lengths, columns, values)."""
    m, N = A[0], B[1]
    arp, brp = A[2].long(), B[2].long()
    acol, bcol = A[3].long(), B[3].long()
    blen = brp[1:] - brp[:-1]
    pcum = torch.zeros(A[3].numel() + 1, dtype=torch.int64, device=DEV)
    pcum[1:] = blen[acol].cumsum(0)
    prod = pcum[arp]  # products before each row
    ends, r0 = [0], 0
    hp = prod.cpu()
    while r0 < m:  # at most 2^29 slots and about 2^27 products a block
        r1 = int(torch.searchsorted(hp, hp[r0] + (1 << 27), right=True)) - 1
        r0 = min(m, r0 + max(1, (1 << 29) // N), max(r0 + 1, r1))
        ends.append(r0)
    for r0, r1 in zip(ends[:-1], ends[1:]):
        hit = torch.zeros((r1 - r0) * N, dtype=torch.bool, device=DEV)
        acc = torch.zeros((r1 - r0) * N, dtype=torch.float64, device=DEV) if want_values else None
        e0, e1 = int(arp[r0]), int(arp[r1])
        if e1 > e0:
            rows = torch.repeat_interleave(torch.arange(r1 - r0, device=DEV), arp[r0 + 1:r1 + 1] - arp[r0:r1])
            k = acol[e0:e1]
            entry = torch.repeat_interleave(torch.arange(e1 - e0, device=DEV), blen[k])
            at = torch.arange(entry.numel(), device=DEV) - (pcum[e0:e1] - pcum[e0])[entry] + brp[k][entry]
            key = rows[entry] * N + bcol[at]
            hit[key] = True
            if want_values:
                acc.index_add_(0, key, A[4][e0:e1].double()[entry] * B[4][at].double())
            del entry, at, key
        idx = hit.nonzero().squeeze(1)
        lens = torch.bincount(idx // N, minlength=r1 - r0)
        yield lens, (idx % N).to(torch.int32) if want_values else None, acc[idx] if want_values else None
        del hit, acc, idx


@functools.lru_cache(maxsize=64)
def _sizes(items):
    """(nnz(A), nnz(B), products, nnz(C)) of a case's inputs under one seed."""
    case = dict(items)
    A, B = _inputs(case, 1)
    if case["kind"] in ("combine", "propagate"):
        return A[3].numel(), 0, 0, 0
    blen = (B[2][1:] - B[2][:-1]).long()
    products = int(blen[A[3].long()].sum())
    nnzc = int(sum(lens.sum() for lens, _, _ in _unions(A, B, False)))
    return A[3].numel(), B[3].numel(), products, nnzc


def work(case):
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "budget_mb", "values")))
    nnza, nnzb, products, nnzc = _sizes(key)
    n, sA = case["n"], 8 if case["rp64"] else 4
    a = sA * (n + 1) + 8 * nnza
    if case["kind"] in ("combine", "propagate"):
        k = case["f"] if case["kind"] == "combine" else n
        return {"bytes": a + 4 * (k + n) * case["fout"], "flops": 2 * nnza * case["fout"]}
    if case["kind"] == "twohop":
        b = 0  # B is A
    else:
        b = 4 * (n + 1) + 8 * nnzb
        if case.get("values") == "sym_norm":
            a -= 4 * nnza
    return {"bytes": a + b + 8 * (n + 1) + 8 * nnzc, "flops": 2 * products}


def tolerance(case):
    # Measured against 64 bits: fp32 sums 7e-9 to 2e-8 of the result (dense
    # contractions 2.2e-7); two passes on the same inputs, whose sums come in
    # another order, 3e-9.  A two-hop entry may also be summed in 32-bit fixed
    # point, whose absolute error stays below 1e-6.
    if case["kind"] == "twohop":
        return {"rel": 5e-7, "max": 1e-4}
    if case["kind"] == "combine":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 3e-7, "max": 5e-6}


def exact(case, seed):
    A, B = _inputs(case, seed)
    if case["kind"] in ("combine", "propagate"):
        n, f = case["n"], case["fout"]
        Y = torch.zeros((n, f), dtype=torch.float64, device=DEV)
        rp = A[2].long()
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
        step = max(1, (1 << 28) // f)
        for e0 in range(0, rows.numel(), step):
            e = slice(e0, e0 + step)
            Y.index_add_(0, rows[e], A[4][e].double()[:, None] * B[A[3][e].long()].double())
        return Y.clamp_(min=0) if case["kind"] == "combine" else Y
    if case["kind"] == "twohop" and case["n"] > 600000:
        return None
    if case.get("values") == "sym_norm":  # the rounded normalised values are the input
        inv = (A[2][1:] - A[2][:-1]).double()
        rows = torch.repeat_interleave(torch.arange(case["n"], device=DEV), (A[2][1:] - A[2][:-1]).long())
        A = A[:4] + ((1 / torch.sqrt(inv[rows] * inv[A[3].long()])).float(),)
    lens, cols, vals = zip(*_unions(A, B, True))
    rp = torch.zeros(case["n"] + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cat(lens).cumsum(0)
    return [rp, torch.cat(cols), torch.cat(vals)]
