"""Performance cases: what a user of the batched LP solver has it do.

A case names a family and its sizes.  Inputs are made on the GPU from the seed
with the distributions of the paper's LP families (Secs. 4.6, 6, 7):

* type 1: A ~ U(1, 10), b ~ U(10, 100), c ~ U(1, 10), all rows "<=";
* type 2: the first half of the rows "<=", the rest ">=", built around an
  interior point x0 ~ U(1, 5)^n with margins U(1, 10) (needs phase 1);
* hyperbox: l ~ U(-10, -1), u ~ U(1, 10), unit objectives;
* shared constraints: one type-1 polytope queried in directions swept around
  a circle (support-function sampling).

`run` is one call of the public entry points with everything a program keeps
(the handle, the batch) already in hand; result tensors are allocated by the
call, as `Solver.solve` does by default.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1609_08114_amd as blp

F64 = torch.float64


def listed():
    return [
        # the smallest call: a thousand tiny LPs, where launches and latency count
        {"name": "tiny_5x5_1k", "family": "uniform", "type": 1, "m": 5, "n": 5, "count": 1000},
        # tiny LPs in bulk
        {"name": "tiny_5x5_200k", "family": "uniform", "type": 1, "m": 5, "n": 5, "count": 200_000},
        # small LPs in bulk
        {"name": "small_30x30_20k", "family": "uniform", "type": 1, "m": 30, "n": 30, "count": 20_000},
        # ragged rectangular LPs that need both phases
        {"name": "twophase_47x61_4k", "family": "uniform", "type": 2, "m": 47, "n": 61, "count": 4001},
        # the headline batch: 50,000 LPs of 100 x 100
        {"name": "type1_100x100_50k", "family": "uniform", "type": 1, "m": 100, "n": 100, "count": 50_000},
        # both phases at the headline size
        {"name": "twophase_100x100_4k", "family": "uniform", "type": 2, "m": 100, "n": 100, "count": 4000},
        # both phases, beyond any register tile
        {"name": "twophase_200x200_1k", "family": "uniform", "type": 2, "m": 200, "n": 200, "count": 1000},
        # simplex and hyperbox LPs of every size in one batch (40% type 1, 40% type 2, 20% hyperbox)
        {"name": "mixed_5_300_2k", "family": "mixed", "lo": 5, "hi": 300, "count": 2000},
        # a training step over type-1 LPs of mixed sizes: optimum and its gradients
        {"name": "sizes_20_150_20k_grad", "family": "sizes", "lo": 20, "hi": 150, "count": 20_000},
        # support functions of many small boxes
        {"name": "box_5_4M", "family": "box", "n": 5, "count": 4_000_000, "grad": False},
        # larger boxes, forward and backward
        {"name": "box_28_6M_grad", "family": "box", "n": 28, "count": 6_000_000, "grad": True},
        # one polytope, many directions, forward and backward
        {"name": "shared_100x100_50k_grad", "family": "shared", "m": 100, "n": 100, "count": 50_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# what a drawn case may cost at most: pivot flops, and bytes in and out
_MAX_FLOPS = 2.0e11
_MAX_BYTES = 3.5e9


def draw(rng):
    family = rng.choice(["uniform", "uniform", "uniform", "uniform", "mixed", "sizes", "box", "shared"])
    if family == "uniform":
        ty = rng.choice([1, 1, 2])
        m = _log_int(rng, 4, 250 if ty == 1 else 210)
        n = min(250 if ty == 1 else 210, max(4, int(m * math.exp(rng.uniform(-0.7, 0.7)))))
        case = {"family": family, "type": ty, "m": m, "n": n, "count": 1}
        w = work(case)
        most = min(200_000, int(_MAX_FLOPS / w["flops"]), int(_MAX_BYTES / w["bytes"]))
        case["count"] = _log_int(rng, min(500, most), most)
        return case
    if family == "mixed":
        hi = rng.randint(60, 300)
        return {"family": family, "lo": rng.randint(4, 30), "hi": hi, "count": _log_int(rng, 300, 2000)}
    if family == "sizes":
        return {"family": family, "lo": rng.randint(4, 40), "hi": rng.randint(60, 160), "count": _log_int(rng, 500, 16_000)}
    if family == "box":
        n = _log_int(rng, 2, 64)
        return {"family": family, "n": n, "count": _log_int(rng, 2000, 60_000_000 // n), "grad": rng.random() < 0.5}
    return {"family": family, "m": rng.randint(15, 110), "n": rng.randint(15, 110), "count": _log_int(rng, 1000, 50_000)}


# --------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uni(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=F64) * (hi - lo) + lo


def _shapes(case):
    """(type 1/2/3, m, n) of every LP of a mixed or ragged batch (host arrays):
    one draw for the case, so that its results keep their length for every
    seed of the data."""
    K, lo, hi = case["count"], case["lo"], case["hi"]
    r = np.random.default_rng([lo, hi, K])
    m = r.integers(lo, hi + 1, K).astype(np.int32)
    n = r.integers(lo, hi + 1, K).astype(np.int32)
    ty = np.ones(K, np.int32)
    if case["family"] == "sizes":
        n = m.copy()
    else:
        ty = 1 + np.searchsorted([0.4, 0.8], r.random(K), side="right").astype(np.int32)
        m[ty == 3] = 0
    return ty, m, n


def _batch(m, n, kind, A, b, sense, c, l, u, uniform):
    m64, n64 = m.astype(np.int64), n.astype(np.int64)

    def off(v):
        return np.concatenate([[0], np.cumsum(v)[:-1]]).astype(np.int64)

    db = blp.DeviceBatch(m=m, n=n, kind=kind, a_off=off(m64 * n64), row_off=off(m64), col_off=off(n64), A=A, b=b,
                         sense=sense, c=c, l=l, u=u, uniform=uniform)
    db._count = len(m)
    return db


def _uniform_data(case, seed):
    """A (K, m, n), b, sense (K, m), c (K, n) of a uniform simplex batch."""
    g = _gen(seed)
    K, m, n = case["count"], case["m"], case["n"]
    A = _uni(g, 1, 10, K, m, n)
    c = _uni(g, 1, 10, K, n)
    sense = torch.zeros(K, m, dtype=torch.int8, device="cuda")
    if case["type"] == 1:
        b = _uni(g, 10, 100, K, m)
    else:
        x0, d = _uni(g, 1, 5, K, n), _uni(g, 1, 10, K, m)
        sense[:, m // 2:] = 1
        b = torch.empty(K, m, dtype=F64, device="cuda")
        for k in range(0, K, 4096):  # (bounds the product's temporary)
            s = slice(k, k + 4096)
            b[s] = (A[s] * x0[s, None, :]).sum(-1) + torch.where(sense[s] == 0, d[s], -d[s])
    return A, b, sense, c


def _ragged_data(case, seed):
    """Flat A, b, sense, c, l, u of a batch of LPs of several sizes, and its shapes."""
    g = _gen(seed)
    ty, m, n = _shapes(case)
    K, tm, tn = len(m), int(m.astype(np.int64).sum()), int(n.astype(np.int64).sum())
    A = _uni(g, 1, 10, max(1, int((m.astype(np.int64) * n).sum())))
    b = _uni(g, 10, 100, max(1, tm))
    c = _uni(g, 1, 10, tn)
    l, u = _uni(g, -10, -1, tn), _uni(g, 1, 10, tn)
    x0, d = _uni(g, 1, 5, tn), _uni(g, 1, 10, max(1, tm))
    gauss = torch.randn(tn, generator=g, device="cuda", dtype=F64)
    sense = torch.zeros(max(1, tm), dtype=torch.int8, device="cuda")
    a = r = q = 0
    for k in range(K):
        mk, nk = int(m[k]), int(n[k])
        if ty[k] == 2:
            h = mk // 2
            sense[r + h:r + mk] = 1
            ax = (A[a:a + mk * nk].view(mk, nk) * x0[q:q + nk]).sum(1)
            b[r:r + h] = ax[:h] + d[r:r + h]
            b[r + h:r + mk] = ax[h:] - d[r + h:r + mk]
        elif ty[k] == 3:
            c[q:q + nk] = gauss[q:q + nk]
        a, r, q = a + mk * nk, r + mk, q + nk
    return ty, m, n, A, b, sense, c, l, u


def _box_data(case, seed):
    g = _gen(seed)
    K, n = case["count"], case["n"]
    c = torch.randn(K, n, generator=g, device="cuda", dtype=F64)
    c /= c.square().sum(1, keepdim=True).sqrt()
    return c, _uni(g, -10, -1, K, n), _uni(g, 1, 10, K, n), _uni(g, 0, 1, K)


def _shared_data(case, seed):
    g = _gen(seed)
    K, m, n = case["count"], case["m"], case["n"]
    A, b = _uni(g, 1, 10, m, n), _uni(g, 10, 100, m)
    u, v = torch.randn(2, n, generator=g, device="cuda", dtype=F64)
    t = torch.arange(K, device="cuda", dtype=F64)[:, None] * (2 * math.pi / K)
    C = torch.cos(t) * u + torch.sin(t) * v
    return A, b, torch.zeros(m, dtype=torch.int8, device="cuda"), C, _uni(g, 0, 1, K)


def prepare(case, seed):
    f = case["family"]
    st = {"family": f, "solver": blp.Solver()}
    if f == "uniform":
        A, b, sense, c = _uniform_data(case, seed)
        K = case["count"]
        st["db"] = _batch(np.full(K, case["m"], np.int32), np.full(K, case["n"], np.int32), np.zeros(K, np.int32),
                          A.view(-1), b.view(-1), sense.view(-1), c.view(-1), None, None, True)
    elif f in ("mixed", "sizes"):
        ty, m, n, A, b, sense, c, l, u = _ragged_data(case, seed)
        box = bool((ty == 3).any())
        st["db"] = _batch(m, n, (ty == 3).astype(np.int32), A, b, sense, c, l if box else None, u if box else None, False)
        if f == "sizes":
            st["g"] = _uni(_gen(seed + 1), 0, 1, len(m))
    elif f == "box":
        c, l, u, w = _box_data(case, seed)
        K = case["count"]
        st["db"] = _batch(np.zeros(K, np.int32), np.full(K, case["n"], np.int32), np.ones(K, np.int32), None, None,
                          None, c.view(-1), l.view(-1), u.view(-1), True)
        if case["grad"]:
            st["g"] = w
    else:
        st["A"], st["b"], st["sense"], st["C"], st["g"] = _shared_data(case, seed)
    return st


# ----------------------------------------------------------------------- runs
def run(st):
    s, f = st["solver"], st["family"]
    if f == "shared":
        out = s.solve_shared(st["A"], st["b"], st["sense"], st["C"])
        m, n = st["A"].shape
        return {**out, **s.backward_shared(out, m, n, st["g"])}
    out = s.solve(st["db"])
    if "g" not in st:
        return out
    want = ("dc", "db", "dA") if f == "sizes" else ("dc", "dl", "du")
    return {**out, **s.backward(st["g"], want=want)}


# ----------------------------------------------------------------------- work
def _pivots(ty, m, n):
    """Mean pivots of the largest-coefficient rule on the two LP types (fitted
    to 5..300 rows and columns)."""
    return 2.0 + 0.125 * math.sqrt(m * n) if ty == 1 else 0.045 * m * n + min(m, n)


def _simplex_work(ty, m, n):
    # one FMA per entry of the condensed tableau and pivot (type 2: half of
    # the surplus columns of the >= rows on average)
    cols = n + 1 + (m // 4 if ty == 2 else 0)
    flops = 2.0 * _pivots(ty, m, n) * (m + 1) * cols
    return 8.0 * (m * n + 2 * m + 2 * n) + m + 16.0, flops


def work(case):
    f, K = case["family"], case["count"]
    if f == "uniform":
        by, fl = _simplex_work(case["type"], case["m"], case["n"])
        return {"bytes": K * by, "flops": K * fl}
    if f in ("mixed", "sizes"):
        by = fl = 0.0
        sample = dict(case, count=1000)
        for ty, m, n in zip(*(v.tolist() for v in _shapes(sample))):
            if ty == 3:
                by, fl = by + 32.0 * n + 16, fl + 2.0 * n
                continue
            p, q = _simplex_work(ty, m, n)
            by, fl = by + p, fl + q
            if f == "sizes":  # x, y, g read; dc, db, dA written
                by, fl = by + 8.0 * (m * n + 2 * m + 2 * n + 1), fl + m * n
        return {"bytes": by * K / 1000, "flops": fl * K / 1000}
    n = case["n"]
    if f == "box":
        # c, l, u, x and the result; backward: c, x, g in, dc, dl, du out
        return {"bytes": K * (32.0 * n + 16 + (40.0 * n + 12 if case["grad"] else 0)), "flops": 2.0 * K * n}
    m = case["m"]
    # objectives in, x and y out; backward: x, y, g in, dC out; 0.3 pivots per
    # objective along the sweep and the contraction for dA
    return {"bytes": K * (8.0 * (4 * n + 2 * m + 3) + 12) + 24.0 * m * n,
            "flops": K * (0.6 * (m + 1) * (n + 1) + 2.0 * m * n)}


# ---------------------------------------------------------------- exact values
def _simplex64(A, b, sense, c, nrow, ncol):
    """obj, x, y of a stack of padded LPs by a plain batched two-phase tableau
    simplex in 64 bits.  A (K, m, n); rows past nrow[k] and columns past
    ncol[k] are padding."""
    K, m, n = A.shape
    dev = A.device
    row = torch.arange(m, device=dev) < nrow[:, None]
    sg = torch.where(sense != 0, -1.0, 1.0).to(F64)
    A, b = A * sg[..., None], b * sg
    art = (b < 0) & row
    flip = torch.where(art, -1.0, 1.0).to(F64)
    A, b = A * flip[..., None], b * flip
    na = int(art.sum(1).max()) if K else 0
    # columns: structural, surplus of the artificial rows, rhs; rows: constraints, phase 1, objective
    T = torch.zeros(K, m + 2, n + na + 1, dtype=F64, device=dev)
    T[:, :m, :n] = A
    T[:, :m, -1] = b
    T[:, m + 1, :n] = c
    rank = torch.cumsum(art, 1) - 1
    kk, ii = torch.nonzero(art, as_tuple=True)
    T[kk, ii, n + rank[kk, ii]] = -1.0
    T[:, m] = (T[:, :m] * art[..., None]).sum(1)
    # variables: 0..n-1 structural, n + i logical of row i, n + m + i artificial of row i
    cv = torch.full((K, n + na), n + 2 * m, dtype=torch.int64, device=dev)
    cv[:, :n] = torch.arange(n, device=dev)
    cv[kk, n + rank[kk, ii]] = n + ii
    bs = torch.where(art, n + m, n) + torch.arange(m, device=dev)
    w0 = T[:, m, -1].clone()
    res = [torch.zeros(K, s, dtype=F64, device=dev) for s in (1, n + m, n + m)]  # objective, values, reduced costs
    live = torch.arange(K, device=dev)
    mode = torch.where(art.any(1), 1, 2)
    step = 0
    while live.numel():
        k = torch.arange(T.shape[0], device=dev)
        d = torch.where((mode == 1)[:, None], T[:, m, :-1], T[:, m + 1, :-1])
        d = torch.where(cv < n + m, d, -1.0)
        best, e = d.max(1)
        stop = best <= 1e-9
        # a finished phase 1: basic artificials (at zero) leave on any usable
        # column; then phase 2
        basic_art = (bs >= n + m).any(1)
        drive = stop & (mode == 1) & basic_art
        to2 = stop & (mode == 1) & ~basic_art
        done = stop & (mode == 2)
        f = T[k, :, e]
        r = torch.where((f[:, :m] > 1e-9), T[:, :m, -1].clamp_min(0) / f[:, :m].clamp_min(1e-300), math.inf)
        low, lrow = r.min(1)
        if bool(drive.any()):
            ra = (bs >= n + m).to(torch.int8).argmax(1)
            cand = torch.where(cv < n + m, T[k, ra, :-1].abs(), 0.0)
            lrow, e = torch.where(drive, ra, lrow), torch.where(drive, cand.argmax(1), e)
            f = T[k, :, e]
        go = ((~stop) & torch.isfinite(low)) | drive
        bad = (~stop) & ~torch.isfinite(low)  # unbounded: not in these families
        f = torch.where(go[:, None], f, 0.0)
        pe = torch.where(go, f[k, lrow], 1.0)
        p = torch.where(go[:, None], T[k, lrow] / pe[:, None], 0.0)
        T[k, :, e] = torch.where(go[:, None], 0.0, T[k, :, e])
        p[k, e] = torch.where(go, 1.0 / pe, 0.0)
        T.sub_(f[:, :, None] * p[:, None, :])
        T[k, lrow] = torch.where(go[:, None], p, T[k, lrow])
        leave = bs[k, lrow]
        bs[k, lrow] = torch.where(go, cv[k, e], leave)
        cv[k, e] = torch.where(go, leave, cv[k, e])
        mode = torch.where(to2, 2, mode)
        end = done | bad
        step += 1
        if step % 8 == 0 and bool(end.any()) or T.shape[0] == 1 and bool(end.all()):
            q = torch.nonzero(end)[:, 0]
            res[0][live[q], 0] = -T[q, m + 1, -1]
            val = torch.zeros(q.numel(), n + 2 * m + 1, dtype=F64, device=dev)
            red = torch.zeros_like(val)
            val.scatter_(1, bs[q], T[q, :m, -1])
            red.scatter_(1, cv[q], T[q, m + 1, :-1])
            res[1][live[q]], res[2][live[q]] = val[:, :n + m], red[:, :n + m]
            stay = torch.nonzero(~end)[:, 0]
            if stay.numel() < 0.8 * T.shape[0] or not stay.numel():
                T, cv, bs, mode, live = T[stay], cv[stay], bs[stay], mode[stay], live[stay]
        if step > 50 * (m + n):
            break
    y = -res[2][:, n:] * sg  # d obj / d b_i
    return res[0][:, 0], res[1][:, :n], y


def _solve64(A, b, sense, c, nrow, ncol):
    """_simplex64 in chunks that bound its memory."""
    K, m, n = A.shape
    per = max(1, int(6e9 / (8.0 * (m + 2) * (n + m // 2 + 1))))
    parts = [_simplex64(A[k:k + per], b[k:k + per], sense[k:k + per], c[k:k + per], nrow[k:k + per], ncol[k:k + per])
             for k in range(0, K, per)]
    return [torch.cat(v) for v in zip(*parts)]


def _none(**kw):
    return {"status": None, "iters": None, **kw}


def exact(case, seed):
    f, K = case["family"], case["count"]
    if f == "uniform":
        A, b, sense, c = _uniform_data(case, seed)
        nr = torch.full((K,), case["m"], device="cuda")
        obj, x, y = _solve64(A, b, sense, c, nr, torch.full((K,), case["n"], device="cuda"))
        return _none(obj=obj, x=x.reshape(-1), y=y.reshape(-1))
    if f == "box":
        c, l, u, w = _box_data(case, seed)
        h = torch.where(c < 0, l, u)
        out = _none(obj=(c * h).sum(1), x=h.view(-1))
        out["y"] = None
        if case["grad"]:
            out["dc"] = (w[:, None] * h).view(-1)
            out["dl"] = (w[:, None] * c.clamp_max(0)).view(-1)
            out["du"] = (w[:, None] * c.clamp_min(0)).view(-1)
        return out
    if f == "shared":
        A, b, sense, C, g = _shared_data(case, seed)
        m, n = A.shape
        obj, x, y = [], [], []
        for k in range(0, K, 25_000):
            kk = min(25_000, K - k)
            r = _solve64(A.expand(kk, m, n), b.expand(kk, m), sense.expand(kk, m), C[k:k + kk],
                         torch.full((kk,), m, device="cuda"), torch.full((kk,), n, device="cuda"))
            for v, w in zip((obj, x, y), r):
                v.append(w)
        obj, x, y = torch.cat(obj), torch.cat(x), torch.cat(y)
        wy = g[:, None] * y
        return _none(obj=obj, x=x.reshape(-1), y=y.reshape(-1), dC=(g[:, None] * x).reshape(-1), db=wy.sum(0),
                     dA=-(wy.t() @ x).reshape(-1))
    # ragged: LPs of similar size are padded to one shape
    ty, m, n, A, b, sense, c, l, u = _ragged_data(case, seed)
    m64, n64 = m.astype(np.int64), n.astype(np.int64)
    ao, ro, co = [np.concatenate([[0], np.cumsum(v)[:-1]]) for v in (m64 * n64, m64, n64)]
    obj = torch.zeros(K, dtype=F64, device="cuda")
    x, y = torch.zeros(int(n64.sum()), dtype=F64, device="cuda"), torch.zeros(max(1, int(m64.sum())), dtype=F64, device="cuda")
    groups = {}
    for k in range(K):
        groups.setdefault((0, 0, 0) if ty[k] == 3 else (int(ty[k]), -(-int(m[k]) // 60), -(-int(n[k]) // 60)), []).append(k)
    for (t, _, _), ks in groups.items():
        if t == 0:
            for k in ks:
                q = slice(int(co[k]), int(co[k]) + int(n[k]))
                x[q] = torch.where(c[q] < 0, l[q], u[q])
                obj[k] = (c[q] * x[q]).sum()
            continue
        ks = np.array(ks)
        M, N = int(m[ks].max()), int(n[ks].max())
        for s in range(0, len(ks), 4000):
            kq = ks[s:s + 4000]
            ai, ri, ci = (torch.from_numpy(v[kq]).cuda() for v in (ao, ro, co))
            mm, nn = (torch.from_numpy(v[kq]).cuda() for v in (m64, n64))
            i, j = torch.arange(M, device="cuda"), torch.arange(N, device="cuda")
            rok, cok = i < mm[:, None], j < nn[:, None]
            ok = rok[:, :, None] & cok[:, None, :]
            at = torch.where(ok, ai[:, None, None] + i[:, None] * nn[:, None, None] + j, 0)
            Ak = torch.where(ok, A[at], 0.0)
            del at
            rx, cx = torch.where(rok, ri[:, None] + i, 0), torch.where(cok, ci[:, None] + j, 0)
            o, xs, ys = _solve64(Ak, torch.where(rok, b[rx], 0.0), torch.where(rok, sense[rx], 0),
                                 torch.where(cok, c[cx], 0.0), mm, nn)
            obj[torch.from_numpy(kq).cuda()] = o
            x[cx[cok]] = xs[cok]
            y[rx[rok]] = ys[rok]
    if f == "mixed":
        return _none(obj=obj, x=x, y=y)
    g = _uni(_gen(seed + 1), 0, 1, K)
    gm, gn = (torch.repeat_interleave(g, torch.from_numpy(v).cuda()) for v in (m64, n64))
    dA = torch.empty_like(A)
    for k in range(K):
        dA[ao[k]:ao[k] + m64[k] * n64[k]] = torch.outer(-(g[k] * y[ro[k]:ro[k] + m64[k]]), x[co[k]:co[k] + n64[k]]).view(-1)
    return _none(obj=obj, x=x, y=y, dc=gn * x, db=gm * y, dA=dA)
