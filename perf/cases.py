"""Performance cases of the framework's public entry points, over the range its users meet.

Each case is one call sequence of a user's program on matrices of its size:

  step     pack + factor (in place, as the benchmark does) + selected inverse of one matrix
  logdet   pack + factor out of place: one evaluation of log det, the input kept
  selinv   the selected inverse of a factor already in hand
  batch    pack + batched factor + batched selected inverse of many uneven matrices
  grad     log det of the space-time model and its gradient (forward and backward)
  inverse  every entry of the inverse from a factor in hand
  select   chosen entries of the inverse from a factor in hand

Matrices: N(0, 1) band, arrow and corner with a strictly dominant diagonal, drawn on the device from the
seed.  All data is float64, the only type the framework takes.  `exact` is plain torch: a block
tridiagonal Cholesky and backward recurrence on blocks at least as wide as the band.
"""
import math

import numpy as np
import torch

from paper_2504_19171_amd import grad, stiles

F64 = torch.float64
DEV = "cuda"
TILES = (64, 128, 192, 256)


def listed():
    return [
        # the smallest workload of the benchmark: 32 tile columns, where launches and latency count
        {"name": "step_small", "kind": "step", "nb": 2000, "w": 32, "a": 20, "tile": 64},
        # a long narrow band (the narrowest of the batched workload): 500 short dependent tile columns
        {"name": "step_narrow", "kind": "step", "nb": 31987, "w": 32, "a": 57, "tile": 64},
        # one served job with a wide arrow, nothing a multiple of the tile
        {"name": "step_ragged", "kind": "step", "nb": 15999, "w": 553, "a": 413, "tile": 128},
        # the benchmark's main workload
        {"name": "step_large", "kind": "step", "nb": 100000, "w": 1024, "a": 100, "tile": 256},
        # an objective evaluation that needs log det alone, odd sizes, the input kept
        {"name": "logdet_odd", "kind": "logdet", "nb": 30011, "w": 501, "a": 7, "tile": 192},
        # marginal variances from a factor in hand, a band without an arrow
        {"name": "selinv_band", "kind": "selinv", "nb": 20000, "w": 700, "a": 0, "tile": 256},
        # 64 uneven matrices of the batched workload's ranges, at its tile size
        {"name": "batch64", "kind": "batch", "count": 64, "nb_lo": 5000, "nb_hi": 50000, "w_lo": 32, "w_hi": 512,
         "a_lo": 10, "a_hi": 200, "tile": 64},
        # one batch of the serving loop: 8 jobs of very different sizes
        {"name": "batch_served", "kind": "batch", "count": 8, "nb_lo": 2000, "nb_hi": 60000, "w_lo": 16, "w_hi": 1024,
         "a_lo": 0, "a_hi": 500, "tile": 128},
        # many small matrices at once
        {"name": "batch_small", "kind": "batch", "count": 24, "nb_lo": 400, "nb_hi": 3000, "w_lo": 8, "w_hi": 100,
         "a_lo": 0, "a_hi": 30, "tile": 64},
        # the gradient workload: 50 times x 2,000 sites, 50 fixed effects
        {"name": "grad_large", "kind": "grad", "nt": 50, "ns": 2000, "a": 50, "tile": 256},
        # the whole inverse of a modest matrix
        {"name": "inverse_mid", "kind": "inverse", "nb": 6000, "w": 256, "a": 37, "tile": 128},
        # a few hundred entries towards the end of a long matrix
        {"name": "select_tail", "kind": "select", "nb": 40000, "w": 256, "a": 50, "tile": 128, "pairs": 300, "tail": 6000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: single steps and batches most often, sizes over their logarithm."""
    kind = rng.choice(["step", "step", "step", "batch", "batch", "logdet", "selinv", "grad", "inverse", "select"])
    tile = rng.choice(TILES)
    if kind == "batch":
        tile = rng.choice((64, 128, 256))
        nb_lo, w_lo = _log(rng, 400, 5000), _log(rng, 8, 64)
        return {"kind": kind, "count": _log(rng, 4, 32), "nb_lo": nb_lo, "nb_hi": nb_lo * rng.randint(2, 8), "w_lo": w_lo,
                "w_hi": w_lo * rng.randint(2, 8), "a_lo": rng.randint(0, 30), "a_hi": rng.randint(31, 300), "tile": tile}
    if kind == "grad":
        return {"kind": kind, "nt": _log(rng, 8, 50), "ns": _log(rng, 60, 1200), "a": rng.randint(1, 80), "tile": tile}
    a = rng.choice((0, rng.randint(1, 40), rng.randint(41, 500)))
    if kind == "inverse":
        return {"kind": kind, "nb": _log(rng, 500, 7000), "w": _log(rng, 8, 500), "a": min(a, 200), "tile": tile}
    nb, w = _log(rng, 1500, 100000), _log(rng, 16, 1024)
    c = {"kind": kind, "nb": nb, "w": w, "a": a, "tile": tile}
    if kind == "select":
        c.update(pairs=_log(rng, 10, 2000), tail=_log(rng, 500, 8000))
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _matrix(nb, w, a, seed):
    """(ab, P, C) in canonical band form: A[j+d, j] = ab[d, j], A[nb+r, j] = P[r, j], corner C."""
    w = min(w, nb - 1)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    ab = torch.randn((w + 1, nb), generator=g, dtype=F64, device=DEV)
    col = torch.arange(nb, device=DEV)
    ab.masked_fill_(col[None, :] >= nb - torch.arange(w + 1, device=DEV)[:, None], 0.0)
    ab[0] = 0.0
    sheared = torch.zeros((w + 1, nb + w), dtype=F64, device=DEV)        # row d moved right by d
    sheared.as_strided((w + 1, nb), (nb + w + 1, 1)).copy_(ab)
    rows = ab.abs().sum(0) + sheared.abs_().sum(0)[:nb]
    del sheared
    P = C = None
    if a:
        P = torch.randn((a, nb), generator=g, dtype=F64, device=DEV)
        C = torch.tril(torch.randn((a, a), generator=g, dtype=F64, device=DEV), -1)
        C = C + C.T
        rows = rows + P.abs().sum(0)
        C.diagonal().copy_(P.abs().sum(1) + C.abs().sum(1) + 1.0)
    ab[0] = rows + 1.0
    return ab, P, C


def _batch_sizes(case):
    """The batch's sizes: the same for every seed, spread over the case's ranges."""
    r = np.random.default_rng(case["count"] * 1000003 + case["nb_hi"])
    out = []
    for _ in range(case["count"]):
        nb = int(r.integers(case["nb_lo"], case["nb_hi"] + 1))
        w = int(round(math.exp(r.uniform(math.log(case["w_lo"]), math.log(case["w_hi"])))))
        out.append((nb, w, int(r.integers(case["a_lo"], case["a_hi"] + 1))))
    return out


def _pairs(case, seed):
    """Selected (i, j): within the band in the last `tail` columns, some of them in the arrow rows."""
    r = np.random.default_rng(seed)
    nb, a, k = case["nb"], case["a"], case["pairs"]
    j = r.integers(max(0, nb - case["tail"]), nb, size=k)
    i = np.minimum(nb - 1, j + r.integers(0, min(case["w"], nb - 1) + 1, size=k))
    if a:
        arrow = r.random(k) < 0.25
        i = np.where(arrow, nb + r.integers(0, a, size=k), i)
    return np.stack([i, j], axis=1)


def _theta(seed):
    r = np.random.default_rng(seed)
    return [float(r.uniform(-1.0, 1.0)), float(r.uniform(-1.0, 1.0))]


KAPPA = 0.5


def prepare(case, seed):
    kind, tile = case["kind"], case["tile"]
    s = {"kind": kind}
    if kind == "grad":
        model = grad.SpatioTemporal(case["nt"], case["ns"], KAPPA, case["a"], seed, torch.device(DEV))
        s["f"] = grad.LogDet(model, tile=tile)
        s["theta"] = torch.tensor(_theta(seed), dtype=F64)
        return s
    if kind == "batch":
        sizes = _batch_sizes(case)
        s["lays"] = [stiles.layout(nb + a, w, a, tile) for nb, w, a in sizes]
        s["mats"] = [_matrix(nb, w, a, seed * 1000 + k) for k, (nb, w, a) in enumerate(sizes)]
        total = [lay.total_doubles for lay in s["lays"]]
        s["L"] = torch.empty(sum(total), dtype=F64, device=DEV)
        s["S"] = torch.empty(sum(total), dtype=F64, device=DEV)
        s["Ls"], s["Ss"] = list(s["L"].split(total)), list(s["S"].split(total))
        s["ws"] = torch.empty(stiles.batch_workspace_bytes(s["lays"]), dtype=torch.uint8, device=DEV)
        return s
    lay = s["lay"] = stiles.layout(case["nb"] + case["a"], case["w"], case["a"], tile)
    m = _matrix(case["nb"], case["w"], case["a"], seed)
    if kind in ("step", "logdet"):
        s["m"] = m
        s["A"] = torch.empty(lay.total_doubles, dtype=F64, device=DEV)
        s["out"] = torch.empty_like(s["A"])
        s["wf"] = torch.empty(lay.factor_workspace_bytes, dtype=torch.uint8, device=DEV)
    else:
        A = stiles.pack(*m, lay)
        s["L"] = stiles.factor(A, lay, out=A)[0]
    if kind in ("step", "selinv"):
        s["ws"] = torch.empty(lay.selinv_workspace_bytes, dtype=torch.uint8, device=DEV)
    if kind == "selinv":
        s["out"] = torch.empty_like(s["L"])
    if kind == "select":
        s["pairs"] = _pairs(case, seed)
    return s


def run(s):
    kind = s["kind"]
    if kind == "step":
        L = stiles.pack(*s["m"], s["lay"], out=s["A"])
        L, ld, info = stiles.factor(L, s["lay"], out=L, workspace=s["wf"])
        S, sinfo = stiles.selinv(L, s["lay"], out=s["out"], workspace=s["ws"])
        return {"L": L, "Sigma": S, "logdet": ld, "info": info, "sinfo": sinfo}
    if kind == "logdet":
        A = stiles.pack(*s["m"], s["lay"], out=s["A"])
        L, ld, info = stiles.factor(A, s["lay"], out=s["out"], workspace=s["wf"])
        return {"L": L, "logdet": ld, "info": info}
    if kind == "selinv":
        S, sinfo = stiles.selinv(s["L"], s["lay"], out=s["out"], workspace=s["ws"])
        return {"Sigma": S, "sinfo": sinfo}
    if kind == "batch":
        for m, lay, L in zip(s["mats"], s["lays"], s["Ls"]):
            stiles.pack(*m, lay, out=L)
        _, ld, info = stiles.factor_batched(s["Ls"], s["lays"], outs=s["Ls"], workspace=s["ws"])
        _, info = stiles.selinv_batched(s["Ls"], s["lays"], outs=s["Ss"], workspace=s["ws"], info=info)
        return {"L": s["L"], "Sigma": s["S"], "logdet": ld, "info": info}
    if kind == "grad":
        theta = s["theta"].clone().requires_grad_(True)
        ld = s["f"](theta)
        ld.backward()
        return {"logdet": ld.detach(), "grad": theta.grad}
    if kind == "inverse":
        X, info = stiles.inverse(s["L"], s["lay"])
        return {"inverse": X, "info": info}
    v, info = stiles.select(s["L"], s["lay"], s["pairs"])
    return {"values": v, "info": info}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _tile_shape(nb, w, a, b):
    n_t = -(-nb // b)
    bt = min(-(-min(w, nb - 1) // b), n_t - 1)
    return n_t, bt, -(-a // 16) * 16


def _tile_doubles(nb, w, a, b):
    n_t, bt, ap = _tile_shape(nb, w, a, b)
    return n_t * (bt + 1) * b * b + n_t * ap * b + ap * ap


def _flops(nb, w, a, selinv):
    """Element-level count of the factor (1 part) or of the selected inverse (2 parts)."""
    w = min(w, nb - 1)
    full = nb - w
    f = full * (w + a) ** 2 + sum((k + a) ** 2 for k in range(w)) + a ** 3 / 3
    return (2.0 if selinv else 1.0) * f


def work(case):
    kind, b = case["kind"], case["tile"]
    if kind == "grad":
        nb, w, a = case["nt"] * case["ns"], case["ns"] + 2, case["a"]
        return {"bytes": 8.0 * (8 * nb + a * nb), "flops": _flops(nb, w, a, False) + _flops(nb, w, a, True)}
    if kind == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        for nb, w, a in _batch_sizes(case):
            one = work({"kind": "step", "nb": nb, "w": w, "a": a, "tile": b})
            tot = {k: tot[k] + one[k] for k in tot}
        return tot
    nb, w, a = case["nb"], min(case["w"], case["nb"] - 1), case["a"]
    tiles, given = _tile_doubles(nb, w, a, b), (w + 1 + a) * nb + a * a
    if kind == "step":
        return {"bytes": 8.0 * (given + 2 * tiles), "flops": _flops(nb, w, a, False) + _flops(nb, w, a, True)}
    if kind == "logdet":
        return {"bytes": 8.0 * (given + tiles), "flops": _flops(nb, w, a, False)}
    if kind == "selinv":
        return {"bytes": 8.0 * 2 * tiles, "flops": _flops(nb, w, a, True)}
    if kind == "inverse":
        return {"bytes": 8.0 * (tiles + (nb + a) ** 2), "flops": 1.0 * (nb + a) ** 2 * (w + a)}
    tail = min(case["tail"], nb)
    return {"bytes": 8.0 * _tile_doubles(tail, w, a, b) + 24.0 * case["pairs"], "flops": _flops(tail, w, a, True)}


# ---------------------------------------------------------------------------
# The same results by plain torch
# ---------------------------------------------------------------------------

class _Plain:
    """Block tridiagonal-plus-arrow Cholesky and selected inverse, blocks of q >= B b columns (q a multiple
    of the tile b), so that every tile of the pattern lies in a diagonal or subdiagonal block."""

    def __init__(self, m, nb, w, a, b, selinv=True):
        ab, P, C = m
        w = min(w, nb - 1)
        self.nb, self.a, self.b = nb, a, b
        self.nt, self.bt, self.ap = _tile_shape(nb, w, a, b)
        q = self.q = b * max(1, self.bt, -(-min(512, nb) // b))
        self.nq = -(-nb // q)
        ap, nq, dev = self.ap, self.nq, ab.device
        eye = torch.eye(q, dtype=F64, device=dev)
        r, c = torch.arange(2 * q, device=dev)[:, None], torch.arange(q, device=dev)[None, :]
        k = (r - c).abs()
        inside = k <= w
        k = k.clamp(max=w)

        def column(J):   # rows J q .. (J + 2) q of block column J
            i, j = J * q + r, J * q + c
            ok = inside & (i < nb) & (j < nb)
            v = torch.where(ok, ab[k, torch.minimum(i, j).clamp(max=nb - 1)], torch.zeros((), dtype=F64, device=dev))
            v[:q].diagonal()[max(0, nb - J * q):] = 1.0
            return v

        self.L, self.E, self.F, self.X = [], [], [], []
        corner = torch.eye(ap, dtype=F64, device=dev)
        if a:
            corner[:a, :a] = C
        d_carry = f_carry = None
        for J in range(nq):
            col = column(J)
            D, E = col[:q], col[q:]
            F = torch.zeros((ap, q), dtype=F64, device=dev)
            if a:
                n = min(q, nb - J * q)
                F[:a, :n] = P[:, J * q:J * q + n]
            if J:
                D, F = D - d_carry, F - f_carry
            L = torch.linalg.cholesky(D)
            X = torch.linalg.solve_triangular(L, eye, upper=False)
            Xt = X.T.contiguous()
            E, F = E @ Xt, F @ Xt
            Et, Ft = E.T.contiguous(), F.T.contiguous()
            d_carry, f_carry = E @ Et, F @ Et
            corner = corner - F @ Ft
            self.L.append(L), self.E.append(E), self.F.append(F), self.X.append(X)
        self.Lc = torch.linalg.cholesky(corner) if ap else corner
        self.logdet = 2.0 * sum(float(L.diagonal().log().sum()) for L in self.L)
        if ap:
            self.logdet += 2.0 * float(self.Lc.diagonal().log().sum())
        if not selinv:
            return
        Xc = torch.linalg.solve_triangular(self.Lc, torch.eye(ap, dtype=F64, device=dev), upper=False) if ap else corner
        self.Sc = Xc.T.contiguous() @ Xc
        self.D, self.G, self.H = [None] * nq, [None] * nq, [None] * nq   # diagonal, subdiagonal, arrow blocks
        D1 = torch.zeros((q, q), dtype=F64, device=dev)
        H1 = torch.zeros((ap, q), dtype=F64, device=dev)
        for J in range(nq - 1, -1, -1):
            X, E, F = self.X[J], self.E[J], self.F[J]
            Eh, Fh = E @ X, F @ X
            H1t = H1.T.contiguous()
            G = -(D1 @ Eh + H1t @ Fh)
            H = -(H1 @ Eh + self.Sc @ Fh)
            D = X.T.contiguous() @ X - Eh.T.contiguous() @ G - Fh.T.contiguous() @ H
            self.D[J], self.G[J], self.H[J] = D, G, H
            D1, H1 = D, H
        self.X = None

    def tiles(self, diag, sub, arrow, corner):
        """The flat tile buffer (every tile column-major) of these blocks."""
        b, g, bt = self.b, self.q // self.b, self.bt
        band = torch.zeros((self.nt, bt + 1, b, b), dtype=F64, device=corner.device)
        arw = torch.zeros((self.nt, b, self.ap), dtype=F64, device=corner.device)
        for J in range(self.nt):
            o = (J % g) * b
            col = torch.cat([diag[J // g], sub[J // g]])[o:o + (bt + 1) * b, o:o + b]
            live = min(bt, self.nt - 1 - J) + 1
            band[J, :live] = col.reshape(bt + 1, b, b).transpose(1, 2)[:live]
            arw[J] = arrow[J // g][:, o:o + b].T
        return torch.cat([band.reshape(-1), arw.reshape(-1), corner.T.reshape(-1)])

    def factor_tiles(self):
        return self.tiles(self.L, self.E, self.F, self.Lc)

    def sigma_tiles(self):
        return self.tiles(self.D, self.G, self.H, self.Sc)

    def entry(self, i, j):
        i, j = max(i, j), min(i, j)
        q, nb = self.q, self.nb
        if j >= nb:
            return float(self.Sc[i - nb, j - nb])
        J, c = divmod(j, q)
        if i >= nb:
            return float(self.H[J][i - nb, c])
        return float((self.D[J] if i // q == J else self.G[J])[i % q, c])


def _space_time(nt, ns, theta, a, seed):
    """A(theta) of the space-time model, and its derivatives by both parameters, as (ab, P, C)."""
    nb, w = nt * ns, ns + 2 if nt > 1 else 2

    def path(m):
        G = torch.zeros((m, m), dtype=F64)
        i = torch.arange(m - 1)
        G[i, i] += 1.0
        G[i + 1, i + 1] += 1.0
        G[i, i + 1] = G[i + 1, i] = -1.0
        return G

    R = path(nt)
    M = KAPPA ** 2 * torch.eye(ns, dtype=F64) + path(ns)
    Q = M @ M
    K = torch.zeros((w + 1, nb), dtype=F64)
    for t in range(nt):
        for dt in (0, 1):
            if t + dt >= nt:
                continue
            for e in range(-2, 3):
                d = dt * ns + e
                if d < 0 or abs(e) >= ns:
                    continue
                q = torch.diagonal(Q, -e)
                s0 = max(0, -e)
                K[d, t * ns + s0:t * ns + s0 + q.numel()] += R[t + dt, t] * q
    K = K.to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    X = torch.randn((nb, a), generator=g, dtype=F64, device=DEV)
    e1, e2 = math.exp(theta[0]), math.exp(theta[1])
    ab = e1 * K
    ab[0] += e2 + 1.0
    Xt = X.T.contiguous()
    return (ab, Xt, Xt @ X + e2 * torch.eye(a, dtype=F64, device=DEV)), K


def exact(case, seed):
    kind, b = case["kind"], case["tile"]
    zero = torch.zeros(1, dtype=torch.int32)
    if kind == "grad":
        nt, ns, a, theta = case["nt"], case["ns"], case["a"], _theta(seed)
        m, K = _space_time(nt, ns, theta, a, seed)
        nb, w = nt * ns, K.shape[0] - 1
        f = _Plain(m, nb, w, a, b)
        q, e1, e2 = f.q, math.exp(theta[0]), math.exp(theta[1])
        r, c = torch.arange(2 * q, device=DEV)[:, None], torch.arange(q, device=DEV)[None, :]
        k = r - c
        t1, t2 = 0.0, float(f.Sc.diagonal()[:a].sum())
        for J in range(f.nq):
            col = torch.cat([f.D[J], f.G[J]])
            j = J * q + c
            ok = (k >= 0) & (k <= w) & (J * q + r < nb) & (j < nb)
            Kv = torch.where(ok, K[k.clamp(0, w), j.clamp(max=nb - 1)], torch.zeros((), dtype=F64, device=DEV))
            t1 += float((torch.where(k == 0, 1.0, 2.0) * Kv * col).sum())
            t2 += float(f.D[J].diagonal()[:max(0, min(q, nb - J * q))].sum())
        return {"logdet": torch.tensor(f.logdet, dtype=F64), "grad": torch.tensor([e1 * t1, e2 * t2], dtype=F64)}
    if kind == "batch":
        L, S, ld = [], [], []
        for k, (nb, w, a) in enumerate(_batch_sizes(case)):
            f = _Plain(_matrix(nb, w, a, seed * 1000 + k), nb, w, a, b)
            L.append(f.factor_tiles())
            S.append(f.sigma_tiles())
            ld.append(f.logdet)
        return {"L": torch.cat(L), "Sigma": torch.cat(S), "logdet": torch.tensor(ld, dtype=F64),
                "info": torch.zeros((len(ld), 2), dtype=torch.int32)}
    nb, w, a = case["nb"], case["w"], case["a"]
    m = _matrix(nb, w, a, seed)
    if kind == "inverse":
        n = nb + a
        A = torch.zeros((n, n), dtype=F64, device=DEV)
        for d in range(m[0].shape[0]):
            A.diagonal(-d)[:nb - d] = m[0][d, :nb - d]
        if a:
            A[nb:, :nb] = m[1]
            A[nb:, nb:] = m[2]
        X = torch.cholesky_inverse(torch.linalg.cholesky(A.cpu()))
        return {"inverse": X, "info": zero}
    f = _Plain(m, nb, w, a, b, selinv=kind != "logdet")
    ld = torch.tensor([f.logdet], dtype=F64)
    if kind == "step":
        return {"L": f.factor_tiles(), "Sigma": f.sigma_tiles(), "logdet": ld, "info": zero, "sinfo": zero}
    if kind == "logdet":
        return {"L": f.factor_tiles(), "logdet": ld, "info": zero}
    if kind == "selinv":
        return {"Sigma": f.sigma_tiles(), "sinfo": zero}
    return {"values": torch.tensor([f.entry(int(i), int(j)) for i, j in _pairs(case, seed)], dtype=F64), "info": zero}
