"""Performance cases: what a program that reconstructs tracks with this
library has it do, from one small event in a latency-bound loop to batches of
hundreds of thousands of seeds, through the public binding.

Every case is a dict of plain values:

  kind    fit    kf_fit / kf_fit_hybrid over fixed hit lists
          bin    hit_bin of a batch of events
          event  seed, bin, build, gather and fit of one event, call by call
          build  hit_bin and kf_build of a batch (plain or learned window)
          step   the whole step of uneven events as one replayed graph
          det    hit_bin_det, kf_build_det, gather, kf_fit_det (barrel + disks)
          mlp    one optimiser step of the window network (gradient, Adam)
  events, tracks    events and tracks per event (fit: tracks; mlp: rows)
  layers  barrel layers at r = 4, 8, ... cm
  f64     FP64 arithmetic on FP32 data, else FP32
  hybrid  the hybrid state (q/pT, phi, theta), else Cartesian
  cap     candidates per seed
  learned the network's search window
  ordered hits grouped by layer (as read out), else in any order
  refit   (fit) seeds are an earlier pass's estimates (momentum to 2 %), else
          the three-hit seeds; the FP32 fit, whose rounding decides where a
          badly seeded filter ends, takes estimates

The inputs follow the paper's toy scenario: tracks with pT in [0.5, 10] GeV
and |eta| <= 1 from a beam spot, cylinders in a 3.8 T field, Gaussian hits,
multiple scattering, 20 % noise hits; seeds from the first three hits with
the beam-spot convention of kf_seed.  They are made here with torch in FP64
from the seed alone; the events with disks come from the repository's
generator.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1711_06571_amd import kftrack as kf
from paper_1711_06571_amd import presets, workloads

DEV = "cuda:0"
D = torch.float64
KAPPA = 0.299792458e-2  # GeV / (T cm)
F = 3                   # first searched or fitted layer


def _case(name, kind, events, tracks, layers=17, f64=True, hybrid=False, cap=6, learned=False, ordered=True,
          refit=False):
    return dict(name=name, kind=kind, events=events, tracks=tracks, layers=layers, f64=f64, hybrid=hybrid, cap=cap,
                learned=learned, ordered=ordered, refit=refit)


def listed():
    return [
        # the refit of one small event's tracks: a call bound by latency
        _case("fit_small", "fit", 1, 1000, layers=10),
        # the fit of built lists at scale, FP64, with holes
        _case("fit_scale", "fit", 1, 1000000, refit=True),
        # an odd number of tracks in the hybrid state, FP32
        _case("fit_hybrid_f32", "fit", 1, 99991, f64=False, hybrid=True, refit=True),
        # binning alone: many events as read out, grouped by layer
        _case("bin_batch", "bin", 100, 5000),
        # one small event through every step, call by call (an online loop)
        _case("event_small", "event", 1, 500),
        # one ordinary event, binned and built in the default arithmetic
        _case("event_20k_f32", "build", 1, 20000, f64=False),
        # uneven events (500 to 50 000 tracks) binned, built and fitted by one graph
        _case("step_batch", "step", 16, 0),
        # a batch of full events, binned and built in FP64 (the benchmark's step)
        _case("build_batch", "build", 20, 20000),
        # the hybrid state, which recovers seeds of the wrong charge
        _case("build_hybrid", "build", 9, 9973, hybrid=True),
        # the learned search window in the default arithmetic
        _case("build_learned_f32", "build", 8, 20000, f64=False, learned=True),
        # barrel closed by disks with displaced modules: two-step propagation
        _case("det_step", "det", 4, 20000, layers=24),
        # training the window network: one optimiser step of a batch of rows
        _case("mlp_step", "mlp", 1, 4096, layers=0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "fit", "bin", "event", "build", "build", "build", "step", "det", "mlp"])
    c = _case("", kind, 1, 0)
    c.pop("name")
    if kind == "fit":
        c.update(tracks=_logint(rng, 64, 1000000), layers=rng.randint(5, 17), f64=rng.random() < 0.6,
                 hybrid=rng.random() < 0.4)
        c["refit"] = not c["f64"] or c["tracks"] > 20000
    elif kind == "bin":
        c["tracks"] = _logint(rng, 100, 50000)
        c["events"] = max(1, min(200, _logint(rng, 500, 500000) // c["tracks"]))
        c["ordered"] = rng.random() < 0.75
    elif kind == "event":
        c.update(tracks=_logint(rng, 100, 5000), f64=rng.random() < 0.6, hybrid=rng.random() < 0.4)
    elif kind == "build":
        c["tracks"] = _logint(rng, 500, 50000)
        c["cap"] = rng.choice([4, 6, 6, 6, 8])
        c["events"] = max(1, min(64, _logint(rng, 1000, 400000 * 6 // c["cap"]) // c["tracks"]))
        c.update(layers=rng.choice([10, 17, 17]), f64=rng.random() < 0.6, hybrid=rng.random() < 0.35)
        c["learned"] = not c["hybrid"] and rng.random() < 0.3
    elif kind == "step":
        c.update(events=rng.randint(2, 16), f64=rng.random() < 0.6, hybrid=rng.random() < 0.4)
    elif kind == "det":
        c.update(events=rng.randint(1, 4), tracks=_logint(rng, 500, 20000), layers=24, f64=rng.random() < 0.6)
    else:
        c.update(tracks=_logint(rng, 256, 65536), layers=0)
    return c


# ------------------------------------------------------------- FP64 helpers
#
# States X [n, 6], covariances P [n, 6, 6], charges q [n].

def _turn(X, q, R, bz):
    """Turning angle to the first crossing with the cylinder r = R along the
    motion, and the curvature h (alpha = h s); NaN where there is none."""
    px, py = X[:, 3], X[:, 4]
    pt = torch.sqrt(px * px + py * py)
    h = -q * KAPPA * bz / pt
    tx, ty = px / pt, py / pt
    u = X[:, 0] * tx + X[:, 1] * ty
    v = -X[:, 0] * ty + X[:, 1] * tx
    a, b, c = h * u, 1 + h * v, 0.5 * h * h * (R * R - X[:, 0] ** 2 - X[:, 1] ** 2)
    A2 = 2 * b - c
    disc = a * a + c * A2
    sd = torch.sqrt(disc)
    qq = -(a + torch.where(a >= 0, sd, -sd))
    sg = torch.sign(h)
    big = torch.full_like(a, math.inf)
    half = [torch.atan(sg * t) for t in (qq / A2, -c / qq)]
    half = [torch.where(t > 0, t, t + math.pi) for t in half]
    half = torch.minimum(*[torch.where(torch.isnan(t), big, t) for t in half])
    alpha = torch.where(torch.isinf(half) | ~(disc >= 0), torch.full_like(a, math.nan), 2 * half * sg)
    return alpha, h, pt


def _move(X, alpha, h, pt):
    tx, ty = X[:, 3] / pt, X[:, 4] / pt
    sa, omc = torch.sin(alpha), 2 * torch.sin(alpha / 2) ** 2
    A, B = sa / h, omc / h
    ca = 1 - omc
    s = alpha / h
    Xo = torch.stack([X[:, 0] + tx * A - ty * B, X[:, 1] + ty * A + tx * B, X[:, 2] + X[:, 5] * s / pt,
                      X[:, 3] * ca - X[:, 4] * sa, X[:, 4] * ca + X[:, 3] * sa, X[:, 5]], 1)
    return Xo, s, A, B, sa, ca


def _highland(X, x0, mass):
    """(scattering angle)^2 at a cylinder crossing, and p^2."""
    p2 = (X[:, 3:] ** 2).sum(1)
    p = torch.sqrt(p2)
    r = torch.sqrt(X[:, 0] ** 2 + X[:, 1] ** 2)
    xe = x0 * r * p / (X[:, 0] * X[:, 3] + X[:, 1] * X[:, 4]).abs()
    ib2 = (p2 + mass * mass) / p2
    th = 0.0136 * torch.sqrt(ib2) / p * torch.sqrt(xe) * (1 + 0.038 * torch.log(xe * ib2))
    return th * th, p2


def _scatter(P, X, x0, mass):
    t2, p2 = _highland(X, x0, mass)
    m = X[:, 3:]
    P[:, 3:, 3:] += t2[:, None, None] * (p2[:, None, None] * torch.eye(3, dtype=D, device=X.device) -
                                         m[:, :, None] * m[:, None, :])


def _predict(X, P, q, R, g):
    """To r = R with the surface-constrained Jacobian and the scattering."""
    alpha, h, pt = _turn(X, q, R, g.bz)
    Xo, s, A, B, sa, ca = _move(X, alpha, h, pt)
    px, py, pz = X[:, 3], X[:, 4], X[:, 5]
    n = X.shape[0]
    sp3, aox = s / pt ** 3, alpha / pt ** 2
    J = torch.eye(6, dtype=D, device=X.device).repeat(n, 1, 1)
    J[:, 0, 3], J[:, 0, 4] = A / pt - Xo[:, 3] * px * sp3, -B / pt - Xo[:, 3] * py * sp3
    J[:, 1, 3], J[:, 1, 4] = B / pt - Xo[:, 4] * px * sp3, A / pt - Xo[:, 4] * py * sp3
    J[:, 2, 3], J[:, 2, 4], J[:, 2, 5] = -pz * px * sp3, -pz * py * sp3, s / pt
    J[:, 3, 3], J[:, 3, 4] = ca + Xo[:, 4] * aox * px, -sa + Xo[:, 4] * aox * py
    J[:, 4, 3], J[:, 4, 4] = sa - Xo[:, 3] * aox * px, ca - Xo[:, 3] * aox * py
    w = torch.stack([Xo[:, 3] / pt, Xo[:, 4] / pt, pz / pt, -h * Xo[:, 4], h * Xo[:, 3], torch.zeros_like(pz)], 1)
    r = torch.sqrt(Xo[:, 0] ** 2 + Xo[:, 1] ** 2)
    nx, ny = Xo[:, 0] / r, Xo[:, 1] / r
    gs = -(nx[:, None] * J[:, 0] + ny[:, None] * J[:, 1]) / (nx * w[:, 0] + ny * w[:, 1])[:, None]
    J = J + w[:, :, None] * gs[:, None, :]
    P = J @ P @ J.transpose(1, 2).contiguous()
    _scatter(P, Xo, g.x_over_x0, g.mass)
    return Xo, P


def _update(X, P, m, V):
    """Tangent-plane update with hits m [n, 3], V [n, 6]; returns chi2, det."""
    r = torch.sqrt(X[:, 0] ** 2 + X[:, 1] ** 2)
    tx, ty = -X[:, 1] / r, X[:, 0] / r
    r0 = tx * (m[:, 0] - X[:, 0]) + ty * (m[:, 1] - X[:, 1])
    r1 = m[:, 2] - X[:, 2]
    U = tx[:, None] * P[:, :, 0] + ty[:, None] * P[:, :, 1]
    W = P[:, :, 2].clone()
    s00 = tx * U[:, 0] + ty * U[:, 1] + tx * tx * V[:, 0] + 2 * tx * ty * V[:, 1] + ty * ty * V[:, 3]
    s01 = U[:, 2] + tx * V[:, 2] + ty * V[:, 4]
    s11 = W[:, 2] + V[:, 5]
    det = s00 * s11 - s01 * s01
    i00, i01, i11 = s11 / det, -s01 / det, s00 / det
    K0 = U * i00[:, None] + W * i01[:, None]
    K1 = U * i01[:, None] + W * i11[:, None]
    chi2 = r0 * (i00 * r0 + i01 * r1) + r1 * (i01 * r0 + i11 * r1)
    Xn = X + K0 * r0[:, None] + K1 * r1[:, None]
    Pn = P - K0[:, :, None] * U[:, None, :] - K1[:, :, None] * W[:, None, :]
    return Xn, Pn, chi2, (s00 > 0) & (det > 0)


def _to_hybrid(X, P, q):
    px, py, pz = X[:, 3], X[:, 4], X[:, 5]
    pt2 = px * px + py * py
    pt, p2 = torch.sqrt(pt2), pt2 + pz * pz
    Y = torch.stack([X[:, 0], X[:, 1], X[:, 2], q / pt, torch.atan2(py, px), torch.atan2(pt, pz)], 1)
    B = torch.eye(6, dtype=D, device=X.device).repeat(X.shape[0], 1, 1)
    B[:, 3, 3], B[:, 3, 4] = -q * px / pt ** 3, -q * py / pt ** 3
    B[:, 3, 5] = 0
    B[:, 4, 3], B[:, 4, 4], B[:, 4, 5] = -py / pt2, px / pt2, 0
    B[:, 5, 3], B[:, 5, 4], B[:, 5, 5] = px * pz / (pt * p2), py * pz / (pt * p2), -pt / p2
    return Y, B @ P @ B.transpose(1, 2).contiguous()


def _to_cartesian(Y, P):
    k = Y[:, 3]
    pt, sg = 1 / k.abs(), torch.where(k < 0, -1.0, 1.0).to(D)
    sf, cf, st, ct = torch.sin(Y[:, 4]), torch.cos(Y[:, 4]), torch.sin(Y[:, 5]), torch.cos(Y[:, 5])
    cot = ct / st
    X = torch.stack([Y[:, 0], Y[:, 1], Y[:, 2], pt * cf, pt * sf, pt * cot], 1)
    d = -sg * pt * pt
    A = torch.eye(6, dtype=D, device=Y.device).repeat(Y.shape[0], 1, 1)
    A[:, 3, 3], A[:, 3, 4], A[:, 3, 5] = d * cf, -pt * sf, 0
    A[:, 4, 3], A[:, 4, 4], A[:, 4, 5] = d * sf, pt * cf, 0
    A[:, 5, 3], A[:, 5, 4], A[:, 5, 5] = d * cot, 0, -pt / (st * st)
    return X, A @ P @ A.transpose(1, 2).contiguous(), sg


_UT = [(i, j) for i in range(6) for j in range(i, 6)]


def _pack(P):
    return torch.stack([P[:, i, j] for i, j in _UT], 0)


def _unpack(C):
    P = torch.empty((C.shape[1], 6, 6), dtype=D, device=C.device)
    for k, (i, j) in enumerate(_UT):
        P[:, i, j] = C[k]
        P[:, j, i] = C[k]
    return P


def _seed64(H, g, layers=3):
    """The beam-spot seed of hits H [3, 9, n] in FP64: X, P, q, ok."""
    h = H[:3].to(D)
    n = h.shape[2]
    Bx, By, Cx, Cy = h[0, 0], h[0, 1], h[2, 0], h[2, 1]
    d = 2 * (Bx * Cy - By * Cx)
    l1, l2 = Bx * Bx + By * By, Cx * Cx + Cy * Cy
    ox, oy = (Cy * l1 - By * l2) / d, (Bx * l2 - Cx * l1) / d
    r1x, r1y, r3x, r3y = Bx - ox, By - oy, Cx - ox, Cy - oy
    rho = torch.sqrt(r1x * r1x + r1y * r1y)
    turn = Bx * (Cy - By) - By * (Cx - Bx)
    q = torch.where((turn < 0) == (g.bz > 0), 1.0, -1.0).to(D)
    pt = KAPPA * abs(g.bz) * rho
    sg = torch.where(turn > 0, 1.0, -1.0).to(D)
    dal = torch.atan2(r1x * r3y - r1y * r3x, r1x * r3x + r1y * r3y).abs()
    X = torch.stack([Bx, By, h[0, 2], pt * -sg * r1y / rho, pt * sg * r1x / rho,
                     pt * (h[2, 2] - h[0, 2]) / (rho * dal)], 1)
    p2 = (X[:, 3:] ** 2).sum(1)
    r0 = torch.sqrt(l1)
    tx, ty = -By / r0, Bx / r0
    P = torch.zeros((n, 6, 6), dtype=D, device=h.device)
    P[:, 0, 0], P[:, 0, 1], P[:, 1, 0], P[:, 1, 1], P[:, 2, 2] = tx * tx, tx * ty, tx * ty, ty * ty, 100.0
    for k in (3, 4, 5):
        P[:, k, k] = p2
    # impact parameter 0 +- the beam spot
    k = q * KAPPA * g.bz
    cx, cy = X[:, 0] + X[:, 4] / k, X[:, 1] - X[:, 3] / k
    cn, pt = torch.sqrt(cx * cx + cy * cy), torch.sqrt(X[:, 3] ** 2 + X[:, 4] ** 2)
    f = cn - pt / k.abs()
    z = torch.zeros_like(cn)
    Hm = torch.stack([cx / cn, cy / cn, z, -cy / (k * cn) - X[:, 3] / (pt * k.abs()),
                      cx / (k * cn) - X[:, 4] / (pt * k.abs()), z], 1)
    PH = (P * Hm[:, None, :]).sum(2)
    S = g.beam_sigma ** 2 + (Hm * PH).sum(1)
    ok = S > 0
    X = X - PH * (f / S)[:, None]
    P = P - PH[:, :, None] * PH[:, None, :] / S[:, None, None]
    _scatter(P, X, g.x_over_x0, g.mass)
    for l in range(3):
        if l:
            X, P = _predict(X, P, q, g.r[l], g)
            ok &= ~(X[:, 2].abs() > g.z_half)
        X, P, _, pd = _update(X, P, h[l, :3].T, h[l, 3:].T)
        ok &= pd
    ok &= torch.isfinite(X).all(1) & torch.isfinite(P).all(2).all(1)
    X = torch.where(ok[:, None], X, 0.0)
    P = torch.where(ok[:, None, None], P, 0.0)
    return X, P, torch.where(ok, q, 1.0), ok


def _seeds(H, g, ld):
    """What kf_seed gives a program: FP32 par [6, ld], cov [21, ld], q."""
    n = H.shape[2]
    par = torch.zeros((6, ld), dtype=torch.float32, device=DEV)
    cov = torch.zeros((21, ld), dtype=torch.float32, device=DEV)
    q = torch.ones(ld, dtype=torch.int8, device=DEV)
    for a in range(0, n, 1 << 18):
        b = min(n, a + (1 << 18))
        X, P, qq, _ = _seed64(H[:, :, a:b], g)
        par[:, a:b], cov[:, a:b], q[a:b] = X.T.float(), _pack(P).float(), qq.to(torch.int8)
    return dict(par=par, cov=cov, q=q)


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + 17)


def _geometry(case):
    return presets.barrel(case["layers"])


def _cov_rows(phi, gs):
    a, b = gs.sig_rphi ** 2, gs.sig_z ** 2
    s, c, z = torch.sin(phi), torch.cos(phi), torch.zeros_like(phi)
    return torch.stack([a * s * s, -a * s * c, z, a * c * c, z, b + z], 0)


def _tracks(n, g, G, truth=False):
    """Track hits [L, 9, n] FP32 of n tracks through every layer; with truth
    also the states on layer 2 (before its scattering) and the charges."""
    gs = presets.GenSettings()
    out, have, at2, qs = [], 0, [], []
    while have < n:
        m = int((n - have) * 1.05) + 64
        U = lambda: torch.rand(m, dtype=D, device=DEV, generator=G)
        N = lambda: torch.randn(m, dtype=D, device=DEV, generator=G)
        q = torch.where(U() < 0.5, -1.0, 1.0).to(D)
        pt, phi, eta = gs.pt_min + U() * (gs.pt_max - gs.pt_min), 2 * math.pi * U(), gs.eta_max * (2 * U() - 1)
        X = torch.stack([N() * gs.vtx_sxy, N() * gs.vtx_sxy, N() * gs.vtx_sz, pt * torch.cos(phi), pt * torch.sin(phi),
                         pt * torch.sinh(eta)], 1)
        H = torch.empty((g.n_layers, 9, m), dtype=torch.float32, device=DEV)
        ok = torch.ones(m, dtype=torch.bool, device=DEV)
        for l in range(g.n_layers):
            X = _move(X, *_turn(X, q, g.r[l], g.bz))[0]
            ok &= X[:, 2].abs() < g.z_half
            ph = torch.atan2(X[:, 1], X[:, 0]) + N() * gs.sig_rphi / g.r[l]
            H[l, 0], H[l, 1] = (g.r[l] * torch.cos(ph)).float(), (g.r[l] * torch.sin(ph)).float()
            H[l, 2] = (X[:, 2] + N() * gs.sig_z).float()
            H[l, 3:] = _cov_rows(ph, gs).float()
            if l == F - 1:
                X2 = X
            t2, p2 = _highland(X, g.x_over_x0, g.mass)
            p, mom = torch.sqrt(p2), X[:, 3:]
            v = torch.stack([N(), N(), N()], 1) * torch.sqrt(t2 * p2)[:, None]
            v -= mom * ((v * mom).sum(1) / p2)[:, None]
            mom = mom + v
            X = torch.cat([X[:, :3], mom * (p / mom.norm(dim=1))[:, None]], 1)
            ok &= torch.isfinite(X).all(1)
        H = H[:, :, ok][:, :, :n - have]
        out.append(H)
        at2.append(X2[ok][:n - have])
        qs.append(q[ok][:n - have])
        have += H.shape[2]
    H = torch.cat(out, 2) if len(out) > 1 else out[0]
    return (H, torch.cat(at2), torch.cat(qs)) if truth else H


def _estimates(X, q, g, ld, G):
    """Seeds as an earlier pass leaves them: the true state on layer 2 moved
    by its stated covariance (hit resolution, 2 % of the momentum)."""
    gs, n = presets.GenSettings(), X.shape[0]
    ph, p = torch.atan2(X[:, 1], X[:, 0]), X[:, 3:].norm(dim=1)
    N = lambda: torch.randn(n, dtype=D, device=DEV, generator=G)
    ph2 = ph + N() * gs.sig_rphi / g.r[F - 1]
    Y = torch.stack([g.r[F - 1] * torch.cos(ph2), g.r[F - 1] * torch.sin(ph2), X[:, 2] + N() * gs.sig_z] +
                    [X[:, 3 + k] + N() * 0.02 * p / math.sqrt(3) for k in range(3)], 1)
    C = torch.zeros((21, n), dtype=D, device=DEV)
    V = _cov_rows(ph2, gs)
    for k, v in zip((0, 1, 2, 6, 7, 11), V):
        C[k] = v
    for k in (15, 18, 20):
        C[k] = (0.02 * p) ** 2 / 3
    par = torch.zeros((6, ld), dtype=torch.float32, device=DEV)
    cov = torch.zeros((21, ld), dtype=torch.float32, device=DEV)
    qo = torch.ones(ld, dtype=torch.int8, device=DEV)
    par[:, :n], cov[:, :n], qo[:n] = Y.T.float(), C.float(), q.to(torch.int8)
    return dict(par=par, cov=cov, q=qo)


def _pad(n):
    return max(64, (n + 63) // 64 * 64)


def _event_sizes(case):
    if case["kind"] == "step":  # uneven: log-uniform in [500, 50 000]
        r = np.random.default_rng(7919 + case["events"])
        return np.exp(r.uniform(math.log(500), math.log(50000), case["events"])).astype(np.int64)
    return np.full(case["events"], case["tracks"], dtype=np.int64)


def _events(case, seed):
    """Hits of all events (tracks + 20 % noise per layer) as hit_bin takes
    them, grouped by layer and in random order inside a layer, and the seeds."""
    g, G = _geometry(case), _gen(seed)
    L, gs = g.n_layers, presets.GenSettings()
    nt = _event_sizes(case)
    E, n = len(nt), int(nt.sum())
    ld = _pad(n)
    H = _tracks(n, g, G)
    sev = torch.repeat_interleave(torch.arange(E, device=DEV, dtype=torch.int32), torch.from_numpy(nt).to(DEV))
    nn = np.rint(0.2 * nt).astype(np.int64)
    nev = torch.repeat_interleave(torch.arange(E, device=DEV, dtype=torch.int32), torch.from_numpy(nn).to(DEV))
    m = nev.shape[0]
    rows, ev, lay = [], [], []
    for l in range(L):
        ph = 2 * math.pi * torch.rand(m, dtype=D, device=DEV, generator=G)
        z = g.z_half * (2 * torch.rand(m, dtype=D, device=DEV, generator=G) - 1)
        noise = torch.cat([torch.stack([g.r[l] * torch.cos(ph), g.r[l] * torch.sin(ph), z], 0), _cov_rows(ph, gs)], 0)
        rows += [H[l], noise.float()]
        ev += [sev, nev]
        lay += [torch.full((n + m,), l, dtype=torch.int32, device=DEV)]
    rows, ev, lay = torch.cat(rows, 1), torch.cat(ev), torch.cat(lay)
    key = ev.long() * 64 + (lay.long() if case["ordered"] else 0)
    key = (key << 32) + torch.randint(0, 1 << 32, key.shape, device=DEV, generator=G)
    o = torch.argsort(key)
    cnt = torch.from_numpy((nt + nn) * L)
    hoff = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(cnt, 0)]).to(torch.int32).to(DEV)
    H3 = torch.zeros((3, 9, ld), dtype=torch.float32, device=DEV)
    H3[:, :, :n] = H[:3]
    return dict(g=g, n=n, E=E, nt=nt, ld=ld, layer=lay[o].contiguous(), xyz=rows[:3, o].contiguous(),
                cov=rows[3:, o].contiguous(), hoff=hoff, sev=sev, H3=H3)


def _network():
    """A window network of trained size and spread: widths near 0.12 cm along
    the arc and 0.6 cm in z, consulted where the plain window is wider than
    the gates of the trained ones."""
    r = np.random.default_rng(5)
    p = dict(W1=r.normal(0, math.sqrt(2 / 27), (64, 27)), b1=np.zeros(64), W2=r.normal(0, math.sqrt(2 / 64), (64, 64)),
             b2=np.zeros(64), W3=r.normal(0, math.sqrt(1 / 64), (2, 64)), b3=np.array([20.0, 10.0]))
    sd = np.array([25.0, 25, 20, 3, 3, 3] + [0.1] * 6 + [0.1] * 5 + [0.3] * 4 + [1.0] * 6)
    return kf.mlp_block(kf.mlp_join(p), np.zeros(27), sd, [0.01, 0.1], kappa=0.6, gate_rphi=0.135, gate_z=0.627)


def _arith(case):
    return kf.ARITH_F64 if case["f64"] else kf.ARITH_F32


def _fit_rows(case, seed):
    g, n = _geometry(case), case["tracks"]
    ld = _pad(n)
    G = _gen(seed)
    H = torch.zeros((g.n_layers, 9, ld), dtype=torch.float32, device=DEV)
    H[:, :, :n], X2, q = _tracks(n, g, G, truth=True)
    s = _estimates(X2, q, g, ld, G) if case["refit"] else _seeds(H[:3, :, :n], g, ld)
    # lists as the build leaves them: a hole on about 4 % of the layers
    hole = torch.zeros(ld, dtype=torch.int32, device=DEV)
    for l in range(F, g.n_layers):
        b = torch.rand(ld, device=DEV, generator=G) < 0.04
        hole |= b.to(torch.int32) << l
    return g, n, H, s, hole


def _mlp_rows(case, seed):
    n, G = case["tracks"], _gen(seed)
    rows = torch.zeros((n, kf.MLP_ROW), dtype=torch.float32, device=DEV)
    rows[:, :27] = torch.randn((n, 27), device=DEV, generator=G) * 1.5 + 0.3
    rows[:, 27:29] = torch.randn((n, 2), device=DEV, generator=G).abs() * torch.tensor([0.02, 0.2], device=DEV)
    r = np.random.default_rng(seed)
    p = dict(W1=r.normal(0, math.sqrt(2 / 27), (64, 27)), b1=r.normal(0, 0.05, 64),
             W2=r.normal(0, math.sqrt(2 / 64), (64, 64)), b2=r.normal(0, 0.05, 64),
             W3=r.normal(0, math.sqrt(1 / 64), (2, 64)), b3=np.array([1.0, 1.0]))
    w = kf.mlp_join(p).astype(np.float32)
    w = torch.from_numpy(w).to(torch.bfloat16).float().numpy()  # masters on working values, as training starts
    # moments of a run under way
    m = r.normal(0, 0.01, w.shape).astype(np.float32)
    v = (m * m + r.uniform(1e-4, 1e-3, w.shape)).astype(np.float32)
    return rows, w, m, v


_MU, _SD, _SCALE = np.full(27, 0.3), np.full(27, 1.5), np.array([0.01, 0.1])


def prepare(case, seed):
    kind = case["kind"]
    c = presets.BuildCuts(cand_cap=case["cap"])
    if kind == "fit":
        g, n, H, s, hole = _fit_rows(case, seed)
        return dict(case=case, g=g, n=n, H=H, s=s, hole=hole)
    if kind == "mlp":
        rows, w, m, v = _mlp_rows(case, seed)
        T = lambda a: torch.from_numpy(a.copy()).to(DEV)
        ws = torch.empty(int(kf.lib().kf_mlp_grad_workspace_bytes(case["tracks"])) // 4, dtype=torch.float32, device=DEV)
        return dict(case=case, rows=rows, block=kf.mlp_block(w, _MU, _SD, _SCALE), w=T(w), m=T(m), v=T(v), ws=ws,
                    step=100)
    if kind == "det":
        wl = presets.lids()
        wl.gen.seed = presets.SEED_BASE + 100 + int(seed)
        eb = workloads.det_event_batch(wl, range(case["events"]), n_tracks=case["tracks"])
        T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        n, ld = eb.n_seeds, eb.ld
        H3 = T(eb.track_rows[:3])
        st = dict(case=case, d=wl.detector, cuts=c, n=n, E=case["events"], layer=T(eb.layer), xyz=T(eb.xyz),
                  cov=T(eb.cov), hoff=T(eb.hit_offsets), sev=T(eb.seed_event),
                  s=_seeds(H3[:, :, :n], wl.detector.seed_geometry(), ld), out=None, fit=None, rows=None, hole=None)
        st["binned"] = kf.BinnedHits(st["E"], st["d"].n_layers, c.n_phi_bins, c.n_z_bins, st["layer"].shape[0], DEV)
        st["bp"] = kf.build_params(c, arith=_arith(case))
        return dict(st, **_workspaces(st, st["d"].n_layers))
    e = _events(case, seed)
    L, nh = e["g"].n_layers, e["layer"].shape[0]
    state = kf.STATE_HYBRID if case["hybrid"] else kf.STATE_CARTESIAN
    if kind == "event":
        return dict(e, case=case, cuts=c, bp=kf.build_params(c, arith=_arith(case), state=state))
    if kind == "bin":
        binned = kf.BinnedHits(e["E"], L, c.n_phi_bins, c.n_z_bins, nh, DEV)
        ws = torch.empty(kf.hit_bin_workspace_bytes(e["E"], L, c.n_phi_bins, c.n_z_bins, nh), dtype=torch.uint8,
                         device=DEV)
        return dict(e, case=case, cuts=c, binned=binned, bin_ws=ws)
    e["s"] = _seeds(e["H3"][:, :, :e["n"]], e["g"], e["ld"])
    net = _network() if case["learned"] else None
    bp = kf.build_params(c, arith=_arith(case), state=state, window_mode=1 if case["learned"] else 0, mlp_block=net,
                         tuned=kind == "step")
    e.update(case=case, cuts=c, bp=bp, net=net, out=None)
    if kind == "step":
        # seeds of the largest events first, completion not asked for
        nt = e["nt"]
        off = np.concatenate([[0], np.cumsum(nt)])
        order = np.concatenate([np.arange(off[k], off[k + 1]) for k in np.argsort(-nt, kind="stable")])
        e["order"] = torch.from_numpy(order.astype(np.int32)).to(DEV)
        ex = kf.BuildExtra()
        ex.seed_event, ex.seed_order = e["sev"].data_ptr(), e["order"].data_ptr()
        e["plan"] = kf.BatchPlan(e["g"], bp, e["layer"], e["xyz"], e["cov"], e["hoff"], c.n_phi_bins, c.n_z_bins,
                                 e["n"], e["s"]["par"], e["s"]["cov"], e["s"]["q"], extra=ex,
                                 stream=torch.cuda.current_stream() if torch.cuda.current_stream().cuda_stream else None,
                                 fit_arith=_arith(case), keep=(e["sev"], e["order"]))
        return e
    e["binned"] = kf.BinnedHits(e["E"], L, c.n_phi_bins, c.n_z_bins, nh, DEV)
    return dict(e, **_workspaces(e, L))


def _workspaces(e, L):
    c, nh = e["cuts"], e["layer"].shape[0]
    return dict(bin_ws=torch.empty(kf.hit_bin_workspace_bytes(e["E"], L, c.n_phi_bins, c.n_z_bins, nh),
                                   dtype=torch.uint8, device=DEV),
                build_ws=torch.empty(kf.kf_build_workspace_bytes(e["bp"], e["binned"], e["n"]), dtype=torch.uint8,
                                     device=DEV))


# --------------------------------------------------------------------- run

def _built(out, n, more=()):
    return {k: out[k][..., :n] for k in ("hits", "par", "cov", "chi2", "nhits", "status") + tuple(more)}


def _fitted(out, n):
    return {k: out[k][..., :n] for k in ("par", "cov", "chi2", "ndof", "status")}


def run(s):
    case = s["case"]
    kind, arith = case["kind"], _arith(case)
    fit = kf.kf_fit_hybrid if case["hybrid"] else kf.kf_fit
    if kind == "fit":
        s["out"] = fit(s["g"], s["n"], F, s["H"], s["s"]["par"], s["s"]["cov"], s["s"]["q"], hole_mask=s["hole"],
                       out=s.get("out"), arith=arith)
        return _fitted(s["out"], s["n"])
    if kind == "mlp":
        g = kf.kf_mlp_grad(s["block"], s["rows"], ws=s["ws"])
        kf.kf_mlp_adam(s["block"], s["w"], s["m"], s["v"], g, s["step"])
        s["step"] += 1
        return dict(grad=g, w=s["w"], m=s["m"], v=s["v"])
    c = s["cuts"] if kind != "step" else None
    if kind == "bin":
        b = kf.hit_bin(s["g"], c.n_phi_bins, c.n_z_bins, s["layer"], s["xyz"], s["cov"], event_offsets=s["hoff"],
                       out=s["binned"], ws=s["bin_ws"])
        return dict(offsets=b.offsets, xyzphi=b.xyzphi, cov=b.cov, orig=b.orig, bad=b.bad)
    if kind == "event":
        n, g = s["n"], s["g"]
        sd = kf.kf_seed(g, n, s["H3"])
        b = kf.hit_bin(g, c.n_phi_bins, c.n_z_bins, s["layer"], s["xyz"], s["cov"])
        o = kf.kf_build(g, s["bp"], b, n, sd["par"], sd["cov"], sd["q"])
        rows, hole = kf.kf_gather_hits(g.n_layers, F, n, o["hits"], s["xyz"], s["cov"])
        f = fit(g, n, F, rows, sd["par"], sd["cov"], sd["q"], hole_mask=hole, arith=arith)
        return dict(seed=dict(par=sd["par"], cov=sd["cov"], q=sd["q"]), build=_built(o, n), fit=_fitted(f, n))
    if kind == "det":
        n, d = s["n"], s["d"]
        kf.hit_bin_det(d, c.n_phi_bins, c.n_z_bins, s["layer"], s["xyz"], s["cov"], event_offsets=s["hoff"],
                       out=s["binned"], ws=s["bin_ws"])
        ex = kf.BuildExtra()
        ex.seed_event = s["sev"].data_ptr()
        o = s["out"] = kf.kf_build_det(d, s["bp"], s["binned"], n, s["s"]["par"], s["s"]["cov"], s["s"]["q"], extra=ex,
                                       out=s["out"], ws=s["build_ws"])
        s["rows"], s["hole"] = kf.kf_gather_hits(d.n_layers, F, n, o["hits"], s["xyz"], s["cov"], seed_event=s["sev"],
                                                 event_offsets=s["hoff"], fit_hits=s["rows"], hole_mask=s["hole"])
        s["fit"] = kf.kf_fit_det(d, n, F, s["rows"], o["visit"], s["s"]["par"], s["s"]["cov"], s["s"]["q"],
                                 hole_mask=s["hole"], out=s["fit"], arith=arith)
        return dict(build=_built(o, n, ("visit",)), fit=_fitted(s["fit"], n))
    if kind == "step":
        p = s["plan"]
        here = torch.cuda.current_stream()
        p.stream.wait_stream(here)
        p.launch()
        here.wait_stream(p.stream)
        return dict(build=_built(p.out, s["n"]), fit=_fitted(p.fit, s["n"]))
    kf.hit_bin(s["g"], c.n_phi_bins, c.n_z_bins, s["layer"], s["xyz"], s["cov"], event_offsets=s["hoff"],
               out=s["binned"], ws=s["bin_ws"])
    ex = kf.BuildExtra()
    ex.seed_event = s["sev"].data_ptr()
    s["out"] = kf.kf_build(s["g"], s["bp"], s["binned"], s["n"], s["s"]["par"], s["s"]["cov"], s["s"]["q"], extra=ex,
                           out=s["out"], ws=s["build_ws"])
    return _built(s["out"], s["n"])


# ------------------------------------------------------------ work, exact

def work(case):
    """Bytes: every input read and every output written once.  Operations:
    per track and layer one prediction (610) and update (202); a build has at
    least one candidate per seed and layer, the seed's cap once it branches
    (counted here as one)."""
    kind, L = case["kind"], case["layers"]
    n = float(_event_sizes(case).sum())
    S = L - F
    fit_b, fit_f = n * (36.0 * S + 113 + 120), n * S * 822.0
    hits = 1.2 * n * (L if kind != "det" else 10)
    S = S if kind != "det" else 7
    bin_b = hits * (40 + 44) + case["events"] * L * 1009 * 4.0
    build_b, build_f = n * (109 + 4.0 * (L - F) + 120) + hits * 44, n * S * 822.0
    if kind == "fit":
        return dict(bytes=fit_b, flops=fit_f)
    if kind == "bin":
        return dict(bytes=bin_b, flops=hits * 20.0)
    if kind == "mlp":
        return dict(bytes=n * 116 + kf.MLP_NPARAM * 28.0, flops=n * 6.0 * (64 * 27 + 64 * 64 + 128))
    if kind == "build":
        return dict(bytes=hits * 40 + build_b, flops=build_f)
    return dict(bytes=hits * 40 + build_b + fit_b, flops=build_f + fit_f)


def _exact_fit(case, seed):
    g, n, H, s, hole = _fit_rows(case, seed)
    par = torch.empty((6, n), dtype=D, device=DEV)
    cov = torch.empty((21, n), dtype=D, device=DEV)
    chi2 = torch.empty(n, dtype=D, device=DEV)
    for a in range(0, n, 1 << 17):
        b = min(n, a + (1 << 17))
        X, P = s["par"][:, a:b].T.to(D).contiguous(), _unpack(s["cov"][:, a:b].to(D))
        q = s["q"][a:b].to(D)
        c2 = torch.zeros(b - a, dtype=D, device=DEV)
        if case["hybrid"]:
            X, P = _to_hybrid(X, P, q)
        live = torch.isfinite(X).all(1) & torch.isfinite(P).all(2).all(1)
        for l in range(F, g.n_layers):
            h = H[l, :, a:b].to(D)
            use = (hole[a:b] >> l & 1) == 0
            if case["hybrid"]:
                Xc, Pc, qc = _to_cartesian(X, P)
                Xc, Pc = _predict(Xc, Pc, qc, g.r[l], g)
                out = Xc[:, 2].abs() > g.z_half
                Xp, Pp = _to_hybrid(Xc, Pc, qc)
            else:
                Xp, Pp = _predict(X, P, q, g.r[l], g)
                out = Xp[:, 2].abs() > g.z_half
            Xu, Pu, d, pd = _update(Xp, Pp, h[:3].T, h[3:].T)
            Xn = torch.where(use[:, None], Xu, Xp)
            Pn = torch.where(use[:, None, None], Pu, Pp)
            live = live & ~out & (pd | ~use) & torch.isfinite(Xn).all(1) & torch.isfinite(Pn).all(2).all(1)
            X = torch.where(live[:, None], Xn, X)
            P = torch.where(live[:, None, None], Pn, P)
            c2 = torch.where(live & use, c2 + d, c2)
        par[:, a:b], cov[:, a:b], chi2[a:b] = X.T, _pack(P), c2
    return dict(par=par, cov=cov, chi2=chi2, ndof=None, status=None)


def _exact_bin(case, seed):
    e, c = _events(case, seed), presets.BuildCuts()
    g, L, nb = e["g"], e["g"].n_layers, c.n_phi_bins * c.n_z_bins
    x, y, z = e["xyz"].to(D)
    ph = torch.atan2(y, x)
    ph = torch.where(ph < 0, ph + 2 * math.pi, ph).float()
    ip = torch.floor(ph.to(D) * c.n_phi_bins / (2 * math.pi)).clamp(0, c.n_phi_bins - 1).long()
    iz = torch.floor((z + g.z_half) * c.n_z_bins / (2 * g.z_half)).clamp(0, c.n_z_bins - 1).long()
    ev = torch.bucketize(torch.arange(len(x), device=DEV), e["hoff"].long(), right=True) - 1
    gb = (ev * L + e["layer"].long()) * nb + iz * c.n_phi_bins + ip
    o = torch.argsort(ph, stable=True)
    o = o[torch.argsort(gb[o], stable=True)]
    return dict(offsets=None, xyzphi=torch.cat([e["xyz"].to(D), ph.to(D)[None]], 0)[:, o], cov=e["cov"].to(D)[:, o],
                orig=None, bad=None)


def _exact_mlp(case, seed):
    rows, w, m, v = _mlp_rows(case, seed)
    T = lambda a: torch.from_numpy(a.astype(np.float64)).to(DEV)
    p = T(w).requires_grad_(True)
    o, parts = 0, []
    for shp in ((64, 27), (64,), (64, 64), (64,), (2, 64), (2,)):
        k = int(np.prod(shp))
        parts.append(p[o:o + k].reshape(shp))
        o += k
    W1, b1, W2, b2, W3, b3 = parts
    x = (rows[:, :27].to(D) - T(_MU)) / T(_SD)
    a = torch.nn.functional.gelu(x @ W1.t() + b1)
    a = torch.nn.functional.gelu(a @ W2.t() + b2)
    wd = T(_SCALE) * torch.nn.functional.softplus(a @ W3.t() + b3)
    d = rows[:, 27:29].to(D)
    loss = (20 * (d - wd).clamp(min=0) + (wd - d).clamp(min=0)).mean()
    loss.backward()
    gr = p.grad
    mm, vv = 0.9 * T(m) + 0.1 * gr, 0.999 * T(v) + 0.001 * gr * gr
    new = p.detach() - 1e-3 * (mm / (1 - 0.9 ** 100)) / (torch.sqrt(vv / (1 - 0.999 ** 100)) + 1e-8)
    return dict(grad=torch.cat([gr, loss.detach()[None]]), w=new, m=mm, v=vv)


def exact(case, seed):
    """FP64 values by plain torch.  A build has none: its lists hang on
    thresholds (chi2 cut, window edges, ranks), so the value of a later layer
    is not a function that can be taken in 64 bits alone; the event's seeds
    are."""
    kind = case["kind"]
    if kind == "fit":
        return _exact_fit(case, seed)
    if kind == "bin":
        return _exact_bin(case, seed)
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if kind == "event":
        e = _events(case, seed)
        n = e["n"]
        X, P, _, _ = _seed64(e["H3"][:, :, :n], e["g"])
        par = torch.zeros((6, e["ld"]), dtype=D, device=DEV)
        cov = torch.zeros((21, e["ld"]), dtype=D, device=DEV)
        par[:, :n], cov[:, :n] = X.T, _pack(P)
        return dict(seed=dict(par=par, cov=cov, q=None), build=None, fit=None)
    return None
