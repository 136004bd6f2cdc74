"""Measured cases: the work that a user of the detector has it do.

Four families, each through the package's public calls: detection of a block
of received vectors with a frozen model, training of one detector (and the
cyclic projections that continue one), a batch of detectors trained and
detected together, and the differentiable unrolled training (loss and
gradient).  Inputs follow the uplink model of `synth`: i.i.d. Rayleigh
channel, QPSK or 16-QAM, AWGN, one real scale per instance so that the pilots
have unit mean squared norm.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2201_05024_amd as A

MODS = ("qpsk", "qam16")
LEVELS = {"qpsk": (-1 / math.sqrt(2), 1 / math.sqrt(2)),
          "qam16": tuple(v / math.sqrt(10) for v in (-3, -1, 1, 3))}


def listed():
    return [
        # ---- detection: K users, M antennas, D dictionary entries, S vectors
        # the small plain call, where launch latency counts
        dict(name="detect_small", kind="detect", K=4, M=8, D=256, S=2048, mod="qpsk", snr=10.0),
        # the paper's own shape (Sec. V): 685 pilots, 3840 data symbols
        dict(name="detect_paper", kind="detect", K=6, M=16, D=1370, S=3840, mod="qpsk", snr=20.0),
        # a whole slot of one 16-antenna receiver
        dict(name="detect_slot", kind="detect", K=6, M=16, D=1024, S=1048576, mod="qpsk", snr=10.0),
        # the large array: 16 users, 64 antennas, a full dictionary
        dict(name="detect_array", kind="detect", K=16, M=64, D=8192, S=1048576, mod="qam16", snr=20.0),
        # ---- training of one detector: P pilots, window W, capacity cap
        # the small plain call
        dict(name="train_small", kind="train", K=4, M=8, P=256, W=16, cap=256, mod="qpsk", snr=10.0),
        # the slot's pilots; the capacity binds halfway
        dict(name="train_slot", kind="train", K=6, M=16, P=1024, W=32, cap=1024, mod="qpsk", snr=10.0),
        # the large array's shape, 16 users on 64 antennas
        dict(name="train_array", kind="train", K=16, M=64, P=2048, W=32, cap=2048, mod="qam16", snr=20.0),
        # cyclic projections from a linear MMSE start: mixed set kinds, weights
        # by violation, continued cycles and the ball; odd sizes
        dict(name="pocs_warm", kind="pocs", K=5, M=11, P=333, W=20, cap=500, mod="qpsk", snr=12.0, cycles=3,
             radius=3.0),
        # ---- batches, trained and detected together
        # many small cells of mixed shapes (K 2..8, 8/16/32 antennas)
        dict(name="batch_mixed", kind="batch_mixed", detectors=64, pmin=64, pmax=2048, S=16384, W=32, shapes=11),
        # several large arrays
        dict(name="batch_array", kind="batch_array", detectors=4, K=16, M=64, P=4096, W=32, cap=4096, S=131072,
             mod="qam16", snr=20.0),
        # ---- unrolled training, loss and gradient: n detectors, `passes` iterations
        # a small one, as in a first trial of the design parameters
        dict(name="unrolled_small", kind="unrolled", n=4, K=4, M=8, P=64, S=256, W=8, passes=4, every=2, snr=10.0),
        # learning the design parameters over 64 slots
        dict(name="unrolled_slots", kind="unrolled", n=64, K=6, M=16, P=512, S=4096, W=32, passes=20, every=5,
             snr=10.0),
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["detect", "detect", "train", "train", "pocs", "batch_mixed", "batch_array", "unrolled"])
    mod, snr = rng.choice(MODS), round(rng.uniform(5.0, 20.0), 1)
    if kind == "detect":
        M, K, D = _log_int(rng, 8, 64), rng.randint(2, 16), _log_int(rng, 64, 8192)
        top = min(1 << 20, (1 << 33) * 144 // (D * (2 * M + K)))
        return dict(kind=kind, K=K, M=M, D=D, S=_log_int(rng, 1024, top), mod=mod, snr=snr)
    if kind == "train":
        P = _log_int(rng, 64, 1536)
        return dict(kind=kind, K=rng.randint(2, 16), M=_log_int(rng, 8, 64), P=P, W=rng.randint(8, 32),
                    cap=_log_int(rng, max(64, P // 2), 2048), mod=mod, snr=snr)
    if kind == "pocs":
        P = _log_int(rng, 64, 512)
        return dict(kind=kind, K=rng.randint(2, 8), M=_log_int(rng, 8, 32), P=P,
                    W=rng.randint(8, 32), cap=_log_int(rng, max(64, P // 2), 1024), mod=mod, snr=snr, cycles=rng.randint(2, 4),
                    radius=round(rng.uniform(1.0, 6.0), 2))
    if kind == "batch_mixed":
        return dict(kind=kind, detectors=_log_int(rng, 4, 64), pmin=64, pmax=_log_int(rng, 128, 2048),
                    S=_log_int(rng, 1024, 16384), W=rng.randint(8, 32), shapes=rng.randint(0, 1 << 30))
    if kind == "batch_array":
        P = _log_int(rng, 512, 4096)
        return dict(kind=kind, detectors=rng.randint(2, 4), K=rng.randint(9, 16), M=rng.randint(33, 64), P=P,
                    W=rng.randint(16, 32), cap=rng.randint(max(512, P // 2), 4096), S=_log_int(rng, 4096, 131072), mod="qam16",
                    snr=snr)
    return dict(kind=kind, n=_log_int(rng, 2, 64), K=rng.randint(2, 8), M=_log_int(rng, 4, 16),
                P=_log_int(rng, 32, 512), S=_log_int(rng, 128, 4096), W=rng.randint(4, 32),
                passes=rng.randint(2, 20), every=rng.randint(1, 6), snr=snr)


# ---------------------------------------------------------------- inputs

def _gen(seed: int, salt: int = 0):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + salt * 7919 + 17) % (1 << 62))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _block(g, n, H, mod, n0):
    """n received vectors [n][2M] (unscaled), symbols [n][K][2], labels [n][K]."""
    lv = torch.tensor(LEVELS[mod], device="cuda")
    K, M = H.shape[1], H.shape[0]
    idx = torch.randint(0, len(LEVELS[mod]), (n, K, 2), generator=g, device="cuda")
    sym = lv[idx]
    br, bi = sym[..., 0], sym[..., 1]
    hr, hi = H.real.T.contiguous(), H.imag.T.contiguous()
    rx = torch.cat([br @ hr - bi @ hi, br @ hi + bi @ hr], dim=1)
    rx += _randn(g, n, 2 * M) * math.sqrt(n0 / 2)
    gray = idx ^ (idx >> 1)
    bits = 1 if mod == "qpsk" else 2
    return rx, sym.contiguous(), ((gray[..., 0] << bits) | gray[..., 1]).to(torch.uint8)


def _instance(seed, salt, K, M, P, S, mod, snr):
    """One instance: pilots, data and the channel scaled as the stored vectors."""
    g = _gen(seed, salt)
    H = torch.complex(_randn(g, M, K), _randn(g, M, K)) / math.sqrt(2)
    n0 = 10.0 ** (-snr / 10)
    rp, sp, _ = _block(g, P, H, mod, n0)
    scale = 1.0 / torch.sqrt((rp * rp).sum(1).mean())
    inst = dict(rx_pilot=(rp * scale).contiguous(), sym_pilot=sp, n0=n0 * float(scale) ** 2,
                h=(torch.cat([H.real, H.imag]).T * scale).contiguous())
    if S:
        rd, sd, truth = _block(g, S, H, mod, n0)
        inst.update(rx=(rd * scale).contiguous(), sym=sd, truth=truth)
    return inst


def _real_rows(rx):
    """Training sequence r_{2t} = r1(t), r_{2t+1} = r2(t) of pilots [P][2M]."""
    M = rx.shape[1] // 2
    return torch.stack([rx, torch.cat([rx[:, M:], -rx[:, :M]], 1)], 1).reshape(-1, 2 * M).contiguous()


def _detect_inputs(c, seed):
    """A detector as training leaves it: the pilots' newest D real vectors as
    dictionary, a least-squares linear part, small Gaussian coefficients."""
    i = _instance(seed, 1, c["K"], c["M"], (c["D"] + 1) // 2, c["S"], c["mod"], c["snr"])
    R = _real_rows(i["rx_pilot"])
    B = i["sym_pilot"].transpose(1, 2).reshape(-1, c["K"])
    eye = torch.eye(R.shape[1], device="cuda")
    w = torch.linalg.solve(R.T @ R + 0.05 * eye, R.T @ B).T.contiguous()
    alpha = _randn(_gen(seed, 2), c["D"], c["K"]) * 0.02
    return dict(i, dict_rows=R[:c["D"]].contiguous(), alpha=alpha, w=w)


def _set_types(seed, P, K):
    """Mostly hyperslabs, some hyperplanes and halfspaces."""
    g = _gen(seed, 3)
    u = torch.rand((P, K, 2), generator=g, device="cuda")
    t = torch.randint(1, 4, (P, K, 2), generator=g, device="cuda")
    return torch.where(u < 0.8, torch.zeros_like(t), t).to(torch.uint8).contiguous()


def _mixed_shapes(c):
    rng = random.Random(c["shapes"])
    out = []
    for _ in range(c["detectors"]):
        out.append(dict(K=rng.randint(2, 8), M=rng.choice([8, 16, 32]), P=rng.randint(c["pmin"], c["pmax"]),
                        mod=rng.choice(MODS), snr=rng.uniform(5.0, 20.0)))
    for s in out:
        s["cap"] = max(s["P"], c["W"])
    return out


def _batch_shapes(c):
    if c["kind"] == "batch_mixed":
        return _mixed_shapes(c)
    return [dict(K=c["K"], M=c["M"], P=c["P"], mod=c["mod"], snr=c["snr"], cap=c["cap"])] * c["detectors"]


def _params(c, **kw):
    return A.Params(sigma2=0.5, eps=0.05, mu=1.0, window=c["W"], w_lin=0.5, w_gauss=0.5, **kw)


def _unrolled_inputs(c, seed):
    insts = [_instance(seed, 100 + b, c["K"], c["M"], c["P"], c["S"], "qpsk", c["snr"]) for b in range(c["n"])]
    data = [torch.stack([i[k] for i in insts]).contiguous() for k in ("rx_pilot", "sym_pilot", "rx", "sym")]
    om = 0.5 + torch.rand(c["W"], generator=_gen(seed, 5), device="cuda")
    # over-relaxed, with a wide slab: at mu = 1 the first projection of a pass
    # ends exactly on the threshold, where the loss has no derivative
    return data, torch.cat([torch.tensor([0.7, 0.2, 1.3], device="cuda"), om])


# The arrays of a batch's detectors are views of one tensor each, every one
# from a 256-byte boundary on: the models and the soft values come back whole.
_PARTS = ("dict", "alpha", "w", "state", "soft")


def _batch_sizes(c):
    for s in _batch_shapes(c):
        M2, K = 2 * s["M"], s["K"]
        yield dict(dict=(M2, s["cap"]), alpha=(s["cap"], K), w=(K, M2), state=(4,), soft=(c["S"], K, 2))


def _flat(sizes, part, make):
    at, n = [], 0
    for z in sizes:
        at.append(n)
        n += (math.prod(z[part]) + 63) // 64 * 64
    whole = make(n)
    return whole, [whole[o:o + math.prod(z[part])].view(z[part]) for o, z in zip(at, sizes)]


def _batch_state(c, seed):
    shapes, sizes = _batch_shapes(c), list(_batch_sizes(c))
    whole, views = {}, {}
    for p in _PARTS:
        dt = torch.int32 if p == "state" else torch.float32
        whole[p], views[p] = _flat(sizes, p, lambda n: torch.zeros(n, dtype=dt, device="cuda"))
    items = []
    for b, s in enumerate(shapes):
        i = _instance(seed, 10 + b, s["K"], s["M"], s["P"], c["S"], s["mod"], s["snr"])
        m = A.Model(2 * s["M"], s["K"], s["cap"], sigma2=0.5)
        for p in _PARTS[:4]:
            setattr(m, p, views[p][b])
        # soft values only: they feed a channel decoder
        items.append(A.BatchItem(model=m, rx_pilot=i["rx_pilot"], sym_pilot=i["sym_pilot"], rx=i["rx"],
                                 modulation=None, soft=views["soft"][b], sigma2=0.5))
    return dict(case=c, batch=A.Batch(_params(c), items), whole=[whole[p] for p in _PARTS])


def prepare(c, seed):
    k = c["kind"]
    if k == "detect":
        i = _detect_inputs(c, seed)
        m = A.Model(2 * c["M"], c["K"], c["D"], sigma2=0.5)
        m.dict.copy_(i["dict_rows"].T)
        m.alpha.copy_(i["alpha"])
        m.w.copy_(i["w"])
        m.state.copy_(torch.tensor([c["D"], 0, c["D"], 0], dtype=torch.int32))
        m.pack()
        return dict(case=c, model=m, rx=i["rx"], truth=i["truth"])
    if k in ("train", "pocs"):
        i = _instance(seed, 1, c["K"], c["M"], c["P"], 0, c["mod"], c["snr"])
        m = A.Model(2 * c["M"], c["K"], max(c["cap"], c["W"]), sigma2=0.5)
        if k == "train":
            return dict(case=c, model=m, params=_params(c, dict_cap=m.dict_cap), **i)
        p = _params(c, dict_cap=m.dict_cap, init="linear", weights="violation",
                    set_types=_set_types(seed, c["P"], c["K"]))
        return dict(case=c, model=m, params=p, ws=A.ball_workspace(m), **i)
    if k in ("batch_mixed", "batch_array"):
        return _batch_state(c, seed)
    data, theta = _unrolled_inputs(c, seed)
    return dict(case=c, data=data, theta=theta.requires_grad_(True))


def _model_out(m):
    return [m.dict, m.alpha, m.w, m.state]


def run(st):
    c = st["case"]
    k = c["kind"]
    if k == "detect":
        o = A.detect(st["model"], st["rx"], modulation=c["mod"], truth=st["truth"])
        return [o["soft"], o["hard"], o["errors"]]
    if k == "train":
        return _model_out(A.train(st["rx_pilot"], st["sym_pilot"], st["params"], model=st["model"]))
    if k == "pocs":
        A.linear_mmse(st["h"], st["n0"], w=st["model"].w)
        return _model_out(A.pocs(st["rx_pilot"], st["sym_pilot"], st["params"], radius=c["radius"],
                                 cycles=c["cycles"], model=st["model"], workspace=st["ws"]))
    if k in ("batch_mixed", "batch_array"):
        st["batch"].train().detect()
        return st["whole"]
    st["theta"].grad = None
    loss = A.unrolled_loss(st["theta"], *st["data"], passes=c["passes"], ckpt_every=c["every"])
    loss.backward()
    return [loss.detach(), st["theta"].grad]


# ---------------------------------------------------------------- work

def _train_work(K, M, P, W, cap):
    """Kernel values of every step against the entries it sees, the new
    member's prediction, the update of the window's predictions and of w."""
    T, M2 = 2 * P, 2 * M
    cap = min(max(cap, W), T)
    vals = cap * (cap + 1) // 2 + (T - cap) * cap
    flops = vals * (2 * M2 + 3 + 2 * K) + T * (2 * W * W * K + 2 * W * K * M2)
    return 4 * (P * M2 + 2 * P * K + cap * (M2 + K) + K * M2), flops


def _detect_work(K, M, D, S):
    M2 = 2 * M
    return (4 * S * M2 + S * K * 10 + 4 * (D * (M2 + K) + K * M2),
            2 * S * (D * (2 * M2 + 3 + 2 * K) + 2 * M2 * (K + 1)))


def work(c):
    k = c["kind"]
    if k == "detect":
        parts = [_detect_work(c["K"], c["M"], c["D"], c["S"])]
    elif k == "train":
        parts = [_train_work(c["K"], c["M"], c["P"], c["W"], c["cap"])]
    elif k == "pocs":
        b, f = _train_work(c["K"], c["M"], c["P"], c["W"], c["cap"])
        D = min(c["cap"], 2 * c["P"])
        parts = [(b, c["cycles"] * (f + D * D * (4 * c["M"] + 3 + 2 * c["K"])))]
    elif k in ("batch_mixed", "batch_array"):
        parts = []
        for s in _batch_shapes(c):
            parts.append(_train_work(s["K"], s["M"], s["P"], c["W"], s["cap"]))
            parts.append(_detect_work(s["K"], s["M"], min(s["cap"], 2 * s["P"]), c["S"]))
    else:
        n, K, M2, T, S, W = c["n"], c["K"], 2 * c["M"], 2 * c["P"], c["S"], c["W"]
        step = 2 * T * K + 2 * W * W * K + 2 * W * K * M2
        # forward: Gram matrix, passes, validation; backward: the forward again
        # with the sigma sums, the reverse sweep, the validation's adjoint
        fl = T * T * (2 * M2 + 3) + c["passes"] * T * step * 4 + 2 * S * T * (4 * M2 + 6 + 6 * K)
        parts = [(4 * n * (c["P"] + S) * (M2 + 2 * K), n * fl)]
    return {"bytes": int(sum(p[0] for p in parts)), "flops": int(sum(p[1] for p in parts))}


# ---------------------------------------------------------------- exact

def _exact_detect(dict_rows, alpha, w, rx, mod, truth):
    """Soft outputs, labels and error counts in 64 bits (on the GPU)."""
    d, a, w = dict_rows.double(), alpha.double(), w.double()
    S, K, M = rx.shape[0], w.shape[0], rx.shape[1] // 2
    dn = (d * d).sum(1)
    soft = torch.empty((S, K, 2), dtype=torch.float64, device=rx.device)
    step = max(256, (1 << 27) // max(d.shape[0], 1))
    for s0 in range(0, S, step):
        x = rx[s0:s0 + step].double()
        for p in range(2):
            v = x if p == 0 else torch.cat([x[:, M:], -x[:, :M]], 1)
            d2 = (v * v).sum(1)[:, None] + dn[None] - 2.0 * (v @ d.T)
            soft[s0:s0 + step, :, p] = torch.exp(-d2.clamp_(min=0.0)) @ a + v @ w.T
    if mod == "qpsk":
        idx, bits = (soft >= 0).int(), 1
    else:
        th = 2 / math.sqrt(10)
        idx, bits = (soft >= -th).int() + (soft >= 0).int() + (soft >= th).int(), 2
    gray = idx ^ (idx >> 1)
    hard = ((gray[..., 0] << bits) | gray[..., 1]).to(torch.uint8)
    return soft, hard, (hard != truth).sum(0)


class _Trainer64:
    """The windowed parallel projections in 64 bits: a ring of `cap` Gaussian
    entries, running window predictions (exact up to rounding)."""

    def __init__(self, M2, K, cap, W, w0=None):
        self.M2, self.K, self.cap, self.W = M2, K, cap, W
        self.d, self.a, self.n0 = np.zeros((cap, M2)), np.zeros((cap, K)), 0
        self.w = np.zeros((K, M2)) if w0 is None else w0.copy()

    def block(self, R, B, violation=False, types=None, eps=np.float64(np.float32(0.05))):
        T, cap, W, K = len(R), self.cap, self.W, self.K
        nrm = (R * R).sum(1)
        lin = R @ R.T
        G = np.exp(-np.maximum(nrm[:, None] + nrm[None] - 2 * lin, 0.0))       # 2 sigma^2 = 1
        np.fill_diagonal(G, 1.0)
        lin *= 0.5
        lin += 0.5 * G
        Kf, old, n0 = lin, self.d, self.n0
        used = min(n0, cap)
        if used:
            on = (old[:used] ** 2).sum(1)
            Go = np.exp(-np.maximum(nrm[:, None] + on[None] - 2 * (R @ old[:used].T), 0.0))
        e = np.zeros((T, K))
        src = np.full(cap, -1)                   # block sample in each slot (-1: an older entry)
        krow = np.zeros(cap)
        a, w = self.a, self.w
        for n in range(T):
            slot = (n0 + n) % cap
            J = np.arange(max(0, n - W + 1), n + 1)
            if n0 + n >= cap and n:              # the oldest entry leaves
                kv = G[J[:-1], src[slot]] if src[slot] >= 0 else Go[J[:-1], slot]
                e[J[:-1]] -= kv[:, None] * a[slot][None]
            a[slot] = 0.0
            src[slot] = n
            if used:
                krow[:used] = Go[n]
            lo = max(0, n - cap + 1)
            krow[np.arange(n0 + lo, n0 + n + 1) % cap] = G[n, lo:n + 1]
            e[n] = krow @ a + w @ R[n]
            x = e[J] - B[J]
            res = np.sign(x) * np.maximum(np.abs(x) - eps, 0.0)
            if types is not None:
                t = types[J]
                res = np.where(t == 1, x, np.where(t == 2, np.maximum(x - eps, 0.0),
                                                   np.where(t == 3, np.minimum(x + eps, 0.0), res)))
            beta = -res / Kf[J, J][:, None]
            if violation:
                v = np.abs(res)
                tot = v.sum(0)
                c = beta * v / np.where(tot > 0, tot, 1.0)
            else:
                c = beta / len(J)
            e[J] += Kf[np.ix_(J, J)] @ c
            a[(n0 + J) % cap] += 0.5 * c
            w += 0.5 * (c.T @ R[J])
        i = np.arange(max(0, T - cap), T)
        self.d[(n0 + i) % cap] = R[i]
        self.n0 += T

    def ball(self, radius):
        used = min(self.n0, self.cap)
        d, a = self.d[:used], self.a[:used]
        dn = (d * d).sum(1)
        G = np.exp(-np.maximum(dn[:, None] + dn[None] - 2 * (d @ d.T), 0.0))
        nrm = np.sqrt(np.maximum((self.w ** 2).sum(1) / 0.5 + (a * (G @ a)).sum(0) / 0.5, 0.0))
        sc = np.where(nrm > radius, radius / np.maximum(nrm, 1e-300), 1.0)
        self.w *= sc[:, None]
        self.a *= sc[None]

    def outputs(self):
        st = torch.tensor([min(self.n0, self.cap), self.n0 % self.cap, self.n0, 0], dtype=torch.int32)
        return [torch.from_numpy(self.d.T.copy()), torch.from_numpy(self.a.copy()), torch.from_numpy(self.w.copy()), st]


def _sequence64(i):
    R = _real_rows(i["rx_pilot"]).double().cpu().numpy()
    K = i["sym_pilot"].shape[1]
    return R, i["sym_pilot"].transpose(1, 2).reshape(-1, K).double().cpu().numpy()


def _mmse64(h, n0):
    M = h.shape[1] // 2
    h = h.double().cpu().numpy()
    H = (h[:, :M] + 1j * h[:, M:]).T
    U = H @ np.linalg.inv(H.conj().T @ H + np.float64(np.float32(n0)) * np.eye(H.shape[1]))
    return np.concatenate([U.real, U.imag]).T.copy()


def _exact_unrolled(c, seed):
    """Loss and gradient by automatic differentiation in 64 bits (on the GPU)."""
    data, theta = _unrolled_inputs(c, seed)
    th = theta.double().requires_grad_(True)
    sigma, eps, mu, om = th[0], th[1], th[2], th[3:]
    W, K, T, n = c["W"], c["K"], 2 * c["P"], c["n"]
    rows = lambda x: torch.stack([_real_rows(v) for v in x.double()])                    # noqa: E731
    syms = lambda s: s.double().transpose(2, 3).reshape(n, -1, K)                        # noqa: E731
    R, B, V, BV = rows(data[0]), syms(data[1]), rows(data[2]), syms(data[3])

    def gauss(x, y):
        d2 = (x * x).sum(2)[:, :, None] + (y * y).sum(2)[:, None] - 2 * torch.matmul(x, y.transpose(1, 2).contiguous())
        return torch.exp(-d2.clamp(min=0.0) / (2 * sigma * sigma))

    G = gauss(R, R)
    Kf = 0.5 * torch.matmul(R, R.transpose(1, 2).contiguous()) + 0.5 * G
    kd = 0.5 * (R * R).sum(2) + 0.5
    C = torch.zeros((n, T, K), dtype=torch.float64, device="cuda")
    for _ in range(c["passes"]):
        e = torch.matmul(Kf, C)                  # predictions of every sample, kept up to date
        for t in range(T):
            lo = max(0, t - W + 1)
            x = e[:, lo:t + 1] - B[:, lo:t + 1]
            q = om[:t + 1 - lo].flip(0)
            beta = -torch.sign(x) * torch.relu(x.abs() - eps) / kd[:, lo:t + 1, None]
            cs = mu * (q / q.sum())[None, :, None] * beta
            C = C + torch.nn.functional.pad(cs, (0, 0, lo, T - t - 1))
            e = e + torch.matmul(Kf[:, :, lo:t + 1].contiguous(), cs)
    w = 0.5 * torch.matmul(C.transpose(1, 2).contiguous(), R)
    f = 0.5 * torch.matmul(gauss(V, R), C) + torch.matmul(V, w.transpose(1, 2).contiguous())
    loss = ((f - BV) ** 2).sum() / (n * c["S"] * K)
    loss.backward()
    return [loss.detach(), th.grad]


def exact(c, seed):
    k = c["kind"]
    if k == "detect":
        i = _detect_inputs(c, seed)
        return list(_exact_detect(i["dict_rows"], i["alpha"], i["w"], i["rx"], c["mod"], i["truth"]))
    if k == "train":
        i = _instance(seed, 1, c["K"], c["M"], c["P"], 0, c["mod"], c["snr"])
        t = _Trainer64(2 * c["M"], c["K"], max(c["cap"], c["W"]), c["W"])
        t.block(*_sequence64(i))
        return t.outputs()
    if k == "pocs":
        i = _instance(seed, 1, c["K"], c["M"], c["P"], 0, c["mod"], c["snr"])
        t = _Trainer64(2 * c["M"], c["K"], max(c["cap"], c["W"]), c["W"], _mmse64(i["h"], i["n0"]))
        ty = _set_types(seed, c["P"], c["K"]).transpose(1, 2).reshape(-1, c["K"]).cpu().numpy()
        R, B = _sequence64(i)
        for _ in range(c["cycles"]):
            t.block(R, B, violation=True, types=ty)
            t.ball(float(np.float32(c["radius"])))
        return t.outputs()
    if k in ("batch_mixed", "batch_array"):
        shapes, sizes = _batch_shapes(c), list(_batch_sizes(c))
        if sum(2 * s["P"] * (1 + s["cap"] * s["K"] / 40000) for s in shapes) > 200000:
            return None
        whole, views = {}, {}
        for p in _PARTS:
            dt = torch.int32 if p == "state" else torch.float64
            whole[p], views[p] = _flat(sizes, p, lambda n: torch.zeros(n, dtype=dt))
        for b, s in enumerate(shapes):
            i = _instance(seed, 10 + b, s["K"], s["M"], s["P"], c["S"], s["mod"], s["snr"])
            t = _Trainer64(2 * s["M"], s["K"], s["cap"], c["W"])
            t.block(*_sequence64(i))
            m = t.outputs()
            soft, _, _ = _exact_detect(m[0].T.contiguous().cuda(), m[1].cuda(), m[2].cuda(), i["rx"], s["mod"],
                                       i["truth"])
            for p, v in zip(_PARTS, m + [soft.cpu()]):
                views[p][b].copy_(v)
        return [whole[p] for p in _PARTS]
    steps = 2 * c["P"] * c["passes"]
    if steps > 3000 or steps * c["n"] * 2 * c["P"] * c["W"] > 4e9:     # its tape would not be held
        return None
    return _exact_unrolled(c, seed)
