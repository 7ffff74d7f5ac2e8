"""The workloads the library's speed is judged on, and their exact results.

Each case is one call of a public entry point of ``paper_1702_04458_amd.api`` at
a shape that the configurations, the tests or ``bench.py`` use, or at an odd one
of the same ranges.  A case is a dict of plain values:

``op``      ``admm`` (Algorithm 1), ``cg`` (Algorithm 2), ``precode``
            (Algorithm 3), ``resident`` (iterations against a static channel's
            factors; ``h16``: H packed as complex FP16) or ``batch`` (uneven
            frames of one U in one call).
``B U C``   antennas, users, clusters; ``n_sc`` subcarriers, ``n_sym`` received
            (or target) vectors per subcarrier; ``T`` iterations.
``qam snr`` constellation and average receive SNR per antenna in dB.

Channels are i.i.d. Rayleigh CN(0, 1), symbols uniform over unit-energy QAM,
noise CN(0, U / SNR), rho = gamma = Es = 1.  ``prepare`` makes what a frame loop
holds: inputs, output buffers, the workspace of the exact hard decisions, and
for a static channel its factors.
"""
from __future__ import annotations

import math

import torch

from paper_1702_04458_amd import api, inputs

DEV = "cuda"
RHO = 1.0


# -- the cases ---------------------------------------------------------------

def _ul(name, op, B, U, C, n_sc, n_sym, T, qam, snr, reg="mmse", prec="fp32"):
    return {"name": name, "op": op, "B": B, "U": U, "C": C, "n_sc": n_sc, "n_sym": n_sym, "T": T, "qam": qam,
            "snr": float(snr), "reg": reg, "prec": prec}


def _dl(name, B, U, C, n_sc, n_sym, T, qam, layout="uplink", eps=0.0, power="none", P=0.0):
    return {"name": name, "op": "precode", "B": B, "U": U, "C": C, "n_sc": n_sc, "n_sym": n_sym, "T": T, "qam": qam,
            "layout": layout, "eps": float(eps), "power": power, "P": float(P)}


def listed():
    return [
        # The smallest call: 16 subcarriers of the 64-antenna configuration,
        # QPSK at 10 dB.  Latency of a lone small allocation.
        _ul("admm_u8_16sc", "admm", 64, 8, 4, 16, 1, 3, 4, 10),
        # One 1200-subcarrier OFDM symbol by conjugate gradients at 10 dB: the
        # per-frame latency of Algorithm 2, exact hard decisions included.
        _ul("cg_u16_frame", "cg", 128, 16, 8, 1200, 1, 5, 16, 10),
        # 32 such frames in one call by ADMM: the throughput form of the
        # 128-antenna configuration.
        _ul("admm_u16_32frames", "admm", 128, 16, 8, 38400, 1, 5, 16, 10),
        # An odd allocation: 731 subcarriers, 33 antennas in each of 6
        # clusters, box regulariser, 16-QAM at 10 dB.
        _ul("admm_u32_odd_box", "admm", 198, 32, 6, 731, 1, 5, 16, 10, reg="box"),
        # The headline shape: 32 frames of 1200 subcarriers, 64-QAM at 25 dB.
        _ul("admm_u32_32frames", "admm", 256, 32, 8, 38400, 1, 5, 64, 25),
        # The largest array, one frame at 10 dB: the tail of a serving mix,
        # where many subcarriers need the exact FP64 decisions.
        _ul("admm_u64_frame", "admm", 512, 64, 8, 1200, 1, 5, 16, 10),
        # Mixed precision (split FP16 Gram) at the largest array, 8 frames of
        # 64-QAM at 25 dB.
        _ul("mixed_u64_8frames", "admm", 512, 64, 8, 9600, 1, 5, 64, 25, prec="fp16"),
        # Seven symbols per subcarrier over one channel (half a slot), one
        # factorisation reused over them.
        _ul("admm_u32_7symbols", "admm", 256, 32, 8, 5485, 7, 5, 64, 25),
        # A served static channel kept as FP16 with FP32 factors: the
        # iterations alone, soft outputs.
        _ul("resident_h16_u32", "resident", 256, 32, 8, 38400, 1, 5, 64, 25, prec="h16"),
        # Downlink precoding, 32 frames, per-cluster budgets met by the common
        # gain.
        _dl("precode_u32_32frames", 256, 32, 16, 38400, 1, 5, 64, power="common_gain", P=0.013),
        # One precoded frame with the budgets inside every x-update (binding on
        # about half of the clusters).
        _dl("precode_u32_budget", 256, 32, 16, 1200, 1, 5, 64, power="per_cluster", P=0.013),
        # Eight uneven frames of 16 users in one call, as the serving loop
        # batches them.
        {"name": "batch_u16_uneven", "op": "batch", "U": 16, "n_frames": 8, "mix": 1, "T": 5},
    ]


# Valid (B, U, C) of the serving mix, and uneven cluster sizes besides.
_SHAPES = inputs.serving_shapes()
_MOST = 38400 * 8 * (32 * 32 * 32 * 1.5 + 32.0 ** 3)   # matrix work of the headline call


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _uplink_shape(rng):
    if rng.random() < 0.5:
        return rng.choice(_SHAPES)
    U = rng.choice((8, 16, 32, 64))
    C = rng.randint(1, min(16, 512 // U))
    S = min(_log_int(rng, U, 4 * U), 1024 // C) if 1024 // C >= U else U
    return (S * C, U, C)


def _capped(rng, per_sc, lo=16, hi=38400):
    """Subcarriers of a call that costs no more than the headline one."""
    return _log_int(rng, lo, max(lo + 1, min(hi, int(_MOST / per_sc))))


def draw(rng):
    op = rng.choice(("admm", "admm", "admm", "cg", "precode", "precode", "resident", "batch"))
    if op == "batch":
        return {"op": "batch", "U": rng.choice((8, 16, 32)), "n_frames": rng.randint(2, 12),
                "mix": rng.randint(2, 1 << 20), "T": rng.randint(3, 6)}
    T = rng.randint(3, 8)
    if op == "precode":
        U = rng.choice((8, 16, 32, 64))
        C = rng.choice([c for c in (2, 3, 4, 6, 8, 12, 16) if c * U <= 512])
        S = rng.randint(max(-(-U // C), U // 4), U)
        power = rng.choice(("none", "none", "common_gain", "per_cluster"))
        n_sym = rng.choice((1, 1, 2, 7))
        # each x-update of the budgeted form factors up to six times
        per = C * (U * S * S * 1.5 + S ** 3 + 4.0 * n_sym * T * U * S) * (6 * T * n_sym if power == "per_cluster" else 1)
        return {"op": "precode", "B": S * C, "U": U, "C": C, "n_sc": _capped(rng, 4 * per, hi=9600), "n_sym": n_sym,
                "T": T, "qam": rng.choice((4, 16, 64)), "layout": rng.choice(("uplink", "downlink")),
                "eps": rng.choice((0.0, 0.0, 0.3)), "power": power,
                # about the mean per-cluster energy of an unbudgeted precoder with S C > U
                "P": 0.0 if power == "none" else 0.9 * U / C / max(S * C - U, U / 2)}
    B, U, C = _uplink_shape(rng)
    n_sym = rng.choice((1, 1, 1, 2, 7, 14))
    per = 2 * C * ((B // C) * U * U * 1.5 + U ** 3 + n_sym * T * U * U)
    prec = "fp32"
    if op == "admm" and U >= 32 and rng.random() < 0.3:
        prec = rng.choice(("fp16", "bf16"))
    if op == "resident":
        prec = rng.choice(("fp32", "h16"))
    return {"op": op, "B": B, "U": U, "C": C, "n_sc": _capped(rng, per), "n_sym": n_sym, "T": T,
            "qam": rng.choice((4, 16, 64)), "snr": float(rng.randint(0, 25)),
            "reg": rng.choice(("mmse", "mmse", "zf") if op == "cg" else ("mmse", "mmse", "zf", "box")), "prec": prec}


# -- inputs --------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7fffffff)
    return g


def _cn(g, shape, var=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.complex64) * math.sqrt(var)


def _symbols(g, shape, qam):
    L, kappa = inputs.qam_side(qam), inputs.qam_kappa(qam)
    i = torch.randint(0, L, shape, generator=g, device=DEV)
    q = torch.randint(0, L, shape, generator=g, device=DEV)
    return (torch.complex((2 * i - (L - 1)).float(), (2 * q - (L - 1)).float()) / kappa).contiguous()


def _uplink(g, n_sc, n_sym, B, U, qam, snr):
    H = _cn(g, (n_sc, B, U))
    N0 = U / 10.0 ** (snr / 10.0)
    s = _symbols(g, (n_sc, U, n_sym), qam)
    y = torch.matmul(H, s).transpose(1, 2) + _cn(g, (n_sc, n_sym, B), N0)
    return H.contiguous(), y.contiguous(), N0


def _mix(case):
    """The frames of a batch: (B, C, n_sc, qam, snr) drawn from the serving
    shapes of this U (subcarriers 72, 300, 600 or 1200)."""
    import random

    r = random.Random(case["mix"])
    shapes = [s for s in _SHAPES if s[1] == case["U"]]
    frames = []
    for _ in range(case["n_frames"]):
        B, _, C = r.choice(shapes)
        frames.append((B, C, r.choice((72, 300, 600, 1200)), r.choice((16, 64)), float(r.choice((0, 5, 10, 15, 20)))))
    return frames


def prepare(case, seed):
    g = _gen(seed)
    op, U = case["op"], case["U"]
    if op == "batch":
        frames = []
        for B, C, n_sc, qam, snr in _mix(case):
            H, y, N0 = _uplink(g, n_sc, 1, B, U, qam, snr)
            frames.append(dict(H=H, y=y, N0=N0, C=C, T=case["T"], qam=qam, workspace=api.workspace(n_sc, U, C)))
        return {"case": case, "frames": frames}
    B, C, n_sc, n_sym = case["B"], case["C"], case["n_sc"], case["n_sym"]
    if op == "precode":
        H = _cn(g, (n_sc, B, U) if case["layout"] == "uplink" else (n_sc, U, B))
        s = _symbols(g, (n_sc, n_sym, U), case["qam"])
        P = None if case["power"] == "none" else torch.full((C,), case["P"], dtype=torch.float32, device=DEV)
        out = (torch.empty((n_sc, n_sym, B), dtype=torch.complex64, device=DEV),
               torch.empty((n_sc, n_sym), dtype=torch.float32, device=DEV))
        return {"case": case, "H": H, "s": s, "P": P, "out": out}
    H, y, N0 = _uplink(g, n_sc, n_sym, B, U, case["qam"], case["snr"])
    st = {"case": case, "H": H, "y": y, "N0": N0}
    s_hat = torch.empty((n_sc, n_sym, U), dtype=torch.complex64, device=DEV)
    hard = torch.empty((n_sc, n_sym, U), dtype=torch.uint8, device=DEV)
    if op == "resident" and case["prec"] == "h16":
        st["factors"], st["packed"] = api.factor_h16(H, C, RHO)
        st["out"] = (s_hat, None)
        return st
    if op == "resident":
        st["factors"] = api.factor(H, C, RHO)
    st["out"] = (s_hat, hard)
    st["workspace"] = api.workspace(n_sc, U, C)
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "batch":
        return api.detect_batch(st["frames"])
    if op == "precode":
        kw = {} if st["P"] is None else {"P_cluster": st["P"], "power": case["power"]}
        return api.precode(st["H"], st["s"], case["C"], RHO, case["T"], eps=case["eps"], layout=case["layout"],
                           out=st["out"], **kw)
    kw = dict(reg=case["reg"], qam=case["qam"], out=st["out"])
    if op == "resident" and case["prec"] == "h16":
        s_hat, _ = api.detect_factored_h16(st["packed"], st["factors"], st["y"], st["N0"], case["B"], case["U"],
                                           case["C"], RHO, case["T"], hard=False, **kw)
        return s_hat
    if op == "resident":
        return api.detect_factored(st["H"], st["factors"], st["y"], st["N0"], case["C"], RHO, case["T"],
                                   workspace=st["workspace"], **kw)
    return api.detect(st["H"], st["y"], st["N0"], case["C"], RHO, case["T"], algo=op, prec=case["prec"],
                      workspace=st["workspace"], **kw)


# -- what one pass cannot do without ---------------------------------------------

def _ul_work(op, prec, B, U, C, n_sc, n_sym, T):
    """Complex multiply-adds (8 flops): the Hermitian Gram, a U^3 / 6
    factorisation and one U x U solve per estimate; for CG H p and H^H (H p)."""
    S = B // C
    h = 4 if prec == "h16" else 8
    nbytes = h * B * U + n_sym * (8 * B + 8 * U + (0 if prec == "h16" else U))
    if op == "cg":
        cm = n_sym * B * U * (1 + 2 * T)
    else:
        cm = n_sym * (B * U + T * C * U * U)
        if op == "resident":
            nbytes += 8 * C * (U * (U + 1) // 2)
        else:
            cm += C * S * U * (U + 1) / 2 + C * U ** 3 / 6
    return n_sc * nbytes, 8.0 * n_sc * cm


def work(case):
    op, U, T = case["op"], case["U"], case["T"]
    if op == "batch":
        parts = [_ul_work("admm", "fp32", B, U, C, n_sc, 1, T) for B, C, n_sc, _, _ in _mix(case)]
        return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}
    B, C, n_sc, n_sym = case["B"], case["C"], case["n_sc"], case["n_sym"]
    if op != "precode":
        nbytes, flops = _ul_work(op, case["prec"], B, U, C, n_sc, n_sym, T)
        return {"bytes": float(nbytes), "flops": float(flops)}
    S = B // C
    cm = C * U * S * (S + 1) / 2 + C * S ** 3 / 6 + n_sym * C * (T * (S * U + S * S) + (T - 1) * S * U)
    return {"bytes": float(n_sc * (8 * B * U + n_sym * (8 * U + 8 * B + 4))), "flops": 8.0 * n_sc * cm}


# -- the same results in 64 bits ---------------------------------------------------

def _inverse(M):
    """Inverses of Hermitian positive definite matrices [..., N, N]
    (Gauss-Jordan elimination; no pivoting is needed)."""
    N = M.shape[-1]
    A = M.clone()
    for k in range(N):
        p = 1.0 / A[..., k, k].clone()
        row = A[..., k, :] * p[..., None]
        row[..., k] = p
        col = A[..., :, k].clone()
        col[..., k] = 0
        A[..., :, k] = 0
        A -= col[..., :, None] * row[..., None, :]
        A[..., k, :] = row
    return A


def _mv(M, v):
    return (M * v[..., None, :]).sum(-1)


def _herm(M):
    return M.conj().transpose(-1, -2).resolve_conj().contiguous()


def _slice(s, qam):
    L, kappa = inputs.qam_side(qam), inputs.qam_kappa(qam)
    i = torch.clamp(torch.floor((kappa * s.real + L) / 2), 0, L - 1)
    q = torch.clamp(torch.floor((kappa * s.imag + L) / 2), 0, L - 1)
    return (i + L * q).to(torch.uint8)


def _admm(H, y, C, T, N0, reg, qam):
    """Algorithm 1 on [n, B, U] and [n, n_sym, B] complex128."""
    n, B, U = H.shape
    S, n_sym = B // C, y.shape[1]
    Hc = H.reshape(n, C, S, U)
    Hh = _herm(Hc)
    Binv = _inverse(torch.matmul(Hh, Hc) + RHO * torch.eye(U, dtype=H.dtype, device=H.device))
    yc = y.reshape(n, n_sym, C, S).permute(0, 2, 3, 1).contiguous()
    yreg = torch.matmul(Binv, torch.matmul(Hh, yc))          # [n, C, U, n_sym]
    nu = N0 / RHO if reg == "mmse" else 0.0
    r = (inputs.qam_side(qam) - 1) / inputs.qam_kappa(qam)

    def prox(w):
        if reg == "box":
            v = w / C
            return torch.complex(v.real.clamp(-r, r), v.imag.clamp(-r, r))
        return w / (nu + C)

    z, lam = yreg, torch.zeros_like(yreg)
    s = prox(z.sum(1, keepdim=True))
    for _ in range(T - 1):
        lam = lam + (z - s)
        z = yreg + RHO * torch.matmul(Binv, (s - lam).contiguous())
        s = prox((z + lam).sum(1, keepdim=True))
    return s[:, 0].transpose(1, 2).contiguous()


def _cg(H, y, T, N0, reg):
    """Algorithm 2 (whose sums over clusters run over all rows of H)."""
    mu = N0 if reg == "mmse" else 0.0
    Hh = _herm(H)
    r = torch.matmul(Hh, y.transpose(1, 2).contiguous())      # [n, U, n_sym]
    p, x = r.clone(), torch.zeros_like(r)
    rr = (r.abs() ** 2).sum(1, keepdim=True)
    for _ in range(T):
        e = mu * p + torch.matmul(Hh, torch.matmul(H, p))
        a = rr / (p.conj() * e).real.sum(1, keepdim=True)
        x = x + a * p
        r = r - a * e
        new = (r.abs() ** 2).sum(1, keepdim=True)
        p = r + (new / rr) * p
        rr = new
    return x.transpose(1, 2).contiguous()


def _precode(Hu, s, C, T, eps, power, P):
    """Algorithm 3 (S <= U) on the uplink block Hu [n, B, U] and s [n, n_sym, U]."""
    n, B, U = Hu.shape
    S, n_sym = B // C, s.shape[1]
    Hc = Hu.reshape(n, C, S, U).transpose(-1, -2).contiguous()     # downlink blocks, U x S
    Hh = _herm(Hc)
    G = torch.matmul(Hh, Hc)
    eye = torch.eye(S, dtype=Hu.dtype, device=Hu.device)
    A = _inverse(G + eye / RHO)
    target = s.transpose(1, 2).contiguous()[:, None]                # [n, 1, U, n_sym]

    def apply(v):
        h = torch.matmul(Hh, v.contiguous())
        x = torch.matmul(A, h)
        if power != "per_cluster":
            return x
        # budgeted step: the root tau of ||(G + tau I)^{-1} h||^2 = P where the
        # unconstrained step exceeds the budget (Newton on 1 / ||x||)
        cols = []
        for j in range(n_sym):
            hj, xj = h[..., j].contiguous(), x[..., j].contiguous()
            tau = torch.full(xj.shape[:-1], 1.0 / RHO, dtype=torch.float64, device=xj.device)
            over = (xj.abs() ** 2).sum(-1) > P
            for _ in range(14):
                inv = _inverse(G + tau[..., None, None] * eye)
                xn = _mv(inv, hj)
                e = (xn.abs() ** 2).sum(-1)
                q = (xn.conj() * _mv(inv, xn)).real.sum(-1)
                step = e * (torch.sqrt(e) - math.sqrt(P)) / (math.sqrt(P) * q)
                tau = torch.where(over, tau + step, tau)
            xn = _mv(_inverse(G + tau[..., None, None] * eye), hj)
            cols.append(torch.where(over[..., None], xn, xj))
        return torch.stack(cols, -1)

    z = (max(U / B, 1.0 / C) * target).expand(n, C, U, n_sym)
    lam = torch.zeros_like(z)
    x = apply(z)
    for _ in range(T - 1):
        m = torch.matmul(Hc, x.contiguous())
        w = m - lam
        d = target - w.sum(1, keepdim=True)
        f = 1.0
        if eps > 0.0:
            f = torch.clamp(1.0 - eps / torch.sqrt((d.abs() ** 2).sum(2, keepdim=True)), min=0.0)
        z = w + f * d / C
        lam = lam - (m - z)
        x = apply(z + lam)
    beta = torch.ones((n, n_sym), dtype=torch.float64, device=Hu.device)
    if power == "common_gain":
        e = (x.abs() ** 2).sum(2)                                   # [n, C, n_sym]
        beta = torch.clamp(torch.sqrt(P / e).amin(1), max=1.0)
    x = x * beta[:, None, None, :]
    return x.permute(0, 3, 1, 2).reshape(n, n_sym, B).contiguous(), beta


def _f32(v):
    """The call takes N0 (and budgets) in single precision."""
    return float(torch.tensor(v, dtype=torch.float32))


def _chunks(n_sc, entries):
    """Slices of the subcarriers of at most about 2^26 matrix entries."""
    step = max(1, (1 << 26) // max(1, entries))
    return [slice(i, min(n_sc, i + step)) for i in range(0, n_sc, step)]


def _exact_uplink(op, H, y, C, T, N0, reg, qam):
    n_sc, B, U = H.shape
    N0 = _f32(N0)
    parts = []
    for k in _chunks(n_sc, C * U * U + 2 * B * U):
        Hk, yk = H[k].to(torch.complex128), y[k].to(torch.complex128)
        parts.append(_cg(Hk, yk, T, N0, reg) if op == "cg" else _admm(Hk, yk, C, T, N0, reg, qam))
    return torch.cat(parts)


def exact(case, seed):
    st = prepare(case, seed)
    op, T = case["op"], case["T"]
    if op == "batch":
        outs = []
        for f in st["frames"]:
            s = _exact_uplink("admm", f["H"], f["y"], f["C"], T, f["N0"], "mmse", f["qam"])
            outs.append((s, _slice(s, f["qam"])))
        return outs
    C = case["C"]
    if op == "precode":
        H = st["H"] if case["layout"] == "uplink" else st["H"].transpose(1, 2)
        n_sc, B, U = H.shape
        parts = []
        for k in _chunks(n_sc, 2 * B * U + C * (B // C) ** 2):
            parts.append(_precode(H[k].to(torch.complex128).contiguous(), st["s"][k].to(torch.complex128), C, T,
                                  _f32(case["eps"]), case["power"], _f32(case["P"])))
        return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
    s = _exact_uplink("cg" if op == "cg" else "admm", st["H"], st["y"], C, T, st["N0"], case["reg"], case["qam"])
    if op == "resident" and case["prec"] == "h16":
        return s
    return s, _slice(s, case["qam"])
