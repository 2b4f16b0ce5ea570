"""The evaluation work of this library as cases to time: what a parameter-estimation program has it do,
through its public entry points, over the range of sizes, types and options in use.

A case is a dict of plain values.  ``prepare`` makes what such a program holds before the call (the handle on
its intrinsic points and the extrinsic samples, or the host arrays of the precompute), ``run`` makes one pass,
``exact`` gives the same outputs from plain torch in 64 bits.  The synthetic points follow the workloads of the
benchmark: detectors at published sites, random mode overlaps scaled to a network SNR, a Gaussian-windowed
signal plus noise of the same covariance.
"""
import math

import numpy as np
import torch

from paper_2210_07912_amd import ile

C_LIGHT = 299792458.0
F_S = 4096.0
D_REF, D_MIN, D_MAX = 100.0, 10.0, 1000.0

# vertex (m, Earth-fixed), x arm, y arm of the H1, L1 and V1 sites
SITES = (
    ((-2.16141492636e06, -3.83469517889e06, 4.60035022664e06), (-0.22389266154, 0.79983062746, 0.55690487831),
     (-0.91397818574, 0.02609403989, -0.40492342125)),
    ((-7.42760447238e04, -5.49628371971e06, 3.22425701744e06), (-0.95457412153, -0.14158077340, -0.26218911324),
     (0.29774156894, -0.48791033647, -0.82054461286)),
    ((4.54637409900e06, 8.42989697626e05, 4.37857696241e06), (-0.70045821479, 0.20848948619, 0.68256166277),
     (-0.05379255368, -0.96908180549, 0.24080451708)),
)
MODES = {
    2: [(2, 2), (2, -2)],
    5: [(2, m) for m in (2, 1, 0, -1, -2)],
    9: [(2, m) for m in (2, 1, 0, -1, -2)] + [(3, 3), (3, -3), (3, 2), (3, -2)],
    12: [(l, m) for l in (2, 3) for m in range(l, -l - 1, -1)],
    21: [(l, m) for l in (2, 3, 4) for m in range(l, -l - 1, -1)],
}


# ---- cases ------------------------------------------------------------------
def listed():
    return [
        # one small call on one point, as an optimiser or a test of a proposal makes it: launches and latency
        dict(name="lnl_small", kind="lnl", points=1, K=3, M=5, n_t=100, n=4096, snr=12.0),
        # the two-detector quadrupole point in full precision at the size of one workflow job
        dict(name="lnl_fp64_plain", kind="lnl", fp64=True, points=1, K=2, M=2, n_t=410, n=10007, snr=15.0),
        # the FP64 replay of samples that a FP32 run weighted, at the three-detector l = 2..4 shape
        dict(name="lnl_fp64_replay", kind="lnl", fp64=True, points=1, K=3, M=21, n_t=820, n=200000, snr=25.0),
        # one intrinsic point, three detectors, l = 2..4, a long window: the large single call
        dict(name="lnl_single", kind="lnl", points=1, K=3, M=21, n_t=820, n=1000000, snr=25.0),
        # many heterogeneous intrinsic points in one call, as a grid of them is marginalized
        dict(name="lnl_batched", kind="lnl", points=48, K=0, M=0, n_t=0, n=0, snr=0.0),
        # the distance-marginalized likelihood of a call's points (production setting of the integrator)
        dict(name="lnl_dmarg", kind="lnl", dmarg=True, points=4, K=3, M=9, n_t=500, n=50000, snr=20.0),
        # the gradient of one point's samples (gradient-informed proposals), FP32 with the FP64 refinement
        dict(name="grad_single", kind="grad", points=1, K=3, M=21, n_t=820, n=100000, snr=25.0, tau=True),
        # forward and backward through autograd on a few samples of several points, as an ascent steps
        dict(name="grad_small", kind="grad", points=8, K=3, M=5, n_t=200, n=64, snr=15.0, forward=True),
        # the gradient in full precision
        dict(name="grad_fp64", kind="grad", fp64=True, points=1, K=3, M=9, n_t=410, n=20000, snr=20.0),
        # a round of an adaptive run from the tables of an earlier one: draw, evaluate, reduce, refit the histograms
        dict(name="run_adaptive", kind="run", points=8, K=3, M=21, n_t=820, n=100000, snr=10.0, rounds=1, mask=0x3F,
             tables=True),
        # the same with the Gaussian-mixture proposal and correlated pairs
        dict(name="run_mixture", kind="run", points=8, K=2, M=5, n_t=400, n=50000, snr=6.0, rounds=1, mask=0x3F,
             tables=True, gmm=3, graph=True),
        # the overlaps of one point from frequency-domain inputs on the host: 8 s at 4096 Hz
        dict(name="precompute", kind="quv", K=3, M=21, N=32768, n_rows=999),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; none costs more than the largest listed ones."""
    kind = rng.choice(("lnl", "lnl", "lnl64", "dmarg", "grad", "grad", "grad64", "run", "quv"))
    K, M = rng.choice((1, 2, 2, 3, 3, 3)), rng.choice((2, 5, 9, 12, 21))
    n_t = _log_int(rng, 100, 820)
    snr = rng.uniform(8.0, 40.0)
    points = rng.choice((1, 1, 2, 5, 16))
    if kind == "lnl":
        return dict(kind="lnl", points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 1000, 1000000 // points), snr=snr,
                    V=rng.random() < 0.2, graph=rng.random() < 0.3)
    if kind == "lnl64":
        return dict(kind="lnl", fp64=True, points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 1000, 150000 // points),
                    snr=snr, V=rng.random() < 0.2)
    if kind == "dmarg":
        return dict(kind="lnl", dmarg=True, points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 1000, 100000 // points),
                    snr=snr)
    if kind == "grad":
        return dict(kind="grad", points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 64, 100000 // points), snr=snr,
                    tau=rng.random() < 0.5, forward=rng.random() < 0.5)
    if kind == "grad64":
        return dict(kind="grad", fp64=True, points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 64, 10000 // points),
                    snr=snr, tau=rng.random() < 0.5)
    if kind == "run":
        # several rounds from the prior, or one that refits the proposal after it
        mask = rng.choice((0, 0x3F, 0x1F))
        gmm = rng.choice((0, 0, 2)) if mask else 0
        return dict(kind="run", points=points, K=K, M=M, n_t=n_t, n=_log_int(rng, 4000, 400000 // points),
                    snr=6.0 if gmm else rng.uniform(6.0, 12.0), rounds=1 if mask else rng.randint(1, 4), mask=mask,
                    gmm=gmm, tables=bool(mask), graph=rng.random() < 0.5)
    return dict(kind="quv", K=K, M=M, N=rng.choice((4096, 8192, 9600, 16384, 32768)), n_rows=rng.randint(200, 1100))


# ---- plain 64-bit reference --------------------------------------------------
def _harmonics(modes, iota, phi):
    """Spin-weight -2 harmonics [M, n] complex128 by the Wigner-d sum."""
    c, s = torch.cos(0.5 * iota), torch.sin(0.5 * iota)
    f = math.factorial
    out = []
    for l, m in modes:
        d = torch.zeros_like(iota)
        norm = math.sqrt((2 * l + 1) / (4 * math.pi)) * math.sqrt(f(l + m) * f(l - m) * f(l + 2) * f(l - 2))
        for k in range(max(0, m - 2), min(l + m, l - 2) + 1):
            den = f(l + m - k) * f(l - 2 - k) * f(k) * f(k + 2 - m)
            d = d + (-1.0) ** k * norm / den * c ** (2 * l + m - 2 - 2 * k) * s ** (2 * k + 2 - m)
        out.append(torch.polar(torch.ones_like(phi), m * phi) * d)
    return torch.stack(out)


def _geometry(p, th):
    """Antenna patterns F [K, n] complex and delays dt [K, n] (s) at th [7, n]."""
    h = th[0] - p["gmst"]
    ch, sh, cd, sd = torch.cos(h), torch.sin(h), torch.cos(th[1]), torch.sin(th[1])
    cp, sp = torch.cos(th[2]), torch.sin(th[2])
    e1 = torch.stack([-sh, ch, torch.zeros_like(h)])
    e2 = torch.stack([sd * ch, sd * sh, -cd])
    X, Y = cp * e1 + sp * e2, cp * e2 - sp * e1
    F, dt = [], []
    for k in range(len(p["det_pos"])):
        D = torch.as_tensor(p["det_resp"][k], device=th.device)
        r = torch.as_tensor(p["det_pos"][k], device=th.device) / C_LIGHT
        F.append(torch.complex((X * (D @ X)).sum(0) - (Y * (D @ Y)).sum(0), 2.0 * (X * (D @ Y)).sum(0)))
        dt.append(-(r[0] * cd * ch + r[1] * cd * sh + r[2] * sd))
    return torch.stack(F), torch.stack(dt)


def _window(p, th, unit_distance=False):
    """Data terms A [n, n_t] of the window and the quadratic term B [n] at th [7, n] (float64, differentiable)."""
    dev = th.device
    K, M, n_t, pad = len(p["det_pos"]), len(p["ell"]), p["n_t"], p["pad"]
    F, dt = _geometry(p, th)
    Y = _harmonics(list(zip(p["ell"].tolist(), p["em"].tolist())), th[3], th[4])
    x = torch.ones_like(th[5]) if unit_distance else D_REF / th[5]
    A = torch.zeros((th.shape[1], n_t), dtype=torch.float64, device=dev)
    B = torch.zeros_like(th[0])
    j = torch.arange(n_t, device=dev)
    for k in range(K):
        a = x * F[k] * Y
        U = torch.as_tensor(p["U"][k], device=dev)
        B = B + 0.25 * (a.conj() * (U @ a)).sum(0).real
        if p["V"] is not None:
            B = B + 0.25 * (a * (torch.as_tensor(p["V"][k], device=dev) @ a)).sum(0).real
        Q = torch.as_tensor(p["Q"][k], device=dev)
        z = a.real.T @ Q.real.T + a.imag.T @ Q.imag.T  # Re sum_m conj(a_m) Q[r, m], all rows
        s = (th[6] + dt[k]) * F_S
        n = torch.floor(s.detach())
        mu = s - n
        w = (0.5 * (-mu ** 3 + 2 * mu ** 2 - mu), 0.5 * (3 * mu ** 3 - 5 * mu ** 2 + 2),
             0.5 * (-3 * mu ** 3 + 4 * mu ** 2 + mu), 0.5 * (mu ** 3 - mu ** 2))
        row = pad + n.long()[:, None] + j[None, :]
        for q in range(4):
            A = A + w[q][:, None] * torch.gather(z, 1, row + q)
    return A, B


def _lnl_exact(p, th, dmarg):
    A, B = _window(p, th, dmarg)
    if not dmarg:
        return torch.logsumexp(A, 1) - B - math.log(p["n_t"])
    # over t = ln(D_ref / D) with p(D) dD = c e^{-3t} dt: composite Gauss-Legendre on the part of the prior's
    # range where the envelope of the integrand is within 60 nats of its peak
    lo, hi = math.log(D_REF / D_MAX), math.log(D_REF / D_MIN)
    c = 3.0 * D_REF ** 3 / (D_MAX ** 3 - D_MIN ** 3)
    am = A.max(1).values
    t = torch.linspace(lo, hi, 2001, dtype=torch.float64, device=th.device)
    env = am[:, None] * t.exp() - B[:, None] * (2 * t).exp() - 3 * t
    near = env >= env.max(1, keepdim=True).values - 60.0
    first = near.to(torch.int8).argmax(1)
    last = 2000 - near.flip(1).to(torch.int8).argmax(1)
    ta, tb = t[(first - 1).clamp(min=0)], t[(last + 1).clamp(max=2000)]
    gx, gw = np.polynomial.legendre.leggauss(12)
    panels = 10
    total = torch.full_like(am, -math.inf)
    width = (tb - ta) / panels
    for i in range(panels):
        for g, w in zip(gx, gw):
            tq = ta + width * (i + 0.5 + 0.5 * g)
            x = tq.exp()
            term = torch.logsumexp(x[:, None] * A, 1) - x * x * B - 3 * tq + torch.log(0.5 * width * w * c)
            total = torch.logaddexp(total, term)
    return total - math.log(p["n_t"])


def _chunks(items, per):
    for point, off, cnt in items:
        for o in range(off, off + cnt, per):
            yield point, o, min(o + per, off + cnt)


# ---- inputs -----------------------------------------------------------------
def _shape(case, i):
    """Shape of point i of a case: the given one, or (zeros) drawn per point as in the batched workload."""
    if case["n"]:
        return case["K"], case["M"], case["n_t"], case["n"], case["snr"]
    s = np.random.default_rng([11, i])  # the shapes are the case's, only the values come from the seed
    return (int(s.choice((2, 3))), int(s.choice((2, 5, 9, 21))), int(s.integers(200, 801)),
            int(round(10 ** s.uniform(5, 6))), float(s.uniform(8, 40)))


def _point(g, K, M, n_t, snr, V=False):
    pos = np.array([SITES[k][0] for k in range(K)])
    resp = np.array([0.5 * (np.outer(x, x) - np.outer(y, y)) for _, x, y in SITES[:K]])
    pad = int(math.ceil(F_S * max(np.linalg.norm(r) for r in pos) / C_LIGHT + 0.5))
    L = n_t + 2 * pad + 3
    ell, em = (np.array(v, dtype=np.int32) for v in zip(*MODES[M]))
    u = g.random(7)
    th = np.array([2 * math.pi * u[0], math.asin(2 * u[1] - 1), math.pi * u[2], math.acos(2 * u[3] - 1),
                   2 * math.pi * u[4], 100.0 + 500.0 * u[5], 0.0])
    p = dict(det_pos=pos, det_resp=resp, ell=ell, em=em, n_t=n_t, pad=pad, f_s=F_S, d_ref=D_REF,
             gmst=2 * math.pi * u[6], theta_inj=th, V=None)
    U = np.empty((K, M, M), dtype=np.complex128)
    for k in range(K):
        G = g.standard_normal((M, M + 2)) + 1j * g.standard_normal((M, M + 2))
        U[k] = (0.5 + 0.5 * g.random()) * (G @ G.conj().T) / (2.0 * (M + 2))
        U[k] = 0.5 * (U[k] + U[k].conj().T)
    t = torch.tensor(th)[:, None]
    F, dt = _geometry(p, t)
    a = (D_REF / th[5] * F[:, None, :] * _harmonics(MODES[M], t[3], t[4])[None]).numpy()[:, :, 0]  # [K, M]
    rho2 = 0.5 * sum((a[k].conj() @ U[k] @ a[k]).real for k in range(K))
    U *= snr ** 2 / rho2
    r = (np.arange(L) - (pad + 1 + n_t // 2)) / F_S
    Q = np.empty((K, L, M), dtype=np.complex128)
    for k in range(K):
        tau = r - float(dt[k, 0])
        kern = np.exp(-tau ** 2 / (2 * 3e-3 ** 2) - 2j * math.pi * 100.0 * tau)
        chol = np.linalg.cholesky(U[k] + 1e-12 * np.trace(U[k]).real / M * np.eye(M))
        xi = (g.standard_normal((L, M)) + 1j * g.standard_normal((L, M))) / math.sqrt(2)
        Q[k] = kern[:, None] * (0.5 * (U[k] @ a[k]))[None, :] + xi @ chol.T
    p.update(Q=Q, U=U)
    if V:
        S = 0.02 * np.abs(U).max() * (g.standard_normal((K, M, M)) + 1j * g.standard_normal((K, M, M)))
        p["V"] = S + S.transpose(0, 2, 1)
    return p


def _points(case, seed):
    g = np.random.default_rng([int(seed), 1])
    pts, items, off = [], [], 0
    for i in range(case["points"]):
        K, M, n_t, n, snr = _shape(case, i)
        pts.append(_point(g, K, M, n_t, snr, case.get("V", False)))
        items.append((i, off, n))
        off += n
    return pts, items


def _theta(pts, items, seed, tau):
    """Half prior draws, half scattered around each point's injection, in no order; FP32 values, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    n = sum(c for _, _, c in items)
    u = torch.rand((7, n), generator=g, device="cuda", dtype=torch.float64)
    z = torch.randn((7, n), generator=g, device="cuda", dtype=torch.float64)
    near = torch.rand(n, generator=g, device="cuda") < 0.5
    th = torch.stack([2 * math.pi * u[0], torch.asin(2 * u[1] - 1), math.pi * u[2], torch.acos(2 * u[3] - 1),
                      2 * math.pi * u[4], (D_MIN ** 3 + u[5] * (D_MAX ** 3 - D_MIN ** 3)) ** (1.0 / 3.0),
                      (u[6] - 0.5) * (1.0 / F_S if tau else 0.0)])
    for point, o, c in items:
        t0 = pts[point]["theta_inj"]
        for d, sc in enumerate((0.02, 0.02, 0.05, 0.1, 0.1, 0.1 * t0[5])):
            v = t0[d] + sc * z[d, o:o + c]
            th[d, o:o + c] = torch.where(near[o:o + c], v.abs() + 1.0 if d == 5 else v, th[d, o:o + c])
    return th.to(torch.float32)


def _fd(case, seed):
    """Host arrays of the precompute: coloured PSDs, power-law modes with smooth phases, Gaussian data."""
    K, M, N = case["K"], case["M"], case["N"]
    df, f_low = F_S / N, 20.0
    g = np.random.default_rng([int(seed), 2])
    f = np.fft.fftfreq(N, d=1.0 / (N * df))
    fs = np.maximum(np.abs(f), df)
    psd = g.uniform(0.5, 2.0, (K, 1)) * (1.0 + (40.0 / fs) ** 4 + (fs / 300.0) ** 2)
    band = (np.abs(f) > f_low) & (np.abs(f) < 0.4 * N * df)
    c = g.normal(size=(M, 4))
    phase = (c[:, :1] + c[:, 1:2] * fs / 100.0 + c[:, 2:3] * np.sign(f) * (fs / 100.0) ** 2
             + c[:, 3:] * (100.0 / fs))
    modes = np.where(band, g.uniform(0.5, 2.0, (M, 1)) * (fs / 100.0) ** (-7.0 / 6.0) * np.exp(1j * phase), 0.0)
    data = np.sqrt(psd / (4.0 * df)) * (g.normal(size=(K, N)) + 1j * g.normal(size=(K, N)))
    return dict(data=data, psd=psd, modes=modes, df=df, f_low=f_low, row0=N // 3, n_rows=case["n_rows"])


def _tables(p, width=0.06, floor=0.1):
    """Histogram tables [7, 101] of an earlier round: a bump about the injection over a uniform floor, each in the
    parameter's prior-CDF coordinate."""
    t = p["theta_inj"]
    u0 = (t[0] / (2 * math.pi), (math.sin(t[1]) + 1) / 2, t[2] / math.pi, (1 - math.cos(t[3])) / 2,
          t[4] / (2 * math.pi), (t[5] ** 3 - D_MIN ** 3) / (D_MAX ** 3 - D_MIN ** 3), 0.5)
    u = (np.arange(100) + 0.5) / 100
    h = np.array([np.exp(-0.5 * ((u - c) / width) ** 2) for c in u0])
    h = floor + (1 - floor) * 100 * h / h.sum(axis=1, keepdims=True)
    cdf = np.concatenate([np.zeros((7, 1)), np.cumsum(h, axis=1)], axis=1)
    return cdf / cdf[:, -1:]


def prepare(case, seed):
    if case["kind"] == "quv":
        return dict(case=case, fd=_fd(case, seed))
    pts, items = _points(case, seed)
    tau = bool(case.get("tau"))
    h = ile.RiftILE(pts, precision="fp64" if case.get("fp64") else "fp32", d_min=D_MIN, d_max=D_MAX,
                    tau_width=1.0 / F_S if tau else 0.0)
    if case.get("graph"):
        h.set_graph(True)
    if case.get("dmarg"):
        h.set_distance_marginalization(True)
    s = dict(case=case, h=h, items=items, seed=int(seed))
    if case.get("tables"):
        s["tables"] = [_tables(p) for p in pts]
    if case["kind"] != "run":
        s["theta"] = _theta(pts, items, seed, tau).to(h.dtype)
    if case["kind"] == "grad":
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed) + 1)
        s["g"] = torch.rand(s["theta"].shape[1], generator=g, device="cuda", dtype=torch.float32).to(h.dtype) + 0.5
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "quv":
        return dict(zip("QUV", ile.precompute(**s["fd"])))
    h = s["h"]
    if case["kind"] == "lnl":
        return h.lnL(s["theta"], s["items"])
    if case["kind"] == "grad":
        if not case.get("forward"):
            return h.backward(s["theta"], s["g"], s["items"])
        th = s["theta"].detach().requires_grad_(True)
        l = ile.lnL_autograd(h, th, s["items"])
        l.backward(s["g"])
        return dict(lnL=l.detach(), grad=th.grad)
    # the pooled estimate of every point, every sample with its weight (the sample-size ratios of the result are
    # functions of those weights) and the proposal that the next round draws from, at the run's precision
    mask, gmm = case["mask"], case.get("gmm", 0)
    for i, cdf in enumerate(s.get("tables", ())):
        h.set_proposal(i, cdf, mask)
    res, th, lw = h.marginalize(seed=s["seed"], n_per_point=case["n"], n_rounds=case["rounds"], adapt_mask=mask,
                                reset=not case.get("tables"), return_samples=True, gmm_components=gmm,
                                gmm_pairs=((2, 4), (3, 5)) if gmm and mask == 0x3F else ())
    out = dict(lnL_marg=np.array([r["lnL_marg"] for r in res], dtype=np.float32),
               n=np.array([r["n"] for r in res]), theta=th, lnw=lw)
    if mask and gmm:
        out["proposal"] = [np.stack([g[k] for k in ("w", "mu", "sd")]).astype(np.float32)
                           for g in map(h.get_gmm, range(case["points"]))]
    elif mask:
        out["proposal"] = np.stack([h.get_proposal(i)[0] for i in range(case["points"])]).astype(np.float32)
    return out


def exact(case, seed):
    if case["kind"] == "run":
        return None  # the draws are the library's own generator's
    if case["kind"] == "quv":
        fd = _fd(case, seed)
        d, S, h = (torch.as_tensor(fd[k], device="cuda") for k in ("data", "psd", "modes"))
        N = case["N"]
        f = torch.fft.fftfreq(N, d=1.0 / (N * fd["df"]), device="cuda", dtype=torch.float64)
        w = torch.where(f.abs() > fd["f_low"], 2.0 * fd["df"] / S, torch.zeros_like(S))
        X = torch.fft.ifft(w[:, None] * h.conj()[None] * d[:, None], dim=2) * N
        rows = (fd["row0"] + torch.arange(case["n_rows"], device="cuda")) % N
        neg = h.roll(-1, 1).flip(1)  # h(-f)
        U = torch.stack([(h.conj() * w[k]) @ h.T for k in range(case["K"])])
        V = torch.stack([(neg * w[k]) @ h.T for k in range(case["K"])])
        return dict(Q=X[:, :, rows].transpose(1, 2).contiguous(), U=U, V=V)
    pts, items = _points(case, seed)
    th = _theta(pts, items, seed, bool(case.get("tau"))).double()
    if case["kind"] == "lnl":
        out = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
        for point, a, b in _chunks(items, 2000 if case.get("dmarg") else 20000):
            out[a:b] = _lnl_exact(pts[point], th[:, a:b], bool(case.get("dmarg")))
        return out
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 1)
    up = (torch.rand(th.shape[1], generator=g, device="cuda", dtype=torch.float32)
          .to(torch.float64 if case.get("fp64") else torch.float32) + 0.5).double()
    lnl, grad = torch.empty_like(th[0]), torch.empty_like(th)
    for point, a, b in _chunks(items, 4000):
        t = th[:, a:b].clone().requires_grad_(True)
        v = _lnl_exact(pts[point], t, False)
        (grad[:, a:b],) = torch.autograd.grad(v, t, up[a:b])
        lnl[a:b] = v.detach()
    return dict(lnL=lnl, grad=grad) if case.get("forward") else grad


# ---- what a pass cannot do without -------------------------------------------
def _eval_work(K, M, n_t, n, elem, grad=False, dmarg=False):
    """Flops and bytes of n evaluations on one point: the contraction of the rows the window needs, the 4-tap
    interpolation, the log-sum-exp, the quadratic term and the coefficients; samples in, results out, Q once."""
    f = K * (n_t + 3) * 4 * M + 8 * K * n_t + 4 * n_t + 4 * K * M * M + 6 * K * M + 200
    if grad:  # transposed contraction and interpolation, derivative interpolation, softmax, U a, chain rule
        f += K * (n_t + 3) * 4 * M + 8 * K * (n_t + 3) + 8 * K * n_t + 2 * n_t + 8 * K * M * M + 40 * K * M
    if dmarg:  # the window's sum at each node of the distance rule
        f += 24 * 3 * n_t
    pad = int(math.ceil(F_S * max(np.linalg.norm(SITES[k][0]) for k in range(K)) / C_LIGHT + 0.5))
    q = K * (n_t + 2 * pad + 3) * 2 * M * elem
    return float(n) * f, n * elem * (7 + 1 + (8 if grad else 0)) + q


def work(case):
    if case["kind"] == "quv":
        K, M, N, r = case["K"], case["M"], case["N"], case["n_rows"]
        return dict(flops=K * M * (10 * N + 5 * N * math.log2(N)) + 16.0 * K * M * M * N,
                    bytes=16 * (K + M) * N + 8 * K * N + 16 * K * r * M + 32 * K * M * M)
    flops = nbytes = 0.0
    for i in range(case["points"]):
        K, M, n_t, n, _ = _shape(case, i)
        f, b = _eval_work(K, M, n_t, n, 8 if case.get("fp64") else 4, case["kind"] == "grad", bool(case.get("dmarg")))
        flops, nbytes = flops + f, nbytes + b
    r = case.get("rounds", 1)
    return dict(flops=flops * r, bytes=nbytes * r)
