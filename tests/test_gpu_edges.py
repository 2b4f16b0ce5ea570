"""GPU parity at the edges of what the sorted matrix-core forms take: window
values that overflow, results that may not depend on a sample's neighbours,
calls of very many delay bins, grids of the precompute with long sums."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import _handle, _say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ile():
    from paper_2210_07912_amd import ile as m
    m.lib()
    return m


@pytest.mark.parametrize("prec,big", [("fp32", 3e38), ("fp64", 1.7e308)])
def test_overflow_far_below_the_peak(ile, orc, prec, big):
    """A row of Q that overflows the near samples' window values (one detector
    at the geocentre, whose interpolation weights are 0, 1, 0, 0: -inf and NaN,
    no +inf), 1900 nats below their peak: ln L_t and gradient of those samples
    are NaN in every form, also where the sorted forms leave blocks without
    mass out; the others, 20 times as far away, do not overflow and agree with
    the oracle."""
    n_t, n = 200, 40000
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1700, dets=("H1",), n_modes=2, n_t=n_t, snr=1.0, kernel="none")
    d = dict(synth.make_point(spec))
    d["det_pos"] = np.zeros((1, 3))
    th = synth.mixed_samples(d, 37, 4)[:, :1]
    th[6], th[5] = 0.0, 100.0
    a = np.asarray(orc.coeffs(orc.Point.from_dict(d), th[:, 0])[0])[0]
    th[5] = np.float32(100.0 * np.abs(a).max() / 3.0)  # the largest coefficient is 3
    a *= 3.0 / np.abs(a).max()
    m = int(np.argmax(np.abs(a)))
    L = d["Q"].shape[1]
    row = L - (n_t + 3)  # first row of the window is (L - n_t - 3) / 2 + 1
    row //= 2
    d["U"] = 1e-3 * np.eye(2)[None].astype(complex)
    d["Q"] = np.zeros((1, L, 2), dtype=complex)
    d["Q"][0, row + 9] = 2000.0 * a / (np.abs(a) ** 2).sum()
    bad = row + 151
    part = np.array([a[m].real, a[m].imag])
    q = -0.9 * big * (part / np.abs(part).max())
    d["Q"][0, bad, m] = q[0] + 1j * q[1]
    ths = np.repeat(th, n, axis=1)
    near = np.arange(n) % 2 == 0
    ths[5, ~near] = np.float32(20.0 * th[5, 0])
    ths = ths.astype(np.float32).astype(np.float64)
    far = orc.lnL_t(orc.Point.from_dict(d, complex64=(prec == "fp32")), ths[:, 1:2])[0]
    h = _handle(ile, [d], prec)
    _say(f"overflow far below the peak {prec}: far samples {far}")
    t = torch.tensor(ths)
    out = h.lnL(t).cpu().numpy()
    g, lg = h.backward(t, want_lnL=True)
    small = h.lnL(t[:, :64]).cpu().numpy()
    h.close()
    for v in (small, out, lg.cpu().numpy()):
        assert np.isnan(v[near[:v.size]]).all()
        assert np.abs(v[~near[:v.size]] - far).max() <= 2e-5 * abs(far)  # (FP32: the data term of 100)
    g = g.cpu().numpy()
    assert np.isnan(g[:, near]).all() and np.isfinite(g[:, ~near]).all()


def test_gradient_does_not_depend_on_the_neighbours(ile, orc):
    """Two peaks, the later one higher: within 40 nats of each other for the
    far samples, 60 and more apart for the near ones, so that samples of one
    tile need different blocks.  The peaks are symmetric about a row (one
    detector, at the geocentre), so that the derivative in tau is zero but for
    the rounding of its terms, which shows the order and the references of every
    sum: it and all else of the near samples are the same, bit for bit, alone
    and among the far ones, in any order."""
    n = 96
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1701, dets=("H1",), n_modes=2, n_t=160, snr=1.0, kernel="none")
    d = dict(synth.make_point(spec))
    d["ell"], d["em"] = d["ell"][:1], d["em"][:1]
    d["U"] = 1e-3 * np.ones((1, 1, 1), dtype=complex)
    d["det_pos"] = np.zeros((1, 3))
    th = synth.mixed_samples(d, 38, 4)[:, 3:]
    th[6], th[5] = 0.0, 200.0
    d["Q"] = np.zeros((1, d["Q"].shape[1], 1), dtype=complex)
    a = np.asarray(orc.coeffs(orc.Point.from_dict(d), th[:, 0])[0])[0]
    r = np.arange(d["Q"].shape[1]) - d["Q"].shape[1] // 2
    peaks = 970.0 * np.maximum(0, 1 - ((r + 40) / 20) ** 2) + 1000.0 * np.maximum(0, 1 - ((r - 40) / 20) ** 2)
    d["Q"][0] = (peaks[:, None] * (a / (np.abs(a) ** 2).sum())[None, :])
    ths = np.repeat(th, n, axis=1)
    near = np.arange(n) % 3 != 0
    ths[5, near] = 95.0 - 0.1 * np.arange(near.sum())
    ths[5, ~near] = 200.0 + np.arange((~near).sum())
    h = _handle(ile, [d], "fp32")
    _say("gradient beside other samples")
    g, l = (x.cpu().numpy() for x in h.backward(torch.tensor(ths), want_lnL=True))
    perm = np.random.default_rng(3).permutation(n)
    gp, lp = (x.cpu().numpy() for x in h.backward(torch.tensor(ths[:, perm]), want_lnL=True))
    ga, la = (x.cpu().numpy() for x in h.backward(torch.tensor(ths[:, near]), want_lnL=True))
    h.close()
    assert np.isfinite(g).all() and np.abs(g[6]).max() < 1e-6 and (g[6, near] != 0.0).any()
    assert np.array_equal(g[:, near], ga) and np.array_equal(l[near], la)
    assert np.array_equal(g[:, perm], gp) and np.array_equal(l[perm], lp)


def _row_sum_bound(N):
    """Largest error of Q over its largest value: an FFT's, of log2 N levels
    that round each value once by 2^-53 in quadrature, four times over."""
    return 4.0 * 2.0 ** -53 * np.sqrt(np.log2(N))


@pytest.mark.parametrize("N", [4096, 9600, 32749, 131071, 2 ** 18])
def test_precompute_long_sums(ile, N):
    """Rows of Q against sums in extended precision, on grids with many and
    (32749 and 131071 are prime) no divisors: the error does not grow with the
    number of terms of a row."""
    M, R = 2, 24
    data, psd, modes, f = synth.fd_inputs(90 + N, n_det=1, n_modes=M, N=N, df=0.25, f_low=0.3)
    row0 = N // 3
    Q, _, _ = ile.precompute(data, psd, modes, 0.25, 0.3, row0, R)
    ld = np.longdouble
    w = np.where(np.abs(f) > 0.3, 2.0 * ld(0.25) / psd[0].astype(ld), ld(0))
    i = np.arange(N, dtype=np.int64)
    err = big = 0.0
    for r in range(R):
        ph = 2 * ld("3.14159265358979323846264338327950288") * ((i * (row0 + r)) % N).astype(ld) / ld(N)
        x = (np.cos(ph) + 1j * np.sin(ph)) * w * data[0].astype(np.clongdouble)
        for m in range(M):
            ref = (np.conj(modes[m].astype(np.clongdouble)) * x).sum()
            err, big = max(err, float(abs(Q[0, r, m] - ref))), max(big, float(abs(ref)))
    _say(f"precompute sums N={N}: {err / big:.2e}, bound {_row_sum_bound(N):.2e}")
    assert err <= _row_sum_bound(N) * big


def test_precompute_rows_at_the_ends_of_int64(ile):
    """Rows wrap modulo N from any first row, also the smallest and largest
    64-bit ones (N = 4095, whose divisors are odd)."""
    data, psd, modes, f = synth.fd_inputs(92, n_det=2, n_modes=3, N=4095, df=0.25, f_low=0.3)
    for row0 in (-2 ** 63, -2 ** 63 + 5, 2 ** 63 - 70):
        a = ile.precompute(data, psd, modes, 0.25, 0.3, row0, 65)
        b = ile.precompute(data, psd, modes, 0.25, 0.3, row0 % 4095, 65)
        _say(f"precompute row0 = {row0}")
        assert all(np.array_equal(x, y) for x, y in zip(a, b))


def _wide(key, K=2, n_modes=2, n_t=16, bins_per_det=256):
    """A point whose pad gives bins_per_det delay bins (of 14 rows) per detector."""
    spec = synth.PointSpec(seed=synth.BASE_SEED + key, dets=("H1", "L1", "V1")[:K], n_modes=n_modes, n_t=n_t, snr=1.0,
                           kernel="none")
    d = dict(synth.make_point(spec))
    pad = (14 * bins_per_det - 1) // 2
    g = np.random.default_rng(key)
    L = n_t + 2 * pad + 3
    d["pad"] = pad
    d["Q"] = g.standard_normal((K, L, n_modes)) + 1j * g.standard_normal((K, L, n_modes))
    return d


def test_fp64_items_of_very_many_bins(ile, orc):
    """More delay bins in one FP64 call (4200 items of 65536) than one sort
    takes: evaluated, not refused, as every call of the plain form."""
    d = _wide(1710, n_t=64)
    n, per = 4200, 32
    th = synth.mixed_samples(d, 40, n * per)
    items = [(0, per * i, per) for i in range(n)]
    h = _handle(ile, [d], "fp64")
    _say(f"{n} items of {h.meta[0]}, 65536 bins each")
    out = h.lnL(torch.tensor(th), items).cpu().numpy()
    sub = np.arange(0, n * per, 1311)
    ref = orc.lnL_t(orc.Point.from_dict(d), th[:, sub])
    h.close()
    assert np.all(np.abs(out[sub] - ref) <= 1e-9 * (1 + np.abs(ref)))


def test_fp32_tiles_beyond_one_group(ile, orc):
    """3.4e7 samples in 520 items of 65536 delay bins, most of them alone in
    theirs: more tiles, padded to pairs, than one group holds (2^26); such a
    call is evaluated in several (of some 100 GB of workspace)."""
    d = _wide(1711, n_t=4)
    n, per = 520, 65536
    base = torch.tensor(synth.mixed_samples(d, 41, per, tau_width=2.0 * (d["pad"] / 4096.0 - 0.03)), dtype=torch.float32)
    th = base.cuda().repeat(1, n)
    h = _handle(ile, [d], "fp32", plain=False)
    _say(f"{n} items of {per} samples, 65536 bins each")
    out = h.lnL(th, [(0, per * i, per) for i in range(n)]).reshape(n, per)
    one = h.lnL(base)
    h.close()
    assert torch.isfinite(one).all()
    assert (out == one[None]).all()


def test_workspace_of_many_small_points(ile):
    """The adjoint pads a bin to one tile: 200 items of 2000 samples, 2197 bins
    each, take no more device memory than those tiles do, a quarter more (the
    growth) and half of that again (the rest of the arrays)."""
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1712, dets=("H1", "L1", "V1"), n_modes=21, n_t=16, snr=1.0,
                           kernel="none")
    d = synth.make_point(spec)
    n, per = 200, 2000
    th = torch.tensor(synth.mixed_samples(d, 42, n * per), dtype=torch.float32).cuda()
    h = _handle(ile, [d], "fp32")
    h.lnL(th[:, :64])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    out = torch.empty_like(th)
    g = h.backward(th, items=[(0, per * i, per) for i in range(n)])
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    tiles = n * (per / 16 + per + 4)
    bound = 1.25 * 1.5 * tiles * (2 * 3 * 2 * 22 * 16 * 4)
    _say(f"workspace {used / 1e9:.2f} GB, bound {bound / 1e9:.2f} GB")
    h.close()
    assert torch.isfinite(g).all() and used <= bound + out.numel() * 8


@pytest.mark.parametrize("M,K,n_t", [(1, 1, 16), (2, 3, 16), (3, 2, 17), (5, 3, 15), (12, 3, 47), (15, 1, 64),
                                     (21, 3, 48), (28, 2, 33), (32, 3, 33)])
def test_fp64_sorted_and_plain_forward(ile, orc, M, K, n_t):
    """One FP64 call of 2e8 units of work (K n_t (M + 4) per sample), far above
    the size rule of the sorted form, against the same samples in calls of 1e7,
    far below it.  ln L_t agrees to the rounding of its terms, and not bit for
    bit: both forms have run."""
    rng = np.random.default_rng([94, M, K, n_t])
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1720 + M, dets=("H1", "L1", "V1")[:K], n_modes=2, n_t=n_t, snr=1.0,
                           kernel="none")
    d = dict(synth.make_point(spec))
    lm = [(l, m) for l in range(2, 9) for m in range(-l, l + 1)]
    pick = rng.choice(len(lm), M, replace=False)
    d["ell"] = np.array([lm[i][0] for i in pick], dtype=np.int32)
    d["em"] = np.array([lm[i][1] for i in pick], dtype=np.int32)
    L = d["Q"].shape[1]
    G = rng.standard_normal((K, M, M + 2)) + 1j * rng.standard_normal((K, M, M + 2))
    d["U"] = 100.0 * G @ G.conj().transpose(0, 2, 1) / (M + 2)
    d["Q"] = 30.0 * (rng.standard_normal((K, L, M)) + 1j * rng.standard_normal((K, L, M)))
    unit = K * n_t * (M + 4)
    n, part = int(2e8 / unit) + 1, int(1e7 / unit)
    th = torch.tensor(synth.mixed_samples(d, 43, n))
    h = _handle(ile, [d], "fp64")
    _say(f"fp64 sorted and plain M={M} K={K} n_t={n_t} n={n}")
    out = h.lnL(th).cpu().numpy()
    cut = np.arange(0, n, max(part, n // 4))[:4]
    small = np.concatenate([h.lnL(th[:, a:a + part]).cpu().numpy() for a in cut])
    h.close()
    same = np.concatenate([out[a:a + part] for a in cut])
    assert np.isfinite(out).all() and np.allclose(same, small, rtol=1e-11, atol=1e-9)
    assert (same != small).any()
    cols = rng.choice(n, 40, replace=False)
    ref = orc.lnL_t(orc.Point.from_dict(d), th.numpy()[:, cols])
    assert np.all(np.abs(out[cols] - ref) <= 1e-9 * (1 + np.abs(ref)))


def test_precompute_by_the_fft(ile):
    """A precompute of more products than the pruned transform takes (a prime
    grid, 40000 rows, ten series): the rows come from the FFT, and agree with
    extended-precision sums as closely as those of a call of a few rows, which
    does not take it."""
    N, K, M, R, row0 = 131071, 2, 5, 40000, 100000
    data, psd, modes, f = synth.fd_inputs(93, n_det=K, n_modes=M, N=N, df=0.25, f_low=0.3)
    Q, U, V = ile.precompute(data, psd, modes, 0.25, 0.3, row0, R)
    big = np.abs(Q).max()
    for r in (0, 7001, 31070, R - 8):
        q, u, v = ile.precompute(data, psd, modes, 0.25, 0.3, row0 + r, 8)
        err = np.abs(Q[:, r:r + 8] - q).max() / big
        _say(f"precompute by the FFT, rows {row0 + r}...: {err:.2e}")
        assert 0.0 < err <= 8.0 * _row_sum_bound(N)  # (a prime grid: three transforms of twice the length and more)
        assert np.array_equal(u, U) and np.array_equal(v, V)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_calls_of_many_shapes_on_one_handle(ile, prec):
    """Forward and adjoint calls, of one item and of several, large and small,
    in turn on one handle (graph replay on, in FP32): each gives what it gives
    alone on a handle of its own, the first time and again, whatever the calls
    before it left in the shared workspace."""
    pts = [synth.make_point(synth.PointSpec(seed=synth.BASE_SEED + 1750 + i, dets=("H1", "L1", "V1")[:2 + i],
                                            n_modes=(5, 9)[i], n_t=60, snr=1.0, kernel="none")) for i in range(2)]
    th = torch.tensor(synth.mixed_samples(pts[0], 44, 60000))
    calls = [(60000, [(0, 0, 60000)]), (50000, [(1, 20000, 30000), (0, 0, 20000)]), (500, [(1, 0, 200), (0, 200, 300)]),
             (60000, [(1, 0, 60000)]), (50000, [(0, 20000, 30000), (1, 0, 20000)])]

    def run(h, c, grad):
        n, items = c
        if not grad:
            return [h.lnL(th[:, :n], items).cpu().numpy()]
        return [x.cpu().numpy() for x in h.backward(th[:, :n], items=items, want_lnL=True)]

    alone = {}
    for i, c in enumerate(calls):
        for grad in (False, True):
            h = _handle(ile, pts, prec)
            alone[i, grad] = run(h, c, grad)
            h.close()
    h = _handle(ile, pts, prec)
    h.set_graph(True)
    _say(f"calls of many shapes {prec}")
    for i, grad in [(i, g) for _ in range(3) for g in (False, True) for i in range(len(calls))] + [(1, False), (4, False)]:
        for a, b in zip(run(h, calls[i], grad), alone[i, grad]):
            assert np.array_equal(a, b, equal_nan=True), (i, grad)
    h.close()


def test_gradient_of_partly_refined_units(ile):
    """One delay bin, of which every third sample's mass lies in one block and
    the others' in all ten: work units of 64 slots with 0 to 22 samples to
    refine, around the tiles of 16 they are gathered in.  Every sample gets what
    it gets alone, refined or not."""
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1702, dets=("H1",), n_modes=2, n_t=160, snr=1.0, kernel="none")
    d = dict(synth.make_point(spec))
    d["det_pos"] = np.zeros((1, 3))
    th = synth.mixed_samples(d, 45, 200)
    th[6] = 0.0
    th[5] = np.where(np.arange(200) % 3 == 0, 20.0, 4000.0) + 0.25 * np.arange(200)
    r = np.arange(d["Q"].shape[1]) - d["Q"].shape[1] // 2
    g = np.random.default_rng(46)
    d["Q"] = 30.0 * (g.standard_normal((1, r.size, 2)) + 1j * g.standard_normal((1, r.size, 2)))
    d["Q"] *= (0.01 + 30.0 * np.exp(-0.5 * ((r - 5) / 3.0) ** 2))[None, :, None]
    t = torch.tensor(th.astype(np.float32))
    h = _handle(ile, [d], "fp32")
    alone = np.concatenate([h.backward(t[:, i:i + 1]).cpu().numpy() for i in range(200)], axis=1)
    h.set_grad_refine(False)
    changed = (h.backward(t).cpu().numpy() != alone).any(axis=0)
    h.set_grad_refine(True)
    _say(f"partly refined units: {changed[::3].sum()} of {changed[::3].size} near samples refined")
    assert changed[::3].mean() > 0.5
    for n in (1, 3, 46, 48, 49, 64, 65, 97, 128, 145, 200):
        assert np.array_equal(h.backward(t[:, :n]).cpu().numpy(), alone[:, :n]), n
    h.close()


@pytest.mark.parametrize("K,M,n_t,n,sorted_form", [
    (3, 21, 800, 1020, False), (2, 21, 800, 1100, False), (3, 9, 400, 3900, False), (3, 5, 569, 5012, False),
    (2, 2, 410, 10007, True), (3, 21, 800, 20000, True)])
def test_fp64_form_by_size(ile, K, M, n_t, n, sorted_form):
    """Which form an FP64 forward call takes: at long windows and many modes
    the sorted form pays later than its units of work say (1000 samples at K =
    3, M = 21, n_t = 800 are 2.7 times as fast in the plain form).  Small parts
    of the call, plain by their size, agree with it bit for bit only where
    the whole call is plain, too."""
    spec = synth.PointSpec(seed=synth.BASE_SEED + 1760 + M, dets=("H1", "L1", "V1")[:K], n_modes=M, n_t=n_t, snr=1.0,
                           kernel="none")
    d = synth.make_point(spec)
    th = torch.tensor(synth.mixed_samples(d, 47, n))
    h = _handle(ile, [d], "fp64")
    _say(f"fp64 form K={K} M={M} n_t={n_t} n={n}")
    out = h.lnL(th).cpu().numpy()
    part = n // 40
    parts = np.concatenate([h.lnL(th[:, a:a + part]).cpu().numpy() for a in range(0, n, part)])
    h.close()
    assert np.array_equal(out, parts) != sorted_form
    assert np.allclose(out, parts, rtol=1e-12, atol=1e-11)


def test_autotune_cache_of_earlier_kernels(ile, tmp_path):
    """Lines of a cache file that name no kernels, or other ones, are of
    evaluation kernels that are gone: the class is measured again and its line
    appended; the lines appended are read back."""
    d = synth.make_point(synth.workload("tiny").points[0])
    th = torch.tensor(synth.mixed_samples(d, 48, 500))
    T, K, bucket = (len(d["ell"]) + 1) // 2, len(d["det_pos"]), int(np.log2(d["n_t"]))
    path = tmp_path / "tune.txt"
    h = _handle(ile, [d], "fp32")
    h.set_autotune_cache(path)
    h.lnL(th)
    h.close()
    tag = path.read_text().split()[0]
    arch = tag.split("/")[0]
    text = f"{arch} {T} {K} {bucket} 3\n{arch}/1 {T} {K} {bucket} 3\n"
    path.write_text(text)
    _say(f"autotune cache of earlier kernels, tag {tag}")
    for again in range(2):
        h = _handle(ile, [d], "fp32")
        h.set_autotune_cache(path)
        ref = h.lnL(th)
        assert torch.equal(h.lnL(th), ref)
        h.close()
        new = path.read_text()[len(text):].split()
        assert path.read_text().startswith(text) and len(new) == 5 and new[0] == tag and tag != arch, again
