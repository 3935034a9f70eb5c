"""The work a search program asks of this package, as cases that can be timed.

A case is a dict of plain values: its kind, its sizes and its options.  ``prepare`` makes what the
program holds before the call (spectra, series, planes, weights, the prepared template bank),
``run`` is one pass through the package's public calls, ``exact`` the same results in 64 bits from
the definitions, and ``work`` the bytes and operations a pass cannot do without.

Definitions used by ``exact``: Y[z][r] = sum_j A[r + j - M/2] conj T[z][j] with A zero outside
[0, N), P = |Y|^2; T[z][j] = R(j - M/2, z) with R(q, z) the integral over u in [0, 1] of
exp(2 pi i (q u + z (u^2 - u) / 2)); half bins (pi/4)^2 |Y_r - Y_{r+1}|^2 (interbinned) or the
filter at r + 1/2 over the M bins around it (two-bin interpolation); the H-fold sum
S_H[k][r] = sum_{h <= H} P[c + h (k - c)][h r].
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1804_05335_amd as fdas
from paper_1804_05335_amd import autograd as fdas_autograd

DEV = "cuda"
DZ = 2.0
# detection thresholds per fold on unit-mean noise power (a few noise peaks pass each)
THRESHOLDS = {1: 14.0, 2: 17.5, 4: 23.0, 8: 31.0, 16: 45.0, 32: 70.0}
TABLE = 4096        # rows of the program's candidate table, per fold


def listed():
    return [
        # one short spectrum and few templates: the call's latency
        dict(name="plane_short", kind="plane", N=1 << 16, zmax=20.0, M=64, L=512, bank="full"),
        # the ordinary search plane: 2^21 bins, 85 templates of 256 taps
        dict(name="plane_main", kind="plane", N=1 << 21, zmax=84.0, M=256, L=2048, bank="full"),
        # a wide acceleration range on the longest segments, spectrum of odd length
        dict(name="plane_wide", kind="plane", N=1500007, zmax=200.0, M=512, L=8192, bank="full"),
        # half-bin plane by interbinning, odd length
        dict(name="interbin", kind="interbin", N=1000003, zmax=84.0, M=256, L=2048),
        # half-bin plane by two-bin interpolation, shorter templates and segments
        dict(name="fourier2", kind="fourier2", N=300007, zmax=40.0, M=128, L=1024),
        # spectra of many dedispersion trials and beams, ragged lengths, one call
        dict(name="batch_ragged", kind="batch", nspec=64, lo=15, hi=20, lengths=3, zmax=84.0,
             M=256, L=2048),
        # a training step on templates and spectrum: plane and both gradients
        dict(name="train", kind="train", N=1 << 20, zmax=84.0, M=128, L=512),
        # spectrum gradients of a ragged batch over a wide acceleration range
        dict(name="adjoint_batch", kind="adjoint", nspec=6, lo=16, hi=19, lengths=5, zmax=200.0,
             M=512, L=2048, taps=False),
        # the transform that opens a search: one long time series
        dict(name="series_long", kind="series", n=1 << 24, nseries=1),
        # harmonic sums of a finished plane up to 32 harmonics
        dict(name="folds", kind="folds", N=1 << 20, K=85, max_fold=32),
        # a whole search of one series: transform, templates, plane, folds, candidates
        dict(name="search", kind="search", n=1 << 21, nseries=1, zmax=84.0, M=256, L=2048,
             max_fold=8),
        # the same for the series of a few dedispersion trials at once
        dict(name="search_batch", kind="search", n=1 << 18, nseries=8, zmax=40.0, M=128, L=1024,
             max_fold=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plane", "plane", "interbin", "fourier2", "batch", "train", "adjoint",
                       "series", "folds", "search", "search"])
    zmax, M = rng.choice([(20.0, 64), (40.0, 128), (84.0, 128), (84.0, 256), (120.0, 256),
                          (200.0, 512)])
    K = int(2 * zmax / DZ) + 1
    L = rng.choice([l for l in (512, 1024, 2048, 4096, 8192) if 4 * M <= l <= 32 * M])
    most = 3e8 / K                      # bins of a plane of at most 3e8 points
    if kind == "plane":
        return dict(kind=kind, N=_log_int(rng, 5000, most), zmax=zmax, M=M, L=L,
                    bank=rng.choice(["full", "full", "sym"]))
    if kind in ("interbin", "fourier2"):
        return dict(kind=kind, N=_log_int(rng, 5000, most / 2), zmax=zmax, M=M, L=L)
    if kind == "batch":
        lo = rng.choice([11, 12, 14])
        return dict(kind=kind, nspec=_log_int(rng, 2, 48), lo=lo, hi=lo + 4,
                    lengths=rng.randrange(1 << 20), zmax=zmax, M=M, L=L)
    if kind == "train":
        return dict(kind=kind, N=_log_int(rng, 5000, most / 3), zmax=zmax, M=M, L=L)
    if kind == "adjoint":
        lo = rng.choice([12, 14, 15])
        return dict(kind=kind, nspec=_log_int(rng, 2, 12), lo=lo, hi=lo + 3,
                    lengths=rng.randrange(1 << 20), zmax=zmax, M=M, L=L,
                    taps=rng.random() < 0.5)
    if kind == "series":
        log2n = rng.randint(13, 24)
        return dict(kind=kind, n=1 << log2n,
                    nseries=_log_int(rng, 1, max(1, min(64, 1 << (25 - log2n)))))
    if kind == "folds":
        return dict(kind=kind, N=_log_int(rng, 5000, most / 2), K=K,
                    max_fold=rng.choice([4, 8, 16, 32]))
    # searches make their own templates: up to the listed search's count of them
    zmax, M = rng.choice([(20.0, 64), (40.0, 128), (84.0, 128), (84.0, 256)])
    K, L = int(2 * zmax / DZ) + 1, rng.choice([512, 1024, 2048]) * (M // 64)
    log2n = rng.randint(14, 21)
    nseries = min(_log_int(rng, 1, 16), max(1, int(9e7 / K) >> (log2n - 1)))
    return dict(kind=kind, n=1 << log2n, nseries=nseries, zmax=zmax, M=M, L=L,
                max_fold=rng.choice([4, 8, 16, 32]))


# ---- inputs -----------------------------------------------------------------------


def _templates(case):
    return int(2 * case["zmax"] / DZ) + 1


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _response(q, z):
    """R(q, z) for 1-D tensors q and z, [len(z)][len(q)] complex128 (Gauss-Legendre panels)."""
    x, w = np.polynomial.legendre.leggauss(16)
    panels = 192
    u = ((np.arange(panels)[:, None] + 0.5 + 0.5 * x[None, :]) / panels).reshape(-1)
    w = np.tile(0.5 * w / panels, panels)
    u, w = torch.from_numpy(u).to(DEV), torch.from_numpy(w).to(DEV)
    turn = 2.0 * math.pi * u
    eq = torch.polar(torch.ones((), dtype=torch.float64, device=DEV), q[:, None] * turn[None, :])
    ez = torch.polar(w[None, :].expand(len(z), -1).contiguous(),
                     math.pi * z[:, None] * (u * u - u)[None, :])
    return ez @ eq.T


def _drifts(zmax):
    K = int(2 * zmax / DZ) + 1
    return (torch.arange(K, dtype=torch.float64, device=DEV) - (K - 1) / 2) * DZ


def _taps(zmax, M, half=False):
    """The templates, rounded to complex64 as the calls take them."""
    if half:
        q = 0.5 - (torch.arange(M + 2, dtype=torch.float64, device=DEV) - (M + 2) // 2)
        T = _response(q, _drifts(zmax))
        T[:, :2] = 0
    else:
        T = _response(torch.arange(M, dtype=torch.float64, device=DEV) - M // 2, _drifts(zmax))
    return T.to(torch.complex64)


def _spectrum(n, zmax, g, signals=4):
    """Normalised noise (mean power 1) with a few drifting signals of power 50."""
    a = torch.randn(n, dtype=torch.complex64, device=DEV, generator=g)
    draws = torch.rand(signals, 3, generator=g, device=DEV, dtype=torch.float64)
    wide = min(256, n)
    for r, z, phase in draws.tolist():
        r, z = wide / 2 + r * (n - wide), 0.9 * zmax * (2 * z - 1)
        k0 = int(r) - wide // 2
        k = torch.arange(k0, k0 + wide, dtype=torch.float64, device=DEV)
        R = _response(k - r, torch.tensor([z], dtype=torch.float64, device=DEV))[0]
        a[k0:k0 + wide] += (math.sqrt(50.0) * R * np.exp(2j * math.pi * phase)).to(a.dtype)
    return a


def _lengths(case):
    rng = np.random.default_rng(case["lengths"])
    e = rng.uniform(case["lo"], case["hi"], case["nspec"])
    return [int(v) for v in np.floor(2.0 ** e)]


def _series(case, g):
    """White noise with a pulsed drifting signal of eight harmonics in each series."""
    n, nseries = case["n"], case["nseries"]
    x = torch.randn(nseries, n, dtype=torch.float32, device=DEV, generator=g)
    u = torch.arange(n, dtype=torch.float64, device=DEV) / n
    zmax = case.get("zmax", 20.0)
    amp = 2.0 * math.sqrt(60.0 / n)
    for b, (r, z, phase) in enumerate(
            torch.rand(nseries, 3, generator=g, device=DEV, dtype=torch.float64).tolist()):
        r0, z0 = n / 40 + r * n / 20, zmax / 8 * (2 * z - 1)
        cycles = r0 * u + 0.5 * z0 * (u * u - u) + phase
        for h in range(1, 9):
            x[b] += (amp * torch.cos(2.0 * math.pi * torch.frac(h * cycles))).float()
    return x


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    s = dict(case)
    if kind in ("plane", "interbin", "fourier2"):
        s["K"] = _templates(case)
        s["spec"] = _spectrum(case["N"], case["zmax"], g)
        taps, s["bank"] = fdas.make_bank(case["zmax"], DZ, case["M"], case["L"], device=DEV)
        s["symmetric"] = case.get("bank") == "sym"
        if s["symmetric"]:
            s["bank"] = fdas.prepare_bank_sym(taps, case["L"])
        if kind == "fourier2":
            _, s["bank_half"] = fdas.make_bank_half(case["zmax"], DZ, case["M"], case["L"],
                                                    device=DEV)
    elif kind in ("batch", "adjoint"):
        s["K"] = _templates(case)
        s["specs"], s["offsets"] = fdas.pack(
            [_spectrum(n, case["zmax"], g, signals=1) for n in _lengths(case)], device=DEV)
        _, s["bank"] = fdas.make_bank(case["zmax"], DZ, case["M"], case["L"], device=DEV)
        if kind == "adjoint":
            s["w"] = torch.rand(s["K"] * s["specs"].numel(), device=DEV, generator=g)
    elif kind == "train":
        s["spec"] = _spectrum(case["N"], case["zmax"], g).requires_grad_()
        taps = _taps(case["zmax"], case["M"])       # templates in training: a little off
        taps += 1e-3 * torch.randn(taps.shape, dtype=taps.dtype, device=DEV, generator=g)
        s["taps"] = taps.requires_grad_()
        s["w"] = torch.rand(taps.shape[0], case["N"], device=DEV, generator=g)
    elif kind == "folds":
        s["plane"] = -torch.log1p(-torch.rand(case["K"], case["N"], device=DEV, generator=g))
    else:                                           # series, search
        x = _series(case, g)
        s["x"] = x[0].contiguous() if case["nseries"] == 1 else x
    return s


def _column(v):
    """A column of a candidate list in the program's fixed-size table (counts stay numbers)."""
    if isinstance(v, int):
        return v
    out = np.zeros(TABLE, dtype=v.dtype)
    out[:len(v)] = v[:TABLE]
    return out


def run(s):
    kind = s["kind"]
    if kind == "plane":
        call = fdas.correlate_sym if s["symmetric"] else fdas.correlate
        return call(s["spec"], s["bank"], s["K"], s["M"], s["L"])
    if kind == "interbin":
        return fdas.correlate_interbin(s["spec"], s["bank"], s["K"], s["M"], s["L"])
    if kind == "fourier2":
        return fdas.correlate_fourier2(s["spec"], s["bank"], s["bank_half"], s["K"], s["M"],
                                       s["L"])
    if kind == "batch":
        return fdas.correlate_batched(s["specs"], s["offsets"], s["bank"], s["K"], s["M"], s["L"])
    if kind == "adjoint":
        return fdas.correlate_backward_batched(s["specs"], s["offsets"], s["bank"], s["K"],
                                               s["M"], s["L"], s["w"], want_taps=s["taps"])
    if kind == "train":
        plane = fdas_autograd.correlate(s["spec"], s["taps"], s["L"])
        # the gradient that reaches the plane from the layers above it
        gs, gt = torch.autograd.grad(plane, (s["spec"], s["taps"]), grad_outputs=s["w"])
        return plane, gs, gt
    if kind == "series":
        scale = 1.0 / math.sqrt(s["n"])
        if s["nseries"] == 1:
            return fdas.spectrum_from_series(s["x"], scale)
        return fdas.spectra_from_series(s["x"], scale)
    if kind == "folds":
        return fdas.harmonic_sums(s["plane"], s["max_fold"])[1:]
    thresholds = {H: t for H, t in THRESHOLDS.items() if H <= s["max_fold"]}
    call = fdas.search if s["nseries"] == 1 else fdas.search_batched
    found = call(s["x"], s["zmax"], DZ, s["M"], s["L"], s["max_fold"], thresholds)
    return {H: [_column(v) for v in columns] for H, columns in found.items()}


# ---- the same in 64 bits ------------------------------------------------------------


def _pow2(n):
    return 1 << (n - 1).bit_length()


def _filters(T, P):
    """Transforms of the filters h[(M/2 - j) mod P] = conj T[j], for rows T [k][M]."""
    M = T.shape[1]
    h = torch.zeros(T.shape[0], P, dtype=torch.complex128, device=DEV)
    h[:, (M // 2 - torch.arange(M, device=DEV)) % P] = T.to(torch.complex128).conj()
    return torch.fft.fft(h)


def _rows_at_once(P):
    return max(1, (1 << 24) // P)


def _correlation(A, T, count):
    """Y[z][r] for r in [0, count), a block of rows at a time."""
    P = _pow2(max(A.numel(), count) + T.shape[1])
    Af = torch.fft.fft(A.to(torch.complex128), n=P)
    step = _rows_at_once(P)
    for z in range(0, T.shape[0], step):
        yield z, torch.fft.ifft(Af * _filters(T[z:z + step], P))[:, :count]


def _power(y):
    return y.real.square() + y.imag.square()


def _plane(A, T):
    out = torch.empty(T.shape[0], A.numel(), dtype=torch.float64, device=DEV)
    for z, y in _correlation(A, T, A.numel()):
        out[z:z + y.shape[0]] = _power(y)
    return out


def _gradients(A, T, w):
    """Gradients of sum w P: (spectrum, taps)."""
    N, (K, M) = A.numel(), T.shape
    P = _pow2(N + M)
    Af = torch.fft.fft(A.to(torch.complex128), n=P)
    acc = torch.zeros(P, dtype=torch.complex128, device=DEV)
    gt = torch.empty(K, M, dtype=torch.complex128, device=DEV)
    lags = (torch.arange(M, device=DEV) - M // 2) % P
    step = _rows_at_once(P)
    for z in range(0, K, step):
        Hf = _filters(T[z:z + step], P)
        g = 2 * w[z:z + step].double() * torch.fft.ifft(Af * Hf)[:, :N]
        Gf = torch.fft.fft(g, n=P)
        acc += (Hf.conj() * Gf).sum(0)
        gt[z:z + step] = torch.fft.ifft(Gf.conj() * Af)[:, lags]
    return torch.fft.ifft(acc)[:N], gt


def _folds(plane, max_fold):
    K, N = plane.shape
    c, out, H = (K - 1) // 2, [plane], 2
    while H <= max_fold:
        kc, n = c // H, -(-N // H)
        prev = out[-1]
        pc = (prev.shape[0] - 1) // 2
        s = prev[pc - kc:pc + kc + 1, :n].clone()
        for h in range(H // 2 + 1, H + 1):
            s += plane[c - h * kc:c + h * kc + 1:h, ::h][:, :n] if kc else plane[c:c + 1, ::h][:, :n]
        out.append(s)
        H *= 2
    return out


def _peaks(S, threshold):
    """Powers of the points above the threshold and no lower than any neighbour."""
    p = torch.nn.functional.pad(S, (1, 1, 1, 1), value=-math.inf)
    near = S
    for a in range(3):
        for b in range(3):
            near = torch.maximum(near, p[a:a + S.shape[0], b:b + S.shape[1]])
    return S[(S > threshold) & (S >= near)]


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "plane":
        return _plane(s["spec"], _taps(case["zmax"], case["M"]))
    if kind == "interbin":
        N, K = case["N"], s["K"]
        out = torch.empty(K, N, 2, dtype=torch.float64, device=DEV)
        for z, y in _correlation(s["spec"], _taps(case["zmax"], case["M"]), N + 1):
            out[z:z + y.shape[0], :, 0] = _power(y[:, :N])
            out[z:z + y.shape[0], :, 1] = (math.pi / 4) ** 2 * _power(y[:, :N] - y[:, 1:])
        return out.view(K, 2 * N)
    if kind == "fourier2":
        whole = _plane(s["spec"], _taps(case["zmax"], case["M"]))
        half = _plane(s["spec"], _taps(case["zmax"], case["M"], half=True))
        return torch.stack([whole, half], -1).view(s["K"], -1)
    if kind == "batch":
        T, at, parts = _taps(case["zmax"], case["M"]), 0, []
        for n in _lengths(case):
            parts.append(_plane(s["specs"][at:at + n], T).reshape(-1))
            at += n
        return torch.cat(parts)
    if kind == "adjoint":
        T, K, at, gs, gt = _taps(case["zmax"], case["M"]), s["K"], 0, [], 0
        for n in _lengths(case):
            a, t = _gradients(s["specs"][at:at + n], T, s["w"][K * at:K * (at + n)].view(K, n))
            gs.append(a)
            gt = gt + t
            at += n
        return torch.cat(gs), gt if case["taps"] else None
    if kind == "train":
        A, T = s["spec"].detach(), s["taps"].detach()
        return (_plane(A, T), *_gradients(A, T, s["w"]))
    if kind == "series":
        return torch.fft.rfft(s["x"].double()) / math.sqrt(case["n"])
    if kind == "folds":
        return _folds(s["plane"].double(), case["max_fold"])[1:]
    # search: the candidates' powers, in the order (series, row, r); their places are whole numbers
    x = s["x"].double().view(case["nseries"], -1)
    spec = torch.fft.rfft(x) / math.sqrt(case["n"])
    one = case["nseries"] == 1
    if one:
        spec = spec[:, :-1]
    T = _response(torch.arange(case["M"], dtype=torch.float64, device=DEV) - case["M"] // 2,
                  _drifts(case["zmax"]))
    found = {H: [] for H in THRESHOLDS if H <= case["max_fold"]}
    for A in spec:
        for H, S in zip(sorted(found), _folds(_plane(A, T), case["max_fold"])):
            found[H].append(_peaks(S, THRESHOLDS[H]))
    powers = {H: _column(torch.cat(v).cpu().numpy()) for H, v in found.items()}
    return {H: [None, None, v, None] if one else [None, None, None, v, None]
            for H, v in powers.items()}


# ---- what a pass cannot do without ---------------------------------------------------


def _fft_flops(L):
    return 4.25 * L * math.log2(L)


def _forward(N, K, M, L, planes=1):
    """Bytes and operations of the plane of N bins: spectrum and bank in, plane out; a transform of
    each segment, and per template the product, a transform back and the powers."""
    segments = -(-N // (L - M))
    return (8 * N + planes * 8 * K * L + planes * 4 * K * N,
            segments * (_fft_flops(L) + planes * K * (6 * L + _fft_flops(L))) + planes * 3 * K * N)


def _fold_sizes(N, K, max_fold):
    c, H, out = (K - 1) // 2, 2, []
    while H <= max_fold:
        out.append((2 * (c // H) + 1) * -(-N // H))
        H *= 2
    return out


def work(case):
    kind = case["kind"]
    if kind in ("plane", "interbin", "fourier2"):
        K = _templates(case)
        b, f = _forward(case["N"], K, case["M"], case["L"], 2 if kind == "fourier2" else 1)
        if kind == "interbin":
            b, f = b + 4 * K * case["N"], f + 6 * K * case["N"]
        return {"bytes": b, "flops": f}
    if kind in ("batch", "adjoint"):
        K, L, M = _templates(case), case["L"], case["M"]
        each = [_forward(n, K, M, L) for n in _lengths(case)]
        b = sum(x for x, _ in each) - 8 * K * L * (len(each) - 1)
        f = sum(y for _, y in each)
        if kind == "adjoint":   # weights in, gradients out; a second transform per template
            b += 8 * sum(_lengths(case)) + (8 * K * M if case["taps"] else 0)
            f = 2 * f
        return {"bytes": b, "flops": f}
    if kind == "train":         # plane, then weights in and gradients out
        K, N, M = _templates(case), case["N"], case["M"]
        b, f = _forward(N, K, M, case["L"])
        return {"bytes": b + 4 * K * N + 16 * N + 16 * K * M, "flops": 3 * f}
    if kind == "series":
        n = case["n"] * case["nseries"]
        return {"bytes": 8 * n, "flops": 2.5 * n * math.log2(case["n"])}
    if kind == "folds":
        sizes = _fold_sizes(case["N"], case["K"], case["max_fold"])
        return {"bytes": 4 * (case["K"] * case["N"] + sum(sizes)),
                "flops": sum(s * 2 ** i for i, s in enumerate(sizes))}
    n, ns, K = case["n"], case["nseries"], _templates(case)
    _, f = _forward(n // 2 + (ns > 1), K, case["M"], case["L"])
    sizes = _fold_sizes(n // 2, K, case["max_fold"])
    # series in and bank; the plane and the folds between the steps are written and read once
    return {"bytes": ns * (4 * n + 16 * (n // 2) + 8 * (K * (n // 2) + sum(sizes))) +
            8 * K * case["L"],
            "flops": ns * (f + 2.5 * n * math.log2(n) +
                           sum(s * 2 ** i for i, s in enumerate(sizes)))}
