"""Performance cases of the training-data generator: what its users have it do, through the public entry points.

A case is a dict of plain values.  ``prepare`` makes what a user's program holds before the call (the resident
background, the context, the workspace and the output buffers), ``run`` is one pass, ``work`` the bytes and flops that
the path cannot do without, and ``exact`` the same outputs computed in 64 bits with plain torch and numpy.
"""

import math

import numpy as np
import torch

from paper_2407_19048_amd import gwgen, inputs
from paper_2407_19048_amd import surrogate as surrogate_module

DEV = "cuda"
BATCH_INDEX = 5          # any batch of a run
LR_NODES = 1024          # surrogate node grid
TRIM_SECONDS = 2.0       # duration of the per-run whitening filter (1 s cropped at each end)


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # one sample on demand: the shortest call of an interactive or online program, bound by latency and launches
        dict(name="one_sample", kind="batch", base="paper_scale", batch=1, log2_bg=24),
        # the small workload: 64 TaylorF2 signals, two detectors, 4 s at 1024 Hz, Welch over 32 s
        dict(name="small_batch", kind="batch", base="pr1_plain", batch=64, log2_bg=22),
        # the training batch at the paper's scale: 2048 signals, three detectors, 8 s at 2048 Hz, Welch over 64 s
        dict(name="paper_batch", kind="batch", base="paper_scale", batch=2048, log2_bg=27),
        # the reference precision (binary64 throughout), used to judge the other modes
        dict(name="binary64_batch", kind="batch", base="paper_scale", batch=100, log2_bg=24, precision=2),
        # an uneven batch: six (rate, duration) classes drawn per signal, an eighth of the full workload's 16384
        dict(name="uneven_batch", kind="uneven", batch=2048, log2_bg=25),
        # long binary-neutron-star windows: 256 s at 2048 Hz
        dict(name="long_windows", kind="batch", base="bns_long", batch=32, log2_bg=24),
        # batches whitened with one fixed filter per run instead of a PSD per sample
        dict(name="run_filter_batch", kind="runpsd", base="paper_scale", batch=2048, log2_bg=25),
        # the noise fit of that mode, once per resident background: run PSD and truncated filter
        dict(name="run_filter_fit", kind="runfit", base="paper_scale", chunks=200, log2_bg=25),
        # view pairs for self-supervised pre-training, an odd batch
        dict(name="view_pairs", kind="pairs", base="paper_scale", batch=301, log2_bg=25),
        # the learned waveform in place of the closed form
        dict(name="surrogate_batch", kind="surrogate", base="paper_scale", batch=2048, log2_bg=25),
        # forward and backward pass of the surrogate's network at its training batch
        dict(name="surrogate_gradients", kind="train", base="paper_scale", batch=8192),
        # the six steps one by one, every intermediate product kept: analysis programs
        dict(name="single_steps", kind="steps", base="paper_scale", batch=200, log2_bg=25),
    ]


def draw(rng):
    """One more case of those ranges: batches over three decades, every window length, odd stretches and counts."""
    kind = rng.choice(("batch", "batch", "batch", "batch", "uneven", "long", "runpsd", "runfit", "pairs", "surrogate",
                       "train", "steps"))
    if kind == "train":
        return dict(kind=kind, base="paper_scale", batch=_log_int(rng, 64, 8192))
    if kind == "uneven":
        return dict(kind=kind, batch=_log_int(rng, 48, 2048), log2_bg=25)
    if kind == "long":
        t_window = rng.choice((32.0, 64.0, 128.0, 256.0, 512.0))
        return dict(kind="batch", base="bns_long", t_window=t_window, batch=_log_int(rng, 1, int(32 * 256 / t_window)),
                    log2_bg=24, psd_length=float(rng.randrange(16, 65)))
    fs = rng.choice((1024.0, 2048.0))
    t_window = rng.choice((4.0, 8.0, 16.0) if kind in ("runpsd", "runfit", "surrogate") else (2.0, 4.0, 8.0, 16.0))
    case = dict(kind=kind, base="paper_scale", fs=fs, t_window=t_window, psd_length=float(rng.randrange(16, 65)),
                log2_bg=25, detectors=rng.randrange(1, 4))
    if kind == "runfit":
        case["chunks"] = _log_int(rng, 4, int(200 * 64 / case["psd_length"]))
        return case
    case["batch"] = _log_int(rng, 1, int({"batch": 2048, "runpsd": 2048, "pairs": 512, "surrogate": 1024,
                                          "steps": 256}[kind] * 16384 / max(16384, fs * t_window)))
    if kind in ("batch", "pairs", "steps"):
        case["base"] = rng.choice(("paper_scale", "pr1_plain", "sine_gaussian"))
        case["f_min"] = 20.0
    if kind == "batch":
        case["precision"] = rng.choice((1, 1, 1, 0, 2))
        if case["precision"] == 2:
            case["batch"] = min(case["batch"], 100)
            if fs * t_window > 16384:
                case["t_window"] = 8.0
    return case


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _config(case):
    """The configuration of a case: one of the repository's workloads with the case's changes."""
    cfg = inputs.config(case["base"])
    for key in ("fs", "t_window", "psd_length", "f_min", "precision"):
        if key in case:
            cfg[key] = case[key]
    if "detectors" in case:
        cfg["det_ids"] = tuple(range(case["detectors"]))
    if cfg["approximant"] == 2:
        cfg["f0"] = (32.0, min(1000.0, 0.45 * cfg["fs"]))
    return cfg


def _sizes(cfg):
    n, p, l = (int(round(cfg[k] * cfg["fs"])) for k in ("t_window", "psd_length", "fftlen"))
    return dict(N=n, P=p, L=l, K=2 * (p - l) // l + 1, F=n // 2 + 1, Fw=l // 2 + 1, D=len(cfg["det_ids"]))


def _uneven_classes(case):
    return inputs.ragged_classes(), inputs.ragged_assignment(case["batch"], seed=11)


# ------------------------------------------------------------------ inputs

def _background(n_det, log2_len, fs, seed):
    """Stationary Gaussian noise coloured like the detectors' design curve, [n_det][2^log2_len] binary32 on the GPU."""
    taps = int(4 * fs)
    f = torch.arange(taps // 2 + 1, dtype=torch.float64, device=DEV) * fs / taps
    x = f.clamp(min=10.0) / 215.0
    psd = 2.0 ** 140 * 1e-49 * (x ** -4.14 - 5 * x ** -2 + 111 * (1 - x ** 2 + x ** 4 / 2) / (1 + x ** 2 / 2))
    h = torch.roll(torch.fft.irfft(torch.sqrt(fs * psd / 2), n=taps), taps // 2)
    h = h * torch.hann_window(taps, dtype=torch.float64, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + int(fs))
    piece = min(log2_len, 20)
    bg = torch.empty((n_det, 1 << log2_len), dtype=torch.float32, device=DEV)
    colour = torch.fft.rfft(h, n=1 << piece).to(torch.complex64)
    for d in range(n_det):
        white = torch.randn((1 << (log2_len - piece), 1 << piece), generator=gen, device=DEV)
        bg[d] = torch.fft.irfft(torch.fft.rfft(white) * colour, n=1 << piece).reshape(-1)
    return bg


def _network_inputs(cfg, batch, seed):
    """Parameters within the prior and standardised targets of the surrogate's network."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 17)
    u = torch.rand((batch, 4), generator=gen, device=DEV)
    lo = torch.tensor([cfg["mc"][0], cfg["q"][0], cfg["chi"][0], cfg["chi"][0]], device=DEV)
    hi = torch.tensor([cfg["mc"][1], cfg["q"][1], cfg["chi"][1], cfg["chi"][1]], device=DEV)
    return lo + u * (hi - lo), torch.randn((batch, 128), generator=gen, device=DEV)


def _surrogate(gen, cfg, seed):
    """A surrogate with a smooth basis, its skip path fitted to the plain model and a head that sends some samples to
    the plain model; the network has its initial weights."""
    s = surrogate_module.Surrogate(gen, max_batch=2048)
    j = np.arange(LR_NODES) + 0.5
    dct = np.cos(np.pi * np.arange(64)[:, None] * j[None, :] / LR_NODES) * math.sqrt(2.0 / LR_NODES)
    dct[0] *= math.sqrt(0.5)
    n = 1024
    params = torch.empty((12, n), dtype=torch.float64, device=DEV)
    offsets = torch.empty(n, dtype=torch.int64, device=DEV)
    z = gen.sizes
    gen.sample_params(seed + 1, 0, n, z["P"] + z["N"], params, offsets)
    ratio = torch.empty((n, LR_NODES), dtype=torch.float32, device=DEV)
    dpsi = torch.empty_like(ratio)
    feat = torch.empty((n, 9), dtype=torch.float64, device=DEV)
    s.targets(params, ratio, dpsi, feat)
    mean = torch.stack([ratio.double().mean(0), dpsi.double().mean(0)]).cpu().numpy()
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    head = np.concatenate([rng.standard_normal(256) * 0.05, [-3.3]]).astype(np.float32)
    state = [np.stack([dct, dct]), mean, np.zeros((9, 128)), np.zeros(128), np.ones(128), head]
    s.set_state(*state)
    coef = torch.empty((n, 128), dtype=torch.float32, device=DEV)
    resid = torch.empty_like(coef)
    s.project(ratio, dpsi, coef)
    s.fit_skip(feat, coef, resid)
    s.set_weights(surrogate_module.init_weights(int(seed)))
    return s


def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind, case=case, seed=int(seed))
    if kind == "uneven":
        classes, cls = _uneven_classes(case)
        plan = gwgen.Ragged(classes, cls)
        bg = {fs: _background(plan.D, case["log2_bg"] - (fs == 1024.0), fs, seed) for fs in inputs.RAGGED_RATES}
        st.update(plan=plan, bgs=[bg[c["fs"]] for c in classes], out=plan.alloc_out(), ws=plan.alloc_workspace(),
                  params=_f32((12, plan.B)), status=_i32(plan.B))
        return st
    cfg = _config(case)
    gen = gwgen.Generator(cfg)
    z = gen.sizes
    st.update(gen=gen, cfg=cfg)
    if kind == "train":
        s = surrogate_module.Surrogate(gen, max_batch=case["batch"])
        s.set_weights(surrogate_module.init_weights(int(seed)))
        theta, targets = _network_inputs(cfg, case["batch"], seed)
        st.update(s=s, theta=theta, targets=targets, grads=_f32(s.n_weights), loss=_f32(1))
        return st
    bg = st["bg"] = _background(z["D"], case["log2_bg"], cfg["fs"], seed)
    if kind == "runfit":
        st.update(psd=_f32((z["D"], z["Fw"])), filt=_f32((z["D"], z["F"])), status=_i32(z["D"]))
        return st
    b = case["batch"]
    st.update(params=_f32((12, b)), status=_i32(b), ws=gen.alloc_workspace(b))
    if kind == "runpsd":
        psd = _f32((z["D"], z["Fw"]))
        st["filt"] = _f32((z["D"], z["F"]))
        gen.run_psd(bg, _fit_chunks(cfg, case), psd)
        taps = int(TRIM_SECONDS * cfg["fs"])
        gen.whiten_filter(psd, taps, st["filt"])
        torch.cuda.synchronize()  # the fit's workspace may go
        st["out"] = _f32((b, z["D"], z["N"] - taps))
        return st
    st["out"] = _f32((b, z["D"], z["N"]))
    if kind == "pairs":
        st["ref"] = _f32((b, z["D"], z["N"]))
    elif kind == "surrogate":
        st["s"] = _surrogate(gen, cfg, seed)
        st["ws"] = gen.alloc_workspace_surrogate(b)
    elif kind == "steps":
        c64 = lambda shape: torch.zeros(shape, dtype=torch.complex64, device=DEV)
        st.update(params=torch.zeros((12, b), dtype=torch.float64, device=DEV),
                  offset=torch.zeros(b, dtype=torch.int64, device=DEV), hp=c64((b, z["F"])), hc=c64((b, z["F"])),
                  hdet=c64((b, z["D"], z["F"])), strain=_f32((b, z["D"], z["N"])), psd=_f32((b, z["D"], z["Fw"])))
    return st


def _f32(shape):
    return torch.zeros(shape, dtype=torch.float32, device=DEV)


def _i32(n):
    return torch.zeros(n, dtype=torch.int32, device=DEV)


def _fit_chunks(cfg, case):
    """Stretches of the run PSD behind a filter batch: 32 of them."""
    z = _sizes(cfg)
    return min(32, ((1 << case["log2_bg"]) - z["P"]) // (z["K"] * z["L"] // 2) + 1)


# ------------------------------------------------------------------ one pass

def run(st):
    kind = st["kind"]
    if kind == "uneven":
        st["plan"].generate(st["seed"], BATCH_INDEX, st["bgs"], st["out"], st["ws"], params_f32=st["params"],
                            status=st["status"])
        return {"out": st["out"], "params": st["params"], "status": st["status"]}
    gen = st["gen"]
    if kind == "train":
        st["s"].gradients(st["theta"], st["targets"], st["grads"], st["loss"])
        return {"grads": st["grads"], "loss": st["loss"]}
    if kind == "runfit":
        ws = gen.run_psd(st["bg"], st["case"]["chunks"], st["psd"])
        gen.whiten_filter(st["psd"], int(TRIM_SECONDS * st["cfg"]["fs"]), st["filt"], st["status"])
        del ws
        return {"psd": st["psd"], "filt": st["filt"], "status": st["status"]}
    b, bg, out = st["case"]["batch"], st["bg"], st["out"]
    if kind == "steps":
        gen.sample_params(st["seed"], BATCH_INDEX * b, b, bg.shape[1], st["params"], st["offset"])
        gen.gen_fd_waveform(st["params"], st["hp"], st["hc"])
        gen.project_detectors(st["params"], st["hp"], st["hc"], st["hdet"])
        gen.inject(bg, st["offset"], st["hdet"], st["strain"])
        gen.welch_psd(bg, st["offset"], st["psd"])
        gen.whiten(st["strain"], st["psd"], out, st["status"])
        return {k: st[k] for k in ("params", "offset", "hp", "hc", "hdet", "strain", "psd", "out", "status")}
    common = dict(params_f32=st["params"], status=st["status"])
    got = {"out": out, "params": st["params"], "status": st["status"]}
    if kind == "batch":
        gen.generate_batch(st["seed"], BATCH_INDEX, b, bg, out, st["ws"], **common)
    elif kind == "runpsd":
        gen.generate_batch_runpsd(st["seed"], BATCH_INDEX, b, bg, st["filt"], int(TRIM_SECONDS * st["cfg"]["fs"]) // 2,
                                  out, st["ws"], **common)
    elif kind == "pairs":
        gen.generate_batch_pairs(st["seed"], BATCH_INDEX, b, bg, st["ref"], out, st["ws"], **common)
        got["ref"] = st["ref"]
    else:
        gen.generate_batch_surrogate(st["s"], st["seed"], BATCH_INDEX, b, bg, out, st["ws"], **common)
    return got


# ------------------------------------------------------------------ work

def _fft_flops(n):
    return 2.5 * n * math.log2(n)


def _item_work(z, welch=True, windows=1):
    """Bytes and flops of one (sample, detector): each background sample read once, each output written once."""
    b = 4.0 * (z["N"] + windows * z["N"])
    f = (1 + windows) * _fft_flops(z["N"]) + 30.0 * windows * z["F"]
    if welch:
        b += 4.0 * z["P"]
        f += z["K"] * (_fft_flops(z["L"]) + 3.0 * z["L"])
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "uneven":
        classes, cls = _uneven_classes(case)
        items = [_item_work(_sizes(c)) for c in classes]
        b, f = (sum(3 * items[c][k] for c in cls) for k in (0, 1))
        return {"bytes": b + 52.0 * case["batch"], "flops": f}
    cfg = _config(case)
    z = _sizes(cfg)
    if kind == "train":
        n = 16 * 256 + 2 * 65536 + 256 * 128
        return {"bytes": case["batch"] * 4.0 * (4 + 128) + 4.0 * 2 * (n + 896), "flops": 6.0 * n * case["batch"]}
    if kind == "runfit":
        segs = case["chunks"] * z["K"]
        b = z["D"] * (4.0 * (segs + 1) * z["L"] / 2 + 4.0 * (z["Fw"] + z["F"]))
        return {"bytes": b, "flops": z["D"] * (segs * (_fft_flops(z["L"]) + 3.0 * z["L"]) + 2 * _fft_flops(z["N"]))}
    items = case["batch"] * z["D"]
    if kind == "steps":
        # every product of the six steps written once, the background read once for the noise and once for the PSD
        b = items * (4.0 * (z["N"] + z["P"]) + 4.0 * 2 * z["N"] + 8.0 * z["F"] + 4.0 * z["Fw"])
        b += case["batch"] * (16.0 * z["F"] + 104.0)
        f = items * (_item_work(z)[1] + _fft_flops(z["N"]))
        return {"bytes": b, "flops": f}
    b, f = _item_work(z, welch=kind != "runpsd", windows=2 if kind == "pairs" else 1)
    if kind == "runpsd":
        b -= 4.0 * int(TRIM_SECONDS * cfg["fs"])
    return {"bytes": items * b + 52.0 * case["batch"], "flops": items * f}


# ------------------------------------------------------------------ the same in 64 bits

def _philox(seed, index, stream):
    """Binary64 uniforms of Philox4x32-10 at counters (index, stream, 0)."""
    m32 = np.uint64(0xFFFFFFFF)
    index = np.asarray(index, dtype=np.uint64)
    c = [index & m32, index >> np.uint64(32), np.full_like(index, stream), np.zeros_like(index)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for r in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m32, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return ((c[0] >> np.uint64(5)).astype(np.float64) * 67108864.0 + (c[1] >> np.uint64(6)).astype(np.float64) + 0.5) * 2.0 ** -53


def _prior(cfg, seed, index, span):
    """Parameters [12][n] and background offsets [n] of the global sample indices."""
    u = [_philox(seed, index, s) for s in range(11)]
    p = np.zeros((12, len(index)))
    if cfg["approximant"] == 2:
        p[0] = cfg["f0"][0] + u[0] * (cfg["f0"][1] - cfg["f0"][0])
        p[1] = cfg["quality"][0] + u[1] * (cfg["quality"][1] - cfg["quality"][0])
        p[2] = cfg["hrss"][0] * (cfg["hrss"][1] / cfg["hrss"][0]) ** u[2]
    else:
        for row, key in ((0, "mc"), (1, "q"), (2, "chi"), (3, "chi")):
            p[row] = cfg[key][0] + u[row] * (cfg[key][1] - cfg[key][0])
        p[4] = np.cbrt(cfg["dl"][0] ** 3 + u[4] * (cfg["dl"][1] ** 3 - cfg["dl"][0] ** 3))
    p[5], p[6], p[7] = np.arccos(2 * u[5] - 1), 2 * np.pi * u[6], np.arcsin(2 * u[7] - 1)
    p[8], p[9], p[10] = np.pi * u[8], 2 * np.pi * u[9], cfg["t_window"] - 1.5 + u[10]
    return p, np.floor(_philox(seed, index, 12) * span).astype(np.int64)


def _taylor_f2(v, eta, q, chi1, chi2):
    """TaylorF2 phase to 3.5PN order and its derivative with respect to v."""
    pi, dm, cs, ca = math.pi, (1 - q) / (1 + q), (chi1 + chi2) / 2, (chi1 - chi2) / 2
    lnv = torch.log(v)
    p5 = pi * (38645 / 756 - 65 / 9 * eta)
    psi = [torch.ones_like(eta), None, 3715 / 756 + 55 / 9 * eta,
           -16 * pi + 113 / 3 * dm * ca + (113 / 3 - 76 / 3 * eta) * cs,
           15293365 / 508032 + 27145 / 504 * eta + 3085 / 72 * eta ** 2 - 395 / 4 * eta * chi1 * chi2,
           p5 * (1 + 3 * lnv + 1.5 * math.log(6.0)),
           11583231236531 / 4694215680 - 640 / 3 * pi ** 2 - 6848 / 21 * (0.5772156649015329 + math.log(4.0) + lnv)
           + (-15737765635 / 3048192 + 2255 / 12 * pi ** 2) * eta + 76055 / 1728 * eta ** 2 - 127825 / 1296 * eta ** 3,
           pi * (77096675 / 254016 + 378515 / 1512 * eta - 74045 / 756 * eta ** 2)]
    slope = {5: 3 * p5, 6: -6848 / 21}
    phase = sum(c * v ** (k - 5) for k, c in enumerate(psi) if c is not None)
    deriv = sum((k - 5) * c * v ** (k - 6) for k, c in enumerate(psi) if c is not None)
    deriv = deriv + sum(c * v ** (k - 6) for k, c in slope.items())
    pre = 3 / (128 * eta)
    return pre * phase, pre * deriv


def _polarisations(cfg, p, f):
    """h+ and hx, complex128 [n][F], of parameters [12][n] (device tensor) at frequencies f."""
    col = lambda i: p[i][:, None]
    ci = torch.cos(col(5))
    pos = f.clamp(min=0.5 / cfg["t_window"])[None, :]
    keep = (f >= cfg["f_min"]) & (f > 0)
    keep[-1] = False
    if cfg["approximant"] == 2:
        f0, qual, hrss = col(0), col(1), col(2)
        tau = qual / (math.sqrt(2.0) * math.pi * f0)
        amp = 2.0 ** 70 * hrss / torch.sqrt(tau * math.sqrt(math.pi / 2))
        gauss = lambda x: 0.5 * math.sqrt(math.pi) * tau * torch.exp(-(math.pi * tau * x) ** 2)
        em = torch.polar(gauss(f - f0), col(9).expand(-1, f.numel()))
        ep = torch.polar(gauss(f + f0), -col(9).expand(-1, f.numel()))
        return keep * amp * 0.5 * (1 + ci ** 2) * (em + ep), keep * amp * ci * 1j * (ep - em)
    mc, q, chi1, chi2, dist = (col(i) for i in range(5))
    eta = q / (1 + q) ** 2
    ms = mc * eta ** -0.6 * 4.925490947641267e-6
    amp0 = (2.0 ** 70 * math.sqrt(5 / 24) * math.pi ** (-2 / 3) * (mc * 4.925490947641267e-6) ** (5 / 6)
            / (dist * (3.085677581491367e22 / 299792458.0)))
    v = (math.pi * ms * pos) ** (1 / 3)
    phase = _taylor_f2(v, eta, q, chi1, chi2)[0]
    amp = amp0 * pos ** (-7 / 6)
    if cfg["approximant"] == 0:
        keep = keep & (f < 1 / (6 ** 1.5 * math.pi * ms))
    else:
        keep = keep & (f < 0.2 / ms)
        at = (chi1 + chi2 * q ** 2) / (1 + q ** 2)
        af = (at - 0.1229 * at ** 2 * eta + 0.4537 * at * eta ** 2 - 2.8904 * at * eta + 2 * math.sqrt(3.0) * eta
              - 3.5171 * eta ** 2 + 2.5763 * eta ** 3).clamp(-0.99, 0.99)
        mf = ms * (1 - (0.0559745 * eta + 0.580951 * eta ** 2 - 0.960673 * eta ** 3 + 3.35241 * eta ** 4))
        f_rd = (1.5251 - 1.1568 * (1 - af) ** 0.1292) / (2 * math.pi * mf)
        f_damp = f_rd / (2 * (0.7 + 1.4187 * (1 - af) ** -0.4990))
        ft = f_rd / 2
        vt = (math.pi * ms * ft) ** (1 / 3)
        pt, dpt = _taylor_f2(vt, eta, q, chi1, chi2)
        x = (ft - f_rd) / f_damp
        b1 = dpt * vt / (3 * ft) - 1 / f_damp / (1 + x ** 2)
        b0 = pt - b1 * ft - torch.atan(x)
        phase = torch.where(pos < ft, phase, b0 + b1 * pos + torch.atan((pos - f_rd) / f_damp))
        a_t = amp0 * ft ** (-7 / 6)
        late = torch.where(pos < f_rd, a_t * (pos / ft) ** (-2 / 3),
                           a_t * 2 ** (-2 / 3) * f_damp ** 2 / ((pos - f_rd) ** 2 + f_damp ** 2))
        amp = torch.where(pos < ft, amp, late)
    e = torch.polar(torch.ones_like(phase), -(phase - col(9) - math.pi / 4)) * (keep * amp)
    return e * 0.5 * (1 + ci ** 2), -1j * e * ci


_SITES = ((46.45514, -119.40766, 324.0, 234.0), (30.56289, -90.77424, 252.2835, 162.2835),
          (43.63141, 10.50450, 19.4326, 289.4326))


def _response(det, p):
    """Antenna patterns and delay of a detector for the sky positions of p: three tensors [n]."""
    lat, lon, ax, ay = (math.radians(v) for v in _SITES[det])
    flat = 1 / 298.257223563
    e2 = flat * (2 - flat)
    nu = 6378137.0 / math.sqrt(1 - e2 * math.sin(lat) ** 2)
    site = np.array([nu * math.cos(lat) * math.cos(lon), nu * math.cos(lat) * math.sin(lon), nu * (1 - e2) * math.sin(lat)])
    east = np.array([-math.sin(lon), math.cos(lon), 0.0])
    north = np.array([-math.sin(lat) * math.cos(lon), -math.sin(lat) * math.sin(lon), math.cos(lat)])
    arm = [math.cos(a) * north + math.sin(a) * east for a in (ax, ay)]
    tensor = torch.from_numpy((np.outer(arm[0], arm[0]) - np.outer(arm[1], arm[1])) / 2).to(p)
    sr, cr, sd, cd, sp, cp = (g(p[i]) for i in (6, 7, 8) for g in (torch.sin, torch.cos))
    zero = torch.zeros_like(sr)
    theta, phi = torch.stack([sd * cr, sd * sr, -cd]), torch.stack([-sr, cr, zero])
    a, b = cp * theta + sp * phi, -sp * theta + cp * phi
    n = torch.stack([cd * cr, cd * sr, sd])
    pair = lambda x, y: ((tensor @ x) * y).sum(0)
    return pair(a, a) - pair(b, b), 2 * pair(a, b), -(n * torch.from_numpy(site).to(p)[:, None]).sum(0) / 299792458.0


def _projected(cfg, p, hp, hc, t_signal):
    """DFT coefficients of the detectors' strain, complex128 [n][D][F]."""
    f = torch.arange(hp.shape[1], dtype=torch.float64, device=DEV) / cfg["t_window"]
    got = []
    for det in cfg["det_ids"]:
        fp, fx, dt = _response(det, p)
        turn = torch.remainder(f[None, :] * (t_signal + dt)[:, None], 1.0)
        got.append(cfg["fs"] * (fp[:, None] * hp + fx[:, None] * hc) * torch.exp(-2j * math.pi * turn))
    return torch.stack(got, 1)


def _welch(x, l, fs):
    """One-sided Welch PSD of the rows of x (last axis): periodic Hann, half overlap, mean."""
    win = torch.hann_window(l, periodic=True, dtype=torch.float64, device=DEV)
    spec = torch.fft.rfft(x.unfold(-1, l, l // 2) * win).abs().square().mean(-2) / (fs * win.square().sum())
    spec[..., 1:-1] *= 2
    return spec


def _gain(psd, cfg, z):
    """Whitening gain on the window grid from PSD rows."""
    k = torch.arange(z["F"], device=DEV)
    r = z["N"] // z["L"]
    i = torch.clamp(k // r, max=z["Fw"] - 2)
    t = (k - i * r).double() / r
    g = 1 / torch.sqrt(cfg["fs"] / 2 * ((1 - t) * psd[..., i] + t * psd[..., i + 1]))
    return torch.where((k > 0) & (k < z["F"] - 1) & (k / cfg["t_window"] >= cfg["f_min"]), g, torch.zeros_like(g))


def _rows(bg, offset, start, length):
    """[n][D][length] binary64 slices of the background at offset + start."""
    at = torch.from_numpy(offset).to(DEV)[:, None] + start + torch.arange(length, device=DEV)
    return bg[:, at].permute(1, 0, 2).double()


def _irfft(x, n):
    """irfft with the imaginary parts of DC and Nyquist dropped."""
    x = x.clone()
    x[..., 0].imag.zero_()
    x[..., -1].imag.zero_()
    return torch.fft.irfft(x, n=n)


def _batch_exact(cfg, bg, p, offset, filt=None, trim=0, pair=False):
    """Whitened windows [n][D][N] (and the reference views), a few samples at a time."""
    z = _sizes(cfg)
    f = torch.arange(z["F"], dtype=torch.float64, device=DEV) / cfg["t_window"]
    got, ref = [], []
    step = max(1, (1 << 24) // (z["D"] * (z["N"] + 2 * z["P"])))
    for i in range(0, p.shape[1], step):
        pi = torch.from_numpy(p[:, i:i + step]).to(DEV)
        o = offset[i:i + step]
        noise = torch.fft.rfft(_rows(bg, o, z["P"], z["N"]))
        gain = filt if filt is not None else _gain(_welch(_rows(bg, o, 0, z["P"]), z["L"], cfg["fs"]), cfg, z)
        hp, hc = _polarisations(cfg, pi, f)
        t_ref = torch.full_like(pi[10], cfg["t_window"] - 1.5)
        for keep, t in ((got, pi[10]),) + (((ref, t_ref),) if pair else ()):
            y = torch.fft.irfft((noise + _projected(cfg, pi, hp, hc, t)) * gain, n=z["N"])
            keep.append(y[..., trim:z["N"] - trim])
    return torch.cat(got), torch.cat(ref) if pair else None


def _run_fit(cfg, bg, chunks):
    """Run PSD [D][Fw] and truncated whitening filter [D][F]."""
    z = _sizes(cfg)
    seg = chunks * z["K"]
    psd = torch.stack([_welch_long(row[:(seg + 1) * z["L"] // 2], z["L"], cfg["fs"]) for row in bg])
    h = torch.fft.irfft(_gain(psd, cfg, z).to(torch.complex128), n=z["N"])
    taps = int(TRIM_SECONDS * cfg["fs"])
    lag = torch.arange(z["N"], device=DEV)
    lag = torch.where(lag <= z["N"] // 2, lag, lag - z["N"]).double()
    h = h * torch.where(2 * lag.abs() < taps, torch.cos(math.pi * lag / taps) ** 2, torch.zeros_like(lag))
    return psd, torch.fft.rfft(h).abs()


def _welch_long(x, l, fs):
    """Welch PSD of one long row, some segments at a time."""
    total, n, seg = 0.0, 0, x.numel() // (l // 2) - 1
    for s in range(0, seg, 4096):
        m = min(4096, seg - s)
        total = total + m * _welch(x[s * l // 2:(s + m + 1) * l // 2].double(), l, fs)
        n += m
    return total / n


def exact(case, seed):
    kind, seed = case["kind"], int(seed)
    if kind == "surrogate":
        return None  # the network's bfloat16 rounding and the routing that follows from it are part of its result
    if kind == "uneven":
        return _exact_uneven(case, seed)
    cfg = _config(case)
    z = _sizes(cfg)
    if kind == "train":
        return _exact_train(cfg, case, seed)
    bg = _background(z["D"], case["log2_bg"], cfg["fs"], seed)
    if kind == "runfit":
        psd, filt = _run_fit(cfg, bg, case["chunks"])
        return {"psd": psd, "filt": filt, "status": None}
    b = case["batch"]
    index = np.arange(BATCH_INDEX * b, (BATCH_INDEX + 1) * b)
    p, offset = _prior(cfg, seed, index, (1 << case["log2_bg"]) - z["P"] - z["N"] + 1)
    if kind == "steps":
        f = torch.arange(z["F"], dtype=torch.float64, device=DEV) / cfg["t_window"]
        pt = torch.from_numpy(p).to(DEV)
        hp, hc = _polarisations(cfg, pt, f)
        hdet = _projected(cfg, pt, hp, hc, pt[10])
        strain = _rows(bg, offset, z["P"], z["N"]) + _irfft(hdet, z["N"])
        psd = torch.cat([_welch(_rows(bg, offset[i:i + 16], 0, z["P"]), z["L"], cfg["fs"]) for i in range(0, b, 16)])
        out = torch.fft.irfft(torch.fft.rfft(strain) * _gain(psd, cfg, z), n=z["N"])
        return dict(params=pt, offset=None, hp=hp, hc=hc, hdet=hdet, strain=strain, psd=psd, out=out, status=None)
    filt, trim = None, 0
    if kind == "runpsd":
        filt = _run_fit(cfg, bg, _fit_chunks(cfg, case))[1]
        trim = int(TRIM_SECONDS * cfg["fs"]) // 2
    out, ref = _batch_exact(cfg, bg, p, offset, filt, trim, kind == "pairs")
    got = {"out": out, "params": torch.from_numpy(p), "status": None}
    if ref is not None:
        got["ref"] = ref
    return got


def _exact_uneven(case, seed):
    classes, cls = _uneven_classes(case)
    sizes = [_sizes(c) for c in classes]
    start = np.concatenate([[0], np.cumsum([sizes[c]["D"] * sizes[c]["N"] for c in cls])])
    out = torch.zeros(int(start[-1]), dtype=torch.float64, device=DEV)
    params = np.zeros((12, case["batch"]))
    for fs in inputs.RAGGED_RATES:
        log2 = case["log2_bg"] - (fs == 1024.0)
        bg = _background(3, log2, fs, seed)
        for c, cfg in enumerate(classes):
            at = np.flatnonzero(cls == c)
            if cfg["fs"] != fs or not at.size:
                continue
            z = sizes[c]
            p, offset = _prior(cfg, seed, BATCH_INDEX * case["batch"] + at, (1 << log2) - z["P"] - z["N"] + 1)
            p[11] = c
            params[:, at] = p
            rows = torch.from_numpy(start[at]).to(DEV)[:, None] + torch.arange(z["D"] * z["N"], device=DEV)
            out[rows] = _batch_exact(cfg, bg, p, offset)[0].reshape(at.size, -1).double()
    return {"out": out, "params": torch.from_numpy(params), "status": None}


def _exact_train(cfg, case, seed):
    theta, targets = _network_inputs(cfg, case["batch"], seed)
    flat = torch.from_numpy(surrogate_module.init_weights(seed)).to(DEV).double().requires_grad_(True)
    lo = torch.tensor([cfg["mc"][0], cfg["q"][0], cfg["chi"][0], cfg["chi"][0]], dtype=torch.float64, device=DEV)
    hi = torch.tensor([cfg["mc"][1], cfg["q"][1], cfg["chi"][1], cfg["chi"][1]], dtype=torch.float64, device=DEV)
    x = torch.nn.functional.pad(2 * (theta.double() - lo) / (hi - lo) - 1, (0, 12))
    at = 0
    for n, (nin, nout) in enumerate(((16, 256), (256, 256), (256, 256), (256, 128))):
        w = flat[at:at + nin * nout].view(nin, nout)
        x = x @ w + flat[at + nin * nout:at + nin * nout + nout]
        at += nin * nout + nout
        if n < 3:
            x = torch.nn.functional.silu(x)
    square = (x - targets.double()).square().sum()
    grads, = torch.autograd.grad(square / targets.numel(), flat)
    return {"grads": grads, "loss": square.detach().reshape(1)}
