"""Performance cases of the correlator library: what a user's program has it do, through the
public binding (``paper_1801_04834_amd.binding`` / ``.autograd``), over the range of sizes it
serves: observations of 2 to 80 stations, 1 to 128 subbands, blocks of a few dozen to 3072
channel samples, 8-bit / 16-bit / float samples, the three correlator modes, coarse delay with
lost-sample flags, the beamformer (Stokes I or IQUV, voltages, incoherent beam), the
output-resolution transform of its voltages, and the differentiable gains.

A case is a dict of plain values; ``kind`` names the entry point:

``correlate``   Plan.correlate: one block of the FX chain (steady state of an observation)
``ex``          Plan.correlate_ex: the same with coarse delays, lost-sample flags and weights
``noalloc``     correlate_noalloc: one block without a plan, history passed by the caller
``channelize``  Plan.channelize: the F stage into a caller buffer (two-stream schedule)
``xstage``      Plan.correlate_channelized: the X stage on a caller buffer (two-stream schedule)
``beamform``    Plan.beamform: F stage + beamformer at 256 channels
``transform``   Plan.beam_transform: beam voltages from 256 to c_out channels per subband
``gains``       autograd.gain_correlate, forward and backward

Streams are taken in their steady state: the plan has already seen one block, and every pass
feeds the block again, so the carried history is the block's own tail (the input is a periodic
stream) and every pass of a state gives the same result.
"""

import math

import numpy as np
import torch

from paper_1801_04834_amd import autograd, binding

SAMPLE_RATE = 195312.5                       # subband sample rate (Hz): 5.12 us samples
TAPS = 16
TYPES = {"ci8": binding.CI8, "ci16": binding.CI16, "cf32": binding.CF32}
MODES = {"fp32": binding.X_FP32, "fp16": binding.X_FP16_SPLIT, "int8": binding.X_INT8}
DTYPES = {"ci8": torch.int8, "ci16": torch.int16, "cf32": torch.float32}
SIGMA = {"ci8": 16.0, "ci16": 64.0, "cf32": 64.0}
SAMPLE_BYTES = {"ci8": 2, "ci16": 4, "cf32": 8}
CHAN_BYTES = {"fp32": 8, "fp16": 8, "int8": 2}
GUARD = 2048                                 # extra samples per row for the coarse delay


def listed():
    return [
        # the smallest call: a short block of a few stations without a plan (a serving loop or
        # stream capture that must not allocate); launches and latency count
        dict(name="noalloc_8st_2sb_short", kind="noalloc", S=8, SB=2, C=64, n_c=512, st="ci16", mode="fp16"),
        # one subband of a small array, the plain single-precision form, a full ~1 s block: what
        # a commissioning run looks at first
        dict(name="plain_8st_1sb_fp32", kind="correlate", S=8, SB=1, C=64, n_c=3072, st="ci16", mode="fp32"),
        # one of several concurrent observations of the streaming service: 24 stations, 32 subbands
        dict(name="obs_24st_32sb", kind="correlate", S=24, SB=32, C=64, n_c=3072, st="ci16", mode="fp16"),
        # a full GPU share of a 16-bit observation with every station: the headline block
        dict(name="share_76st_64sb", kind="correlate", S=76, SB=64, C=64, n_c=3072, st="ci16", mode="fp16"),
        # the 8-bit mode of the same array: twice the subbands, int8 matrix products
        dict(name="int8_76st_128sb", kind="correlate", S=76, SB=128, C=64, n_c=3072, st="ci8", mode="int8"),
        # an observation as it really arrives: odd station and subband counts, a ragged block,
        # coarse delays into guarded rows, 0.2 % of the packets lost, weights written
        dict(name="flagged_37st_11sb_ragged", kind="ex", S=37, SB=11, C=64, n_c=1501, st="ci16", mode="fp16"),
        # float samples through the plain single-precision form (validation against recorded or
        # simulated voltages), a mid-sized array
        dict(name="float_60st_8sb_fp32", kind="correlate", S=60, SB=8, C=64, n_c=3072, st="cf32", mode="fp32"),
        # the X stage alone on a channelised buffer of the caller (F of the next block runs on
        # another stream), one subband at the finest resolution, 256 channels
        dict(name="xstage_48st_1sb_256ch", kind="xstage", S=48, SB=1, C=256, n_c=768, st="ci16", mode="fp16"),
        # the beamformer's survey setting: 127 tied-array beams, Stokes I over 16 samples + incoherent
        dict(name="beams_48st_61sb_I", kind="beamform", S=48, SB=61, C=256, n_c=768, st="ci16", mode="fp16", NB=127, NS=1,
             n_int=16, volt=0, inc=True),
        # a few full-polarisation beams at full time resolution with their complex voltages, a
        # small array and a ragged block (pulsar timing on a few subbands)
        dict(name="beams_13st_5sb_iquv_volt", kind="beamform", S=13, SB=5, C=256, n_c=300, st="ci16", mode="fp16", NB=40,
             NS=4, n_int=1, volt=48, inc=False),
        # beam voltages back to one channel per subband (time series, full Stokes over 64 samples)
        dict(name="transform_61beams_c1_iquv", kind="transform", SB=8, n_c=768, NB=61, stride=64, c_out=1, NS=4, n_int=64,
             volt=False),
        # one step of a gain solver: gain-applied visibilities and the gradient of the gains
        dict(name="gains_48st_16sb", kind="gains", S=48, SB=16),
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], uniform in its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["correlate", "correlate", "correlate", "ex", "noalloc", "channelize", "xstage", "beamform", "beamform",
                       "transform", "gains"])
    if kind == "gains":
        return dict(kind=kind, S=rng.randint(2, 80), SB=_log(rng, 1, 32))
    if kind == "transform":
        NB = _log(rng, 1, 127)
        c_out = rng.choice([1, 2, 4, 8, 16])
        c = dict(kind=kind, SB=_log(rng, 1, 16), n_c=_log(rng, 32, 768), NB=NB, stride=rng.choice([0, (NB + 15) // 16 * 16]),
                 c_out=c_out, NS=rng.choice([1, 4]), n_int=1 << rng.randint(0, int(math.log2(256 // c_out))), volt=rng.random() < 0.4)
        return c
    if kind == "beamform":
        C = rng.choice([256, 256, 256, 64])
        n_int = rng.choice([1, 4, 8, 16, 32, 96])
        c = dict(kind=kind, S=rng.randint(2, 48), SB=_log(rng, 1, 32), C=C, n_c=max(1, _log(rng, 48, 196608 // C) // n_int) * n_int,
                 st=rng.choice(["ci16", "ci16", "ci8"]), mode="fp16", NB=_log(rng, 1, 127), NS=rng.choice([1, 4]), n_int=n_int,
                 volt=0, inc=rng.random() < 0.5)
        if rng.random() < 0.35:
            c["volt"] = rng.choice([c["NB"], (c["NB"] + 15) // 16 * 16])
        return c
    st, mode = rng.choice([("ci16", "fp16"), ("ci16", "fp16"), ("ci16", "fp32"), ("ci8", "int8"), ("ci8", "fp16"), ("cf32", "fp32")])
    C = rng.choice([64, 64, 64, 256])
    c = dict(kind=kind, S=rng.randint(2, 76), SB=_log(rng, 1, 64), C=C, n_c=_log(rng, 48, 196608 // C), st=st, mode=mode)
    if kind == "noalloc":                       # its intermediate data live in a fixed 256 MiB
        c["S"], c["SB"] = rng.randint(2, 24), _log(rng, 1, 4)
        c["n_c"] = _log(rng, 48, 131072 // C)
    if mode == "fp32":                          # keeps the single-precision form below the largest listed case
        c["SB"] = min(c["SB"], 16)
    return c


# ---- settings and inputs -----------------------------------------------------------------

def _fir(C):
    """Blackman-windowed sinc prototype of a C-channel, 16-tap filter bank, sum 1 (float32)."""
    m = np.arange(TAPS * C, dtype=np.float64)
    h = np.sinc((m - (TAPS * C - 1) / 2.0) / C) * np.blackman(TAPS * C)
    return (h / h.sum()).astype(np.float32)


def _bandpass(C):
    c = np.arange(C, dtype=np.float64)
    return (1.0 + 0.05 * np.cos(2 * np.pi * (c - C / 2) / C)).astype(np.float32)


def _freqs(SB):
    return 100e6 + (256 + np.arange(SB, dtype=np.float64)) * SAMPLE_RATE


def _gain(C, sigma):
    return float(np.float32(16.0 / (sigma * math.sqrt(float(np.sum(_fir(C).astype(np.float64) ** 2))))))


def _settings(case):
    C = case["C"]
    return dict(n_stations=case["S"], n_subbands=case["SB"], samples_per_block=C * case["n_c"], sample_type=TYPES[case["st"]],
                x_mode=MODES[case["mode"]], fir=_fir(C), subband_freqs=_freqs(case["SB"]), sample_rate=SAMPLE_RATE,
                bandpass=_bandpass(C), requant_gain=_gain(C, SIGMA[case["st"]]) if case["mode"] == "int8" else 1.0,
                fp16_prescale_log2=-1 if case["mode"] == "fp16" else 0, n_channels=C)


def _generator(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + what)
    return g


def _delays(case, seed):
    rng = np.random.default_rng([int(seed), 1])
    t0 = rng.uniform(-5e-6, 5e-6, case["S"])
    return np.stack([t0, t0 + rng.uniform(-25e-9, 25e-9, case["S"])], axis=1)


def _samples(case, seed, row):
    """Station noise [S][2][SB][row][2] in the storage type, on the GPU."""
    g = _generator(seed, 0)
    x = torch.empty((case["S"], 2, case["SB"], row, 2), dtype=DTYPES[case["st"]], device="cuda")
    flat, step = x.view(-1), 1 << 28
    lim = {"ci8": 127, "ci16": 32767}.get(case["st"])
    for i in range(0, flat.numel(), step):
        v = torch.randn(min(step, flat.numel() - i), generator=g, device="cuda") * SIGMA[case["st"]]
        flat[i:i + step] = v if lim is None else v.round_().clamp_(-lim, lim)
    return x


def _lost(case, seed, row):
    """Lost 16-sample packets (0.2 %) as a bool tensor [S][SB][row] on the GPU."""
    g = _generator(seed, 1)
    packets = torch.rand((case["S"], case["SB"], (row + 15) // 16), generator=g, device="cuda") < 0.002
    return packets.repeat_interleave(16, dim=2)[..., :row]


def _flag_words(lost):
    S, SB, row = lost.shape
    words = (row + 31) // 32
    bits = torch.zeros((S, SB, words * 32), dtype=torch.int64, device="cuda")
    bits[..., :row] = lost
    w = (bits.view(S, SB, words, 32) << torch.arange(32, device="cuda")).sum(-1)
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _coarse(case, seed):
    return np.random.default_rng([int(seed), 2]).integers(0, GUARD + 1, case["S"]).astype(np.int32)


def _dtau(case, seed):
    d = np.random.default_rng([int(seed), 3]).uniform(-2e-6, 2e-6, (case["NB"], case["S"]))
    return torch.from_numpy(d).cuda()


def _complex_noise(shape, seed, what):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=_generator(seed, what), device="cuda"))


def _gain_inputs(case, seed):
    S, SB, C = case["S"], case["SB"], 64
    B = S * (S + 1) // 2
    vis0 = _complex_noise((SB, C, B, 4), seed, 4) * 3072.0
    gains = 1.0 + 0.1 * _complex_noise((SB, C, 2 * S), seed, 5)
    grad = _complex_noise((SB, C, B, 4), seed, 6)
    return vis0, gains, grad


def _beam_voltages(case, seed):
    nbs = case["stride"] or case["NB"]
    return torch.randn((case["SB"], 256, case["n_c"], 2, nbs, 2), generator=_generator(seed, 7), device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case}
    if kind == "gains":
        s["plan"] = binding.Plan(**_settings(dict(case, C=64, n_c=64, st="ci16", mode="fp16")))
        s["vis0"], gains, s["grad"] = _gain_inputs(case, seed)
        s["gains"] = gains.requires_grad_()
        return s
    if kind == "transform":
        s["plan"] = binding.Plan(**_settings(dict(case, S=1, C=256, st="ci16", mode="fp16")))
        s["voltages"] = _beam_voltages(case, seed)
        ov, os_ = s["plan"].transform_shapes(case["NB"], case["c_out"], case["NS"], case["n_int"], case["stride"])
        s["out_voltages"] = torch.zeros(ov, device="cuda") if case["volt"] else None
        s["out_stokes"] = torch.empty(os_, device="cuda")
        return s
    kw = _settings(case)
    N = kw["samples_per_block"]
    s["delays"] = _delays(case, seed)
    s["x"] = _samples(case, seed, N + (GUARD if kind == "ex" else 0))
    if kind == "noalloc":
        s["settings"] = kw
        B = case["S"] * (case["S"] + 1) // 2
        s["vis"] = torch.empty((case["SB"], case["C"], B, 4, 2), dtype=torch.int32 if case["mode"] == "int8" else torch.float32,
                               device="cuda")
        hist = (TAPS - 1) * case["C"]
        head = torch.cat([s["x"]] * (1 + hist // N), dim=3)[:, :, :, -hist:]      # the periodic stream before the block
        s["hist_in"] = head.reshape(case["S"] * 2 * case["SB"], hist, 2).contiguous()
        s["hist_out"] = torch.empty_like(s["hist_in"])
        return s
    plan = s["plan"] = binding.Plan(**kw)
    if kind == "ex":
        s["coarse"] = _coarse(case, seed)
        s["flags"] = _flag_words(_lost(case, seed, N + GUARD))
        s["weights"] = torch.empty(plan.weights_shape(), dtype=torch.int32, device="cuda")
    if kind in ("correlate", "ex", "xstage"):
        s["vis"] = plan.empty_vis()
    if kind in ("channelize", "xstage"):
        s["chan"] = plan.empty_chan()
    if kind == "xstage":
        plan.channelize(s["x"], s["delays"], out=s["chan"])
        plan.channelize(s.pop("x"), s["delays"], out=s["chan"])
        return s
    if kind == "beamform":
        s["dtau"] = _dtau(case, seed)
        cs, vs, is_ = plan.beam_shapes(case["NB"], case["NS"], case["n_int"], case["volt"])
        s["coherent"] = torch.empty(cs, device="cuda")
        s["voltages"] = torch.zeros(vs, device="cuda") if case["volt"] else None
        s["incoherent"] = torch.empty(is_, device="cuda") if case["inc"] else None
    for _ in range(1 + (TAPS - 2) // case["n_c"]):       # the blocks before: fill the carried history
        run(s)
    return s


def run(s):
    kind, c = s["kind"], s["case"]
    if kind == "gains":
        vis = autograd.gain_correlate(s["plan"], s["vis0"], s["gains"])
        (grad,) = torch.autograd.grad(vis, s["gains"], s["grad"])
        return {"vis": vis.detach(), "grad": grad}
    if kind == "transform":
        v, st = s["plan"].beam_transform(s["voltages"], c["c_out"], c["NS"], c["n_int"], out_voltages=s["out_voltages"],
                                         out_stokes=s["out_stokes"], n_beams=c["NB"])
        return {"voltages": None if v is None else v[..., :c["NB"], :], "stokes": st}
    if kind == "noalloc":
        binding.correlate_noalloc(s["x"], s["delays"], s["vis"], hist_in=s["hist_in"], hist_out=s["hist_out"], **s["settings"])
        return {"vis": s["vis"], "history": s["hist_out"]}
    if kind == "channelize":
        return {"chan": s["plan"].channelize(s["x"], s["delays"], out=s["chan"])}
    if kind == "xstage":
        return {"vis": s["plan"].correlate_channelized(s["chan"], out=s["vis"])}
    if kind == "ex":
        s["plan"].correlate_ex(s["x"], s["delays"], coarse=s["coarse"], flags=s["flags"], weights=s["weights"], out=s["vis"])
        return {"vis": s["vis"], "weights": s["weights"]}
    if kind == "beamform":
        co, vo, inc = s["plan"].beamform(s["x"], s["delays"], s["dtau"], c["NS"], c["n_int"], coherent=s["coherent"],
                                         voltages=s["voltages"], incoherent=s["incoherent"])
        return {"coherent": co, "voltages": None if vo is None else vo[..., :c["NB"], :], "incoherent": inc}
    return {"vis": s["plan"].correlate(s["x"], s["delays"], out=s["vis"])}


# ---- work --------------------------------------------------------------------------------

def work(case):
    """Bytes: inputs once, outputs once (the channelised data between F and X stay inside).
    Flops: 2 T + 5 log2 C + 8 real operations per sample for the filter bank's FIR (2 x 2 T),
    FFT and rotation, 8 per complex multiply-add of the stored products."""
    kind = case["kind"]
    if kind == "gains":
        S, SB = case["S"], case["SB"]
        entries, g = SB * 64 * S * (S + 1) // 2 * 4, SB * 64 * 2 * S
        return {"bytes": 8.0 * (4 * entries + 3 * g), "flops": 14.0 * entries + 32.0 * entries}
    if kind == "transform":
        G = case["n_c"] * 256 // case["c_out"]
        v = case["SB"] * 256 * case["n_c"] * 2 * case["NB"]
        st = case["SB"] * (G // case["n_int"]) * case["c_out"] * case["NS"] * case["NB"]
        return {"bytes": 8.0 * v * (2 if case["volt"] else 1) + 4.0 * st,
                "flops": v * (5.0 * 8 + 5.0 * math.log2(case["c_out"]) + 6 + 4)}
    S, SB, C, n_c = case["S"], case["SB"], case["C"], case["n_c"]
    M, B = 2 * S, S * (S + 1) // 2
    samples = float(M * SB * C * n_c)
    x_in = samples * SAMPLE_BYTES[case["st"]]
    f_flops = samples * (4 * TAPS + 5 * math.log2(C) + 8)
    vis = SB * C * B * 4 * 8.0
    x_flops = 8.0 * B * 4 * SB * C * n_c
    chan = SB * C * M * ((n_c + 31) // 32 * 32) * float(CHAN_BYTES[case["mode"]])
    if kind == "channelize":
        return {"bytes": x_in + chan, "flops": f_flops}
    if kind == "xstage":
        return {"bytes": chan + vis, "flops": x_flops}
    if kind == "beamform":
        NB, n_out = case["NB"], n_c // case["n_int"]
        out = 4.0 * SB * C * n_out * case["NS"] * (NB + (1 if case["inc"] else 0))
        out += 16.0 * SB * C * n_c * NB if case["volt"] else 0.0
        return {"bytes": x_in + out, "flops": f_flops + 8.0 * NB * samples}
    extra = 0.0
    if kind == "ex":
        extra = S * SB * C * n_c / 8.0 + 4.0 * SB * B
    if kind == "noalloc":
        extra = 2.0 * M * SB * (TAPS - 1) * C * SAMPLE_BYTES[case["st"]]
    return {"bytes": x_in + vis + extra, "flops": f_flops + x_flops}


# ---- the same results in 64 bits -----------------------------------------------------------

def _exact_channels(case, seed, x, sb, lost=None, coarse=None):
    """Channelised samples of subband sb [S, 2, n_c, C] in complex128: filter bank over the
    periodic stream, delay phase, bandpass, lost samples' channel samples zero."""
    S, C, n_c = case["S"], case["C"], case["n_c"]
    N = C * n_c
    if coarse is None:
        t = x[:, :, sb, :N].double()
    else:
        t = torch.stack([x[s, :, sb, int(g):int(g) + N] for s, g in enumerate(coarse)]).double()
    t = torch.view_as_complex(t).view(S, 2, n_c, C)
    h = torch.from_numpy(_fir(C).astype(np.float64)).cuda().view(TAPS, C)
    y = torch.zeros_like(t)
    for k in range(TAPS):                                  # row j - T + 1 + k of the periodic stream
        y += h[k] * torch.roll(t, TAPS - 1 - k, dims=2)
    p = torch.arange(C, device="cuda", dtype=torch.float64)
    turns = torch.remainder(p[:, None] * (p[None, :] - C // 2), C) / C          # channel c holds bin c - C/2
    X = y.view(-1, C) @ torch.polar(torch.ones_like(turns), -2 * math.pi * turns)
    X = X.view(S, 2, n_c, C)
    f_c = _freqs(case["SB"])[sb] + (p - C / 2) * (SAMPLE_RATE / C)
    d = torch.from_numpy(_delays(case, seed)).cuda()
    j = torch.arange(n_c, device="cuda", dtype=torch.float64) / n_c
    cyc = (d[:, :1] + (d[:, 1:] - d[:, :1]) * j)[:, :, None] * f_c               # [S, n_c, C]
    cyc = cyc - cyc.round()
    b = torch.from_numpy(_bandpass(C).astype(np.float64)).cuda()
    X = X * (torch.polar(torch.ones_like(cyc), 2 * math.pi * cyc) * b)[:, None]
    if lost is not None:
        rows = torch.stack([lost[s, sb, int(g):int(g) + N] for s, g in enumerate(coarse)]).view(S, n_c, C).any(-1)
        bad = torch.zeros_like(rows)
        for k in range(TAPS):
            bad |= torch.roll(rows, k, dims=1)
        X[bad[:, None, :, None].expand_as(X)] = 0
        return X, bad
    return X, None


def _lower(S):
    s1 = np.concatenate([np.full(i + 1, i) for i in range(S)])
    s2 = np.concatenate([np.arange(i + 1) for i in range(S)])
    a = (2 * s1[:, None] + np.array([0, 0, 1, 1])[None]).astype(np.int64)
    b = (2 * s2[:, None] + np.array([0, 1, 0, 1])[None]).astype(np.int64)
    return torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()


def _exact_vis(Z, S):
    """[S, 2, n_c, C] -> [C, B, 4, 2]: sums over n_c of Z_a conj(Z_b), a >= b pairs."""
    C, n_c = Z.shape[3], Z.shape[2]
    z = Z.permute(3, 0, 1, 2).reshape(C, 2 * S, n_c).contiguous()
    full = torch.bmm(z, z.conj().transpose(1, 2).contiguous())
    a, b = _lower(S)
    return torch.view_as_real(full[:, a, b])


def _exact_stokes(X, Y, NS):
    xx, yy = X.abs() ** 2, Y.abs() ** 2
    if NS == 1:
        return (xx + yy)[..., None]
    xy = X * Y.conj()
    return torch.stack([xx + yy, xx - yy, 2 * xy.real, 2 * xy.imag], dim=-1)


def _exact_transform(case, seed):
    v = torch.view_as_complex(_beam_voltages(case, seed).double())[..., :case["NB"]]        # [SB, 256, n_c, 2, NB]
    SB, co, ni = case["SB"], case["c_out"], case["n_int"]
    k = torch.arange(256, device="cuda", dtype=torch.float64)
    turns = torch.remainder(k[:, None] * (k[None, :] - 128), 256) / 256
    E = torch.polar(torch.full_like(turns, 1.0 / 256), 2 * math.pi * turns)
    m = torch.arange(co, device="cuda", dtype=torch.float64)
    fturns = m[:, None] * (m[None, :] - co // 2) / co
    F = torch.polar(torch.ones_like(fturns), -2 * math.pi * fturns)                       # [m, c']
    G = case["n_c"] * 256 // co
    volts, stokes = [], []
    for sb in range(SB):
        u = (E @ v[sb].reshape(256, -1)).view(256, case["n_c"], 2, -1).permute(1, 0, 2, 3)   # [n_c, n, 2, NB]
        u = u.reshape(G, co, -1).permute(0, 2, 1).reshape(-1, co)
        O = (u @ F).view(G, 2, case["NB"], co).permute(0, 3, 1, 2)                            # [G, co, 2, NB]
        st = _exact_stokes(O[:, :, 0], O[:, :, 1], case["NS"]).view(G // ni, ni, co, case["NB"], case["NS"]).sum(1)
        stokes.append(st.permute(0, 1, 3, 2).contiguous())
        if case["volt"]:
            volts.append(torch.view_as_real(O.contiguous()))
    return {"voltages": torch.stack(volts) if case["volt"] else None, "stokes": torch.stack(stokes)}


def _exact_gains(case, seed):
    vis0, gains, grad = (t.to(torch.complex128) for t in _gain_inputs(case, seed))
    a, b = _lower(case["S"])
    ga, gb = gains[:, :, a], gains[:, :, b]
    g = torch.zeros_like(gains)
    shape = g.shape[:2] + (-1,)
    for idx, t in ((b, grad.conj() * ga * vis0), (a, grad * gb * vis0.conj())):
        t = t.reshape(shape)
        at = idx.reshape(-1).expand(t.shape)
        g += torch.complex(torch.zeros(g.shape, dtype=torch.float64, device="cuda").scatter_add_(2, at, t.real.contiguous()),
                           torch.zeros(g.shape, dtype=torch.float64, device="cuda").scatter_add_(2, at, t.imag.contiguous()))
    return {"vis": ga * gb.conj() * vis0, "grad": g}


def _exact_beams(case, seed, x):
    S, C, n_c, ni = case["S"], case["C"], case["n_c"], case["n_int"]
    dtau = _dtau(case, seed)
    p = torch.arange(C, device="cuda", dtype=torch.float64)
    out = {"coherent": [], "voltages": [], "incoherent": []}
    for sb in range(case["SB"]):
        Z, _ = _exact_channels(case, seed, x, sb)
        f_c = _freqs(case["SB"])[sb] + (p - C / 2) * (SAMPLE_RATE / C)
        cyc = f_c[:, None, None] * dtau
        W = torch.polar(torch.ones_like(cyc), 2 * math.pi * (cyc - cyc.round()))              # [C, NB, S]
        z = Z.permute(3, 0, 1, 2).reshape(C, S, 2 * n_c).contiguous()
        beams = torch.bmm(W, z).view(C, -1, 2, n_c).permute(0, 3, 2, 1)                     # [C, n_c, 2, NB]
        st = _exact_stokes(beams[:, :, 0], beams[:, :, 1], case["NS"]).view(C, n_c // ni, ni, -1, case["NS"]).sum(2)
        out["coherent"].append(st.permute(0, 1, 3, 2).contiguous())
        if case["volt"]:
            out["voltages"].append(torch.view_as_real(beams.contiguous()))
        if case["inc"]:
            inc = _exact_stokes(Z[:, 0], Z[:, 1], case["NS"]).sum(0)                         # [n_c, C, NS]
            out["incoherent"].append(inc.view(n_c // ni, ni, C, case["NS"]).sum(1).permute(1, 0, 2).contiguous())
    return {k: torch.stack(v) if v else None for k, v in out.items()}


def exact(case, seed):
    """What run() returns, computed in 64 bits.  8-bit requantised data (and the integer sums over
    them) are whole numbers and have no such value, nor have the split halves of the FP16 planes."""
    kind = case["kind"]
    if kind == "gains":
        return _exact_gains(case, seed)
    if kind == "transform":
        return _exact_transform(case, seed)
    if case["mode"] == "int8" or (kind == "channelize" and case["mode"] == "fp16"):
        return None
    N = case["C"] * case["n_c"]
    x = _samples(case, seed, N + (GUARD if kind == "ex" else 0))
    if kind == "beamform":
        return _exact_beams(case, seed, x)
    lost = _lost(case, seed, N + GUARD) if kind == "ex" else None
    coarse = _coarse(case, seed) if kind == "ex" else None
    vis, chan = [], []
    for sb in range(case["SB"]):
        Z, _ = _exact_channels(case, seed, x, sb, lost, coarse)
        if kind == "channelize":                            # [C, n_kb, M, 32, 2], zeros past the block
            S, C, n_c = case["S"], case["C"], case["n_c"]
            z = torch.zeros((C, 2 * S, (n_c + 31) // 32 * 32), dtype=torch.complex128, device="cuda")
            z[:, :, :n_c] = Z.permute(3, 0, 1, 2).reshape(C, 2 * S, n_c)
            chan.append(torch.view_as_real(z.view(C, 2 * S, -1, 32).permute(0, 2, 1, 3).contiguous()))
        else:
            vis.append(_exact_vis(Z, case["S"]))
    if kind == "channelize":
        return {"chan": torch.stack(chan)}
    return {"vis": torch.stack(vis), "weights": None} if kind == "ex" else {"vis": torch.stack(vis), "history": None} \
        if kind == "noalloc" else {"vis": torch.stack(vis)}
