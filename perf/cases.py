"""The work that programs using this library have it do, as measurable cases.

Each case is one call of a public entry point (`Plan.execute`, `Plan.power_spectrum`,
`Batch.execute`) on device-resident input, with the plan, its workspace and the output buffer kept
between calls as a search pipeline keeps them.  The sizes are those of this repository's own
workloads (`workloads/`) or generic ones of the same ranges: from one 64-channel circular
transform of 4096 samples, where launches and latency count, to a 1024-channel 8-bit observation
of 2^20 samples dedispersed at 2048 trial DMs.

A case is a dict:
  kind       "execute" (dedispersed series), "power" (power spectra) or "batch" (several beams)
  n_chan, n_samp, n_dm, log_len (FFT length L = 2^log_len), single (one circular transform)
  band       lower and upper band edge in MHz as f_lo, f_hi; tsamp is 64 us everywhere
  dm_max     trial DMs run from 0 to dm_max; dms = "uniform" (equal steps) or "stepped" (three
             runs with steps 1 : 2 : 4, as a search that widens its steps with DM uses)
  input      "f32" (channel-major float32) or "u8" (time-major 8-bit)
  precision  "fp32", "fp16_split", "bf16_split";  mode "exact" or "round" (nearest-sample delays)
  downsample largest output down-sampling factor (1: none), factors from the smearing
  beams      number of beams (batch): beam i has its own shape, drawn from beam_seed
"""
import math

import numpy as np
import torch

import paper_2110_03482_amd as fdd

TSAMP = 64e-6
K_DM = 4.148808e3
COST_MAX = 1.3e13          # 8 n_dm n_chan bins chunks of the largest drawn case


def _case(name, kind, n_chan, n_samp, n_dm, log_len, *, single=False, f_lo=1250.0, f_hi=1550.0, dm_max=1000.0,
          dms="uniform", input="f32", precision="fp32", mode="exact", downsample=1, beams=1, beam_seed=0):
    c = dict(kind=kind, n_chan=n_chan, n_samp=n_samp, n_dm=n_dm, log_len=log_len, single=single, f_lo=f_lo, f_hi=f_hi,
             dm_max=dm_max, dms=dms, input=input, precision=precision, mode=mode, downsample=downsample, beams=beams,
             beam_seed=beam_seed)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one circular transform per channel, as a quick-look or a unit of a
        # streaming program; launches and latency count.
        _case("small_f32", "execute", 64, 4096, 64, 12, single=True, f_lo=1350.0, f_hi=1450.0, dm_max=63.0),
        # The same band with a fine DM grid in split precision (the precision sweep's shape).
        _case("fine_grid_f16", "execute", 64, 4096, 2048, 12, single=True, f_lo=1350.0, f_hi=1450.0, dm_max=63.97,
              precision="fp16_split"),
        # An ordinary float observation with no size a power of two.
        _case("odd_f32", "execute", 200, 100001, 301, 13, dm_max=90.0),
        # A short 8-bit observation in bfloat16 split precision, odd sizes.
        _case("odd_u8_bf16", "execute", 336, 150007, 700, 14, dm_max=220.0, input="u8", precision="bf16_split"),
        # One beam of a multi-beam receiver.
        _case("beam_f32", "execute", 512, 1 << 18, 1024, 16),
        # Nearest-sample delays (results equal to time-domain shift-and-sum) on 8-bit data.
        _case("round_u8_f32", "execute", 1024, 1 << 18, 1024, 16, input="u8", mode="round"),
        # A DM list whose steps widen with DM, split precision.
        _case("stepped_u8_f16", "execute", 512, 1 << 18, 1500, 16, input="u8", dms="stepped", precision="fp16_split"),
        # The paper-shaped observation (1024 channels, 2^20 8-bit samples, 2048 trials): FP32,
        # FP16 split, and with the output down-sampled where the smearing allows it.
        _case("paper_u8_f32", "execute", 1024, 1 << 20, 2048, 16, input="u8"),
        _case("paper_u8_f16", "execute", 1024, 1 << 20, 2048, 16, input="u8", precision="fp16_split"),
        _case("paper_u8_downsampled", "execute", 1024, 1 << 20, 2048, 16, input="u8", downsample=16),
        # Periodicity search: power spectra of one unchunked 2^22-sample transform.
        _case("periodicity_f16", "power", 512, 1 << 22, 2048, 22, single=True, dm_max=500.0, precision="fp16_split"),
        # Beams of uneven shapes in one batched call.
        _case("batch_8_beams", "batch", 1024, 1 << 18, 2048, 16, beams=8, beam_seed=3),
    ]


# ------------------------------------------------------------------------------ problem set-up

def _freqs(case):
    bw = (case["f_hi"] - case["f_lo"]) / case["n_chan"]
    return case["f_lo"] + (np.arange(case["n_chan"], dtype=np.float64) + 0.5) * bw


def _dms(case):
    n, top = case["n_dm"], case["dm_max"]
    if case["dms"] == "uniform" or n < 8:
        return np.linspace(0.0, top, n) if n > 1 else np.zeros(1)
    steps = np.ones(n - 1)
    steps[n // 3:] = 2.0
    steps[2 * n // 3:] = 4.0
    d = np.concatenate([[0.0], np.cumsum(steps)])
    return d * (top / d[-1])


def _kappa(case):
    f, ref = _freqs(case), case["f_hi"]
    return (K_DM * (1.0 / (f * f) - 1.0 / (ref * ref))) / TSAMP


def _factors(case):
    if case["downsample"] <= 1:
        return None
    return fdd.fdd_smearing_factors(_freqs(case), TSAMP, _dms(case), case["downsample"])


def _split(case):
    """The beams of a batch as cases of their own (one, the case itself, otherwise)."""
    if case["kind"] != "batch":
        return [case]
    rng = np.random.default_rng(case["beam_seed"])
    out = []
    for _ in range(case["beams"]):
        n_chan = case["n_chan"] >> int(rng.integers(0, 3))
        n_samp = case["n_samp"] >> int(rng.integers(0, 3))
        n_dm = case["n_dm"] >> int(rng.integers(0, 3))
        out.append(dict(case, kind="execute", n_chan=n_chan, n_samp=n_samp, n_dm=n_dm))
    return out


def _geometry(case):
    """(L, stride, chunks) of the overlap-save split, as the planner documents it."""
    L = 1 << case["log_len"]
    if case["single"]:
        return L, L, 1
    need = int(math.ceil(float(_dms(case).max()) * float(_kappa(case).max())))
    f = _factors(case)
    top = int(f.max()) if f is not None else 1
    stride = (L - need) // top * top
    return L, stride, -(-case["n_samp"] // stride)


def _data(case, seed):
    """Noise with a bright dispersed pulse, made on the GPU from the seed."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, c = case["n_samp"], case["n_chan"]
    d = torch.from_numpy(np.floor(0.4 * case["dm_max"] * _kappa(case) + 0.5).astype(np.int64)).cuda()
    t = (n // 3 + d) % n
    ch = torch.arange(c, device="cuda")
    if case["input"] == "u8":
        x = torch.empty((n, c), dtype=torch.uint8, device="cuda")
        rows = max(1, (1 << 26) // c)
        for r in range(0, n, rows):
            v = torch.randn((min(rows, n - r), c), generator=g, device="cuda")
            x[r:r + rows] = v.mul_(16.0).add_(128.0).round_().clamp_(0.0, 255.0).to(torch.uint8)
        x[t, ch] = 255
        return x
    x = torch.randn((c, n), generator=g, device="cuda")
    x[ch, t] += 5.0
    return x


def _plan(case, workspace=True):
    return fdd.Plan(_freqs(case), case["f_hi"], TSAMP, _dms(case), case["n_samp"], 1 << case["log_len"],
                    single_chunk=case["single"], input=case["input"], precision=case["precision"], mode=case["mode"],
                    power_only=case["kind"] == "power", downsample=_factors(case), workspace=workspace,
                    device=torch.device("cuda", torch.cuda.current_device()))


def prepare(case, seed):
    parts = _split(case)
    plans = [_plan(p, workspace=case["kind"] != "batch") for p in parts]
    xs = [_data(p, 1000 * seed + i) for i, p in enumerate(parts)]
    outs = []
    for p, pl in zip(parts, plans):
        if case["kind"] == "power":
            shape = (p["n_dm"], 1 << (p["log_len"] - 1))
        elif pl.downsampled:
            shape = (int(pl.geometry.out_samples),)
        else:
            shape = (p["n_dm"], p["n_samp"])
        outs.append(torch.empty(shape, dtype=torch.float32, device="cuda"))
    batch = fdd.Batch(plans) if case["kind"] == "batch" else None
    return dict(kind=case["kind"], plans=plans, x=xs, out=outs, batch=batch)


def run(state):
    if state["kind"] == "batch":
        return state["batch"].execute(state["x"], state["out"])
    plan, x, out = state["plans"][0], state["x"][0], state["out"][0]
    if state["kind"] == "power":
        return plan.power_spectrum(x, out)
    return plan.execute(x, out)


# ------------------------------------------------------------------------------ work and truth

def work(case):
    """Input read once and output written once; real transforms at 2.5 n log2 n.  The phasor sum of
    exact delays on equally spaced trials is a non-uniform discrete Fourier transform along the
    trial axis, counted as a fast one, 5 n log2 n with n = max(n_dm, n_chan) per bin and chunk;
    nearest-sample delays and unequal steps have no such structure and count the matrix product,
    8 n_dm n_chan.  Power spectra add 3 per value."""
    nbytes = flops = 0.0
    for p in _split(case):
        L, _, chunks = _geometry(p)
        f = _factors(p)
        d = np.ones(p["n_dm"]) if f is None else f.astype(np.float64)
        nbytes += p["n_chan"] * p["n_samp"] * (1 if p["input"] == "u8" else 4)
        flops += 2.5 * L * math.log2(L) * p["n_chan"] * chunks
        if p["kind"] == "power":
            nbytes += 4.0 * p["n_dm"] * (L // 2)
            flops += 3.0 * p["n_dm"] * (L // 2)
        else:
            nbytes += 4.0 * float(np.sum(np.ceil(p["n_samp"] / d)))
            flops += float(np.sum(2.5 * (L / d) * np.log2(L / d))) * chunks
        bins = float(np.sum(L / (2.0 * d))) / p["n_dm"]        # mean bins per trial
        n = max(p["n_dm"], p["n_chan"])
        if p["mode"] == "exact" and p["dms"] == "uniform":
            flops += 5.0 * n * math.log2(max(2, n)) * bins * chunks
        else:
            flops += 8.0 * p["n_dm"] * p["n_chan"] * bins * chunks
    return {"bytes": nbytes, "flops": flops}


def _exact_one(case, x):
    """Eqs. 3, 4, 7 and 6 in float64 with torch's transforms and matrix products."""
    L, stride, chunks = _geometry(case)
    n, c, nd = case["n_samp"], case["n_chan"], case["n_dm"]
    dev = x.device
    tau = torch.from_numpy(np.outer(_dms(case), _kappa(case))).to(dev)              # samples
    if case["mode"] == "round":
        tau = torch.floor(tau + 0.5)
    frac = torch.remainder(tau, float(L)) / L                                       # turns per bin
    xt = x.t() if case["input"] == "u8" else x
    nb = L // 2 + 1
    f = _factors(case)
    fac = np.ones(nd, dtype=np.int64) if f is None else f.astype(np.int64)
    runs = [(int(j[0]), int(j[-1]) + 1) for j in np.split(np.arange(nd), np.flatnonzero(np.diff(fac)) + 1)]
    X = torch.empty((nb, c, chunks), dtype=torch.complex128, device=dev)
    for k in range(chunks):
        s = k * stride
        w = min(L, n - s)
        X[:, :, k] = torch.fft.rfft(xt[:, s:s + w].to(torch.float64), n=L).t()
    if case["kind"] == "power":
        out = torch.empty((nd, L // 2), dtype=torch.float64, device=dev)
    else:
        out = torch.empty(int(sum((b - a) * -(-n // int(fac[a])) for a, b in runs)), dtype=torch.float64, device=dev)
    at = 0
    for a, b in runs:
        d = int(fac[a])
        M = L // d
        cols = M // 2 + (0 if case["kind"] == "power" else 1)
        Y = torch.empty((b - a, chunks, cols), dtype=torch.complex128, device=dev)
        block = max(1, (1 << 27) // ((b - a) * c))
        for f0 in range(0, cols, block):
            ff = torch.arange(f0, min(cols, f0 + block), dtype=torch.float64, device=dev)
            ph = torch.remainder(ff[:, None, None] * frac[None, a:b], 1.0).mul_(2.0 * math.pi)
            W = torch.polar(torch.ones_like(ph), ph)
            Y[:, :, f0:f0 + block] = torch.matmul(W, X[f0:f0 + W.shape[0]]).permute(1, 2, 0)
        if case["kind"] == "power":
            out[a:b] = Y[:, 0].real.square() + Y[:, 0].imag.square()
            continue
        no = -(-n // d)
        row = out[at:at + (b - a) * no].view(b - a, no)
        at += (b - a) * no
        Y[:, :, 0].imag.zero_()
        Y[:, :, M // 2].imag.zero_()
        keep = stride // d
        for k in range(chunks):
            w = min(no, keep) if case["single"] else min(keep, no - k * keep)
            row[:, k * keep:k * keep + w] = (torch.fft.irfft(Y[:, k], n=M) * (M / L))[:, :w]
    return out if case["kind"] == "power" or f is not None else out.view(nd, n)


def _direct_cost(case):
    L, _, chunks = _geometry(case)
    return 8.0 * case["n_dm"] * case["n_chan"] * (L / 2) * chunks


def exact(case, seed):
    parts = _split(case)
    # the phasors of 2^21 bins take minutes in float64
    if sum(_direct_cost(p) for p in parts) > 2e13 or any(p["n_dm"] * p["n_chan"] << p["log_len"] > 2e11 for p in parts):
        return None
    res = [_exact_one(p, _data(p, 1000 * seed + i)) for i, p in enumerate(parts)]
    return res if case["kind"] == "batch" else res[0]


# ------------------------------------------------------------------------------ further cases

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["execute"] * 7 + ["power"] * 2 + ["batch"])
        n_chan = _log_int(rng, 32, 1024)
        n_dm = _log_int(rng, 32, 2048)
        precision = rng.choice(["fp32", "fp32", "fp16_split", "bf16_split"])
        mode = rng.choice(["exact"] * 4 + ["round"])
        dms = rng.choice(["uniform"] * 4 + ["stepped"])
        inp = rng.choice(["f32", "u8"])
        if kind == "power":
            log_len = rng.randint(12, 20)
            L = 1 << log_len
            case = _case("", kind, n_chan, rng.choice([L, rng.randint(L // 2 + 1, L)]), n_dm, log_len, single=True,
                         dm_max=1.0, dms=dms, input=inp, precision=precision, mode="exact")
        elif kind == "batch":
            case = _case("", kind, 4 * max(16, n_chan // 4), _log_int(rng, 1 << 15, 1 << 18), max(128, n_dm), 16,
                         dm_max=1.0, beams=rng.randint(3, 8), beam_seed=rng.randint(0, 1 << 20), precision=precision)
        else:
            log_len = rng.randint(12, 16)
            single = rng.random() < 0.2
            n_samp = rng.randint((1 << log_len) // 2 + 1, 1 << log_len) if single else _log_int(rng, 1 << 14, 1 << 20)
            case = _case("", kind, n_chan, n_samp, n_dm, log_len, single=single, dm_max=1.0, dms=dms, input=inp,
                         precision=precision, mode=mode,
                         downsample=1 if single else rng.choice([1, 1, 1, 8]))
        # the largest delay takes between a tenth and four tenths of the transform, of 2^16 at most
        top = float(max(_kappa(p).max() for p in _split(case)))
        case["dm_max"] = round(rng.uniform(0.1, 0.4) * (1 << min(16, case["log_len"])) / top, 3)
        parts = _split(case)
        cost = sum(_direct_cost(p) for p in parts)
        values = sum(p["n_dm"] * p["n_samp"] + p["n_chan"] * p["n_samp"] for p in parts)
        if cost <= COST_MAX / 4 and values <= 1.2e9 and all(_geometry(p)[2] <= 400 for p in parts):
            return case
