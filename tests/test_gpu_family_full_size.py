"""The matrix-product families at full size (GPU), and the plans that take the grid form instead.

`Plan.kernel` names the family of a plan, which does the phasor sums where the plan has no grid form
(`Plan.grid == (0, 0)`): with unequal DM steps, short lists, plans that the planner's rule declines, and
FDD_GRID=0, which is how these tests ask for it.  A plan's default may be the grid form at the same
name, so a test of a family checks `Plan.grid` beside `Plan.kernel`.

The reference is float64 on the GPU: rows of Eqs. 3, 4, 7 and 6 by torch's transforms, a row at a
time.  Tolerances are those of the families' other tests (1e-5; bfloat16 split 1e-4).
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity import check_power, check_rows, raw_start

torch = pytest.importorskip("torch")
fdd = pytest.importorskip("paper_2110_03482_amd")

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp16_split": 1e-5, "bf16_split": 1e-4}
ROWS = [0, 921, 2047]
PULSES = ((100.0, 205), (450.0, 921), (900.0, 1842))          # DM and its trial


def plan_of(w, **kw):
    return fdd.Plan(w.freqs, w.ref_freq_mhz, w.tsamp_s, w.dms, w.n_samp, w.chunk_len, single_chunk=w.single_chunk,
                    input=w.input_kind, **kw)


def phases(w, row, bins):
    """exp(2 pi i f tau / L) of every channel and bin, complex128."""
    tau = torch.from_numpy(O.delays(w.dms[row:row + 1], w.freqs, w.ref_freq_mhz, w.tsamp_s)[0]).cuda()
    frac = torch.remainder(tau, float(w.chunk_len)) / w.chunk_len
    f = torch.arange(bins, dtype=torch.float64, device="cuda")
    ph = torch.remainder(frac[:, None] * f[None, :], 1.0).mul_(2.0 * np.pi)
    return torch.polar(torch.ones_like(ph), ph)


def exact_rows(w, x, g, rows, factors=None):
    """Dedispersed rows of a chunked plan; x is the 8-bit input on the device."""
    L, S, n = w.chunk_len, int(g.stride), w.n_samp
    d = {r: 1 if factors is None else int(factors[r]) for r in rows}
    out = {r: torch.zeros(-(-n // d[r]), dtype=torch.float64, device="cuda") for r in rows}
    turn = {r: phases(w, r, L // d[r] // 2 + 1) for r in rows}
    for k in range(int(g.n_chunks)):
        seg = x[k * S:k * S + L].t().to(torch.float64)
        X = torch.fft.rfft(seg, n=L, dim=1)
        for r in rows:
            M, keep = L // d[r], S // d[r]
            y = torch.fft.irfft((X[:, :M // 2 + 1] * turn[r]).sum(dim=0), n=M) / d[r]
            part = out[r][k * keep:(k + 1) * keep]
            part.copy_(y[:part.numel()])
    return [out[r].cpu().numpy() for r in rows]


@pytest.fixture(scope="module")
def paper():
    """1024 channels, 2048 trials (0..1000), 2^21 8-bit samples with three dispersed pulses; the shorter
    workload is its first half."""
    w = W.paper_shaped_u8()
    x = torch.empty((1 << 21, w.n_chan), dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    for r in range(0, x.shape[0], 1 << 18):
        v = torch.randn((1 << 18, w.n_chan), generator=gen, device="cuda")
        x[r:r + (1 << 18)] = v.mul_(16.0).add_(128.0).round_().clamp_(0.0, 255.0).to(torch.uint8)
    ch = torch.arange(w.n_chan, device="cuda")
    for i, (dm, _) in enumerate(PULSES):
        offs = O.nearest_sample(O.delays([dm], w.freqs, w.ref_freq_mhz, w.tsamp_s))[0]
        x[pulse_at(i) + torch.from_numpy(np.asarray(offs, dtype=np.int64)).cuda(), ch] = 255
    return x


def pulse_at(i):
    return (i + 1) << 18


def workload(chunks):
    w = W.paper_shaped_u8()
    w.n_samp = 1 << 20 if chunks == 21 else 1 << 21
    return w


@pytest.fixture(scope="module")
def truth(paper):
    done = {}

    def get(chunks, g):
        if chunks not in done:
            w = workload(chunks)
            done[chunks] = exact_rows(w, paper[:w.n_samp], g, ROWS)
        return done[chunks]
    return get


#            chunks, precision, kernel, FDD_GRID
FAMILIES = [(21, "fp32", "mfma_f32", "0"), (21, "fp16_split", "facw_f16_split", "0"),
            (21, "bf16_split", "facw_bf16_split", "0"), (42, "fp32", "mfma_f32", "0"), (21, "fp32", "mfma_f32", None)]


@pytest.mark.parametrize("case", FAMILIES, ids=[f"{c[1]}_{c[0]}chunks_{'grid' if c[3] is None else c[2]}" for c in FAMILIES])
def test_paper_shaped_rows(case, paper, truth, monkeypatch):
    chunks, precision, kernel, form = case
    if form is not None:
        monkeypatch.setenv("FDD_GRID", form)
    w = workload(chunks)
    print(f"full size {case}", flush=True)
    with plan_of(w, precision=precision) as p:
        g = p.geometry
        assert p.kernel == kernel and g.n_chunks == chunks
        assert p.grid == ((0, 0) if form == "0" else (1, 4096))
        y = p.execute(paper[:w.n_samp])
        torch.cuda.synchronize()
    check_rows(y[ROWS].cpu().numpy(), np.stack(truth(chunks, g)), TOL[precision],
               raw_from=raw_start("u8", w.n_samp, w.chunk_len, int(g.stride), int(g.n_chunks), False), label=f"full size {case}")
    assert bool(torch.isfinite(y).all())
    for i, (_, trial) in enumerate(PULSES):
        t0 = pulse_at(i)
        assert abs(int(y[:, t0 - 2:t0 + 3].amax(dim=1).argmax()) - trial) <= 2


def test_paper_shaped_downsampled_rows(paper, monkeypatch):
    monkeypatch.setenv("FDD_GRID", "0")
    w = workload(21)
    factors = fdd.fdd_smearing_factors(w.freqs, w.tsamp_s, w.dms, 16)
    rows = [0] + [int(np.flatnonzero(factors == d)[-1]) for d in np.unique(factors)]
    with plan_of(w, downsample=factors) as p:
        g = p.geometry
        assert p.kernel == "mfma_f32" and p.grid == (0, 0)
        y = p.rows(p.execute(paper[:w.n_samp]))
        torch.cuda.synchronize()
        y = [y[r].cpu().numpy() for r in rows]
    raw = [raw_start("u8", w.n_samp, w.chunk_len, int(g.stride), int(g.n_chunks), False, int(factors[r])) for r in rows]
    check_rows(y, exact_rows(w, paper[:w.n_samp], g, rows, factors), TOL["fp32"], raw_from=raw,
               label="full size, down-sampled")


def test_periodicity_rows(monkeypatch):
    """512 channels x 2^22 samples x 4096 trials (0..500), power spectra in float16 split."""
    monkeypatch.setenv("FDD_GRID", "0")
    w = W.periodicity()
    x = torch.randn((w.n_chan, w.n_samp), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    rows = [0, 467, 4095]
    with plan_of(w, precision="fp16_split", power_only=True) as p:
        assert p.kernel == "fac_f16_split" and p.grid == (0, 0)
        P = p.power_spectrum(x)
        torch.cuda.synchronize()
    assert bool(torch.isfinite(P).all())
    ref = torch.zeros((len(rows), w.n_samp // 2), dtype=torch.complex128, device="cuda")
    tau = torch.from_numpy(O.delays(w.dms[rows], w.freqs, w.ref_freq_mhz, w.tsamp_s)).cuda()
    f = torch.arange(w.n_samp // 2, dtype=torch.float64, device="cuda")
    for c in range(w.n_chan):
        X = torch.fft.rfft(x[c].to(torch.float64))[:-1]
        ph = torch.remainder(torch.remainder(tau[:, c:c + 1], float(w.chunk_len)) / w.chunk_len * f, 1.0).mul_(2.0 * np.pi)
        ref += X * torch.polar(torch.ones_like(ph), ph)
    check_power(P[rows].cpu().numpy(), (ref.real ** 2 + ref.imag ** 2).cpu().numpy(), TOL["fp16_split"],
                label="full size, periodicity")
