"""GPU parity of the grid form of the phasor sum (equal DM steps, exact delays).

FDD_GRID=1 makes a plan take the grid kernel wherever it applies, so that small shapes reach every
instance: grids of 2^8 .. 2^12 points, one and several columns per wave, several blocks of trials,
channel counts around the 64 of a batch, stepped DM lists (several runs), down-sampled segments,
long transforms, power spectra, and channels out of order.

Tolerance 2e-6 of the row norm (centred and per sample as tests/parity.py does): the forward and
inverse transforms keep within 4e-7 each, the grid adds at most 3e-7 of aliasing on the outermost
rows and 5e-7 of float32 rounding (12 butterfly stages and 8 weights).
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import paper_2110_03482_amd as fdd  # noqa: E402
import workloads as W  # noqa: E402
from parity import check_power, check_rows, raw_start  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 2e-6


def workload(seed, n_chan, n_samp, n_dm, L, single, kind, dm_max, steps=(1.0,)):
    w = W.tiny_random(seed, n_chan, n_samp, n_dm, L, single_chunk=single, input_kind=kind, dm_max=dm_max)
    d = np.concatenate([np.full(n, s) for s, n in zip(steps, np.diff(np.linspace(0, n_dm, len(steps) + 1).astype(int)))])
    d = np.concatenate([[0.0], np.cumsum(d[1:])])
    w = dataclasses.replace(w, dms=d * (dm_max / d[-1]))
    x = W.gaussian_u8(n_samp, n_chan, seed) if kind == "u8" else W.gaussian_f32(n_chan, n_samp, seed)
    return w, x


def plan_of(w, freqs=None, **kw):
    return fdd.Plan(w.freqs if freqs is None else freqs, w.ref_freq_mhz, w.tsamp_s, w.dms, w.n_samp, w.chunk_len,
                    single_chunk=w.single_chunk, input=w.input_kind, **kw)


#         channels, samples, trials, L, single, input, DM max, steps
CASES = [(64, 4096, 64, 4096, True, "f32", 20.0, (1.0,)),          # one column, one batch of channels
         (63, 9000, 127, 2048, False, "f32", 4.0, (1.0,)),         # 2^8 points, 16 columns per wave
         (65, 9000, 128, 2048, False, "u8", 4.0, (1.0,)),          # the most trials of 2^8 points
         (130, 30000, 129, 4096, False, "f32", 12.0, (1.0,)),      # 2^9 points
         (100, 30000, 512, 4096, False, "u8", 12.0, (1.0,)),       # the most trials of 2^10 points
         (40, 30000, 600, 8192, False, "f32", 30.0, (1.0,)),       # 2^11 points
         (257, 12000, 1100, 4096, False, "f32", 9.0, (1.0,)),      # 2^12 points
         (1024, 9000, 1030, 4096, False, "u8", 9.0, (1.0,)),       # the most channels whose values are staged
         (1030, 4096, 1030, 4096, True, "f32", 9.0, (1.0,)),       # one part more: values read where they are used
         (33, 5000, 2049, 2048, False, "f32", 3.0, (1.0,)),        # two blocks of trials
         (48, 4096, 4500, 4096, True, "f32", 12.0, (1.0,)),        # three blocks, one chunk
         (1, 5000, 70, 2048, False, "f32", 3.0, (1.0,)),           # one channel
         (70, 20000, 300, 4096, False, "f32", 10.0, (1.0, 2.0, 4.0)),   # three runs
         (72, 9000, 200, 1024, False, "u8", 2.0, (1.0,)),          # short transforms, many chunks
         (200, 4096, 64, 4096, True, "f32", 100.0, (1.0,))]        # coarse steps: the channels go round many times


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}ch_{c[2]}dm_L{c[3]}_{c[5]}_{len(c[7])}runs" for c in CASES])
def test_grid_matches_oracle(case, monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    w, x = workload(40 + case[0], *case)
    precision = {0: "fp32", 1: "fp16_split", 2: "bf16_split"}[case[0] % 3]
    print(f"grid {case} {precision}", flush=True)
    with plan_of(w, precision=precision) as p:
        assert p.grid[0] == len(case[7])
        xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
        y = p.execute(xd)
        again = p.execute(xd.clone())
        torch.cuda.synchronize()
        assert torch.equal(y, again)
        g, y = p.geometry, y.cpu().numpy()
    ref = O.fdd(x, w.input_kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, single_chunk=w.single_chunk,
                mode="exact")
    raw = raw_start(w.input_kind, w.n_samp, w.chunk_len, int(g.stride), int(g.n_chunks), w.single_chunk)
    check_rows(y, ref, TOL, raw_from=raw, label=f"grid {case}")


@pytest.mark.parametrize("kind", ["f32", "u8"])
def test_grid_power_and_channel_order(kind, monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    w, x = workload(7, 90, 4096, 2100, 4096, True, kind, 15.0)
    order = np.random.default_rng(3).permutation(w.n_chan)
    xs = np.ascontiguousarray(x[:, order] if kind == "u8" else x[order])
    with plan_of(w, freqs=w.freqs[order], power_only=True) as p:
        assert p.grid[0] == 1
        P = p.power_spectrum(torch.from_numpy(xs).cuda())
        torch.cuda.synchronize()
        P = P.cpu().numpy()
    ref = O.fdd_power(x, kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, mode="exact")
    check_power(P, ref, TOL, skip_dc=kind == "u8", label=f"grid power {kind}")
    if kind == "u8":                             # the offset of all channels, coherent in every trial
        np.testing.assert_allclose(P[:, 0], ref[:, 0], rtol=2 * TOL)


def test_grid_downsampled_and_long(monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    w, x = workload(11, 50, 20000, 260, 4096, False, "f32", 10.0)
    factors = np.repeat([1, 2, 4], [100, 90, 70]).astype(np.int32)
    with plan_of(w, downsample=factors) as p:
        assert p.grid[0] == 3
        rows = [r.cpu().numpy() for r in p.rows(p.execute(torch.from_numpy(x).cuda()))]
    ref = O.fdd(x, "f32", w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, mode="exact", factors=factors)
    for r, e in zip(rows, ref):
        check_rows(r[None], np.asarray(e)[None], TOL, label="grid down-sampled")
    w, x = workload(12, 20, 150000, 80, 1 << 17, False, "f32", 100.0)
    with plan_of(w) as p:
        assert p.grid[0] == 1
        y = p.execute(torch.from_numpy(x).cuda()).cpu().numpy()
    ref = O.fdd(x, "f32", w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, mode="exact")
    check_rows(y, ref, TOL, label="grid, long transforms")


@pytest.mark.parametrize("share", [False, True])
def test_grid_batch(share, monkeypatch):
    """Beams of the grid form next to others in one batch, replayed on new data."""
    monkeypatch.setenv("FDD_GRID", "1")
    shapes = [(64, 9000, 200, 2048, False, "f32", 4.0), (70, 12000, 300, 2048, False, "u8", 4.0),
              (64, 7000, 200, 2048, False, "f32", 4.0), (30, 9000, 20, 2048, False, "f32", 4.0)]
    made = [workload(60 if s[0] == 64 else 61 + i, *s) for i, s in enumerate(shapes)]
    xs = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for _, x in made]
    plans = [plan_of(w, workspace=False) for w, _ in made]
    assert [p.grid[0] for p in plans] == [1, 1, 1, 0]
    outs = [torch.empty((w.n_dm, w.n_samp), dtype=torch.float32, device="cuda") for w, _ in made]
    with fdd.Batch(plans, autotune=False, share_phasors=share) as b:
        assert any(c["choice"] == "grid" for c in b.describe()["classes"])
        for rep in range(3):
            for x in xs:
                if x.dtype == torch.float32:
                    x.mul_(-0.5).add_(0.25)
            b.execute(xs, outs)
            for (w, _), x, y in zip(made, xs, outs):
                with plan_of(w) as p:
                    e = p.execute(x)
                    torch.cuda.synchronize()
                if share:
                    assert float((y - e).norm() / e.norm()) < TOL
                else:
                    assert torch.equal(y, e), (rep, w.name)
    for p in plans:
        p.close()
