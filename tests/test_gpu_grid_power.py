"""Power spectra of the grid form of the phasor sum on plans that also down-sample (GPU).

Down-sampling factors do not apply to power spectra, so one plan runs its trials over fewer bins in
execute() and over all bins in power_spectrum().  The DM steps are coarse enough that the channels
go round the grid in the high bins, whose orders come from the plan's scratch.

Tolerance as in test_gpu_grid.py; the same trials without down-sampling run the same sums, bit for bit.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import paper_2110_03482_amd as fdd  # noqa: E402
import workloads as W  # noqa: E402
from parity import check_power  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 2e-6


def make(seed, n_chan, L, n_dm, kind, dm_max):
    w = W.tiny_random(seed, n_chan, L, n_dm, L, single_chunk=True, input_kind=kind, dm_max=dm_max)
    w = dataclasses.replace(w, dms=np.linspace(0.0, dm_max, n_dm))
    return w, W.gaussian_u8(L, n_chan, seed) if kind == "u8" else W.gaussian_f32(n_chan, L, seed)


def plan_of(w, **kw):
    return fdd.Plan(w.freqs, w.ref_freq_mhz, w.tsamp_s, w.dms, w.n_samp, w.chunk_len, single_chunk=True, input=w.input_kind,
                    **kw)


#         channels, L, trials, input, DM max, factors
CASES = [(64, 4096, 70, "f32", 120.0, (4,)), (200, 4096, 140, "u8", 150.0, (2, 8)), (64, 16384, 128, "f32", 500.0, (16,))]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}ch_L{c[1]}_{c[3]}_{len(c[5])}runs" for c in CASES])
def test_power_of_a_down_sampling_plan(case, monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    n_chan, L, n_dm, kind, dm_max, fs = case
    w, x = make(9, n_chan, L, n_dm, kind, dm_max)
    print(f"power of a down-sampling plan {case}", flush=True)
    xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    factors = np.repeat(fs, n_dm // len(fs)).astype(np.int32)
    with plan_of(w, downsample=factors) as p:
        assert p.grid[0] == len(fs)
        P = p.power_spectrum(xd)
        y = p.execute(xd)
        again, y2 = p.power_spectrum(xd), p.execute(xd)
        torch.cuda.synchronize()
        assert torch.equal(P, again) and torch.equal(y, y2)
    if len(fs) == 1:
        with plan_of(w) as p:
            assert p.grid[0] == 1
            assert torch.equal(P, p.power_spectrum(xd))
    ref = O.fdd_power(x, kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, mode="exact")
    check_power(P.cpu().numpy(), ref, TOL, skip_dc=kind == "u8", label=f"power of a down-sampling plan {case}")


def test_power_into_an_output_at_any_float(monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    w, x = make(10, 70, 2048, 100, "f32", 20.0)
    xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    with plan_of(w, power_only=True) as p:
        assert p.grid[0] == 1
        P = p.power_spectrum(xd)
        for off in (1, 2, 3):
            flat = torch.full((P.numel() + 8,), -1.0, device="cuda")
            out = flat[off:off + P.numel()].view(P.shape)
            assert p.power_spectrum(xd, out) is out
            torch.cuda.synchronize()
            assert torch.equal(out, P)
            assert bool((flat[:off] == -1.0).all()) and bool((flat[off + P.numel():] == -1.0).all())
