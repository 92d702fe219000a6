"""GPU parity of the phasor sum on the vector ALUs: plans of one or two chunks with few equally spaced
trials (increments from the coarse and fine tables) and with rounded delays (increments from the
(channel, DM) table), at every number of bins per lane, trial and channel counts that are not multiples
of the 4 waves, and power spectra.

Tolerance 2e-6 of the row norm: the two transforms keep within 4e-7 each, the sum of up to 130 channels
in four parts within 5e-7 and the product of two evaluated phasors within 2e-7.
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

#        channels, samples, trials, L, single, input, DM max, mode, precision
CASES = [(64, 4096, 64, 4096, True, "f32", 20.0, "exact", "fp32"),           # one bin per lane
         (33, 4000, 33, 4096, True, "u8", 20.0, "exact", "fp16_split"),      # partial waves and rows
         (3, 1024, 5, 1024, True, "f32", 4.0, "exact", "bf16_split"),        # fewer channels than waves
         (30, 16384, 65, 16384, True, "f32", 60.0, "exact", "fp32"),         # 4 bins per lane
         (18, 65536, 66, 65536, True, "f32", 200.0, "exact", "fp32"),        # 16 bins per lane
         (21, 3000, 70, 2048, False, "f32", 5.0, "exact", "fp32"),           # two chunks, one bin per lane
         (17, 50000, 67, 32768, False, "u8", 100.0, "exact", "fp16_split"),  # two chunks, 8 bins per lane
         (130, 4096, 301, 4096, True, "f32", 20.0, "round", "fp32"),         # rounded delays
         (10, 3000, 9, 2048, False, "u8", 5.0, "round", "fp32")]             # and two chunks


def plan_of(w, mode, precision):
    return fdd.Plan(w.freqs, w.ref_freq_mhz, w.tsamp_s, w.dms, w.n_samp, w.chunk_len, single_chunk=w.single_chunk,
                    input=w.input_kind, mode=mode, precision=precision)


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}ch_{c[2]}dm_L{c[3]}_{c[7]}_{c[8]}" for c in CASES])
def test_valu_matches_oracle(case, monkeypatch):
    n_chan, n_samp, n_dm, L, single, kind, dm_max, mode, precision = case
    monkeypatch.setenv("FDD_GRID", "0")
    w = W.tiny_random(n_chan + n_dm, n_chan, n_samp, n_dm, L, single_chunk=single, input_kind=kind, dm_max=dm_max)
    w = dataclasses.replace(w, dms=np.linspace(0.0, dm_max, n_dm))
    x = W.gaussian_u8(n_samp, n_chan, n_dm) if kind == "u8" else W.gaussian_f32(n_chan, n_samp, n_dm)
    with plan_of(w, mode, precision) as p:
        g = p.geometry
        assert int(g.n_chunks) == (1 if single else 2)
        xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
        y = p.execute(xd).cpu().numpy()
        power = p.power_spectrum(xd).cpu().numpy() if single else None
        raw = raw_start(kind, n_samp, L, int(g.stride), int(g.n_chunks), single)
    ref = O.fdd(x, kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, single_chunk=single, mode=mode)
    check_rows(y, ref, TOL, raw_from=raw, label=str(case))
    if single:
        ref = O.fdd_power(x, kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len, mode=mode)
        check_power(power, ref, TOL, skip_dc=kind == "u8", label=str(case))
