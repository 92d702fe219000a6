"""GPU parity of the forward transform of long series (two passes over memory), seen through the power
spectrum of two channels at DM 0, which is |X_0[f] + X_1[f]|^2: every factorisation, both input types,
whole and short series, and a second channel whose start is not aligned for 8-byte (or 2-byte) loads.

Tolerance: a transform of N points in two passes rounds each value in at most log2 N butterfly levels
and 6 twiddle products, about sqrt(log2 N + 6) 6e-8 = 3.2e-7 of the root mean square value.  The power
has twice that: 1e-6 of the norm, in every 64th of the spectrum.  Samples of 8 bits that are not centred
(short series) have twice the root mean square of their spectrum without bin 0: 2e-6.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2110_03482_amd as fdd  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-6, "u8": 2e-6}


@pytest.mark.parametrize("log_len", [17, 18, 19, 20, 21, 22])
@pytest.mark.parametrize("kind", ["f32", "u8"])
@pytest.mark.parametrize("short", [0, 1, 12345])
def test_long_forward(log_len, kind, short):
    L = 1 << log_len
    n = L - short
    rng = np.random.default_rng(log_len + short)
    if kind == "u8":
        x = rng.integers(0, 256, (n, 2), dtype=np.uint8)
        ref_in = x.T.astype(np.float64)
    else:
        x = rng.standard_normal((2, n), dtype=np.float32)
        ref_in = x.astype(np.float64)
    plan = fdd.Plan(np.array([1300.0, 1400.0]), 1500.0, 64e-6, np.array([0.0, 1e-3]), n, L, single_chunk=True, input=kind)
    out = plan.power_spectrum(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)[0]
    ref = np.abs(np.fft.rfft(ref_in.sum(axis=0), L)[: out.size]) ** 2
    if kind == "u8":                                 # bin 0 is the sum of the samples
        assert abs(out[0] - ref[0]) <= 1e-5 * ref[0]
        out[0] = ref[0] = 0.0
    out, ref = out.reshape(64, -1), ref.reshape(64, -1)
    assert np.all(np.linalg.norm(out - ref, axis=1) <= TOL[kind] * np.linalg.norm(ref, axis=1))
