"""The threaded steps of the oracle give the oracle's own results, bit for bit (CPU)."""
import numpy as np
import pytest

import oracle_threads
import workloads as W
from oracle import fdd_oracle


@pytest.mark.parametrize("kind,single,mode", [("f32", True, "exact"), ("u8", False, "round"), ("u8", False, "exact")])
def test_threaded_oracle_is_the_oracle(kind, single, mode, monkeypatch):
    w = W.tiny_random(5, 37, 9000 if not single else 4096, 6, 4096, single_chunk=single, input_kind=kind, dm_max=20.0)
    x = W.gaussian_u8(w.n_samp, 37, 1) if kind == "u8" else W.gaussian_f32(37, w.n_samp, 1)
    args = (x, kind, w.dms, w.freqs, w.ref_freq_mhz, w.tsamp_s, w.chunk_len)
    want = fdd_oracle.fdd(*args, single_chunk=single, mode=mode)
    power = fdd_oracle.fdd_power(*args, mode=mode) if single else None
    undo = oracle_threads.install(fdd_oracle, small=1)
    try:
        got = fdd_oracle.fdd(*args, single_chunk=single, mode=mode)
        gotp = fdd_oracle.fdd_power(*args, mode=mode) if single else None
    finally:
        undo()
    assert np.array_equal(want, got)
    assert power is None or np.array_equal(power, gotp)
