"""What a batch may choose from (GPU).

A tuned choice is kept for the class, for later batches of the process and in the tuning file,
whatever their trial counts.  So a class must not offer a kernel that only a part of its trial counts
should run.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
fdd = pytest.importorskip("paper_2110_03482_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [1, 2])
def test_factorised_classes_do_not_offer_the_vector_kernel(chunks, monkeypatch, tmp_path):
    monkeypatch.setenv("FDD_GRID", "0")
    L = 2048
    n_samp = L if chunks == 1 else L * 5 // 4
    plans, xs = [], []
    for n_dm in (300, 900, 40):
        w = W.tiny_random(n_dm, 20, n_samp, n_dm, L, single_chunk=chunks == 1, input_kind="f32", dm_max=4.0)
        plans.append(fdd.Plan(w.freqs, w.ref_freq_mhz, w.tsamp_s, np.linspace(0.0, 4.0, n_dm), n_samp, L,
                              single_chunk=chunks == 1, workspace=False))
        assert plans[-1].geometry.n_chunks == chunks and plans[-1].kernel == "fac_f32"
        xs.append(torch.from_numpy(W.gaussian_f32(20, n_samp, n_dm)).cuda())
    with fdd.Batch(plans, tune_cache=str(tmp_path / "tune.json")) as b:
        b.execute(xs)
        torch.cuda.synchronize()
        classes = {c["key"].split("+")[1]: c for c in b.describe()["classes"]}
    assert set(classes) == {"fac0", "fac0few"}                  # 300 and 900 trials; 40 trials
    assert all(k.startswith("fac_f32/") for k in classes["fac0"]["candidates"])
    assert any(k.startswith("fac_few/") for k in classes["fac0few"]["candidates"])
    for p in plans:
        p.close()
