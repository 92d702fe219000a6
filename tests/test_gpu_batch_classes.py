"""What a batch may choose from (GPU).

A tuned choice is kept for the class, for later batches of the process and in the tuning file,
whatever their trial counts.  So a class must not offer a kernel that only a part of its trial counts
should run.
"""
import json
import os
import subprocess
import sys

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


_FRESH = """
import json
import numpy as np
import torch
import paper_2110_03482_amd as fdd
n = 1 << 16
freqs = 1250.0 + (np.arange(64) + 0.5) * (300.0 / 64)
plans = [fdd.Plan(freqs, 1550.0, 64e-6, np.linspace(0.0, 400.0, 64), n + n // 4, n, precision="fp16_split", workspace=False)
         for _ in range(2)]
assert all(p.geometry.n_chunks == 2 and p.grid[0] == 0 for p in plans)
xs = [torch.randn((64, n + n // 4), device="cuda") for _ in plans]
with fdd.Batch(plans) as b:
    b.execute(xs)
    torch.cuda.synchronize()
    print(json.dumps(b.describe()["classes"]))
"""


def test_first_launches_in_a_process_do_not_prune_a_candidate():
    """64 trials and two chunks: the direct split kernel measures 0.4 to 0.6 of the vector kernel's time, which
    is timed before it.  The direct kernel's first launch also loads it, several times that."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _FRESH], cwd=root, env=dict(os.environ, PYTHONPATH=root), capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    (c,) = json.loads(r.stdout.strip().splitlines()[-1])
    print(c["key"], c["choice"], c["candidates"])
    assert c["key"].endswith("+fac0few")
    assert c["choice"] == "mfma_f16_split/grid"


@pytest.mark.parametrize("n_chan,tuned", [(360, False), (1000, True)])
def test_grid_beams_win_against_the_shared_launch(n_chan, tuned):
    """360 channels, 128 trials, one split chunk of 65536 samples: alone the grid kernel is the fastest,
    in a tuned batch the direct kernel, whose beams share a launch.  With 1000 channels the grid is in
    both.  Untuned batches run what the beams' own plans run."""
    n = 1 << 16
    freqs = 1250.0 + (np.arange(n_chan) + 0.5) * (300.0 / n_chan)
    plans = [fdd.Plan(freqs, 1550.0, 64e-6, np.linspace(0.0, 400.0, 128), n, n, single_chunk=True, precision="fp16_split",
                      workspace=False) for _ in range(2)]
    assert all(p.grid[0] == 1 for p in plans)
    xs = [torch.randn((n_chan, n), device="cuda") for _ in plans]
    outs = {}
    for autotune in (False, True):
        with fdd.Batch(plans, autotune=autotune) as b:
            outs[autotune] = [y.clone() for y in b.execute(xs)]
            torch.cuda.synchronize()
            grid = [c["choice"] == "grid" for c in b.describe()["classes"]]
        assert grid == [tuned if autotune else True]
    for y, e in zip(outs[True], outs[False]):
        assert float((y - e).norm() / e.norm()) < 1e-5          # the split products keep within 1e-6
    for p in plans:
        p.close()
