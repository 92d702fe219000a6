"""Planning of the grid form of the phasor sum, on dry-run plans (no GPU)."""
import time

import numpy as np
import pytest

fdd = pytest.importorskip("paper_2110_03482_amd")


def dry(n_chan, n_samp, dms, L, **kw):
    freqs = 1250.0 + (np.arange(n_chan) + 0.5) * (300.0 / n_chan)
    return fdd.Plan(freqs, 1550.0, 64e-6, dms, n_samp, L, dry_run=True, **kw)


@pytest.mark.parametrize("factor", [2, 16])
@pytest.mark.parametrize("L,dm_max", [(16384, 500.0), (65536, 2000.0)])
def test_scratch_of_a_down_sampled_single_chunk_plan_holds_all_bins(L, dm_max, factor, monkeypatch):
    """Its power spectra are those of the full resolution: beyond the twiddles of the shortened
    inverse it needs no less memory than the plan without down-sampling."""
    monkeypatch.setenv("FDD_GRID", "1")
    dms = np.linspace(0.0, dm_max, 1024)
    with dry(64, L, dms, L, single_chunk=True) as p:
        assert p.grid[0] == 1
        full = p.geometry.workspace_bytes
    with dry(64, L, dms, L, single_chunk=True, downsample=[factor] * 1024) as p:
        assert p.grid[0] == 1
        assert p.geometry.workspace_bytes >= full + 8 * (L // factor)


@pytest.mark.parametrize("n_chan,n_dm", [(200, 400), (256, 1000), (512, 2048)])
def test_no_schedules_where_values_are_staged(n_chan, n_dm, monkeypatch):
    """Up to 16 spread steps per column group the grid kernel writes no schedule: beyond the plan of the
    family it needs 1 MiB for rows that are no trials, its channel tables and row divisors (under 64
    KiB), and a few groups of bins (small DM steps: 1024 bins a group)."""
    got = {}
    for form in ("0", "1"):
        monkeypatch.setenv("FDD_GRID", form)
        with dry(n_chan, 100000, np.linspace(0.0, 2.0, n_dm), 8192) as p:
            assert p.grid[0] == int(form)
            got[form] = p.geometry.workspace_bytes
    assert got["1"] <= got["0"] + (1 << 20) + (1 << 16)


def test_plans_keep_fitting_the_static_scratch(monkeypatch):
    """A plan that fits the 64 MiB of fdd_execute_noalloc without the grid's schedules fits them with
    FDD_GRID=1, too: it gives up the grid form instead."""
    limit = 64 << 20
    kept = dropped = 0
    for n_dm in range(100, 520, 20):
        size, grid = {}, {}
        for form in ("0", "1"):
            monkeypatch.setenv("FDD_GRID", form)
            with dry(420, 1 << 14, np.linspace(0.0, 30.0, n_dm), 4096) as p:
                size[form], grid[form] = p.geometry.workspace_bytes, p.grid[0]
        assert grid["0"] == 0
        if size["0"] <= limit:
            assert size["1"] <= limit
            kept += grid["1"] == 1
            dropped += grid["1"] == 0
        else:
            assert grid["1"] == 1
    assert kept > 0 and dropped > 0


STEPPED = np.cumsum(np.concatenate([[0.0], np.full(99, 0.5), np.full(100, 1.0), np.full(101, 2.0)]))


@pytest.mark.parametrize("dms,kw,runs", [
    (np.linspace(0.0, 50.0, 64), {}, 1), (np.linspace(0.0, 50.0, 63), {}, 0),             # the shortest run
    (STEPPED, {}, 3), (STEPPED[:170], {}, 2), (STEPPED[:163], {}, 0),                     # a run of 63 trials
    (STEPPED[::-1], {}, 0), (np.sqrt(np.arange(300.0)), {}, 0), (np.zeros(100), {}, 0),
    (np.linspace(7.0, 50.0, 300), {}, 1),                                                 # does not begin at 0
    (np.linspace(0.0, 50.0, 300), {"mode": "round"}, 0),
    (np.linspace(0.0, 50.0, 300), {"downsample": [1] * 150 + [2] * 150}, 2),              # runs end with a segment
    (np.linspace(0.0, 50.0, 300), {"downsample": [1] * 250 + [2] * 50}, 0),
    (np.linspace(0.0, 50.0, 5000), {}, 1)])
def test_runs_of_equal_steps(dms, kw, runs, monkeypatch):
    monkeypatch.setenv("FDD_GRID", "1")
    with dry(40, 40000, dms, 8192, **kw) as p:
        assert p.grid[0] == runs
        assert p.grid[1] == 0 if runs == 0 else 256 <= p.grid[1] <= 4096
        assert runs == 0 or p.grid[1] == 4096 or p.grid[1] >= 2 * dms.size // runs - 4


@pytest.mark.parametrize("env", ["FDD_FACTOR", "FDD_TILE_VARIANT", "FDD_PHASE_TABLE"])
def test_a_family_asked_for_by_name_keeps_its_kernels(env, monkeypatch):
    dms = np.linspace(0.0, 1000.0, 2048)
    with dry(1024, 1 << 20, dms, 1 << 16) as p:
        assert p.grid[0] == 1
    monkeypatch.setenv(env, {"FDD_FACTOR": "direct", "FDD_TILE_VARIANT": "0", "FDD_PHASE_TABLE": "linear"}[env])
    with dry(1024, 1 << 20, dms, 1 << 16) as p:
        assert p.grid == (0, 0)


def test_planning_takes_no_longer_than_the_family(monkeypatch):
    """The row divisors depend on the grid alone and are made once.  Per plan the grid form then does
    less than the factorised one (no phase table): 1.29 against 1.57 ms of this thread's time."""
    best = {"0": 1.0, "1": 1.0}
    dms = np.linspace(0.0, 20.0, 2048)
    for _ in range(40):
        for form in best:
            monkeypatch.setenv("FDD_GRID", form)
            t0 = time.thread_time()
            with dry(64, 4096, dms, 4096, single_chunk=True) as p:
                best[form] = min(best[form], time.thread_time() - t0)
                assert p.grid[0] == int(form)
    assert best["1"] <= best["0"]


# Measured phasor stages of both forms on an MI355X, us (family, grid): chunks, L, channels, trials, precision.
# A single chunk is a circular transform, two are 1.25 L samples.
MEASURED = [
    # the factorised kernels are the faster ones: a workgroup has 64 coarse rows of 32 / N trials
    (2, 1 << 16, 91, 218, "fp16_split", 267, 407), (2, 1 << 16, 93, 830, "bf16_split", 343, 442),
    (2, 1 << 16, 128, 192, "fp16_split", 346, 429), (2, 1 << 14, 91, 535, "bf16_split", 92, 127),
    (2, 1 << 15, 83, 106, "fp16_split", 138, 216), (2, 1 << 12, 118, 132, "bf16_split", 39, 58),
    (2, 1 << 16, 77, 2216, "bf16_split", 886, 1430), (2, 1 << 16, 52, 388, "fp32", 323, 427),
    (2, 1 << 14, 48, 129, "fp32", 84, 124), (2, 1 << 13, 51, 288, "fp32", 59, 80), (2, 1 << 16, 40, 3022, "fp32", 911, 1490),
    # the grid is
    (2, 1 << 16, 256, 316, "bf16_split", 651, 470), (2, 1 << 16, 195, 1065, "fp16_split", 1144, 765),
    (2, 1 << 16, 105, 139, "fp32", 592, 410), (2, 1 << 16, 117, 1681, "fp32", 1313, 816),
    (1, 1 << 13, 359, 1999, "fp32", 311, 105), (2, 1 << 15, 163, 968, "fp32", 480, 289)]


@pytest.mark.parametrize("case", MEASURED, ids=[f"{c[2]}ch_{c[3]}dm_L{c[1]}x{c[0]}_{c[4]}" for c in MEASURED])
def test_rule_takes_the_form_that_measures_faster(case):
    chunks, L, n_chan, n_dm, precision, family, grid = case
    top = 0.3 * L * 64e-6 / (4148.808 * (1250.0 ** -2 - 1550.0 ** -2))
    with dry(n_chan, L if chunks == 1 else L * 5 // 4, np.linspace(0.0, top, n_dm), L, single_chunk=chunks == 1,
             precision=precision) as p:
        assert p.geometry.n_chunks == chunks and p.kernel.startswith("fac_")
        assert (p.grid[0] > 0) == (grid < family)


@pytest.mark.parametrize("precision", ["fp32", "fp16_split"])
def test_rule_over_trials_of_two_chunks(precision):
    """The line is the fewest channels that take the grid; it lies where a stage of channels of the
    factorised kernels begins (8, or 16 in the split precisions).  Up to 1024 trials both forms do the
    same work, but the families write more sums, so the line falls.  With twice the trials past 1024
    the families do twice the work; the grid kernel makes a bin's entries once (36 of 480 us) and a
    column of 4096 points takes half the spread steps (0.6 of 12.9 us), so 1.8 times: the line falls by
    up to 14 % (46 us of at least 350 us of products), in whole stages."""
    L = 1 << 16

    def line(n_dm):
        for n_chan in range(16, 400, 4):
            with dry(n_chan, L * 5 // 4, np.linspace(0.0, 500.0, n_dm), L, precision=precision) as p:
                if p.grid[0] > 0:
                    return n_chan
        return 400

    assert line(300) >= line(600) >= line(1024)
    stage = 8 if precision == "fp32" else 16
    for n_dm in (600, 800, 1024):
        assert line(n_dm) - (0.14 * line(n_dm) + stage) <= line(2 * n_dm) <= line(n_dm)
