"""Planning of the grid form of the phasor sum, on dry-run plans (no GPU)."""
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
