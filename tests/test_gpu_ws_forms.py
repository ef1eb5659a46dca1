"""The generator-wave launches around the wave count from which their waves share SIMDs (more pairs
than half the SIMDs): which form runs, and each form against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED, FIRST = 17, 0x5EED5EED, 2


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


# (L, waves beyond half the SIMDs, speculate, form): only L = 6 changes to one read there
@pytest.mark.parametrize("L,over,spec,form", [(4, 1, 0, "paired"), (6, 0, 0, "paired"), (6, 1, 0, "single"),
                                              (6, 1, 1, "paired"), (8, 0, 0, "paired"), (8, 1, 0, "paired"),
                                              (8, 100, 1, "paired")])
def test_form_and_results_where_waves_share_simds(nfm, orc, L, over, spec, form):
    import torch
    n, T = 2 * torch.cuda.get_device_properties(0).multi_processor_count + over, 3
    print("generator wave: L", L, "waves", n, "speculate", spec, flush=True)
    b = nfm.Batch([L] * n, [64] * n, DSEED, WSEED, first_real_id=FIRST)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    b.rec_init(0)
    b.set_tuning(speculate=spec, sweeps_per_launch=2)
    b.run_sweeps(T)
    (kernel, got, grid, threads, _), = b.last_launch()
    assert (kernel, got, grid, threads) == (f"k_sweeps_ws{'_spec' if spec else ''}<{L}>", form, n, 128)
    S, ws, H = b.get_spins(0, b.n_walkers).reshape(n, 64, -1), b.read_walkers(), b.read_histograms()
    for r in (0, n // 2, n - 1):
        thr, row0 = b.get_thresholds(r)
        rz = orc.make_realization(L, DSEED, FIRST + r, WSEED, 64)
        e_bot = b.e_base(r) + 4 * int(b.rec_read_info()["k_lo"][r])
        Hr, _ = orc.sample(rz, thr, row0, e_bot, 0, T)
        off, w0 = b.level_offset(r), b.walker_offset(r)
        assert np.array_equal(H[off:off + rz.K], Hr)
        assert np.array_equal(S[r], rz.S)
        for f in ("E", "E_min", "rt_state", "new_min", "rt_count", "t_first", "t_last"):
            assert np.array_equal(ws[f][w0:w0 + 64], rz.w[f]), f
    b.close()
