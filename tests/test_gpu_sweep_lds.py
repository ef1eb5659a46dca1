"""On-chip memory of the L = 12 sweep kernels: what a workgroup asks for decides how many of them a
compute unit holds, so a form is charged for what it uses and for nothing else."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED = 5, 0xD1CE5EED
L, MARGIN = 12, 64
JK_BYTES = 4 * 2 * L * 6 * 3     # two colours, L planes, six bonds, three words a plane
LDS_PER_CU = 160 * 1024


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


def _batch(nfm, Ls, rows, **tuning):
    """Tables of `rows` rows up to E = 0 (one extra level of slack at the top) for every realization."""
    b = nfm.Batch(Ls, [64] * len(Ls), DSEED, WSEED)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    lnw, k_lo, k_top = np.zeros(b.levels_total), [], []
    for r in range(len(Ls)):
        eb, off = b.e_base(r), b.level_offset(r)
        top = (-eb + 3) // 4
        lo = max(0, top - rows + 1)
        lnw[off + lo:off + top + 1] = -0.7 * (eb + 4.0 * np.arange(lo, top + 1))
        k_lo.append(lo)
        k_top.append(top)
    b.set_weights_lnw(lnw, k_lo, k_top)
    b.set_tuning(**tuning)
    return b


def _plain(b, rows):
    """Table, couplings and the histogram's window: what every form needs."""
    return 32 * rows + JK_BYTES + 4 * min(b.levels(0), rows + 2 * MARGIN)


@pytest.mark.parametrize("schedule", [0, 2])
def test_speculative_forms_hold_no_staged_words(nfm, schedule):
    b = _batch(nfm, [L, 4], 300, schedule=schedule, speculate=1, hist=1)
    b.run_sweeps(2)
    print("speculative L = 12, schedule", schedule, b.last_launch(), flush=True)
    launch = [x for x in b.last_launch() if x[0].endswith("<12>")]
    assert len(launch) == 1 and "spec" in launch[0][0]
    rows = max(len(b.get_thresholds(0)[0]), 1)
    assert launch[0][4] == _plain(b, rows)
    b.close()


# (waves per compute unit, rows): waves alone; SIMDs shared with room for staged words; without room
# (as many workgroups as fit 160 KB without the words, or fewer)
@pytest.mark.parametrize("per_cu,rows,form", [(4, 720, "vector"), (5, 720, "vector"), (6, 660, "vector"),
                                              (5, 60, "staged"), (7, 200, "staged"), (8, 400, "vector")])
def test_staged_words_cost_no_resident_workgroup(nfm, orc, per_cu, rows, form):
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n, T = (per_cu - 1) * n_cu + 40, 2
    print("L = 12:", n, "waves,", rows, "rows", flush=True)
    b = _batch(nfm, [L] * n, rows, schedule=0)
    table_rows = max(len(b.get_thresholds(r)[0]) for r in range(n))
    b.run_sweeps(T)
    (kernel, got, grid, threads, lds), = b.last_launch()
    assert (kernel, got, grid, threads) == ("k_sweeps<12>", form, n, 64)
    fit = LDS_PER_CU // _plain(b, table_rows)
    assert LDS_PER_CU // lds >= min(fit, per_cu)
    # the last realization against the oracle
    r = n - 1
    thr, row0 = b.get_thresholds(r)
    w0, off = b.walker_offset(r), b.level_offset(r)
    rz = orc.make_realization(L, DSEED, r, WSEED, 64)
    Hr, _ = orc.sample(rz, thr, row0, 0, 0, T)
    assert np.array_equal(b.read_histograms()[off:off + rz.K], Hr)
    assert np.array_equal(b.get_spins(w0, 64).reshape(64, -1), rz.S)
    assert np.array_equal(b.read_walkers()["E"][w0:w0 + 64], rz.w["E"])
    b.close()
