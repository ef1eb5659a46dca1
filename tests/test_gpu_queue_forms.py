"""The persistent kernels that share SIMDs (k_sweeps_queue, compiled for sizes up to 8, 10 and 12):
batches of more waves than the GPU has SIMDs, with and without speculation, under every extent of the
on-chip histogram. Bit for bit as the launches per size, and against the oracle for one realization
of every size; the report of the launch shows that the form under test is the one that ran."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED, FIRST = 31, 0xC0FFEE11, 3
FIELDS = ("E", "E_min", "rt_state", "new_min", "rt_count", "t_first", "t_last")


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


def _simds():
    import torch
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def _run(nfm, Ls, n, tuning):
    b = nfm.Batch(Ls, [64] * len(Ls), DSEED, WSEED, first_real_id=FIRST)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    b.rec_init(1, 1.0, -1.0)     # tables from the walkers' levels: short ones, left on both sides
    b.set_tuning(sweeps_per_launch=3, **tuning)
    b.run_sweeps(n)
    return b, (b.get_spins(0, b.n_walkers), b.read_walkers(), b.read_histograms())


def _against_oracle(orc, b, state, Ls, n):
    S, ws, H = state
    w0s = np.concatenate([[0], np.cumsum([64 * L ** 3 for L in Ls])])
    for L in sorted(set(Ls)):
        r = Ls.index(L)
        thr, row0 = b.get_thresholds(r)
        rz = orc.make_realization(L, DSEED, FIRST + r, WSEED, 64)
        e_bot = b.e_base(r) + 4 * int(b.rec_read_info()["k_lo"][r])
        Hr, _ = orc.sample(rz, thr, row0, e_bot, 0, n)
        off, w0 = b.level_offset(r), b.walker_offset(r)
        assert np.array_equal(H[off:off + rz.K], Hr), L
        assert np.array_equal(S[w0s[r]:w0s[r + 1]].reshape(64, -1), rz.S), L
        for f in FIELDS:
            assert np.array_equal(ws[f][w0:w0 + 64], rz.w[f]), (L, f)


@pytest.mark.parametrize("spec", [0, 1])
@pytest.mark.parametrize("largest", [8, 10, 12])
def test_shared_forms_match_oracle_and_launches_per_size(nfm, orc, largest, spec):
    Ls = [largest, largest - 2, 6, 4] + [2] * _simds() + [largest, 4]
    n = 5
    b, want = _run(nfm, Ls, n, dict(schedule=0))
    _against_oracle(orc, b, want, Ls, n)
    b.close()
    name = "k_sweeps_queue_spec" if spec else "k_sweeps_queue"
    for hist in (0, 1, 2, 3):
        print("shared queue: largest", largest, "speculate", spec, "hist", hist, "waves", len(Ls), flush=True)
        b, got = _run(nfm, Ls, n, dict(schedule=1, speculate=spec, hist=hist))
        (kernel, form, grid, threads, lds), = b.last_launch()
        assert (kernel, form, grid, threads) == (f"{name}<{largest}>", "shared", len(Ls), 64)
        assert b.last_kernel() == name
        for x, y in zip(got, want):
            assert np.array_equal(x, y), hist
        b.close()


@pytest.mark.parametrize("L", [2, 6])
def test_one_size_with_more_waves_than_simds_is_queued(nfm, L):
    Ls = [L] * (_simds() + 7)
    b, want = _run(nfm, Ls, 4, dict(schedule=0))
    b.close()
    for schedule in (1, 2):
        print("one size, queued: L", L, "schedule", schedule, flush=True)
        b, got = _run(nfm, Ls, 4, dict(schedule=schedule))
        (kernel, form, grid, _, _), = b.last_launch()
        assert (kernel, form, grid) == ("k_sweeps_queue<8>", "shared", len(Ls))
        for x, y in zip(got, want):
            assert np.array_equal(x, y)
        b.close()
