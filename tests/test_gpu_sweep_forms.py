"""Every kernel form of the sweeps at the edges of its table: a table of one row, of a few rows
around the walkers' energies and of all levels, so that the clamped compact rows, the expanded
table's copies of the first and last row and the rows of both outcomes are read below, inside and
above the window; all table entries distinct, so that a wrong row or entry shows. Against the
oracle, bit for bit (spins, walker records, histograms)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED = 77, 0xBEEF5EED


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


def _table(rng, rows):
    """Random thresholds, a third of them near 0 and a third near 2^32 - 1 (long runs of refused
    and of taken moves), so that walkers leave the window on both sides."""
    t = rng.integers(0, 2 ** 32, (rows, 8), dtype=np.uint64)
    edge = rng.integers(0, 3, (rows, 8))
    t[edge == 0] >>= 20
    t[edge == 1] |= 0xFFF00000
    return t.astype(np.uint32)


# L = 4 (four planes a block), 6 (unrolled, rows with unused bits), 8 (whole words), 10 and 12
# (several words a plane); plain and paired forms, a launch per size and the persistent ones
@pytest.mark.parametrize("tuning", [dict(ws=1), dict(ws=2), dict(speculate=1, ws=1), dict(hist=3), dict(schedule=1),
                                    dict(schedule=2), dict(schedule=2, speculate=1)],
                         ids=lambda d: "-".join(f"{k}{v}" for k, v in d.items()))
@pytest.mark.parametrize("rows", [1, 5, 0])
def test_table_windows_match_oracle(nfm, orc, tuning, rows):
    Ls, W, T = [12, 10, 8, 6, 4], 64, 3
    rng = np.random.default_rng(rows)
    print("table windows: rows", rows, "tuning", tuning, flush=True)
    groups = [Ls] if "schedule" in tuning else [[L] for L in Ls]
    for Lg in groups:
        b = nfm.Batch(Lg, [W] * len(Lg), DSEED, WSEED, first_real_id=40)
        b.set_tuning(sweeps_per_launch=2, **tuning)
        b.init_couplings()
        b.init_spins()
        b.compute_energies()
        E0 = b.read_walkers()["E"].copy()
        refs = []
        for r, L in enumerate(Lg):
            J = orc.couplings(L, DSEED, 40 + r)
            K, eb = orc.n_levels(L, J), orc.e_base(L, J)
            n = rows or K
            row0 = 0 if rows == 0 else int(np.median(E0[r * W:(r + 1) * W]) - eb) // 4 - n // 2
            thr = _table(rng, n)
            b.set_thresholds(r, thr, row0)
            b.set_rt_bounds(r, eb, 0)
            refs.append((L, J, K, eb, thr, row0))
        b.run_sweeps(T)
        ws, H = b.read_walkers(), b.read_histograms()
        for r, (L, J, K, eb, thr, row0) in enumerate(refs):
            spins = b.get_spins(b.walker_offset(r), W).reshape(W, L ** 3)
            Href = np.zeros(K, np.uint64)
            for w in range(W):
                s = orc.spins(L, WSEED, 40 + r, w)
                wr = orc.new_walkers(1, orc.energy(L, J, s))
                orc.muca_sweeps(L, J, s, wr, thr, row0, eb, 0, WSEED, 40 + r, w, 0, T, hist=Href)
                assert np.array_equal(spins[w], s), (L, w)
                for f in ("E", "E_min", "rt_state", "new_min", "rt_count"):
                    assert ws[f][r * W + w] == wr[f][0], (f, L, w)
            assert np.array_equal(H[b.level_offset(r):b.level_offset(r) + K], Href), L
        b.close()


@pytest.mark.parametrize("L", [2, 6, 12])
def test_one_size_under_the_persistent_schedule(nfm, L):
    """A batch of one size with at most one wave per SIMD has nothing to queue and runs as the size's
    own launch, unless the queue's options are set; the results are the same in each form, and in the
    queue of a grid with several waves per SIMD."""
    print("one size, persistent schedule: L", L, flush=True)
    out = []
    for tuning, form in ((dict(schedule=1), f"k_sweeps_ws<{L}>"), (dict(schedule=2), f"k_sweeps_ws<{L}>"),
                         (dict(schedule=1, ws=1), f"k_sweeps_xt<{L}>"), (dict(schedule=1, waves_per_cu=1), "k_sweeps_queue"),
                         (dict(schedule=1, hist=1), "k_sweeps_queue"), (dict(schedule=1, speculate=1), "k_sweeps_queue_spec")):
        b = nfm.Batch([L] * 3, [64, 128, 64], DSEED, WSEED, first_real_id=7)
        b.set_tuning(sweeps_per_launch=3, **tuning)
        b.init_couplings()
        b.init_spins()
        b.compute_energies()
        b.rec_init(0)
        b.run_sweeps(5)
        assert b.last_kernel() == form, tuning
        out.append((b.get_spins(0, b.n_walkers), b.read_walkers(), b.read_histograms()))
        b.close()
    for o in out[1:]:
        assert np.array_equal(o[0], out[0][0]) and np.array_equal(o[1], out[0][1]) and np.array_equal(o[2], out[0][2])
