"""The device update where its work is split: more levels than one staged chunk of the chains (768;
L = 12 with a prior down to level 0 has 1297), counts with gaps across whole 64-level mask words,
one counted level, none at all, and L = 2 with fewer levels than a batch of eight additions.

The device keeps the oracle's operation order, so the results differ by the last bits of log and
exp alone (2^-52 relative each, on log-weights below 2^12): a step by about 4 * 2^-40 / 2^12 of
the largest, S by that times the square root of 1297 levels. 1e-12 normwise bounds both."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED = 5, 0xFEED


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


@pytest.mark.parametrize("L", [2, 10, 12])
@pytest.mark.parametrize("profile", [0, 1, 2])
@pytest.mark.parametrize("seeded", [False, True])
def test_update_blocks(nfm, orc, L, profile, seeded):
    kinds = ["full", "gaps", "one", "none"]
    print("update blocks: L", L, "profile", profile, "seeded", seeded, flush=True)
    R, dE, alpha = len(kinds), 24.0, -2.0
    b = nfm.Batch([L] * R, [64] * R, DSEED, WSEED)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    E_min = b.read_walkers()["E_min"].reshape(R, 64).min(1)
    rng = np.random.default_rng(100 * L + 10 * profile + seeded)
    Hs = np.zeros(b.levels_total, np.uint64)
    cases = []
    for r, kind in enumerate(kinds):
        J = orc.couplings(L, DSEED, r)
        K, eb = orc.n_levels(L, J), orc.e_base(L, J)
        k_top = (-eb + 3) // 4
        k_min = (int(E_min[r]) - eb) // 4
        # the state's lowest level: far below the walkers (so that the estimate is long), but in the
        # first realization just above them (new levels below)
        k_lo = min(k_top, k_min + 1) if r == 0 else min(k_min, k_top // 4)
        low = 0 if seeded else k_lo
        bv, pv = np.zeros(K), np.zeros(K)
        bv[low:k_top] = rng.normal(-1.0, 0.5, k_top - low)
        pv[k_lo:k_top] = rng.uniform(0, 50, k_top - k_lo) * (rng.random(k_top - k_lo) < 0.7)
        vis = (rng.random(K) < 0.5).astype(np.uint8)
        _, lnP, lnW = orc.rec_weights_ext(K, eb, k_lo, k_top, low, profile, dE, alpha, bv)
        H, lo = np.zeros(K, np.uint64), min(k_min, k_lo)
        if kind in ("full", "gaps"):
            H[lo:k_top + 2] = rng.integers(1, 1000, min(k_top + 2, K) - lo)
        if kind == "gaps":
            H[rng.random(K) < 0.5] = 0
            H[lo + 5:lo + 5 + 150] = 0
        if kind == "one":
            H[(lo + k_top) // 2] = 12
        Hs[b.level_offset(r):b.level_offset(r) + K] = H
        b.rec_set_state(r, bv, pv, lnP, lnW, vis, k_lo, k_top, profile, dE, alpha, k_seed=0 if seeded else -1)
        cases.append((K, eb, k_top, min(k_min, k_lo), k_lo, low, bv, pv, vis, lnP, lnW, H))
    b.set_histograms(Hs)
    info = b.rec_update(0.3)
    for r, (K, eb, k_top, k_min, k_lo, low, bv, pv, vis, lnP0, lnW0, H) in enumerate(cases):
        k_new, flat = orc.rec_update_ext(K, k_lo, k_top, low, seeded, k_min, lnW0, lnP0, H, bv, pv, vis)
        low_new = min(low, k_new)
        S, lnP, lnW = orc.rec_weights_ext(K, eb, k_new, k_top, low_new, profile, dE, alpha, bv)
        st = b.rec_get_state(r)
        assert info["k_lo"][r] == k_new == st["info"]["k_lo"]
        assert info["converged"][r] == int(flat >= 0.3 and k_new == k_lo)
        assert abs(info["flatness"][r] - flat) <= 1e-12 * abs(flat), (r, info["flatness"][r], flat)
        assert np.array_equal(st["visited"][:K], vis), r
        sl = slice(low_new, k_top + 1)
        for name, ref in (("b", bv), ("p", pv), ("S", S), ("lnP", lnP), ("lnW", lnW)):
            err = np.max(np.abs(st[name][sl] - ref[sl]))
            assert err <= 1e-12 * np.max(np.abs(ref[sl]), initial=1e-300), (name, r, err)
    b.close()
