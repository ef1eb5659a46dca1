"""Couplings, starts, energies and the couplings' statistics of one batch of all lattice sizes with
uneven walker counts, against the oracle: rows that straddle words (L = 6, 10, 12), stream words cut
at any bit (N = 216, 1000), rows with unused bits, L = 2 whose neighbours on both sides are one site.
Random and uniform couplings (all bonds of either sign: the extremes of the energy and of every
count). Integers are compared exactly; the statistics are counts over N, formed in FP64 and rounded
once to FP32, moments to within 2^-22 relative."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED = 31337, 0xC0FFEE12345


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


@pytest.mark.parametrize("couplings", ["drawn", "plus", "minus"])
def test_batch_of_all_sizes(nfm, orc, couplings):
    Ls, Ws = [12, 2, 6, 10, 4, 8], [64, 128, 192, 64, 64, 128]
    print("samples: couplings", couplings, flush=True)
    b = nfm.Batch(Ls, Ws, DSEED, WSEED, first_real_id=1000)
    if couplings == "drawn":
        b.init_couplings()
    else:
        v = 1 if couplings == "plus" else -1
        for r, L in enumerate(Ls):
            b.set_couplings(r, nfm.pack_couplings(np.full(3 * L ** 3, v, np.int8), L))
    b.init_spins()
    b.compute_energies()
    b.reset_histograms()
    ws = b.read_walkers()
    x = b.features().cpu().numpy()
    for r, L in enumerate(Ls):
        J = orc.couplings(L, DSEED, 1000 + r) if couplings == "drawn" else np.full(3 * L ** 3, v, np.int8)
        assert np.array_equal(b.get_couplings(r, 1), nfm.pack_couplings(J, L)), L
        assert b.levels(r) == orc.n_levels(L, J) and b.e_base(r) == orc.e_base(L, J), L
        g = b.walker_offset(r)
        spins = b.get_spins(g, Ws[r]).reshape(Ws[r], L ** 3)
        for w in range(Ws[r]):
            S = orc.spins(L, WSEED, 1000 + r, w)
            assert np.array_equal(spins[w], S), (L, w)
            assert ws["E"][g + w] == ws["E_min"][g + w] == orc.energy(L, J, S), (L, w)
        assert x[r][0] == np.float32(L / 12.0)
        for k, ref in enumerate(orc.features(L, J)):
            got = x[r][1 + k]
            assert abs(got - ref) <= 2.0 ** -22 * max(abs(ref), 2.0 ** -20), (L, k, got, ref)
    b.close()
