"""The persistent kernels for grids of at most one workgroup per SIMD (k_sweeps_queue_lone): results
bit for bit as the launches per size, and room on every SIMD for kernels of other streams."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DSEED, WSEED = 13, 0xABCDEF01


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


def _batch(nfm, Ls, tuning, stream=None):
    b = nfm.Batch(Ls, [64] * len(Ls), DSEED, WSEED, stream=stream)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    b.rec_init(1, 1.0, -1.0)
    b.set_tuning(**tuning)
    return b


@pytest.mark.parametrize("spec", [0, 1])
@pytest.mark.parametrize("Ls", [[8, 6, 4, 2, 6], [10, 2, 8, 6], [12, 10, 8, 6, 4, 2]], ids=lambda v: str(v[0]))
def test_lone_forms_match_launches_per_size(nfm, Ls, spec):
    out = []
    for tuning in (dict(schedule=0), dict(schedule=1, speculate=spec), dict(schedule=1, speculate=spec, hist=1),
                   dict(schedule=1, speculate=spec, hist=3, waves_per_cu=2)):
        print("lone queue", Ls, tuning, flush=True)
        b = _batch(nfm, Ls, dict(tuning, sweeps_per_launch=4))
        b.run_sweeps(10)
        if tuning["schedule"]:
            (kernel, form, grid, _, _), = b.last_launch()
            name = "k_sweeps_queue_spec" if spec else "k_sweeps_queue"
            assert (kernel, form, grid) == (f"{name}<{max(Ls)}>", "lone", len(Ls))
            assert b.last_kernel() == name
        out.append((b.get_spins(0, b.n_walkers), b.read_walkers(), b.read_histograms()))
        b.close()
    for o in out[1:]:
        for x, y in zip(o, out[0]):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("L", [8, 10, 12])
def test_other_streams_run_beside_the_queue(nfm, L):
    """A wave on every SIMD, for many milliseconds: a small kernel on another stream ends before the
    queue's launch does. (On one of four streams: those that share the queue's hardware queue wait.)"""
    import torch
    n = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    queue = torch.cuda.Stream()
    b = _batch(nfm, [L] * n, dict(schedule=1, waves_per_cu=4), stream=queue)
    b.run_sweeps(2)
    assert b.last_launch()[0][1:3] == ("lone", n)
    sweeps = 40960 // L ** 3 + 200          # one launch of 8 ms or more
    x = torch.zeros(4096, device="cuda")
    beside = []
    for _ in range(4):
        other, done = torch.cuda.Stream(), torch.cuda.Event()
        torch.cuda.synchronize()
        b.run_sweeps(sweeps)
        done.record(queue)
        time.sleep(0.001)                   # its waves are placed
        with torch.cuda.stream(other):
            x.add_(1.0)
        other.synchronize()
        beside.append(not done.query())
        torch.cuda.synchronize()
    print("beside the queue, L =", L, beside, flush=True)
    assert any(beside)
    b.close()
