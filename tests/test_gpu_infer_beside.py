"""The network's BF16 inference on another stream while sampling waves are on every compute unit: it
ends before the sampling launch does, with the same rows as alone. (On one of four streams: those
that share the sampling launch's hardware queue wait.)"""
import time

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


@pytest.mark.parametrize("L,per_cu,tuning", [(8, 2, dict(schedule=0)), (6, 4, dict(schedule=0)),
                                             (12, 4, dict(schedule=1, waves_per_cu=4))],
                         ids=["L8 generator waves", "L6 generator waves", "L12 queue"])
def test_inference_beside_sampling(nfm, L, per_cu, tuning):
    import torch
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    sampling = torch.cuda.Stream()
    b = nfm.Batch([L] * n, [64] * n, 3, 4, stream=sampling)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    b.rec_init(1, 1.0, -1.0)
    b.set_tuning(**tuning)
    b.run_sweeps(2)
    sweeps = 40960 // L ** 3 + 500          # one launch of 6 ms or more
    rows = 256
    x = torch.randn(rows, 81, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    y = torch.zeros(rows, 256, device="cuda")
    beside = []
    for _ in range(4):
        other, done = torch.cuda.Stream(), torch.cuda.Event()
        net = nfm.Mlp(batch_max=rows, stream=other)
        net.init(5)
        net.to_bf16()
        torch.cuda.synchronize()
        want = net.infer_bf16(x)
        torch.cuda.synchronize()
        b.run_sweeps(sweeps)
        done.record(sampling)
        time.sleep(0.001)                   # the waves are placed
        net.infer_bf16(x, out=y)
        other.synchronize()
        beside.append(not done.query())
        torch.cuda.synchronize()
        assert torch.equal(y, want)
        y.zero_()
        torch.cuda.synchronize()
        net.close()
    print("inference beside", b.last_kernel(), beside, flush=True)
    assert any(beside)
    b.close()
