"""nfm_mlp_infer_bf16_noalloc where the output rows overlap the input rows (they go through the
library's static rows then): bit for bit as into separate rows, call after call with more and with
fewer rows than the one before, whose rows must not show."""
import numpy as np
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


# where the input starts in the output rows: their start, inside a row, their last element
@pytest.mark.parametrize("at", [0, 93, -1], ids=["start", "inside", "end"])
def test_output_over_input_matches_separate_rows(nfm, at):
    import torch
    rng = np.random.default_rng(11)
    mlp = nfm.Mlp(batch_max=1024)
    mlp.init(7)
    p, _ = mlp.get_params()
    mlp.set_params(p + rng.normal(0, 0.05, p.shape).astype(np.float32),
                   np.stack([rng.normal(0, 1, 81), rng.uniform(0.5, 2, 81)]).astype(np.float32))
    mlp.to_bf16()
    for rows in (1000, 37, 1024, 1):
        print("no-alloc inference over its input:", rows, "rows, at", at, flush=True)
        x = torch.tensor(rng.normal(0, 1.5, (rows, 81)).astype(np.float32), device="cuda")
        want = mlp.infer_bf16(x)
        off = rows * 256 - 1 if at < 0 else at
        both = torch.full((rows * (256 + 81),), float("nan"), dtype=torch.float32, device="cuda")
        both[off:off + rows * 81] = x.view(-1)
        out = mlp.infer_bf16_noalloc(both[off:off + rows * 81].view(rows, 81), both[:rows * 256].view(rows, 256))
        torch.cuda.synchronize()
        assert torch.equal(out, want), rows
    mlp.close()
