"""GPU tests of the level-0 Prod at the sizes and run shapes that only large plans have."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    import paper_1402_6081_amd.lgf as L
    L.library()
    return L


def test_more_near_targets_than_half_the_offset_range(L):
    """Separate sets with 4251528 near targets (162^3 blocks, every 27th a source) in FP32: the
    field spectra of a wave's two chunks span more than 2^32 bytes, its offsets less.  Against the
    same sources evaluated on 4000 of the blocks: bit for bit (a target's sums do not depend on
    which other targets there are)."""
    e, n, p = 162, 4, 2
    print("case: near targets", e ** 3, flush=True)
    b = np.arange(e, dtype=np.int32)
    ev = np.stack(np.meshgrid(b, b, b, indexing="ij"), -1).reshape(-1, 3)
    c = np.arange(1, e, 3, dtype=np.int32)
    src = np.stack(np.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.default_rng(162)
    some = np.unique(np.concatenate([rng.integers(0, len(ev), 4000), [0, len(ev) - 1]]))
    plan = L.Plan(src, n, p, 0, "f32", eval_blocks=ev)
    f = torch.randn(plan.shape(), dtype=torch.float32, generator=torch.Generator().manual_seed(1)).to("cuda:0")
    u = plan.solve(f)[torch.from_numpy(some).to("cuda:0")].clone()
    plan.close()
    small = L.Plan(src, n, p, 0, "f32", eval_blocks=ev[some])
    v = small.solve(f)
    torch.cuda.synchronize()
    small.close()
    assert torch.equal(u, v)
