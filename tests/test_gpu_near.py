"""GPU tests of the level-0 Prod at the sizes and run shapes that only large plans have, and of the
interpolation passes at every block edge and node count."""
import numpy as np
import pytest
import torch

from oracle import flgf
from paper_1402_6081_amd import workloads as W
from tolerances import FP32_BAR, fp64_tol, lebesgue, rel

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


def _towers():
    """Towers of 2 x 2 x (16, 16, 16, 16, 10, 5) blocks side by side, with a hole and an odd top."""
    b = [(2 * i + dx, dy, z) for i, h in enumerate((16, 16, 16, 16, 10, 5)) for dx in (0, 1) for dy in (0, 1)
         for z in range(h)]
    return np.array([t for t in b if t not in ((3, 1, 7), (10, 0, 4))], dtype=np.int32)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,copies", [(8, 25), (4, 171)])
def test_lockstep_and_free_workgroups(L, n, copies, prec):
    """A batch of towers whose runs are 8, 8, 8, 8, 5 and 3 groups: workgroups whose four waves march
    in lockstep beside such whose waves do not, and a last one with two runs
    (tests/test_host_rules.py counts them).  Against the towers alone, whose runs are single groups,
    bit for bit, in workgroups of 4, 2 and 8 waves; alone against the oracle (tolerances.py).  n = 4
    has an odd number of chunks, the second half of FP32's last wave none."""
    p = 4
    print("case: lockstep", n, prec, flush=True)
    blocks = _towers()
    rng = np.random.default_rng(n)
    if prec == "f64":
        f = rng.standard_normal((len(blocks), n, n, n))
    else:
        f, _ = W.zero_mean_gaussians(blocks, n, rng, len(blocks) // 8)
    plan = L.Plan(blocks, n, p, 0, prec)
    fd = torch.from_numpy(f).to("cuda:0", plan.dtype)
    u = plan.solve(fd)
    ref = flgf.FLGF(blocks, n, p, 0).solve(fd.cpu().numpy().astype(np.float64))
    assert rel(u.cpu().numpy().astype(np.float64), ref) <= (fp64_tol(p) if prec == "f64" else FP32_BAR)
    batch = L.Plan.batch([blocks] * copies, n, p, 0, prec)
    fb = fd.repeat(copies, 1, 1, 1).contiguous()
    want = u.repeat(copies, 1, 1, 1)
    for waves in (4, 2, 8):
        batch.set_tuning(near_waves=waves)
        assert torch.equal(batch.solve(fb), want), waves
    batch.close()
    plan.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [4, 6, 8, 12, 16])
def test_every_block_edge_and_node_count(L, n, prec):
    """Reg, Interp and the final pass share their outputs among the waves differently for every
    (n, p): all of p = 2..10 on a small layout of two far-field levels, against the oracle.  Bound:
    rounding of a level's node values (eps of the path's transforms) grows by at most Lambda^3 in each
    Interp below it and, adjointly, each Reg: Lambda^6 eps for two levels, and never less than the
    bars of tolerances.py."""
    blocks = np.array([(x, y, z) for x in range(7) for y in (0, 1) for z in (0, 1) if (x + 2 * y + z) % 4 != 3],
                      dtype=np.int32)
    rng = np.random.default_rng(n)
    f64 = prec == "f64"
    for p in range(2, 11):
        print("case: shares", n, p, prec, flush=True)
        f = rng.standard_normal((len(blocks), n, n, n)) if f64 else W.zero_mean_gaussians(blocks, n, rng, 3)[0]
        plan = L.Plan(blocks, n, p, 0, prec)
        fd = torch.from_numpy(f).to("cuda:0", plan.dtype)
        u = plan.solve(fd).cpu().numpy().astype(np.float64)
        plan.close()
        ref = flgf.FLGF(blocks, n, p, 0).solve(fd.cpu().numpy().astype(np.float64))
        grown = lebesgue(p) ** 6 * (2.0 ** -52 if f64 else 2.0 ** -23)
        assert rel(u, ref) <= max(grown, fp64_tol(p) if f64 else FP32_BAR), p
