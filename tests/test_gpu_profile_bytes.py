"""GPU test of the bytes that the step profile reports for Reg and its forward transform."""
import pytest
import torch

from paper_1402_6081_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,es", [("f64", 8), ("f32", 4)])
def test_reg_bytes(prec, es):
    """Input read, spectra written, and node values written where a level above reads them: not at
    the top level, whose node values stay in LDS."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    import paper_1402_6081_amd.lgf as L
    n, p = 8, 6
    spectrum = 2 * es * 4 * p * p * (p + 1)
    expected = {4: {"reg_l0_l1": 64 * (n ** 3 * es + spectrum)},
                8: {"reg_l0_l1": 512 * ((n ** 3 + p ** 3) * es + spectrum),
                    "reg_l1_l2": 512 * p ** 3 * es + 64 * spectrum}}
    for edge, steps in expected.items():
        print("case: Reg bytes", prec, edge, flush=True)
        plan = L.Plan(W.cube_layout(edge), n, p, 0, prec)
        f = torch.randn(plan.shape(), dtype=plan.dtype, device="cuda:0")
        plan.profile_enable(1)
        plan.solve(f)
        torch.cuda.synchronize()
        got = {s["name"]: s["bytes"] for s in plan.profile_collect()["steps"] if s["name"].startswith("reg_")}
        assert got == steps
        plan.close()
