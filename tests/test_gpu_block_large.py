"""Bands held in registers where they are the default from 1024^2: the FP64
fused launch in its two-waves-per-SIMD form and several waves to a workgroup,
whose tile sums meet in LDS (three waves leave a remainder: 1280 tiles), against
the row march in bands of 32 rows; and, in the FP32 cycles of mixed solves,
every height of band on the levels below the finest.  The same bits; singular
FP64 problems, whose means are summed over tiles cut differently, to 1e-12 of
the largest value.  (Singular mixed solves round those means to FP32, where two
cuts of the row march differ as well, and are not compared.)"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")

N = 1024


def solve(bc, prec, fv, finest, fused, levels):
    """Four cycles; shapes (rows, waves) of the finest level's two launches, of
    the fused one and of the 512^2 to 128^2 levels."""
    plan = cc.Plan(cc.Problem(n=N, bc=tuple(bc), prec=prec, max_cycles=4, rtol=0.0))
    for level in range(4):
        for kind in (0, 1):
            cc.ccmg_plan_set_shape(plan, level, kind, *(levels if level else finest))
    cc.ccmg_plan_set_shape(plan, 0, 2 if prec == cc.FP64 else 3, *fused)
    f = torch.zeros((N + 2, N + 2 + 3), dtype=torch.float64, device="cuda")
    f[1:N + 1, 1:N + 1] = torch.from_numpy(fv).cuda()
    phi = torch.zeros_like(f)
    r = cc.ccmg_solve(plan, f, phi)
    assert r.status == cc.NOT_CONVERGED and r.cycles == 4
    return phi.cpu().numpy(), r.history


def rhs():
    fv = np.random.default_rng(61).standard_normal((N, N))
    return fv - fv.mean()


@pytest.mark.parametrize("bc", ["DDDD", "DNPP", "PPPP"])
def test_fp64_default_forms_match_the_row_march(bc):
    print(f"block {N}^2 {bc}", flush=True)
    fv = rhs()
    ref, href = solve(bc, cc.FP64, fv, (32, 1), (32, 1), (32, 1))
    for finest, fused, levels in (((16, 1), (8, 1), (8, 1)), ((16, 4), (8, 4), (8, 4)), ((8, 3), (8, 3), (16, 3))):
        got, h = solve(bc, cc.FP64, fv, finest, fused, levels)
        if bc == "PPPP":
            assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max(), (finest, fused, levels)
        else:
            assert np.array_equal(got, ref), (finest, fused, levels)
        np.testing.assert_allclose(h, href, rtol=1e-9)


@pytest.mark.parametrize("bc", ["DDDD", "DNPP"])
def test_fp32_levels_match_the_row_march(bc):
    print(f"block {N}^2 mixed {bc}", flush=True)
    fv = rhs()
    ref, href = solve(bc, cc.MIXED, fv, (32, 1), (32, 1), (32, 1))
    for fused, levels in (((16, 1), (8, 1)), ((16, 4), (16, 3)), ((8, 3), (16, 4)), ((32, 1), (0, 1))):  # (0: as 8)
        got, h = solve(bc, cc.MIXED, fv, (32, 1), fused, levels)
        assert np.array_equal(got, ref), (fused, levels)
        np.testing.assert_allclose(h, href, rtol=1e-9)
