"""Launch shapes set by hand for the 64 x 64 level below the finest.  It runs in
one launch with the tail, which writes one of the level's two arrays; launches
of its own, which a shape or a visit set for it asks for, write both (two
launches) or the same one (a visit).  The iterates are the same bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")

POISON = 0xA5


def vcycle(n, prec, shapes, tune=False):
    """One V-cycle from zero; the field and how many of the workspace's bytes
    it left as they were."""
    plan = cc.Plan(cc.Problem(n=n, bc=tuple("DNDD"), prec=prec))
    fv = np.random.default_rng(5).standard_normal((n, n))
    f = torch.zeros((n + 2, n + 2), dtype=torch.float64, device="cuda")
    f[1:n + 1, 1:n + 1] = torch.from_numpy(fv).cuda()
    phi = torch.zeros_like(f)
    level = n.bit_length() - 1 - 6
    for kind, ty, wpb in shapes:
        cc.ccmg_plan_set_shape(plan, level, kind, ty, wpb)
    if tune:
        cc.ccmg_plan_autotune(plan, f, phi)
        assert cc.ccmg_plan_shape(plan, level, 0) == cc.ccmg_plan_shape(plan, level, 1) == (8, 1)
        assert cc.ccmg_plan_shape(plan, level, 5)[0] == 0
    plan.workspace.fill_(POISON)
    cc.ccmg_vcycle(plan, f, phi)
    torch.cuda.synchronize()
    return phi[1:n + 1, 1:n + 1].cpu().numpy(), int((plan.workspace == POISON).sum())


@pytest.mark.parametrize("prec", [cc.FP64, cc.MIXED])
@pytest.mark.parametrize("n", [128, 256])
def test_shapes_set_for_the_64_level_are_run(n, prec):
    ref, left = vcycle(n, prec, [])
    level_bytes = 64 * 64 * (8 if prec == cc.FP64 else 4)
    for shapes in ([(0, 16, 1)], [(1, 32, 2)], [(0, 0, 1)]):
        got, left_own = vcycle(n, prec, shapes)
        assert np.array_equal(got, ref), shapes
        # a value's bytes are seldom all unlike the pattern: a tenth is far above that
        assert left - left_own > 0.9 * level_bytes, shapes
    for shapes in ([(0, 8, 1), (1, 8, 1)], [(5, 32, 1), (5, 0, 1)]):  # the defaults
        got, same = vcycle(n, prec, shapes)
        assert np.array_equal(got, ref) and abs(same - left) < 0.1 * level_bytes, shapes
    got, _ = vcycle(n, prec, [(5, 32, 1)])  # a visit
    assert np.array_equal(got, ref)
    # the tuner goes back to the launch with the tail
    got, same = vcycle(n, prec, [(0, 16, 1), (5, 32, 1)], tune=True)
    assert np.array_equal(got, ref) and abs(same - left) < 0.1 * level_bytes
