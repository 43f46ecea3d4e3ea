"""Launch shapes of untuned plans: bands held in registers are short; a launch
that has no such variant keeps the row march's taller bands at 2048^2, where
the halo rows of short ones are the cost."""
import pytest

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")


def shapes(n, bc, prec, nu1, nu2):
    plan = cc.Plan(cc.Problem(n=n, bc=tuple(bc), prec=prec, nu1=nu1, nu2=nu2))
    return {n >> l: (pre, post) for l, (pre, _, post, _) in enumerate(cc.ccmg_plan_shapes(plan)) if n >> l >= 64}


@pytest.mark.parametrize("bc", ["DDDD", "PPPP"])
def test_untuned_bands(bc):
    held = {64: 8, 128: 8, 256: 8, 512: 8, 1024: 16, 2048: 16}
    march = dict(held) | {2048: 32}
    big = {4096: 64}
    for prec, nu1, nu2, pre, post in [(cc.FP64, 2, 2, held, held), (cc.FP64, 3, 1, held, march),
                                      (cc.FP64, 1, 4, march, held), (cc.FP64, 0, 3, march, march),
                                      (cc.MIXED, 1, 1, march, march), (cc.MIXED, 2, 2, held, held)]:
        for n in (512, 2048, 4096):
            for m, got in shapes(n, bc, prec, nu1, nu2).items():
                # (a mixed plan's finest prolongating launch also updates the FP64 iterate: marched)
                q = march if prec == cc.MIXED and m == n else post
                assert got == ((pre | big)[m], (q | big)[m]), (prec, nu1, nu2, n, m)
