"""The end of a cycle (its residual, the done flag, the mean of phi) when it
runs inside the next cycle's first coarse launch: what is queued behind a
cycle that converged leaves the finest level alone."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")


def field(v):
    n = v.shape[0]
    t = torch.zeros((n + 2, n + 2), dtype=torch.float64, device="cuda")
    t[1:n + 1, 1:n + 1] = torch.from_numpy(v).cuda()
    return t


def workspace(plan):
    """The plan's workspace from its first (256-byte aligned) byte."""
    return plan.workspace[-plan.workspace.data_ptr() % 256:]


def finest_buffers(plan):
    """The two finest-level buffers of an FP64 plan (the workspace's first regions)."""
    n = plan.n
    size = 8 * (n + 2) * ((n + 2 + 31) & ~31)
    return workspace(plan)[:2 * ((size + 255) & ~255)].clone()


@pytest.mark.parametrize("bc", ["DDDD", "DNPP"])
def test_cycle_queued_past_the_last_one_does_nothing(bc):
    """A cycle expected to be the last ends without the next one's
    pre-smoothing; a residual that falls more slowly than extrapolated has the
    next cycle queued all the same, before the residual is read.  If the cycle
    did converge, that next cycle must not touch the finest level: the buffers
    are those of the same solve that may not queue it (max_cycles)."""
    n = 256
    fv = np.random.default_rng(0).standard_normal((n, n))

    def solve(rtol, max_cycles):
        plan = cc.Plan(cc.Problem(n=n, bc=tuple(bc), rtol=rtol, max_cycles=max_cycles))
        workspace(plan).zero_()
        phi = field(np.zeros((n, n)))
        r = cc.ccmg_solve(plan, field(fv), phi)
        torch.cuda.synchronize()
        return r, phi.cpu().numpy(), finest_buffers(plan)

    h = solve(1e-12, 30)[0].history
    # cycle 4 is queued with cycles 1 and 2 known, cycle 5 with cycle 3 known:
    # the first extrapolation meets half the tolerance, the second doesn't
    lo = max(2 * h[2] ** 3 / h[1] ** 2, h[4])
    hi = min(2 * h[3] ** 2 / h[2], 2 * h[2] ** 2 / h[1], h[3])
    assert 1.1 * lo < hi
    rtol = (lo * hi) ** 0.5
    r, phi, buf = solve(rtol, 30)
    s, ref, ref_buf = solve(rtol, 4)
    assert r.status == s.status == cc.OK and r.cycles == s.cycles == 4
    assert np.array_equal(phi, ref)
    assert torch.equal(buf, ref_buf)


def history_region(plan):
    """The device history of a plan: behind it lie the flags (256 bytes) and
    the exact bottom's inverse (8^4 doubles), the workspace's end."""
    ws, nbytes = workspace(plan), cc.ccmg_workspace_bytes(plan.prob)
    end = nbytes - 8 * 8 ** 4 - 256
    return ws[end - 8 * cc.HISTORY:end].clone().view(torch.float64)


@pytest.mark.parametrize("value", [0.0, np.inf])
def test_refused_solve_leaves_no_end_behind(value):
    """A right-hand side that ends a solve is seen after its first cycle, when
    the second is queued and its end not yet launched; that end must not be run
    by whatever uses the plan next (here the autotuner's coarse cycles, which
    write no history: it is cleared and stays clear)."""
    n = 4096
    plan = cc.Plan(cc.Problem(n=n, bc=tuple("DDDD")))
    good = np.random.default_rng(3).standard_normal((n, n))
    bad = field(np.full((n, n), value))
    phi = torch.zeros_like(bad)
    if value == 0.0:
        r = cc.ccmg_solve(plan, bad, phi)
        assert r.status == cc.OK and r.cycles == 0
    else:
        with pytest.raises(cc.CcmgError) as e:
            cc.ccmg_solve(plan, bad, phi)
        assert e.value.status == cc.ENONFINITE
    f = field(good)
    phi.zero_()
    cc.ccmg_plan_autotune(plan, f, phi)
    torch.cuda.synchronize()
    assert not history_region(plan).any()
    r = cc.ccmg_solve(plan, f, phi)
    assert r.status == cc.OK and r.cycles > 5
