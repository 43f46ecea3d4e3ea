"""A batch's levels on either side of the sizes from which the iterate of the way
down is recomputed rather than stored: each problem against the same problem
alone (one FP32 cycle per refinement step).  A problem with a Dirichlet side has
no mean to remove, so its iterates are the same bits whatever the tiles, and its
history differs by the order of a sum of n^2 squares."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")


def field(n, pad, seed=None):
    a = torch.zeros((n + 2, n + 2 + pad), dtype=torch.float64, device="cuda")
    if seed is not None:
        g = torch.Generator().manual_seed(seed)
        a[1:n + 1, 1:n + 1] = torch.randn((n, n), dtype=torch.float64, generator=g).cuda()
    return a


@pytest.mark.parametrize("tuned", [False, True])
def test_recomputed_levels_match_single_solves(tuned):
    cases = [(n, bc) for n in (64, 128, 256, 512, 1024, 2048) for bc in ("DDDD", "PPDN", "NDPP")]
    probs = [cc.Problem(n=n, bc=tuple(bc), rtol=1e-9, prec=cc.MIXED) for n, bc in cases]
    batch = cc.Batch(probs)
    fs = [field(n, i % 3, seed=i) for i, (n, _) in enumerate(cases)]
    phis = [field(n, i % 3) for i, (n, _) in enumerate(cases)]
    if tuned:
        cc.ccmg_batch_autotune(batch, fs, phis)
    res, info = cc.ccmg_batch_solve(batch, fs, phis)
    assert info["status"] == cc.OK
    for (n, bc), p, f, phi, r in zip(cases, probs, fs, phis, res):
        plan = cc.Plan(p)
        cc.ccmg_plan_set_option(plan, cc.OPT_MIXED_INNER, 1)
        one = torch.zeros_like(f)
        r1 = cc.ccmg_solve(plan, f, one)
        assert r1.cycles == r.cycles, (n, bc)
        np.testing.assert_allclose(r.history, r1.history, rtol=n * n * 2.0 ** -52)
        assert torch.equal(phi[1:n + 1, 1:n + 1], one[1:n + 1, 1:n + 1]), (n, bc)


@pytest.mark.parametrize("counts", [{256: 63}, {256: 64, 512: 16}, {1024: 33}, {1024: 24, 2048: 8}])
def test_size_classes_on_either_side_of_the_cell_counts(counts):
    """Batches whose size classes hold just fewer or just enough cells to
    recompute (4 M of finest levels, 8 M of a coarser level): two of each size
    against the same problems alone."""
    cases = [(n, ("DDDD", "NDPP")[i % 2]) for n, c in counts.items() for i in range(c)]
    probs = [cc.Problem(n=n, bc=tuple(bc), rtol=1e-9, prec=cc.MIXED) for n, bc in cases]
    fs = [field(n, 0, seed=i) for i, (n, _) in enumerate(cases)]
    phis = [field(n, 0) for n, _ in cases]
    res, info = cc.ccmg_batch_solve(cc.Batch(probs), fs, phis)
    assert info["status"] == cc.OK
    seen = {}
    for (n, bc), p, f, phi, r in zip(cases, probs, fs, phis, res):
        seen[n, bc] = seen.get((n, bc), 0) + 1
        if seen[n, bc] > 1:
            continue
        plan = cc.Plan(p)
        cc.ccmg_plan_set_option(plan, cc.OPT_MIXED_INNER, 1)
        one = torch.zeros_like(f)
        r1 = cc.ccmg_solve(plan, f, one)
        assert r1.cycles == r.cycles, (n, bc)
        np.testing.assert_allclose(r.history, r1.history, rtol=n * n * 2.0 ** -52)
        assert torch.equal(phi[1:n + 1, 1:n + 1], one[1:n + 1, 1:n + 1]), (n, bc)


def test_recomputed_levels_with_a_guess_and_a_mean():
    """A singular problem (its mean is removed as the iterate is read) from a
    guess: the residual of what is returned is the one reported."""
    n = 512
    g = torch.Generator().manual_seed(9)
    f, phi = field(n, 1, seed=5), field(n, 1)
    f[1:n + 1, 1:n + 1] -= f[1:n + 1, 1:n + 1].mean()
    phi[1:n + 1, 1:n + 1] = torch.randn((n, n), dtype=torch.float64, generator=g).cuda()
    batch = cc.Batch([cc.Problem(n=n, bc=("P",) * 4, rtol=1e-9, prec=cc.MIXED)])
    (r,), info = cc.ccmg_batch_solve(batch, [f], [phi], use_guess=True)
    assert r.status == cc.OK
    u = phi[1:n + 1, 1:n + 1]
    lap = sum(torch.roll(u, s, d) for s in (1, -1) for d in (0, 1)) - 4 * u
    res = f[1:n + 1, 1:n + 1] - lap * float(n * n)
    assert res.norm().item() / f[1:n + 1, 1:n + 1].norm().item() <= 1.5e-9
    assert abs(u.mean().item()) <= 1e-12 * u.abs().max().item()


def test_problems_done_before_their_first_step_return_zero():
    """From zero, whatever the array held: a zero right-hand side, a tolerance
    that zero meets, and a right-hand side that isn't finite; a problem beside
    them that takes steps is solved."""
    n = 64
    fs = [field(n, 0), field(n, 1, seed=1), field(n, 0, seed=2), field(n, 1, seed=3)]
    fs[2][5, 7] = float("nan")
    phis = [field(n, i % 2, seed=20 + i) for i in range(4)]
    probs = [cc.Problem(n=n, bc=tuple("DDDD"), rtol=r, prec=cc.MIXED) for r in (1e-9, 2.0, 1e-9, 1e-9)]
    res, _ = cc.ccmg_batch_solve(cc.Batch(probs), fs, phis)
    assert [r.status for r in res] == [cc.OK, cc.OK, cc.ENONFINITE, cc.OK]
    assert [r.cycles for r in res[:3]] == [0, 0, 0] and res[3].cycles > 0
    for p in phis[:3]:
        # (the four corner ghosts are nobody's)
        assert torch.count_nonzero(p[1:n + 1, :n + 2]).item() == 0
        assert torch.count_nonzero(p[:, 1:n + 1]).item() == 0
    assert phis[3][1:n + 1, 1:n + 1].abs().max().item() > 0
