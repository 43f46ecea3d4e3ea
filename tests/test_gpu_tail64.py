"""The 64 x 64 level in one launch with the tail under it: V-cycles with other
smoothing counts than two (none, one, odd) against the oracle, element by
element, where that level is the second and the third of the hierarchy.  (With
two, whole solves against the separate launches, bit for bit, are
test_gpu_visit's.)  Bound: 1e-11 of the largest value over three cycles, as for
every V-cycle against the oracle (FP64 rounding carried through the levels)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")


def dev_field(a, pad=5):
    n = a.shape[0] - 2
    t = torch.zeros((n + 2, n + 2 + pad), dtype=torch.float64, device="cuda")
    t[:, :n + 2] = torch.from_numpy(a).cuda()
    return t


@pytest.mark.parametrize("nu", [(0, 2), (1, 0), (1, 1), (3, 1)])
@pytest.mark.parametrize("bc,ab", [("DNND", (0.0, -1.0)), ("PPPP", (0.0, -1.0)), ("PPDN", (1.0, 0.01))])
@pytest.mark.parametrize("n", [128, 256])
def test_vcycles_match_oracle(n, bc, ab, nu):
    print(f"tail64 n={n} bc={bc} ab={ab} nu={nu}", flush=True)
    plan = cc.Plan(cc.Problem(n=n, bc=tuple(bc), alpha=ab[0], beta=ab[1], nu1=nu[0], nu2=nu[1]))
    p = oracle.Problem(n=n, h=1.0 / n, alpha=ab[0], beta=ab[1], bc=bc, nu1=nu[0], nu2=nu[1])
    fv = np.random.default_rng(41).standard_normal((n, n))
    if p.singular:
        fv -= fv.mean()
    f, ref = oracle.embed(fv), oracle.embed(np.random.default_rng(42).standard_normal((n, n)))
    d_f, d_phi = dev_field(f), dev_field(ref)
    for k in range(3):
        cc.ccmg_vcycle(plan, d_f, d_phi)
        oracle.vcycle(p, ref, f)
        got, want = oracle.interior(d_phi[:, :n + 2].cpu().numpy()), oracle.interior(ref)
        if p.singular:
            got, want = got - got.mean(), want - want.mean()
        assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max(), k
