"""Bands of 8 and 16 rows held in registers whole against the row march (bands
of 32 rows): the same bits, launch by launch, for solves from zero and from a
guess, at the smallest level (where a band's halo reaches past the next band
to the domain's side), at strip edges and over several bands.  Singular
problems remove means summed over the tiles, which are cut differently, so
there FP64 iterates agree to rounding (1e-12 of the largest value); the FP32
cycles of a singular mixed solve round those means to FP32, where two cuts of
the row march differ as well, and are not compared."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")


def field(v, pad):
    n = v.shape[0]
    t = torch.zeros((n + 2, n + 2 + pad), dtype=torch.float64, device="cuda")
    t[1:n + 1, 1:n + 1] = torch.from_numpy(v).cuda()
    return t


def solve(n, bc, ab, prec, ty, fv, guess, pad):
    plan = cc.Plan(cc.Problem(n=n, bc=tuple(bc), alpha=ab[0], beta=ab[1], prec=prec, max_cycles=4, rtol=0.0))
    for level in range(n.bit_length() - 1 - 5):
        cc.ccmg_plan_set_shape(plan, level, 0, ty, 1)
        cc.ccmg_plan_set_shape(plan, level, 1, ty, 1)
    cc.ccmg_plan_set_shape(plan, 0, 2 if prec == cc.FP64 else 3, ty, 1)
    phi = field(guess if guess is not None else np.zeros_like(fv), pad)
    r = cc.ccmg_solve(plan, field(fv, pad), phi, use_guess=guess is not None)
    assert r.status == cc.NOT_CONVERGED and r.cycles == 4
    return phi.cpu().numpy(), r.history


@pytest.mark.parametrize("prec,bc,ab", [(cc.FP64, "DDDD", (0.0, -1.0)), (cc.MIXED, "DDDD", (0.0, -1.0)),
                                        (cc.FP64, "NDPP", (0.0, -1.0)), (cc.MIXED, "NDPP", (0.0, -1.0)),
                                        (cc.FP64, "PPND", (1.0, 3e-5)), (cc.MIXED, "PPND", (1.0, 3e-5)),
                                        (cc.FP64, "PPPP", (0.0, -1.0))])
@pytest.mark.parametrize("n", [64, 128, 512])
def test_bands_in_registers_match_the_row_march(n, prec, bc, ab):
    print(f"block n={n} bc={bc} ab={ab} prec={prec}", flush=True)
    singular = ab[0] == 0.0 and "D" not in bc
    fv = np.random.default_rng(31).standard_normal((n, n))
    fv -= fv.mean()
    g = W.fourier_modes(n, seed=2, count=8, kmax=4) * 1e-3
    for guess in (None, g):
        ref, href = solve(n, bc, ab, prec, 32, fv, guess, 3)
        for ty in (8, 16):
            got, h = solve(n, bc, ab, prec, ty, fv, guess, 3)
            if singular:
                assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max(), (ty, guess is None)
            else:
                assert np.array_equal(got, ref), (ty, guess is None)
            np.testing.assert_allclose(h, href, rtol=1e-9)
