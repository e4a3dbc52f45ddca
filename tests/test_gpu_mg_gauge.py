"""The potential's mean is removed: of the iterate that is returned, also where the solve
stops at its first test, on a guess far from the solution whose mean the smoothing moves
(by up to 1e-2 of its rms here).

Bound: the mean is subtracted in FP32, which rounds it (2^-25 of the guess's mean of 3) and
each value (2^-24 of at most its size, about zero on average): 2^-22 of the largest value.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [20, 48, 96, 224, 256])
@pytest.mark.parametrize("kw", [dict(), dict(omega=1.5), dict(pre=1, post=1, omega=0.6)])
def test_returned_potential_has_no_mean(n, kw):
    import paper_2410_20501_amd as lib
    g = torch.Generator("cuda").manual_seed(n)
    rho = 1.0 + 0.3 * torch.randn((n, n, n), device="cuda", generator=g)
    ctx = lib.Context(n)
    for stop in (dict(tol=1e30), dict(tol=1e-30, max_cycles=1)):
        phi = 3.0 + torch.randn((n, n, n), device="cuda", generator=g)
        st = lib.pm_solve_mg(ctx, rho, 0.15, phi, guess="warm", **stop, **kw)
        mean, top = float(phi.double().mean()), float(phi.abs().max())
        print(f"[case] n={n} {kw} {stop}: {st.cycles} cycles, mean {mean:.1e} of {top:.1e}", flush=True)
        assert abs(mean) <= 2.0 ** -22 * max(top, 3.0)
    ctx.close()
