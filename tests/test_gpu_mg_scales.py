"""Tolerance-driven multigrid solves of sources of any size that FP32 holds.

The solve is linear, so a source scaled by a power of two gives the same cycles, residual
history and, scaled back, the same bits, as long as no value leaves FP32's normal range
(2^+-80: squares of such sources lie far outside it). At 2^+-100 corrections near the
denormal range round differently: the solutions agree within the tolerance of the solve.
The reverse mode's solves take cotangents of any size through the same test; its sums are
FP32 atomics in any order, so both sides differ by the solve's tolerance (1e-6) and
roundings: 2e-5.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _fluctuations(n, seed):
    x = np.random.default_rng(seed).standard_normal((n, n, n))
    for d in range(3):
        x = x + np.roll(x, 1, d) + np.roll(x, 2, d)
    return torch.from_numpy((0.3 * (x - x.mean()) / x.std()).astype(np.float32)).cuda()


def _solve(lib, ctx, f, coef, **kw):
    phi = torch.zeros_like(f)
    st = lib.pm_solve_mg(ctx, f, coef, phi, tol=1e-5, **kw)
    return phi.double().cpu().numpy() / coef, st


def _check_scales(n, kws, exact=(-80, 80)):
    import paper_2410_20501_amd as lib
    f, ctx = _fluctuations(n, n), lib.Context(n)
    for kw in kws:
        ref, sr = _solve(lib, ctx, f, 1.0, **kw)
        assert sr.status == lib.PM_OK and sr.cycles > 1
        for e in (-100, -80, -60, 66, 80, 100):
            x, st = _solve(lib, ctx, f, 2.0 ** e, **kw)
            print(f"[case] n={n} {kw} 2^{e}: status {st.status}, {st.cycles} cycles", flush=True)
            assert st.status == lib.PM_OK and st.cycles == sr.cycles
            if exact[0] <= e <= exact[1]:
                assert list(st.history()) == list(sr.history()) and np.array_equal(x, ref)
            else:
                assert np.linalg.norm(x - ref) <= 1e-5 * np.linalg.norm(ref)
    ctx.close()


@pytest.mark.parametrize("n", [20, 64, 96, 160])
def test_solutions_scale_with_the_source(n):
    _check_scales(n, (dict(), dict(pre=0), dict(pre=3, omega=1.1)))


def test_solutions_scale_with_the_source_streaming():
    # (h^2 / 6 of a source of 2^-80 reaches the denormal range where a residual crosses zero)
    _check_scales(256, (dict(), dict(pre=3, omega=1.1)), exact=(-60, 80))


@pytest.mark.parametrize("n", [40])
def test_force_transpose_scales_with_the_cotangent(n):
    import paper_2410_20501_amd as lib
    rng = np.random.default_rng(7)
    q = (np.indices((n, n, n)).reshape(3, -1).T + 0.5) / n
    pos = torch.from_numpy(((q + 0.3 / n * rng.standard_normal(q.shape)) % 1.0).astype(np.float32) % 1.0).cuda()
    lam = torch.from_numpy(rng.standard_normal(q.shape).astype(np.float32)).cuda()
    p = lib.default_step_params(tol=1e-6)
    out = {}
    for size in (1.0, 2.0 ** -80, 2.0 ** 80):
        ctx = lib.Context(n, n ** 3)
        phi, acc, bar = torch.zeros((n, n, n), device="cuda"), torch.empty_like(pos), torch.zeros_like(pos)
        lib.pm_accel(ctx, pos, 0.5, phi, acc, params=p)
        st = lib.pm_accel_vjp(ctx, pos, 0.5, phi, lam * size, bar, params=p)
        out[size] = bar.double() / size
        print(f"[case] n={n} cotangents of {size:g}: status {st.status}, {st.cycles} cycles", flush=True)
        ctx.close()
    for size in (2.0 ** -80, 2.0 ** 80):
        assert float((out[size] - out[1.0]).norm()) <= 2e-5 * float(out[1.0].norm())
