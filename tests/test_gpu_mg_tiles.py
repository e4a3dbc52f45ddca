"""Tile kernels of the multigrid's smaller levels and the exact coarsest solve.

The tile kernels (two launches per level and visit) are compared with a context that runs
one kernel per half-sweep, residual, restriction and prolongation: sizes around the edges
of the three tile shapes, one tile or less, remainders of a tile along each axis, and the
largest sizes of the range. Both run the same operations; a half-sweep rounds each value a
few times (2^-24 each) and three cycles smooth those errors, so the iterates agree within
2e-6 (the bound of the streaming kernels' tests). The coarsest solve is compared with the
oracle's exact seven-point solution; its transforms add about 2^-24 per butterfly level and
the source's mean is subtracted in FP32, together below 2e-6.
"""
import numpy as np
import pytest
import torch

from oracle import pm as opm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2410_20501_amd as pm
    return pm


def rel_l2(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


def density(n, seed):
    """Correlated fluctuations of rms 0.3 about 1 (white noise averaged over neighbours)."""
    x = np.random.default_rng(seed).standard_normal((n, n, n))
    for d in range(3):
        x = x + np.roll(x, 1, d) + np.roll(x, 2, d)
    return (1.0 + 0.3 * (x - x.mean()) / x.std()).astype(np.float32)


SWEEPS = [dict(pre=2, post=2), dict(pre=1, post=0, omega=1.25), dict(pre=0, post=1),
          dict(pre=5, post=3, restrict_kind="avg"), dict(pre=2, post=1, omega=1.1, cycle="W")]


@pytest.mark.parametrize("n", [20, 28, 32, 36, 48, 72, 80, 96, 112, 160, 224])
def test_tile_levels_match_one_kernel_per_half_sweep(lib, n):
    print(f"tile levels n={n}", flush=True)
    rho = torch.from_numpy(density(n, n)).cuda()
    guess = torch.from_numpy(density(n, n + 1) - 1.0).cuda()
    tile, plain = lib.Context(n), lib.Context(n, 0, lib.PM_CREATE_REFERENCE_KERNELS)
    for kw in SWEEPS:
        for start in ("jacobi", "warm"):
            out = []
            for ctx in (tile, plain):
                phi = guess.clone()
                lib.pm_solve_mg(ctx, rho, 0.15, phi, fixed_cycles=3, guess=start, **kw)
                out.append(phi.cpu().numpy())
            assert np.isfinite(out[0]).all()
            assert rel_l2(out[0], out[1].astype(np.float64)) <= 2e-6, (kw, start)
    for ctx in (tile, plain):
        ctx.close()


@pytest.mark.parametrize("n", [20, 48, 96])
def test_tile_norms_match_the_separate_pass(lib, n):
    """The residual norms that the first pass of a cycle sums (tolerance-driven solves)."""
    print(f"tile norms n={n}", flush=True)
    rho = torch.from_numpy(density(n, 3 * n)).cuda()
    hist = []
    for flags in (0, lib.PM_CREATE_REFERENCE_KERNELS):
        ctx = lib.Context(n, 0, flags)
        for kw in (dict(), dict(pre=3), dict(pre=0), dict(guess="warm")):
            phi = torch.from_numpy(density(n, 5) - 1.0).cuda()
            st = lib.pm_solve_mg(ctx, rho, 0.15, phi, tol=1e-3, max_cycles=30, **kw)
            assert st.status == lib.PM_OK
            hist.append(st.history())
        ctx.close()
    for a, b in zip(hist[:4], hist[4:]):
        # FP32 residuals near 1e-3 of the source carry a relative rounding of about 1e-3
        assert len(a) == len(b) and np.allclose(a, b, rtol=5e-3, atol=1e-6), (a, b)


@pytest.mark.parametrize("n", [8, 10, 12, 14, 16, 18])
def test_coarsest_solve_is_exact(lib, n):
    print(f"coarsest solve n={n}", flush=True)
    rho = density(n, n)
    ctx = lib.Context(n)
    phi = torch.empty((n, n, n), device="cuda")
    lib.pm_solve_mg(ctx, torch.from_numpy(rho).cuda(), 0.15, phi, fixed_cycles=1)
    ref = opm.solve_exact7(opm.source(rho.astype(np.float64), 0.1), 1.0 / n)
    assert rel_l2(phi.cpu().numpy(), ref) <= 2e-6
    ctx.close()


@pytest.mark.parametrize("sizes", [[32], [12, 18, 20, 36, 80, 16], [64] * 5 + [48, 96], [32] * 40])
def test_batched_tile_levels_match_single_boxes(lib, sizes):
    """The batched passes in each of their tile shapes, with sweep counts that leave the
    iterate in either buffer, against single boxes that run one kernel per half-sweep: the
    documented bound between the batched and the single-box force, 1e-5."""
    print(f"batched tile levels {sizes}", flush=True)
    batch = lib.Batch(sizes, [n ** 3 for n in sizes])
    rng = np.random.default_rng(len(sizes))
    pos = []
    for n in sizes:
        q = (np.indices((n, n, n)).reshape(3, -1).T + 0.5) / n
        pos.append(((q + 0.3 / n * rng.standard_normal(q.shape)) % 1.0).astype(np.float32) % 1.0)
    x = torch.from_numpy(np.concatenate(pos)).cuda()
    plain = {n: lib.Context(n, n ** 3, lib.PM_CREATE_REFERENCE_KERNELS) for n in set(sizes)}
    for kw in (dict(), dict(pre=3, post=1), dict(pre=1, post=3, omega=1.2), dict(pre=0, post=0),
               dict(pre=2, post=1, restrict_kind="avg")):
        p = lib.default_step_params(fixed_cycles=2, **kw)
        acc, phi = torch.empty_like(x), torch.zeros(batch.ncell_total, device="cuda")
        lib.pm_batch_accel(batch, x, acc, phi, 0.1, p)
        for b in range(0, len(sizes), max(1, len(sizes) // 6)):
            n = sizes[b]
            rows, cells = slice(*batch.p_off[b:b + 2]), slice(*batch.c_off[b:b + 2])
            one, pot = torch.empty_like(x[rows]), torch.zeros((n, n, n), device="cuda")
            lib.pm_accel(plain[n], x[rows].contiguous(), 0.1, pot, one, params=p)
            assert rel_l2(phi[cells].cpu().numpy(), pot.reshape(-1).cpu().numpy()) <= 1e-5, (n, kw)
            assert rel_l2(acc[rows].cpu().numpy(), one.cpu().numpy()) <= 1e-5, (n, kw)
    batch.close()
    for ctx in plain.values():
        ctx.close()
