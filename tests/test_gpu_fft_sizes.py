"""The FFT passes at the lengths that the parity tests leave out, and grids that are only
4-byte aligned (rows are read and written as pairs of floats).

Bound: 1e-5, the configured tolerance of potentials and forces (the transforms' rounding,
about 2^-24 per butterfly level, stays near 1e-6).
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


def grid(shape, shift):
    """A contiguous tensor whose data begin `shift` floats after an aligned address."""
    return torch.empty(int(np.prod(shape)) + shift, device="cuda")[shift:].view(shape)


def case(n, seed):
    rho = (1.0 + 0.3 * np.random.default_rng(seed).standard_normal((n, n, n))).astype(np.float32)
    r = rho.astype(np.float64)
    return rho, 0.3 * (r - r.mean())


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [8, 64, 256])
def test_force_in_fourier_space_other_lengths(lib, n, shift):
    print(f"full_fft n={n} shift={shift}", flush=True)
    rho, f = case(n, n)
    ctx = lib.Context(n)
    x, g = grid((n, n, n), shift), grid((n, n, n, 3), shift)
    x.copy_(torch.from_numpy(rho))
    lib.pm_solve_fft_kernel(ctx, x, 0.3, g, kernel="full", deconv=2)
    assert rel_l2(g.cpu().numpy(), opm.force_full_fft(f, 1.0 / n, 2)) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("n", [8, 64, 512])
def test_seven_point_kernel_other_lengths(lib, n):
    print(f"fft_7pt n={n}", flush=True)
    rho, f = case(n, n + 1)
    ctx = lib.Context(n)
    x, phi = grid((n, n, n), 1), grid((n, n, n), 1)
    x.copy_(torch.from_numpy(rho))
    lib.pm_solve_fft_kernel(ctx, x, 0.3, phi, kernel="7pt")
    assert rel_l2(phi.cpu().numpy(), opm.solve_fft_7pt(f, 1.0 / n)) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("n", [16, 32, 80])
def test_multigrid_on_unaligned_grids(lib, n):
    print(f"multigrid unaligned n={n}", flush=True)
    rho, _ = case(n, n + 2)
    ctx = lib.Context(n)
    out = []
    for shift in (0, 1):
        x, phi = grid((n, n, n), shift), grid((n, n, n), shift)
        x.copy_(torch.from_numpy(rho))
        lib.pm_solve_mg(ctx, x, 0.15, phi, fixed_cycles=4)
        out.append(phi.cpu().numpy())
    # the same kernels; the final mean may be summed in another order
    assert rel_l2(out[0], out[1].astype(np.float64)) <= 1e-6
    ctx.close()
