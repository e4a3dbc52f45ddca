"""pm_ic_lpt at the edges of its transforms' ranges, against the FP64 oracle: the smallest
grids (a band narrower than one tile of columns, rows of 4), both product grids, a product
grid taken in several chunks of planes (128, dealiased), and one context used for
different orders and outputs, whose scratch it keeps between calls.

Bound on velocities: relative L2 <= 1e-5, that of the larger grids (test_gpu_ics.py): FP32
rounding of transforms of at most 24 butterfly stages, each below 2^-23 of the field's norm.
Positions: 2e-5 cell, and half an ulp of a box position more.
"""
import numpy as np
import pytest
import torch

from oracle import ics as oics

pytestmark = pytest.mark.gpu

A0 = 0.5
K_TAB, P_TAB = oics.power_law_table(0.1, -2.0, kmin=1.0, kmax=1e4)


def _noise(n, seed):
    return np.random.Generator(np.random.PCG64(seed)).standard_normal((n, n, n)).astype(np.float32)


def _check(pos, vel, noise, order, dealias):
    n = noise.shape[0]
    xr, vr = oics.lpt_state(noise.astype(np.float64), K_TAB, P_TAB, A0, order, dealias)
    e = np.linalg.norm(vel.cpu().numpy().astype(np.float64) - vr) / np.linalg.norm(vr)
    d = pos.cpu().numpy().astype(np.float64) - xr
    d -= np.round(d)
    print(f"[case] n={n} order={order} dealias={dealias}: velocities {e:.2e}, positions {np.abs(d).max():.2e}",
          flush=True)
    assert e <= 1e-5
    assert np.abs(d).max() <= 2e-5 / n + 2.0 ** -23


@pytest.mark.parametrize("n,order,dealias", [(8, 1, False), (8, 2, False), (8, 3, True), (16, 2, True),
                                             (16, 3, False), (128, 2, True)])
def test_small_and_chunked_sizes(n, order, dealias):
    import paper_2410_20501_amd as lib
    noise = _noise(n, 3 + n)
    ctx = lib.Context(n, n ** 3)
    pos, vel = torch.empty((n ** 3, 3), device="cuda"), torch.empty((n ** 3, 3), device="cuda")
    lib.pm_ic_lpt(ctx, torch.from_numpy(noise).cuda(), K_TAB, P_TAB, A0, pos, vel, order=order, dealias=dealias)
    _check(pos, vel, noise, order, dealias)
    ctx.close()


def test_kept_scratch_and_unaligned_outputs():
    """Orders 2, 3, 1, 2 on one context and two streams; outputs one particle into their
    buffers (12 bytes on: aligned to a float only), what lies around them untouched."""
    import paper_2410_20501_amd as lib
    n = 32
    ctx = lib.Context(n, n ** 3)
    side = torch.cuda.Stream()
    for i, order in enumerate((2, 3, 1, 2)):
        noise = _noise(n, 60 + i)
        w = torch.from_numpy(noise).cuda()
        bufs = [torch.full((n ** 3 + 2, 3), 7.5, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        with torch.cuda.stream(side if i % 2 else torch.cuda.current_stream()):
            lib.pm_ic_lpt(ctx, w, K_TAB, P_TAB, A0, bufs[0][1:-1], bufs[1][1:-1], order=order, dealias=True)
        _check(bufs[0][1:-1], bufs[1][1:-1], noise, order, True)
        for b in bufs:
            assert (b[0] == 7.5).all() and (b[-1] == 7.5).all()
    ctx.close()
