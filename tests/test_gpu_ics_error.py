"""Error of the first-order velocities, where the Fourier-space factors and the transforms are
all that rounds.

Bounds: the mean relative error, on these noises, of the spectral passes that the band
passes replaced (each factor one FP64 product, radix-4 transforms), and 1 % more.
"""
import numpy as np
import pytest
import torch

from oracle import ics as oics

pytestmark = pytest.mark.gpu

K_TAB, P_TAB = oics.power_law_table(0.1, -2.0, kmin=1.0, kmax=1e4)


@pytest.mark.parametrize("n,noises,bound", [(16, 20, 1.870e-7), (32, 20, 2.408e-7), (128, 6, 2.469e-7),
                                            (256, 2, 2.613e-7)])
def test_velocity_error_is_no_larger_than_that_of_the_earlier_passes(n, noises, bound):
    import paper_2410_20501_amd as lib
    ctx, err = lib.Context(n, n ** 3), []
    pos, vel = torch.empty((n ** 3, 3), device="cuda"), torch.empty((n ** 3, 3), device="cuda")
    for s in range(noises):
        w = np.random.Generator(np.random.PCG64(100 * n + s)).standard_normal((n, n, n)).astype(np.float32)
        _, ref = oics.lpt_state(w.astype(np.float64), K_TAB, P_TAB, 0.5, 1, False)
        lib.pm_ic_lpt(ctx, torch.from_numpy(w).cuda(), K_TAB, P_TAB, 0.5, pos, vel, order=1, dealias=False)
        err.append(np.linalg.norm(vel.cpu().numpy() - ref) / np.linalg.norm(ref))
    ctx.close()
    print(f"[case] n={n}: {np.mean(err):.3e} of {bound:.3e}", flush=True)
    assert np.mean(err) <= 1.01 * bound
