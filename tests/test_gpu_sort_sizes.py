"""The tile sort at the edges of its scan and histogram: grids whose number of tiles lies on
either side of the one-workgroup scan's two sizes (5120 and 33792 entries) and of the block
histogram (2048 keys), one tile, more keys than particles. The sorted deposit and the
interpolation that reads its order are compared with the kernels that use no sort: the
deposits sum the same 2^-30 fixed-point weights, with one FP32 rounding per box or chunk that
covers a cell (at most 8 and 16 of 2^-24 of a value: 1.5e-6), the interpolations the same 27
products in FP32 (27 2^-24 of the largest force: 1.7e-6). A step's drift makes the histogram
itself: its positions are those of an unsorted step, bit for bit.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 96, 112, 128, 144, 256, 288])
def test_sorted_paths_match_unsorted(n):
    import paper_2410_20501_amd as lib
    print(f"[case] n={n}", flush=True)
    rng = np.random.default_rng(n)
    pos = rng.random((30000, 3)).astype(np.float32) % 1.0
    pos[:10000] = (0.3 + 2.0 / n * rng.standard_normal((10000, 3))).astype(np.float32) % 1.0
    x = torch.from_numpy(pos).cuda()
    ctx = lib.Context(n, len(pos))
    rho = {o: torch.empty((n, n, n), device="cuda") for o in ("sorted", "atomic")}
    for order, r in rho.items():
        lib.pm_deposit(ctx, x, r, order=order)
    a, b = (rho[o].cpu().numpy().astype(np.float64) for o in ("sorted", "atomic"))
    assert np.abs(a - b).max() <= 1.5e-6 * np.abs(b).max()
    assert abs(a.sum() / n ** 3 - 1.0) <= 1e-5
    phi = torch.randn((n, n, n), device="cuda", generator=torch.Generator("cuda").manual_seed(n)) / n
    states = {}
    for order in ("sorted", "atomic"):
        xs, vs = x.clone(), torch.zeros_like(x)
        acc = torch.zeros_like(x)
        ph = phi.clone()
        p = lib.default_step_params(order=order, fixed_cycles=1)
        lib.pm_accel(ctx, xs, 0.1, ph, acc, params=p)
        vs.copy_(0.01 * torch.sin(37.0 * x))
        lib.pm_kdk(ctx, xs, vs, 0.1, 0.101, ph, torch.zeros_like(x), params=p)
        states[order] = (xs.cpu().numpy(), acc.cpu().numpy().astype(np.float64))
    assert np.array_equal(states["sorted"][0], states["atomic"][0])
    fa, fb = states["sorted"][1], states["atomic"][1]
    assert np.abs(fa - fb).max() <= 1e-5 * np.abs(fb).max()
    ctx.close()
