"""The chunked deposit with the nearest-grid-point window, whose boxes are taken only where
they are small for their particles: chunks, parts and waves of both kinds at each number of
particles per thread, against the sorted deposit.

Bound: a cell's value is its particles' number times the mass, added in at most as many
FP32 steps: with up to 30 particles a cell 30 roundings of 2^-24, below 2e-6 of it.
"""
import pytest
import torch

from test_gpu_deposit_parts import _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,planes,rms", [
    (16, 16, 0.3), (32, 32, 0.05), (64, 40, 0.3), (64, 64, 0.05), (128, 10, 0.3), (128, 60, 0.3),
    (256, 2, 0.3), (256, 10, 3.0), (256, 64, 0.3)])
def test_lattice_rows_ngp(n, planes, rms):
    import paper_2410_20501_amd as lib
    x = _rows(n, planes, rms, n + planes)
    dense = (0.4 + 0.1 * x[: len(x) // 8]).contiguous()  # 125 times as dense: boxes of shared cells
    for p in (x, torch.cat([x, dense]).contiguous()):
        ctx = lib.Context(n, len(p))
        rho = {o: torch.empty((n, n, n), device="cuda") for o in ("sorted", "atomic")}
        for order, r in rho.items():
            lib.pm_deposit(ctx, p, r, order=order, mas="ngp")
        ctx.close()
        a, b = rho["atomic"].double(), rho["sorted"].double()
        err, top = float((a - b).abs().max()), float(b.max())
        print(f"[case] n={n} np={len(p)}: max difference {err / top:.1e}", flush=True)
        assert err <= 2e-6 * top
        assert abs(float(a.sum()) / n ** 3 - 1.0) <= 1e-5
