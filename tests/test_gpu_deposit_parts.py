"""The chunked deposit's ways of taking a chunk (whole, by parts of a slot per thread, by
waves, weight by weight) at each number of particles per thread, against the sorted deposit,
which sums the same 2^-30 fixed-point weights exactly.

Bound: a cell takes at most 27 windows' worth of particles per particle around it, each part
that covers it one FP32 addition, so up to 27 roundings of 2^-24 of the cell's value for the
lattice (1.6e-6) and, weight by weight, one per weight (0.3 particles a cell there: fewer).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(n, x):
    import paper_2410_20501_amd as lib
    ctx = lib.Context(n, len(x))
    rho = {o: torch.empty((n, n, n), device="cuda") for o in ("sorted", "atomic")}
    for order, r in rho.items():
        lib.pm_deposit(ctx, x, r, order=order)
    a, b = (rho[o].double() for o in ("atomic", "sorted"))
    err, top = float((a - b).abs().max()), float(b.abs().max())
    print(f"[case] n={n} np={len(x)}: max difference {err / top:.1e} of the largest value", flush=True)
    ctx.close()
    assert err <= 2e-6 * top


def _rows(n, planes, rms, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    i = torch.arange(n, device="cuda", dtype=torch.float32)
    q = torch.stack(torch.meshgrid(i[:planes], i, i, indexing="ij"), -1).reshape(-1, 3)
    x = ((q + 0.5 + rms * torch.randn(q.shape, device="cuda", generator=g)) / n) % 1.0
    x[x >= 1.0] = 0.0
    return x.contiguous()


@pytest.mark.parametrize("n,planes,rms", [
    (16, 16, 0.3), (64, 40, 0.3), (64, 64, 0.3),      # whole chunks, one and two a thread
    (128, 10, 0.3), (128, 60, 0.3),                   # parts of 256
    (256, 2, 0.3), (256, 10, 0.3), (256, 64, 0.3),    # waves; one, two and eight a thread
    (256, 2, 3.0)])                                   # weight by weight
def test_lattice_rows(n, planes, rms):
    _check(n, _rows(n, planes, rms, n + planes))


def test_ragged_and_mixed_chunks():
    """Coherent chunks, scattered ones and a short last one in one call."""
    a, g = _rows(64, 3, 0.2, 1), torch.Generator("cuda").manual_seed(2)
    b = torch.rand((5000, 3), device="cuda", generator=g)
    b[b >= 1.0] = 0.0
    for tail in (0, 1, 63, 255):
        _check(64, torch.cat([a, b, a[: 4000 + tail]]).contiguous())
