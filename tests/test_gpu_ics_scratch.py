"""Device memory of the initial conditions: what a call keeps with the context is no more than
it documents, 12 (first order), 24 or 40 (second, without or with dealiasing), 92 or 444
(third) bytes per cell and 128 MiB of half-transformed fields, and 4 MiB for tables and the
allocator's granules; the fields share places, which must not show in the result: every
order after every other one, on one context, equals a fresh context's bits."""
import numpy as np
import pytest
import torch

from oracle import ics as oics

pytestmark = pytest.mark.gpu

K_TAB, P_TAB = oics.power_law_table(0.1, -2.0, kmin=1.0, kmax=1e4)
CASES = [(1, False), (2, False), (2, True), (3, False), (3, True)]


def _call(lib, ctx, w, order, dealias):
    n = w.shape[0]
    pos, vel = torch.empty((n ** 3, 3), device="cuda"), torch.empty((n ** 3, 3), device="cuda")
    lib.pm_ic_lpt(ctx, w, K_TAB, P_TAB, 0.5, pos, vel, order=order, dealias=dealias)
    return pos, vel


@pytest.mark.parametrize("order,dealias,per_cell", [(1, False, 12), (2, False, 24), (2, True, 40), (3, False, 92)])
@pytest.mark.parametrize("n", [128, 256])
def test_kept_bytes(n, order, dealias, per_cell):
    import paper_2410_20501_amd as lib
    w = torch.randn((n, n, n), device="cuda")
    pos, vel = torch.empty((n ** 3, 3), device="cuda"), torch.empty((n ** 3, 3), device="cuda")
    ctx = lib.Context(n, n ** 3)  # (its kernels are loaded by a call of a context that is gone)
    lib.pm_ic_lpt(ctx, w, K_TAB, P_TAB, 0.5, pos, vel, order=order, dealias=dealias)
    ctx.close()
    ctx = lib.Context(n, n ** 3)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    lib.pm_ic_lpt(ctx, w, K_TAB, P_TAB, 0.5, pos, vel, order=order, dealias=dealias)
    kept = before - torch.cuda.mem_get_info()[0]
    fields = min(6 * (2 if dealias else 1) * 4 * n ** 3, 128 << 20)
    print(f"[case] n={n} order {order} dealias {dealias}: {kept / n ** 3:.1f} bytes per cell", flush=True)
    ctx.close()
    assert 0 < kept <= per_cell * n ** 3 + (fields if order == 2 else 0) + (4 << 20)


@pytest.mark.parametrize("n", [8, 16, 32, 64])
def test_shared_places_do_not_show(n):
    import paper_2410_20501_amd as lib
    w = torch.from_numpy(np.random.default_rng(n).standard_normal((n, n, n)).astype(np.float32)).cuda()
    fresh = {}
    for c in CASES:
        ctx = lib.Context(n, n ** 3)
        fresh[c] = _call(lib, ctx, w, *c)
        ctx.close()
    ctx = lib.Context(n, n ** 3)
    for a in CASES:
        for b in CASES:
            for c in (a, b):
                x, v = _call(lib, ctx, w, *c)
                assert torch.equal(x, fresh[c][0]) and torch.equal(v, fresh[c][1]), (a, b, c)
    ctx.close()


def test_release():
    import paper_2410_20501_amd as lib
    n = 128
    w = torch.randn((n, n, n), device="cuda")
    ctx = lib.Context(n, n ** 3)
    lib.pm_ic_release(ctx)  # (nothing kept)
    x, v = _call(lib, ctx, w, 2, True)
    kept = torch.cuda.mem_get_info()[0]
    lib.pm_ic_release(ctx)
    back = torch.cuda.mem_get_info()[0] - kept
    print(f"[case] released {back >> 20} MiB", flush=True)
    assert back >= 40 * n ** 3
    lib.pm_ic_release(ctx)
    y, u = _call(lib, ctx, w, 2, True)
    assert torch.equal(x, y) and torch.equal(v, u)
    ctx.close()
