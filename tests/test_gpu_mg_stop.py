"""The multigrid's convergence test, made while the cycle goes on.

A solve that stops by tolerance has launched part of the next cycle when the test is made;
one that stops by its number of cycles has not. The same solve ended either way returns the
same bits, the same history and the same number of cycles: nothing of what was launched in
vain may show. Levels: two (the whole next cycle may be queued), three, four, and a streaming
finest level; sweep counts and cycle shapes that change which launches those are.
"""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rho(n, seed):
    x = np.random.default_rng(seed).standard_normal((n, n, n))
    for d in range(3):
        x = x + np.roll(x, 1, d) + np.roll(x, 2, d)
    return torch.from_numpy((1.0 + 0.3 * (x - x.mean()) / x.std()).astype(np.float32)).cuda()


def _solve(lib, ctx, rho, **kw):
    phi = torch.zeros_like(rho)
    st = lib.pm_solve_mg(ctx, rho, 0.15, phi, **kw)
    return phi.cpu().numpy(), st


def _both_ends(lib, ctx, rho, kw, cycles):
    a, sa = _solve(lib, ctx, rho, tol=1e-30, max_cycles=cycles, **kw)
    h = list(sa.history())
    assert sa.cycles == cycles and sa.status == lib.PM_WARN_NOT_CONVERGED
    assert h[cycles] < 0.5 * h[cycles - 1]  # (so that a tolerance between the two exists)
    b, sb = _solve(lib, ctx, rho, tol=1.5 * h[cycles], max_cycles=30, **kw)
    assert sb.cycles == cycles and sb.status == lib.PM_OK and list(sb.history()) == h
    assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [20, 32, 64, 80, 128, 256])
def test_stop_by_tolerance_equals_stop_by_cycles(n):
    import paper_2410_20501_amd as lib
    print(f"[case] n={n}", flush=True)
    ctx, rho = lib.Context(n), _rho(n, n)
    for kw in (dict(), dict(pre=1, post=1), dict(pre=2, post=3), dict(cycle="W"), dict(cycle="F"),
               dict(pre=3), dict(guess="warm")):
        for cycles in (1, 2):
            _both_ends(lib, ctx, rho, kw, cycles)
    zero, st = _solve(lib, ctx, torch.ones_like(rho))
    assert st.cycles == 0 and st.status == lib.PM_OK and not zero.any()
    _both_ends(lib, ctx, rho, dict(), 2)  # (after a solve that ended early)
    ctx.close()


def test_contexts_in_threads_on_their_own_streams():
    import paper_2410_20501_amd as lib
    sizes = (32, 48, 96)
    failed = []

    def work(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                ctx, rho = lib.Context(n), _rho(n, n)
                for _ in range(8):
                    _both_ends(lib, ctx, rho, dict(), 2)
                ctx.close()
        except BaseException as e:  # noqa: BLE001 (reported below)
            failed.append((n, repr(e)))

    threads = [threading.Thread(target=work, args=(n,)) for n in sizes]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
