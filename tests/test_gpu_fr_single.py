"""The scalaron on grids without a coarser one: every coarsest sweep of a cycle is part of
one launch (10^3 and 14^3), and the result is the oracle's (both sides take each root to
FP64 rounding: 1e-9, the bound of the scalaron's other tests)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import fr as ofr

pytestmark = pytest.mark.gpu


def _nodes_of(call):
    """Nodes of the graph that captures `call` on a stream of its own."""
    hip = ctypes.CDLL("libamdhip64.so")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        h, graph, count = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
        torch.cuda.synchronize()
        assert hip.hipStreamBeginCapture(h, 2) == 0  # (relaxed)
        call()
        assert hip.hipStreamEndCapture(h, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("n", [10, 14])
@pytest.mark.parametrize("n_exp,cycles,sweeps", [(1, 2, 32), (2, 1, 7)])
def test_single_level_grid(n, n_exp, cycles, sweeps):
    import paper_2410_20501_amd as lib
    rho = np.exp(np.random.Generator(np.random.PCG64(n)).standard_normal((n, n, n)))
    rho = (rho / rho.mean()).astype(np.float32)
    a, f0, c2 = 0.5, -1e-6, ofr.c_tilde(100.0) ** 2
    p = lib.default_step_params(omega_m=0.3, omega_l=0.7, fr_f0=f0, fr_n=n_exp, fr_c2=c2, fr_cycles=cycles,
                                fr_coarse_sweeps=sweeps)
    ctx, r = lib.Context(n), torch.from_numpy(rho).cuda()
    u = torch.ones((n, n, n), dtype=torch.float64, device="cuda")
    lib.pm_solve_fr(ctx, r, a, p, u)
    ref, _ = ofr.solve(rho.astype(np.float64), ofr.Coeffs(a, f0, n_exp, c2, 0.3, 0.7), cycles=cycles,
                       coarse_sweeps=sweeps)
    assert float(np.abs(u.cpu().numpy() - ref).max()) <= 1e-9
    nodes = _nodes_of(lambda: lib.pm_solve_fr(ctx, r, a, p, u))
    print(f"[case] n={n} nexp={n_exp} {cycles} cycles of {sweeps} sweeps: {nodes} launches", flush=True)
    lib.pm_kernel_timer(ctx, "fr_sweep", 64)
    lib.pm_solve_fr(ctx, r, a, p, u)
    ms, launches, nbytes = lib.pm_kernel_timer_read(ctx)
    assert launches == cycles and ms > 0 and nbytes == 32.0 * sweeps * cycles * n ** 3
    ctx.close()
    assert nodes <= 2 + cycles  # the mean, the source, the cycles
