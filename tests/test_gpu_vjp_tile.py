"""interp^T through the tile buckets (fixed-point sums in LDS): one tile that wraps onto
itself, few tiles, several passes of a workgroup over one tile; cotangents at the ends of
FP32's range; non-finite ones.

Bounds against the FP64 oracle: a contribution rounds four products in FP32 and its integer
at 2^-38 of the tile's largest cotangent, the cell's sum rounds once, so the largest error
over the largest value stays below 1e-5 (the bound of the transposes' tests).
"""
import numpy as np
import pytest
import torch

import icgen
from oracle import adjoint as oa

pytestmark = pytest.mark.gpu


def _rel_max(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def _case(n, np_, seed):
    rng = np.random.default_rng(seed)
    pos = rng.random((np_, 3)).astype(np.float32) % 1.0
    pos[: np_ // 2] = (0.5 + 0.5 / n * rng.standard_normal((np_ // 2, 3))).astype(np.float32) % 1.0
    # away from the kinks of CIC's derivative, which FP32 and FP64 may take on either side
    frac = np.abs((pos.astype(np.float64) * n + 0.5) % 1.0 - 0.0)
    pos = pos[(np.minimum(frac, 1.0 - frac) > 1e-3).all(axis=1)]
    return pos, rng.standard_normal((n, n, n, 3)).astype(np.float32), rng.standard_normal(pos.shape).astype(np.float32)


@pytest.mark.parametrize("n,np_", [(8, 100), (8, 5000), (16, 3000), (40, 20000)])
@pytest.mark.parametrize("mas", ["tsc", "cic"])
def test_tiles_match_oracle(n, np_, mas):
    import paper_2410_20501_amd as lib
    pos, g, lam = _case(n, np_, n + np_)
    ctx = lib.Context(n, len(pos))
    for kind in ("box", "celloff"):
        if kind == "box":
            x, kw = pos, {}
            x64 = pos.astype(np.float64)
        else:
            cell, x = icgen.to_cell_offset(pos, n)
            kw = dict(cell=torch.from_numpy(np.asarray(cell, dtype=np.int32)).cuda())
            x64 = icgen.from_cell_offset(cell, x, n)
        for size in (1.0, 1e-30, 1e30):
            l = (lam * np.float32(size)).astype(np.float32)
            gbar, xbar = torch.zeros((n, n, n, 3), device="cuda"), torch.zeros(pos.shape, device="cuda")
            lib.pm_interp_vjp(ctx, torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda(),
                              torch.from_numpy(l).cuda(), g=torch.from_numpy(g).cuda(), g_bar=gbar, pos_bar=xbar,
                              mas=mas, **kw)
            gr, xr = oa.interp_vjp(x64, g.astype(np.float64), l.astype(np.float64), mas)
            eg = _rel_max(gbar.cpu().numpy().astype(np.float64), gr)
            ex = _rel_max(xbar.cpu().numpy().astype(np.float64), xr)
            print(f"[case] n={n} np={len(pos)} {mas} {kind} {size:g}: g_bar {eg:.2e} pos_bar {ex:.2e}", flush=True)
            assert eg < 1e-5 and ex < 1e-5
    ctx.close()


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_cotangent_stays_in_its_window(value):
    """One particle's non-finite cotangent reaches the 27 cells of its window and no other."""
    import paper_2410_20501_amd as lib
    n = 16
    pos, g, lam = _case(n, 2000, 5)
    lam[7] = value
    ctx = lib.Context(n, len(pos))
    gbar = torch.zeros((n, n, n, 3), device="cuda")
    lib.pm_interp_vjp(ctx, torch.from_numpy(pos).cuda(), torch.from_numpy(lam).cuda(), g_bar=gbar)
    ctx.close()
    got = gbar.cpu().numpy().astype(np.float64)
    c = np.floor(pos[7].astype(np.float64) * n).astype(int)
    window = np.zeros((n, n, n), dtype=bool)
    window[np.ix_(*[[(i - 1) % n, i % n, (i + 1) % n] for i in c])] = True
    assert (~np.isfinite(got[window])).all()
    keep = np.arange(len(pos)) != 7
    ref, _ = oa.interp_vjp(pos[keep].astype(np.float64), g.astype(np.float64), lam[keep].astype(np.float64), "tsc")
    assert np.abs(got[~window] - ref[~window]).max() <= 1e-5 * np.abs(ref).max()
