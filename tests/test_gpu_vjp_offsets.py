"""interp^T of particles whose in-cell offset lies far outside [0, 1) or is not finite: their
weights are beyond the tile boxes' fixed point and still add up, and spread no further than
their window.

Bound: one particle's 27 contributions of four FP32 roundings each, among others of order
one: 1e-5 of the largest.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, AT = 16, 37


def _window(o, mas):
    if mas == "tsc":
        d = o - 0.5
        return 0, np.array([0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2])
    d, first = (o - 0.5, 1) if o >= 0.5 else (o + 0.5, 0)
    return first, np.array([1.0 - d, d])


def _case(offset, mas):
    import paper_2410_20501_amd as lib
    rng = np.random.default_rng(3)
    cell = rng.integers(0, N ** 3, 400).astype(np.int32)
    off = rng.random((400, 3)).astype(np.float32) * np.float32(0.999)
    off[AT] = offset
    lam = rng.standard_normal((400, 3)).astype(np.float32)
    ref, mark = np.zeros((N, N, N, 3)), np.zeros((N, N, N), dtype=bool)
    for p in range(400):
        c = np.array([cell[p] // (N * N), cell[p] // N % N, cell[p] % N])
        with np.errstate(invalid="ignore"):
            fw = [_window(float(o), mas) for o in off[p]]
        ix = np.ix_(*[(c[d] - 1 + fw[d][0] + np.arange(len(fw[d][1]))) % N for d in range(3)])
        if p == AT:
            mark[ix] = True
        if np.isfinite(off[p]).all():
            ref[ix] += np.einsum("i,j,k,d->ijkd", *[f[1] for f in fw], lam[p])
    ctx, g = lib.Context(N, 400), torch.zeros((N, N, N, 3), device="cuda")
    print(f"[case] offset {offset} {mas}", flush=True)
    lib.pm_interp_vjp(ctx, torch.from_numpy(off).cuda(), torch.from_numpy(lam).cuda(), g_bar=g, mas=mas,
                      cell=torch.from_numpy(cell).cuda())
    ctx.close()
    return g.cpu().numpy(), ref, mark


@pytest.mark.parametrize("mas", ["tsc", "cic"])
@pytest.mark.parametrize("offset", [1.5, -0.75, 9.0, -30.0, 1000.0, 1e6])
def test_large_offsets(offset, mas):
    got, ref, _ = _case(offset, mas)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("offset", [np.inf, -np.inf, np.nan])
def test_offsets_that_are_not_finite(offset):
    got, ref, mark = _case(offset, "tsc")
    assert (~np.isfinite(got[mark])).all()
    assert np.abs(got[~mark] - ref[~mark]).max() <= 1e-5 * np.abs(ref).max()
