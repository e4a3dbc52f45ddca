"""The power spectrum at the sizes and numbers of shells that take its other paths: grids
narrower than a tile of columns (8, 16), the register transforms of 256, tiles of 8 and 4
columns (512, 1024), block sums in the reduction scratch and in the force grid, shells
beyond the last mode. Against a plain FP64 transform; at 1024 against plane waves and the
exact counts of lattice points.

Bounds: mode counts equal, mean |k| to FP64 rounding (1e-12), power within 1e-5 per shell
(the estimator's bound: FP32 transforms of at most 30 butterfly stages, 2^-24 each).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(rho, deconv, nbins):
    n = rho.shape[0]
    r = rho.double()
    f = torch.fft.rfftn(r / r.mean() - 1.0)
    power = (f.real ** 2 + f.imag ** 2) / float(n) ** 6
    del f
    m = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
    mz = torch.arange(n // 2 + 1, dtype=torch.float64, device="cuda")
    out = torch.zeros((3, nbins + 1), dtype=torch.float64, device="cuda")
    wz = torch.where((mz == 0) | (mz == n // 2), 1.0, 2.0).double()
    for i in range(n):  # (a plane at a time)
        k = torch.sqrt(m[i] ** 2 + m[:, None] ** 2 + mz ** 2)
        w = (torch.sinc(m[i] / n) * torch.sinc(m[:, None] / n) * torch.sinc(mz / n)) ** (2 * deconv)
        b = torch.round(k).long().clamp_max(nbins + 1)
        sel = (b >= 1) & (b <= nbins)
        c = wz.expand(n, -1)
        for o, v in zip(out, (c * power[i] / w, c * 2 * np.pi * k, c)):
            o.index_add_(0, b[sel], v[sel])
    return out[:, 1:].cpu().numpy()


@pytest.mark.parametrize("n,nbins,deconv", [(8, 4, 3), (16, 14, 0), (64, 64, 2), (256, 128, 3), (256, 256, 2),
                                            (512, 256, 3), (512, 512, 0)])
def test_shells(n, nbins, deconv):
    import paper_2410_20501_amd as lib
    g = torch.Generator("cuda").manual_seed(n + nbins)
    rho = 1.0 + 0.2 * torch.randn((n, n, n), device="cuda", generator=g)  # (power in every shell)
    ctx = lib.Context(n)
    pk, km, nm = (np.array(v) for v in lib.pm_power_spectrum(ctx, rho, deconv=deconv, nbins=nbins))
    ctx.close()
    p, k, c = _reference(rho, deconv, nbins)
    assert np.array_equal(nm, c.astype(np.int64))
    full = c > 0
    e = np.abs(pk[full] - p[full] / c[full]) / (p[full] / c[full])
    print(f"[case] n={n} {nbins} shells, deconv {deconv}: max rel per shell {e.max():.1e}", flush=True)
    assert np.allclose(km[full], k[full] / c[full], rtol=1e-12, atol=0.0)
    assert e.max() <= 1e-5
    assert not pk[~full].any() and not km[~full].any()


def test_plane_waves_at_1024():
    import paper_2410_20501_amd as lib
    n, nbins, deconv = 1024, 1024, 3
    h = n // 2
    waves = [((3, -4, 12), 0.05), ((-500, 37, 255), 0.02), ((0, 0, 300), 0.03), ((1, 512, 2), 0.04),
             ((-511, -511, 511), 0.03)]
    i = torch.arange(n, dtype=torch.float64, device="cuda")
    rho = torch.ones((n, n, n), device="cuda")
    for m, a in waves:  # a cos(2 pi m x), the phase of each axis modulo n in integers
        e = [torch.exp(2j * np.pi * ((md * i) % n) / n).to(torch.complex64) for md in m]
        for x in range(n):
            rho[x] += a * ((e[0][x] * e[1])[:, None] * e[2]).real
    ctx = lib.Context(n)
    pk, km, nm = (np.array(v) for v in lib.pm_power_spectrum(ctx, rho, deconv=deconv, nbins=nbins))
    ctx.close()
    # modes per |m|^2, from one octant
    ax = np.arange(h + 1, dtype=np.int64)
    w = np.where((ax == 0) | (ax == h), 1, 2)
    count = np.zeros(3 * h * h + 1, dtype=np.int64)
    p2, wp = (ax[:, None] ** 2 + ax ** 2).ravel(), (w[:, None] * w).ravel()
    for x in range(h + 1):
        count += np.bincount(p2 + x * x, weights=wp * w[x], minlength=len(count)).astype(np.int64)
    k = np.sqrt(np.arange(len(count), dtype=np.float64))
    b = np.rint(k).astype(int)
    c = np.bincount(b, weights=count, minlength=nbins + 1)[1:]
    s = np.bincount(b, weights=2 * np.pi * k * count, minlength=nbins + 1)[1:]
    full = c > 0
    assert np.array_equal(nm, c.astype(np.int64))
    assert np.allclose(km[full], s[full] / c[full], rtol=1e-12, atol=0.0)
    for m, a in waves:
        shell = int(np.rint(np.sqrt(sum(v * v for v in m))))
        # (1, 512, 2) and its conjugate (-1, 512, -2) are two modes of amplitude a / 2 as well
        power = 2 * (a / 2) ** 2 / np.prod([np.sinc(v / n) for v in m]) ** (2 * deconv)
        got = pk[shell - 1] * nm[shell - 1]
        print(f"[case] n=1024 wave {m}: shell {shell}, {got:.8e} of {power:.8e}", flush=True)
        assert abs(got / power - 1.0) <= 1e-5
