"""Gauge transform, vortex fields and projection with each combination of ordinary and streaming link
accesses (small fields; fields whose result, then whose links, exceed the last-level cache), on tiled and
lexicographic launches, against the same products in plain torch."""
import pytest

pytestmark = pytest.mark.gpu

# links (and a transform of 144 bytes per site) against 256 MB: both fit; the links written do not; the
# links read do not either; and slices of fewer than 2048 half-sites
CASES = [((6, 4, 4, 8), 0), ((6, 4, 4, 8), 1), ((20, 20, 20, 40), 1), ((20, 20, 20, 40), 0), ((24, 24, 24, 48), 1),
         ((24, 24, 24, 48), 0), ((10, 12, 14, 300), 0)]


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0264_amd import _abi, api
    return api, _abi, torch


def product(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


@pytest.mark.parametrize("L,prec", CASES)
def test_products(S, env, L, prec):
    api, A, torch = env
    U = S.haar_links_gpu(L, 81)
    if prec:
        U = U.to(torch.complex64).to(torch.complex128)
    g = S.haar_gauge_gpu(L, 82, 0)
    Ud, Gd = api.to_links(U, prec), api.to_gauge(g)
    # one rounding of each entry (of modulus at most 1) to the links' type, and FP64 products
    tol = 1e-14 if prec == 0 else 2.0 ** -23

    def close(out, want):
        got = api.from_links(out, torch.complex128)
        for mu in range(4):
            assert (got[..., mu, :, :] - want[mu]).abs().max().item() <= tol, (L, prec, mu)

    V = [product(product(g, U[..., mu, :, :]), torch.roll(g, -1, 3 - mu).conj().transpose(-1, -2)) for mu in range(4)]
    close(api.apply_gauge(Ud, Gd), V)
    for G, F in ((Gd, V), (None, [U[..., mu, :, :] for mu in range(4)])):
        Z, margin = api.center_project(Ud, G)
        t = [f[..., 0, 0] + f[..., 1, 1] + f[..., 2, 2] for f in F]
        m = [torch.round(torch.angle(x) * (3 / (2 * torch.pi))) for x in t]  # -1, 0 or 1
        off = [torch.pi / 3 - (torch.angle(x) - k * (2 * torch.pi / 3)).abs() for x, k in zip(t, m)]
        zint = Z.view(4, L[3], L[2], L[1], L[0])
        for mu in range(4):
            sure = off[mu] > 1e-9
            assert torch.equal(zint[mu][sure], m[mu].to(torch.int8)[sure]), (L, prec, mu)
        assert abs(margin - min(x.min().item() for x in off)) <= 1e-9
        z = [torch.polar(torch.ones_like(k), k * (2 * torch.pi / 3))[..., None, None] for k in zint.double()]
        close(api.vortex_field(Ud, G, Z, A.MCG_VORTEX_REMOVED), [x.conj() * f for x, f in zip(z, F)])
        one = torch.eye(3, dtype=torch.complex128, device=U.device)
        close(api.vortex_field(Ud, G, Z, A.MCG_VORTEX_ONLY), [x * one for x in z])
        del t, m, off, z
