"""Gauge transform, projection, vortex fields and counts on the GPU against the oracle on lattices whose
slices are tiled along t (with whole and ragged last tiles), with Z at every byte alignment; layout
conversion of ragged tiles in every pair of precisions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    from paper_0807_0264_amd import api
    return api, gpu_util, torch


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("L", [(16, 16, 16, 2), (18, 12, 20, 10), (6, 10, 4, 4)])
def test_transform_and_projection(S, O, env, L, prec):
    api, g, torch = env
    U = g.rounded(S.heatbath_field(L, S.sub_seed(7400), 5.7, 2), prec)
    G = S.haar_gauge(L, S.sub_seed(7401))
    Ud, Gd = g.links(U, prec), g.gauge(G)
    tol = 1e-14 if prec == 0 else 1e-6
    assert np.abs(g.host_links(api.apply_gauge(Ud, Gd)) - O.apply_gauge(U, G)).max() < tol
    Zo, margin = O.center_project(U, G)
    want = O.count_vortices(Zo)["total"]
    V = api.volume(L)
    for off in (0, 1, 2):  # pairs and single bytes out; words and single bytes in
        Z = torch.empty(4 * V + 4, dtype=torch.int8, device="cuda")[off:off + 4 * V].view(4, V)
        _, mm = api.center_project_noalloc(Ud, Gd, Z=Z)
        assert np.array_equal(g.z_interchange(Z, L), Zo) and abs(mm - np.min(margin)) < 1e-12
        assert api.count_vortices(Z, L)["total"] == want
    for mode in (0, 1):
        got = g.host_links(api.vortex_field(Ud, Gd, api.center_project(Ud, Gd)[0], mode))
        assert np.abs(got - O.vortex_field(U, G, Zo, mode)).max() < tol


@pytest.mark.parametrize("L", [(8, 4, 4, 6), (6, 4, 2, 4), (4, 2, 2, 2)])
def test_counts_of_any_integers(env, L):
    """Counts of integers beyond -1, 0, 1, in words and in single bytes, against the definition."""
    api, g, torch = env
    V = api.volume(L)
    Z = np.random.default_rng(5).integers(-128, 128, (4, V)).astype(np.int8)
    z = np.moveaxis(Z.reshape(4, L[3], L[2], L[1], L[0]), 0, -1).astype(int)
    planes, charge = [], [0, 0]
    for mu in range(4):
        for nu in range(mu + 1, 4):
            n = (z[..., mu] + np.roll(z[..., nu], -1, 3 - mu) - np.roll(z[..., mu], -1, 3 - nu) - z[..., nu]) % 3
            planes.append(int((n != 0).sum()))
            charge = [charge[0] + int((n == 1).sum()), charge[1] + int((n == 2).sum())]
    for off in (0, 1):
        t = torch.empty(4 * V + 1, dtype=torch.int8, device="cuda")[off:off + 4 * V].view(4, V)
        t.copy_(torch.from_numpy(Z))
        got = api.count_vortices(t, L)
        assert got["per_plane"] == planes and got["per_charge"] == charge and got["total"] == sum(planes)


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 2, 10, 6), (10, 6, 8, 14)])
def test_conversion_round_trips(S, env, L):
    api, g, torch = env
    U = torch.from_numpy(S.haar_links(L, S.sub_seed(7402))).cuda()
    G = torch.from_numpy(S.haar_gauge(L, S.sub_seed(7403))).cuda()
    assert torch.equal(api.from_gauge(api.to_gauge(G)), G)
    U32 = U.to(torch.complex64)
    for src, prec, want in ((U, 0, U), (U, 1, U32), (U32, 1, U32), (U32, 0, U32.to(torch.complex128))):
        W = api.to_links(src, prec)
        for dt in (torch.complex64, torch.complex128):
            assert torch.equal(api.from_links(W, dt), want.to(dt))
        # the layout itself: element (mu, parity, k, h)
        Lx, Ly, Lz, Lt = L
        V = Lx * Ly * Lz * Lt
        f = torch.view_as_complex(W.data.view(4, 2, 9, V // 2, 2)).cpu().numpy()
        for x, y, z, t in ((0, 0, 0, 0), (Lx - 1, Ly - 1, Lz - 1, Lt - 1), (1, 0, Lz - 1, 1)):
            i = x + Lx * (y + Ly * (z + Lz * t))
            assert np.array_equal(f[:, (x + y + z + t) % 2, :, i // 2].reshape(4, 3, 3),
                                  want[t, z, y, x].cpu().numpy())
