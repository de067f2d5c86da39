"""The half-sweep with one wave per link (launches too small to fill the device) against the one with
a site per lane, bit for bit: raw sweeps in every pairing and ring setting, single and batched fixes
with their trajectories and stop tests, slabs, on lattices whose last block is ragged and on both sides
of the sizes at which the form and its stop test change."""
import ctypes as C
import itertools

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


@pytest.fixture
def contexts(env):
    """(a context with its default launches, one whose variant was set: a site per lane)"""
    api, _, _ = env
    from paper_0807_0264_amd import _abi as A
    lib, out, saved = A.load(), [], api.context(0)
    for narrow in (False, True):
        h = C.c_void_p()
        assert lib.mcg_create(C.byref(h), 0) == A.MCG_OK
        if narrow:
            for prec in (0, 1):
                assert lib.mcg_set_variant(h, prec, 1) == A.MCG_OK
        out.append(h)
    yield out
    api._ctx_cache[0] = saved
    for h in out:
        lib.mcg_destroy(h)


def both(api, contexts, run):
    res = []
    for h in contexts:
        api._ctx_cache[0] = h
        res.append(run())
    return res


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 4, 4, 8), (10, 6, 8, 14), (16, 16, 16, 12)])
def test_raw_sweeps(S, env, contexts, L, prec):
    api, g, torch = env
    U = g.links(S.heatbath_field_gpu(L, S.sub_seed(7500), 5.7, 2).cpu().numpy(), prec)
    G0 = g.gauge(S.haar_gauge(L, S.sub_seed(7501)))

    def run():
        out = []
        for paired, defer, slabs in itertools.product((0, 1, 2), (True, False), (1, 2)):
            api.set_paired(paired), api.set_defer_g(defer), api.set_slabs(slabs)
            W, G = U.clone(), G0.clone()
            api.sweeps(W, G, 3)
            out += [W.data, G.data]
        return out

    for a, b in zip(*both(api, contexts, run)):
        assert torch.equal(a, b)


# 192 blocks of 64 half-sites and 256 (FP64) or 512 (FP32) are the lines of the stop test and the form
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("lats", [[(4, 4, 4, 4)], [(10, 6, 8, 14)], [(16, 16, 16, 6)], [(16, 16, 16, 8)],
                                  [(4, 4, 4, 4), (10, 6, 8, 14), (2, 2, 2, 2)]])
def test_fixes(S, env, contexts, lats, prec):
    api, g, torch = env
    Us = [g.links(S.heatbath_field_gpu(L, S.sub_seed(7502, k), 5.7, 2).cpu().numpy(), prec)
          for k, L in enumerate(lats)]

    def run():
        out = []
        for tol, n in ((-1.0, 60), (1e-4, 2000)):  # two blocks of sweeps; stopped by the tolerance
            if len(Us) == 1:
                G, r = api.fix(Us[0], None, tol=tol, max_sweeps=n, reunit_every=25, want_traj=True)
                out.append(([G], [r]))
            out.append(api.fix_batch(Us, None, tol=tol, max_sweeps=n, reunit_every=25, want_traj=True))
        return out

    for (Ga, ra), (Gb, rb) in zip(*both(api, contexts, run)):
        assert all(torch.equal(a.data, b.data) for a, b in zip(Ga, Gb))
        for a, b in zip(ra, rb):
            assert np.array_equal(a.pop("traj"), b.pop("traj")) and a == b
