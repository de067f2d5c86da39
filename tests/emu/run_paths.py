"""More runs of the library built against the emulated HIP runtime (AddressSanitizer + UBSan), one
function per path; started by tests/test_emu_paths.py in a subprocess with libasan preloaded.  Test
infrastructure only."""
import ctypes as C
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path[:0] = [ROOT, os.path.dirname(HERE), HERE]

import emu_api as E  # noqa: E402
from oracle import oracle as O  # noqa: E402
from paper_0807_0264_amd import _abi as A  # noqa: E402
from paper_0807_0264_amd import synth as S  # noqa: E402


def rounded(U, prec):
    return U if prec == 0 else U.astype(np.complex64).astype(np.complex128)


def field(L, seed, sweeps=3):
    return S.heatbath_field(L, S.sub_seed(seed), 5.7, sweeps)


def path_theta():
    """The stationarity residual of a field as given, first call of its context."""
    for L in ((4, 4, 4, 4), (2, 2, 2, 2), (6, 4, 4, 8)):
        for prec in (0, 1):
            U = rounded(field(L, 2100), prec)
            want = O.theta(U)
            got = E.theta(E.links(U, prec))
            assert abs(got - want) <= (1e-12 if prec == 0 else 1e-5) * want, (L, prec, got, want)


def loop_field(L, seed, prec, bad=None):
    """A thermalised field; bad: one time link made non-unitary (a factor) so that the temporal gauge
    does not apply."""
    U = rounded(field(L, seed, 2), prec)
    if bad is not None:
        U[1, 0, 1, 1, 3] *= bad
    return U


def path_loops():
    """Wilson loops at the edges of the temporal-gauge kernels: several rounds of 16 extents, time
    ranges split over blocks, extents beyond a block (the general kernels), spatial sizes below and
    above a wave, a non-unitary time link (general kernels) and a non-unitary spatial link."""
    cases = [((2, 2, 2, 20), 1, 20, None), ((6, 4, 4, 6), 2, 3, None), ((2, 2, 2, 34), 1, 30, None),
             ((2, 2, 2, 60), 1, 60, None), ((4, 2, 2, 8), 1, 8, 1.001)]
    for L, rmax, tmax, bad in cases:
        for prec in (0, 1):
            U = loop_field(L, 2200, prec, bad)
            if bad is None:
                U[0, 1, 0, 1, 0] = 0.9 * U[0, 1, 0, 1, 0]
                U = rounded(U, prec)
            vecs = [(1, 0, 0), (1, 1, 0)] if L[0] > 2 else [(1, 0, 0)]
            got = E.wilson_loops(E.links(U, prec), vecs, rmax, tmax)
            want = O.wilson_loops(U, vecs, rmax, tmax)
            # FP32: the products of a loop round at 6e-8 each, averaged over few sites
            err = np.abs(got - want).max()
            assert err < (1e-13 if prec == 0 else 2e-6), (L, prec, tmax, bad, err)


def path_loops_extents():
    """Wilson loops at the edges of every set of extents that the correlations are built for."""
    L = (2, 2, 2, 18)
    for prec in (0, 1):
        U = loop_field(L, 2250, prec)
        want = O.wilson_loops(U, [(1, 0, 0)], 2, 18)
        for tmax in (1, 4, 5, 8, 9, 10, 11, 12, 13, 16, 17, 18):
            before = E.lib().emu_launches(b"k_wl_corr")
            n = 4 if tmax < 5 else 1  # directions asked for: so many loops that the gauge pays
            got = E.wilson_loops(E.links(U, prec), n * [(1, 0, 0)], 2, tmax)
            assert E.lib().emu_launches(b"k_wl_corr") == before + n, (prec, tmax)
            assert np.abs(got - want[..., :tmax]).max() < (1e-13 if prec == 0 else 2e-6), (prec, tmax)


def path_loops_few():
    """Few loops are multiplied out, without the gauge; many take it."""
    L = (4, 4, 4, 16)
    for prec in (0, 1):
        U = E.links(loop_field(L, 2290, prec), prec)
        for vecs, rmax, tmax, gauged in (([(1, 0, 0)], 1, 4, False), ([(1, 0, 0)], 4, 4, True),
                                         (2 * [(1, 0, 0)], 2, 1, False)):
            before = E.lib().emu_launches(b"k_wl_gauge")
            E.wilson_loops(U, vecs, rmax, tmax)
            assert E.lib().emu_launches(b"k_wl_gauge") - before == gauged, (prec, rmax, tmax)


def path_loops_directions():
    """More directions in one call than the library keeps path images of, on either path."""
    L = (4, 4, 4, 4)
    vecs = [(1, 0, 0), (1, 1, 0), (1, 1, 1)] * 7
    for bad in (None, 1.001):
        U = loop_field(L, 2300, 0, bad)
        got = E.wilson_loops(E.links(U, 0), vecs, 1, 2)
        want = O.wilson_loops(U, vecs[:3], 1, 2)
        assert np.abs(got - np.tile(want, (7, 1, 1))).max() < 1e-13


def cold_field(L, prec, steps):
    """Unit links, the time links scaled by 1 + steps * (unit in the last place of 1): W(R, T) is the
    scale to the power 2 T, whatever the path multiplies out."""
    scale = 1 + steps * 2.0 ** (-52 if prec == 0 else -23)
    U = np.zeros((L[3], L[2], L[1], L[0], 4, 3, 3), np.complex128)
    U[...] = np.eye(3)
    U[..., 3, :, :] *= scale
    return U, scale


def path_loops_scaled():
    """Wilson loops of time links all off by the same few units in the last place come out to the
    rounding of the 2 T + 2 R products of a loop, within the temporal gauge's tolerance and beyond."""
    L, tmax = (4, 2, 2, 8), 8
    for prec, ulp in ((0, 2.0 ** -52), (1, 2.0 ** -23)):
        for steps in (1, 2, 3, 5, 6, 40, 200):
            U, scale = cold_field(L, prec, steps)
            got = E.wilson_loops(E.links(U, prec), [(1, 0, 0)], 2, tmax)[0, 0]
            for T in range(1, tmax + 1):
                err = abs(got[T - 1] / scale ** (2 * T) - 1)
                assert err <= (2 * T + 2) * ulp, (prec, steps, T, err)


def path_loops_precision():
    """FP64 Wilson loops far along the period, where the transform to the temporal gauge has gone through
    80 products: the 50 products of a loop round at 2^-53 each, independently over 1,856 sites, so their
    mean is as good as its own rounding (below 2^-53), whichever way it was formed."""
    L = (4, 4, 2, 58)
    U = field(L, 2255, 3)
    before = E.lib().emu_launches(b"k_wl_corr")
    got = E.wilson_loops(E.links(U, 0), [(1, 0, 0)], 2, 24)
    assert E.lib().emu_launches(b"k_wl_corr") == before + 1
    err = np.abs(got - O.wilson_loops(U, [(1, 0, 0)], 2, 24)).max()
    assert err <= 5e-16, err


def path_loops_scratch():
    """Wilson loops under a scratch limit that admits either path alone but not their buffers added up:
    a call refused by the temporal gauge after it was set up (a non-unitary time link), a call that its
    plan refuses after one that it took, and what a gauged call leaves for other calls."""
    limit = 6
    L, tmax = (4, 4, 4, 32), 32  # a line is 147 kB: the general path holds 4.8 MB

    def context():
        h = C.c_void_p()
        assert E.lib().mcg_create(C.byref(h), 0) == 0
        assert E.lib().mcg_set_option(h, A.MCG_OPT_SCRATCH_LIMIT_MIB, limit) == 0
        E._ctx = h

    def loops(U, tmax):
        got = E.wilson_loops(E.links(U, 1), [(1, 0, 0)], 1, tmax)
        assert np.abs(got - O.wilson_loops(U, [(1, 0, 0)], 1, tmax)).max() < 2e-6

    saved = E.ctx()
    U, bad = loop_field(L, 2210, 1), loop_field(L, 2210, 1, 1.001)
    context()
    loops(rounded(bad, 1), tmax)
    E.check(E.lib().mcg_destroy(E.ctx()))
    context()
    loops(U, tmax)
    E.smear(E.links(field(L, 2211, 1), 0), 0.1, 1.0, 2)  # its temporary is a field of 1.2 MB
    E.check(E.lib().mcg_destroy(E.ctx()))
    context()
    loops(U, tmax)
    loops(loop_field((4, 4, 2, 64), 2212, 1), 62)
    E.check(E.lib().mcg_destroy(E.ctx()))
    E._ctx = saved


def path_loops_refused():
    """A field with a non-unitary time link, under a scratch limit that admits the temporal gauge and not
    the general path: the call is refused and W is not touched."""
    L, tmax = (4, 4, 4, 32), 8
    saved = E.ctx()
    h = C.c_void_p()
    assert E.lib().mcg_create(C.byref(h), 0) == 0
    assert E.lib().mcg_set_option(h, A.MCG_OPT_SCRATCH_LIMIT_MIB, 4) == 0
    E._ctx = h
    for bad, rmax, status in ((None, 1, A.MCG_OK), (None, 4, A.MCG_OK), (1.001, 4, A.MCG_ENOMEM)):
        U = E.links(rounded(loop_field(L, 2220, 1, bad), 1), 1)
        f = U.abi()
        W = np.full((1, rmax, tmax), 7.0)
        st = E.lib().mcg_wilson_loops(h, C.byref(f), 1, (C.c_int32 * 3)(1, 0, 0), rmax, tmax,
                                      W.ctypes.data_as(C.POINTER(C.c_double)), None)
        assert st == status, (st, E.lib().mcg_last_error(h))
        assert (W == 7.0).all() == (bad is not None), W
    E.check(E.lib().mcg_destroy(h))
    E._ctx = saved


def path_launch_form():
    """The form of the half-sweep that a small fix launches: one wave per link until a variant was chosen,
    by the autotuner or by the caller, which then is what runs."""
    saved = E.ctx()
    launches = E.lib().emu_launches
    for prec in (0, 1):
        U = E.links(field((4, 4, 4, 4), 2230, 1), prec)
        for choose in (None, lambda: E.autotune_batch([U]), lambda: E.set_variant(prec, 1)):
            h = C.c_void_p()
            assert E.lib().mcg_create(C.byref(h), 0) == 0
            E._ctx = h
            if choose:
                choose()
            else:  # the two-row form, then the full one
                assert E.get_variant(prec) == (0 if prec == 0 else 2)
                E.set_two_row(False)
                assert E.get_variant(prec) == 2
                E.set_two_row(True)
            before = launches(b"k_halfsweep_wide"), launches(b"k_halfsweep<")
            E.fix(U, None, tol=-1.0, max_sweeps=2)
            wide, plain = (launches(k) - n for k, n in zip((b"k_halfsweep_wide", b"k_halfsweep<"), before))
            assert (wide, plain) == ((4, 0) if choose is None else (0, 4)), (prec, wide, plain)
            E.check(E.lib().mcg_destroy(h))
    E._ctx = saved


def path_stout_form():
    """The kernel of a stout step, by the rounds of 256 blocks that either would take."""
    launches = E.lib().emu_launches
    for L, blocks in (((4, 4, 4, 4), (False, False)), ((2, 2, 2, 66), (False, False)), ((2, 2, 2, 128), (False, True)),
                      ((2, 2, 2, 400), (True, True))):
        for prec in (0, 1):
            U = rounded(field(L, 2260, 1), prec)
            before = launches(b"k_smear_stout")
            got = E.host_links(E.smear(E.links(U, prec), 0.1, 1.0, 1))
            assert launches(b"k_smear_stout") - before == blocks[prec == 0], (L, prec)
            assert np.abs(got - O.smear(U, 0.1, 1.0, 1)).max() < (1e-14 if prec == 0 else 1e-6), (L, prec)


def path_field_accesses():
    """Small fields stay in the caches: gauge transform, projection and vortex fields of them run the
    kernels with ordinary accesses."""
    launches = E.lib().emu_launches
    U, G = E.links(field((4, 4, 4, 4), 2270, 1), 1), E.gauge(S.haar_gauge((4, 4, 4, 4), S.sub_seed(2271)))
    Z, _ = E.center_project(U, G)
    for name, run in ((b"k_apply_gauge<T, false, false>", lambda: E.apply_gauge(U, G)),
                      (b"k_center_project<T, false>", lambda: E.center_project(U, G)),
                      (b"k_center_project<T, false>", lambda: E.center_project(U, None)),
                      (b"k_vortex_field<T, false, false>", lambda: E.vortex_field(U, G, Z, 0)),
                      (b"k_vortex_field<T, false, false>", lambda: E.vortex_field(U, G, Z, 1)),
                      (b"k_vortex_field<T, false, false>", lambda: E.vortex_field(U, None, Z, 1))):
        before = launches(name)
        run()
        assert launches(name) == before + 1, name


def path_backward_workspace():
    """The gradient's smallest workspace, as mcg.h states it: ceil(n/c) - 1 + (c - 1) + 5 fields."""
    L, n, c = (4, 4, 4, 16), 3, 1  # 7 fields of 590 kB
    U, G = E.links(field(L, 2240, 1), 0), E.gauge(S.haar_gauge(L, S.sub_seed(2241)))
    want = E.smear_mcg_backward(U, 0.1, 1.0, n, G, c)
    saved = E.ctx()
    h = C.c_void_p()
    assert E.lib().mcg_create(C.byref(h), 0) == 0
    assert E.lib().mcg_set_option(h, A.MCG_OPT_SCRATCH_LIMIT_MIB, 4) == 0
    E._ctx = h
    got = E.smear_mcg_backward(U, 0.1, 1.0, n, G, c)
    assert np.abs(E.host_links(got[0]) - E.host_links(want[0])).max() <= 1e-13 * np.abs(E.host_links(want[0])).max()
    assert all(abs(a - b) <= 1e-12 * abs(b) for a, b in zip(got[1:], want[1:])), (got[1:], want[1:])
    E.check(E.lib().mcg_destroy(h))
    E._ctx = saved


if __name__ == "__main__":
    for name in sys.argv[1:]:
        globals()["path_" + name]()
        print("ok", name, flush=True)
