"""More runs of the library built against the emulated HIP runtime (AddressSanitizer + UBSan), one
function per path; started by tests/test_emu_paths.py in a subprocess with libasan preloaded.  Test
infrastructure only."""
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path[:0] = [ROOT, os.path.dirname(HERE), HERE]

import emu_api as E  # noqa: E402
from oracle import oracle as O  # noqa: E402
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


if __name__ == "__main__":
    for name in sys.argv[1:]:
        globals()["path_" + name]()
        print("ok", name, flush=True)
