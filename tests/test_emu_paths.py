"""Single paths of the library on the emulated HIP runtime under AddressSanitizer and UBSan, against
the oracle (tests/emu/run_paths.py)."""
import os
import subprocess
import sys

import pytest

from test_emu import EMU, emu_lib  # noqa: F401

PATHS = ["theta", "loops", "loops_extents", "loops_scaled", "loops_precision", "loops_few", "loops_directions", "loops_scratch", "loops_refused", "launch_form", "stout_form", "field_accesses", "backward_workspace"]


@pytest.mark.parametrize("path", PATHS)
def test_emulated_path(emu_lib, path):  # noqa: F811
    asan = subprocess.check_output(["gcc", "-print-file-name=libasan.so"], text=True).strip()
    env = dict(os.environ, LD_PRELOAD=asan, ASAN_OPTIONS="detect_leaks=0", OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, os.path.join(EMU, "run_paths.py"), path], env=env, timeout=600,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
