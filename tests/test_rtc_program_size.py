"""The program of an order compiled at run time stays small: the first set-up of
the order waits for its compilation (about 1.1 s with the set-up kernel's loops
over the planes unrolled, 140 kB of code; 0.55 s and about 100 kB rolled)."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# a process of its own: the library keeps what it has compiled
CODE = """
import ctypes, sys
from paper_2606_12650_amd import _lib as L
size = ctypes.c_size_t(0)
assert L.lib().sem_rtc_build(int(sys.argv[1]), b"gfx950", ctypes.byref(size)) == L.SEM_OK
print(size.value)
"""


@pytest.mark.parametrize("N", [13, 14, 15])
def test_rtc_program_is_small(N, tmp_path):
    env = dict(os.environ, SEM_RTC_CACHE=str(tmp_path))
    r = subprocess.run([sys.executable, "-c", CODE, str(N)], cwd=ROOT, env=env, stdout=subprocess.PIPE, text=True,
                       timeout=120, check=True)
    assert 10000 < int(r.stdout.split()[-1]) < 112 * 1024
