"""What the launch plans promise, over the shapes they accept (host functions: nothing is launched)."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest
from scipy import stats

import paper_2510_05485_amd as tb
from paper_2510_05485_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
LDS = 160 * 1024


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if not os.path.exists(build.LIB):
        build.build(verbose=False)
    so = str(tmp_path_factory.mktemp("plans") / "plans.so")
    subprocess.check_call([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC",
                           "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(HERE, "plans.cpp"),
                           "-o", so, "-L", build.PKG, "-ltensorbleu", "-Wl,-rpath," + build.PKG])
    tb.load_library()
    lib = ctypes.CDLL(so)
    i64, i32, flag = ctypes.c_int64, ctypes.c_int, ctypes.c_bool
    lib.runs_plan.restype = flag
    lib.runs_plan.argtypes = [i64, i64, i64, i32, i32, i32, flag, flag, ctypes.POINTER(i64)]
    return lib


def test_sorted_runs_leave_their_tables_room(plans):
    # Every table (where n-grams have more than 64 bits: every part of one) receives a binomial share
    # of the distinct n-grams, at most one per position.  That a share outgrows its table has to stay
    # below exp(-40) each.
    out = (ctypes.c_int64 * 5)()
    shapes, entries, tables, slots = [], [], [], []
    for R, cs, of, N, bits in itertools.product(
            (1, 2, 3, 4, 6, 8, 12, 16, 31, 62),
            (100, 1000, 3000, 4096, 8192, 12000, 30000, 65536, 131072, 262144, 1000000),
            (0.01, 0.5, 1.0, 2.0), (1, 3, 4, 8), (1, 8, 13, 14, 16, 17, 18, 19, 22, 23, 24, 25, 31)):
        rs = max(int(of * cs), 1)
        cap = cs + R * rs
        if not 12288 < cap <= 2097152:
            continue
        for B, (rouge, sizes) in itertools.product((1, 50), ((False, False), (False, True), (True, False))):
            if plans.runs_plan(B, cs, rs, R, N, bits, rouge, sizes, out):
                shapes.append((B, cs, rs, R, N, bits, rouge, sizes))
                entries.append(cap if sizes else cs)
                tables.append(out[0])
                slots.append(out[1])
                assert out[2] <= 512 and out[3] * out[2] <= cap and out[4] + 1024 <= LDS, shapes[-1]
    assert len(shapes) > 10000
    assert (8192, 8192, 16, 4, 18) in {s[1:6] for s in shapes}
    chance = stats.binom.logsf(slots, entries, 1.0 / np.array(tables, dtype=np.float64))
    worst = int(np.argmax(chance))
    assert chance[worst] <= -40.0, (shapes[worst], tables[worst], slots[worst], chance[worst])
