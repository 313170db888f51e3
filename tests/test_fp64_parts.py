"""How the FP64 contraction deals a batch to its tiles (csrc/fp64_parts.h), on the
CPU: the same source, built host-only with the shim in tests/host/.  The parts
cover the batch, start where their 16-byte loads are aligned, and read no entry of
the basis rows past the rows' leading dimension."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2508_04172_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE_Q = (64, 128, 64, 128, 64, 256, 128)    # proposals of each variant's tile


@pytest.fixture(scope="module")
def fp(tmp_path_factory):
    hipcc = shutil.which("hipcc") or os.path.join(build.ROCM, "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    out = str(tmp_path_factory.mktemp("fp64parts") / "libfp64parts.so")
    cmd = [hipcc, "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", f"-I{build.CSRC}",
           f"-I{build.ROCM}/include", os.path.join(ROOT, "tests", "host", "fp64_parts_shim.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    lib = C.CDLL(out)
    lib.fp_parts.argtypes = [C.c_int, C.c_int, C.c_longlong, C.c_int, C.POINTER(C.c_longlong)]
    lib.fp_rows_ld.restype = C.c_longlong
    lib.fp_rows_ld.argtypes = [C.c_longlong]
    return lib


# one, two, ten and twenty column tiles of 128
@pytest.mark.parametrize("K", [41, 243, 1275, 2475])
def test_parts_cover_the_batch_and_stay_in_its_rows(fp, K):
    Kp = (K + 127) // 128 * 128
    rng = np.random.default_rng(K)
    sizes = [1, 7, 8, 9, 30_011, 90_000, 99_999, 110_000] + [int(n) for n in np.exp(rng.uniform(0, np.log(2e6), 3000))]
    out = (C.c_longlong * 6)()
    handed_over = 0
    for n in sizes:
        ldb = fp.fp_rows_ld(n)
        assert n <= ldb < n + 8
        for v in range(7):
            fp.fp_parts(K, Kp, n, v, out)
            first, count, read_end, first2, count2, read_end2 = out
            what = f"K {K}, {n} proposals, variant {v}: {list(out)}"
            assert first == 0 and first2 == count and count + count2 == n and min(count, count2) >= 0, what
            assert count2 == 0 or count % TILE_Q[v] == 0, what
            handed_over += count > 0 and count2 > 0
            for at, cnt, end in ((first, count, read_end), (first2, count2, read_end2)):
                if cnt == 0:
                    continue                          # not launched
                # pairs from even entries on: a tile's last load ends at read_end at most
                assert at % 2 == 0 and end % 2 == 0 and end >= cnt, what
                assert at + end <= ldb, what
    assert handed_over > 0 or Kp == 128
