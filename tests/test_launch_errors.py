"""A launch that fails is reported, and nothing that depends on it is launched.

Runs on the CPU: a stub in front of the HIP runtime counts the launches and
fails the n-th one, in a process of its own that loads the stub before the
library. No pointer is dereferenced and nothing reaches a device."""

import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
static int launches, fail_at, last;
void stub_reset(int n) { launches = last = 0; fail_at = n; }
int stub_launches(void) { return launches; }
int __hipPushCallConfiguration(void) { return 0; }
int __hipPopCallConfiguration(void) { return 0; }
int hipLaunchKernel(void) { if (++launches == fail_at) return last = 719; return 0; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
"""

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
from tests.test_abi import FAKE, _with_host_indptr, d2sd, good_args, ws_size
one = dict(batch=1, total_nodes=48, max_nodes=48, max_ctx_len=32768, max_pages=2048, num_pages=2048)
eight = dict(batch=8, total_nodes=384, max_nodes=48, max_ctx_len=8192, max_pages=512, num_pages=4096)
ip = np.arange(33, dtype=np.int32) * 80
plans = {
    "even division": good_args(**eight), "even division, fp32": good_args(dtype=d2sd.F32, **eight),
    "four waves": good_args(kv_split=256, **one), "fp32": good_args(kv_split=256, dtype=d2sd.F32, **one),
    "twelve waves": good_args(kv_split=4096, row_group=384),
    "packed": _with_host_indptr(good_args(kv_split=4096, row_group=384, packed=2), ip),
}
for name, a in plans.items():
    st, need = ws_size(a)
    assert st == 0 and need > 0, name
    for n, status, launched in ((0, d2sd.OK, 2), (1, d2sd.ERR_HIP, 1), (2, d2sd.ERR_HIP, 2)):
        stub.stub_reset(n)
        got = d2sd._cascade(ctypes.byref(a), ctypes.c_void_p(FAKE), need, None)
        assert (got, stub.stub_launches()) == (status, launched), (name, n, got, stub.stub_launches())
print("ok")
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs a C compiler")
def test_a_failed_launch_is_reported(tmp_path):
    src, lib = tmp_path / "stub.c", tmp_path / "libstub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr[-2000:]
