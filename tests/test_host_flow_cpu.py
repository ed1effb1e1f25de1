"""The host side of the library (launch bookkeeping) with HIP calls that fail,
over a stand-in for HIP that runs no kernel (hip_host_stub.cpp), in a process of
its own."""
import json
import os
import shutil
import subprocess
import sys

import pytest

from paper_1607_00908_amd import _build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PRELUDE = """
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library
from paper_1607_00908_amd import dv
lib = dv.load()
field = (ctypes.c_float * (64 * 64))()

def create(flags=dv.KEEP_RESULTS, max_batch=1):
    cfg = dv.DVConfig(ctypes.sizeof(dv.DVConfig), 64, 64, 0.5, 0, 8, 16, 8, 0, flags, max_batch)
    h = ctypes.c_void_p()
    assert lib.dv_create(ctypes.byref(cfg), ctypes.c_void_p(8), ctypes.byref(h)) == dv.OK
    return h

def headers():   # the sequence header that each launch read
    buf = (ctypes.c_int * 256)()
    return [buf[i] for i in range(stub.stub_headers(buf, 256))]

def take(h, wait):
    infos = (dv.DVFrameInfo * 256)()
    n, f = ctypes.c_int32(), ctypes.c_int32()
    assert lib.dv_get_results(h, wait, infos, 256, ctypes.byref(n), None, 0, ctypes.byref(f)) == dv.OK
    return n.value
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not shutil.which(_build.HIPCC):
        pytest.skip("no hipcc")
    so = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run([_build.HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-I" + _build.INCLUDE, "-I" + _build.CSRC,
                    os.path.join(ROOT, "tests", "hip_host_stub.cpp"), "-o", so], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", _PRELUDE + body, so], cwd=ROOT, capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, (r.returncode, r.stderr)
        return json.loads(r.stdout)
    return go


# Every launch commits into the header it did not read: the next one reads that,
# whatever host call failed in between, and no frame that was sent is lost.
@pytest.mark.parametrize("fault", ["stub_fail_record", "stub_stale_error"])
def test_the_host_follows_the_devices_header_past_failed_calls(run, fault):
    out = run(f"""
h = create()
st = []
for k in range(6):
    stub.{fault}(1 if k in (1, 4) else 0)
    st.append(lib.dv_push_frame(h, field))
print(json.dumps([st, headers(), take(h, 0), take(h, 1)]))
""")
    assert out[0] == [0, 4, 0, 0, 4, 0]
    assert out[1] == [0, 1, 0, 1, 0, 1]
    if fault == "stub_fail_record":
        assert out[2:] == [6, 0]


@pytest.mark.parametrize("fault", ["stub_fail_record", "stub_stale_error"])
def test_groups_follow_the_headers_past_failed_calls(run, fault):
    out = run(f"""
m = [create(), create()]
g = ctypes.c_void_p()
assert lib.dv_group_create((ctypes.c_void_p * 2)(*m), 2, ctypes.byref(g)) == dv.OK
st = []
for k in range(20):
    stub.{fault}(1 if k in (1, 18, 19) else 0)
    st.append(lib.dv_group_push(g, (ctypes.c_void_p * 2)(*[ctypes.addressof(field)] * 2)))
print(json.dumps([st, headers(), [take(x, 0) for x in m], [take(x, 1) for x in m]]))
""")
    assert out[0] == [4 if k in (1, 18, 19) else 0 for k in range(20)]
    assert out[1] == [k & 1 for k in range(20)]
    if fault == "stub_fail_record":   # (nothing vouches for the last two without waiting)
        assert out[2] == [18, 18] and out[3] == [2, 2]
