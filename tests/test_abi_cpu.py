"""Host-side checks of the C ABI (no GPU needed): the library loads, exports
every entry point include/dv.h declares, and rejects invalid configurations
on the host before any device work."""
import ctypes
import os
import re

import pytest

from paper_1607_00908_amd import dv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "dv.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(dv_[a-z_]+)\s*\(", src)))


def test_header_and_binding_agree():
    assert _declared() == sorted(dv.EXPORTS)


def test_library_exports_every_declared_symbol():
    lib = dv.load()
    for name in _declared():
        assert hasattr(lib, name), name


def test_struct_sizes_match_header_layout():
    assert ctypes.sizeof(dv.DVConfig) == 44
    assert ctypes.sizeof(dv.DVFlip) == 24
    assert ctypes.sizeof(dv.DVFrameInfo) == 48


def _cfg(**kw):
    base = dict(lx=64, ly=64, threshold=0.5, phase=0, connectivity=8, max_components=100,
                max_degree=0, device=0, flags=1, max_batch=0)
    base.update(kw)
    c = dv.DVConfig(ctypes.sizeof(dv.DVConfig), base["lx"], base["ly"], base["threshold"],
                    base["phase"], base["connectivity"], base["max_components"],
                    base["max_degree"], base["device"], base["flags"], base["max_batch"])
    return c


@pytest.mark.parametrize("bad", [
    dict(lx=2), dict(ly=0), dict(lx=70000), dict(lx=65536, ly=65536), dict(phase=2),
    dict(connectivity=6), dict(max_components=0), dict(max_components=(1 << 24) + 1),
    dict(max_degree=3), dict(max_degree=65), dict(threshold=float("nan")), dict(flags=128), dict(flags=0x80000000),
    dict(max_batch=-1), dict(max_batch=65)])
def test_invalid_config_is_rejected_on_the_host(bad):
    lib = dv.load()
    h = ctypes.c_void_p()
    st = lib.dv_create(ctypes.byref(_cfg(**bad)), None, ctypes.byref(h))
    assert st == dv.ERR_ARG
    assert not h.value
    assert lib.dv_last_error(None)
    n = ctypes.c_uint64(7)
    assert lib.dv_device_bytes(ctypes.byref(_cfg(**bad)), ctypes.byref(n)) == dv.ERR_ARG
    assert n.value == 0


def test_device_bytes_follows_the_configuration():
    """The layout size (computed on the host) grows with every quantity that
    sizes a buffer: sites and batch slots, K_max, the row length, an obstacle
    mask; each slot holds at least the per-site maps (parent, 16-bit piece
    slots, piece lists, label and owner maps: 16 B/site)."""
    lib = dv.load()
    assert lib.dv_device_bytes(None, None) == dv.ERR_ARG
    assert lib.dv_device_bytes(ctypes.byref(_cfg()), None) == dv.ERR_ARG
    b = lambda **kw: dv.device_bytes(**{"lx": 256, "ly": 256, "max_components": 1000,
                                         "max_batch": 1, **kw})
    base = b()
    assert base >= 256 * 256 * 16
    assert b(lx=512) - base >= 256 * 256 * 16
    two = b(max_batch=2)
    assert two - base >= 256 * 256 * 16
    assert b(max_batch=3) - two == two - base          # slots are all alike
    assert b(max_components=2000) > base
    assert b(max_degree=64) > base                      # default rows: 48 slots
    assert b(max_degree=45) == b(max_degree=48)         # rows rounded up to 4
    assert b(with_obstacles=True) - base >= 256 * 256   # one byte per site
    assert b(max_batch=0) == b(max_batch=dv.DEFAULT_BATCH)


# Weight sums lie in memory that is free while they are needed.
@pytest.mark.parametrize("cfg", [
    dict(lx=256, ly=256, max_components=1024), dict(lx=1024, ly=1024, max_components=1536, max_batch=2),
    dict(lx=3, ly=65536, max_components=1, max_batch=1), dict(lx=33, ly=1000, max_components=1, keep_maps=False),
    dict(lx=4096, ly=4096, max_components=32768, keep_maps=False)])
@pytest.mark.parametrize("obstacles", [False, True])
def test_weighted_contexts_take_no_more_memory(cfg, obstacles):
    b = [dv.device_bytes(weighted=w, with_obstacles=obstacles, **cfg) for w in (False, True)]
    assert b[1] <= b[0]


def test_size_guard():
    lib = dv.load()
    c = _cfg()
    c.size = 12
    h = ctypes.c_void_p()
    assert lib.dv_create(ctypes.byref(c), None, ctypes.byref(h)) == dv.ERR_ARG


def test_null_arguments():
    lib = dv.load()
    assert lib.dv_create(None, None, None) == dv.ERR_ARG
    assert lib.dv_push_frame(None, None) == dv.ERR_ARG
    assert lib.dv_set_obstacles(None, None, 0) == dv.ERR_ARG
    n = ctypes.c_int32(0)
    assert lib.dv_get_flips(None, None, 0, ctypes.byref(n)) == dv.ERR_ARG
    assert lib.dv_results_ready(None, 1, ctypes.byref(n), ctypes.byref(n)) == dv.ERR_ARG
    assert lib.dv_get_results(None, 1, None, 0, ctypes.byref(n), None, 0, ctypes.byref(n)) == dv.ERR_ARG
    lib.dv_destroy(None)   # NULL-safe
    assert lib.dv_status_str(2) == b"capacity exceeded"


def test_group_arguments_are_checked_on_the_host():
    lib = dv.load()
    h = ctypes.c_void_p()
    assert lib.dv_group_create(None, 1, ctypes.byref(h)) == dv.ERR_ARG
    arr = (ctypes.c_void_p * 1)(None)
    assert lib.dv_group_create(arr, 1, ctypes.byref(h)) == dv.ERR_ARG
    assert lib.dv_group_create(arr, 0, ctypes.byref(h)) == dv.ERR_ARG
    assert lib.dv_group_create(arr, 65, ctypes.byref(h)) == dv.ERR_ARG
    assert lib.dv_group_create(arr, 1, None) == dv.ERR_ARG
    assert not h.value
    assert lib.dv_group_push(None, None) == dv.ERR_ARG
    lib.dv_group_destroy(None)


def test_group_subset_arguments_are_checked_on_the_host():
    lib = dv.load()
    idx = (ctypes.c_int32 * 1)(0)
    arr = (ctypes.c_void_p * 1)(None)
    assert lib.dv_group_push_some(None, idx, arr, 1) == dv.ERR_ARG
