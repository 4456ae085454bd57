"""The library's host code on a stand-in HIP runtime (host_runtime.cpp): what
a call does when a runtime call fails, and what it plans and launches."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2609_36452_amd import binding as rpd
from paper_2609_36452_amd.build import CSRC, INCLUDE

HERE = os.path.dirname(os.path.abspath(__file__))
OUT_OF_MEMORY, INVALID_VALUE = 2, 1


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    so = str(d / "host.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=(x)", "-I/opt/rocm/include",
                    "-I", INCLUDE, "-I", CSRC, os.path.join(CSRC, "rpd_api.cpp"), os.path.join(CSRC, "proj_plan.cpp"),
                    os.path.join(HERE, "host_runtime.cpp"), "-o", so], check=True, capture_output=True)
    return so


@pytest.fixture
def host(built, tmp_path):
    # a copy of its own: the library keeps what it set up on first use
    L = ctypes.CDLL(shutil.copy(built, str(tmp_path / "host.so")))
    L.rpd_workspace_size.restype = ctypes.c_size_t
    L.rpd_last_error.restype = L.host_log.restype = ctypes.c_char_p
    L.host_reset()
    return L


def _call(L, max_masked=-1, K=4, B=1, n=64, d=4096, V=126464, dtype=0, flags=0):
    """One rpd_score_commit; returns the status and the launches it made."""
    p = rpd.RpdProblem(K, B, n, d, V, dtype, 4096, 8192, 64, max_masked, None, 1e-5, 0)
    q = rpd.Params().to_c()
    q.flags = flags
    o = rpd.RpdOutputs(*([4096] * 10 + [None] * 4))
    need = L.rpd_workspace_size(ctypes.byref(p))
    buf = ctypes.create_string_buffer(512)     # the header is all that the stand-in kernels write
    at = (ctypes.addressof(buf) + 255) // 256 * 256
    before = len(L.host_log())
    s = L.rpd_score_commit(ctypes.byref(p), ctypes.byref(q), ctypes.byref(o), ctypes.c_void_p(at),
                           ctypes.c_size_t(need), None)
    return s, L.host_log()[before:].decode().split()


def test_a_count_comes_through_the_pinned_slot(host):
    host.host_add_count(24)
    assert _call(host) == (0, ["compact", "sync", "big24", "reduce24", "commit0"])


@pytest.mark.parametrize("what", ["host_fail_malloc", "host_fail_capturing"])
def test_without_a_pinned_slot_the_count_is_copied(host, what):
    # the failed runtime call stays the thread's last error unless it is taken: the launch that follows would report it
    ctypes.c_int.in_dll(host, what).value = OUT_OF_MEMORY
    for n in (24, 7):
        host.host_add_count(n)
        s, log = _call(host)
        assert s == 0, host.rpd_last_error()
        assert log[:3] == ["compact", "copy", "sync"] and log[3:] == ["big24" if n == 24 else "stream7",
                                                                      f"reduce{n}", "commit0"]


def test_a_slot_that_a_kernel_may_still_store_to_is_not_given_back(host):
    # the launch check reports an earlier failure of the program's own although the compaction is enqueued: the call
    # fails, and the compaction stores its count later, when the next call already waits for another
    host.host_set_last_error(INVALID_VALUE)
    host.host_add_count(64)
    assert _call(host)[0] == 6
    host.host_add_count(7)
    assert _call(host) == (0, ["compact", "sync", "stream7", "reduce7", "commit0"])


class _Plan(ctypes.Structure):   # rpd::ProjPlan
    _fields_ = [(n, ctypes.c_int) for n in ("variant", "rows_per_tile", "vocab_cap", "nvt", "nrt", "per_xcd",
                                            "split_rows", "grid")]


def _plan(L, dtype, rows, V):
    f = L._ZN3rpd15plan_projectionEixi   # rpd::plan_projection(int, long long, int)
    f.restype, f.argtypes = _Plan, [ctypes.c_int, ctypes.c_longlong, ctypes.c_int]
    return f(dtype, rows, V)


def _busiest(p):
    """Tiles of the XCD that has most of them."""
    share = lambda n: max((x + 1) * n // 8 - x * n // 8 for x in range(8))   # noqa: E731
    return share(p.nrt) * p.nvt if p.split_rows else share(p.nvt) * p.nrt


@pytest.mark.parametrize("V", [126464, 32000])
def test_fp32_tiles_are_spread_evenly_over_the_xcds(host, V):
    for rows in [*range(1, 1400, 7), 2048, 2049, 4096, 4400, 12288]:
        p = _plan(host, 1, rows, V)
        assert 8 * _busiest(p) <= 1.03 * p.nvt * p.nrt, (rows, p.rows_per_tile, p.nrt)


def test_fp32_tile_height_by_the_cost_of_its_rows(host):
    # 128-row tiles cost least a row, then 96 and 64, then 32: a shorter tile has to save its padding
    rows = (32, 48, 96, 128, 160, 208, 224, 240, 256, 288, 320, 352, 384, 544, 640, 736, 800, 864, 992, 1136)
    assert [_plan(host, 1, r, 126464).rows_per_tile for r in rows] == \
        [32, 64, 96, 128, 32, 32, 32, 128, 128, 96, 64, 32, 128, 32, 128, 128, 64, 96, 128, 128]
