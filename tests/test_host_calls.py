"""The library's host code on a stand-in HIP runtime (host_runtime.cpp): what
a call does when a runtime call fails, and what it plans and launches."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_36452_amd import binding as rpd
from paper_2609_36452_amd.build import CSRC, INCLUDE
from tests.f32_forms import F32_FORMS
from tests.lazy_walks import WALKS

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
    L.kept = getattr(L, "kept", []) + [buf]    # which they may do after the call
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


@pytest.mark.parametrize("name,rows,vocab,ov,seed", F32_FORMS, ids=[c[0] for c in F32_FORMS])
def test_the_shapes_of_the_fp32_forms_take_them(host, name, rows, vocab, ov, seed):
    p = _plan(host, 1, ov["K"] * ov["B"] * ov["n_masked"], ov["V"])
    assert (p.rows_per_tile, p.vocab_cap, p.split_rows) == (rows, vocab, int(name.endswith("row_split")))
    assert p.nrt == {"tile128_two_row_tiles": 2, "tile64_row_split": 16, "small": 4}.get(name, 1)


def test_fp32_tiles_by_rounds_on_the_busiest_xcd(host):
    # V = 15460: 121 vocabulary tiles, 16 on an XCD: two row tiles of 32 or 64 rows are one round of its 32 CUs; at V =
    # 3285 (26, 4 on an XCD; or 52 of 64 vocabulary rows, 7) four to seven row tiles of 32
    assert [_plan(host, 1, r, 15460).rows_per_tile for r in (32, 64, 96, 128)] == [32, 32, 64, 64]
    assert [(p.rows_per_tile, p.vocab_cap) for p in (_plan(host, 1, r, 3285) for r in (32, 128, 200))] == \
        [(32, 64), (32, 64), (32, 128)]


LAZY, LAZY_ALL = 1, 3


def _projections(log):
    """Launches of a lazy call, pass by pass: bounds on the rows of the projections in it."""
    passes = [[]]
    for w in log:
        if w == "next":
            passes.append([])
        elif w.startswith(("big", "stream", "f32_")):
            passes[-1].append(int(re.search(r"\d+$", w.replace("f32_", "")).group()))
    return passes


def test_lazy_calls_that_project_every_layer_at_once(host):
    # Where every position walks, one pass over all layers may cost 1.3 times the least that walking can (d = 4096, V =
    # 126464: 144 positions at K = 4 and 72 at K = 8 are 576 rows, three 192-row tiles)
    one = lambda n, K, flags: "score%d" % n not in _call(host, n, K=K, n=256, flags=flags)[1]   # noqa: E731
    assert [n for n in range(1, 257) if one(n, 4, LAZY_ALL)] == list(range(1, 145))
    assert [n for n in range(1, 257) if one(n, 8, LAZY_ALL)] == list(range(1, 73))
    assert all(one(n, 2, LAZY_ALL) for n in range(1, 257)) and all(one(n, 1, LAZY) for n in range(1, 257))
    # two layers of positions that all walk are projected whatever they hold
    assert all("reduce%d" % n in _call(host, n, K=2, n=n, d=1536, V=31574, flags=LAZY_ALL)[1] for n in range(2, 900, 40))
    # in the band, where one more pass over few positions is all that walking is likely to take, far fewer
    assert not one(64, 4, LAZY) and one(24, 4, LAZY)


@pytest.mark.parametrize("K", [3, 4, 8, 20])
@pytest.mark.parametrize("flags", [LAZY, LAZY_ALL])
def test_lazy_passes_take_no_more_rows_than_are_worth_one(host, K, flags):
    # passes after the final layer: the 256 rows of one tile, or 1, 2, 4 .. layers of every position
    for n in (70, 129, 160, 200, 256):
        s, log = _call(host, n, K=K, n=256, flags=flags)
        if "score%d" % n not in log:
            continue
        passes = _projections(log)
        assert s == 0 and passes[0] == [n]
        for t, rows in enumerate(passes[1:], 1):
            assert max(rows) <= max(256, n * 2 ** (t - 1)), (n, t, rows)
            assert sorted(rows) == rows and len(rows) <= 5
        assert 2 ** (len(passes) - 2) < K


def test_lazy_counts_above_the_bound_are_waited_for(host):
    # 300 positions, of which 280 and 150 walk on: two counts through the slot, then size classes
    for c in (300, 280, 150):   # the first by the compaction
        host.host_add_count(c)
    s, log = _call(host, 300, K=6, n=512, flags=LAZY_ALL)
    assert s == 0 and log[:3] == ["compact", "big300", "walk300"]
    assert log[3:7] == ["next", "sync", "big280", "walk280"] and log[7:11] == ["next", "sync", "big300", "walk150"]
    assert "sync" not in log[11:] and log[-2:] == ["score300", "commit0"]
    passes = _projections(log)[3:]
    assert passes and all(len(p) > 1 for p in passes)


def test_a_lazy_call_without_a_bound_decides_by_its_count(host):
    # 180 of 200 positions: the whole canvas is projected in one pass (its final layer takes a 256-row tile), the 180
    # (192 rows) walk; a bound of 180 walks, and so does no bound
    shape = dict(K=5, n=200, d=2048, V=60013, flags=LAZY_ALL)
    for bound, want in ((200, "reduce200"), (180, "score180"), (-1, "score180")):
        host.host_reset()
        host.host_add_count(180)
        assert want in _call(host, bound, **shape)[1], bound


@pytest.mark.parametrize("name,K,B,n,d,V,dtype,every,norm,ties", WALKS, ids=[c[0] for c in WALKS])
def test_the_shapes_of_the_walking_tests_walk(host, name, K, B, n, d, V, dtype, every, norm, ties):
    # of the positions n_t are left walking after pass t: counts are waited for above 256 positions, else each pass
    # after the first is enqueued once per size class
    counts = [B * n, B * n * 9 // 10, B * n // 4]
    for bound in (B * n, -1):
        host.host_reset()
        for c in counts:
            host.host_add_count(c)
        s, log = _call(host, bound, K=K, B=B, n=n + 9, d=d, V=V, dtype=int(dtype == "f32"), flags=3 if every else 1)
        assert s == 0 and "score%d" % (B * n) in log and log.count("next") >= 1
        assert log.count("sync") == (bound < 0) + (2 if B * n > 256 else 0)
        passes = _projections(log)
        assert len(passes) >= 2 and (B * n > 256 or max(len(p) for p in passes[1:]) >= 2)
