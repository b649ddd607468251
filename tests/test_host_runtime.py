"""The runtime's host code on the CPU: api.cpp and kb_host.cpp linked against
stand-ins for the HIP runtime and the kernel launchers (host_stub.cpp), which
log streams, allocations and launches."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1710_03197_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_03197_amd", "csrc")
HERE = os.path.dirname(os.path.abspath(__file__))
CXX = ["g++", "-O1", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
       f"-I{CSRC}"]

if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
    pytest.skip("needs g++ and the HIP headers", allow_module_level=True)


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    procs = []
    for src in (os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "kb_host.cpp"), os.path.join(HERE, "host_stub.cpp")):
        obj = str(d / (os.path.basename(src) + ".o"))
        procs.append((obj, subprocess.Popen([*CXX, "-c", src, "-o", obj])))
    assert all(p.wait() == 0 for _, p in procs)
    return d, [obj for obj, _ in procs]


class Host:
    """The library's entry points over the stand-ins."""

    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        for name, args in _lib._SIGS.items():
            getattr(self.lib, name).argtypes = args
        self.lib.nufft_last_error.restype = self.lib.stub_log.restype = ctypes.c_char_p
        self.lib.stub_fail_allocations.argtypes = [ctypes.c_size_t, ctypes.c_int]
        self.lib.stub_live_bytes.restype = ctypes.c_size_t
        self.keep = []

    def call(self, name, *args, status=0):
        self.lib.stub_clear()
        st = getattr(self.lib, name)(*args)
        assert st == status, (name, st, self.lib.nufft_last_error())
        return [dict([("what", line.split()[0])] + [kv.split("=") for kv in line.split()[1:]])
                for line in self.lib.stub_log().decode().splitlines()]

    def points(self, om):
        om = np.ascontiguousarray(om, dtype=np.float32)
        self.keep.append(om)
        return om.ctypes.data

    def plan(self, N, K, J, om, stream=None, **options):
        from paper_1710_03197_amd.plan import options_struct
        opt = options_struct(options)
        h = ctypes.c_void_p()
        i64 = ctypes.c_int64 * len(N)
        log = self.call("nufft_plan_ex", len(N), i64(*N), i64(*K), J, len(om), self.points(om), ctypes.byref(opt),
                        stream, ctypes.byref(h))
        return h, log

    def multi(self, problems):
        """problems: (N, K, J, om, coils, options)."""
        from paper_1710_03197_amd.plan import options_struct
        descs = (_lib.ProblemDesc * len(problems))()
        for de, (N, K, J, om, C, options) in zip(descs, problems):
            de.d, de.J, de.M, de.om = len(N), J, len(om), self.points(om)
            de.N[:len(N)], de.K[:len(K)] = N, K
            if C:
                maps = np.ones((C,) + tuple(N), np.complex64)
                self.keep.append(maps)
                de.C, de.coils = C, maps.ctypes.data
            opt = options_struct(options)
            self.keep.append(opt)
            de.opt = ctypes.addressof(opt)
        h = ctypes.c_void_p()
        self.call("nufft_multi_plan", len(problems), descs, None, ctypes.byref(h))
        return h


@pytest.fixture(scope="module")
def host(objects):
    d, objs = objects
    so = str(d / "libhost.so")
    subprocess.run(["g++", "-shared", *objs, "-o", so], check=True)
    return Host(so)


def _buf(n=1):
    return ctypes.c_void_p(0x1000 + n)  # never dereferenced: nothing runs


# ---- 32-bit offsets of the strided FFT passes
OFFSETS = r"""
#include <cstdio>
#include "nufft_internal.h"
using namespace nufft;
int main() {
    long wide_n = 0;
    for (int K = 2; K <= 4096; K += 2)
        for (int sched = 0; sched < 4; ++sched) {
            StridedPassArgs a{};
            if (!radix_plan(K, &a.rp, sched)) continue;
            a.K = K;
            // the largest array of the axis: below 2^31 cells, two axes of at most 4096 after it
            for (int64_t inner : {std::min<int64_t>(4096 * 4096, ((int64_t(1) << 31) - 1) / K), int64_t(4096)}) {
                a.inner = inner;
                for (bool inverse : {false, true}) {
                    a.inverse = inverse;
                    const int p = inverse ? 0 : a.rp.n - 1;
                    const int64_t last = (int64_t(a.rp.nbl[p] - 1) * inner + inner - 1) * 8;
                    if (strided_wide(a) != (last >= int64_t(1) << 32)) {
                        printf("K=%d schedule %d inner %lld\n", K, sched, (long long)inner);
                        return 1;
                    }
                    wide_n += strided_wide(a);
                    // Toeplitz grids (2N, N even, the default schedule) take no wide pass
                    if (K % 4 == 0 && sched == 0 && strided_wide(a)) return 2;
                }
            }
        }
    printf("%ld\n", wide_n);
    return wide_n > 0 ? 0 : 3;
}
"""


def test_strided_offset_width_covers_every_length(objects):
    """Over every grid length and radix schedule at the largest array: offsets
    are 64 bits wide exactly where 32 do not reach."""
    d, objs = objects
    src, exe = d / "offsets.cpp", d / "offsets"
    src.write_text(OFFSETS)
    kb = [o for o in objs if "kb_host" in o]
    subprocess.run([*CXX, str(src), *kb, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stdout)


def test_multi_problem_passes_take_the_offset_width_of_each_problem(host):
    """A grid whose forward pass along axis 0 ends in radix 3 over 4 GiB of rows,
    beside a small one: two launches, the large one wide."""
    om = np.full((4, 3), 0.5, np.float32)
    m = host.multi([((2, 2, 2), (162, 4096, 3200), 6, om, 0, {}), ((8, 8, 8), (16, 16, 16), 6, om, 0, {})])
    ptrs = (ctypes.c_void_p * 2)(_buf(1), _buf(2))
    log = [e for e in host.call("nufft_multi_forward", m, ptrs, ptrs, None) if e["what"] == "strided_multi"]
    assert [(e["K"], e["wide"]) for e in log] == [("4096", "0"), ("162", "1"), ("16", "0")]
    host.call("nufft_multi_destroy", m)


# ---- re-binning a plan in use
@pytest.mark.parametrize("before,now,waits", [(None, 16, True), (32, 16, True), (16, None, True), (16, 16, False),
                                              (None, None, False)])
def test_set_points_waits_for_the_previous_calls_stream(host, before, now, waits):
    """Re-binning on another stream than the previous call's, the default stream
    (NULL) among them, waits for that stream before it writes anything."""
    om = np.full((50, 2), 0.5, np.float32)
    p, _ = host.plan((16, 16), (32, 32), 6, om)
    host.call("nufft_forward", p, _buf(1), _buf(2), before)
    log = host.call("nufft_set_points", p, host.points(om), now)
    name = {None: "(nil)"}.get(before, f"{before or 0:#x}")
    first_write = next(i for i, e in enumerate(log) if e["what"] == "write")
    waited = [e["stream"] for e in log[:first_write] if e["what"] == "sync"]
    assert waited == ([name] if waits else [])
    host.call("nufft_destroy", p)


def test_set_points_of_an_uncalled_plan_waits_for_no_stream(host):
    om = np.full((50, 2), 0.5, np.float32)
    p, _ = host.plan((16, 16), (32, 32), 6, om)
    log = host.call("nufft_set_points", p, host.points(om), 16)
    assert log[0]["what"] == "write"
    host.call("nufft_destroy", p)


def _trajectories(M=200000):
    """One whose samples share a tile (few work items) and one dealt over all tiles (many)."""
    return np.full((M, 2), -0.5, np.float32), np.full((M, 2), 0.5, np.float32)


@pytest.mark.parametrize("failures", [0, 1, 2, 3, 4])
def test_rebin_without_memory_leaves_no_dangling_lists(host, failures):
    """Larger work lists whose allocation fails: once, the old ones make room;
    two or three times, the re-bin reports it and the plan keeps its previous
    trajectory; four times, not even that one's lists fit again and transforms are
    refused.  No launch reads freed lists in any case."""
    few, many = _trajectories()
    p, _ = host.plan((64, 64), (128, 128), 6, few)
    host.lib.stub_fail_allocations(4096, failures)
    host.call("nufft_set_points", p, host.points(many), None, status=-3 if failures > 1 else 0)
    for name in ("nufft_forward", "nufft_adjoint"):
        log = host.call(name, p, _buf(1), _buf(2), None, status=-3 if failures > 3 else 0)
        launches = [e for e in log if e["what"] in ("grid", "interp", "reduce")]
        assert bool(launches) == (failures < 4)
        assert all(e["live"] == "1" for e in launches)
    host.lib.stub_fail_allocations(0, 0)
    # with memory again, a re-bin makes the plan whole
    host.call("nufft_set_points", p, host.points(many), None)
    log = host.call("nufft_adjoint", p, _buf(1), _buf(2), None)
    assert [e["live"] for e in log if e["what"] in ("grid", "reduce")][0] == "1"
    host.call("nufft_destroy", p)


# ---- the window table
@pytest.mark.parametrize("option,d,M,table", [
    (0, 2, 1000, True), (1, 2, 1000, True), (-1, 2, 1000, False),
    (0, 3, 3355443, True), (0, 3, 3355444, False),  # 80 bytes a sample, 256 MiB
    (1, 3, 3355444, True),
    (0, 2, 524288, True),
])
def test_window_table_option(host, option, d, M, table):
    """0 takes a table within its limit, 1 always, -1 never."""
    p, log = host.plan((16,) * d, (32,) * d, 6, np.full((M, d), 0.5, np.float32), weight_table=option)
    assert [e for e in log if e["what"] == "table"] == ([dict(what="table")] if table else [])
    for name, what in (("nufft_forward", "interp"), ("nufft_adjoint", "grid")):
        log = host.call(name, p, _buf(1), _buf(2), None)
        assert [e["table"] for e in log if e["what"] == what] == [str(int(table))]
    host.call("nufft_destroy", p)


@pytest.mark.parametrize("option", [0, 1])
def test_large_2d_gathers_evaluate_their_windows(host, option):
    """Above 32 MiB of records the 2D gather is faster on the fly; the gridding,
    which visits a sample more than once, still reads the table."""
    p, _ = host.plan((16, 16), (32, 32), 6, np.full((524289, 2), 0.5, np.float32), weight_table=option)
    log = host.call("nufft_forward", p, _buf(1), _buf(2), None)
    assert [e["table"] for e in log if e["what"] == "interp"] == ["0"]
    log = host.call("nufft_adjoint", p, _buf(1), _buf(2), None)
    assert [e["table"] for e in log if e["what"] == "grid"] == ["1"]
    host.call("nufft_destroy", p)


def test_window_table_option_range(host):
    from paper_1710_03197_amd.plan import options_struct
    om = np.full((10, 2), 0.5, np.float32)
    i64 = ctypes.c_int64 * 2
    for bad in (-2, 2):
        h = ctypes.c_void_p()
        host.call("nufft_plan_ex", 2, i64(16, 16), i64(32, 32), 6, 10, host.points(om),
                  ctypes.byref(options_struct(dict(weight_table=bad))), None, ctypes.byref(h), status=-1)


def test_toeplitz_spectrum_is_made_without_a_table(host):
    """Its point-spread function is one transform of a plan that then goes."""
    p, _ = host.plan((16, 16), (32, 32), 6, np.full((1000, 2), 0.5, np.float32))
    t = ctypes.c_void_p()
    log = host.call("nufft_toeplitz_plan", p, None, None, ctypes.byref(t))
    assert [e for e in log if e["what"] == "table"] == []
    host.call("nufft_toeplitz_destroy", t)
    host.call("nufft_destroy", p)


@pytest.mark.parametrize("option,status", [(0, 0), (1, -3)])
def test_default_table_gives_way_to_the_workspace(host, option, status):
    """A workspace that does not fit beside a table taken by default fits without
    it; a table that was asked for stays."""
    p, _ = host.plan((16, 16), (32, 32), 6, np.full((1000, 2), 0.5, np.float32), weight_table=option)
    host.lib.stub_fail_allocations(4096, 1)
    log = host.call("nufft_forward_batched", p, 8, _buf(1), _buf(2), None, status=status)
    assert [(e["table"], e["live"]) for e in log if e["what"] == "interp"] == ([("0", "1")] if status == 0 else [])
    host.lib.stub_fail_allocations(0, 0)
    log = host.call("nufft_adjoint_batched", p, 8, _buf(1), _buf(2), None)
    assert [(e["table"], e["live"]) for e in log if e["what"] == "grid"] == [("01"[option], "1")]
    host.call("nufft_destroy", p)


# ---- which gridding and gather forms a call takes
def _adjoint_cols(host, N, C, M, **options):
    p, _ = host.plan(N, tuple(2 * n for n in N), 6, np.full((M, 2), 0.5, np.float32), **options)
    log = host.call("nufft_adjoint_batched", p, C, _buf(1), _buf(2), None)
    host.call("nufft_destroy", p)
    return [int(e["cols"]) for e in log if e["what"] == "grid"]


@pytest.mark.parametrize("N,grids,cols", [
    ((320, 320), 3, 0), ((320, 320), 4, 0),     # one group of the row-tile form
    ((320, 320), 5, 4), ((320, 320), 8, 4),     # 1600 tiles
    ((128, 128), 8, 0), ((128, 128), 16, 4),    # 256 tiles: 512 and 1024 workgroups of four grids
    ((64, 64), 24, 0),
    ((320, 320), 24, 4), ((320, 320), 32, 1),   # 4800 and 6400 groups of eight grids
])
def test_column_gridding_is_taken_where_it_is_faster(host, N, grids, cols):
    """Few grids and few workgroups stay with the row-tile form, whatever the
    number of samples in a tile's one work item."""
    for M in (1000, 15000):
        assert _adjoint_cols(host, N, grids, M) == [cols]


def test_multi_problem_forms_follow_the_whole_launch(host):
    """One and two problems take the forms of their single plans; many take one
    wavefront a gridding item and all coils in a gather workgroup.  Row-tile or
    column gridding is each problem's own choice in every launch."""
    om = np.full((5000, 2), 0.5, np.float32)
    big, small = ((256, 256), (512, 512), 6, om, 8, {}), ((64, 64), (128, 128), 6, om[:2000], 8, {})
    single, _ = host.plan((256, 256), (512, 512), 6, om)
    gather = [int(e["grids_per_wg"]) for e in host.call("nufft_forward_batched", single, 8, _buf(1), _buf(2), None)
              if e["what"] == "interp"]
    host.call("nufft_destroy", single)
    for problems, waves in (([big], 4), ([big, small], 4), ([big] * 2, 4), ([big] * 16, 1), ([small] + [big] * 16, 1)):
        m = host.multi(problems)
        ptrs = (ctypes.c_void_p * len(problems))(*[_buf(k + 1) for k in range(len(problems))])
        adj = [e for e in host.call("nufft_multi_adjoint", m, ptrs, ptrs, None) if e["what"] == "grid_multi"]
        fwd = [e for e in host.call("nufft_multi_forward", m, ptrs, ptrs, None) if e["what"] == "interp_multi"]
        assert {int(e["cols"]) for e in adj} == ({0, waves} if small in problems else {waves})
        if problems == [big]:
            assert int(fwd[0]["grids_per_wg"]) == gather[0]
        host.call("nufft_multi_destroy", m)
    m = host.multi([((256, 256), (512, 512), 6, np.full((40000, 2), 0.5, np.float32), 8, {})] * 40)
    ptrs = (ctypes.c_void_p * 40)(*[_buf(k + 1) for k in range(40)])
    fwd = [e for e in host.call("nufft_multi_forward", m, ptrs, ptrs, None) if e["what"] == "interp_multi"]
    assert fwd[0]["grids_per_wg"] == "8"
    host.call("nufft_multi_destroy", m)


# ---- the Toeplitz operator's workspace
@pytest.mark.parametrize("failures", [0, 1])
def test_toeplitz_operator_is_made_with_room_for_the_coils(host, failures):
    """A first application allocates nothing; where the room does not fit, the
    operator is made with one grid's and grows in the application."""
    p, _ = host.plan((64, 64), (128, 128), 6, np.full((1000, 2), 0.5, np.float32))
    maps = np.ones((8, 64, 64), np.complex64)
    host.call("nufft_set_coils", p, 8, maps.ctypes.data)
    t = ctypes.c_void_p()
    host.lib.stub_fail_allocations(8 * 128 * 128 * 8, failures)
    host.call("nufft_toeplitz_plan", p, None, None, ctypes.byref(t))
    host.lib.stub_fail_allocations(0, 0)
    before = host.lib.stub_live_bytes()
    host.call("nufft_toeplitz_apply", t, 1, _buf(1), _buf(2), None)
    assert (host.lib.stub_live_bytes() == before) == (failures == 0)
    host.call("nufft_toeplitz_destroy", t)
    host.call("nufft_destroy", p)


@pytest.mark.parametrize("N", [(120, 120, 96), (80, 72, 60), (30, 50, 18), (100, 60), (162, 90), (54,)])
def test_toeplitz_spectrum_is_scaled_by_one_rounding(host, N):
    """1 / prod(2N) reaches the spectrum to half a unit in the last place."""
    p, _ = host.plan(N, tuple(2 * n for n in N), 6, np.full((10, len(N)), 0.5, np.float32))
    t = ctypes.c_void_p()
    log = host.call("nufft_toeplitz_plan", p, None, None, ctypes.byref(t))
    scale = float.fromhex([e["scale"] for e in log if e["what"] == "first"][-1])
    assert abs(scale * np.prod([2.0 * n for n in N]) - 1.0) <= 2.0 ** -24
    host.call("nufft_toeplitz_destroy", t)
    host.call("nufft_destroy", p)
