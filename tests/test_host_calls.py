"""What the library's calls ask of the HIP runtime, followed on the CPU: the
built library runs against a host-only stand-in for the runtime
(tests/hostrt/fake_hip.cpp), in a process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

from paper_2407_11290_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, os, threading
import numpy as np
from paper_2407_11290_amd import _lib, FN_HILBERT, PREC_FP64, EDEVICE, EINVAL, ENOMEM, ESTATE
from paper_2407_11290_amd.api import TTCross, default_options
L = _lib.load()
F = C.CDLL(os.environ["FAKE_HIP"])
F.fake_malloc.restype = C.c_void_p
F.fake_malloc.argtypes = [C.c_size_t, C.c_int]
F.fake_limit.argtypes = [C.c_size_t]
F.fake_in_use.restype = C.c_size_t
HOOK = C.CFUNCTYPE(None, C.c_char_p, C.c_void_p)

def lines(f):
    b = C.create_string_buffer(1 << 20)
    f(b, len(b))
    return b.value.decode().splitlines()

def faults():
    return lines(F.fake_faults)

def log(what=""):
    return [x for x in lines(F.fake_log) if what in x]

def solved(n=(6, 5, 7), stream=None):
    p = TTCross(list(n), 1e-8, FN_HILBERT, precision=PREC_FP64, stream=stream)
    assert p.run() == 0 and list(p.ranks()) == [1] * (len(n) + 1)
    return p

def read(p, ptr, cap=None):
    m = int(sum(p.n))
    got = L.tt_cross_get_cores(p.h, C.c_void_p(ptr), m if cap is None else cap, 1)
    return got, np.ctypeslib.as_array((C.c_double * m).from_address(ptr)).copy()

def sampled(p, R, seed=1):
    e = C.c_double()
    return L.tt_cross_sampled_error(p.h, R, C.c_uint64(seed), C.byref(e))
"""


@pytest.fixture(scope="session")
def fake(tmp_path_factory):
    """Runs code in a process of its own, on the stand-in runtime."""
    lib = tmp_path_factory.mktemp("hostrt") / "libfakehip.so"
    subprocess.run([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I",
                    os.path.join(ROOT, "include"), "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "hostrt", "fake_hip.cpp"), "-o", str(lib)], check=True)

    def run(code):
        env = dict(os.environ, LD_PRELOAD=str(lib), FAKE_HIP=str(lib), PYTHONPATH=ROOT)
        env.pop("TT_CROSS_LIB", None)
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code)], env=env, cwd=ROOT, timeout=60,
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout
    return run


def test_core_read_goes_to_the_buffer(fake):
    fake("""
    p = solved()
    m = sum(p.n)
    buf = F.fake_malloc(8 * m, 0)
    F.fake_clear()
    got, x = read(p, buf)
    assert got == m and list(x) == list(range(1, m + 1)), (got, x)
    assert len(log("k_copy_one")) == 1 and not faults(), (log(), faults())
    """)


def test_core_read_runs_on_the_handles_device(fake):
    """A handle made on one GPU and read while another is current: before, a
    copy on the handle's own stream, and it may not become a kernel of the
    other GPU, which has no access to the cores."""
    fake("""
    F.fake_set_device(0)
    a = solved()
    m = sum(a.n)
    buf0 = F.fake_malloc(8 * m, 0)
    assert read(a, buf0)[0] == m                 # the first read, on GPU 0
    F.fake_set_device(1)
    b = solved()
    buf1 = F.fake_malloc(8 * m, 0)
    for cur in (1, 0):
        F.fake_set_device(cur)
        F.fake_clear()
        got, x = read(b, buf1)
        assert got == m and list(x) == list(range(1, m + 1)), (cur, got, x)
        assert not faults(), (cur, faults())
    F.fake_set_device(1)
    F.fake_clear()
    assert read(a, buf0)[0] == m and not faults(), faults()
    """)


@pytest.mark.parametrize("target", ["host", "pinned", "peer", "short", "misaligned"])
def test_core_read_into_other_memory(fake, target):
    """Targets that a copy command takes or refuses by itself go to it, as
    before: pageable and pinned host memory, another GPU's memory, a range
    past its allocation (an error), an address between two doubles."""
    fake(f"""
    target = {target!r}
    p = solved()
    m = sum(p.n)
    if target == "host":
        room = (C.c_char * (8 * m + 64))()
        ptr = C.addressof(room)
    elif target == "peer":
        F.fake_set_device(1)
        ptr = F.fake_malloc(8 * m, 0)
        F.fake_set_device(0)
    else:
        ptr = F.fake_malloc(8 * m + 16, int(target == "pinned"))
        ptr += {{"pinned": 0, "short": 24, "misaligned": 4}}[target]
    F.fake_clear()
    got, x = read(p, ptr)
    assert not faults() and not log("k_copy_one") and len(log("hipMemcpyAsync %d " % (8 * m))) == 1, (faults(), log())
    if target == "short":
        assert got == EDEVICE, got
    else:
        assert got == m and list(x) == list(range(1, m + 1)), (got, x)
    """)


def test_last_handle_destroyed_beside_a_new_ones_core_read(fake):
    """One thread destroys the last handle and is stopped while the check's
    workspace is given back; another makes a handle, solves, and is stopped
    as its core copy is launched; the first goes on.  What the copy uses (its
    flag, its stream) must still be there."""
    fake("""
    a = solved()
    m = sum(a.n)
    buf = F.fake_malloc(8 * m, 0)
    assert read(a, buf)[0] == m                  # the flag page and its stream are there
    F.fake_clear()
    assert sampled(a, 1000) >= 0                 # and the workspace
    size = int(log("hipMalloc")[-1].split()[1])
    launched, destroyed = threading.Event(), threading.Event()
    made, state, result = [], {"at": None}, []

    def second():
        p = solved()
        made.append(p)
        result.append(read(p, buf))

    def hook(name, arg):
        me = threading.current_thread()
        if me is first and name == b"hipFree" and a.h is None and not made:
            # the handle's own buffers go first; the workspace is the last
            pending["frees"] += 1
            if pending["frees"] == pending["stop_at"]:
                t2.start()
                assert launched.wait(30)
        if me is t2 and name == b"hipLaunchKernel" and b"k_copy_one" in C.string_at(arg):
            launched.set()
            assert destroyed.wait(30)

    def destroy(p):
        h, p.h = p.h, None
        L.tt_cross_destroy(C.c_void_p(h))

    # how many frees a destroyed last handle makes, the workspace's included
    pending = {"frees": 0, "stop_at": -1}
    first = threading.current_thread()
    t2 = threading.Thread(target=second)
    cb = HOOK(hook)
    F.fake_hook(cb)
    destroy(a)
    F.fake_hook(HOOK())
    total = pending["frees"]
    for stop_at in range(1, total + 1):
        a = solved()
        assert read(a, buf)[0] == m and sampled(a, 1000) >= 0
        made.clear(); result.clear(); launched.clear(); destroyed.clear()
        pending = {"frees": 0, "stop_at": stop_at}
        t2 = threading.Thread(target=second)
        F.fake_clear()
        F.fake_hook(cb)
        destroy(a)
        destroyed.set()
        t2.join()
        F.fake_hook(HOOK())
        assert not faults(), (stop_at, total, faults())
        got, x = result[0]
        assert got == m and list(x) == list(range(1, m + 1)), (stop_at, got)
        made[0].close()
    """)


def test_everything_is_given_back_with_the_last_handle(fake):
    fake("""
    for rep in range(3):
        ps = [solved() for _ in range(3)]
        m = sum(ps[0].n)
        buf = F.fake_malloc(8 * m, 0)
        for p in ps:
            assert read(p, buf)[0] == m and sampled(p, 1000) >= 0
        before = F.fake_in_use()
        for p in ps:
            p.close()
        left = F.fake_in_use()
        if rep == 0:
            base = left
        assert left == base + 8 * m * rep and before > left, (rep, left, base)
        assert not faults(), faults()
    """)


@pytest.mark.parametrize("name,nth", [("hipMemcpyAsync", 1), ("hipLaunchKernel", 2), ("hipLaunchKernel", 4)])
def test_failed_check_leaves_nothing_queued_on_the_kept_workspace(fake, name, nth):
    """A check that fails on the way has kernels queued that write the
    workspace; the next check, on another stream, gets the same memory, so
    the failed one waits for its stream before it returns."""
    fake(f"""
    p = solved()
    assert sampled(p, 1000) >= 0
    F.fake_clear()
    F.fake_fail({name.encode()!r}, {nth})
    assert sampled(p, 1000) == EDEVICE
    calls = log()
    stream = [x for x in calls if x.startswith("launch")][0].split("stream ")[1].split()[0]
    last = max(i for i, x in enumerate(calls) if x.startswith("launch"))
    assert any(x == "hipStreamSynchronize " + stream for x in calls[last + 1:]), calls
    assert sampled(p, 1000) >= 0 and not faults()
    """)


@pytest.mark.parametrize("R", [-(-2**64 // 28), -(-2**64 // 28) + 100, 2**62, 2**63 - 1])
def test_check_of_too_many_samples_is_refused(fake, R):
    """Sample counts whose buffers pass what an address can hold: refused
    before anything is launched (one buffer's size may not wrap around to a
    small one)."""
    fake(f"""
    p = solved()
    F.fake_clear()
    assert sampled(p, {R}) == ENOMEM, _lib.last_error()
    assert not log("launch") and not faults(), (log(), faults())
    assert sampled(p, 1000) >= 0
    """)


def test_time_of_the_last_bulk_evaluation_that_completed(fake):
    """A later evaluation that fails does not count."""
    fake("""
    n = np.array([9, 9, 9], dtype=np.int32)

    def evaluate(m):
        idx = np.zeros((m, 3), dtype=np.int32)
        out = np.zeros(m)
        return L.tt_fn_eval(FN_HILBERT, 3, n.ctypes.data_as(C.POINTER(C.c_int32)), None, 0, m, idx.ctypes.data_as(C.c_void_p),
                            out.ctypes.data_as(C.c_void_p), 0)

    ms = C.c_double()
    assert L.tt_fn_eval_last_kernel_ms(C.byref(ms)) == ESTATE
    F.fake_fail(b"hipStreamSynchronize", 1)
    assert evaluate(5000) == EDEVICE
    assert L.tt_fn_eval_last_kernel_ms(C.byref(ms)) == ESTATE
    for m, want in ((5000, 4.0), (20000, 15.0), (1000, 1.0)):
        assert evaluate(m) == 0 and L.tt_fn_eval_last_kernel_ms(C.byref(ms)) == 0 and ms.value == want, (m, ms.value)
        for name, nth in ((b"hipStreamSynchronize", 1), (b"hipLaunchKernel", 1)):
            F.fake_fail(name, nth)
            assert evaluate(100000) == EDEVICE
            ms.value = -1.0
            assert L.tt_fn_eval_last_kernel_ms(C.byref(ms)) == 0 and ms.value == want, (m, name, ms.value)
    """)


def test_kept_workspace_makes_room_for_a_solve(fake):
    """Memory that a solve needs and only the check's kept workspace holds."""
    fake("""
    p = solved()
    q = TTCross([40, 50, 60], 1e-8, FN_HILBERT, precision=PREC_FP64)
    before = F.fake_in_use()
    assert q.run() == 0
    need = F.fake_in_use() - before
    q.close()
    assert sampled(p, 2000000) >= 0              # 2.8e7 bytes
    assert need < 2e7
    F.fake_limit(need // 2)
    q = TTCross([40, 50, 60], 1e-8, FN_HILBERT, precision=PREC_FP64)
    assert q.run() == 0
    # and a check too large to be kept gets the room of the kept one
    F.fake_limit(0)
    assert sampled(p, 2000000) >= 0
    F.fake_limit(int(2.8e8))
    assert sampled(p, 10500000) >= 0             # 2.94e8 bytes
    F.fake_limit(0)
    assert sampled(p, 1000) >= 0 and not faults(), faults()
    """)


@pytest.mark.parametrize("count", [1, 3])
def test_batched_sweeps_have_a_workgroup_per_new_tile(fake, count):
    """The device finishes every round before the host looks: with no round
    queued the next one still has the new tiles of the last commit (64 points
    in two blocks: 2 x 2 tiles of a new prefix or suffix, two unfoldings)."""
    fake(f"""
    from paper_2407_11290_amd.api import batch_run
    F.fake_sweeps(6)
    ps = [TTCross([64] * 3, 1e-8, FN_HILBERT, precision=PREC_FP64, grid=[2] * 3, seed=i, lookahead=1)
          for i in range({count})]
    batch_run(ps[:1])                            # (buffers)
    F.fake_clear()
    batch_run(ps)
    grids = [int(x.split("grid ")[1]) for x in log("k_sweep_b")]
    assert len(grids) >= 6 and not faults(), (grids, faults())
    assert all(g >= {count} * 8 for g in grids[2:6]), grids
    assert all(list(p.ranks()) == [1, 6, 6, 1] for p in ps)
    """)


@pytest.mark.parametrize("count,least", [(1, 128), (4, 4 * 128), (64, 64 * 16)])
def test_stored_tiles_are_cut_while_few_problems_share_a_launch(fake, count, least):
    """Tiles of 256 rows (16 a superblock of 512 x 512 points): one problem's
    are searched in parts of 16 rows, and so on until the launch has 4096."""
    fake(f"""
    from paper_2407_11290_amd.api import batch_run
    F.fake_sweeps(2)
    ps = [TTCross([512] * 3, 1e-8, FN_HILBERT, precision=PREC_FP64, seed=i, r_max=2, tile_rows=256, tile_cols=64)
          for i in range({count})]
    F.fake_clear()
    batch_run(ps)
    grids = [int(x.split("grid ")[1]) for x in log("k_sweep_b")]
    assert grids[0] >= {least} and not faults(), (grids, faults())
    """)


# where the kernels' measured times lie well apart (lane groups / other, us)
TT_EVAL_KERNELS = [
    ([1000] * 3, 5, 65536, "9k_tt_evalE"),                 # 30 / 52
    ([1000] * 3, 5, 262144, "k_tt_eval_sortILi16E"),       # 66 / 53
    ([1000] * 3, 12, 65536, "9k_tt_evalE"),                # 38 / 52
    ([1000] * 3, 20, 98304, "k_tt_eval_sortILi32E"),       # 100 / 86
    ([1000] * 3, 20, 132000, "9k_tt_evalE"),               # 124 / 149
    ([1000] * 3, 40, 98304, "9k_tt_evalE"),                # 265 / 342
    ([1000] * 3, 40, 1000000, "9k_tt_evalE"),              # 2430 / 2583
    ([250] * 4, 24, 132000, "9k_tt_evalE"),                # 167 / 267
    ([250] * 4, 9, 200000, "k_tt_eval_sortILi16E"),        # 99 / 53
    ([64] * 4, 9, 65536, "k_tt_eval_sortILi16E"),          # 46 / 35
    ([64] * 4, 20, 98304, "k_tt_eval_sortILi32E"),         # 135 / 48
    ([64] * 4, 48, 132000, "9k_tt_evalE"),                 # 560 / 658
    ([64] * 4, 56, 131072, "k_tt_eval_sortILi64E"),        # 642 / 475
    ([30, 500, 40, 600, 30], 5, 65536, "9k_tt_evalE"),     # 40 / 86
    ([20] * 6, 8, 4096, "9k_tt_evalE"),                    # 18 / 29
    ([20] * 6, 8, 65536, "k_tt_eval_lds"),                 # 44 / 30
    ([128] * 6, 2, 20000, "k_tt_eval_lds"),
    ([40, 30, 20], 1, 4097, "k_tt_eval_lds"),
    ([64] * 6, 16, 1000000, "k_tt_eval_sortILi16E"),       # 623 / 169
]


def test_tt_values_take_the_kernel_that_is_faster(fake):
    fake(f"""
    for n, r, m, want in {TT_EVAL_KERNELS!r}:
        F.fake_ranks(r)
        p = TTCross(n, 1e-8, FN_HILBERT, precision=PREC_FP64, r_max=64, n_samples=1)
        p.run()
        assert max(p.ranks()) == r, p.ranks()
        idx, out = F.fake_malloc(4 * m * len(n), 0), F.fake_malloc(8 * m, 0)
        F.fake_clear()
        assert L.tt_eval(p.h, m, C.c_void_p(idx), C.c_void_p(out), 1) == 0
        got = [x.split()[1] for x in log("k_tt_eval")]
        assert len(got) == 1 and want in got[0], (n, r, m, want, got)
        p.close()
    """)


def test_bulk_evaluation_has_one_kernel_for_every_alignment(fake):
    """Index lists that start between 16-byte lines (slices of a larger list)
    take the kernel that aligned ones take: a second one was slower."""
    fake("""
    for f32 in (0, 1):
        names = set()
        for d in (2, 3, 5, 6):
            n = np.array([9] * d, dtype=np.int32)
            idx, out = F.fake_malloc(4 * 5000 * d + 64, 0), F.fake_malloc(8 * 5000, 0)
            for shift in (0, 4, 8, 12):
                F.fake_clear()
                assert (L.tt_fn_eval_f32 if f32 else L.tt_fn_eval)(
                    FN_HILBERT, d, n.ctypes.data_as(C.POINTER(C.c_int32)), None, 0, 5000, C.c_void_p(idx + shift),
                    C.c_void_p(out), 1) == 0
                names.add(log("k_fn_eval")[0].split()[1])
        assert len(names) == 1, names
    """)
