"""The library's host code on a model of the HIP runtime (tests/hostmodel): device
memory is host memory, kernels do nothing, streams and events keep vector
clocks.  A launch that runs before what it needs shows here for certain, where
a GPU would show it now and then, and failures of the runtime can be asked for."""
import concurrent.futures as cf
import ctypes as C
import glob
import os
import shutil
import subprocess
import threading

import pytest

import paper_1311_1006_amd as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1311_1006_amd", "csrc")


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if shutil.which("hipcc") is None or shutil.which("g++") is None:
        pytest.skip("hipcc / g++ not available")
    tmp = str(tmp_path_factory.mktemp("hostmodel"))
    gxx = ["g++", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include")]

    def compile_(src):
        obj = os.path.join(tmp, os.path.basename(src) + ".o")
        cc = ["hipcc", "--offload-host-only"] if src.endswith(".hip") else gxx
        subprocess.run(cc + ["-O1", "-std=c++17", "-fPIC", "-c", src, "-o", obj], check=True, capture_output=True)
        return obj

    srcs = glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp"))
    srcs.append(os.path.join(ROOT, "tests", "hostmodel", "runtime.cpp"))
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_, srcs))
    syms = subprocess.run(["nm", "-u"] + objs, check=True, capture_output=True, text=True).stdout.split()
    code = ["-Wl,--defsym=%s=0" % s for s in sorted(set(syms)) if s.startswith("__hip_fatbin_")]
    so = os.path.join(tmp, "model.so")
    subprocess.run(["g++", "-shared", "-Wl,-z,defs", "-Wl,-Bsymbolic", "-o", so] + objs + code, check=True)
    return so


class Model:
    """A fresh copy of the library with a runtime of its own."""

    def __init__(self, so):
        self.lib = C.CDLL(so)
        for f in ("fmm_last_error",):
            getattr(self.lib, f).restype = C.c_char_p
        self.lib.model_stream.restype = C.c_void_p
        self.lib.model_now.restype = C.c_long
        self.buf = (C.c_double * 4096)()      # no kernel reads or writes it

    def stream(self):
        return C.c_void_p(self.lib.model_stream())

    def ok(self, rc):
        assert rc == 0, self.lib.fmm_last_error().decode()

    def tree(self, n, L, s, nprob=1):
        off = (C.c_int64 * (nprob + 1))(*[n * b for b in range(nprob + 1)])
        h = C.c_void_p()
        self.ok(self.lib.fmm_build_tree(self.buf, off, nprob, (C.c_int * nprob)(*[L] * nprob), s, C.byref(h)))
        return h

    def plan(self, tree, s, p=12, prec=0, flags=0, theta=0.5):
        t = F._Tuning()
        t.flags = flags
        h = C.c_void_p()
        self.ok(self.lib.fmm_plan(tree, p, C.c_double(theta), prec, C.byref(t), s, C.byref(h)))
        return h

    def call(self, op, pl, s):
        L, b = self.lib, self.buf
        if op == "evaluate":
            return L.fmm_evaluate(pl, b, b, s)
        if op == "parts":
            return L.fmm_evaluate_parts(pl, b, b, b, s)
        if op == "field":
            return L.fmm_evaluate_field(pl, b, b, b, s)
        if op == "log":
            return L.fmm_evaluate_log(pl, b, b, s)
        if op == "adjoint":
            return L.fmm_evaluate_adjoint(pl, b, b, b, b, s)
        if op == "static":
            return L.fmm_evaluate_static(pl, b, b, s)
        points, field = op.split(":")
        return L.fmm_evaluate_points(pl, b, b, C.c_int64(int(points)), b, b if field == "field" else None, s)

    def before(self, s, at):
        name = C.create_string_buffer(256)
        return self.lib.model_before(s, C.c_long(at), name, 256), name.value.decode()


@pytest.fixture
def model(library, tmp_path):
    # a copy of its own: the library's statics are fresh
    so = str(tmp_path / "model.so")
    shutil.copy(library, so)
    return Model(so)


OPS = ["evaluate", "parts", "field", "log", "100:phi", "100:field", "60000:phi", "60000:field"]


@pytest.mark.parametrize("flag", [0, 4, 12])      # no long lists; long strong lists; long weak ones too
@pytest.mark.parametrize("op", OPS)
def test_first_call_on_another_stream_follows_the_plan(model, op, flag):
    # tree and plan on one stream, the first call on another: no kernel of the
    # call may run before the tree is built (they gather through its permutation)
    a, b = model.stream(), model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))
    model.plan(model.tree(5000, 5, a), a)      # the first of a layout waits on the host
    pl = model.plan(model.tree(5000, 5, a), a)
    at = model.lib.model_now(a)
    model.lib.model_clear()
    model.ok(model.call(op, pl, b))
    assert model.lib.model_launches(b"") > 0
    assert model.before(a, at) == (0, "")
    # and the caller's stream comes after everything that the call launched
    assert model.lib.model_not_joined(b) == 0


def live(model):
    n = C.c_int64()
    model.ok(model.lib.fmm_debug_live_blocks(C.byref(n)))
    return n.value


@pytest.mark.parametrize("flag", [0, 12])
@pytest.mark.parametrize("op", OPS + ["adjoint"])
def test_call_after_a_failed_allocation_has_its_buffers(model, op, flag):
    # a buffer whose allocation failed is allocated by the next call: it must not
    # count as there (its kernels would get a null pointer)
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))

    def plan():
        pl = model.plan(model.tree(5000, 5, s), s)
        model.ok(model.lib.fmm_plan_stats(pl, C.byref(F._Stats())))       # the lists are final
        if op == "adjoint":
            model.ok(model.call("evaluate", pl, s))
        return pl

    pl = plan()
    before = live(model)
    model.ok(model.call(op, pl, s))
    kept = live(model) - before
    for k in range(100):
        pl = plan()
        before = live(model)
        model.lib.fmm_debug_fail_alloc(C.c_int64(k))
        rc = model.call(op, pl, s)
        model.lib.fmm_debug_fail_alloc(C.c_int64(-1))
        if rc == 0:
            break
        assert rc == -2, k
        model.ok(model.call(op, pl, s))
        assert live(model) - before == kept, k
    else:
        pytest.fail("the call never succeeded")


def fresh_models(library, tmp_path, name="fresh"):
    """(k, a copy of the library that has done nothing yet), k = 0, 1, ..."""
    for k in range(200):
        so = str(tmp_path / ("%s%d.so" % (name, k)))
        shutil.copy(library, so)
        yield k, Model(so)
    pytest.fail("the sequence never ran out of allocations")


def test_first_plan_of_a_process_is_retried_when_memory_is_short(library, tmp_path):
    # every hipMalloc of the sequence fails once (the tables that depend on
    # nothing are made here): the library gives its cached blocks back and tries again
    for k, m in fresh_models(library, tmp_path):
        s = m.stream()
        m.lib.model_fail_malloc(k)
        m.ok(m.call("evaluate", m.plan(m.tree(5000, 5, s), s), s))
        if m.lib.model_mallocs() <= k:
            break


def test_failed_allocations_reach_the_constant_tables(library, tmp_path):
    def failures(models):
        for k, m in models:
            s, off, tree, pl = m.stream(), (C.c_int64 * 2)(0, 5000), C.c_void_p(), C.c_void_p()
            m.lib.fmm_debug_fail_alloc(C.c_int64(k))
            rc = m.lib.fmm_build_tree(m.buf, off, 1, C.byref(C.c_int(5)), s, C.byref(tree))
            if rc == 0:
                rc = m.lib.fmm_plan(tree, 12, C.c_double(0.5), 0, None, s, C.byref(pl))
            if rc == 0:
                return k
            assert rc == -2, k

    def warm():                  # another layout has been used before
        for k, m in fresh_models(library, tmp_path, "warm"):
            s = m.stream()
            m.lib.fmm_plan_destroy(m.plan(m.tree(300, 3, s), s))
            yield k, m

    # the first plan of a process makes one block more: the tables
    assert failures(fresh_models(library, tmp_path)) == failures(warm()) + 1


@pytest.mark.parametrize("p", [12, 40])
@pytest.mark.parametrize("flag", [0, 4, 8, 12])
def test_nothing_is_created_inside_a_capture(model, flag, p):
    # the first use of a process is a graph plan, its lists split or not
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))
    pl = model.plan(model.tree(5000, 5, s), s, p=p, flags=F.FMM_FLAG_GRAPH)
    model.ok(model.call("evaluate", pl, s))
    assert model.lib.model_created_in_capture() == 0


@pytest.mark.parametrize("flag", [0, 12])
def test_fixed_memory_evaluation_creates_nothing(model, flag):
    # under a caller's capture: the plan's lists final, nothing evaluated yet
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))
    pl = model.plan(model.tree(5000, 5, s), s)
    model.ok(model.lib.fmm_plan_stats(pl, C.byref(F._Stats())))
    model.lib.hipStreamBeginCapture(s, 0)
    model.ok(model.call("static", pl, s))
    assert model.lib.model_created_in_capture() == 0


@pytest.mark.parametrize("prec,per_leaf", [(0, 3), (1, 2)])
@pytest.mark.parametrize("n,L", [(300, 3), (70000, 8)])
def test_points_with_the_derivative_few_per_leaf_are_descended(model, n, L, prec, per_leaf):
    s = model.stream()
    pl = model.plan(model.tree(n, L, s), s, prec=prec)
    line = max(8192, per_leaf * 4 ** (L - 1))
    for M, own in ((1, 0), (line, 0), (line + 1, 1)):
        model.lib.model_clear()
        model.ok(model.call("%d:field" % M, pl, s))
        assert model.lib.model_launches(b"k_pts_near_der") == own, M


@pytest.mark.parametrize("flag,longest", [(0, 2 ** 31 - 1), (4, 512)])
def test_long_lists_of_points_with_the_derivative_are_descended(model, flag, longest):
    # split strong lists: the own kernel (its 14th argument) leaves out what the
    # descents (their 5th) take, leaves with more than 512 boxes in their list
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))
    pl = model.plan(model.tree(5000, 5, s), s)
    for part, arg, value in ((b"k_pts_near_der", 13, longest), (b"k_pts_descend", 4, 512 if flag else 0)):
        model.lib.model_watch(part, arg)
        model.ok(model.call("20000:field", pl, s))
        assert model.lib.model_watched() == value, part


@pytest.mark.parametrize("L,M,theta,line", [(6, 32768, 0.5, 64), (6, 32769, 0.5, 512), (8, 131072, 0.5, 64),
                                            (8, 131073, 0.5, 512), (6, 32768, 0.1875, 85), (6, 32768, 0.01, 512)])
def test_the_line_of_long_lists_by_the_number_of_points(model, L, M, theta, line):
    # up to 32 points per leaf (1024 leaves) and up to 131,072 points (16,384 leaves)
    # the larger of 64 and 3 / theta^2 boxes, else 512 (which is also the most)
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(4))
    pl = model.plan(model.tree(70000, L, s), s, theta=theta)
    for part, arg in ((b"k_pts_near_der", 13), (b"k_pts_descend", 4)):
        model.lib.model_watch(part, arg)
        model.ok(model.call("%d:field" % M, pl, s))
        assert model.lib.model_watched() == line, (part, M)


@pytest.mark.parametrize("n,L,p,flag,apart", [(5000, 5, 12, 12, 0), (16384, 5, 12, 12, 0), (16385, 5, 12, 0, 0),
                                              (16385, 5, 12, 12, 1), (16385, 6, 12, 12, 0), (2048, 3, 40, 0, 0),
                                              (2049, 3, 40, 0, 1), (2049, 5, 40, 0, 0), (4096, 4, 40, 0, 0),
                                              (4097, 4, 40, 0, 1)])
def test_near_field_of_fat_leaves_gathers_for_itself(model, n, L, p, flag, apart):
    # a gather of the strengths apart from P2M's: only on the second stream (split
    # lists above 16,384 points, or more than 32 terms above 2048) and with more
    # than 64 points per leaf; the adjoint afterwards needs nothing of it
    s = model.stream()
    model.lib.model_list_flag(C.c_longlong(flag))
    pl = model.plan(model.tree(n, L, s), s, p=p)
    model.ok(model.lib.fmm_plan_stats(pl, C.byref(F._Stats())))
    model.lib.model_clear()
    model.ok(model.call("evaluate", pl, s))
    assert model.lib.model_launches(b"k_gather") == apart
    assert model.lib.model_not_joined(s) == 0


@pytest.mark.parametrize("n,L,fat", [(4096, 3, 0), (4097, 3, 1), (16384, 4, 0), (16385, 4, 1), (3000, 2, 0)])
def test_leaves_of_many_points_have_their_own_launches(model, n, L, fat):
    # above 256 points per leaf (three levels and more): P2M and L2P apart from the
    # subtrees'; problems of one or two levels have no subtrees
    s = model.stream()
    pl = model.plan(model.tree(n, L, s), s)
    model.ok(model.lib.fmm_plan_stats(pl, C.byref(F._Stats())))
    for kind, l2p in (("evaluate", b"5k_l2pI"), ("field", b"13k_field_finalI")):
        model.lib.model_clear()
        model.ok(model.call(kind, pl, s))
        assert model.lib.model_launches(b"5k_p2mI") == model.lib.model_launches(l2p) == (fat or L < 3), kind
        assert model.lib.model_launches(b"k_up_leaf") == model.lib.model_launches(b"k_down_leaf") == (L >= 3), kind
        assert model.lib.model_not_joined(s) == 0


def test_two_threads_make_plans_of_one_layout(model):
    # trees of their own that share a layout: while one thread prepares the layout's
    # launch lists (here: waits for their copy) the other's fmm_plan waits
    s, t = model.stream(), model.stream()
    model.plan(model.tree(300, 3, s), s)               # the constant tables are there
    mine, other = model.tree(5000, 5, s), model.tree(5000, 5, t)
    waited, made = [], []
    thread = threading.Thread(target=lambda: made.append(model.plan(other, t)))

    def meanwhile():
        thread.start()
        thread.join(0.3)
        waited.append(thread.is_alive())

    hook = C.CFUNCTYPE(None)(meanwhile)
    model.lib.model_on_sync(hook)
    pl = model.plan(mine, s)
    thread.join()
    assert waited == [True] and len(made) == 1
    for p, st in ((pl, s), (made[0], t)):
        model.ok(model.call("evaluate", p, st))


@pytest.mark.parametrize("n,L,wide", [(1024, 3, 0), (1025, 3, 1), (100, 1, 1), (64, 1, 0)])
def test_log_l2p_takes_a_workgroup_for_fat_leaves(model, n, L, wide):
    s = model.stream()
    pl = model.plan(model.tree(n, L, s), s)
    model.lib.model_clear()
    model.ok(model.call("log", pl, s))
    assert model.lib.model_launches(b"k_l2p_logIdLi256E") == wide
    assert model.lib.model_launches(b"k_l2p_logIdLi32E") == 1 - wide
