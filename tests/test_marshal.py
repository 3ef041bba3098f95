"""The native argument marshalling (csrc/lcsa_marshal.cpp) against the Python functions it stands in for: the same results, and for
whatever it does not take, the same errors."""
import ctypes
import importlib.util
import os
import subprocess
import sys
import threading
import types
import weakref

import pytest
import torch

from paper_2510_12747_amd import binding as B
from paper_2510_12747_amd import build

NOTHING = types.SimpleNamespace(append=lambda *a: None, pool_select=lambda *a: None, forward=lambda *a: None)


PROBES = """
#include <ATen/ATen.h>
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
extern "C" {
__attribute__((visibility("default"))) int fail_wraps = 0, fail_allocations = 0, locked_allocations = 0, allocations = 0;
}
static at::Tensor probed_empty(at::IntArrayRef sizes, at::TensorOptions options) {
    ++allocations;
    locked_allocations += PyGILState_Check();
    if (fail_allocations && --fail_allocations == 0) throw 1;
    return at::empty(sizes, options);
}
static PyObject *probed_wrap(at::Tensor x) {
    if (fail_wraps && --fail_wraps == 0) throw 1;
    return THPVariable_Wrap(std::move(x));
}
"""
LIBRARY = """
#include <stdint.h>
#include <stdlib.h>
#include <unistd.h>
int calls, status, delay_us;
int64_t seen[12];
int append(void *c, const void *k, const void *v, int64_t st, int64_t sh, int32_t n, void *s) {
    int64_t a[] = {(int64_t)c, (int64_t)k, (int64_t)v, st, sh, n, (int64_t)s};
    for (int i = 0; i < 7; ++i) seen[i] = a[i];
    usleep(delay_us); ++calls; return status;
}
int pool_select(const void *g, const void *q, int64_t st, int64_t sh, const void *c, float *p, int32_t *i_, int32_t *n, float *gap, void *s) {
    int64_t a[] = {(int64_t)g, (int64_t)q, st, sh, (int64_t)c, (int64_t)p, (int64_t)i_, (int64_t)n, (int64_t)gap, (int64_t)s};
    for (int i = 0; i < 10; ++i) seen[i] = a[i];
    usleep(delay_us); ++calls; return status;
}
int forward(const void *g, const void *q, int64_t st, int64_t sh, const void *c, const int32_t *i_, const int32_t *n, void *o, int64_t ost, int64_t osh,
            float *l, float scale, void *s) {
    int64_t a[] = {(int64_t)g, (int64_t)q, st, sh, (int64_t)c, (int64_t)i_, (int64_t)n, (int64_t)o, ost, osh, (int64_t)l, (int64_t)s};
    for (int i = 0; i < 12; ++i) seen[i] = a[i];
    usleep(delay_us); ++calls; return status;
}
static void linger(void) { usleep(1000000); }
void linger_at_exit(void) { atexit(linger); }
"""


def load_on_cpu(folder):
    """The marshalling's source built for CPU tensors in front of a library that only notes its arguments."""
    spec = importlib.util.spec_from_file_location("_marshal", os.path.join(folder, "_marshal.so"))
    native = importlib.util.module_from_spec(spec)
    library = ctypes.CDLL(os.path.join(folder, "library.so"))
    native.bind(*(ctypes.cast(f, ctypes.c_void_p).value for f in (library.append, library.pool_select, library.forward)))
    return native, library


@pytest.fixture(scope="module")
def on_cpu(tmp_path_factory):
    folder = tmp_path_factory.mktemp("marshal")
    with open(os.path.join(build.CSRC, "lcsa_marshal.cpp")) as f:
        source = f.read()
    for old, new in (("is_cuda()", "is_cpu()"), ("THPVariable_Wrap(", "probed_wrap("), ("at::empty(", "probed_empty(")):
        assert old in source
        source = source.replace(old, new)
    (folder / "marshal.cpp").write_text(PROBES + source)
    (folder / "library.c").write_text(LIBRARY)
    build.build_marshal(source=str(folder / "marshal.cpp"), out=str(folder / "_marshal.so"))
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(folder / "library.so"), str(folder / "library.c")], check=True)
    return (str(folder), *load_on_cpu(folder))


GEOM = (2, 32, 6, 8, 4, 4, 2, 4, 4, 4, 4, B.LCSA_F32)


def arguments():
    """Of a layer's three calls, without their streams."""
    g = B.Geom(*GEOM)
    x = torch.zeros(96, 2, 32)
    i, n = torch.zeros(2, 8, 4, dtype=torch.int32), torch.zeros(2, 8, dtype=torch.int32)
    return (g._plan(), 5, x, x, 2), (g._plan(), x, 5, True), (g._plan(), x, 5, i, n, None, None, 0.0)


@pytest.mark.parametrize("how", ["absent", "unloadable", "another torch", "of before it told"])
def test_the_library_loads_without_it(monkeypatch, tmp_path, how):
    """Callers that need none of its functions, and those that do: the Python functions are all there."""
    B.lib()
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_marshal", B._marshal)
    if how == "another torch":
        monkeypatch.setattr(B._marshal, "torch_version", "1.0.0")
    elif how == "of before it told":
        monkeypatch.delattr(B._marshal, "torch_version")
    else:
        if how == "unloadable":
            (tmp_path / "_marshal.so").write_bytes(b"no object file")
        monkeypatch.setattr(sys.modules[B.__package__], "__path__", [str(tmp_path)])
        monkeypatch.delattr(sys.modules[B.__package__], "_marshal", raising=False)
        monkeypatch.delitem(sys.modules, B.__package__ + "._marshal", raising=False)
    with pytest.warns(RuntimeWarning, match="_marshal.so not loaded"):
        assert B.lcsa_cache_device_bytes(B.Geom(*GEOM)) > 0
    (plan, *a), (_, *b), (_, *c) = arguments()
    assert B._marshal.append(plan, *a, 7) is B._marshal.pool_select(plan, *b, 7) is B._marshal.forward(plan, *c, 7) is None
    with pytest.raises(B.LcsaError, match="device tensor"):
        B._tok(a[1])


def test_a_thread_that_the_interpreter_ends_in_a_call_ends_quietly(on_cpu):
    """The interpreter shuts down while daemon threads are in the library: they are ended when they come back, not the process."""
    folder = on_cpu[0]
    script = f"""
import ctypes, sys, threading, time
sys.path[:0] = {[os.path.dirname(__file__), os.path.dirname(build.HERE)]!r}
import test_marshal as t
native, library = t.load_on_cpu({folder!r})
append, pool_select, forward = t.arguments()
ctypes.c_int.in_dll(library, "delay_us").value = 500000
for f, a in ((native.append, append), (native.pool_select, pool_select), (native.forward, forward)):
    threading.Thread(target=f, args=(*a, 7), daemon=True).start()
time.sleep(0.2)
library.linger_at_exit()
print("leaving", flush=True)
"""
    done = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True, timeout=120)
    assert done.stdout == "leaving\n" and done.returncode == 0, (done.returncode, done.stderr)


def test_a_result_that_python_cannot_take_is_an_error_and_not_a_second_launch(on_cpu):
    _, native, library = on_cpu
    calls, fail = ctypes.c_int.in_dll(library, "calls"), ctypes.c_int.in_dll(ctypes.CDLL(native.__file__), "fail_wraps")
    _, pool_select, forward = arguments()
    for f, a, results in ((native.pool_select, pool_select, 4), (native.forward, forward, 1)):
        for nth in range(1, results + 1):
            calls.value, fail.value = 0, nth
            with pytest.raises(RuntimeError):
                f(*a, 7)
            assert calls.value == 1 and fail.value == 0


def test_outputs_are_allocated_without_the_interpreter_lock(on_cpu):
    """As torch.empty allocates; and where an allocation throws, the Python function is to go on."""
    _, native, library = on_cpu
    probes = ctypes.CDLL(native.__file__)
    calls, fail, made, locked = ctypes.c_int.in_dll(library, "calls"), *(ctypes.c_int.in_dll(probes, p) for p in ("fail_allocations", "allocations", "locked_allocations"))
    _, pool_select, forward = arguments()
    for f, a, outputs in ((native.pool_select, pool_select, 4), (native.forward, forward, 1)):
        calls.value = made.value = locked.value = 0
        assert f(*a, 7) is not None and [calls.value, made.value, locked.value] == [1, outputs, 0]
        for nth in range(1, outputs + 1):
            fail.value = nth
            assert f(*a, 7) is None and calls.value == 1 and fail.value == 0


def test_what_it_takes_reaches_the_library(on_cpu):
    _, native, library = on_cpu
    calls, status, seen = (t.in_dll(library, n) for t, n in ((ctypes.c_int, "calls"), (ctypes.c_int, "status"), (ctypes.c_int64 * 12, "seen")))
    head_major = lambda x: x.transpose(0, 1).contiguous().transpose(0, 1)
    g = B.Geom(*GEOM)
    plan, at = g._plan(), g._plan()[0]
    i, n = torch.zeros(2, 8, 4, dtype=torch.int32), torch.zeros(2, 8, dtype=torch.int32)
    for x in (torch.zeros(96, 2, 32), head_major(torch.zeros(96, 2, 32)), torch.zeros(96, 4, 64)[:, ::2, :32], torch.nn.Parameter(torch.zeros(96, 2, 32))):
        y = x.detach().clone(memory_format=torch.preserve_format) if x.is_contiguous() else x
        st, sh = x.stride()[:2]
        assert native.append(plan, 5, x, y, 2, 7) == 0 and list(seen[:7]) == [5, x.data_ptr(), y.data_ptr(), st, sh, 2, 7]
        for want_gap in (True, False):
            pooled, idx, cnt, gap = native.pool_select(plan, x, 5, want_gap, 7)
            assert (gap is not None) == want_gap
            assert list(seen[:10]) == [at, x.data_ptr(), st, sh, 5, pooled.data_ptr(), idx.data_ptr(), cnt.data_ptr(), gap.data_ptr() if want_gap else 0, 7]
            assert [(tuple(t.shape), t.dtype) for t in (pooled, idx, cnt)] == [((2, 8, 32), torch.float32), ((2, 8, 4), torch.int32), ((2, 8), torch.int32)]
            assert not want_gap or (tuple(gap.shape), gap.dtype) == ((2, 8), torch.float32)
        for o, lse in ((None, None), (torch.zeros(96, 2, 32), torch.zeros(96, 2)), (head_major(torch.zeros(96, 2, 32)), None)):
            got = native.forward(plan, x, 5, i, n, o, lse, 0.0, 7)
            assert got is o or (o is None and tuple(got.shape) == (96, 2, 32) and got.is_contiguous())
            assert list(seen) == [at, x.data_ptr(), st, sh, 5, i.data_ptr(), n.data_ptr(), got.data_ptr(), *got.stride()[:2], lse.data_ptr() if lse is not None else 0, 7]
    x = torch.zeros(96, 2, 32)
    status.value = -2
    assert native.append(plan, 5, x, x, 2, 7) == native.pool_select(plan, x, 5, True, 7) == native.forward(plan, x, 5, i, n, None, None, 0.0, 7) == -2
    status.value = calls.value = 0
    # what it leaves to the Python functions: each by itself, everything else being in order
    wrong = [x[:-1], x[:, :1], x[..., :16], x.double(), x.bfloat16(), x[..., ::2], x.reshape(-1), x.to_sparse(), torch.zeros(96, 32, 2).transpose(1, 2),
             x.as_subclass(type("Sub", (torch.Tensor,), {}))]
    for bad in wrong:
        assert native.append(plan, 5, bad, x, 2, 7) is native.append(plan, 5, x, bad, 2, 7) is native.pool_select(plan, bad, 5, True, 7) is None
        assert native.forward(plan, bad, 5, i, n, None, None, 0.0, 7) is native.forward(plan, x, 5, i, n, bad, None, 0.0, 7) is None
    assert native.append(plan, 5, x, head_major(x), 2, 7) is native.append(plan, 5, x, x, 1, 7) is native.append(plan, 5, x, x, True, 7) is None
    assert native.pool_select(plan, x, 5, 1, 7) is native.pool_select(plan, x, None, True, 7) is native.pool_select(plan, x, 5, True, None) is None
    for bad_i, bad_n in ((i.long(), n), (i[:, :, :3], n), (i[:1], n), (i, n.long()), (i, torch.zeros(2, 16, dtype=torch.int32)[:, ::2])):
        assert native.forward(plan, x, 5, bad_i, bad_n, None, None, 0.0, 7) is None
    for bad in (torch.zeros(2, 96), torch.zeros(96, 2, dtype=torch.float64), torch.zeros(192), torch.zeros(96, 4)[:, ::2]):
        assert native.forward(plan, x, 5, i, n, None, bad, 0.0, 7) is None
    assert native.forward(plan, x, 5, i, n, None, None, 0, 7) is None
    for bad in (plan[:7], (*plan, 0), list(plan), (1 << 70,) * 8, (None,) * 8, None):
        assert native.append(bad, 5, x, x, 2, 7) is native.pool_select(bad, x, 5, True, 7) is native.forward(bad, x, 5, i, n, None, None, 0.0, 7) is None
    assert calls.value == 0


def test_it_takes_only_plain_device_tensors():
    B.lib()
    g = B.Geom(1, 32, 6, 8, 4, 4, 2, 4, 4, 4, 4, dtype=B.LCSA_F32)
    x = torch.zeros(96, 1, 32)                               # on the CPU
    i, n = torch.zeros(1, 8, 4, dtype=torch.int32), torch.zeros(1, 8, dtype=torch.int32)
    for plan in (g._plan(), g._plan()[:7], list(g._plan()), (1 << 70,) * 8, None):
        assert B._marshal.append(plan, 0, x, x, 2, 0) is None
        assert B._marshal.pool_select(plan, x, 0, True, 0) is None
        assert B._marshal.forward(plan, x, 0, i, n, None, None, 0.0, 0) is None
    for bad in (None, 3, [x], "x"):
        assert B._marshal.append(g._plan(), 0, bad, x, 2, 0) is None
        assert B._marshal.pool_select(g._plan(), bad, 0, True, 0) is None
        assert B._marshal.forward(g._plan(), x, 0, bad, n, None, None, 0.0, 0) is None
    assert B._marshal.append(g._plan(), 0, x, x, 1 << 40, 0) is None and B._marshal.append(g._plan()) is None
    with pytest.raises(TypeError):
        B._marshal.bind(1, 2)
    assert B.Geom(**vars(g))._plan()[1:] == g._plan()[1:]


def test_a_plan_keeps_the_struct_whose_address_it_holds(monkeypatch):
    """Two first uses of one geometry at a time, from two threads: every interleaving leaves an address of a living struct."""
    fields = (1, 32, 6, 8, 4, 4, 2, 4, 4, 4, 4, B.LCSA_F32)
    made, build = [], B.Geom.c

    def interrupted(self):
        """Another thread's whole first use, between the first look at the geometry and the struct that follows from it."""
        monkeypatch.setattr(B.Geom, "c", recorded)
        self._plan()
        return recorded(self)

    def recorded(self):
        struct = build(self)
        made.append(weakref.ref(struct))
        return struct

    alive = lambda address: any(w() is not None and ctypes.addressof(w()) == address for w in made)
    for first in (B.Geom._ref, B.Geom._plan):
        g = B.Geom(*fields)
        monkeypatch.setattr(B.Geom, "c", interrupted)
        first(g)
        assert alive(g._plan()[0])
        plan, seen = g._plan(), bytes(build(g))
        del g
        assert alive(plan[0]) and ctypes.string_at(plan[0], len(seen)) == seen

    monkeypatch.setattr(B.Geom, "c", build)
    geoms, interval, start = [B.Geom(*fields) for _ in range(4000)], sys.getswitchinterval(), threading.Barrier(4)

    def use():
        start.wait()
        for g in geoms:
            g._ref()
            g._plan()

    threads = [threading.Thread(target=use) for _ in range(4)]
    sys.setswitchinterval(1e-7)
    try:
        for t in threads: t.start()
        for t in threads: t.join()
    finally:
        sys.setswitchinterval(interval)
    want = bytes(geoms[0].c())
    assert all(g._plan()[0] == ctypes.addressof(g._plan()[0].struct) and bytes(g._plan()[0].struct) == want for g in geoms)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,tile", [("fp32", 32, (4, 4)), ("bf16", 64, (4, 8)), ("bf16", 128, (8, 16))])
def test_results_and_errors_are_those_of_the_python_functions(monkeypatch, dtype, d, tile):
    h, w, heads, dt = 3 * tile[0] - 1, 2 * tile[1] + 3, 3, torch.float32 if dtype == "fp32" else torch.bfloat16
    g = B.Geom(heads, d, h, w, *tile, 2, 4, 16, 16, 5, dtype=B.LCSA_F32 if dtype == "fp32" else B.LCSA_BF16)
    gen = torch.Generator(device="cuda").manual_seed(0)
    make = lambda frames: torch.randn(frames * h * w, heads, d, generator=gen, device="cuda").to(dt)
    q, k, v = make(2), make(2), make(2)
    head_major = lambda x: x.transpose(0, 1).contiguous().transpose(0, 1)

    class Sub(torch.Tensor):
        pass

    def steps(q, k, v, **kw):
        cache = B.lcsa_cache_init(g)
        for _ in range(2):
            B.lcsa_kv_cache_append(cache, k, v, 2)
        pooled, idx, cnt, gap = B.lcsa_pool_select_blocks(g, q, cache, want_gap=kw.get("want_gap", True))
        lse = torch.empty(q.shape[0], heads, device="cuda") if kw.get("lse") else None
        o = torch.empty_like(q) if kw.get("o") else None
        got = B.lcsa_sparse_attn_fwd(g, q, cache, idx, cnt, o=o, lse=lse, scale=kw.get("scale", 0.0))
        assert o is None or got is o
        assert got.is_contiguous() or o is not None
        return [cache.storage[:0], B.lcsa_cache_pooled_k(cache).clone(), pooled, idx, cnt, gap, lse, got]

    forms = [((q, k, v), {}), ((head_major(q), head_major(k), head_major(v)), dict(lse=True)), ((q, head_major(k), head_major(v)), dict(o=True, want_gap=False)),
             ((torch.nn.Parameter(q, requires_grad=False), k, v), dict(scale=0.3)), ((q.as_subclass(Sub), k, v), dict(scale=1))]
    assert B._marshal is not B._InPython
    answers = []
    note = types.SimpleNamespace(**{f: (lambda *a, f=f, real=getattr(B._marshal, f): answers.append((f, real(*a))) or answers[-1][1])
                                    for f in ("append", "pool_select", "forward")})
    for (a, b, c), kw in forms:
        answers.clear()
        with monkeypatch.context() as m:
            m.setattr(B, "_marshal", note)
            native = steps(a, b, c, **kw)
        # k and v are plain in every form; the last form's q is not, and its scale no float
        assert [f for f, _ in answers] == ["append", "append", "pool_select", "forward"]
        taken = not isinstance(a, Sub)
        assert [x is not None for _, x in answers] == [True, True, taken, taken]
        with monkeypatch.context() as m:
            m.setattr(B, "_marshal", NOTHING)
            python = steps(a, b, c, **kw)
        for x, y in zip(native, python):
            assert (x is None) == (y is None)
            if x is not None:
                assert x.shape == y.shape and x.dtype == y.dtype and x.stride() == y.stride() and torch.equal(x, y)

    cache = B.lcsa_cache_init(g)
    B.lcsa_kv_cache_append(cache, k, v, 2)
    idx, cnt = torch.zeros(heads, g.n_qb, 5, dtype=torch.int32, device="cuda"), torch.zeros(heads, g.n_qb, dtype=torch.int32, device="cuda")
    other = torch.float32 if dt == torch.bfloat16 else torch.bfloat16
    wrong = [lambda: B.lcsa_kv_cache_append(cache, k[:-1], v[:-1], 2), lambda: B.lcsa_kv_cache_append(cache, k, head_major(v), 2),
             lambda: B.lcsa_kv_cache_append(cache, k.to(other), v.to(other), 2), lambda: B.lcsa_kv_cache_append(cache, k.cpu(), v.cpu(), 2),
             lambda: B.lcsa_pool_select_blocks(g, q[:-1], cache), lambda: B.lcsa_pool_select_blocks(g, q.to(other), cache),
             lambda: B.lcsa_sparse_attn_fwd(g, q, cache, idx[:, :, :4], cnt), lambda: B.lcsa_sparse_attn_fwd(g, q, cache, idx.long(), cnt),
             lambda: B.lcsa_sparse_attn_fwd(g, q, cache, idx, cnt, lse=torch.empty(heads, q.shape[0], device="cuda")),
             lambda: B.lcsa_sparse_attn_fwd(g, q, cache, idx, cnt, o=torch.empty(q.shape[0], heads, d, 2, device="cuda", dtype=dt)[..., 0]),
             lambda: B.lcsa_pool_select_blocks(B.Geom(**{**vars(g), "q_frames": 4, "cache_frames": 8}), make(4), cache)]      # another geometry: the library refuses
    for call in wrong:
        with pytest.raises((B.LcsaError, AssertionError)) as native:
            call()
        with monkeypatch.context() as m:
            m.setattr(B, "_marshal", NOTHING)
            with pytest.raises((B.LcsaError, AssertionError)) as python:
                call()
        assert type(native.value) is type(python.value) and str(native.value) == str(python.value)
