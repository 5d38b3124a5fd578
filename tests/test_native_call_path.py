"""The binding's native call path (_launch) against its Python path, which takes over whenever an argument is
not exactly of the plain type (here: the softmax scale as numpy.float64).  Both reach the same kernels, so
results are compared bit for bit; errors must be the Python path's."""
import ctypes
import os
import subprocess
import sys
import threading

import numpy as np
import pytest
import torch

import paper_2506_04421_amd as hm
from paper_2506_04421_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

D = 64
MARKOV_COUNTS = hm.HMAR_MASK_MARKOV | hm.HMAR_SCALE_COUNTS


def _tensors(n, shape, device, seed=0):
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    return [torch.randn(shape, generator=g).to(torch.bfloat16).to(device) for _ in range(n)]


def test_host_tensors_and_other_types_are_left_to_the_python_path():
    hm.load_library()
    native = binding._launch
    q = torch.zeros((1, 1, 5, D), dtype=torch.bfloat16)
    lse = torch.zeros((1, 1, 5))
    binding._sides_array((1, 2))
    known = binding._known_sides((1, 2), 0)
    assert known[1:] == (2, 5) and binding._known_sides([1, 2], 0) == known
    assert binding._known_sides((7, 7, 7), 0) is None and binding._known_sides(([1], 2), 0) is None
    assert binding._known_sides(iter((1, 2)), 0) is None and binding._known_sides((1, 2), MARKOV_COUNTS) is None
    assert native.fwd(q, q, q, None, None, *known, 0, 0.0) is None
    assert native.fwd("Q", q, q, None, None, *known, 0, 0.0) is None
    assert native.fwd(q, q) is None
    assert native.bwd(q, q, q, q, q, lse, None, None, None, None, *known, 0, 0.0) is None
    assert native.bwd_noalloc(q, q, q, q, q, lse, q, q, q, *known, 0.0) is None
    assert native.step(q, q, q, 0, None, None, 0.0) is None
    assert native.rows(q, q, q, 0, torch.zeros(1, dtype=torch.int32), q, lse, 0.0) is None
    assert native.steps([q], [q], [q], [0], None, None, 0.0) is None
    assert native.steps([], [], [], [], None, None, 0.0) is None


def test_the_library_works_without_the_native_path(monkeypatch):
    # the module needs torch's C++ interface and Python's headers where it is built; the library never did
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_launch", None)
    monkeypatch.delattr(hm, "_launch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2506_04421_amd._launch", None)          # importing it fails
    with pytest.warns(RuntimeWarning, match="native call path"):
        assert hm.hmar_schedule_describe((1, 2, 3, 4)) == ([0, 1, 5, 14, 30], 538)
    q = torch.zeros((1, 1, 5, D), dtype=torch.bfloat16)
    binding._sides_array((1, 2))
    for call in (lambda: hm.hmar_attn_fwd(q, q, q, (1, 2)), lambda: hm.hmar_attn_step_fwd(q, q, q, 0),
                 lambda: hm.hmar_attn_bwd(q, q, q, q, q, q, (1, 2))):
        with pytest.raises(hm.HmarError, match="^Q must be a device tensor"):
            call()


def test_the_library_is_built_where_the_native_path_is_not(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "LAUNCH_PATH", str(tmp_path / "_launch.so"))
    monkeypatch.setattr(build, "SOURCES", ["schedule.cpp"])
    for command in (["false"], [str(tmp_path / "no_such_compiler")]):
        monkeypatch.setattr(build, "launch_command", lambda out, c=command: c)
        (tmp_path / "lib.so").unlink(missing_ok=True)
        with pytest.raises(RuntimeError, match="_launch.so"):
            build.build_library()
        assert (tmp_path / "lib.so").exists() and not (tmp_path / "_launch.so").exists()


@pytest.mark.parametrize("moment", ["before", "after"])
def test_two_threads_that_meet_a_schedule_first_share_one_array(monkeypatch, moment):
    # both have found nothing; the second stores its entry just before or just after the first one does.  The address
    # the native path is given must be that of the array that is kept
    class Cache(dict):
        met = blind = False

        def get(self, *a):
            return None if self.blind else super().get(*a)

        def meet(self):
            if not self.met:
                self.met = self.blind = True
                second = threading.Thread(target=binding._sides_array, args=((23, 29),))
                second.start()
                second.join()
                self.blind = False

        def setdefault(self, *a):
            if moment == "before":
                self.meet()
            res = super().setdefault(*a)
            self.meet()
            return res

        def __setitem__(self, *a):
            if moment == "before":
                self.meet()
            super().__setitem__(*a)
            self.meet()
    monkeypatch.setattr(binding, "_SIDES_CACHE", Cache())
    array, count, L = binding._sides_array((23, 29))
    assert binding._SIDES_CACHE.met and list(array) == [23, 29] and (count, L) == (2, 1370)
    kept = binding._sides_array((23, 29))[0]
    assert binding._known_sides((23, 29), 0) == (ctypes.addressof(kept), 2, 1370)


HOST_MODULE = """
import ctypes, importlib.util, sys, threading
import torch
spec = importlib.util.spec_from_file_location("_launch", sys.argv[1])
native = importlib.util.module_from_spec(spec)
spec.loader.exec_module(native)
calls = []
def stand_in(name, code):
    def f(*args):
        calls.append(name)
        return code
    return ctypes.CFUNCTYPE(ctypes.c_int64)(f)          # reads no argument
names = ("fwd", "bwd", "bwd_noalloc", "ws_bytes", "steps", "rows")
keep = [stand_in(n, 4096 if n == "ws_bytes" else 0) for n in names]
native.bind(*[ctypes.cast(f, ctypes.c_void_p).value for f in keep])
q, k, v, o, g = (torch.randn(1, 2, 5, 64).bfloat16() for _ in range(5))
dq, dk, dv = (torch.empty_like(q) for _ in range(3))
lse, rows, ws = torch.zeros(1, 2, 5), torch.zeros(3, dtype=torch.int32), torch.zeros(4096, dtype=torch.uint8)
sides = (ctypes.c_int32 * 2)(1, 2)
s = (ctypes.addressof(sides), 2, 5)
new = {                                                  # these allocate: under a transform they are left to Python
    "fwd": lambda: native.fwd(q, k, v, None, None, *s, 0, 0.0),
    "fwd, O given": lambda: native.fwd(q, k, v, o, None, *s, 0, 0.0),
    "bwd": lambda: native.bwd(q, k, v, o, g, lse, None, None, None, ws, *s, 0, 0.0),
    "bwd, workspace": lambda: native.bwd(q, k, v, o, g, lse, dq, dk, dv, None, *s, 0, 0.0),
    "step": lambda: native.step(q, k, v, 0, None, None, 0.0),
    "steps": lambda: native.steps([q], [k], [v], [0], None, None, 0.0)}
given = {
    "fwd": lambda: native.fwd(q, k, v, o, lse, *s, 0, 0.0),
    "bwd": lambda: native.bwd(q, k, v, o, g, lse, dq, dk, dv, ws, *s, 0, 0.0),
    "bwd_noalloc": lambda: native.bwd_noalloc(q, k, v, o, g, lse, dq, dk, dv, *s, 0.0),
    "step": lambda: native.step(q, k, v, 0, o, lse, 0.0),
    "steps": lambda: native.steps([q], [k], [v], [0], [o], [lse], 0.0),
    "rows": lambda: native.rows(q, k, v, 0, rows, o, lse, 0.0)}
"""

TRANSFORMS = HOST_MODULE + """
def transforms(f):
    res = []
    def body(x):
        res.append(f())
        return (x * x).sum()
    x = torch.ones(3)
    torch.func.grad(body)(x)
    torch.func.vjp(body, x)
    torch.func.jvp(body, (x,), (x,))
    torch.func.vmap(lambda y: body(y))(torch.ones(2, 3))
    return res
for name, f in new.items():
    assert f() is not None, name
    calls.clear()
    res = transforms(f)
    launched = [c for c in calls if c != "ws_bytes"]
    assert res[:3] == [None] * 3 and len(launched) == sum(n is not None for n in res), (name, res, calls)
    assert f() is not None, name
for name, f in given.items():
    calls.clear()
    assert all(r is not None for r in transforms(f)) and len(calls) == 4, (name, calls)
t = threading.Thread(target=lambda: transforms(new["fwd"]))
t.start(); t.join()
print("done")
"""


@pytest.fixture(scope="module")
def host_module(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("host_module") / "_launch.so")
    subprocess.run(build.launch_command(path, ["HMAR_LAUNCH_HOST"]), check=True, timeout=300)
    return path


def _run_on_host_module(program, path):
    res = subprocess.run([sys.executable, "-c", program, path], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert res.returncode == 0 and res.stdout.strip().endswith("done"), res.stdout + res.stderr


def test_function_transforms_around_a_call_are_left_to_the_python_path(host_module):
    # inside torch.func.grad and its like a new tensor is a wrapper without memory, also where every input is a plain
    # constant of the closure; met with the GIL released that ended the process, hence one of its own here
    _run_on_host_module(TRANSFORMS, host_module)


NEW_OUTPUTS = HOST_MODULE + """
# what waits on the way of a new tensor: the fill of deterministic algorithms, and observers.  The stand-ins write
# nothing, so a filled output stays NaN
new["rows"] = lambda: native.rows(q, k, v, 0, rows, None, None, 0.0)
def outputs(x):
    return [t for y in x for t in (y if isinstance(y, list) else [y])]
for name, f in new.items():
    for fill in (True, False):
        torch.use_deterministic_algorithms(True)
        torch.utils.deterministic.fill_uninitialized_memory = fill
        given_too = {o.data_ptr(), dq.data_ptr(), dk.data_ptr(), dv.data_ptr()}
        for i in range(3):
            junk = [torch.zeros(s) for s in ((1, 2, 5, 32), (1, 2, 5))]        # what the allocator hands out next is not NaN
            del junk
            made = [t for t in outputs(f()) if t.data_ptr() not in given_too]
            assert made or name == "bwd, workspace", name
            assert not fill or all(t.float().isnan().all() for t in made), name
        torch.use_deterministic_algorithms(False)
    allocations = {"fwd": 2, "fwd, O given": 1, "bwd": 3, "bwd, workspace": 1, "step": 2, "steps": 2, "rows": 2}[name]
    with torch.autograd.profiler.profile() as prof:
        assert f() is not None
    assert sum(e.name == "aten::empty" for e in prof.function_events) == allocations, (name, prof.function_events)
    assert f() is not None
print("done")
"""


def test_new_outputs_are_filled_and_observed_as_the_python_paths_are(host_module):
    _run_on_host_module(NEW_OUTPUTS, host_module)


@pytest.mark.gpu
def test_new_outputs_of_a_row_list_are_filled_and_observed_on_both_paths():
    dev = torch.device("cuda:0")
    q, k, v = (_tensors(1, (1, 2, n, D), dev, seed=n)[0] for n in (90, 130, 130))
    rows = torch.tensor([3, 70], dtype=torch.int32, device=dev)
    others = [i for i in range(90) if i not in (3, 70)]
    junk = [torch.zeros_like(q) for _ in range(4)] + [torch.zeros((1, 2, 90), device=dev) for _ in range(4)]
    del junk                                            # the blocks the allocator hands out next hold no NaN
    torch.use_deterministic_algorithms(True)
    try:
        for scale in (np.float64(0.0), 0.0):            # the Python path, the native one
            O, LSE = hm.hmar_attn_step_fwd_rows(q, k, v, 40, rows, None, None, scale)
            assert O[:, :, others].isnan().all() and LSE[:, :, others].isnan().all()
            assert O[:, :, [3, 70]].isfinite().all() and LSE[:, :, [3, 70]].isfinite().all()
    finally:
        torch.use_deterministic_algorithms(False)
    with torch.autograd.profiler.profile() as prof:
        hm.hmar_attn_step_fwd(q, k, v, 40)
    assert sum(e.name == "aten::empty" for e in prof.function_events) == 2


@pytest.mark.gpu
def test_a_call_on_constants_inside_a_function_transform_raises_the_python_paths_error():
    dev = torch.device("cuda:0")
    q, k, v, g = _tensors(4, (1, 2, 14, D), dev)
    sizes = (1, 2, 3)
    O, LSE = hm.hmar_attn_fwd(q, k, v, sizes)
    dQ, dK, dV = hm.hmar_attn_bwd(q, k, v, O, g, LSE, sizes)
    ws = torch.empty(8 * 2 * 14 + 16, dtype=torch.uint8, device=dev)
    x = torch.ones(3, device=dev)
    for scale in (np.float64(0.0), 0.0):
        for call in (lambda: hm.hmar_attn_fwd(q, k, v, sizes, scale), lambda: hm.hmar_attn_bwd(q, k, v, O, g, LSE, sizes, scale),
                     lambda: hm.hmar_attn_step_fwd(q, k, v, 0, scale), lambda: hm.hmar_attn_steps_fwd([q], [k], [v], [0], scale)):
            with pytest.raises(RuntimeError, match="storage"):
                torch.func.grad(lambda y: (call(), y.sum())[1])(x)
        o, lse, gq, gk, gv = (torch.full_like(t, float("nan")) for t in (O, LSE, dQ, dK, dV))

        def given(y):
            hm.hmar_attn_fwd(q, k, v, sizes, scale, O=o, LSE=lse)
            hm.hmar_attn_bwd(q, k, v, o, g, lse, sizes, scale, dQ=gq, dK=gk, dV=gv, workspace=ws)
            return (y * y).sum()
        assert torch.equal(torch.func.grad(given)(x), 2 * x)
        for a, b in zip((o, lse, gq, gk, gv), (O, LSE, dQ, dK, dV)):
            assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("sizes,kind", [((1, 2, 3), 0), ([2, 5], hm.HMAR_MASK_BLOCK_CAUSAL), ((3, 40, 77), MARKOV_COUNTS)])
def test_training_calls_give_the_same_bits_on_both_paths(sizes, kind):
    dev = torch.device("cuda:0")
    L = sum(n if kind & hm.HMAR_SCALE_COUNTS else n * n for n in sizes)
    q, k, v, g = _tensors(4, (2, 3, L, D), dev)
    results = []
    for scale in (np.float64(0.1), 0.1):                # the Python path first: it makes the schedule known
        O, LSE = hm.hmar_attn_fwd_masked(q, k, v, sizes, kind, scale)
        results.append((O, LSE) + hm.hmar_attn_bwd_masked(q, k, v, O, g, LSE, sizes, kind, scale))
    known = binding._known_sides(sizes, kind)
    assert binding._launch.fwd(q, k, v, None, None, *known, kind, 0.1) is not None       # it is the native one
    for a, b in zip(*results):
        assert a.dtype == b.dtype and torch.equal(a, b)
    # given buffers come back as the same objects
    O, LSE, dQ, dK, dV = (torch.empty_like(t) for t in results[0])
    ws = torch.empty(8 * 6 * L + 16, dtype=torch.uint8, device=dev)
    got = hm.hmar_attn_fwd_masked(q, k, v, sizes, kind, 0.1, O, LSE)
    assert got[0] is O and got[1] is LSE
    got = hm.hmar_attn_bwd_masked(q, k, v, O, g, LSE, sizes, kind, 0.1, dQ, dK, dV, ws)
    assert got[0] is dQ and got[1] is dK and got[2] is dV
    for a, b in zip((O, LSE, dQ, dK, dV), results[0]):
        assert torch.equal(a, b)
    if kind == 0:
        for scale in (np.float64(0.1), 0.1):
            for t in (dQ, dK, dV):
                t.fill_(float("nan"))
            got = hm.hmar_attn_bwd_noalloc(q, k, v, O, g, LSE, sizes, dQ, dK, dV, scale)
            assert got[0] is dQ and all(torch.equal(a, b) for a, b in zip(got, results[0][2:]))


@pytest.mark.gpu
def test_inference_calls_give_the_same_bits_on_both_paths():
    dev = torch.device("cuda:0")
    shapes = [(0, 1), (9, 16), (50, 130)]
    q = [_tensors(1, (1, 3, c, D), dev, seed=c)[0] for _, c in shapes]
    k, v = zip(*[_tensors(2, (1, 3, p + c, D), dev, seed=99 + c) for p, c in shapes])
    n_prev = [p for p, _ in shapes]
    many = [hm.hmar_attn_steps_fwd(q, k, v, n_prev, scale) for scale in (np.float64(0.0), 0.0)]
    for a, b in zip(many[0][0] + many[0][1], many[1][0] + many[1][1]):
        assert torch.equal(a, b)
    some = [None, torch.empty_like(q[1]), None]
    assert hm.hmar_attn_steps_fwd(q, k, v, n_prev, Os=some)[0][1] is some[1] and some[0] is None
    rows = torch.tensor([5, 0, 129], dtype=torch.int32, device=dev)
    for scale in (np.float64(0.0), 0.0):
        O, LSE = hm.hmar_attn_step_fwd(q[2], k[2], v[2], 50, scale)
        assert torch.equal(O, many[0][0][2]) and torch.equal(LSE, many[0][1][2])
        o, lse = torch.zeros_like(O), torch.zeros_like(LSE)
        got = hm.hmar_attn_step_fwd_rows(q[2], k[2], v[2], 50, rows, o, lse, scale)
        assert got[0] is o and got[1] is lse
        assert (o[:, :, [0, 5, 129]] - O[:, :, [0, 5, 129]]).abs().max().item() <= 1e-2 and not o[:, :, 6].any()


@pytest.mark.gpu
def test_errors_are_those_of_the_python_path():
    dev = torch.device("cuda:0")
    q, k, v, g = _tensors(4, (1, 2, 14, D), dev)
    sizes = (1, 2, 3)
    O, LSE = hm.hmar_attn_fwd(q, k, v, sizes)
    f32 = q.float()
    wide = torch.zeros((1, 2, 14, 2 * D), dtype=torch.bfloat16, device=dev)
    for bad in (f32, q[:, :, :13], wide[..., :D], q.cpu(), "K", None):
        with pytest.raises(hm.HmarError, match="^K "):
            hm.hmar_attn_fwd(q, bad, v, sizes)
        with pytest.raises(hm.HmarError, match="^dO "):
            hm.hmar_attn_bwd(q, k, v, O, bad, LSE, sizes)
    with pytest.raises(hm.HmarError, match="sequence length"):
        hm.hmar_attn_fwd(q, k, v, (1, 2))
    with pytest.raises(hm.HmarError, match="HMAR_ERR_INVALID_ARG"):
        hm.hmar_attn_fwd_masked(q, k, v, sizes, 7)
    with pytest.raises(hm.HmarError, match="HMAR_ERR_WORKSPACE"):
        hm.hmar_attn_bwd(q, k, v, O, g, LSE, sizes, workspace=torch.empty(8, dtype=torch.uint8, device=dev))
    with pytest.raises(hm.HmarError, match="hmar_attn_step_fwd failed: HMAR_ERR_INVALID_ARG"):
        hm.hmar_attn_step_fwd(q, k, v, 0, float("nan"))
    with pytest.raises(hm.HmarError, match="equally long"):
        hm.hmar_attn_steps_fwd([q], [k, k], [v], [0])
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_tensor_subclasses_and_function_modes_see_their_calls():
    class Mine(torch.Tensor):
        pass
    dev = torch.device("cuda:0")
    q, k, v = _tensors(3, (1, 2, 14, D), dev)
    want = hm.hmar_attn_fwd(q, k, v, (1, 2, 3))
    got = hm.hmar_attn_fwd(q.as_subclass(Mine), k, v, (1, 2, 3))
    assert type(got[0]) is Mine and torch.equal(got[0].as_subclass(torch.Tensor), want[0])
    seen = []

    class Watch(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    with Watch():
        got = hm.hmar_attn_fwd(q, k, v, (1, 2, 3))
    assert torch.empty_like in seen and torch.equal(got[0], want[0])
