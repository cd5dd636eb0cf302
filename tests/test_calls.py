"""The extension module that Python makes its compute calls through: what it hands on, argument by argument, to functions that
note what they are given (no GPU and no torch tensors needed)."""
import ctypes as C
import math
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

from paper_2402_02447_amd import binding

VP, U32, U64, I32 = C.c_void_p, C.c_uint32, C.c_uint64, C.c_int
HP = C.POINTER(binding._Adam)
SIGNATURES = [("bucket_clip_norms", (VP, U32, U32, VP, VP)), ("bucket_clip_apply", (VP, U32, U32, VP, VP, VP, VP, VP)),
              ("bucket_clip", (VP, U32, U32, VP, VP, VP, VP, VP)), ("bucket_clip_flat", (VP, U64, I32, VP, VP, VP, VP, VP)),
              ("adam_step", (VP, HP, U64, VP)), ("bucket_clip_adam", (VP, VP, HP, U64, U32, VP, VP, VP, VP)),
              ("lamb_step", (VP, HP, U64, VP, VP)), ("bucket_clip_lamb", (VP, VP, HP, U64, U32, VP, VP, VP, VP, VP))]


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Stream:
    cuda_stream = 0x7000_0000_1234


@pytest.fixture(scope="module")
def noted():
    binding.load_library()
    seen, keep, addresses = [], [], []
    for name, types in SIGNATURES:
        def note(*args, name=name):
            seen.append((name, [[getattr(a.contents, f) for f, _ in binding._Adam._fields_] if isinstance(a, HP) and a else
                                None if isinstance(a, HP) else a for a in args]))
            return 7
        keep.append(C.CFUNCTYPE(I32, *types)(note))
        addresses.append(C.cast(keep[-1], VP).value)
    table = binding._calls.connect(*addresses)
    yield lambda name, *args: (getattr(binding._calls, name)(table, *args), seen.pop())
    del keep


@pytest.mark.parametrize("name,types", SIGNATURES)
def test_every_argument_arrives_in_its_place(noted, name, types):
    hp = binding.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)
    given, want = [], []
    for i, t in enumerate(types):
        if t is HP:
            given.append(hp), want.append([1e-3, 0.9, 0.999, 1e-6, 0.01])
        elif t is VP and i == len(types) - 1:
            given.append(Stream()), want.append(Stream.cuda_stream)
        elif t is VP:
            at = 0x7F00_0000_0000 + 4096 * i
            given.append((at, Tensor(at), np.int64(at))[i % 3]), want.append(at)
        else:
            at = (1 << 40) + i if t is U64 else 1 + i
            given.append(at), want.append(at)
    assert noted(name, *given) == (7, (name, want))
    # nothing where something may be left out, and a stream given as a number
    given = [None if t in (VP, HP) else 0 for t in types[:-1]] + [0x55]
    want = [None if t in (VP, HP) else 0 for t in types[:-1]] + [0x55]
    assert noted(name, *given) == (7, (name, want))


def test_what_is_not_an_argument_is_refused(noted):
    ok = (1, 2, binding.AdamHyper(), 3, 0, 4, 5, 6, None)
    assert noted("bucket_clip_adam", *ok)[0] == 7
    for i, bad, error in ((0, "x", ValueError), (1, object(), TypeError), (2, 5, AttributeError), (3, 1.5, TypeError), (3, "1", TypeError),
                          (4, None, TypeError), (8, object(), TypeError)):
        with pytest.raises(error):
            noted("bucket_clip_adam", *ok[:i], bad, *ok[i + 1:])
    with pytest.raises(TypeError):
        noted("bucket_clip_adam", *ok[:-1])
    with pytest.raises(TypeError):
        noted("bucket_clip_adam", *ok, None)
    with pytest.raises(TypeError):
        noted("adam_step", 1, binding.AdamHyper(lr="fast"), 1, None)
    with pytest.raises((TypeError, ValueError)):
        binding._calls.adam_step(object(), 1, None, 1, None)


def test_numbers_of_any_kind_in_the_hyper_parameters(noted):
    _, (_, args) = noted("adam_step", 1, binding.AdamHyper(np.float32(0.5), 0, np.float64(0.25), float("inf"), -1.0), 2, None)
    assert args[1] == [0.5, 0.0, 0.25, math.inf, -1.0]


def test_only_the_compute_calls_need_the_extension_module():
    """Without it (another interpreter, a library named by BCA_LIB) plans, thresholds and the simulation's host side work, and a compute call
    says what is missing."""
    script = """
import sys
sys.modules["torch"] = sys.modules["paper_2402_02447_amd._calls"] = None
import paper_2402_02447_amd as B, workloads as W
from paper_2402_02447_amd import lbs
assert len(B.alg1_thresholds(1.0, 4)) == 4
lbs.Dataset(W.length_histogram_piecewise_uniform(), W.LENGTH_STRATUM_END, device=-1).close()
with B.Plan.from_layout(W.layout_flat_split([5000], 4096), B.BCA_GRAD_F32, device=-1) as plan:
    assert plan.n_buckets == 2 and plan.work_items()
    for call in (lambda: plan.adam_step(B.AdamHyper(), 1), lambda: plan.bucket_clip(0, 1, 64), lambda: B.bucket_clip_flat(64, 1, 0, 64)):
        try:
            call()
        except ImportError as e:
            assert "_calls" in str(e)
        else:
            raise AssertionError("went through")
print("as it should")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", script], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "as it should" in r.stdout, r.stderr[-2000:]


def test_building_the_package_builds_both_parts(monkeypatch):
    from paper_2402_02447_amd import build
    made = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: made.append(cmd[cmd.index("-o") + 1]))
    build.build()
    assert set(made) == {build.LIB, build.CALLS}
    made.clear()
    build.build(out="/tmp/variant.so")      # a variant of the library alone
    assert made == ["/tmp/variant.so"]


class Parameter:
    def __init__(self, x):
        self._as_parameter_ = x


class Index:
    def __index__(self):
        return 12


NUMBERS = [True, 3, -1, 1 << 70, -(1 << 70), 1.5, "1", b"1", None, np.int64(4), np.uint32(4), C.c_uint32(5), C.c_uint64(6), C.c_int(-7), C.c_long(8), C.c_int64(8),
           C.c_uint16(9), C.c_bool(True), C.c_float(1.0), Parameter(10), Parameter(Parameter(11)), Parameter("x"), Parameter(C.c_uint32(12)),
           Index(), object(), (1,)]
ADDRESSES = [None, True, 0, 5, -1, 1 << 70, -(1 << 70), 2.5, "7", b"8", "x", float("inf"), np.int64(9), np.float32(3), C.c_void_p(3), C.c_uint32(4), Parameter(10), Index(),
             object(), Tensor(0), Tensor(64), Tensor(np.int64(64)), Tensor(64.0), Tensor("64"), Tensor(None)]


def outcome(call):
    try:
        return call()
    except Exception as e:
        return type(e)


def test_arguments_are_taken_and_refused_as_by_ctypes(noted):
    """What arrives for, and which exception comes of, arguments of every kind, against the same call made through ctypes."""
    binding.load_library()

    def note(types):
        seen = []
        f = C.CFUNCTYPE(I32, *types)(lambda *a: seen.append(list(a)) or 7)
        return f, seen
    for name, types in SIGNATURES:
        plain = [None if t in (VP, HP) else 1 for t in types]
        for i, t in enumerate(types):
            if t is HP:
                continue
            stream = t is VP and i == len(types) - 1
            f, seen = note([VP if u is HP else u for u in types])

            def through_ctypes(x):
                if t is VP:
                    x = (binding._stream if stream else binding._ptr)(x)
                assert f(*plain[:i], x, *plain[i + 1:]) == 7
                return seen.pop()

            for x in ADDRESSES if t is VP else NUMBERS:
                want = outcome(lambda: through_ctypes(x))
                got = outcome(lambda: noted(name, *plain[:i], x, *plain[i + 1:])[1][1])
                if isinstance(want, type):
                    assert isinstance(got, type) and issubclass(got, want), (name, i, x, want, got)
                else:
                    assert got == want, (name, i, x, want, got)


class Float:
    def __float__(self):
        return 0.125


HYPER = [0.5, 1, True, -1.0, float("nan"), 1 << 70, 1 << 2000, np.float32(0.25), np.float64(0.25), np.int64(3), np.array(0.5), np.array([0.5, 1.0]), C.c_double(0.75), C.c_float(0.75),
         Float(), Index(), Parameter(0.5), "0.5", None, object()]


def test_hyper_parameters_are_taken_and_refused_as_by_ctypes(noted):
    for i, (field, _) in enumerate(binding._Adam._fields_):
        for x in HYPER:
            values = [0.5] * 5
            values[i] = x
            want = outcome(lambda: repr([getattr(binding._Adam(*values), f) for f, _ in binding._Adam._fields_]))
            got = outcome(lambda: repr(noted("adam_step", 1, binding.AdamHyper(*values), 1, None)[1][1][1]))
            assert got == want, (field, x, want, got)


def test_a_plan_calls_the_library_that_made_it(monkeypatch, tmp_path):
    """Also once another library has been loaded: each of the two keeps its own last error."""
    first = binding.load_library()
    layout = dict(tensor_numel=[5000], bucket_seg_off=[0, 1], seg_tensor=[0], seg_begin=[0], seg_len=[5000])
    with binding.Plan(**layout, device=-1) as plan:
        monkeypatch.setattr(binding, "_lib", None)
        monkeypatch.setenv("BCA_LIB", str(shutil.copy(binding.library_path(), tmp_path / "other.so")))
        second = binding.load_library()
        assert second is not first
        assert first.bca_plan_set_decay_mask(None, None) != 0       # its last error is this one now
        assert second.bca_last_error() == b""
        before = first.bca_last_error()
        for call in (lambda: plan.adam_step(binding.AdamHyper(), 1), lambda: plan.bucket_clip(0, 1, 64, 64, 64, 64)):
            with pytest.raises(binding.BcaError):
                call()
            assert first.bca_last_error() != before and second.bca_last_error() == b""
