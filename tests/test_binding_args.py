"""The binding's native way of a call (csrc/py_args.cpp) hands the C entry points what the Python way hands them, and
leaves every other call to it.  Nothing is launched: the entry points are replaced by recorders."""
import ctypes
import os
import subprocess
import sys
import types

import numpy as np
import pytest
import torch

from paper_2511_05589_amd import binding, build

F32, BF16, I32, I64, U8 = torch.float32, torch.bfloat16, torch.int32, torch.int64, torch.uint8


def cases(dev):
    """entry point -> (function, positional arguments, keyword arguments), every extent different"""
    n = lambda dtype, *shape: torch.zeros(shape, dtype=dtype, device=dev)  # noqa: E731
    f = lambda k: [n(F32, 100) for _ in range(k)]  # noqa: E731
    cu = n(I32, 8)
    attn = dict(scale=0.125, dtype=binding.COPRIS_BF16)
    clip = dict(eps_low=0.2, eps_high=0.28)
    cache = [n(BF16, 11, 3, 16, 64), n(BF16, 11, 3, 16, 64)]
    f32cache = [t.float() for t in cache]
    return {
        "copris_rollout_apply": (binding.rollout_apply, [n(I32, 40), 2, 5, n(I64, 6), n(I32, 6), n(I32, 6), n(I32, 6, 9)], {}),
        "copris_kv_append": (binding.kv_append, [n(BF16, 6, 3, 64), n(BF16, 6, 3, 64), n(I32, 6, 9), n(I32, 6)] + cache,
                             dict(dtype=binding.COPRIS_BF16)),
        "copris_traj_append": (binding.traj_append, [n(I32, 6), n(F32, 6), n(I64, 6), n(I32, 6), n(I32, 6), 4,
                                                     n(I32, 20, 30), n(F32, 20, 30), n(I32, 20, 30)], {}),
        "copris_traj_gather": (binding.traj_gather, [n(I32, 20, 30), n(F32, 20, 30), n(I32, 20, 30), n(I32, 7), cu, 4,
                                                     n(I32, 99), n(F32, 99), n(F32, 99), n(I32, 7)], {}),
        "copris_decode_attn": (binding.decode_attn, [n(BF16, 6, 12, 64)] + cache + [n(I32, 6, 9), n(I32, 6), n(BF16, 6, 12, 64),
                                                                                   n(F32, 6, 12), n(U8, 512)], attn),
        "copris_prefill_attn": (binding.prefill_attn, [n(F32, 50, 12, 64), n(F32, 50, 3, 64), n(F32, 50, 3, 64), cu, n(I32, 7, 9)]
                                + f32cache + [n(F32, 50, 12, 64), None],
                                dict(max_seqlen=33, scale=0.125, dtype=binding.COPRIS_F32)),
        "copris_lmhead_logprob": (binding.lmhead_logprob, [n(BF16, 6, 64), n(BF16, 500, 64), n(I64, 6), n(I32, 6), n(I32, 6),
                                                           n(F32, 6), None, n(U8, 512)],
                                  dict(seed=-3, temperature=0.7, dtype=binding.COPRIS_BF16)),
        "copris_lmhead_token_logprob": (binding.lmhead_token_logprob, [n(F32, 6, 64), n(F32, 500, 64), n(I32, 6), n(F32, 6),
                                                                       n(F32, 6), n(U8, 512)],
                                        dict(temperature=0.7, dtype=binding.COPRIS_F32)),
        "copris_is_ratio": (binding.is_ratio, f(3) + [cu, n(I32, 7), n(U8, 100)] + f(3) + [n(I32, 7), n(I32, 7)], clip),
        "copris_grpo_surrogate": (binding.grpo_surrogate, f(3) + [cu, n(I32, 7), None, n(F32, 7)] + f(3) + [n(I32, 7), n(F32, 1)],
                                  clip),
    }


NAMES = sorted(cases("cpu"))


@pytest.fixture
def recorded(monkeypatch):
    """calls(native) -> the list of recorded calls of the next calls, taken by the native way or by Python's"""
    lib = binding.load_library()
    native, log = binding._args, []
    fake = types.SimpleNamespace()
    for name, (res, argtypes) in binding.SIGNATURES.items():
        if name in native.entry_points:
            record = lambda *a, name=name: log.append((name, a)) or 0  # noqa: E731
            setattr(fake, name, ctypes.CFUNCTYPE(res, *argtypes)(record))
    addresses = lambda l: tuple(ctypes.cast(getattr(l, n), ctypes.c_void_p).value for n in native.entry_points)  # noqa: E731
    monkeypatch.setattr(binding, "_lib", fake)

    def calls(by_native):
        binding._args = native if by_native else None
        log.clear()
        return log

    native.bind(addresses(fake), binding._current_stream())
    yield calls
    native.bind(addresses(lib), binding._current_stream())
    binding._args = native


def test_entry_points():
    binding.load_library()
    assert sorted(binding._args.entry_points) == NAMES and set(NAMES) <= set(binding.SIGNATURES)
    with pytest.raises(ValueError):
        binding._args.bind((1,), None)
    with pytest.raises(ValueError):
        binding._args.bind((0,) * len(NAMES), None)


@pytest.mark.parametrize("name", NAMES)
def test_host_tensors_are_left_to_python(name):
    fn, pos, kw = cases("cpu")[name]
    binding.load_library()
    assert getattr(binding._args, fn.__name__)(*pos, *kw.values(), None) is None
    with pytest.raises(TypeError, match="must be a GPU tensor"):
        fn(*pos, **kw)


# a process in which the module is MODULE (None: it cannot be imported): the library, the manager and the checks work
WITHOUT = """
import sys, types, warnings
sys.modules["paper_2511_05589_amd._args"] = MODULE
from paper_2511_05589_amd import binding
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    binding.load_library()
    binding.load_library()
assert [w.category for w in seen] == [RuntimeWarning] and "ctypes" in str(seen[0].message), seen
assert binding._args is None and binding.version()
from tests import test_binding_args as t
for fn, pos, kw in t.cases("cpu").values():
    try:
        fn(*pos, **kw)
    except TypeError as e:
        assert "must be a GPU tensor" in str(e)
    else:
        raise AssertionError(fn)
"""


@pytest.mark.parametrize("module", ["None", "types.SimpleNamespace(built_for='another version')"])
def test_every_call_goes_the_python_way_without_the_module(module):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    done = subprocess.run([sys.executable, "-c", WITHOUT.replace("MODULE", module)], cwd=root, capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stderr


def test_build_makes_the_module_beside_every_library_and_does_without_it(monkeypatch, tmp_path, capsys):
    ran, old = [], tmp_path / "_args.so"
    compiles = lambda cmd: any(str(c).endswith("py_args.cpp") for c in cmd)  # noqa: E731
    monkeypatch.setattr(build, "ARGS_PATH", str(old))
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: ran.append(cmd))
    other = str(tmp_path / "other.so")
    assert build.build(lib_path=other) == other
    assert sum(compiles(c) for c in ran) == 1

    def no_headers(cmd, verbose):
        if compiles(cmd):
            raise RuntimeError("g++ failed:\nPython.h: No such file or directory")
    monkeypatch.setattr(build, "_run", no_headers)
    old.write_bytes(b"of an older build")
    assert build.build(lib_path=other) == other
    assert not old.exists() and "Python.h" in capsys.readouterr().err


# the module taking host tensors, and an entry point that is under way while the interpreter ends: the thread in it is a
# daemon's, which Python ends where it asks for the interpreter's lock again
SLOW_ENTRY = """
#include <unistd.h>
extern "C" __attribute__((visibility("default"))) int slow_entry(...) { usleep(400000); return 0; }
"""
ENDING = """
import ctypes, importlib.machinery, importlib.util, sys, threading, time, torch
from tests import test_binding_args as t
path = sys.argv[1]
loader = importlib.machinery.ExtensionFileLoader("_args", path)
args = importlib.util.module_from_spec(importlib.util.spec_from_loader("_args", loader))
loader.exec_module(args)
slow = ctypes.cast(ctypes.CDLL(path).slow_entry, ctypes.c_void_p).value
stream = lambda device: time.sleep(WAIT) or 0
args.bind((slow,) * len(args.entry_points), stream)
_, pos, kw = t.cases("cpu")["copris_kv_append"]
assert args.kv_append(*pos, *kw.values(), None) == 0

class Late:                      # goes when the interpreter is ending, and gives up the lock meanwhile
    def __del__(self, sleep=time.sleep):
        sleep(1)

sys.late = Late()
threading.Thread(target=args.kv_append, args=(*pos, *kw.values(), None), daemon=True).start()
time.sleep(0.1)
"""


@pytest.fixture(scope="module")
def host_module(tmp_path_factory):
    with open(os.path.join(build.CSRC, "py_args.cpp")) as f:
        source = f.read()
    assert source.count("t.is_cuda()") == 1
    at = tmp_path_factory.mktemp("args")
    copy, module = str(at / "py_args.cpp"), str(at / "_args.so")
    with open(copy, "w") as f:
        f.write(source.replace("t.is_cuda()", "t.is_cpu()") + SLOW_ENTRY)
    swap = {os.path.join(build.CSRC, "py_args.cpp"): copy, build.ARGS_PATH: module, "-O2": "-O1"}
    subprocess.run([swap.get(c, c) for c in build.args_command()], check=True, capture_output=True)
    return module


@pytest.mark.parametrize("wait", [0, 0.4])   # in the entry point; in the look-up of the stream before it
def test_a_thread_inside_a_call_when_the_interpreter_ends(host_module, wait):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    done = subprocess.run([sys.executable, "-c", ENDING.replace("WAIT", str(wait)), host_module], cwd=root, capture_output=True, text=True,
                          timeout=120)
    assert done.returncode == 0, (done.returncode, done.stderr)


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_same_arguments_by_both_ways(name, recorded):
    fn, pos, kw = cases("cuda")[name]

    def both(pos, kw, native):
        """What both ways do with a call, which has to be the same; native: which way takes it (None: either)."""
        out = []
        for by_native in (False, True):
            log = recorded(by_native)
            try:
                fn(*pos, **kw)
            except Exception as e:
                log.append((type(e), str(e)))
            out.append(list(log))
        assert len(out[0]) == 1 and out[0] == out[1]
        direct = getattr(binding._args, fn.__name__)(*pos, *kw.values(), *([] if "stream" in kw else [None]))
        if native is None:
            native = direct == 0
        assert direct == (0 if native else None) and not (native and isinstance(out[0][0][0], type))
        return out[0][0]

    assert both(pos, kw, True)[0] == name
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert both(pos, kw, True)[1][-1] == side.cuda_stream
    assert both(pos, {**kw, "stream": side}, False)[1][-1] == side.cuda_stream
    for i, t in enumerate(pos):
        if not isinstance(t, torch.Tensor):
            continue
        wide = torch.stack((t, t), dim=-1)[..., 0]            # the same extents, not contiguous unless it is one element
        for other in (t.cpu(), t.tolist(), t.t() if t.dim() == 2 else wide):
            both(pos[:i] + [other] + pos[i + 1:], kw, other.is_contiguous() and other.is_cuda if other is wide else False)
        for other in (t.to(torch.float64), None, t[None], t.flatten()):
            both(pos[:i] + [other] + pos[i + 1:], kw, None)
    for k, x in kw.items():                                   # numbers of other types go the Python way
        both(pos, {**kw, k: np.float32(x) if isinstance(x, float) else np.int64(x)}, False)
