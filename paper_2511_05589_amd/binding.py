"""Thin binding of libcopris.so: argument marshalling only (a good call natively, every other through ctypes).

Every step of the path runs in the library's HIP kernels.  PyTorch is used for
device memory and stream handles, nothing else.  There is no CPU fallback: if
the shared library is missing the import of a symbol fails loudly.
"""
from __future__ import annotations

import ctypes
import os
import warnings
from ctypes import c_char_p, c_float, c_int, c_int64, c_size_t, c_uint64, c_void_p
from typing import Optional

_PKG_DIR = os.path.dirname(os.path.abspath(__file__))
# COPRIS_LIB selects another build of the library (e.g. one with host sanitizers)
LIB_PATH = os.environ.get("COPRIS_LIB") or os.path.join(_PKG_DIR, "libcopris.so")

COPRIS_OK = 0
COPRIS_EINVAL = -1
COPRIS_EWORKSPACE = -2
COPRIS_EUNSUPPORTED = -3
COPRIS_ELAUNCH = -4
COPRIS_F32 = 0
COPRIS_BF16 = 1

# name -> (restype, argtypes), mirroring include/copris.h
SIGNATURES = {
    "copris_strerror": (c_char_p, [c_int]),
    "copris_version": (c_char_p, []),
    "copris_last_error_detail": (c_char_p, []),
    "copris_set_launch_hook": (None, [c_void_p, c_void_p]),
    "copris_decode_attn_workspace_bytes": (c_size_t, [c_int] * 6),
    "copris_decode_attn": (c_int, [c_void_p] * 8 + [c_size_t] + [c_int] * 6 + [c_int64, c_float, c_int, c_void_p]),
    "copris_prefill_attn": (c_int, [c_void_p] * 9 + [c_int, c_int64] + [c_int] * 5 + [c_int64, c_int, c_float,
                                                                                     c_int, c_void_p]),
    "copris_lmhead_logprob_workspace_bytes": (c_size_t, [c_int] * 3),
    "copris_lmhead_logprob": (c_int, [c_void_p] * 4 + [c_uint64, c_float] + [c_void_p] * 4
                              + [c_size_t] + [c_int] * 4 + [c_void_p]),
    "copris_lmhead_logprob_noalloc_max_bytes": (c_size_t, []),
    "copris_lmhead_logprob_noalloc": (c_int, [c_void_p] * 4 + [c_uint64, c_float] + [c_void_p] * 3
                                      + [c_int] * 4 + [c_void_p]),
    "copris_lmhead_token_logprob_workspace_bytes": (c_size_t, [c_int] * 4),
    "copris_lmhead_token_logprob": (c_int, [c_void_p] * 3 + [c_float] + [c_void_p] * 3 + [c_size_t]
                                    + [c_int] * 4 + [c_void_p]),
    "copris_is_ratio": (c_int, [c_void_p] * 6 + [c_float, c_float] + [c_void_p] * 5
                        + [c_int, c_int64, c_void_p]),
    "copris_grpo_surrogate": (c_int, [c_void_p] * 7 + [c_float, c_float] + [c_void_p] * 5
                              + [c_int, c_int64, c_void_p]),
}



class StageStats(ctypes.Structure):
    """copris_stage_stats of include/copris.h."""
    _fields_ = [(n, c_int64) for n in (
        "steps", "generated", "slot_steps_idle", "batch_tokens", "batch_offpolicy",
        "batch_traj_offpolicy", "max_staleness", "resumed", "reprefill_tokens", "paused",
        "buffered_complete", "peak_pages")]


SIGNATURES["copris_rollout_schedule"] = (c_int, [c_void_p, c_void_p] + [c_int] * 6 + [c_void_p] * 3)


class RolloutPlan(ctypes.Structure):
    """copris_rollout_plan of include/copris.h."""
    _fields_ = [(n, ctypes.c_int32) for n in ("stage", "n_active", "n_entered", "n_finishing", "n_slot_cmds",
                                              "n_page_cmds")] + [
        (n, ctypes.POINTER(ctypes.c_int32)) for n in ("slot_traj", "entered", "finishing", "cmds", "block_table")]


ROLLOUT_STEP, ROLLOUT_STAGE_END, ROLLOUT_EXHAUSTED = 0, 1, 2
SIGNATURES.update({
    "copris_rollout_create": (c_int, [c_void_p, c_void_p] + [c_int] * 5 + [c_int64, c_void_p, c_void_p]),
    "copris_rollout_destroy": (None, [c_void_p]),
    "copris_rollout_max_pages": (c_int, [c_void_p]),
    "copris_rollout_free_pages": (c_int64, [c_void_p]),
    "copris_rollout_begin_stage": (c_int, [c_void_p]),
    "copris_rollout_next_step": (c_int, [c_void_p, c_void_p]),
    "copris_rollout_stop": (c_int, [c_void_p, c_void_p, c_int]),
    "copris_rollout_end_stage": (c_int, [c_void_p] * 4),
    "copris_rollout_apply": (c_int, [c_void_p, c_int, c_int] + [c_void_p] * 4 + [c_int, c_int, c_void_p]),
    "copris_kv_append": (c_int, [c_void_p] * 6 + [c_int] * 5 + [c_int64, c_int, c_void_p]),
    "copris_traj_append": (c_int, [c_void_p] * 5 + [c_int] + [c_void_p] * 3 + [c_int, c_int64, c_int, c_void_p]),
    "copris_traj_gather": (c_int, [c_void_p] * 5 + [c_int] + [c_void_p] * 4 + [c_int, c_int64, c_int, c_void_p]),
})

_lib = None
_raw_stream = None
# The native way of a good call (csrc/py_args.cpp), bound to _lib's entry points: it returns the call's code, or None
# where the arguments are for the Python checks to look at.  None until the library is loaded, and where the module is
# not there or not of this PyTorch: every call then goes the Python way.
_args = None


class CoprisError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        detail = load_library().copris_last_error_detail().decode() if code in (COPRIS_ELAUNCH, COPRIS_EWORKSPACE) else ""
        super().__init__(f"{where}: {strerror(code)} (code {code}) {detail}".rstrip())


def load_library(path: Optional[str] = None) -> ctypes.CDLL:
    """Load libcopris.so (built in-tree by paper_2511_05589_amd.build) and type its symbols."""
    global _lib, _args
    if _lib is not None and path is None:
        return _lib
    path = path or LIB_PATH
    if not os.path.exists(path):
        raise FileNotFoundError(
            f"{path} not found: build it with `python -m paper_2511_05589_amd.build` "
            "(there is no fallback path)")
    # PyTorch ships its own HIP runtime (same soname as the system one).  Import it
    # first so that the loader binds libcopris to that already-loaded copy: two HIP
    # runtimes in one process cannot share streams or device memory.
    import torch  # noqa: F401
    lib = ctypes.CDLL(path)
    for name, (res, args) in SIGNATURES.items():
        fn = getattr(lib, name)          # AttributeError if the symbol is not exported
        fn.restype = res
        fn.argtypes = args
    native = _native_args()
    if native is not None:
        native.bind(tuple(ctypes.cast(getattr(lib, name), c_void_p).value for name in native.entry_points),
                    _current_stream())
    _lib, _args = lib, native
    return lib


def _native_args():
    import torch
    try:
        from . import _args as native
        if native.built_for == torch.__version__:
            return native
        why = f"it was built for PyTorch {native.built_for}, this is {torch.__version__}"
    except ImportError as e:
        why = str(e)
    warnings.warn(f"the binding's argument module (_args.so) cannot be used, calls are marshalled by ctypes: {why}; build it "
                  "with `python -m paper_2511_05589_amd.build`", RuntimeWarning, stacklevel=3)
    return None


def _current_stream():
    """device index -> raw handle of torch's current stream"""
    global _raw_stream
    if _raw_stream is None:
        import torch
        # the handle alone: a torch.cuda.Stream object per call costs 2 us
        _raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None) or (
            lambda i: torch.cuda.current_stream(i).cuda_stream)
    return _raw_stream


def strerror(code: int) -> str:
    return load_library().copris_strerror(int(code)).decode()


def version() -> str:
    return load_library().copris_version().decode()


LAUNCH_HOOK = ctypes.CFUNCTYPE(None, c_char_p, c_int, c_void_p, c_void_p)
_hook_ref = None


def set_launch_hook(fn) -> None:
    """fn(kernel: bytes, phase: int, stream: int|None, user) or None to remove the hook."""
    global _hook_ref
    lib = load_library()
    if fn is None:
        lib.copris_set_launch_hook(None, None)
        _hook_ref = None
        return
    _hook_ref = LAUNCH_HOOK(fn)           # keep the trampoline alive
    lib.copris_set_launch_hook(ctypes.cast(_hook_ref, c_void_p), None)


_torch_dtypes = {}   # name -> torch dtype; filled on first use (torch is not imported with this module)


def _dtype(name: str):
    d = _torch_dtypes.get(name)
    if d is None:
        import torch
        d = _torch_dtypes[name] = getattr(torch, name)
    return d


def _arg(t, dtype: Optional[str], name: str, optional: bool = False) -> Optional[int]:
    """The device address of a tensor argument, after the host-side checks it must pass before it
    crosses the C ABI: on the GPU, contiguous, of the expected torch dtype (a name such as "int32";
    None = any).  A call whose arguments are all in order does not come here (_args)."""
    if t is None:
        if optional:
            return None
        raise TypeError(f"{name}: a device tensor is required")
    if t.is_cuda and t.is_contiguous() and (dtype is None or t.dtype == _dtype(dtype)):
        return t.data_ptr()
    if not t.is_cuda:
        raise TypeError(f"{name}: must be a GPU tensor, got device {t.device}")
    if not t.is_contiguous():
        raise TypeError(f"{name}: must be contiguous")
    raise TypeError(f"{name}: expected torch.{dtype}, got {t.dtype}")


def _elem(dtype_code: int) -> str:
    return {COPRIS_F32: "float32", COPRIS_BF16: "bfloat16"}.get(int(dtype_code))


def _stream(stream, ref) -> Optional[int]:
    """The raw stream handle (None = the null stream); `ref` is a tensor argument of the call,
    which must live on the stream's device."""
    if stream is None:
        return _current_stream()(ref.get_device()) or None
    if stream.device != ref.device:
        raise TypeError(f"stream on {stream.device} but tensors on {ref.device}")
    return stream.cuda_stream or None


def _check(code: int, where: str) -> None:
    if code != COPRIS_OK:
        raise CoprisError(code, where)


def decode_attn_workspace_bytes(C, Hq, Hkv, D, page_size, max_pages) -> int:
    return int(load_library().copris_decode_attn_workspace_bytes(C, Hq, Hkv, D, page_size, max_pages))


def decode_attn(q, k_cache, v_cache, block_table, ctx_len, out, lse, workspace, *, scale: float,
                dtype: int, stream=None) -> None:
    """copris_decode_attn on device tensors (shapes as in include/copris.h)."""
    code = _args and _args.decode_attn(q, k_cache, v_cache, block_table, ctx_len, out, lse, workspace, scale, dtype,
                                       stream)
    if code is None:
        e = _elem(dtype)
        ptrs = (_arg(q, e, "q"), _arg(k_cache, e, "k_cache"), _arg(v_cache, e, "v_cache"))
        out_ = _arg(out, e, "out")
        ptrs += (_arg(block_table, "int32", "block_table"), _arg(ctx_len, "int32", "ctx_len"), out_,
                 _arg(lse, "float32", "lse", optional=True), _arg(workspace, "uint8", "workspace"))
        C, Hq, D = q.shape
        num_pages, Hkv, page_size, _ = k_cache.shape
        max_pages = block_table.shape[1]
        code = load_library().copris_decode_attn(
            *ptrs, workspace.numel(), C, Hq, Hkv, D, page_size, max_pages, num_pages, float(scale), int(dtype),
            _stream(stream, q))
    _check(code, "copris_decode_attn")


def lmhead_logprob_workspace_bytes(C, H, V) -> int:
    return int(load_library().copris_lmhead_logprob_workspace_bytes(C, H, V))


def lmhead_logprob(hidden, weight, seq_id, step, token, logprob, lse, workspace, *, seed: int,
                   temperature: float, dtype: int, stream=None) -> None:
    """copris_lmhead_logprob on device tensors."""
    code = _args and _args.lmhead_logprob(hidden, weight, seq_id, step, token, logprob, lse, workspace, seed,
                                          temperature, dtype, stream)
    if code is None:
        e = _elem(dtype)
        ins = (_arg(hidden, e, "hidden"), _arg(weight, e, "weight"), _arg(seq_id, "int64", "seq_id"),
               _arg(step, "int32", "step"))
        outs = (_arg(token, "int32", "token"), _arg(logprob, "float32", "logprob"),
                _arg(lse, "float32", "lse", optional=True), _arg(workspace, "uint8", "workspace"))
        C, H = hidden.shape
        V = weight.shape[0]
        code = load_library().copris_lmhead_logprob(
            *ins, int(seed) & 0xFFFFFFFFFFFFFFFF, float(temperature), *outs, workspace.numel(), C, H, V, int(dtype),
            _stream(stream, hidden))
    _check(code, "copris_lmhead_logprob")


def lmhead_logprob_noalloc(hidden, weight, seq_id, step, token, logprob, lse, *, seed: int,
                           temperature: float, dtype: int, stream=None) -> None:
    """copris_lmhead_logprob_noalloc on device tensors (partials in the library's static array)."""
    e = _elem(dtype)
    ins = (_arg(hidden, e, "hidden"), _arg(weight, e, "weight"), _arg(seq_id, "int64", "seq_id"),
           _arg(step, "int32", "step"))
    outs = (_arg(token, "int32", "token"), _arg(logprob, "float32", "logprob"),
            _arg(lse, "float32", "lse", optional=True))
    C, H = hidden.shape
    V = weight.shape[0]
    code = load_library().copris_lmhead_logprob_noalloc(
        *ins, int(seed) & 0xFFFFFFFFFFFFFFFF, float(temperature), *outs, C, H, V, int(dtype), _stream(stream, hidden))
    _check(code, "copris_lmhead_logprob_noalloc")


def is_ratio(logp_cur, logp_buf, logp_roll, cu_seqlens, split, mask, ratio, ratio_clipped,
             seq_sum, seq_cnt, seq_nclip, *, eps_low: float, eps_high: float, stream=None) -> None:
    """copris_is_ratio on device tensors."""
    code = _args and _args.is_ratio(logp_cur, logp_buf, logp_roll, cu_seqlens, split, mask, ratio, ratio_clipped,
                                    seq_sum, seq_cnt, seq_nclip, eps_low, eps_high, stream)
    if code is None:
        f32, i32 = "float32", "int32"
        cur, buf, roll = _arg(logp_cur, f32, "logp_cur"), _arg(logp_buf, f32, "logp_buf"), _arg(logp_roll, f32, "logp_roll")
        r, rc, ssum = _arg(ratio, f32, "ratio"), _arg(ratio_clipped, f32, "ratio_clipped"), _arg(seq_sum, f32, "seq_sum")
        cu, sp = _arg(cu_seqlens, i32, "cu_seqlens"), _arg(split, i32, "split")
        cnt, nclip = _arg(seq_cnt, i32, "seq_cnt"), _arg(seq_nclip, i32, "seq_nclip")
        m = _arg(mask, "uint8", "mask", optional=True)
        B = cu_seqlens.numel() - 1
        N = logp_cur.numel()
        code = load_library().copris_is_ratio(
            cur, buf, roll, cu, sp, m, float(eps_low), float(eps_high), r, rc, ssum, cnt, nclip, B, N,
            _stream(stream, cu_seqlens))
    _check(code, "copris_is_ratio")


def grpo_surrogate(logp_cur, logp_buf, logp_roll, cu_seqlens, split, mask, adv, surr, grad, seq_surr,
                   seq_cnt, objective, *, eps_low: float, eps_high: float, stream=None) -> None:
    """copris_grpo_surrogate on device tensors."""
    code = _args and _args.grpo_surrogate(logp_cur, logp_buf, logp_roll, cu_seqlens, split, mask, adv, surr, grad,
                                          seq_surr, seq_cnt, objective, eps_low, eps_high, stream)
    if code is None:
        f32, i32 = "float32", "int32"
        cur, buf, roll = _arg(logp_cur, f32, "logp_cur"), _arg(logp_buf, f32, "logp_buf"), _arg(logp_roll, f32, "logp_roll")
        a, sr, gr = _arg(adv, f32, "adv"), _arg(surr, f32, "surr"), _arg(grad, f32, "grad")
        ssurr, obj = _arg(seq_surr, f32, "seq_surr"), _arg(objective, f32, "objective")
        cu, sp, cnt = _arg(cu_seqlens, i32, "cu_seqlens"), _arg(split, i32, "split"), _arg(seq_cnt, i32, "seq_cnt")
        m = _arg(mask, "uint8", "mask", optional=True)
        B = cu_seqlens.numel() - 1
        N = logp_cur.numel()
        code = load_library().copris_grpo_surrogate(
            cur, buf, roll, cu, sp, m, a, float(eps_low), float(eps_high), sr, gr, ssurr, cnt, obj, B, N,
            _stream(stream, objective))
    _check(code, "copris_grpo_surrogate")


def lmhead_token_logprob_workspace_bytes(M, H, V, dtype) -> int:
    return int(load_library().copris_lmhead_token_logprob_workspace_bytes(M, H, V, int(dtype)))


def lmhead_token_logprob(hidden, weight, tokens, logprob, lse, workspace, *, temperature: float,
                         dtype: int, stream=None) -> None:
    """copris_lmhead_token_logprob on device tensors."""
    code = _args and _args.lmhead_token_logprob(hidden, weight, tokens, logprob, lse, workspace, temperature, dtype,
                                                stream)
    if code is None:
        e = _elem(dtype)
        ins = _arg(hidden, e, "hidden"), _arg(weight, e, "weight"), _arg(tokens, "int32", "tokens")
        outs = (_arg(logprob, "float32", "logprob"), _arg(lse, "float32", "lse", optional=True),
                _arg(workspace, "uint8", "workspace"))
        M, H = hidden.shape
        V = weight.shape[0]
        code = load_library().copris_lmhead_token_logprob(
            *ins, float(temperature), *outs, workspace.numel(), M, H, V, int(dtype), _stream(stream, hidden))
    _check(code, "copris_lmhead_token_logprob")


def prefill_attn(q, k, v, cu_seqlens, block_table, k_cache, v_cache, out, lse, *, max_seqlen: int,
                 scale: float, dtype: int, stream=None) -> None:
    """copris_prefill_attn on device tensors (shapes as in include/copris.h)."""
    code = _args and _args.prefill_attn(q, k, v, cu_seqlens, block_table, k_cache, v_cache, out, lse, max_seqlen,
                                        scale, dtype, stream)
    if code is None:
        e = _elem(dtype)
        q_, k_, v_ = _arg(q, e, "q"), _arg(k, e, "k"), _arg(v, e, "v")
        kc, vc, o = _arg(k_cache, e, "k_cache"), _arg(v_cache, e, "v_cache"), _arg(out, e, "out")
        cu, bt = _arg(cu_seqlens, "int32", "cu_seqlens"), _arg(block_table, "int32", "block_table")
        l = _arg(lse, "float32", "lse", optional=True)
        T, Hq, D = q.shape
        Hkv = k.shape[1]
        num_pages, _, page_size, _ = k_cache.shape
        B = cu_seqlens.numel() - 1
        code = load_library().copris_prefill_attn(
            q_, k_, v_, cu, bt, kc, vc, o, l, B, T, Hq, Hkv, D, page_size, block_table.shape[1], num_pages,
            int(max_seqlen), float(scale), int(dtype), _stream(stream, q))
    _check(code, "copris_prefill_attn")


def rollout_schedule(prompt_len, resp_len, pool: int, batch_inputs: int, page_size: int = 16,
                     max_stages: Optional[int] = None) -> list:
    """copris_rollout_schedule on host arrays (numpy); returns a list of per-stage dicts."""
    import numpy as np
    p = np.ascontiguousarray(prompt_len, dtype=np.int32)
    r = np.ascontiguousarray(resp_len, dtype=np.int32)
    n_inputs = int(p.size)
    samples = int(r.shape[1]) if r.ndim == 2 and n_inputs else 1
    if max_stages is None:
        max_stages = n_inputs // max(int(batch_inputs), 1) + 1
    stats = (StageStats * max(max_stages, 1))()
    batch = np.zeros((max(max_stages, 1), max(int(batch_inputs), 1)), dtype=np.int32)
    n = c_int(0)
    code = load_library().copris_rollout_schedule(
        p.ctypes.data, r.ctypes.data, n_inputs, samples, int(pool), int(batch_inputs), int(page_size),
        int(max_stages), ctypes.addressof(stats), batch.ctypes.data, ctypes.addressof(n))
    _check(code, "copris_rollout_schedule")
    out = []
    for k in range(n.value):
        d = {name: int(getattr(stats[k], name)) for name, _ in StageStats._fields_}
        d["batch_inputs"] = batch[k].tolist()
        out.append(d)
    return out


class RolloutManager:
    """The stepwise rollout manager (copris_rollout_* of include/copris.h) on host arrays."""

    def __init__(self, prompt_len, resp_len, pool: int, batch_inputs: int, page_size: int = 16,
                 num_pages: Optional[int] = None, page_order=None):
        import numpy as np
        p = np.ascontiguousarray(prompt_len, dtype=np.int32)
        r = np.ascontiguousarray(resp_len, dtype=np.int32)
        self.n_inputs, self.samples = int(r.shape[0]), int(r.shape[1])
        self.pool, self.batch_inputs, self.page_size = int(pool), int(batch_inputs), int(page_size)
        longest = int((p[:, None].astype(np.int64) + r).max()) if r.size else 1
        if num_pages is None:
            num_pages = self.pool * ((longest + self.page_size - 1) // self.page_size)
        order = None if page_order is None else np.ascontiguousarray(page_order, dtype=np.int32)
        h = c_void_p()
        code = load_library().copris_rollout_create(
            p.ctypes.data, r.ctypes.data, self.n_inputs, self.samples, self.pool, self.batch_inputs,
            self.page_size, int(num_pages), None if order is None else order.ctypes.data, ctypes.addressof(h))
        _check(code, "copris_rollout_create")
        self._h = h
        self.num_pages = int(num_pages)
        self.max_pages = int(load_library().copris_rollout_max_pages(h))

    def close(self) -> None:
        if self._h is not None:
            load_library().copris_rollout_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def free_pages(self) -> int:
        return int(load_library().copris_rollout_free_pages(self._h))

    def begin_stage(self) -> int:
        k = load_library().copris_rollout_begin_stage(self._h)
        if k < 0:
            raise CoprisError(k, "copris_rollout_begin_stage")
        return k

    def next_step(self, copy: bool = True):
        """Returns (code, plan): code is ROLLOUT_STEP / ROLLOUT_STAGE_END / ROLLOUT_EXHAUSTED; plan is a
        dict of the manager's arrays (None unless code is ROLLOUT_STEP): numpy copies, or with
        copy=False views of the manager's own memory that are valid until the next call."""
        import numpy as np
        plan = RolloutPlan()
        code = load_library().copris_rollout_next_step(self._h, ctypes.addressof(plan))
        if code < 0:
            raise CoprisError(code, "copris_rollout_next_step")
        if code != ROLLOUT_STEP:
            return code, None

        def arr(ptr, n):
            if not n:
                return np.zeros(0, np.int32)
            a = np.ctypeslib.as_array(ptr, shape=(n,))
            return a.copy() if copy else a
        return code, {
            "stage": plan.stage, "n_active": plan.n_active,
            "slot_traj": arr(plan.slot_traj, self.pool),
            "entered": arr(plan.entered, 4 * plan.n_entered).reshape(-1, 4),
            "finishing": arr(plan.finishing, plan.n_finishing),
            "n_slot_cmds": plan.n_slot_cmds, "n_page_cmds": plan.n_page_cmds,
            "cmds": arr(plan.cmds, 4 * plan.n_slot_cmds + 3 * plan.n_page_cmds),
            "block_table": arr(plan.block_table, self.pool * self.max_pages).reshape(self.pool, self.max_pages),
        }

    def stop(self, slots) -> None:
        import numpy as np
        s = np.ascontiguousarray(slots, dtype=np.int32)
        _check(load_library().copris_rollout_stop(self._h, s.ctypes.data, int(s.size)), "copris_rollout_stop")

    def end_stage(self) -> dict:
        """Stage statistics (the fields of copris_stage_stats), `batch_inputs` and `batch_traj`
        [B * samples, 3] = (trajectory, response tokens, tokens of earlier stages)."""
        import numpy as np
        stats = StageStats()
        binp = np.zeros(self.batch_inputs, dtype=np.int32)
        btr = np.zeros((self.batch_inputs * self.samples, 3), dtype=np.int32)
        code = load_library().copris_rollout_end_stage(self._h, ctypes.addressof(stats), binp.ctypes.data,
                                                       btr.ctypes.data)
        _check(code, "copris_rollout_end_stage")
        d = {name: int(getattr(stats, name)) for name, _ in StageStats._fields_}
        d["batch_inputs"] = binp.tolist()
        d["batch_traj"] = btr
        return d


def rollout_apply(cmds, n_slot_cmds: int, n_page_cmds: int, seq_id, ctx_len, step, block_table, *,
                  stream=None) -> None:
    """copris_rollout_apply on device tensors (cmds: the plan's commands, already on the device)."""
    code = _args and _args.rollout_apply(cmds, n_slot_cmds, n_page_cmds, seq_id, ctx_len, step, block_table, stream)
    if code is None:
        cm, sid = _arg(cmds, "int32", "cmds"), _arg(seq_id, "int64", "seq_id")
        state = _arg(ctx_len, "int32", "ctx_len"), _arg(step, "int32", "step"), _arg(block_table, "int32", "block_table")
        pool, max_pages = block_table.shape
        code = load_library().copris_rollout_apply(cm, int(n_slot_cmds), int(n_page_cmds), sid, *state, pool, max_pages,
                                                   _stream(stream, block_table))
    _check(code, "copris_rollout_apply")


def kv_append(k_new, v_new, block_table, ctx_len, k_cache, v_cache, *, dtype: int, stream=None) -> None:
    """copris_kv_append on device tensors."""
    code = _args and _args.kv_append(k_new, v_new, block_table, ctx_len, k_cache, v_cache, dtype, stream)
    if code is None:
        kn, vn = _arg(k_new, None, "k_new"), _arg(v_new, None, "v_new")
        kc, vc = _arg(k_cache, None, "k_cache"), _arg(v_cache, None, "v_cache")
        bt, ctx = _arg(block_table, "int32", "block_table"), _arg(ctx_len, "int32", "ctx_len")
        C, Hkv, D = k_new.shape
        num_pages, _, page_size, _ = k_cache.shape
        code = load_library().copris_kv_append(kn, vn, bt, ctx, kc, vc, C, Hkv, D, page_size, block_table.shape[1],
                                               num_pages, int(dtype), _stream(stream, k_cache))
    _check(code, "copris_kv_append")


def traj_append(token, logprob, seq_id, step, ctx_len, stage: int, buf_token, buf_logp, buf_tag, *,
                stream=None) -> None:
    """copris_traj_append on device tensors (buffers [n_traj, max_resp])."""
    code = _args and _args.traj_append(token, logprob, seq_id, step, ctx_len, stage, buf_token, buf_logp, buf_tag,
                                       stream)
    if code is None:
        state = (_arg(token, "int32", "token"), _arg(logprob, "float32", "logprob"), _arg(seq_id, "int64", "seq_id"),
                 _arg(step, "int32", "step"), _arg(ctx_len, "int32", "ctx_len"))
        bufs = (_arg(buf_token, "int32", "buf_token"), _arg(buf_logp, "float32", "buf_logp"),
                _arg(buf_tag, "int32", "buf_tag"))
        n_traj, max_resp = buf_token.shape
        code = load_library().copris_traj_append(*state, int(stage), *bufs, token.numel(), n_traj, max_resp,
                                                 _stream(stream, buf_token))
    _check(code, "copris_traj_append")


def traj_gather(buf_token, buf_logp, buf_tag, traj, cu_seqlens, stage: int, tokens_out, logp_buf_out,
                logp_roll_out, split_out, *, stream=None) -> None:
    """copris_traj_gather on device tensors."""
    code = _args and _args.traj_gather(buf_token, buf_logp, buf_tag, traj, cu_seqlens, stage, tokens_out,
                                       logp_buf_out, logp_roll_out, split_out, stream)
    if code is None:
        ins = (_arg(buf_token, "int32", "buf_token"), _arg(buf_logp, "float32", "buf_logp"),
               _arg(buf_tag, "int32", "buf_tag"), _arg(traj, "int32", "traj"), _arg(cu_seqlens, "int32", "cu_seqlens"))
        outs = (_arg(tokens_out, "int32", "tokens_out"), _arg(logp_buf_out, "float32", "logp_buf_out"),
                _arg(logp_roll_out, "float32", "logp_roll_out"), _arg(split_out, "int32", "split_out"))
        n_traj, max_resp = buf_token.shape
        code = load_library().copris_traj_gather(*ins, int(stage), *outs, traj.numel(), n_traj, max_resp,
                                                 _stream(stream, buf_token))
    _check(code, "copris_traj_gather")
