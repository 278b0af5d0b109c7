"""Shared test plumbing: runs one packed call through the oracle or through the HIP library, and the error
measure of the tolerance."""
from __future__ import annotations

import numpy as np

from paper_2605_05219_amd.device_call import GpuCall, run_call_gpu, to_device  # noqa: F401  (re-exported)


def max_norm_err(x, ref) -> float:
    """max |x - ref| / max |ref| over one tensor (the tolerance's 'max rel err')."""
    x = np.asarray(x, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    if ref.size == 0:
        return 0.0
    den = np.abs(ref).max()
    return float(np.abs(x - ref).max() / (den if den > 0 else 1.0))


QUIET = 2.0 ** -14     # a head quieter than this fraction of the tensor's loudest value is measured against that floor


def worst_head_err(o, o_ref, cu_seqlens):
    """The largest max-normalised error over the tensors the tolerance is stated for: all outputs of one
    (request, layer, value head).  o, o_ref: [L][T][H_v][d_v].  Returns (error, (request, layer, head)).

    The denominator is the head's own max |ref|, but not less than QUIET times the max |ref| of everything passed in: the
    matrix-core operands are fp16 (smallest normal 2^-14), so values that far below the data's scale are below the
    arithmetic's resolution whatever the head they sit in (a head whose state a gate of 1e-30 has just wiped is the case)."""
    o = np.asarray(o, dtype=np.float64)
    o_ref = np.asarray(o_ref, dtype=np.float64)
    floor = QUIET * (float(np.abs(o_ref).max()) if o_ref.size else 0.0)
    worst, where = 0.0, None
    for r in range(len(cu_seqlens) - 1):
        lo, hi = int(cu_seqlens[r]), int(cu_seqlens[r + 1])
        if hi <= lo:
            continue
        diff = np.abs(o[:, lo:hi] - o_ref[:, lo:hi]).max(axis=(1, 3))      # [L][H_v]
        den = np.maximum(np.abs(o_ref[:, lo:hi]).max(axis=(1, 3)), floor)
        e = diff / np.where(den > 0, den, 1.0)
        i = np.unravel_index(int(np.argmax(e)), e.shape)
        if e[i] > worst:
            worst, where = float(e[i]), (r, int(i[0]), int(i[1]))
    return worst, where


def worst_state_err(state, state_ref):
    """The same per value head of one emitted state [L][H_v][d_v][d_k] (floor: QUIET times the state's loudest value)."""
    s = np.asarray(state, dtype=np.float64)
    ref = np.asarray(state_ref, dtype=np.float64)
    diff = np.abs(s - ref).max(axis=(2, 3))
    den = np.maximum(np.abs(ref).max(axis=(2, 3)), QUIET * float(np.abs(ref).max()))
    return float((diff / np.where(den > 0, den, 1.0)).max())


def call_path(call, o_dtype="f32"):
    """The kernels the library runs this call on, with the workspace it asks for (gdn_resume_path)."""
    from paper_2605_05219_amd import binding as B
    shape = B.make_shape(call.L, call.H_qk, call.H_v, call.d_k, call.d_v, call.dtype, o_dtype, call.total_tokens)
    ws = B.gdn_workspace_bytes(shape, call.n_req, call.total_tokens, int(call.emit_pos.size))
    return B.gdn_resume_path(shape, call.cu_seqlens, call.start_pos, call.emit_cu, call.emit_pos, ws)


def run_call_counted(call, pool, o_dtype="f32"):
    """run_call_gpu, and the launches of preparation and of recurrence (or fused) kernels that it took."""
    from paper_2605_05219_amd import binding as B
    B.gdn_profile_enable(True)
    try:
        out = run_call_gpu(call, pool, o_dtype)
        return out + tuple(B.gdn_profile_collect()[3:5])
    finally:
        B.gdn_profile_enable(False)


def run_call_oracle(call, pool):
    from oracle import gdn_oracle as orc
    s = call.streams
    return orc.resume_prefill(s.q, s.k, s.v, s.beta, s.gate, call.cu_seqlens, call.start_pos, call.src_slot,
                              call.emit_cu, call.emit_pos, state_src=pool)
