"""CPU tests of the library's host side: exported symbols, l(t;C), the chunk planner and
every argument check of the entry points (all of them fire before anything is enqueued)."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle import gdn_oracle as orc
from paper_2605_05219_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "gdn_resume.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(gdn_\w+|ckpt_\w+)\s*\(", header))
    assert declared == set(B.EXPORTS)
    L = ctypes.CDLL(B.LIB_PATH)
    for name in declared:
        assert getattr(L, name) is not None
    assert B.gdn_version() >= 100


def test_deepest_checkpoint_matches_brute_force():
    rng = np.random.default_rng(1)
    for _ in range(100):
        N = int(rng.integers(1, 80))
        M = int(rng.integers(0, min(N, 9) + 1))
        pos = sorted(rng.choice(np.arange(1, N + 1), size=M, replace=False).tolist())
        for t in range(0, N + 2):
            assert B.gdn_deepest_ckpt(pos, t) == orc.deepest_ckpt(pos, t)
    assert B.gdn_deepest_ckpt([128, 256, 384], 127) == -1
    assert B.gdn_deepest_ckpt([128, 256, 384], 128) == 0
    assert B.gdn_deepest_ckpt([], 7) == -1


def brute_plan(cu, start, ecu, epos):
    """Reference chunking written independently: walk positions one by one."""
    tok0, ln, em, rcu = [], [], [], [0]
    for r in range(len(start)):
        emits = {int(epos[e]): e for e in range(ecu[r], ecu[r + 1])}
        cur_start, cur_len = None, 0
        for i in range(cu[r + 1] - cu[r]):
            if cur_start is None:
                cur_start, cur_len = cu[r] + i, 0
            cur_len += 1
            pos = start[r] + i + 1
            if pos in emits or cur_len == B.GDN_CHUNK or i == cu[r + 1] - cu[r] - 1:
                tok0.append(cur_start); ln.append(cur_len); em.append(emits.get(pos, -1))
                cur_start = None
        rcu.append(len(tok0))
    return tok0, ln, em, rcu


def test_chunk_planner_matches_position_walk():
    rng = np.random.default_rng(2)
    for _ in range(60):
        n_req = int(rng.integers(1, 6))
        lens = rng.integers(0, 300, size=n_req)
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        start = rng.integers(0, 1000, size=n_req).astype(np.int32)
        epos, ecu = [], [0]
        for r in range(n_req):
            k = int(rng.integers(0, min(4, lens[r]) + 1))
            e = sorted(rng.choice(np.arange(1, lens[r] + 1), size=k, replace=False).tolist()) if k else []
            epos += [int(start[r] + x) for x in e]
            ecu.append(len(epos))
        got = B.gdn_plan_chunks(cu, start, ecu, epos)
        exp = brute_plan(cu, start, ecu, epos)
        for g, e in zip(got, exp):
            assert list(g) == list(e)


def test_chunk_planner_aligned_case():
    tok0, ln, em, rcu = B.gdn_plan_chunks([0, 256], [256], [0, 2], [384, 512])
    assert list(tok0) == [0, 64, 128, 192] and list(ln) == [64] * 4
    assert list(em) == [-1, 0, -1, 1] and list(rcu) == [0, 4]


@pytest.mark.parametrize("cu,start,ecu,epos,code", [
    ([1, 5], [0], [0, 0], [], -4),          # cu does not start at 0
    ([0, 5, 3], [0, 0], [0, 0, 0], [], -4), # decreasing
    ([0, 5], [-1], [0, 0], [], -10),        # negative start
    ([0, 5], [10], [0, 1], [10], -8),       # emit at the start position itself
    ([0, 5], [10], [0, 1], [16], -8),       # emit beyond the end
    ([0, 5], [10], [0, 2], [12, 12], -8),   # not strictly increasing
    ([0, 5], [10], [0, 2], [13, 12], -8),
    ([0, 5], [2**31 - 3], [0, 0], [], -10), # positions overflow int32
])
def test_chunk_planner_rejects(cu, start, ecu, epos, code):
    with pytest.raises(B.GdnError) as ei:
        B.gdn_plan_chunks(cu, start, ecu, epos, capacity=64)
    assert ei.value.code == code


def test_chunk_planner_capacity():
    with pytest.raises(B.GdnError) as ei:
        B.gdn_plan_chunks([0, 200], [0], [0, 0], [], capacity=3)
    assert ei.value.code == -9


def test_workspace_bytes_and_shape_checks():
    ok = B.make_shape(1, 16, 16, 128, 128, "bf16", "f32", 8192)
    n = B.gdn_workspace_bytes(ok, 1, 8192, 16)
    assert n > 0 and n % 256 == 0 or n > 0
    for bad in (B.make_shape(1, 3, 16, 128, 128, "bf16", "f32", 8),     # H_v % H_qk
                B.make_shape(1, 16, 16, 96, 96, "bf16", "f32", 8),      # head size
                B.make_shape(1, 16, 16, 64, 128, "bf16", "f32", 8),
                B.make_shape(0, 16, 16, 128, 128, "bf16", "f32", 8),
                B.make_shape(1, 2, 2, 128, 128, "f32", "f32", 8)):      # fp32 inputs: d = 64 only
        with pytest.raises(B.GdnError) as ei:
            B.gdn_workspace_bytes(bad, 1, 8, 0)
        assert ei.value.code == -3
    with pytest.raises(B.GdnError) as ei:
        B.gdn_workspace_bytes(ok, -1, 8, 0)
    assert ei.value.code == -11


class FakeDev:
    """Stands in for a device tensor: the checks under test return before any pointer is used."""

    def __init__(self, ptr=0x10000, n0=8, stride0=2 * 2 * 64 * 64, nbytes=1 << 30):
        self._ptr, self.shape, self._s0, self._n = ptr, (n0,), stride0, nbytes

    def data_ptr(self): return self._ptr
    def stride(self, i): return self._s0
    def dim(self): return 1
    def numel(self): return self._n
    def element_size(self): return 1
    def __getitem__(self, i): return self


def prefill_args(**over):
    shape = B.make_shape(1, 2, 2, 64, 64, "f32", "f32", 512)
    d = FakeDev()
    a = dict(shape=shape, q=d, k=d, v=d, beta=d, gate=d, cu_seqlens=[0, 256], start_pos=[256],
             state_src=d, src_slot=[1], emit_cu=[0, 2], emit_pos=[384, 512], state_dst=d,
             emit_slot=[3, 4], o=d, workspace=FakeDev(ptr=0x100000), stream=ctypes.c_void_p(0))
    a.update(over)
    return a


def call_prefill(monkeypatch, **over):
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    a = prefill_args(**over)
    B.gdn_resume_prefill(a["shape"], a["q"], a["k"], a["v"], a["beta"], a["gate"], a["cu_seqlens"],
                         a["start_pos"], a["state_src"], a["src_slot"], a["emit_cu"], a["emit_pos"],
                         a["state_dst"], a["emit_slot"], a["o"], a["workspace"], a["stream"])


@pytest.mark.parametrize("over,code", [
    (dict(src_slot=[8]), -5),                                   # source slot outside the pool
    (dict(src_slot=[-2]), -5),
    (dict(emit_slot=[3, 8]), -5),                               # destination outside the pool
    (dict(emit_slot=[3, -1]), -5),
    (dict(emit_slot=[3, 3]), -6),                               # duplicate destination
    (dict(cu_seqlens=[0, 100, 256], start_pos=[256, 0], src_slot=[1, 3], emit_cu=[0, 1, 2],
          emit_pos=[356, 156], emit_slot=[3, 4]), -7),          # request 0 writes request 1's source
    # the same hazard when the destination pool is a view of the source pool two slots further on (slots compared by address)
    (dict(cu_seqlens=[0, 100, 256], start_pos=[256, 0], src_slot=[1, 3], emit_cu=[0, 1, 2],
          emit_pos=[356, 156], emit_slot=[1, 4], state_dst=FakeDev(ptr=0x10000 + 2 * 4 * 2 * 2 * 64 * 64)), -7),
    # a destination that overlaps the writer's own source only partly (view shifted by half a slot)
    (dict(emit_slot=[0, 4], state_dst=FakeDev(ptr=0x10000 + 5 * 2 * 2 * 64 * 64)), -7),
    (dict(emit_pos=[384, 513]), -8),
    (dict(cu_seqlens=[0, 600], emit_pos=[384, 512]), -4),       # more tokens than T_alloc
    (dict(q=FakeDev(ptr=0)), -1),
    (dict(o=FakeDev(ptr=0x10004)), -2),
    (dict(state_src=FakeDev(ptr=0x10008)), -2),
    (dict(state_dst=FakeDev(stride0=2 * 64 * 64 - 4)), -3),      # slot stride smaller than a slot
    (dict(state_dst=FakeDev(stride0=2 * 64 * 64 + 2)), -2),      # slot stride not a multiple of 4 floats
    (dict(workspace=FakeDev(ptr=0x100010)), -9),                # not 256-byte aligned
    (dict(workspace=FakeDev(ptr=0x100000, nbytes=1024)), -9),   # too small
    (dict(state_src=FakeDev(ptr=0)), -1),
    (dict(state_src=None), -5),                                 # no source pool: slot 1 is out of range
])
def test_prefill_argument_errors(monkeypatch, over, code):
    with pytest.raises(B.GdnError) as ei:
        call_prefill(monkeypatch, **over)
    assert ei.value.code == code


def test_own_source_slot_may_be_a_destination(monkeypatch):
    """A request may overwrite the slot it started from; the hazard is only across requests.
    (Checked through a later error so that nothing reaches the device.)"""
    with pytest.raises(B.GdnError) as ei:
        call_prefill(monkeypatch, emit_slot=[1, 4], workspace=FakeDev(ptr=0x100000, nbytes=16))
    assert ei.value.code == -9


def test_empty_call_is_ok(monkeypatch):
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    shape = B.make_shape(1, 2, 2, 64, 64, "f32", "f32", 0)
    B.gdn_resume_prefill(shape, None, None, None, None, None, [0], [], None, [], [0], [], None, [], None, None,
                         ctypes.c_void_p(0))
    B.gdn_resume_prefill(shape, None, None, None, None, None, [0, 0], [5], None, [-1], [0, 0], [], None, [], None,
                         None, ctypes.c_void_p(0))


@pytest.mark.parametrize("fn", ["ckpt_gather", "ckpt_scatter"])
def test_copy_argument_errors(monkeypatch, fn):
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    f = getattr(B, fn)
    pool = FakeDev(n0=8, stride0=64)
    other = FakeDev(ptr=0x20000, n0=2, stride0=64)
    with pytest.raises(B.GdnError) as ei:
        f(pool, [0, 8], other, 64)
    assert ei.value.code == -5
    with pytest.raises(B.GdnError) as ei:
        f(pool, [0, 1], FakeDev(ptr=0x20004, stride0=64), 64)
    assert ei.value.code == -2
    with pytest.raises(B.GdnError) as ei:
        f(pool, [0, 1], other, 62)
    assert ei.value.code == -2
    with pytest.raises(B.GdnError) as ei:
        f(pool, [0, 1], other, 128)          # stride smaller than the state
    assert ei.value.code == -3
    if fn == "ckpt_scatter":
        with pytest.raises(B.GdnError) as ei:
            f(pool, [1, 1], other, 64)
        assert ei.value.code == -6
        with pytest.raises(B.GdnError) as ei:
            f(pool, [-1, 1], other, 64)
        assert ei.value.code == -5
    f(pool, [], other, 64)                    # nothing to copy: fine, nothing enqueued


def test_slab_rounds_knob_bounds_the_workspace():
    """A shorter slab needs a smaller workspace; the knob returns the previous setting."""
    shape = B.make_shape(1, 16, 16, 128, 128, "bf16", "f32", 8192)
    auto = B.gdn_workspace_bytes(shape, 1, 8192, 16)
    assert B.gdn_tune_slab_rounds(4) == 0
    try:
        small = B.gdn_workspace_bytes(shape, 1, 8192, 16)
        assert B.gdn_tune_slab_rounds(8) == 4
        mid = B.gdn_workspace_bytes(shape, 1, 8192, 16)
    finally:
        B.gdn_tune_slab_rounds(0)
    assert 0 < small < mid < auto
    assert B.gdn_workspace_bytes(shape, 1, 8192, 16) == auto


@pytest.mark.parametrize("over,code", [
    (dict(slot=[0, 0]), -6),                                   # two requests share a state
    (dict(slot=[0, 8]), -5),
    (dict(slot=[-1, 1]), -5),
    (dict(q=FakeDev(ptr=0)), -1),
    (dict(o=FakeDev(ptr=0x10004)), -2),
    (dict(pool=FakeDev(stride0=2 * 64 * 64 - 4)), -3),
    (dict(pool=FakeDev(stride0=2 * 64 * 64 + 2)), -2),
    (dict(slot=[0, 1, 2], T_alloc=2), -4),                      # more requests than token rows
])
def test_decode_argument_errors(monkeypatch, over, code):
    """Every check of gdn_decode_step fires on the host, before anything is enqueued."""
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    d = FakeDev()
    args = dict(q=d, k=d, v=d, beta=d, gate=d, pool=FakeDev(), slot=[0, 1], o=d, T_alloc=4)
    args.update(over)
    shape = B.make_shape(1, 2, 2, 64, 64, "f32", "f32", args.pop("T_alloc"))
    with pytest.raises(B.GdnError) as ei:
        B.gdn_decode_step(shape, args["q"], args["k"], args["v"], args["beta"], args["gate"], args["pool"], args["slot"],
                          args["o"], ctypes.c_void_p(0))
    assert ei.value.code == code


@pytest.mark.parametrize("fn", ["ckpt_fetch_host", "ckpt_spill_host"])
def test_host_tier_copy_argument_errors(monkeypatch, fn):
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    f = getattr(B, fn)
    host, dev = FakeDev(ptr=0x20000, n0=4, stride0=64), FakeDev(ptr=0x30000, n0=6, stride0=64)
    cases = [
        (dict(host_ids=[0, 4], dev_ids=[0, 1]), -5),
        (dict(host_ids=[0, 1], dev_ids=[0, 6]), -5),
        (dict(host_ids=[-1, 1], dev_ids=[0, 1]), -5),
        (dict(host_ids=[0, 1], dev_ids=[2, 2]) if fn == "ckpt_fetch_host" else dict(host_ids=[1, 1], dev_ids=[0, 2]), -6),
        (dict(host=FakeDev(ptr=0)), -1),
        (dict(dev=FakeDev(ptr=0x30004, n0=6, stride0=64)), -2),
        (dict(elems=66), -2),
        (dict(host=FakeDev(ptr=0x20000, n0=4, stride0=32)), -3),
    ]
    for over, code in cases:
        a = dict(host=host, dev=dev, host_ids=[0, 1], dev_ids=[0, 1], elems=64)
        a.update(over)
        with pytest.raises(B.GdnError) as ei:
            f(a["host"], a["host_ids"], a["dev"], a["dev_ids"], a["elems"], ctypes.c_void_p(0))
        assert ei.value.code == code, (over, ei.value.code)
    f(host, [], dev, [], 64, ctypes.c_void_p(0))                       # empty: nothing to do


def test_host_tier_workspace_is_the_device_one_plus_staging():
    shape = B.make_shape(1, 16, 16, 128, 128, "bf16", "f32", 8192)
    base = B.gdn_workspace_bytes(shape, 3, 8192, 16)
    assert B.gdn_workspace_bytes_host(shape, 3, 8192, 16) == (base + 255) // 256 * 256 + 3 * 16 * 128 * 128 * 4


@pytest.mark.parametrize("dev,code", [(FakeDev(ptr=0), -1), (FakeDev(ptr=0x10004), -2), (FakeDev(nbytes=1 << 19), -9)])
def test_probe_ceilings_argument_errors(monkeypatch, dev, code):
    """The machine-ceiling probe rejects a null, misaligned or too small scratch before touching the device."""
    monkeypatch.setattr(B, "_stream_ptr", lambda s=None: ctypes.c_void_p(0))
    with pytest.raises(B.GdnError) as ei:
        B.gdn_probe_ceilings(dev)
    assert ei.value.code == code


def test_headers_are_plain_c_and_a_c_program_can_call_the_library(tmp_path):
    """The boundary is a C ABI: the headers compile as strict C99 and a C program linked against the
    library calls host-only entry points through them."""
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = tmp_path / "abi.c"
    src.write_text(
        '#include <stdio.h>\n#include "gdn_resume.h"\n#include "gdn_layer.h"\n#include "attn_resume.h"\n#include "ckpt_place.h"\n'
        "int main(void) {\n"
        "    const int32_t pos[3] = {128, 256, 384};\n"
        "    int32_t out[4];\n"
        "    gdn_shape s = {1, 2, 2, 64, 64, GDN_F32, GDN_F32, 1.0f, 512};\n"
        "    if (gdn_version() < 100) return 1;\n"
        "    if (gdn_deepest_ckpt(pos, 3, 300) != 1 || gdn_deepest_ckpt(pos, 3, 5) != -1) return 2;\n"
        "    if (gdn_workspace_bytes(&s, 1, 256, 2) <= 0) return 3;\n"
        "    if (gdn_layer_workspace_bytes(2, 3) <= 0) return 4;\n"
        "    attn_shape as = {16, 2, 128, GDN_BF16, 0.088f};\n"
        "    if (attn_workspace_bytes(&as, 2, 300) <= 0) return 6;\n"
        "    { const int32_t cu[2] = {0, 64}, st[1] = {8000}; int32_t u[5][64], nu, pk, kt;\n"
        "      if (attn_plan(&as, 1, cu, st, 64, u[0], u[1], u[2], u[3], u[4], &nu, &pk, &kt) != GDN_OK || nu != 64 || pk != 8 || kt != 64) return 7; }\n"
        "    if (ckpt_place_balanced(511, 3, out) != 3 || out[0] != 128 || out[2] != 384) return 5;\n"
        '    printf("ok\\n");\n    return 0;\n}\n')
    exe = tmp_path / "abi"
    pkg = os.path.dirname(B.LIB_PATH)
    subprocess.check_call(["gcc", "-std=c99", "-pedantic", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(root, "include"),
                           str(src), "-o", str(exe), "-L", pkg, "-lgdn_resume", "-Wl,-rpath," + pkg])
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip() == "ok"


def test_bench_refuses_more_than_one_gpu_with_a_message():
    """bench.py --gpus N with N above 1 exits at once with a message that says why (nothing touches a GPU)."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert res.returncode == 2 and res.stdout == "" and "ONE GPU" in res.stderr


def resume_path(lens, L, H, d, ws, host=0, dtype="bf16"):
    """The path of a call of requests of these lengths (tokens), each from a stored state, with a workspace of ws bytes."""
    shape = B.make_shape(L, H, H, d, d, dtype, "f32", sum(lens))
    return B.gdn_resume_path(shape, np.concatenate([[0], np.cumsum(lens)]), [0] * len(lens), [0] * (len(lens) + 1), [], ws, host)


def path_calls():
    """(lengths, layers, heads, d): even and ragged calls of 1 to 300 chains, short and long, some around the limits of the two-kernel
    path's slabs."""
    rng = np.random.default_rng(77)
    calls = [([8192] * 2, 1, 16, 128), ([10600] * 2, 1, 16, 128), ([16384] * 2, 1, 16, 128), ([12000] * 2, 1, 16, 128), ([8192], 3, 16, 64),
             ([6500] * 4, 1, 16, 64), ([8192] * 3, 1, 16, 128), ([2048] * 4, 1, 16, 128), ([4100, 3900, 4000], 1, 16, 128), ([131072] * 2, 1, 16, 128),
             ([1048576], 2, 16, 128), ([65536] * 6, 1, 16, 128)]
    for _ in range(400):
        d, H, L = int(rng.choice([64, 128])), int(rng.choice([2, 8, 13, 16])), int(rng.choice([1, 1, 2, 3]))
        n = int(rng.integers(1, 13))
        hi = int(np.exp(rng.uniform(np.log(64), np.log(40000))))
        lo = hi if rng.random() < 0.4 else int(np.exp(rng.uniform(0, np.log(hi))))
        calls.append(([int(x) for x in np.exp(rng.uniform(np.log(lo), np.log(hi), n))], L, H, d))
    return calls


def queried(lens, L, H, d, host=False):
    f = B.gdn_workspace_bytes_host if host else B.gdn_workspace_bytes
    return f(B.make_shape(L, H, H, d, d, "bf16", "f32", sum(lens)), len(lens), sum(lens), 0)


def test_even_calls_with_halved_slabs_go_by_the_estimate():
    """48 even chains of 128 chunks: no special case next to ragged calls of the same volume."""
    assert resume_path([8192] * 3, 1, 16, 128, 1 << 32) == "split 32"
    assert resume_path([8192, 8192, 7000], 1, 16, 128, 1 << 32) == "split 32"


@pytest.mark.parametrize("n_req,H,d,chunks,path", [(1, 8, 128, 12, "two-kernel"), (1, 8, 128, 24, "two-kernel"), (1, 16, 128, 8, "split 32"), (1, 16, 128, 24, "two-kernel"),
                                                   (2, 16, 128, 256, "split 32"), (1, 8, 64, 32, "two-kernel"), (1, 16, 64, 8, "split 32"), (2, 16, 64, 16, "split 32"),
                                                   (2, 16, 64, 256, "two-kernel"), (2, 16, 64, 512, "two-kernel"), (3, 16, 64, 512, "split 32"), (15, 8, 64, 32, "split 32"), (8, 16, 64, 32, "split 32"),
                                                   (15, 8, 128, 32, "split 64"), (14, 16, 128, 32, "pipelined")])
def test_few_chains_get_the_path_that_was_measured_faster(n_req, H, d, chunks, path):
    assert resume_path([64 * chunks] * n_req, 1, H, d, 1 << 32) == path


@pytest.mark.parametrize("n_req,d,chunks,path", [(12, 128, 1, "fused"), (24, 128, 4, "fused"), (100, 128, 1, "fused"), (16, 128, 8, "pipelined"), (400, 128, 4, "pipelined"),
                                                 (40, 128, 32, "pipelined"), (16, 64, 4, "fused"), (100, 64, 8, "fused"), (16, 64, 16, "pipelined"), (32, 64, 126, "pipelined"),
                                                 (400, 64, 4, "fused")])
def test_short_chains_get_the_fused_kernel_and_long_ones_the_pipelined(n_req, d, chunks, path):
    assert resume_path([64 * chunks] * n_req, 1, 16, d, 1 << 32) == path


@pytest.mark.parametrize("lens,path", [
    ([320] * 16 + [128] * 12 + [64] * 8, "fused"),                    # 576 chains, 1.8 k units, longest 5: volume over longest chain 1.45
    ([384] * 12 + [128] * 24, "fused"),                               # longest 6: 1.3
    ([512] * 18 + [128] * 18, "fused"),                               # longest 8, five chunks a chain on average: 1.46
    ([384] * 12 + [64] * 24, "pipelined"),                            # 1.03
    ([640] * 13 + [128] * 24, "pipelined"),                           # longest 10: 1.15
    ([512] * 30 + [320] * 6, "pipelined"),                            # more than five chunks a chain on average
])
def test_ragged_calls_of_short_chains_get_the_fused_kernel_where_volume_outweighs_the_longest(lens, path):
    """d = 128, 16 heads: at most five chunks a chain on average, and a volume that takes 1.2 times as long as the longest chain."""
    assert resume_path(lens, 1, 16, 128, 1 << 32) == path


def test_pairs_of_value_heads_only_where_volume_outweighs_the_longest_chain_by_far():
    """8 query/key heads under 16 value heads: 1152 even chains of 125 chunks 2.47 ms with single heads, 3.05 in pairs; 32768 chains of 8 2.43 and 2.38."""
    def path(lens, L):
        shape = B.make_shape(L, 8, 16, 128, 128, "bf16", "f32", sum(lens))
        return B.gdn_resume_path(shape, np.concatenate([[0], np.cumsum(lens)]), [0] * len(lens), [0] * (len(lens) + 1), [], 1 << 34)
    assert path([8000] * 24, 3) == "pipelined"
    assert path([512] * 256, 8) == "fused pairs"


def test_ragged_calls_get_the_path_that_was_measured_faster():
    """64 chains of 37 to 256 chunks (two-kernel path 604 us, split 489), 256 of 2 to 32 at d = 64 (pipelined 89, split 74), 32 of 19 and 47 (two-kernel path 92, split 98), 48
    of up to 125 at d = 64 (146 against 164)."""
    assert resume_path([64 * 47, 64 * 19], 1, 16, 128, 1 << 32) == "two-kernel"
    assert resume_path([64 * 125, 64 * 3, 64 * 2], 1, 16, 64, 1 << 32) == "two-kernel"
    assert resume_path([64 * c for c in (256, 120, 44, 37)], 1, 16, 128, 1 << 32) == "split 32"
    assert resume_path([64 * c for c in (32, 31, 28, 22, 20, 16, 15, 11, 8, 7, 5, 4, 3, 3, 2, 2)], 1, 16, 64, 1 << 32) == "split 32"


def test_a_larger_workspace_than_the_queried_one_changes_nothing():
    for lens, L, H, d in path_calls():
        ws = queried(lens, L, H, d)
        assert resume_path(lens, L, H, d, ws) == resume_path(lens, L, H, d, 1 << 40), (lens, L, H, d, ws)


def test_the_slab_length_does_not_change_the_arithmetic():
    """With a forced slab length the call stays with the two-kernel path or with the others, which agree bit for bit, as it is."""
    for lens, L, H, d in path_calls():
        auto = resume_path(lens, L, H, d, queried(lens, L, H, d))
        for rounds in (1, 4, 8, 64, 200):
            prev = B.gdn_tune_slab_rounds(rounds)
            try:
                forced = resume_path(lens, L, H, d, queried(lens, L, H, d))
            finally:
                B.gdn_tune_slab_rounds(prev)
            assert (forced == "two-kernel") == (auto == "two-kernel"), (lens, L, H, d, rounds, auto, forced)


def test_short_calls_from_a_host_pool_get_the_launches_that_fetch_beside_their_work():
    """Copies in front of the fused kernel cost more than the second launch: 15 requests of 2 chunks, 8 heads of 64, 199 us against 49."""
    for n, H, d, chunks in [(3, 16, 64, 2), (15, 8, 64, 2), (7, 16, 128, 128), (15, 8, 64, 128)]:
        lens = [64 * chunks] * n
        assert resume_path(lens, 1, H, d, queried(lens, 1, H, d)) in ("fused", "pipelined", "split 64")
        assert resume_path(lens, 1, H, d, queried(lens, 1, H, d, host=True), n).startswith("split")


def test_host_and_device_pools_get_the_same_arithmetic():
    """Start states from a host pool, all of them or some, with the workspace queried for either."""
    for lens, L, H, d in path_calls():
        dev = resume_path(lens, L, H, d, queried(lens, L, H, d))
        for staged in {1, len(lens) // 2, len(lens)}:
            host = resume_path(lens, L, H, d, queried(lens, L, H, d, host=True), staged)
            assert (host == "two-kernel") == (dev == "two-kernel"), (lens, L, H, d, staged, dev, host)
