"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header
declares, and its host-side argument checks return the documented codes without a GPU."""
import ctypes
import os
import re
import shutil
import subprocess
import sys

import pytest

import paper_2506_09316_amd as dsla
from paper_2506_09316_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(dsla.library_path()):
        from paper_2506_09316_amd import build
        build.build()
    return dsla.load_library()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "dsla.h")).read()
    return sorted(set(re.findall(r"DSLA_API[^;(]*?\b(dsla_\w+)\s*\(", text)))


def test_header_symbols_exported(lib):
    names = declared_symbols()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_status_strings(lib):
    for s in range(6):
        assert lib.dsla_status_string(s)


def test_argument_checks_need_no_gpu(lib):
    d = dsla.make_desc(1, 2, 64, 64, io_dtype=0, gate_dtype=0)
    fake = ctypes.c_void_p(4096)
    # NULL state pointer
    assert lib.dsla_state_init(ctypes.byref(d), None, fake, None) == 1
    # unsupported head size
    bad = dsla.make_desc(1, 2, 48, 48, io_dtype=0, gate_dtype=0)
    assert lib.dsla_state_init(ctypes.byref(bad), fake, fake, None) == 3
    # non-positive batch
    bad = dsla.make_desc(0, 2, 64, 64, io_dtype=0, gate_dtype=0)
    assert lib.dsla_decode(ctypes.byref(bad), *([fake] * 9)) == 2
    # misaligned pointer
    odd = ctypes.c_void_p(4100)
    assert lib.dsla_decode(ctypes.byref(d), odd, *([fake] * 8)) == 2
    # chunk lengths other than 32, 64 and 128 are not built
    big = dsla.make_desc(1, 2, 128, 128, io_dtype=0, gate_dtype=0, chunk=48)
    assert lib.dsla_prefill(ctypes.byref(big), 128, *([fake] * 8), None, 0, None) == 3
    # missing workspace when the plan needs one
    seg = dsla.make_desc(1, 2, 64, 64, io_dtype=0, gate_dtype=0, chunk=64, segments=4)
    need = lib.dsla_prefill_workspace_bytes(ctypes.byref(seg), 1024)
    assert need > 0
    assert lib.dsla_prefill(ctypes.byref(seg), 1024, *([fake] * 8), None, 0, None) == 4
    assert lib.dsla_prefill(ctypes.byref(seg), 1024, *([fake] * 8), fake, need - 1, None) == 4
    # gate mode: unknown mode; pre-activation mode needs a finite positive temperature
    bad = dsla.make_desc(1, 2, 64, 64, io_dtype=0, gate_dtype=0, gate_mode=2)
    assert lib.dsla_decode(ctypes.byref(bad), *([fake] * 9)) == 3
    for tau in (0.0, -1.0, float("inf"), float("nan")):
        bad = dsla.make_desc(1, 2, 64, 64, io_dtype=0, gate_dtype=0, gate_mode=1, tau=tau)
        assert lib.dsla_decode(ctypes.byref(bad), *([fake] * 9)) == 2
        assert lib.dsla_prefill_workspace_bytes(ctypes.byref(bad), 1024) == 0
    ignored = dsla.make_desc(1, 2, 64, 64, io_dtype=0, gate_dtype=0, gate_mode=0, tau=0.0)   # tau unused for log gates
    assert lib.dsla_prefill(ctypes.byref(ignored), 0, None, None, None, None, None, fake, fake, None, None, 0, None) == 0
    # packed sequences: the bound of the lengths cannot exceed the total; the offsets are required
    assert lib.dsla_prefill_varlen(ctypes.byref(d), 100, 101, fake, None, None, *([fake] * 8), None, 0, None) == 2
    assert lib.dsla_prefill_varlen(ctypes.byref(d), 100, 50, None, None, None, *([fake] * 8), None, 0, None) == 1
    assert lib.dsla_prefill_varlen(ctypes.byref(d), 2 ** 31, 50, fake, None, None, *([fake] * 8), None, 0, None) == 2
    assert lib.dsla_prefill_varlen(ctypes.byref(d), 0, 0, fake, None, None, None, None, None, None, None, fake, fake,
                                   None, None, 0, None) == 0
    assert lib.dsla_prefill_varlen(ctypes.byref(seg), 4096, 1024, fake, None, None, *([fake] * 8), None, 0, None) == 4
    assert lib.dsla_prefill_varlen(ctypes.byref(d), 100, 50, fake, ctypes.c_void_p(4098), None, *([fake] * 8), None, 0,
                                   None) == 2
    assert lib.dsla_decode_slots(ctypes.byref(d), *([fake] * 5), None, None, *([fake] * 3), None) == 1
    assert lib.dsla_decode_slots(ctypes.byref(d), *([fake] * 5), None, ctypes.c_void_p(4098), *([fake] * 3), None) == 2
    assert lib.dsla_decode_slots(ctypes.byref(d), *([fake] * 5), ctypes.c_void_p(4098), fake, *([fake] * 3), None) == 2
    # T = 0 does nothing and needs no tensors
    assert lib.dsla_prefill(ctypes.byref(d), 0, None, None, None, None, None, fake, fake, None, None, 0, None) == 0
    assert lib.dsla_prefill(ctypes.byref(d), -1, *([fake] * 8), None, 0, None) == 2


def test_projection_argument_checks(lib):
    fake = ctypes.c_void_p(4096)
    outs = (ctypes.c_void_p * 2)(4096, 8192)
    call = lambda M, K, n_out, width, x=fake, W=fake, o=outs: lib.dsla_project(
        ctypes.c_int64(M), K, n_out, width, x, W, None, o, None)
    assert call(0, 128, 2, 128) == 2                       # no rows
    assert call(16, 48, 2, 128) == 3                       # K is not a multiple of 32
    assert call(16, (1 << 21) + 128, 2, 128) == 3          # K beyond the 32-bit offsets of a tile
    assert call(16, 128, 2, 192) == 3                      # width is not a multiple of 128
    assert call(16, 128, 9, 128) == 3                      # more outputs than DSLA_MAX_PROJECTIONS
    assert call(16, 128, 2, 128, x=None) == 1
    assert call(16, 128, 2, 128, W=ctypes.c_void_p(4100)) == 2
    assert call(16, 128, 2, 128, o=(ctypes.c_void_p * 2)(4096, None)) == 1


def test_attention_entropy_argument_checks_and_plan(lib):
    fake = ctypes.c_void_p(4096)
    call = lambda B, H, d, T, io, q=fake, k=fake, o=fake, ws=None, n=0: lib.dsla_attention_entropy(
        B, H, d, T, io, 1.0, q, k, o, ws, n, None)
    assert call(0, 4, 128, 100, 1) == 2
    assert call(2, 4, 128, 0, 1) == 2
    assert call(2, 4, 96, 100, 1) == 3
    assert call(2, 4, 128, 100, 7) == 3
    assert call(2, 4, 128, 100, 1, q=None) == 1
    assert call(2, 4, 128, 100, 1, k=ctypes.c_void_p(4100)) == 2
    # 8 x 32 (batch, head) pairs: two workgroups each -> parts of 4096 keys, 3 floats per part
    assert lib.dsla_attention_entropy_workspace_bytes(8, 32, 128, 8192) == 256 * 2 * 3 * 4
    # 1024 pairs fill the device on their own: no split, no workspace
    assert lib.dsla_attention_entropy_workspace_bytes(32, 32, 128, 8192) == 0
    # a short sequence is not split below 256 keys per workgroup
    assert lib.dsla_attention_entropy_workspace_bytes(1, 2, 64, 600) == 2 * 3 * 3 * 4
    assert call(1, 2, 64, 600, 1) == 4          # workspace needed and missing
    assert lib.dsla_attention_entropy_workspace_bytes(1, 2, 48, 600) == 0


def test_attention_decode_argument_checks_and_plan(lib):
    fake = ctypes.c_void_p(4096)
    call = lambda B, H, d, T, io, q=fake, k=fake, v=fake, o=fake, ws=None, n=0, lens=None: lib.dsla_attention_decode(
        B, H, d, T, io, 1.0, q, k, v, lens, o, ws, n, None)
    assert call(2, 4, 128, 100, 1, lens=ctypes.c_void_p(4098)) == 2
    assert call(2, 0, 128, 100, 1) == 2
    assert call(2, 4, 100, 100, 1) == 3
    assert call(2, 4, 128, 100, 1, v=None) == 1
    assert call(2, 4, 128, 100, 1, o=ctypes.c_void_p(4104)) == 2
    # same split as the entropy kernel, a record of 2 + d floats per part
    assert lib.dsla_attention_decode_workspace_bytes(8, 32, 128, 8192) == 256 * 2 * 130 * 4
    assert lib.dsla_attention_decode_workspace_bytes(32, 32, 128, 8192) == 0
    assert call(8, 32, 128, 8192, 1) == 4


def test_attention_prefill_argument_checks(lib):
    fake = ctypes.c_void_p(4096)
    call = lambda B, H, d, T, io, q=fake, k=fake, v=fake, o=fake: lib.dsla_attention_prefill(
        B, H, d, ctypes.c_int64(T), io, 1.0, q, k, v, o, None)
    assert call(0, 4, 128, 100, 1) == 2
    assert call(2, 4, 100, 100, 1) == 3                  # head size
    assert call(2, 4, 128, 100, 0) == 3                  # fp32 is not built
    assert call(2, 4, 128, 100, 1, k=None) == 1
    assert call(2, 4, 128, 100, 1, o=ctypes.c_void_p(4104)) == 2
    assert call(1, 32, 128, 1 << 19, 1) == 2             # one sequence's tensor reaches 4 GiB: 32-bit byte offsets


def test_varlen_workspace_plan(lib):
    up = lambda n: (n + 255) // 256 * 256
    # 8 sequences, 32 heads; total 32768 tokens, longest 16384.  The segment length follows the total (about one
    # workgroup per compute unit overall): 32768 * 32 / 256 = 4096 tokens, so the longest sequence has 4 segments.
    # Worst case 32768 / 4096 + 8 = 16 segments in all, 8 of them with a successor.
    d = dsla.make_desc(8, 32, 128, 128, io_dtype=1, gate_dtype=1, chunk=64)
    slots = 16 * 32
    want = slots * 2 * 128 * 128 * 4 + up(slots * 2 * 128 * 4) + up(9 * 4) + 256 + up(16 * 8) + up(8 * 8)
    assert lib.dsla_prefill_varlen_workspace_bytes(ctypes.byref(d), 32768, 16384) == want
    # short sequences only: one segment each, no workspace
    assert lib.dsla_prefill_varlen_workspace_bytes(ctypes.byref(d), 2048, 256) == 0
    # equal lengths and a given segment count: the workspace differs from the dense call's only by the lists
    d3 = dsla.make_desc(3, 2, 128, 128, io_dtype=1, gate_dtype=1, chunk=64, segments=3)
    dense = lib.dsla_prefill_workspace_bytes(ctypes.byref(d3), 384)
    packed = lib.dsla_prefill_varlen_workspace_bytes(ctypes.byref(d3), 3 * 384, 384)
    assert dense == 3 * 6 * 2 * 128 * 128 * 4 + up(2 * 6 * 2 * 128 * 4)
    assert packed == 12 * 2 * 2 * 128 * 128 * 4 + up(12 * 2 * 2 * 128 * 4) + up(4 * 4) + 256 + up(12 * 8) + up(9 * 8)


def test_workspace_plan(lib):
    # one segment: no workspace
    d = dsla.make_desc(8, 32, 128, 128, io_dtype=1, gate_dtype=1, chunk=64)
    assert lib.dsla_prefill_workspace_bytes(ctypes.byref(d), 8192) == 0
    # B*H = 32 at T = 16384: 8 segments of both fp32 states plus the decay vectors
    d = dsla.make_desc(1, 32, 128, 128, io_dtype=1, gate_dtype=1, chunk=64)
    n = lib.dsla_prefill_workspace_bytes(ctypes.byref(d), 16384)
    assert n == 8 * 32 * 2 * 128 * 128 * 4 + 7 * 32 * 2 * 128 * 4
    # B*H = 128: two segments, and the pre-pass on the two halves of the first one (3 slots, 2 decay vectors);
    # a caller who asks for two segments gets two slots
    d = dsla.make_desc(4, 32, 128, 128, io_dtype=1, gate_dtype=1, chunk=64)
    assert lib.dsla_prefill_workspace_bytes(ctypes.byref(d), 16384) == 3 * 128 * 2 * 128 * 128 * 4 + 2 * 128 * 2 * 128 * 4
    d = dsla.make_desc(4, 32, 128, 128, io_dtype=1, gate_dtype=1, chunk=64, segments=2)
    assert lib.dsla_prefill_workspace_bytes(ctypes.byref(d), 16384) == 2 * 128 * 2 * 128 * 128 * 4 + 1 * 128 * 2 * 128 * 4


def test_conversion_logic_against_its_oracle(lib):
    """The host-side conversion logic of the library (C++) against the plain Python statement of the same rules:
    the paper's table, rankings of seeded scores with ties, and conversion plans over a sweep of memory situations."""
    import numpy as np
    from oracle import controller as ctl
    for L in (0, 1, 2047, 2048, 3000, 4095, 4096, 8191, 8192, 100000):
        assert dsla.dsla_max_conversion_rate(L) == ctl.max_conversion_rate(L)
    assert dsla.dsla_kv_cache_bytes(32, 8, 8192, 32, 128, 2) == ctl.kv_cache_bytes(32, 8, 8192, 32, 128, 2)
    rng = np.random.default_rng(11)
    for n in (1, 4, 32):
        sens = np.round(rng.uniform(0, 5, n), 1).astype(np.float32)     # rounded: ties occur
        order = dsla.dsla_rank_layers(sens)
        assert order == ctl.rank_layers(sens)
        kv, st = 64 << 20, 4 << 20
        for used_layers in (0, n // 2, n):
            for thr_layers in (0, n // 4, n // 2, n):
                for rate in (0.0, 0.125, 0.25, 0.5, 1.0):
                    used, thr = 1000 + used_layers * kv, 1000 + thr_layers * kv
                    assert dsla.dsla_conversion_plan(order, used, thr, kv, st, rate) == \
                        ctl.conversion_plan(order, used, thr, kv, st, rate)
    # argument errors
    bad = (ctypes.c_int32 * 3)(0, 0, 1)
    conv = (ctypes.c_uint8 * 3)()
    cnt = ctypes.c_int32()
    assert lib.dsla_conversion_plan(3, bad, 10, 5, 2, 1, 1.0, conv, ctypes.byref(cnt), None, None) == 2
    assert lib.dsla_rank_layers(2, (ctypes.c_float * 2)(1.0, float("nan")), (ctypes.c_int32 * 2)()) == 2


def test_plans_follow_the_work(lib):
    slots = lambda n, H, d: n * H * 2 * d * d * 4
    up = lambda n: (n + 255) // 256 * 256
    dense = lambda B, H, d, io, T: lib.dsla_prefill_workspace_bytes(
        ctypes.byref(dsla.make_desc(B, H, d, d, io_dtype=io, gate_dtype=io, chunk=64)), T)
    want = lambda P, BH, d: slots(P, BH, d) + up((P - 1) * BH * 2 * d * 4)
    assert dense(1, 32, 128, 1, 1000) == want(6, 32, 128)     # 3 chunks per segment
    assert dense(1, 4, 128, 1, 1000) == want(8, 4, 128)       # 2 where that leaves most of the chip idle
    assert dense(1, 4, 64, 0, 256) == want(4, 4, 64)          # fp32: short prompts are cut too, down to a chunk
    assert dense(1, 32, 128, 0, 1000) == want(8, 32, 128)     # and never into more than the chip holds
    assert dense(8, 32, 64, 1, 4000) == 0                     # 256 heads at d = 64: whole
    assert dense(1, 32, 128, 1, 256) == 0
    assert dense(1, 4, 64, 0, 70) == dense(1, 96, 64, 0, 133) == dense(1, 120, 128, 0, 176) == 0   # fp32: too few steps to save
    assert dense(1, 96, 128, 0, 256) == want(2, 96, 128)
    assert dense(1, 24, 64, 1, 2500) == want(10, 24, 64)      # d = 64: one workgroup to a compute unit ...
    assert dense(1, 24, 64, 1, 4000) == want(21, 24, 64)      # ... or as short as two to a unit make them
    packed = lambda B, H, d, total, longest: lib.dsla_prefill_varlen_workspace_bytes(
        ctypes.byref(dsla.make_desc(B, H, d, d, io_dtype=1, gate_dtype=1, chunk=64)), total, longest)
    assert packed(40, 32, 128, 3460, 651) == 0                # many short sequences fill the chip whole
    assert packed(8, 32, 128, 1959, 1900) > 0                 # one long chain is cut
    assert packed(22, 8, 128, 9484, 4015) > 0


def test_plans_of_short_prompts(lib):
    """16 bits, 257 to 1023 tokens: as many segments as pay, and buffers that hold the coarse cut as well."""
    slots = lambda n, H, d: n * H * 2 * d * d * 4
    up = lambda n: (n + 255) // 256 * 256
    dense = lambda BH, d, T, chunk=64: lib.dsla_prefill_workspace_bytes(
        ctypes.byref(dsla.make_desc(1, BH, d, d, io_dtype=1, gate_dtype=1, chunk=chunk)), T)
    want = lambda P, BH, d: slots(P, BH, d) + up((P - 1) * BH * 2 * d * 4)
    assert dense(4, 128, 400) == want(7, 4, 128)              # one chunk per segment
    assert dense(32, 128, 640) == want(5, 32, 128)            # two
    assert dense(32, 128, 400) == dense(64, 64, 400) == 0     # whole, and the coarse cut is whole too
    assert dense(96, 128, 640) == want(2, 96, 128)            # whole, and the buffer holds the coarse cut in two (10 chunks),
    assert dense(128, 128, 1000) == slots(3, 128, 128) + up(2 * 128 * 2 * 128 * 4)   # or in two with the pre-pass on half segments
    # a call that runs whole needs the buffer it was asked for, as one that is cut does
    d = dsla.make_desc(1, 96, 128, 128, io_dtype=1, gate_dtype=1, chunk=64)
    fake = ctypes.c_void_p(4096)
    call = lambda ws, n: lib.dsla_prefill(ctypes.byref(d), 640, *([fake] * 8), ws, n, None)
    assert call(None, 0) == call(fake, want(2, 96, 128) - 1) == 4
    assert call(ctypes.c_void_p(4096 + 64), want(2, 96, 128)) == 2
    assert dense(4, 128, 1400, 128) == slots(3, 4, 128) + up(2 * 4 * 2 * 128 * 4)   # a chunk of 128 keeps its granularity


def test_packed_workspace_of_a_large_batch_serves_smaller_ones(lib):
    """A batch that stays whole because that is faster answers the size query with what cutting it takes: 20 sequences of up
    to 8192 tokens, as the batch shrinks from whole ones to cut ones; none where even one sequence of that length stays
    whole, or where every batch does because nothing is longer than four chunks."""
    ask = lambda B, H, d, total, longest, preact=1: lib.dsla_prefill_varlen_workspace_bytes(
        ctypes.byref(dsla.make_desc(B, H, d, d, io_dtype=1, gate_dtype=1, chunk=64, gate_mode=preact)), total, longest)
    # (within the few per cent that the rounding of the segment length to whole chunks makes between neighbouring totals)
    sizes = [ask(20, 32, 128, total, 8192) for total in (9000, 16384, 20000, 25000, 30000, 37157)]
    assert all(s >= 0.9 * max(sizes) for s in sizes)
    for B, H, d, total, longest in ((64, 32, 128, 41523, 7076), (8, 64, 64, 12913, 4336), (53, 40, 128, 1085, 886)):
        big = ask(B, H, d, total, longest)
        for part in (2, 3, 5):
            assert big >= 0.9 * ask(B, H, d, max(total // part, longest), longest) > 0
    assert ask(40, 32, 128, 3460, 600) == 0 and ask(300, 32, 128, 30000, 256) == 0


def test_native_calls_leave_unusual_arguments_to_the_general_way():
    """Without a GPU: the native calls answer None, with no exception pending, to tensors on the CPU, to what is no tensor and to wrong
    numbers of arguments; the general way then refuses it as it always has.  (One odd argument among right ones takes GPU tensors: test_gpu_06.)"""
    import torch
    dsla.load_library()
    native = dsla.binding._native
    desc = dsla.make_desc(1, 4, 64, 64, io_dtype=0, gate_dtype=0, chunk=64)
    x, S = torch.zeros(1, 4, 64), torch.zeros(1, 4, 64, 64)
    for odd in (x, x.transpose(1, 2), torch.nn.Parameter(x), None, 1, "x", x.numpy()):
        assert native.decode(desc, odd, x, x, x, x, S, S, x) is None
        assert native.prefill(desc, 1, x, x, x, x, x, S, S, x, odd) is None
    assert native.decode() is None and native.decode(desc, x) is None and native.decode(3, *[x] * 8) is None
    assert native.decode_slots(desc, *[x] * 5, None, x, S, S, x) is None
    assert native.prefill(desc, 2.0, *[x] * 8, None) is None and native.prefill(desc, 1 << 70, *[x] * 8, None) is None
    assert native.prefill_varlen(desc, 1, 1, x, None, None, *[x] * 8, None) is None
    assert native.attention_decode(x, x, x, x, 1.0, None, None) is None and native.attention_prefill(x, x, x, x, 1) is None
    assert native.project(x, x, [x], None) is None and native.project(x, x, (x,), None) is None
    with pytest.raises(AssertionError):
        dsla.dsla_decode(desc, x, x, x, x, x, S, S, x)
    with pytest.raises(AssertionError):
        dsla.dsla_project(x[0], x[0], [x])
    with pytest.raises(AttributeError):
        dsla.dsla_prefill(desc, 1, 3, x, x, x, x, S, S, x)
    with pytest.raises(ValueError):
        dsla.dsla_attention_prefill(x, x, x, x, 1.0)


@pytest.mark.parametrize("found", ["nothing", "no library", "another version", "this one"])
def test_the_library_loads_without_its_native_calls(lib, tmp_path, found):
    """_marshal.so missing, unreadable, or built for another header: a warning, and every call goes through ctypes."""
    package = tmp_path / "paper_2506_09316_amd"
    here = os.path.dirname(dsla.library_path())
    shutil.copytree(here, package, ignore=shutil.ignore_patterns("csrc", "__pycache__", *([] if found in ("another version", "this one") else ["_marshal.so"])))
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    if found == "no library":
        (package / "_marshal.so").write_bytes(b"text")
    if found == "another version":
        with open(tmp_path / "include" / "dsla.h", "a") as f:
            f.write("/* changed */\n")
    child = """
import ctypes, sys, warnings
import torch
import paper_2506_09316_amd as dsla
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    dsla.load_library()
native = dsla.binding._native is not dsla.binding._General
x, S = torch.zeros(1, 4, 64), torch.zeros(1, 4, 64, 64)
desc = dsla.make_desc(1, 4, 64, 64, io_dtype=0, gate_dtype=0)
for call in (lambda: dsla.dsla_decode(desc, *[x] * 5, S, S, x), lambda: dsla.dsla_prefill(desc, 1, *[x] * 5, S, S, x),
             lambda: dsla.dsla_prefill_varlen(desc, 1, 1, x, None, *[x] * 5, S, S, x), lambda: dsla.dsla_decode_slots(desc, *[x] * 5, x, S, S, x),
             lambda: dsla.dsla_attention_decode(x, S, S, x, 1.0), lambda: dsla.dsla_attention_prefill(S, S, S, S, 1.0), lambda: dsla.dsla_project(x[0], x[0], [x])):
    try:
        call()
    except AssertionError:   # (not on the GPU)
        continue
    raise SystemExit("taken")
print("native" if native else "general", sum(w.category is RuntimeWarning for w in seen))
"""
    run = subprocess.run([sys.executable, "-c", child], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
    assert run.stdout.split() == (["native", "0"] if found == "this one" else ["general", "1"])
