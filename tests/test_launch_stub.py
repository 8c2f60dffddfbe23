"""What the library does around its launches, with these stubbed out (no GPU; a process of its own, in which the stub comes before
the runtime): launch errors reach the caller, and which calls are accepted with which buffer."""
import os
import subprocess
import sys

import paper_2506_09316_amd as dsla

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(None)
stub.launch_stub_reset(-1)   # (missing where the stub is not loaded: then nothing is called)
from paper_2506_09316_amd import binding
lib = ctypes.CDLL(binding.library_path())
for n in ("dsla_prefill_workspace_bytes", "dsla_prefill_varlen_workspace_bytes", "dsla_prefill_multi_workspace_bytes",
          "dsla_attention_decode_workspace_bytes"):
    getattr(lib, n).restype = ctypes.c_size_t
i64, size, f32, fake = ctypes.c_int64, ctypes.c_size_t, ctypes.c_float, ctypes.c_void_p(4096)
OK, ERR_SHAPE, ERR_WORKSPACE, ERR_HIP = 0, 2, 4, 5
"""

LAUNCH_ERRORS = r"""
def each_launch(name, launches, call):
    stub.launch_stub_reset(-1)
    assert call() == OK and stub.launch_stub_count() == launches, (name, stub.launch_stub_count())
    for n in range(launches):
        stub.launch_stub_reset(n)
        assert call() == ERR_HIP, (name, n)
        assert stub.launch_stub_count() == n + 1, (name, n)   # nothing runs on what a failed launch left unwritten

for io in (0, 1):
    for gate in (0, 1):
        for d in (64, 128):
            desc = lambda B, H, segments: ctypes.byref(binding.make_desc(B, H, d, d, io_dtype=io, gate_dtype=gate, chunk=64, segments=segments))
            for H in (4, 300):                     # at most one workgroup to a compute unit and more
                for segments, launches in ((1, 1), (3, 3)):
                    q = desc(1, H, segments)
                    n = lib.dsla_prefill_workspace_bytes(q, i64(192))
                    each_launch(("prefill", io, gate, d, H, segments), launches,
                                lambda: lib.dsla_prefill(q, i64(192), *[fake] * 8, fake, size(n), None))
                    n = lib.dsla_prefill_varlen_workspace_bytes(q, i64(500), i64(192))
                    each_launch(("packed", io, gate, d, H, segments), launches + (segments > 1),
                                lambda: lib.dsla_prefill_varlen(q, i64(500), i64(192), fake, None, None, *[fake] * 8, fake, size(n), None))
                    vp = ctypes.c_void_p * 2
                    for beta in (None, vp(None, 4096)):
                        multi = binding.DslaMulti(2, 0, vp(4096, 4096), beta, vp(4096, 8192), (ctypes.c_float * 2)(.5, .5), None)
                        n = lib.dsla_prefill_multi_workspace_bytes(q, ctypes.byref(multi), i64(192))
                        # with a beta gate on the second state, the first has an idle partner, whose state is cleared by a launch
                        each_launch(("states", io, gate, d, H, segments, bool(beta)), 2 * launches + 1 if beta else launches,
                                    lambda: lib.dsla_prefill_multi(q, ctypes.byref(multi), i64(192), *[fake] * 5, size(n), None))
            each_launch(("decode", io, gate, d), 1, lambda: lib.dsla_decode(desc(2, 4, 0), *[fake] * 9))
for d in (64, 128):
    for T in (100, 5000):
        each_launch(("attention prefill", d, T), 1, lambda: lib.dsla_attention_prefill(1, 4, d, i64(T), 1, f32(1), *[fake] * 4, None))
    for io, T, launches in ((0, 5000, 2), (1, 5000, 2), (1, 100, 1)):
        n = lib.dsla_attention_decode_workspace_bytes(1, 4, d, i64(T))
        each_launch(("attention decode", d, io, T), launches,
                    lambda: lib.dsla_attention_decode(1, 4, d, i64(T), io, f32(1), *[fake] * 3, None, fake, fake, size(n), None))
for M, K in ((1, 256), (100, 256), (100, 128), (300, 96), (300, 128), (5000, 4096)):
    each_launch(("project", M, K), 1, lambda: lib.dsla_project(i64(M), K, 1, 4096, fake, fake, None, (ctypes.c_void_p * 1)(4096), None))
"""

BUFFERS = r"""
odd = ctypes.c_void_p(4096 + 64)   # not on a multiple of 256

def dense(H, d, T, io, ws, n, B=1):
    stub.launch_stub_reset(-1)
    status = lib.dsla_prefill(ctypes.byref(binding.make_desc(B, H, d, d, io_dtype=io, gate_dtype=io, chunk=64)), i64(T), *[fake] * 8, ws, size(n), None)
    return status, stub.launch_stub_count()

big = 1 << 40
# nothing is asked for where the first rule cuts nothing and the buffer is too small to use: its alignment does not matter
for H, d, T in ((4, 64, 255), (32, 128, 300)):
    assert dense(H, d, T, 0, odd, 1024) == dense(H, d, T, 0, None, 0) == (OK, 1)
    assert dense(H, d, T, 0, fake, big) == (OK, 3) and dense(H, d, T, 0, odd, big) == (ERR_SHAPE, 0)
# 16 bits, 257 tokens and more: cut with a buffer, whole with none that can be used
for H, d, T in ((8, 128, 372), (4, 128, 400), (4, 64, 400)):
    assert dense(H, d, T, 1, fake, big) == (OK, 3)
    assert dense(H, d, T, 1, odd, big) == dense(H, d, T, 1, odd, 1024) == dense(H, d, T, 1, fake, 1024) == dense(H, d, T, 1, None, 0) == (OK, 1)
# the first rule cuts: a buffer is asked for, whatever the estimates make of the call
for H, d, T, launches in ((96, 128, 640, 1), (8, 128, 1000, 3)):
    assert dense(H, d, T, 1, fake, big) == (OK, launches)
    assert dense(H, d, T, 1, odd, big) == (ERR_SHAPE, 0) and dense(H, d, T, 1, None, 0) == dense(H, d, T, 1, odd, 1024) == (ERR_WORKSPACE, 0)

def packed(B, H, d, total, longest, io, ws, n):
    stub.launch_stub_reset(-1)
    status = lib.dsla_prefill_varlen(ctypes.byref(binding.make_desc(B, H, d, d, io_dtype=io, gate_dtype=io, chunk=64)), i64(total), i64(longest), fake, None,
                                     None, *[fake] * 8, ws, size(n), None)
    return status, stub.launch_stub_count()

# packed, fp32: a cut that faster kernels made worth it, which no buffer used to be asked for, and one that always needed its buffer
for B, H, d, total, longest in ((22, 32, 128, 1217, 346), (18, 64, 128, 1323, 641)):
    assert packed(B, H, d, total, longest, 0, fake, big) == (OK, 4)
    assert packed(B, H, d, total, longest, 0, odd, big) == packed(B, H, d, total, longest, 0, fake, 1024) == packed(B, H, d, total, longest, 0, None, 0) == (OK, 1)
for io in (0, 1):
    assert packed(8, 32, 128, 1959, 1900, io, fake, big) == (OK, 4)
    assert packed(8, 32, 128, 1959, 1900, io, odd, big) == (ERR_SHAPE, 0)
    assert packed(8, 32, 128, 1959, 1900, io, fake, 1024) == packed(8, 32, 128, 1959, 1900, io, None, 0) == (ERR_WORKSPACE, 0)
# only the long ones cut: with a buffer; whole without one that holds at least the lists and two slots
assert packed(20, 32, 128, 37157, 8192, 1, fake, big) == (OK, 4)
assert packed(20, 32, 128, 37157, 8192, 1, None, 0) == packed(20, 32, 128, 37157, 8192, 1, fake, 1 << 22) == packed(20, 32, 128, 37157, 8192, 1, odd, big) == (OK, 1)
# d = 64: none of them
for B, H, total, longest in ((8, 32, 41097, 7301), (32, 32, 39561, 7524), (22, 32, 6610, 1924)):
    assert packed(B, H, 64, total, longest, 1, fake, big) == (OK, 1)
# nor at d = 128 where the lists, an empty pre-pass and an empty scan would be much of a call whose bound turns out loose
for B, H, total, longest in ((31, 8, 19014, 1616), (18, 32, 22985, 6652), (3, 32, 5683, 1926), (24, 32, 18417, 5826)):
    assert packed(B, H, 128, total, longest, 1, fake, big) == (OK, 1)

# fp32 prompts of a few hundred tokens from zero states: one launch in the attention form (gates as pre-activations too), whatever the batch is
# cut into otherwise; states carried in, a number of segments that is named, long prompts and many heads take the plan
def short(B, H, d, T, zero_init, segments=0, gate_mode=0, io=0):
    stub.launch_stub_reset(-1)
    desc = ctypes.byref(binding.make_desc(B, H, d, d, io_dtype=io, gate_dtype=io, chunk=64, segments=segments, zero_init=zero_init, gate_mode=gate_mode))
    status = lib.dsla_prefill(desc, i64(T), *[fake] * 8, fake, size(big), None)
    return status, stub.launch_stub_count()

for gate_mode in (0, 1):
    for B, H, d, T in ((1, 4, 64, 256), (2, 3, 64, 270), (1, 2, 64, 600), (2, 3, 128, 140), (1, 2, 128, 300)):
        assert short(B, H, d, T, 1, 0, gate_mode) == (OK, 1) and short(B, H, d, T, 0, 0, gate_mode) == (OK, 3), (B, H, d, T)
        assert short(B, H, d, T, 1, 2, gate_mode) == (OK, 3)
    for B, H, d, T in ((1, 4, 64, 6000), (1, 2, 128, 4000), (8, 8, 64, 2000)):
        assert short(B, H, d, T, 1, 0, gate_mode) == (OK, 3), (B, H, d, T)
assert short(1, 2, 64, 600, 1, io=1) == (OK, 3)
"""


def run_stubbed(tmp_path, body):
    if not os.path.exists(dsla.library_path()):
        from paper_2506_09316_amd import build
        build.build()
    stub = str(tmp_path / "launch_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", stub, os.path.join(HERE, "launch_stub.c")], check=True)
    env = dict(os.environ, LD_PRELOAD=":".join(p for p in (stub, os.environ.get("LD_PRELOAD")) if p))
    run = subprocess.run([sys.executable, "-c", CHILD + body + "print('done')"], env=env, cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout.strip().endswith("done"), run.stderr


def test_launch_errors_reach_the_caller(tmp_path):
    run_stubbed(tmp_path, LAUNCH_ERRORS)


def test_which_buffers_a_call_is_refused_for(tmp_path):
    run_stubbed(tmp_path, BUFFERS)
