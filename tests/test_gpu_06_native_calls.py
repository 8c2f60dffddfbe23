"""The calls of a serving loop in native code (_marshal): what they take, and the same results as through ctypes."""
import pytest

import paper_2506_09316_amd as dsla
from paper_2506_09316_amd import binding

pytestmark = pytest.mark.gpu

B, H, D = 2, 4, 64


def randn(*shape, std=1.0, dtype=None, seed=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty(*shape, device="cuda").normal_(0, std, generator=g).to(dtype or torch.bfloat16)


def layer(*lead, seed=7):
    """q, k, v, g1, g2 in bf16, log-gates"""
    qkv = [randn(*lead, H, D, std=D ** -0.5, seed=seed + i) for i in range(3)]
    return qkv + [-0.1 * randn(*lead, H, D, seed=seed + 3 + i).abs() for i in range(2)]


def states(n):
    import torch
    return [randn(n, H, D, D, std=0.3, dtype=torch.float32, seed=20 + i) for i in range(2)]


def desc(n=B):
    return dsla.make_desc(n, H, D, D, io_dtype=1, gate_dtype=1, gamma=0.4, chunk=64)


def ints(*values):
    import torch
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def scratch(n):
    import torch
    return torch.zeros(n, dtype=torch.uint8, device="cuda") if n else None


def test_a_descriptor_is_a_descriptor():
    """Bytes of a descriptor's size are refused, as ctypes refuses them."""
    x, S = layer(B), states(B)
    o = x[2].clone().zero_()
    before = [t.clone() for t in (o, *S)]
    assert binding.load_library() and binding._native.decode(bytes(desc()), *x, *S, o) is None
    with pytest.raises(TypeError):
        dsla.dsla_decode(bytes(desc()), *x, *S, o)
    assert all(bool((a == b).all()) for a, b in zip(before, (o, *S)))
    assert binding._native.decode(desc(), *x, *S, o) == 0


def calls():
    """name -> (arguments of the native call, indexes of what it writes, indexes that may be None, the public call of the same arguments)"""
    import torch
    T, pool, M, K, W = 70, 5, 40, 64, 128
    one, seq, packed, S, P = layer(B), layer(B, T), layer(T, seed=11), states(B), states(pool)
    out = lambda t: torch.zeros_like(t)
    d = desc()
    cut = dsla.make_desc(B, H, D, D, io_dtype=1, gate_dtype=1, gamma=0.4, chunk=32, segments=2)
    ws = scratch(dsla.dsla_prefill_workspace_bytes(cut, T))
    wsv = scratch(dsla.dsla_prefill_varlen_workspace_bytes(cut, T, 50))
    kv = [randn(B, 300, H, D, seed=40 + i) for i in range(2)]
    wsa = scratch(dsla.dsla_attention_decode_workspace_bytes(B, H, D, 300))
    assert ws is not None and wsv is not None and wsa is not None
    rows = layer(pool, seed=13)
    x, w = randn(M, K, seed=50), randn(3 * W, K, std=K ** -0.5, seed=51)
    outs, bias = [torch.zeros(M, W, dtype=torch.bfloat16, device="cuda") for _ in range(3)], randn(3 * W, dtype=torch.float32, seed=52)
    slots, index = ints(3, 1), ints(4, 0)
    return {
        "decode": ((d, *one, *S, out(one[2])), (6, 7, 8), (), dsla.dsla_decode),
        "decode_slots": ((d, *rows, index, slots, *P, out(rows[2])), (8, 9, 10), (6,),
                         lambda d, q, k, v, g1, g2, row, slot, S1, S2, o: dsla.dsla_decode_slots(d, q, k, v, g1, g2, slot, S1, S2, o, row)),
        "prefill": ((cut, T, *seq, *S, out(seq[2]), ws), (7, 8, 9), (), dsla.dsla_prefill),
        "prefill_varlen": ((cut, T, 50, ints(0, 20, T), ints(1, 0), slots, *packed, *P, out(packed[2]), wsv), (11, 12, 13), (4, 5),
                           lambda d, n, m, cu, seq, slot, *a: dsla.dsla_prefill_varlen(d, n, m, cu, slot, *a, seq_index=seq)),
        "attention_decode": ((one[0], *kv, out(one[0]), 0.125, wsa, ints(300, 170)), (3,), (6,), dsla.dsla_attention_decode),
        "attention_prefill": ((*seq[:3], out(seq[2]), 0.125), (3,), (), dsla.dsla_attention_prefill),
        "project": ((x, w, outs, bias), (2,), (3,), dsla.dsla_project),
    }


NAMES = ("decode", "decode_slots", "prefill", "prefill_varlen", "attention_decode", "attention_prefill", "project")


def tensors(value):
    return value if isinstance(value, list) else [value]


@pytest.mark.parametrize("name", NAMES)
def test_native_calls_equal_the_general_way(name, monkeypatch):
    """Bit for bit, with the optional arguments and without; the native call is the one that answers where it is there."""
    import torch
    args, written, optional, public = calls()[name]
    native = binding._native
    assert native is not binding._General
    start = [[t.clone() for t in tensors(args[i])] for i in written]
    for dropped in {(), optional}:
        a = [None if i in dropped else x for i, x in enumerate(args)]
        results = []
        for way in (native, binding._General):
            for i, was in zip(written, start):
                for t, w in zip(tensors(a[i]), was):
                    t.copy_(w)
            monkeypatch.setattr(binding, "_native", way)
            assert getattr(native, name)(*a) == 0 if way is native else public(*a) is None
            torch.cuda.synchronize()
            results.append([t.clone() for i in written for t in tensors(a[i])])
        assert all(torch.equal(x, y) for x, y in zip(*results)), dropped
        assert not torch.equal(results[0][-1], start[-1][-1])   # (something was computed)


@pytest.mark.parametrize("name", NAMES)
def test_native_calls_leave_single_odd_arguments_to_the_general_way(name):
    """Arguments of a call that it takes, one of them replaced by one that it does not: None, nothing pending, nothing written."""
    import torch
    args, written, optional, _ = calls()[name]
    call = getattr(binding._native, name)

    class Sub(torch.Tensor):
        pass

    def odd(i, x):
        if isinstance(x, dsla.DslaDesc):
            return [None, 3, bytes(x), bytearray(bytes(x))]
        if isinstance(x, int):
            return [float(x), str(x), 1 << 70, None, True]
        if isinstance(x, float):
            return [1, "1", None]
        if isinstance(x, list):
            wide = torch.zeros(2 * x[0].numel(), dtype=x[0].dtype, device="cuda")
            return [tuple(x), None, [], x[:2], [*x[:2], x[2].cpu()], [*x[:2], x[2].t()], [*x[:2], wide]]
        wide = torch.stack([x, x], -1)[..., 0]   # strided
        assert not wide.is_contiguous()
        null = i in optional or x.dtype == torch.uint8 or (name, i) == ("decode_slots", 7)   # (what the library itself takes or refuses)
        return [x.cpu(), wide, x.as_subclass(Sub), 5, "x"] + ([] if null else [None])

    before = [t.clone() for i in written for t in tensors(args[i])]
    for i, x in enumerate(args):
        for value in odd(i, x):
            assert call(*args[:i], value, *args[i + 1:]) is None, (i, type(value))
    assert call(*args[:-1]) is None and call() is None
    assert all(torch.equal(a, b) for a, b in zip(before, [t for i in written for t in tensors(args[i])]))
    assert call(*args) == 0


def test_native_calls_take_parameters_and_refuse_by_status():
    """A Parameter is a tensor to them, a status is the library's; the public call raises it."""
    import torch
    x, S = layer(B), states(B)
    o = torch.zeros_like(x[2])
    assert binding._native.decode(desc(), torch.nn.Parameter(x[0]), *x[1:], *S, o) == 0
    bad = dsla.make_desc(B, H, 48, 48, io_dtype=1, gate_dtype=1)
    assert binding._native.decode(bad, *x, *S, o) == 3
    with pytest.raises(dsla.DslaError):
        dsla.dsla_decode(bad, *x, *S, o)
