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
