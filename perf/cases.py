"""Timing cases of the library: the calls a serving program makes, from one decoding request to a batch of long prompts.

A case is a dict of plain values.  `prepare` makes what a program has in hand before the call (inputs, states, weights,
workspace, descriptor), `run` is one pass through the public entry points, `work` the bytes and operations that pass
cannot do without.  Sizes are those of workloads.py and serving_step.py (a Llama-2-7B attention layer: 32 heads of
width 128, model width 4096), and odd ones between them.

The kinds of calls:
  decode       one token for B sequences (dsla_decode), or for B requests picked from a pool of states and a larger
               batch of rows (dsla_decode_slots)
  prefill      B prompts of T tokens (dsla_prefill), from zero states or continuing from states carried in
  packed       prompts of different lengths back to back, states in a pool (dsla_prefill_varlen)
  project      the projections in front of a layer (dsla_project): q, k, v and two gate pre-activations
  attn_prefill causal softmax attention over a prompt, a layer that has not been converted (dsla_attention_prefill)
  attn_decode  its decode step over a key/value cache, requests at different context lengths (dsla_attention_decode)
"""
import math

import torch

import paper_2506_09316_amd as dsla
from paper_2506_09316_amd.binding import DSLA_BF16, DSLA_F32

TAU = 16.0   # temperature of the gates

# prompt lengths of a mixed batch as a serving system sees it: a few long ones, many short ones, some of a few tokens
SERVING_MIX = "8192,6000,5000,4100,3000,2500,2048,1500,1200,1000,800,600,512,300,200,100,64,33,7,1"


def listed():
    return [
        # an interactive user: one sequence, one token; latency and the host's share count
        dict(name="decode_b1", kind="decode", B=1, H=32, d=128, io="bf16", gates="log", pool=0),
        # a full batch of decoding sequences; the states (270 MB) are the traffic
        dict(name="decode_b64", kind="decode", B=64, H=32, d=128, io="bf16", gates="log", pool=0),
        # the decoding requests of a mixed batch: 37 of 64 pool entries and rows, gates as the projections leave them
        dict(name="decode_pool37", kind="decode", B=37, H=32, d=128, io="bf16", gates="preact", pool=64),
        # the smallest prompt of the configurations, in the fp32 arithmetic a reference run uses
        dict(name="prefill_f32_256", kind="prefill", B=1, T=256, H=4, d=64, io="f32", gates="log", carry=0),
        # the next turn of a conversation: a ragged number of tokens on top of carried states
        dict(name="prefill_1000_carry", kind="prefill", B=1, T=1000, H=32, d=128, io="bf16", gates="preact", carry=1),
        # one long prompt (the headline shape)
        dict(name="prefill_16k", kind="prefill", B=1, T=16384, H=32, d=128, io="bf16", gates="log", carry=0),
        # a batch of long prompts (the hybrid configuration)
        dict(name="prefill_b8_8k", kind="prefill", B=8, T=8192, H=32, d=128, io="bf16", gates="log", carry=0),
        # a mixed batch of prompts of different lengths, gates as the projections leave them
        dict(name="packed_serving", kind="packed", lengths=SERVING_MIX, H=32, d=128, io="bf16", gates="preact"),
        # the projections of one layer for a long prompt, and for the tokens of a decoding batch
        dict(name="project_16k", kind="project", M=16384, K=4096, n_out=5, width=4096),
        dict(name="project_b64", kind="project", M=64, K=4096, n_out=5, width=4096),
        # the softmax layers that stand beside the DSLA layers in a partly converted model
        dict(name="attn_prefill_b8_8k", kind="attn_prefill", B=8, T=8192, H=32, d=128),
        dict(name="attn_decode_b8_8k", kind="attn_decode", B=8, T=8192, H=32, d=128, io="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "prefill", "prefill", "packed", "project", "attn_prefill", "attn_decode"])
    H, d = rng.choice([(32, 128), (32, 128), (32, 128), (8, 128), (32, 64), (4, 64)])
    io = "f32" if rng.random() < 0.15 else "bf16"
    gates = rng.choice(["log", "preact"])
    if kind == "decode":
        B = _log_int(rng, 1, 64)
        return dict(kind=kind, B=B, H=H, d=d, io=io, gates=gates, pool=rng.choice([0, B + rng.randrange(1, 30)]))
    if kind == "prefill":
        # at most the tokens of the largest listed prefill; fp32 prompts are short
        B = _log_int(rng, 1, 8)
        T = _log_int(rng, 17, 2048 if io == "f32" else 65536 // B if B > 4 else 16384)
        return dict(kind=kind, B=B, T=T, H=H, d=d, io=io, gates=gates, carry=rng.randrange(2))
    if kind == "packed":
        n, longest = rng.randrange(2, 41), _log_int(rng, 64, 8192)
        lengths = [_log_int(rng, 1, longest) for _ in range(n)]
        return dict(kind=kind, lengths=",".join(str(x) for x in lengths), H=H, d=d, io="bf16", gates=gates)
    if kind == "project":
        return dict(kind=kind, M=_log_int(rng, 1, 16384), K=rng.choice([512, 1024, 2048, 4096, 4096]),
                    n_out=rng.choice([3, 5, 5]), width=rng.choice([512, 1024, 4096, 4096]))
    if kind == "attn_prefill":
        B = _log_int(rng, 1, 8)
        return dict(kind=kind, B=B, T=_log_int(rng, 33, 8192), H=H, d=d)
    return dict(kind=kind, B=_log_int(rng, 1, 8), T=_log_int(rng, 100, 8192), H=H, d=d, io=io)


# ---------------------------------------------------------------------------------------------------------------
def _type(io):
    return (torch.bfloat16, DSLA_BF16, 2) if io == "bf16" else (torch.float32, DSLA_F32, 4)


class _Draw:
    """Normal values on the GPU from one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(1000003 * int(seed) + 17)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
        return torch.empty(*shape, device="cuda", dtype=torch.float32).normal_(mean, std, generator=self.gen).to(dtype)

    def gates(self, *shape, kind, dtype):
        """Pre-activations z ~ N(2, 1), or their log-gates -softplus(-z) / tau."""
        z = self.normal(*shape, mean=2.0, dtype=torch.float32)
        return (z if kind == "preact" else torch.nn.functional.softplus(-z).div_(-TAU)).to(dtype)

    def order(self, n):
        return torch.randperm(n, device="cuda", generator=self.gen)


def _layer_inputs(r, c, *lead):
    dt = _type(c["io"])[0]
    q, k, v = (r.normal(*lead, c["H"], c["d"], std=c["d"] ** -0.5, dtype=dt) for _ in range(3))
    g1, g2 = (r.gates(*lead, c["H"], c["d"], kind=c["gates"], dtype=dt) for _ in range(2))
    return q, k, v, g1, g2


def _desc(c, B, zero_init=False):
    code = _type(c["io"])[1]
    return dsla.make_desc(B, c["H"], c["d"], c["d"], io_dtype=code, gate_dtype=code, gamma=0.4, chunk=64,
                          gate_mode=int(c["gates"] == "preact"), tau=TAU, zero_init=zero_init)


def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def prepare(case, seed):
    c, r = case, _Draw(seed)
    s = dict(case)
    kind = c["kind"]
    if kind == "decode":
        entries = c["pool"] or c["B"]
        s["x"] = _layer_inputs(r, c, entries)
        s["S"] = [r.normal(entries, c["H"], c["d"], c["d"], std=0.3, dtype=torch.float32) for _ in range(2)]
        s["o"] = torch.zeros_like(s["x"][2])
        s["desc"] = _desc(c, c["B"])
        if c["pool"]:
            s["slots"] = r.order(entries)[:c["B"]].to(torch.int32)
            s["rows"] = r.order(entries)[:c["B"]].to(torch.int32)
    elif kind == "prefill":
        s["x"] = _layer_inputs(r, c, c["B"], c["T"])
        s["S"] = [r.normal(c["B"], c["H"], c["d"], c["d"], std=0.3, dtype=torch.float32) for _ in range(2)]
        s["o"] = torch.empty_like(s["x"][2])
        s["desc"] = _desc(c, c["B"], zero_init=not c["carry"])
        s["ws"] = _scratch(dsla.dsla_prefill_workspace_bytes(s["desc"], c["T"]))
    elif kind == "packed":
        lengths = [int(x) for x in c["lengths"].split(",")]
        s["total"], s["longest"] = sum(lengths), max(lengths)
        s["x"] = _layer_inputs(r, c, s["total"])
        s["S"] = [r.normal(len(lengths), c["H"], c["d"], c["d"], std=0.3, dtype=torch.float32) for _ in range(2)]
        s["o"] = torch.empty_like(s["x"][2])
        s["cu"] = torch.tensor([0] + lengths, dtype=torch.int64).cumsum(0).to(torch.int32).cuda()
        s["slots"] = r.order(len(lengths)).to(torch.int32)
        s["desc"] = _desc(c, len(lengths))
        s["ws"] = _scratch(dsla.dsla_prefill_varlen_workspace_bytes(s["desc"], s["total"], s["longest"]))
    elif kind == "project":
        s["x"] = r.normal(c["M"], c["K"])
        s["W"] = r.normal(c["n_out"] * c["width"], c["K"], std=c["K"] ** -0.5)
        s["outs"] = [torch.empty(c["M"], c["width"], device="cuda", dtype=torch.bfloat16) for _ in range(c["n_out"])]
    elif kind == "attn_prefill":
        s["x"] = [r.normal(c["B"], c["T"], c["H"], c["d"]) for _ in range(3)]
        s["o"] = torch.empty_like(s["x"][2])
    else:
        dt = _type(c["io"])[0]
        s["q"] = r.normal(c["B"], c["H"], c["d"], dtype=dt)
        s["kv"] = [r.normal(c["B"], c["T"], c["H"], c["d"], dtype=dt) for _ in range(2)]
        s["lens"] = torch.tensor(_lens(c), dtype=torch.int32).cuda()
        s["o"] = torch.empty_like(s["q"])
        s["ws"] = _scratch(dsla.dsla_attention_decode_workspace_bytes(c["B"], c["H"], c["d"], c["T"]))
    return s


def _lens(c):
    """Context lengths of the requests in a cache of T positions: from a full one down to a bit more than half."""
    return [c["T"] - (b * c["T"]) // (2 * c["B"]) for b in range(c["B"])]


def run(s):
    kind = s["kind"]
    if kind == "decode":
        if s["pool"]:
            dsla.dsla_decode_slots(s["desc"], *s["x"], s["slots"], s["S"][0], s["S"][1], s["o"], row_index=s["rows"])
        else:
            dsla.dsla_decode(s["desc"], *s["x"], s["S"][0], s["S"][1], s["o"])
        return s["o"], s["S"][0], s["S"][1]
    if kind == "prefill":
        dsla.dsla_prefill(s["desc"], s["T"], *s["x"], s["S"][0], s["S"][1], s["o"], s["ws"])
        return s["o"], s["S"][0], s["S"][1]
    if kind == "packed":
        dsla.dsla_prefill_varlen(s["desc"], s["total"], s["longest"], s["cu"], s["slots"], *s["x"], s["S"][0], s["S"][1], s["o"],
                                 s["ws"])
        return s["o"], s["S"][0], s["S"][1]
    if kind == "project":
        dsla.dsla_project(s["x"], s["W"], s["outs"])
        return s["outs"]
    if kind == "attn_prefill":
        dsla.dsla_attention_prefill(*s["x"], s["o"], s["d"] ** -0.5)
        return s["o"]
    dsla.dsla_attention_decode(s["q"], *s["kv"], s["o"], s["d"] ** -0.5, s["ws"], seq_lens=s["lens"])
    return s["o"]


def work(case):
    """Every input read once, every output written once; the operations of the token recurrence (two states, a
    multiply-add per state element for the update and one for the read-out) or of the products."""
    c = case
    kind = c["kind"]
    if kind == "project":
        N = c["n_out"] * c["width"]
        return {"bytes": 2 * (c["M"] * c["K"] + N * c["K"] + c["M"] * N), "flops": 2 * c["M"] * c["K"] * N}
    H, d = c["H"], c["d"]
    if kind == "attn_prefill":
        return {"bytes": 4 * c["B"] * c["T"] * H * d * 2, "flops": 4 * c["B"] * H * d * (c["T"] * (c["T"] + 1) // 2)}
    e = _type(c["io"])[2]
    if kind == "attn_decode":
        keys = sum(_lens(c))
        return {"bytes": 2 * keys * H * d * e + 2 * c["B"] * H * d * e, "flops": 4 * keys * H * d}
    if kind == "decode":
        tokens, sequences, passes = c["B"], c["B"], 2
    elif kind == "prefill":
        tokens, sequences, passes = c["B"] * c["T"], c["B"], 1 + c["carry"]
    else:
        lengths = [int(x) for x in c["lengths"].split(",")]
        tokens, sequences, passes = sum(lengths), len(lengths), 2
    return {"bytes": tokens * H * d * 6 * e + passes * sequences * H * 2 * d * d * 4, "flops": tokens * H * 8 * d * d}


def tolerance(case):
    """About four times the distance from the same path in 64 bits, measured: 2-norm / largest difference

      prefill, packed   bf16 2.9e-3 / 3.4e-2 (operands of the contractions in bf16)     fp32 2.9e-7 / 3.5e-6
      attn_prefill      bf16 2.6e-3 / 5e-2 (the first rows are many times the root mean square of long prompts)
      decode, project, attn_decode   bf16 1.7e-3 / 3.9e-3 (the rounding of the results)  fp32 2.0e-7 / 6.7e-7
    """
    long = case["kind"] in ("prefill", "packed", "attn_prefill")
    if case.get("io") == "f32":
        return {"rel": 1.2e-6, "max": 2e-5} if long else {"rel": 8e-7, "max": 5e-6}
    return {"rel": 1e-2, "max": 0.3} if long else {"rel": 7e-3, "max": 2e-2}
