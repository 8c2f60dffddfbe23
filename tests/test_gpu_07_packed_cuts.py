"""Which sequences of a packed batch are cut, where the device chooses: every one, only the long ones, or none.  Against the same call
whole (segments = 1) and with every sequence cut (the number of segments named), which are held to the oracle elsewhere."""
import numpy as np
import pytest

import paper_2506_09316_amd as dsla
from tests.gpu_common import check
from tests.util import code

pytestmark = pytest.mark.gpu

NONE, ALL = "none", "all"


class Packed:
    """A packed batch on the GPU; every call starts from the same states.  `take`: which sequences take part, in which order."""

    def __init__(self, lengths, H, d, gate="bf16", preact=False, take=None, seed=98):
        import torch
        g = torch.Generator(device="cuda").manual_seed(seed)
        normal = lambda *shape, std=1.0, mean=0.0: torch.empty(*shape, device="cuda").normal_(mean, std, generator=g)
        self.cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
        self.take = list(range(len(lengths))) if take is None else list(take)
        self.lengths, self.total, self.H, self.d, self.gate, self.preact = [lengths[i] for i in self.take], sum(lengths), H, d, gate, preact
        self.x = [normal(self.total, H, d, std=d ** -0.5).bfloat16() for _ in range(3)]
        for _ in range(2):
            z = normal(self.total, H, d, mean=2.0)
            self.x.append((z if preact else torch.nn.functional.softplus(-z).div_(-16)).to(torch.bfloat16 if gate == "bf16" else torch.float32))
        B = len(self.take)
        self.S0 = [normal(B + 1, H, d, d, std=0.3) for _ in range(2)]   # (one entry more than sequences)
        self.slots = list(range(B))[::-1]
        ints = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
        self.index = (torch.from_numpy(self.cu).cuda(), ints(self.slots), None if take is None else ints(self.take))

    def ask(self, max_T=None, **desc):
        return dsla.dsla_prefill_varlen_workspace_bytes(self.describe(**desc), self.total, max_T or max(self.lengths))

    def describe(self, **desc):
        return dsla.make_desc(len(self.take), self.H, self.d, self.d, io_dtype=code("bf16"), gate_dtype=code(self.gate), gamma=0.6, chunk=64,
                              gate_mode=int(self.preact), **desc)

    def call(self, max_T=None, buffer=None, **desc):
        """o, S1, S2; buffer: bytes given to the call (None: as many as it asks for), followed by some that it must leave alone."""
        import torch
        nbytes, guard = self.ask(max_T, **desc) if buffer is None else buffer, 1 << 20
        ws = torch.full((nbytes + guard,), 0xA5, dtype=torch.uint8, device="cuda")
        S = [s.clone() for s in self.S0]
        if desc.get("zero_init"):
            for s in S:
                s[:-1] = float("nan")
        o = torch.full_like(self.x[2], 7.0)
        cu, slots, seq = self.index
        dsla.dsla_prefill_varlen(self.describe(**desc), self.total, max_T or max(self.lengths), cu, slots, *self.x, *S, o, ws[:nbytes] if nbytes else None,
                                 seq_index=seq)
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 0xA5).all())
        assert all(torch.equal(s[-1], s0[-1]) for s, s0 in zip(S, self.S0))   # no sequence's
        return o, *S

    def rows(self, o, b):
        return o[self.cu[self.take[b]]:self.cu[self.take[b] + 1]]

    def compare(self, got, ref, cut):
        """Bit for bit, but for the sequences `cut`: those differ, within the tolerance."""
        import torch
        for b in range(len(self.take)):
            pairs = [(self.rows(got[0], b), self.rows(ref[0], b))] + [(g[self.slots[b]], r[self.slots[b]]) for g, r in zip(got[1:], ref[1:])]
            if b not in cut:
                assert all(torch.equal(g, r) for g, r in pairs), (b, self.lengths[b])
                continue
            assert not torch.equal(*pairs[0]), (b, self.lengths[b])
            for name, (g, r) in zip(("o", "S1", "S2"), pairs):
                check(f"{name}[{b}]", g.float().cpu().numpy(), r.float().cpu().numpy(), 2e-2)
        others = torch.ones(self.total, dtype=torch.bool, device="cuda")
        for b in self.take:
            others[self.cu[b]:self.cu[b + 1]] = False
        assert bool((got[0][others] == 7.0).all())   # rows of sequences that do not take part


def all_cut(p, max_T=None):
    """The call with every sequence cut as the library would: the number of segments that asks for the same buffer."""
    segments = [n for n in range(2, 200) if p.ask(max_T, segments=n) == p.ask(max_T)]
    return p.call(max_T, segments=segments[0])


@pytest.mark.parametrize("lengths,H,d,preact,max_T,chosen", [
    # as many long ones as there are slots for few: cutting all is better than long segments
    ([2922] * 4 + [2500] * 4 + [2000] * 5, 8, 128, True, None, ALL),
    ([6913, 5500, 6913, 6000, 5911, 5200, 5000], 8, 128, True, None, ALL),
    ([4078, 3000, 3900, 2500] * 5 + [4078, 2100], 4, 64, False, None, ALL),
    # the bound is loose, no sequence is long
    ([1430] * 27 + [1769], 8, 128, True, 7076, NONE),
    # pieces of 512 and of 256, several cut and whole ones among them, an empty one and one of a token
    ([3500, 5451] * 3 + [4500] * 6 + [3500] * 4, 8, 128, False, None, [1, 3, 5, 6, 7, 8, 9, 10, 11]),
    ([2773, 2718, 2982, 1241, 27, 961, 532, 1129, 480, 393, 1469, 964, 1108, 1126, 976, 814, 1309, 309, 475, 0, 1], 8, 128, True, None, [0, 1, 2, 3, 7, 10, 12, 13, 16])])
def test_every_sequence_the_long_ones_or_none(lengths, H, d, preact, max_T, chosen):
    p = Packed(lengths, H, d, preact=preact)
    got = p.call(max_T)
    if chosen == ALL:
        p.compare(got, all_cut(p, max_T), [])
    else:
        p.compare(got, p.call(max_T, segments=1), [] if chosen == NONE else chosen)
