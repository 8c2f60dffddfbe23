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


LONG = [9217, 5] + [1500] * 8 + [8704] + [600] * 6 + [0, 31, 7000]   # one past a multiple of the pieces of 512, a multiple; empty and short ones between
SLOT = 32 * 2 * 128 * 129 * 4                                         # bytes of a state slot and its decays, 32 heads of 128
LISTS = 2048                                                          # of the batch LONG


@pytest.mark.parametrize("gate,preact", [("bf16", True), ("f32", False), ("bf16", False)])
def test_long_ones_from_zero_states(gate, preact):
    """States that are zero by contract hold NaN on entry: a cut sequence's first segment starts from registers, the others from slots."""
    p = Packed(LONG, 32, 128, gate, preact)
    got, whole = (p.call(zero_init=True, segments=n) for n in (0, 1))
    empty = LONG.index(0)
    assert all(bool(s[p.slots[empty]].isnan().all()) for s in (*got[1:], *whole[1:]))   # no token: left as it is
    for s in (*got[1:], *whole[1:]):
        s[p.slots[empty]] = 0
    p.compare(got, whole, [0, 10, 19])


@pytest.mark.parametrize("take,cut", [([10, 19, 2, 3, 4, 0, 5, 6, 7, 8, 9, 17, 18, 1, 11, 12, 13, 14], [0, 1, 5]),
                                      ([21, 10, 2, 3, 4, 0, 5, 6, 7, 17, 18, 1, 11, 12], [1, 5])])
def test_long_ones_among_the_sequences_that_take_part(take, cut):
    p = Packed(LONG + [300, 200], 32, 128, preact=True, take=take)
    p.compare(p.call(), p.call(segments=1), cut)


@pytest.mark.parametrize("slots,cut", [(2, []), (6, []), (9, [0, 10]), (12, [0, 10]), (14, [0, 10, 19]), (27, [0, 10, 19])])
def test_long_ones_in_a_buffer_of_few_slots(slots, cut):
    """The device keeps to the slots there are: longer segments, fewer sequences, or none cut; nothing is written past the buffer."""
    p = Packed(LONG, 32, 128, preact=True)
    assert p.ask() > LISTS + 27 * SLOT
    p.compare(p.call(buffer=LISTS + slots * SLOT + 192), p.call(segments=1), cut)   # (192: not the buffer's whole)


def test_long_ones_with_a_loose_bound():
    """None is long: the lists say so, the pre-pass and the scan do nothing."""
    p = Packed([1858] * 20, 32, 128, preact=True)
    p.compare(p.call(max_T=8192), p.call(segments=1), [])
