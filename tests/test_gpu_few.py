"""The forward of packed sequences with few queries on long key runs, whose keys
are split over workgroups: a sequence's O and LSE depend on its own rows alone."""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def gpa():
    import paper_2609_34272_amd as g
    g.lib()
    return g


class Pack:
    """Sequences of (queries, keys) with random Q, K, V."""

    def __init__(self, runs, Hq, Hkv, d, seed):
        g = torch.Generator().manual_seed(seed)
        self.runs, self.Hq, self.Hkv, self.d = list(runs), Hq, Hkv, d
        self.parts = [[torch.randn(h, n, d, generator=g).to(torch.bfloat16).cuda()
                       for h, n in ((Hq, nq), (Hkv, nk), (Hkv, nk))] for nq, nk in self.runs]

    def args(self, sel):
        """q, k, v, query offsets, longest, key offsets, longest of the chosen ones."""
        q, k, v = (torch.cat([self.parts[s][i] for s in sel], 1).contiguous() for i in range(3))
        nq, nk = ([self.runs[s][i] for s in sel] for i in range(2))
        cu, ck = (torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).cuda()
                  for n in (nq, nk))
        return q, k, v, cu, max(nq), ck, max(nk)

    def run(self, gpa, sel, causal):
        q, k, v, cu, mq, ck, mk = self.args(sel)
        o, lse = gpa.attn_fwd_varlen(q, k, v, cu, mq, causal, cu_seqlens_k=ck, max_seqlen_k=mk)
        return self.split(o, lse, sel)

    def run_c(self, gpa, sel, causal, ws):
        """The C entry point with the workspace tensor `ws`, or none."""
        q, k, v, cu, mq, ck, mk = self.args(sel)
        o = torch.full_like(q, math.nan)
        lse = torch.full(q.shape[:2], math.nan, device="cuda")
        rc = gpa.lib().gpa_attn_fwd_varlen_ws(
            q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), cu.data_ptr(),
            ck.data_ptr(), len(sel), q.shape[1], k.shape[1], self.Hq, self.Hkv, mq, mk, self.d,
            int(causal), 1 / math.sqrt(self.d), None if ws is None else ws.data_ptr(),
            0 if ws is None else ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0, gpa.lib().gpa_last_error()
        torch.cuda.synchronize()
        return self.split(o, lse, sel)

    def split(self, o, lse, sel):
        n = [self.runs[s][0] for s in sel]
        return dict(zip(sel, zip(o.split(n, 1), lse.split(n, 1))))


# Queries and keys: 2 to 8 splits, row tiles that end inside a head, a group's rows
# in one tile and in several, key tails, the lines of the rule (512 keys; 64 rows, or
# 16 keys per row; 128 queries) from both sides, no queries, no keys, a dense
# sequence (nq == nk) and a long one.
RUNS = [(1, 512), (1, 511), (4, 5000), (33, 2300), (128, 4097), (129, 3000), (4, 4), (300, 700),
        (0, 2000), (5, 0), (2, 9000), (16, 1023), (17, 900), (16, 1024), (128, 8192), (3, 1300)]


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (16, 4), (8, 1)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
def test_a_sequence_does_not_depend_on_its_companions(gpa, d, Hq, Hkv, causal):
    """Bit for bit the same alone, in packs of different companions, sizes and order,
    and without a workspace."""
    p = Pack(RUNS, Hq, Hkv, d, 10 * Hq + d)
    everything = list(range(len(RUNS)))
    whole = p.run(gpa, everything, causal)
    others = [(sel, p.run(gpa, sel, causal)) for sel in
              [[s] for s in everything if min(RUNS[s])] + [[15, 6, 4, 2, 9], [13, 7, 0, 3], [2, 0]]]
    others += [(everything, p.run_c(gpa, everything, causal, None))]
    for sel, out in others:
        for s in sel:
            for name, a, b in zip(("O", "LSE"), whole[s], out[s]):
                assert torch.equal(a, b), (name, RUNS[s], sel)
    # nq == nk: the dense forward, bit for bit
    q, k, v = (t[None] for t in p.parts[6])
    o, lse = gpa.attn_fwd(q, k, v, causal)
    assert torch.equal(whole[6][0], o[0]) and torch.equal(whole[6][1], lse[0])


def test_without_memory_for_the_workspace_the_bits_are_the_same(gpa, monkeypatch):
    p = Pack([(4, 3000), (4, 600), (1, 200)], 16, 4, 128, 3)
    want = p.run(gpa, [0, 1, 2], True)
    empty, refused = torch.empty, []

    def full(*a, **kw):
        if kw.get("dtype") is torch.uint8:
            refused.append(a)
            raise torch.OutOfMemoryError("no memory")
        return empty(*a, **kw)

    monkeypatch.setattr(torch, "empty", full)
    got = p.run(gpa, [0, 1, 2], True)
    assert refused
    for s in want:
        assert all(torch.equal(a, b) for a, b in zip(want[s], got[s]))
