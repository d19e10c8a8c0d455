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


@pytest.mark.parametrize("Hq,Hkv,d", [(4, 4, 64), (16, 4, 128), (16, 4, 64), (8, 1, 128)])
def test_calls_stay_inside_their_buffers(gpa, Hq, Hkv, d):
    """O, LSE and a workspace of exactly the reported size between guard regions,
    with the workspace full of NaN bytes: guards intact, every row of O and LSE
    written, the bits of a call with a zeroed workspace."""
    sel = list(range(len(RUNS)))
    p = Pack(RUNS, Hq, Hkv, d, 77)
    q, k, v, cu, mq, ck, mk = p.args(sel)
    L, guard = gpa.lib(), 4096
    shape = (len(sel), q.shape[1], k.shape[1], Hq, Hkv, mq, mk, d)
    n = {"O": 2 * q.numel(), "LSE": 4 * Hq * q.shape[1],
         "workspace": L.gpa_attn_fwd_varlen_workspace_bytes(*shape)}
    assert n["workspace"] > 0
    for causal in (True, False):
        want = p.run_c(gpa, sel, causal, torch.zeros(n["workspace"], dtype=torch.uint8, device="cuda"))
        buf = {name: torch.full((b + 2 * guard,), 0xA5, dtype=torch.uint8, device="cuda")
               for name, b in n.items()}
        for name, b in n.items():
            buf[name][guard:guard + b] = 0xFF
        at = {name: b.data_ptr() + guard for name, b in buf.items()}
        rc = L.gpa_attn_fwd_varlen_ws(
            q.data_ptr(), k.data_ptr(), v.data_ptr(), at["O"], at["LSE"], cu.data_ptr(),
            ck.data_ptr(), *shape, int(causal), 1 / math.sqrt(d), at["workspace"], n["workspace"],
            torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        torch.cuda.synchronize()
        for name, b in buf.items():
            assert (b[:guard] == 0xA5).all() and (b[guard + n[name]:] == 0xA5).all(), name
        o = buf["O"][guard:guard + n["O"]].view(torch.bfloat16).view(q.shape)
        lse = buf["LSE"][guard:guard + n["LSE"]].view(torch.float32).view(q.shape[:2])
        for s, (a, b) in p.split(o, lse, sel).items():
            assert not torch.isnan(a.float()).any() and not torch.isnan(b).any(), s
            assert torch.equal(a, want[s][0]) and torch.equal(b, want[s][1]), s


@pytest.mark.parametrize("value", [math.nan, math.inf, -math.inf])
@pytest.mark.parametrize("which", ["Q", "K", "V"])
def test_non_finite_inputs_reach_what_depends_on_them(gpa, which, value):
    """In one query, or in one early key of one key/value head, of a split sequence:
    the outputs that depend on it are not finite, and those of the other queries or
    heads and of the other sequences keep their bits."""
    p = Pack([(4, 3000), (20, 5000), (2, 100)], 8, 2, 64, 5)
    sel = [0, 1, 2]
    want = p.run(gpa, sel, True)
    x = p.parts[1]["QKV".index(which)]
    if which == "Q":
        x[3, 7, 5] = value
    else:
        x[1, 100, 5] = value
    got = p.run(gpa, sel, True)
    for s in (0, 2):
        assert all(torch.equal(a, b) for a, b in zip(want[s], got[s]))
    (o, lse), (o1, lse1) = want[1], got[1]
    hit = torch.zeros(8, 20, dtype=torch.bool, device="cuda")
    if which == "Q":
        hit[3, 7] = True
    else:
        hit[4:] = True  # the heads of the group see key 100
    assert torch.equal(o[~hit], o1[~hit]) and torch.equal(lse[~hit], lse1[~hit])
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    bad = ~torch.isfinite(o1.float())
    if which == "V":  # the column alone, and not the LSE
        assert bad[hit][:, 5].all() and torch.equal(lse, lse1)
        bad[..., 5] = False
        assert not bad.any()
    elif which == "Q" or math.isnan(value):
        assert bad[hit].all()
        assert not torch.isfinite(lse1[hit]).any()
    else:  # an infinite key: logits of either sign, +inf gives no finite result
        logit = p.parts[1][0][4:, :, 5].float() * value
        assert bad[4:][logit > 0].all()
        assert torch.isfinite(o1[4:][logit < 0].float()).all()


def test_captured_in_a_graph(gpa):
    p = Pack([(4, 3000), (1, 300), (40, 2000), (300, 300)], 8, 2, 128, 9)
    q, k, v, cu, mq, ck, mk = p.args([0, 1, 2, 3])

    def step():
        return gpa.attn_fwd_varlen(q, k, v, cu, mq, True, cu_seqlens_k=ck, max_seqlen_k=mk)

    ref = [t.clone() for t in step()]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = step()
    noise = torch.randn(1 << 18, device="cuda")
    for _ in range(3):
        noise.mul_(0.9999).sum()
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref))
