"""Timed cases of the attention path through the package's public entry points.

Every case is one call sequence a program makes: a forward (evaluation, or the
recomputation of activation checkpointing), a forward plus backward (a training
step's attention, through the plain functions or through autograd), the same
over packed sequences, new queries appended to long key runs, and the FP32
baseline.  `kind` says which:

  fwd     attn_fwd                                  -> O, LSE
  step    attn_fwd, attn_bwd                        -> O, LSE, dQ, dK, dV
  grad    attention under autograd                  -> O, dQ, dK, dV
  packed  attention_varlen under autograd           -> O, dQ, dK, dV
  append  attn_fwd_varlen, few queries, many keys   -> O, LSE
  fp32    fp32_attn                                 -> O, LSE, dQ, dK, dV
"""
from __future__ import annotations

import math
import random

import torch

import paper_2609_34272_amd as gpa


def listed():
    return [
        # The smallest step in use: one head of one short sequence.  Launches
        # and host time decide it.
        dict(name="tiny_step", kind="step", B=1, H=1, Hkv=1, N=128, d=64, causal=True,
             mode="gproj", kbias=8.0, do_std=1.0),
        # Fine-tuning on short texts: many heads, sequences of a few tiles with
        # a ragged end, through autograd.
        dict(name="short_grad", kind="grad", B=8, H=16, Hkv=16, N=500, d=64, causal=True,
             mode="gproj", kbias=4.0, do_std=0.01),
        # The reference training layer: one causal sequence, 16 heads.
        dict(name="h16_n4096_d64_step", kind="step", B=1, H=16, Hkv=16, N=4096, d=64,
             causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # The same layer with wide heads.
        dict(name="h16_n4096_d128_step", kind="step", B=1, H=16, Hkv=16, N=4096, d=128,
             causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # Long-sequence training.
        dict(name="h16_n16384_d64_step", kind="step", B=1, H=16, Hkv=16, N=16384, d=64,
             causal=True, mode="gproj", kbias=8.0, do_std=0.01),
        # The largest: a batch of long sequences with wide heads.
        dict(name="b8_h32_n8192_d128_step", kind="step", B=8, H=32, Hkv=32, N=8192, d=128,
             causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # A decoder layer with grouped-query heads under autograd, query
        # correction only.
        dict(name="gqa_h16kv4_n4096_d64_grad", kind="grad", B=1, H=16, Hkv=4, N=4096, d=64,
             causal=True, mode="gproj_q", kbias=4.0, do_std=0.01),
        # An encoder layer: no causal mask, odd length, uncorrected backward.
        dict(name="encoder_n577_plain", kind="grad", B=8, H=12, Hkv=12, N=577, d=64,
             causal=False, mode="plain", kbias=0.0, do_std=0.01),
        # Evaluation of a long sequence on one GPU of a group that shares the
        # heads: few heads, many tiles each.
        dict(name="shard_h4_n8192_d128_fwd", kind="fwd", B=1, H=4, Hkv=4, N=8192, d=128,
             causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # Training on packed documents of uneven lengths, grouped heads.
        dict(name="packed_h16kv4_d128", kind="packed", nseq=12, H=16, Hkv=4, maxlen=3000, lens=11,
             d=128, causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # A few new tokens per sequence attending to its long past.
        dict(name="append_h16kv4_d128", kind="append", nseq=8, H=16, Hkv=4, newq=4, maxlen=6000,
             lens=5, d=128, causal=True, mode="gproj", kbias=4.0, do_std=0.01),
        # The FP32 baseline on the reference layer.
        dict(name="fp32_h16_n4096_d64", kind="fp32", B=1, H=16, Hkv=16, N=4096, d=64,
             causal=True, mode="plain", kbias=4.0, do_std=0.01),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: the same kinds, sizes over the
    logarithm of their range (mostly odd ones), bounded well below the largest
    listed case."""
    kind = rng.choice(["fwd", "step", "step", "grad", "grad", "packed", "append", "fp32"])
    d = rng.choice([64, 128])
    kv = rng.choice([1, 2, 4, 8])
    G = 1 if kind == "fp32" else rng.choice([1, 1, 2, 4])
    mode = rng.choice(["plain", "gproj_q", "gproj", "gproj"])
    c = dict(kind=kind, H=kv * G, Hkv=kv, d=d, causal=rng.random() < 0.75, mode=mode,
             kbias=0.0 if mode == "plain" else rng.choice([1.0, 4.0, 8.0]),
             do_std=rng.choice([0.01, 1.0]))
    if kind in ("packed", "append"):
        c["nseq"] = rng.randint(2, 24)
        c["maxlen"] = _log_int(rng, 256, 8192)
        c["lens"] = rng.randrange(1 << 20)
        if kind == "append":
            c["newq"] = _log_int(rng, 1, 128)
            c["causal"] = True
    else:
        c["N"] = _log_int(rng, 64, 8192)
        top = 8.0e10 if kind == "fp32" else 1.2e12
        most = top / (2.0 * c["H"] * c["N"] * c["N"] * d)
        c["B"] = max(1, min(_log_int(rng, 1, 32), int(most)))
    return c


# ------------------------------------------------------------------- sizes
def _lengths(case):
    """Query and key counts of the packed sequences of a case."""
    r = random.Random(case["lens"])
    lens = [_log_int(r, max(1, case["maxlen"] // 16), case["maxlen"]) for _ in range(case["nseq"])]
    if case["kind"] == "append":
        return [min(case["newq"], n) for n in lens], lens
    return lens, lens


def _problems(case):
    """(batches, queries, keys) of the attention problems, per head."""
    if case["kind"] in ("packed", "append"):
        return [(1, a, b) for a, b in zip(*_lengths(case))]
    return [(case["B"], case["N"], case["N"])]


def _pairs(nq, nk, causal):
    if not causal:
        return nq * nk
    off = nk - nq  # >= 0 in every case: query i sees keys 0 .. i + off
    return nq * off + nq * (nq + 1) // 2


def work(case):
    H, Hkv, d, kind = case["H"], case["Hkv"], case["d"], case["kind"]
    pairs = H * sum(b * _pairs(nq, nk, case["causal"]) for b, nq, nk in _problems(case))
    rq = H * sum(b * nq for b, nq, nk in _problems(case))
    rk = Hkv * sum(b * nk for b, nq, nk in _problems(case))
    # Products of the forward (Q K^T, P V) and of each backward beyond them:
    # Q K^T, dO V^T, t K, t^T Q, r^T dO; r K with the query correction and r^T z
    # with the key correction.
    products = {"plain": 5, "gproj_q": 6, "gproj": 7}[case["mode"]]
    if kind in ("fwd", "append"):
        return {"bytes": 2 * d * (2 * rq + 2 * rk) + 4 * rq, "flops": 2 * d * pairs * 2}
    # read Q, K, V, dO; write O, LSE, dQ, dK, dV
    return {"bytes": 2 * d * (4 * rq + 4 * rk) + 4 * rq, "flops": 2 * d * pairs * (2 + products)}


# ------------------------------------------------------------------ inputs
def _inputs(case, seed):
    """Q, dO [.., rows, d] and K, V on the GPU: unit normal rows, a common
    per-channel bias on every key of a head (what training drives keys to),
    and upstream gradients of the case's scale."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    H, Hkv, d = case["H"], case["Hkv"], case["d"]
    if case["kind"] in ("packed", "append"):
        nq, nk = _lengths(case)
        sq, sk = (H, sum(nq), d), (Hkv, sum(nk), d)
    else:
        sq, sk = (case["B"], H, case["N"], d), (case["B"], Hkv, case["N"], d)

    def normal(shape, std=1.0, bias=0.0):
        x = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        for i in range(shape[0]):  # one slice at a time: the FP32 draw stays small
            f = torch.randn(shape[1:], generator=g, device="cuda") * std
            if bias:
                b = torch.randn(shape[1:-2] + (1, d), generator=g, device="cuda") * bias
                f += b
            x[i] = f
        return x

    return (normal(sq), normal(sk, 1.0, case["kbias"]), normal(sk), normal(sq, case["do_std"]))


def _offsets(lens):
    return torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32)


def prepare(case, seed):
    q, k, v, do = _inputs(case, seed)
    st = dict(case=case, q=q, k=k, v=v, do=do)
    if case["kind"] in ("packed", "append"):
        nq, nk = _lengths(case)
        st.update(cu_q=_offsets(nq).cuda(), cu_k=_offsets(nk).cuda(), max_q=max(nq), max_k=max(nk))
    if case["kind"] in ("grad", "packed"):
        for n in ("q", "k", "v"):
            st[n].requires_grad_(True)
    return st


def run(st):
    c = st["case"]
    q, k, v, do = st["q"], st["k"], st["v"], st["do"]
    kind, causal, mode = c["kind"], c["causal"], c["mode"]
    if kind == "fwd":
        return gpa.attn_fwd(q, k, v, causal)
    if kind == "step":
        o, lse = gpa.attn_fwd(q, k, v, causal)
        return (o, lse) + gpa.attn_bwd(q, k, v, o, lse, do, mode, causal)
    if kind == "grad":
        o = gpa.attention(q, k, v, causal, mode=mode)
        return (o.detach(),) + torch.autograd.grad(o, (q, k, v), do)
    if kind == "packed":
        o = gpa.attention_varlen(q, k, v, st["cu_q"], st["max_q"], causal, mode=mode)
        return (o.detach(),) + torch.autograd.grad(o, (q, k, v), do)
    if kind == "append":
        return gpa.attn_fwd_varlen(q, k, v, st["cu_q"], st["max_q"], causal,
                                   cu_seqlens_k=st["cu_k"], max_seqlen_k=st["max_k"])
    return gpa.fp32_attn(q, k, v, do, causal)


# ------------------------------------------------------------ what is right
def tolerance(case):
    # BF16 operands and results: 0.16 % (one output cast) to 0.25 % (casts of
    # P, t and the output) from the FP64 result; four times that.
    return {"rel": 6.6e-3 if case["kind"] == "fp32" else 1.0e-2}


def _exact_heads(q, k, v, do, causal):
    """FP64 attention and its gradients for heads [n, Nq, d] x [n, Nk, d]."""
    nq, nk, d = q.shape[1], k.shape[1], q.shape[2]
    a = 1.0 / math.sqrt(d)
    s = torch.matmul(q, k.transpose(1, 2)) * a
    if causal:
        i = torch.arange(nq, device=q.device)[:, None]
        j = torch.arange(nk, device=q.device)[None, :]
        s.masked_fill_(j > i + (nk - nq), -math.inf)
    lse = torch.logsumexp(s, dim=2)
    p = torch.exp(s.sub_(lse[:, :, None]))
    o = torch.matmul(p, v)
    if do is None:
        return o, lse, None, None, None
    dv = torch.matmul(p.transpose(1, 2), do)
    # centred upstream products: the row sum of dS is zero by construction
    ds = torch.matmul(do, v.transpose(1, 2)).sub_((do * o).sum(2, keepdim=True)).mul_(p).mul_(a)
    return o, lse, torch.matmul(ds, k), torch.matmul(ds.transpose(1, 2), q), dv


def exact(case, seed):
    H, Hkv, d, kind, causal = (case[n] for n in ("H", "Hkv", "d", "kind", "causal"))
    G = H // Hkv
    q, k, v, do = _inputs(case, seed)
    if kind in ("fwd", "append"):
        do = None
    packed = kind in ("packed", "append")
    if packed:
        nq, nk = _lengths(case)
        cq, ck = _offsets(nq).tolist(), _offsets(nk).tolist()
        blocks = [(slice(cq[s], cq[s + 1]), slice(ck[s], ck[s + 1])) for s in range(len(nq))]
        q, k, v = q[None], k[None], v[None]
        do = None if do is None else do[None]
    else:
        blocks = [(slice(None), slice(None))]
    B = q.shape[0]

    def new(x):
        return torch.zeros(x.shape, dtype=torch.float64, device="cuda")

    o, lse = new(q), torch.zeros(q.shape[:3], dtype=torch.float64, device="cuda")
    dq, dk, dv = (None, None, None) if do is None else (new(q), new(k), new(v))
    for rq, rk in blocks:
        for b in range(B):
            n = q[0, 0, rq].shape[0] * k[0, 0, rk].shape[0]
            step = max(1, min(H, (1 << 28) // n))
            for h0 in range(0, H, step):
                hs = list(range(h0, min(H, h0 + step)))
                kv = [h // G for h in hs]
                r = _exact_heads(q[b, hs, rq].double(), k[b, kv][:, rk].double(),
                                 v[b, kv][:, rk].double(),
                                 None if do is None else do[b, hs, rq].double(), causal)
                for i, h in enumerate(hs):
                    o[b, h, rq], lse[b, h, rq] = r[0][i], r[1][i]
                    if do is not None:
                        dq[b, h, rq] = r[2][i]
                        dk[b, kv[i], rk] += r[3][i]
                        dv[b, kv[i], rk] += r[4][i]
                del r
    if packed:
        o, lse = o[0], lse[0]
        if do is not None:
            dq, dk, dv = dq[0], dk[0], dv[0]
    if kind in ("fwd", "append"):
        return o, lse
    if kind in ("grad", "packed"):
        return o, dq, dk, dv
    return o, lse, dq, dk, dv
