"""The FP32 baseline's products on the bf16 matrix cores: BF16 inputs exactly,
FP32 factors as three BF16 parts.  Its FP32 results against FP64, at tile edges
and remainders, within a bound that BF16 or two-part factors would break."""
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


def _call(gpa, q, k, v, u, causal, scale):
    """fp32_attn through the C entry point, with the FP32 output its workspace
    begins with."""
    B, H, N, d = q.shape
    nb = gpa.fp32_attn_workspace_bytes(B, H, N, d)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    o, dq, dk, dv = (torch.empty_like(q) for _ in range(4))
    lse = torch.empty((B, H, N), device="cuda")
    rc = gpa.lib().gpa_fp32_attn(q.data_ptr(), k.data_ptr(), v.data_ptr(), u.data_ptr(),
                                 o.data_ptr(), lse.data_ptr(), dq.data_ptr(), dk.data_ptr(),
                                 dv.data_ptr(), B, H, N, d, int(causal), scale, ws.data_ptr(), nb,
                                 torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    return ws[:4 * o.numel()].view(torch.float32).view(o.shape), o, lse, dq, dk, dv


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 128, 191, 257, 448])
def test_fp32_results_against_fp64(gpa, N, d, causal):
    g = torch.Generator().manual_seed(N * d)
    r = lambda: torch.randn(1, 2, N, d, generator=g)  # noqa: E731
    kb = 4 * torch.randn(1, 2, 1, d, generator=g)
    q, k, v, u = (x.to(torch.bfloat16).cuda() for x in (r(), r() + kb, r(), r()))
    scale = float(np.float32(1 / math.sqrt(d)))
    o32, o, lse, dq, dk, dv = _call(gpa, q, k, v, u, causal, scale)
    Q, K, V, U = (t.double().cpu() for t in (q, k, v, u))
    s = Q @ K.transpose(-1, -2) * scale
    if causal:
        s.masked_fill_(torch.ones(N, N, dtype=torch.bool).triu(1), -math.inf)
    l64 = torch.logsumexp(s, -1)
    p = torch.exp(s - l64[..., None])
    o64 = p @ V
    ds = p * (U @ V.transpose(-1, -2) - (U * o64).sum(-1, keepdim=True))
    # FP32 sums: each logit carries the rounding of its d products, bounded by
    # d/32 accumulations of terms no larger than |q||k|, and the exponent's two
    # steps; a row's output 6 accumulations per 64 keys.  Two BF16 parts instead
    # of three would add 2^-17, above it for every size here.
    logit = scale * (Q.norm(dim=-1).max() * K.norm(dim=-1).max()).item()
    eps = 2.0 ** -24
    tol = eps * (logit * (d / 32 + 4) + 6 * (N / 64 + 1))
    rel = lambda a, b: ((a.double().cpu() - b).norm() / b.norm()).item()  # noqa: E731
    assert rel(o32, o64) <= tol
    assert (lse.double().cpu() - l64).abs().max().item() <= tol
    # BF16 results: the cast (2^-9 per value) and the FP32 error of the sums
    for name, a, b in (("O", o, o64), ("dQ", dq, ds @ K * scale),
                       ("dK", dk, ds.transpose(-1, -2) @ Q * scale), ("dV", dv, p.transpose(-1, -2) @ U)):
        if N > 1 or name in ("O", "dV"):
            assert rel(a, b) <= 2.0 ** -9 + 8 * tol, name


def test_non_finite_inputs_reach_what_depends_on_them(gpa):
    """An infinity or NaN in V or dO leaves the outputs that do not depend on it
    as they were and makes those that do non-finite."""
    N, d = 200, 64
    g = torch.Generator().manual_seed(5)
    x = [torch.randn(1, 2, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(4)]
    base = _call(gpa, *x, True, 0.125)
    for bad in (math.inf, math.nan):
        for which, row in ((2, 70), (3, 150)):  # V row 70, dO row 150 of head 1
            y = [t.clone() for t in x]
            y[which][0, 1, row, 3] = bad
            out = _call(gpa, *y, True, 0.125)
            for a, b in zip(base, out):
                assert torch.equal(a[0, 0], b[0, 0])  # the other head
            _, o, _, dq, dk, dv = (t[0, 1] for t in out)
            if which == 2:
                assert not torch.isfinite(o[row:, 3].float()).any()
                assert torch.equal(o[:64], base[1][0, 1, :64])  # tiles before it
            else:
                assert torch.equal(o, base[1][0, 1])
                assert not torch.isfinite(dv[:row + 1, 3].float()).any()
                assert not torch.isfinite(dq[row].float()).any()
                assert torch.equal(dk[192:], base[4][0, 1, 192:])  # keys no such query sees


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_an_infinity_stays_one(gpa, d, causal, sign):
    """P V and P^T dO with an infinite V or dO are infinite where P > 0, as an FP32
    product is (zero BF16 parts of P must not make NaNs of them): rows outside the
    infinity's own tile, where no masked probability meets it."""
    N, row = 200, 70
    g = torch.Generator().manual_seed(6)
    x = [torch.randn(1, 2, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(4)]
    # equal keys: uniform P, whose last two parts are 0 for a power of two of them
    x[1][0, 1] = 0
    base = _call(gpa, *x, causal, 0.125)
    x[2][0, 1, row, 3] = sign * math.inf
    _, o, lse, *_ = _call(gpa, *x, causal, 0.125)
    assert (o[0, 1, 128 if causal else 0:, 3].float() == sign * math.inf).all()
    keep = torch.arange(d, device="cuda") != 3
    assert torch.equal(o[0, 1][:, keep], base[1][0, 1][:, keep]) and torch.equal(lse, base[2])
    x[2][0, 1, row, 3] = 1.0
    x[3][0, 1, row, 3] = sign * math.inf
    _, o, lse, dq, dk, dv = _call(gpa, *x, causal, 0.125)
    assert (dv[0, 1, :64 if causal else N, 3].float() == sign * math.inf).all()
    assert torch.equal(dv[0, 1][:, keep], base[5][0, 1][:, keep])
