"""The FP32 baseline's products on the bf16 matrix cores: BF16 inputs exactly,
FP32 factors as three BF16 parts.  Its results against FP64, at tile edges and
remainders, within a bound that BF16 factors would break; sums that cancel, within a
bound that two-part factors would break; infinities and NaNs."""
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
    # steps; a row's output 6 accumulations per 64 keys.
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


def _two_parts(x):
    """FP32 values cut to two BF16 parts, as a split without its last part gives."""
    x = x.float()
    up = lambda t: (t.contiguous().view(torch.int32) & -65536).view(torch.float32)  # noqa: E731
    hi = up(x)
    return (hi + up(x - hi)).double()


def _cancel(w):
    """BF16 coefficients of three weights whose sum nearly cancels: each takes the
    rest that the ones before it leave, to 8 bits."""
    bf = lambda t: t.to(torch.bfloat16).double()  # noqa: E731
    a = torch.ones_like(w[0])
    b = bf(-w[0] / w[1])
    return torch.stack([a, b, bf(-(w[0] * a + w[1] * b) / w[2])])


def _check_cancelled(name, got, coef, w):
    """Sums of three products of FP32 weights w with BF16 coefficients.  A weight here
    is off by 16 roundings of itself at most: P by 3 of the logit (below 1/4) and the
    exponent, 2 of exp2, 4 of l, 1/l and their product; dS by those, one each of its
    difference and product and, dP being exact and |D| below |dP|/2, 4 of D.  The sum
    adds three and the cast.  Two-part weights are off by up to 2^-16 of themselves."""
    exact, scale_of = (coef * w).sum(0), (coef * w).abs().sum(0)
    tol = 16 * 2.0 ** -24 * scale_of + 2.0 ** -8 * exact.abs()
    two = ((coef * _two_parts(w)).sum(0) - exact).abs()
    assert (two > tol).double().mean() >= 0.4, name  # the bound tells them apart
    assert ((got.double().cpu() - exact).abs() <= tol).all(), name


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [96, 191])
def test_no_part_of_an_fp32_factor_is_lost(gpa, N, d, causal):
    """Outputs whose terms cancel to about 2^-18 of themselves: O and dV (the factor
    P), dQ and dK (the factor dS).  Logits depend on the first d/2 channels only: in the
    next d/4 K is 0 and in the last d/4 Q is, so the other's values there are free."""
    g = torch.Generator().manual_seed(N + d)
    r = lambda: torch.randn(N, d, generator=g)  # noqa: E731
    h, n = d // 2, d // 4
    scale = float(np.float32(1 / math.sqrt(d)))
    q, k = (0.25 * r()).to(torch.bfloat16), (0.25 * r()).to(torch.bfloat16)
    q[:, h:], k[:, h:] = 0, 0
    s = q.double() @ k.double().T * scale
    assert s.abs().max() < 0.25
    if causal:
        s.masked_fill_(torch.ones(N, N, dtype=torch.bool).triu(1), -math.inf)
    p = torch.softmax(s, 1)
    keys, rows = [0, n // 2, n - 1], [n, N // 2, N - 1]  # every target sees / is seen by them
    targets = torch.arange(n)
    late = N - 1 - targets  # queries that see all of `keys`

    def call(q, k, v, u):
        out = _call(gpa, *(t.to(torch.bfloat16)[None, None].cuda() for t in (q, k, v, u)), causal, scale)
        return [t[0, 0] for t in out]

    # O[late, c] = sum over `keys` of P V; dV[c, c] = sum over `rows` of P^T dO
    v, u = torch.zeros(N, d).double(), torch.zeros(N, d).double()
    wo, wv = p[late][:, keys].T, p[rows][:, targets]
    co, cv = _cancel(wo), _cancel(wv)
    v[keys, :n], u[rows, :n] = co, cv
    o32, o, _, _, _, dv = call(q, k, v, u)
    _check_cancelled("O", o32[late, targets], co, wo)
    _check_cancelled("dV", dv[targets, targets], cv, wv)

    # dK[c, h + c] = sum over `rows` of dS^T Q; dQ[late, h + n + c] over `keys` of dS K
    # (dO and V in one channel, V of alternating sign and 1 to 2 in size: D stays small beside
    # every dP)
    v, u = torch.zeros(N, d).double(), torch.zeros(N, d).double()
    v[:, 0] = ((1 + torch.rand(N, generator=g)) * (-1.0) ** torch.arange(N)).to(torch.bfloat16).double()
    u[:, 0] = (0.5 + torch.rand(N, generator=g)).to(torch.bfloat16).double()
    assert (p @ v)[n:, 0].abs().max() < 0.5
    ds = p * (u @ v.T - (u * (p @ v)).sum(1, keepdim=True)) * scale
    wk, wq = ds[rows][:, targets], ds[late][:, keys].T
    ck, cq = _cancel(wk), _cancel(wq)
    q2, k2 = q.double(), k.double()
    q2[rows, h:h + n], k2[keys, h + n:] = ck, cq
    _, _, _, dq, dk, _ = call(q2, k2, v, u)
    _check_cancelled("dK", dk[targets, h + targets], ck, wk)
    _check_cancelled("dQ", dq[late, h + n + targets], cq, wq)


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
