"""Kernels that take fp32 queries, probabilities or score gradients to the bf16 matrix cores have to keep all their bits.

Ordinary inputs do not show it: the outputs are bf16, and 16 significant bits of an operand are already finer.  So the
inputs here cancel: large terms of a sum that leave a small result, which is wrong by the terms' lost bits.  Operands of two
bf16 words (16 to 17 bits, an error of up to 2^-18 of every term) fail each of these tests; 24 bits pass with room."""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from paper_2507_00715_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF = torch.bfloat16


def _B():
    from paper_2507_00715_amd import binding
    binding.lib()
    return binding


def i32(x):
    return torch.tensor(list(x), dtype=torch.int32, device=DEV)


def bf16(x):
    """The nearest bf16 values, as float64."""
    return torch.from_numpy(np.asarray(x, dtype=np.float64)).to(BF).double().numpy()


def cancelling(weights, first, keep=4):
    """Rows x_0 .. x_(keep-1) of bf16 values, x_0 = first, such that sum_i weights[i] x_i nearly vanishes: every row takes
    away what the rows before it leave, to 8 bits.  weights [keep, ...]: non-zero."""
    rows, left = [first], weights[0] * first
    for w in weights[1:keep]:
        rows.append(bf16(-left / w))
        left = left + w * rows[-1]
    return np.stack(rows)


def run_decode(q, k, v, kn, vn, n, scale):
    """One decode step, one stream per sequence, no rotation, one free place in the generated cache."""
    B = _B()
    batch, hq, d = q.shape
    hkv = kn.shape[1]
    to = lambda x: torch.from_numpy(x).to(BF).to(DEV)
    desc = B.make_desc(BF, hq, hkv, d, scale, 0.0)
    gk, gv = (torch.zeros(batch, 1, hkv, d, dtype=BF, device=DEV) for _ in range(2))
    out = torch.full((batch, hq, d), float("nan"), dtype=BF, device=DEV)
    ws = torch.empty(max(B.earn_decode_workspace_bytes(desc, batch, batch, n, 1), 256), dtype=torch.uint8, device=DEV)
    B.earn_decode_attn(desc, to(q), to(kn), to(vn), i32([n] * batch), to(k), to(v), i32(range(0, (batch + 1) * n, n)), None,
                       gk, gv, i32([0] * batch), 1, batch, batch, n, out, ws)
    torch.cuda.synchronize()
    return out.cpu().double().numpy()


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (3, 3, 128), (8, 2, 128)])
def test_decode_scores_that_cancel(hq, hkv, d):
    """Two elements of every key cancel in the score (a b - b a, up to 2^13 each) as long as scale * q keeps its bits."""
    n, batch, gq = 40, 4, hq // hkv
    rng = np.random.default_rng(d + hq)
    rnd = lambda *s: bf16(rng.standard_normal(s))
    q, k, v, kn, vn = rnd(batch, hq, d), rnd(batch * n, hkv, d), rnd(batch * n, hkv, d), rnd(batch, hkv, d), rnd(batch, hkv, d)
    # the heads of a group share the keys: their first two elements differ by a power of two
    a, b = bf16(rng.uniform(1, 2, (batch, hkv))), bf16(rng.uniform(1, 2, (batch, hkv)))
    power = 2.0 ** -(np.arange(hq) % gq)
    q[:, :, 0], q[:, :, 1] = np.repeat(a, gq, 1) * power, np.repeat(b, gq, 1) * power
    size = 2.0 ** rng.integers(6, 14, (batch, n, 1))
    kk = k.reshape(batch, n, hkv, d)
    kk[..., 0], kk[..., 1] = b[:, None] * size, -a[:, None] * size
    scale = d ** -0.5
    got = run_decode(q, k, v, kn, vn, n, scale)
    gk, gv = np.zeros((batch, 1, hkv, d)), np.zeros((batch, 1, hkv, d))
    cu = np.arange(0, (batch + 1) * n, n)
    ref = O.decode_attn(q, kn, vn, [n] * batch, k, v, cu, range(batch), gk, gv, [0] * batch, scale=scale, rope_base=0.0)["out"]
    weight = O.decode_attn(q, kn, np.abs(vn), [n] * batch, k, np.abs(v), cu, range(batch), gk, gv, [0] * batch, scale=scale,
                           rope_base=0.0)["out"]     # sum of probability * |value|
    # fp32: a score is wrong by a few units in the last place of its largest term, all weights by twice that
    term = 4.0 * 2.0 ** 13 * scale
    bound = 2.0 ** -8 * np.abs(ref) + 2.0 * term * 2.0 ** -22 * weight
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound).max())


@pytest.mark.parametrize("h,d", [(4, 64), (3, 128)])
def test_decode_values_that_cancel(h, d):
    """Four rows' values cancel under their probabilities; the other rows' values are zero.  (One head per kv head.)"""
    n, batch, scale = 40, 4, 0.02
    rng = np.random.default_rng(d + h)
    rnd = lambda *s: bf16(rng.standard_normal(s))
    q, k, kn, vn = rnd(batch, h, d), rnd(batch * n, h, d), rnd(batch, h, d), np.zeros((batch, h, d))
    kk = k.reshape(batch, n, h, d)
    s = np.einsum("bhd,bnhd->bnh", q, kk) * scale
    s_new = (q * kn).sum(-1) * scale
    p = np.exp(s) / (np.exp(s).sum(1, keepdims=True) + np.exp(s_new)[:, None])
    v = np.zeros((batch, n, h, d))
    v[:, 3:39:9] = np.moveaxis(cancelling(np.moveaxis(p[:, 3:39:9, :, None], 1, 0), bf16(rng.uniform(1, 2, (batch, h, d)))), 0, 1)
    ref, size = (np.einsum("bnh,bnhd->bhd", p, x) for x in (v, np.abs(v)))
    got = run_decode(q, k, v.reshape(batch * n, h, d), kn, vn, n, scale)
    # small scores (|s| < 1): a probability is right to about 2^-22 of itself in fp32
    bound = 2.0 ** -8 * np.abs(ref) + 2.0 ** -21 * size
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound).max())


@pytest.mark.parametrize("which", ["dq", "dk", "dv"])
@pytest.mark.parametrize("hq,hkv,d,n", [(2, 2, 64, 8), (2, 2, 128, 40), (32, 32, 128, 8)])
def test_backward_sums_that_cancel(hq, hkv, d, n, which):
    """dV of key 0, dK of key 0 or dQ of the last query as a sum of four terms that cancel.  q and k score with their first
    half only, so the second half of the other operand is free to be chosen.  (n = 40 spans two 32-row tiles.)"""
    B = _B()
    batch = 64 if hq == 32 else 2          # 64 x 32 pairs: the 128-row workgroups
    scale, half = 0.02, d // 2
    rng = np.random.default_rng(n + d + len(which))
    q, k = bf16(rng.standard_normal((batch, n, hq, d))), bf16(rng.standard_normal((batch, n, hkv, d)))
    q[..., half:], k[..., half:] = 0.0, 0.0
    # few bits: dP and D come out (almost) exact, the error under test is that of P and dS as operands
    v, g = (rng.integers(-3, 4, (batch, n, hq, d)) / 2.0 for _ in range(2))
    s = np.einsum("bihd,bjhd->bhij", q, k) * scale
    s = np.where(np.arange(n)[:, None] >= np.arange(n)[None], s, -np.inf)
    lse = np.log(np.exp(s).sum(-1))                                    # [batch, h, n]
    lse32 = lse.astype(np.float32).astype(np.float64)
    p = np.exp(s - lse32[..., None])
    rows = np.array([0, 2, n - 3, n - 1])
    if which == "dv":
        w = np.moveaxis(p[:, :, rows, 0], 2, 0)[..., None]             # [4, batch, h, 1]
        g = np.zeros_like(g)
        g[:, rows] = np.moveaxis(cancelling(w, bf16(rng.uniform(1, 2, (batch, hq, d)))), 0, 1)
    out = bf16(np.einsum("bhij,bjhd->bihd", p, v))
    dp = np.einsum("bihd,bjhd->bhij", g, v)
    big_d = np.einsum("bihd,bihd->bhi", out, g)
    ds = p * (dp - big_d[..., None])
    if which in ("dk", "dq"):
        w = np.moveaxis(ds[:, :, rows, 0] if which == "dk" else ds[:, :, n - 1, rows], 2, 0)[..., None]
        w = np.where(np.abs(w) < 1e-3, 1e-3, w)
        first = bf16(rng.uniform(1, 2, (batch, hq, half)))
        x = q if which == "dk" else k
        x[:, rows, :, half:] = np.clip(np.moveaxis(cancelling(w, first), 0, 1), -1e4, 1e4)
    dq, dk, dv = (np.einsum(e, m, x) * f for e, m, x, f in (("bhij,bjhd->bihd", ds, k, scale), ("bhij,bihd->bjhd", ds, q, scale),
                                                            ("bhij,bihd->bjhd", p, g, 1.0)))
    ads = np.abs(p) * (np.abs(dp) + np.abs(big_d)[..., None])
    aq, ak, av = (np.einsum(e, m, np.abs(x)) * f for e, m, x, f in (
        ("bhij,bjhd->bihd", ads, k, scale), ("bhij,bihd->bjhd", ads, q, scale), ("bhij,bihd->bjhd", np.abs(p), g, 1.0)))
    ref, size = {"dq": (dq, aq), "dk": (dk, ak), "dv": (dv, av)}[which]

    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(BF).to(DEV).reshape(batch * n, -1, d)
    desc = B.make_desc(BF, hq, hkv, d, scale, 0.0)
    d_lse = torch.from_numpy(np.ascontiguousarray(np.moveaxis(lse, 1, 2)).astype(np.float32)).to(DEV).reshape(batch * n, hq)
    grads = [torch.full_like(to(x), float("nan")) for x in (q, k, v)]
    B.earn_attn_backward(desc, to(q), to(k), to(v), to(out), d_lse, to(g), i32(range(0, (batch + 1) * n, n)), batch, batch * n, n, *grads)
    torch.cuda.synchronize()
    got = grads[("dq", "dk", "dv").index(which)].cpu().double().numpy().reshape(ref.shape)
    row = n - 1 if which == "dq" else 0
    # every term right to a few units in the last place of fp32
    err, bound = np.abs(got - ref)[:, row], (2.0 ** -8 * np.abs(ref) + 2.0 ** -21 * size)[:, row]
    assert (err <= bound).all(), float((err / np.maximum(bound, 1e-30)).max())
