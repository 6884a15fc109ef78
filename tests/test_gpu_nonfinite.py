"""Infinities and NaN in the inputs of the matrix-core kernels: an element of a key, a value or a gradient reaches exactly the
results that depend on it, as it does when every product and sum is taken on its own in fp32."""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from test_gpu_operand_width import bf16, i32, run_decode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF = torch.bfloat16
INF, NAN = np.inf, np.nan


def same(got, ref, size, what=""):
    """NaN and infinities where the reference has them; the rest right to the rounding of bf16 and of fp32 sums of `size`."""
    assert (np.isnan(got) == np.isnan(ref)).all(), f"{what}: NaN in {np.isnan(got).sum()} places, not {np.isnan(ref).sum()}"
    assert (np.where(np.isinf(ref), ref, 0.0) == np.where(np.isinf(got), got, 0.0)).all(), f"{what}: infinities"
    ok = np.isfinite(ref)
    assert (np.abs(got[ok] - ref[ok]) <= 2.0 ** -8 * np.abs(ref[ok]) + 2.0 ** -16 * size[ok]).all(), what


@pytest.mark.parametrize("n", [20, 300])
@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (3, 3, 128), (8, 2, 128)])
@pytest.mark.parametrize("kind", ["key -inf", "key +inf", "key NaN", "value inf", "values of both signs", "value NaN"])
def test_decode_non_finite_rows(kind, hq, hkv, d, n):
    """Short and medium key lists.  An infinite key element drops its row from the softmax where the score is -inf (every
    query is negative there) and spoils the head where it is +inf; an infinite value is an infinite output."""
    rng = np.random.default_rng(n + d + hq)
    rnd = lambda *s: bf16(rng.standard_normal(s))
    batch = 3
    q, k, v, kn, vn = rnd(batch, hq, d), rnd(batch, n, hkv, d), rnd(batch, n, hkv, d), rnd(batch, hkv, d), rnd(batch, hkv, d)
    q[:, :, 5] = bf16(-np.abs(q[:, :, 5]) - 0.5)
    c = hkv - 1                                   # the kv head; sequence 1 holds the element, the others stay clean
    if kind.startswith("key"):
        k[1, n - 2, c, 5] = {"key -inf": INF, "key +inf": -INF, "key NaN": NAN}[kind]
        k[1, 3, c, 5] = k[1, n - 2, c, 5]
    elif kind == "value inf":
        v[1, n - 2, c, 7] = INF
        v[1, 4, c, 8] = -INF
        vn[1, c, 9] = INF
    elif kind == "values of both signs":
        v[1, n - 2, c, 7], v[1, 4, c, 7] = INF, -INF
    else:
        v[1, n - 2, c, 7] = NAN
    got = run_decode(q, k.reshape(-1, hkv, d), v.reshape(-1, hkv, d), kn, vn, n, d ** -0.5)
    cu, g0 = np.arange(0, (batch + 1) * n, n), lambda: np.zeros((batch, 1, hkv, d))
    with np.errstate(invalid="ignore"):
        ref = O.decode_attn(q, kn, vn, [n] * batch, k.reshape(-1, hkv, d), v.reshape(-1, hkv, d), cu, range(batch), g0(), g0(),
                            [0] * batch, rope_base=0.0)["out"]
    head = c * (hq // hkv)
    if kind == "key -inf":
        assert np.isfinite(ref).all()             # the case is what it says
    elif kind == "key +inf":
        assert np.isnan(ref[1, head:]).all() and np.isfinite(ref[1, :head]).all()
    elif kind == "value inf":
        assert (ref[1, head:, 7] == INF).all() and (ref[1, head:, 8] == -INF).all() and (ref[1, head:, 9] == INF).all()
    same(got, ref, 4.0 * np.ones_like(ref), kind)


@pytest.mark.parametrize("dtype", [BF, torch.float32])
@pytest.mark.parametrize("hq,hkv,d,n,batch", [(2, 2, 64, 40, 2), (4, 2, 128, 70, 2), (4, 1, 128, 70, 1), (32, 32, 128, 40, 32)])
@pytest.mark.parametrize("kind", ["late key inf", "late key NaN", "late value inf", "late value NaN", "early query inf",
                                  "early gradient inf", "early gradient NaN", "gradients of both signs"])
def test_backward_non_finite_rows(kind, hq, hkv, d, n, batch, dtype):
    """A row's infinity or NaN reaches the pairs (query i, key j <= i) that it is part of and no others: what is masked is not
    multiplied by zero.  One sequence holds it; n is past the 32-row tile, the element in the middle of one."""
    from paper_2507_00715_amd import binding as B
    rng = np.random.default_rng(n + d + hq)
    q, g, out = (bf16(rng.standard_normal((batch, n, hq, d))) for _ in range(3))
    k, v = (bf16(rng.standard_normal((batch, n, hkv, d))) for _ in range(2))
    q[..., 5] = bf16(-np.abs(q[..., 5]) - 0.5)      # the sign of an infinite key's scores is known: -inf
    gq, scale, b, c = hq // hkv, d ** -0.5, batch - 1, hkv - 1
    see = np.arange(n)[:, None] >= np.arange(n)[None]
    with np.errstate(invalid="ignore", over="ignore"):
        def scores(bb, a):
            return (q[bb, :, a] @ k[bb, :, a // gq].T) * scale
        lse = np.array([[np.log(np.where(see, np.exp(scores(bb, a)), 0.0).sum(1)) for a in range(hq)] for bb in range(batch)])
        lse = lse.astype(np.float32).astype(np.float64)
        where = {"late": n - 5, "early": 4, "gradients": 4}[kind.split()[0]]
        value = NAN if kind.endswith("NaN") else INF
        if "key" in kind: k[b, where, c, 5] = value
        elif "value" in kind: v[b, where, c, 5] = value
        elif "query" in kind: q[b, where, c * gq, 5] = -value
        else: g[b, where, c * gq, 5] = value
        if kind == "gradients of both signs": g[b, where + 2, c * gq, 5] = -value
        ref = {x: np.zeros_like(t) for x, t in (("dq", q), ("dk", k), ("dv", v))}
        size = {x: np.zeros_like(t) for x, t in ref.items()}

        def add(x, at, term):
            ref[x][at] += term
            size[x][at] += np.abs(np.where(np.isfinite(term), term, 0.0))

        for bb, a in [(b, aa) for aa in range(c * gq, hq)]:     # the heads that share the kv head; the others must just be finite
            cc = a // gq
            d_i = (g[bb, :, a] * out[bb, :, a]).sum(-1)
            for i in range(n):
                for j in range(i + 1):
                    p = np.exp((q[bb, i, a] * k[bb, j, cc]).sum() * scale - lse[bb, a, i])
                    ds = p * ((g[bb, i, a] * v[bb, j, cc]).sum() - d_i[i])
                    add("dq", (bb, i, a), ds * scale * k[bb, j, cc])
                    add("dk", (bb, j, cc), ds * scale * q[bb, i, a])
                    add("dv", (bb, j, cc), p * g[bb, i, a])
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dtype).to(DEV).reshape(batch * n, -1, d)
    d_lse = torch.from_numpy(np.ascontiguousarray(np.moveaxis(lse, 1, 2)).astype(np.float32)).to(DEV).reshape(batch * n, hq)
    grads = [torch.full_like(to(x), 7.0) for x in (q, k, v)]
    B.earn_attn_backward(B.make_desc(dtype, hq, hkv, d, scale, 0.0), to(q), to(k), to(v), to(out), d_lse, to(g),
                         i32(range(0, (batch + 1) * n, n)), batch, batch * n, n, *grads)
    torch.cuda.synchronize()
    for x, t, heads in zip(("dq", "dk", "dv"), grads, (slice(c * gq, hq), slice(c, hkv), slice(c, hkv))):
        got = t.cpu().double().numpy().reshape(ref[x].shape)
        same(got[b][:, heads], ref[x][b][:, heads], size[x][b][:, heads], f"{kind}: {x}")
        assert np.isfinite(got[:b]).all() and np.isfinite(np.delete(got[b], np.arange(heads.start, heads.stop), axis=1)).all()


@pytest.mark.parametrize("value", [INF, NAN])
@pytest.mark.parametrize("hq,hkv,d,lens", [(4, 1, 128, [100, 70, 65]), (8, 2, 64, [128, 75]), (6, 2, 128, [90] * 40)])
def test_short_prefill_non_finite_late_values(hq, hkv, d, lens, value):
    """A value from row 64 on never reaches the queries before it (nor does a key: masked scores are dropped whatever they are).
    The kernel packs the query rows of a group's heads 16 at a time, so early and late rows meet in one product."""
    from paper_2507_00715_amd import binding as B
    T, cu = sum(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    g = torch.Generator().manual_seed(T)
    q, k, v = (torch.randn(T, h, d, generator=g).to(BF) for h in (hq, hkv, hkv))

    def run(k, v):
        desc = B.make_desc(BF, hq, hkv, d)
        out, lse = torch.full((T, hq, d), 7.0, dtype=BF, device=DEV), torch.full((T, hq), 7.0, device=DEV)
        ws = torch.empty(max(B.earn_prefill_workspace_bytes(desc, len(lens), T, max(lens), False), 256), dtype=torch.uint8, device=DEV)
        B.earn_prefill_attn(desc, q.to(DEV), k.to(DEV), v.to(DEV), i32(cu), None, len(lens), T, max(lens), out, None, lse, ws)
        torch.cuda.synchronize()
        return out.cpu(), lse.cpu()

    clean = run(k, v)
    for s, n in enumerate(lens):
        k[cu[s] + 64:cu[s] + n, hkv - 1, 3], v[cu[s] + 64:cu[s] + n, hkv - 1, 3] = value, value
    got = run(k, v)
    early = torch.cat([torch.arange(cu[s], cu[s] + 64) for s in range(len(lens))])
    for x, y in zip(got, clean):
        assert torch.equal(x[early], y[early])
    gq = hq // hkv
    late = torch.cat([torch.arange(cu[s] + 64, cu[s + 1]) for s in range(len(lens))])
    assert torch.equal(got[0][late, :hq - gq], clean[0][late, :hq - gq])          # other kv heads
    assert not torch.isfinite(got[0][late, hq - gq:].float()).all()
