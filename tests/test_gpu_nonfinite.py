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
