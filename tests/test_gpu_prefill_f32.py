"""fp32 prefill (prefill_f32_kernel) at the edges of its 16-key blocks and 16- and 32-row workgroups, rotating the keys itself or
behind a rotation pass, and with infinite values behind the causal mask."""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from paper_2507_00715_amd import workloads as W
from parity import check_attn

pytestmark = pytest.mark.gpu
DEV, F32 = "cuda:0", torch.float32


def _run(lens, hq, hkv, d, rope_base=10000.0, positions=None, in_place=False, edit=None, seed=0, bound=None):
    from paper_2507_00715_amd import binding as B
    g = torch.Generator().manual_seed(seed + sum(lens) + hq)
    T = sum(lens)
    q, k, v = (torch.randn(T, h, d, generator=g) for h in (hq, hkv, hkv))
    if edit:
        edit(q, k, v)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    desc = B.make_desc(F32, hq, hkv, d, 0.0, rope_base)
    d_k = k.to(DEV)
    out, lse = torch.full((T, hq, d), 7.0, device=DEV), torch.empty(T, hq, device=DEV)
    k_rot = d_k if in_place else torch.empty_like(d_k)
    B.earn_prefill_attn(desc, q.to(DEV), d_k, v.to(DEV), torch.from_numpy(cu).to(DEV), None if positions is None else positions.to(DEV),
                        len(lens), T, bound or max(lens), out, k_rot, lse, torch.empty(256, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    return q, k, v, cu, out, k_rot, lse


@pytest.mark.parametrize("rope_base,in_place", [(10000.0, False), (10000.0, True), (0.0, False)])
@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (4, 2, 128), (3, 1, 64)])
@pytest.mark.parametrize("lens", [[1, 15, 16, 17], [33, 31, 0, 32, 2], [129, 127, 128], [47, 48, 49] * 8, [130, 5] * 12])
def test_prefill_f32_at_block_edges(lens, hq, hkv, d, rope_base, in_place):
    pos = torch.randint(0, 9000, (sum(lens),), generator=torch.Generator().manual_seed(1), dtype=torch.int32)
    q, k, v, cu, out, k_rot, lse = _run(lens, hq, hkv, d, rope_base, pos, in_place)
    ref = O.prefill_attn(W.to_f64(q), W.to_f64(k), W.to_f64(v), cu, positions=pos.numpy(), rope_base=rope_base)
    check_attn(out, ref["out"], F32, f"{lens}")
    check_attn(k_rot, ref["k_rot"], F32, "rotated keys")
    assert np.abs(lse.cpu().double().numpy() - ref["lse"]).max() <= 1e-4   # (the bar of the outputs)


@pytest.mark.parametrize("d,batch", [(64, 1), (64, 40), (128, 1), (128, 40)])
def test_values_behind_the_mask_stay_away(d, batch):
    """An infinite value row and a NaN value row reach the queries from their own row on and no other."""
    n, at_inf, at_nan = 37, 21, 30
    def edit(q, k, v):
        for s in range(batch):
            v[s * n + at_inf] = float("inf")
            v[s * n + at_nan] = float("nan")
    clean = _run([n] * batch, 4, 2, d)[4]
    got = _run([n] * batch, 4, 2, d, edit=edit)[4].view(batch, n, 4, d)
    assert torch.equal(got[:, :at_inf - at_inf % 16], clean.view(batch, n, 4, d)[:, :at_inf - at_inf % 16])
    # the block of the first such row is added pair by pair: the same sums in another order
    assert (got[:, :at_inf] - clean.view(batch, n, 4, d)[:, :at_inf]).abs().max() <= 2e-6
    assert bool((got[:, at_inf:at_nan] == float("inf")).all())
    assert bool(torch.isnan(got[:, at_nan:]).all())


@pytest.mark.parametrize("d", [64, 128])
def test_a_bound_far_above_the_sequences(d):
    """max_seqlen is an upper bound: one whose workgroups no grid takes gives what a tight one gives."""
    lens = [20, 1, 33]
    tight, loose = _run(lens, 4, 2, d), _run(lens, 4, 2, d, bound=600_000_000)
    for a, b in zip(tight[4:], loose[4:]):
        assert torch.equal(a, b)
