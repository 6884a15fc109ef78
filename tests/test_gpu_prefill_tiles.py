"""Medium-length bf16 prefill at the edges of its tiles: 32-row waves, 64-key tiles, 128-row workgroups whose queries arrive
and whose outputs leave through LDS, one sequence after another in packed tensors (a row too many would be a neighbour's)."""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from paper_2507_00715_amd import workloads as W
from parity import check_attn

pytestmark = pytest.mark.gpu
DEV, BF = "cuda:0", torch.bfloat16


@pytest.mark.parametrize("rope_base", [10000.0, 0.0])
@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 128), (6, 2, 64), (4, 2, 128)])
@pytest.mark.parametrize("lens", [[129, 1, 31, 128, 32, 33], [193, 64, 65, 127, 63, 191], [257, 96, 97, 160, 255], [385, 0, 2]])
def test_prefill_at_tile_edges(lens, hq, hkv, d, rope_base):
    _check(lens, hq, hkv, d, rope_base)


@pytest.fixture
def long_kernel():
    from paper_2507_00715_amd import binding as B
    B.earn_set_tuning("prefill_block_rows", 256)
    yield
    B.earn_set_tuning("prefill_block_rows", 0)


@pytest.mark.parametrize("rope_base", [10000.0, 0.0])
@pytest.mark.parametrize("hq,hkv,d", [(14, 2, 64), (12, 2, 128), (3, 1, 128), (6, 2, 64)])
@pytest.mark.parametrize("lens", [[200, 1, 31, 32, 33, 63, 64, 65], [321, 0, 129, 96, 257], [577, 2, 449]])
def test_long_prefill_over_heads_that_do_not_fill_a_workgroup(long_kernel, lens, hq, hkv, d, rope_base):
    """Eight waves take units of 32 rows of one head: with groups of 3, 6 and 7 heads a workgroup's units straddle row blocks, and
    the last workgroup of a sequence holds units that do not exist."""
    _check(lens, hq, hkv, d, rope_base)


@pytest.mark.parametrize("offset", [1, 4])
@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (6, 2, 64)])
def test_queries_and_outputs_that_start_anywhere(hq, hkv, d, offset):
    """Rows that do not start on 16 bytes: queries cannot be loaded into LDS directly."""
    _check([129, 1, 31, 128, 32, 33, 200], hq, hkv, d, 10000.0, offset)


def _check(lens, hq, hkv, d, rope_base, offset=0):
    from paper_2507_00715_amd import binding as B
    g = torch.Generator().manual_seed(sum(lens) + hq)
    T = sum(lens)
    q, k, v = (torch.randn(T, h, d, generator=g).to(BF) for h in (hq, hkv, hkv))
    pos = torch.randint(0, 5000, (T,), generator=g, dtype=torch.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    desc = B.make_desc(BF, hq, hkv, d, 0.0, rope_base)
    pad = 3                                      # rows before and behind the batch, which keep their sentinel
    moved = lambda t: torch.cat([t.new_zeros(offset), t.flatten()])[offset:].view(t.shape)   # contiguous, `offset` elements into its memory
    out = moved(torch.full((T + 2 * pad, hq, d), 7.0, dtype=BF, device=DEV))
    lse = torch.empty(T, hq, dtype=torch.float32, device=DEV)
    k_rot = torch.empty(T, hkv, d, dtype=BF, device=DEV)
    B.earn_prefill_attn(desc, moved(q.to(DEV)), k.to(DEV), v.to(DEV), torch.from_numpy(cu).to(DEV), pos.to(DEV), len(lens), T, max(lens),
                        out[pad:pad + T], k_rot, lse, None)
    torch.cuda.synchronize()
    ref = O.prefill_attn(W.to_f64(q), W.to_f64(k), W.to_f64(v), cu, positions=pos.numpy(), rope_base=rope_base)
    check_attn(out[pad:pad + T], ref["out"], BF, f"lengths {lens}")
    check_attn(k_rot, ref["k_rot"], BF, "rotated keys")
    # a query and a key element are rounded once each, 2^-9 apiece: a score is off by at most 2^-8 scale |q| |k|, the
    # log-sum-exp by no more than the worst score and 2^-9 for the rounded weights it sums
    norm = lambda x: float(x.double().norm(dim=-1).max())
    bar = 2.0 ** -8 * norm(q) * norm(k) / d ** 0.5 + 2.0 ** -9
    assert np.abs(lse.cpu().double().numpy() - ref["lse"]).max() <= bar
    assert bool((out[:pad] == 7.0).all()) and bool((out[pad + T:] == 7.0).all())
