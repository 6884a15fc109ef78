"""Decode over streams that share a workgroup (decode_beams_kernel): layouts of the streams, generated rows of any length, an
ancestor table, several layers, and infinite and NaN rows that only some of a group's streams see, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from paper_2507_00715_amd import workloads as W
from parity import check_attn

pytestmark = pytest.mark.gpu
DEV, BF = "cuda:0", torch.bfloat16
# sizes that the rule gives to decode_beams_kernel (test_work_order.py checks that it does): with one layer a launch and with three,
# also with a stream more than the sequences share evenly; 8 generated rows
GROUPED = [(16, 4, 128, 8, 13, 130), (4, 4, 64, 17, 6, 131), (8, 4, 64, 24, 8, 65), (12, 4, 64, 12, 7, 129)]
# ... and in the usual order
ANY_ORDER, ANY_ORDER_ROOM = [(16, 4, 128, 12, 10, 64, 3), (8, 8, 64, 9, 8, 33, 2), (4, 4, 64, 200, 9, 60, 1), (12, 2, 128, 300, 6, 100, 1)], 5
STAY_AWAY = [(16, 4, 128, 12, 9, 100), (8, 8, 64, 12, 9, 100)]
TIMED = [(32, 32, 128, 8, 10, 256), (8, 8, 64, 16, 10, 256)]
I32 = lambda x: torch.tensor([int(v) for v in x], dtype=torch.int32, device=DEV)


def _inputs(seed, streams, lens, hq, hkv, d, cap, layers):
    g = torch.Generator().manual_seed(seed)
    r = lambda *s: torch.randn(layers, *s, generator=g).to(BF)
    rows = sum(lens)
    return dict(q=r(streams, hq, d), k_new=r(streams, hkv, d), v_new=r(streams, hkv, d), k=r(rows, hkv, d), v=r(rows, hkv, d),
                gen_k=r(streams, cap, hkv, d), gen_v=r(streams, cap, hkv, d))


def _run(x, lens, s2s, gen_len, cap, hq, hkv, d, gen_src=None, rope_base=10000.0):
    from paper_2507_00715_amd import binding as B
    layers, streams, batch = x["q"].shape[0], len(s2s), len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q_pos = [lens[s] + g for s, g in zip(s2s, gen_len)]
    desc = B.make_desc(BF, hq, hkv, d, 0.0, rope_base)
    t = {k: v.to(DEV) for k, v in x.items()}
    out = torch.full_like(t["q"], float("nan"))
    ws = torch.empty(max(256, B.earn_decode_layers_workspace_bytes(desc, layers, streams, batch, max(lens), cap)), dtype=torch.uint8, device=DEV)
    if gen_src is not None:
        B.earn_decode_attn_beams(desc, t["q"][0], t["k_new"][0], t["v_new"][0], I32(q_pos), t["k"][0], t["v"][0], I32(cu), I32(s2s),
                                 t["gen_k"][0], t["gen_v"][0], I32(gen_len), I32(np.ravel(gen_src)).view(streams, cap), cap, streams,
                                 batch, max(lens), out[0], ws)
    else:
        B.earn_decode_attn_layers(desc, t["q"], t["k_new"], t["v_new"], I32(q_pos), t["k"], t["v"], I32(cu), I32(s2s), t["gen_k"],
                                  t["gen_v"], I32(gen_len), cap, streams, batch, max(lens), out, ws)
    torch.cuda.synchronize()
    return out.cpu(), t["gen_k"].cpu(), t["gen_v"].cpu(), cu, q_pos


def _oracle(x, l, cu, s2s, gen_len, q_pos, gen_src=None, rope_base=10000.0):
    f = {k: W.to_f64(v[l]) for k, v in x.items()}
    gk, gv = f["gen_k"].copy(), f["gen_v"].copy()
    if gen_src is not None:                      # every stream with a cache of its own: its ancestors' rows copied
        for u, g in enumerate(gen_len):
            for j in range(g):
                gk[u, j], gv[u, j] = f["gen_k"][gen_src[u][j], j], f["gen_v"][gen_src[u][j], j]
    with np.errstate(invalid="ignore", over="ignore"):
        out = O.decode_attn(f["q"], f["k_new"], f["v_new"], q_pos, f["k"], f["v"], cu, s2s, gk, gv, gen_len, rope_base=rope_base)["out"]
    return out, gk, gv


def _layout(name, batch, beams, rng):
    s2s = np.repeat(np.arange(batch), beams)
    if name == "shuffled":
        rng.shuffle(s2s)
    elif name == "uneven":                       # a stream more: the groups follow no sequence
        s2s = np.concatenate([s2s, [batch - 1]])
    elif name == "beams first":                  # the first beam of every sequence, then the second ones
        s2s = np.tile(np.arange(batch), beams)
    elif name == "pairs":                        # two streams of a sequence side by side, its others elsewhere
        s2s = np.tile(np.repeat(np.arange(batch), 2), (beams + 1) // 2)
    elif name == "last two swapped":
        s2s[-1], s2s[-beams - 1] = s2s[-beams - 1], s2s[-1]
    elif name == "few sequences":                # most sequences have no stream, one has most of them
        s2s = np.where(rng.random(batch * beams) < 0.5, 2, rng.integers(0, batch, batch * beams) // 3 * 3)
    return s2s.tolist()


@pytest.mark.parametrize("layout", ["usual", "uneven", "shuffled"])
@pytest.mark.parametrize("hq,hkv,d,batch,beams,longest", [(16, 4, 128, 12, 10, 64), (14, 2, 64, 30, 7, 70), (8, 8, 64, 9, 8, 33),
                                                          (16, 2, 128, 30, 6, 100), (12, 4, 64, 13, 9, 300), *GROUPED])
@pytest.mark.parametrize("table,layers", [(False, 1), (False, 3), (True, 1)])
def test_grouped_streams(layout, hq, hkv, d, batch, beams, longest, table, layers):
    rng = np.random.default_rng(batch + beams + longest)
    s2s, cap = _layout(layout, batch, beams, rng), 8
    lens = rng.integers(1, longest + 1, batch)
    lens[0], lens[-1] = longest, 1
    lens = [int(n) for n in lens]
    # (with a table all streams are at the same step: a call appends to slot gen_len of every stream while others read the slots before)
    gen_len = [cap - 2] * len(s2s) if table else rng.integers(0, cap, len(s2s)).tolist()
    src = rng.integers(0, len(s2s), (len(s2s), cap)).tolist() if table else None
    x = _inputs(batch, len(s2s), lens, hq, hkv, d, cap, layers)
    out, gk, gv, cu, q_pos = _run(x, lens, s2s, gen_len, cap, hq, hkv, d, src)
    for l in range(layers):
        ref, ref_k, ref_v = _oracle(x, l, cu, s2s, gen_len, q_pos, src)
        check_attn(out[l], ref, BF, f"layer {l}")
        for u, g in enumerate(gen_len):          # appended: the new row and nothing else
            check_attn(gk[l, u, g], ref_k[u, g], BF, "appended key")
            assert torch.equal(gv[l, u, g], x["v_new"][l, u])
            gk[l, u, g], gv[l, u, g] = x["gen_k"][l, u, g], x["gen_v"][l, u, g]
        assert torch.equal(gk[l], x["gen_k"][l]) and torch.equal(gv[l], x["gen_v"][l])


@pytest.mark.parametrize("layout", ["beams first", "pairs", "last two swapped", "few sequences"])
@pytest.mark.parametrize("hq,hkv,d,batch,beams,longest,layers", ANY_ORDER)
def test_streams_in_any_order(layout, hq, hkv, d, batch, beams, longest, layers):
    """The groups are cut from the streams in the order of their sequences, whatever order they come in (up to 1800 streams: a
    workgroup's check of the order takes several steps)."""
    rng = np.random.default_rng(batch + beams)
    s2s, cap = _layout(layout, batch, beams, rng), ANY_ORDER_ROOM
    lens = [int(n) for n in rng.integers(1, longest + 1, batch)]
    gen_len = rng.integers(0, cap, len(s2s)).tolist()
    x = _inputs(batch, len(s2s), lens, hq, hkv, d, cap, layers)
    out, gk, gv, cu, q_pos = _run(x, lens, s2s, gen_len, cap, hq, hkv, d)
    for l in range(layers):
        ref, ref_k, _ = _oracle(x, l, cu, s2s, gen_len, q_pos)
        check_attn(out[l], ref, BF, f"layer {l}")
        at = (torch.arange(len(s2s)), torch.tensor(gen_len))
        check_attn(gk[l][at], ref_k[at], BF, "appended keys")
        assert torch.equal(gv[l][at], x["v_new"][l])


@pytest.mark.parametrize("hq,hkv,d,batch,beams,rows", TIMED)
def test_order_of_streams_costs_little(hq, hkv, d, batch, beams, rows):
    """Streams that do not lie side by side: groups of unlike streams walked a cache each, 4 to 6 times the time."""
    from paper_2507_00715_amd import binding as B
    cap, n = 8, batch * beams
    x = {k: v.to(DEV) for k, v in _inputs(1, n, [rows] * batch, hq, hkv, d, cap, 1).items()}
    out, desc = torch.empty_like(x["q"][0]), B.make_desc(BF, hq, hkv, d, 0.0, 10000.0)
    cu, pos, gen = I32(rows * np.arange(batch + 1)), I32([rows + 5] * n), I32([5] * n)
    ws = torch.empty(max(256, B.earn_decode_workspace_bytes(desc, n, batch, rows, cap)), dtype=torch.uint8, device=DEV)

    def us(layout):
        s2s = I32(_layout(layout, batch, beams, np.random.default_rng(0)))
        call = B.bind_decode_attn(desc, x["q"][0], x["k_new"][0], x["v_new"][0], pos, x["k"][0], x["v"][0], cu, s2s, x["gen_k"][0],
                                  x["gen_v"][0], gen, cap, n, batch, rows, out, ws)
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            call()
            a.record()
            for _ in range(20):
                call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 20 * 1e3)
        return best
    assert us("beams first") <= 2 * us("usual")


@pytest.mark.parametrize("n", [40, STAY_AWAY[0][5]])
@pytest.mark.parametrize("hq,hkv,d", [x[:3] for x in STAY_AWAY])
@pytest.mark.parametrize("layout", ["usual", "shuffled"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_rows_of_other_streams_stay_away(hq, hkv, d, layout, value, n):
    """Values of one stream's generated rows, its new token, and one sequence's cache reach only the streams that see them."""
    batch, beams, cap = 12, 9, 8
    rng = np.random.default_rng(5)
    s2s, lens = _layout(layout, batch, beams, rng), [n] * batch
    gen_len = rng.integers(1, cap, len(s2s)).tolist()
    x = _inputs(3, len(s2s), lens, hq, hkv, d, cap, 1)
    clean = _run({k: v.clone() for k, v in x.items()}, lens, s2s, gen_len, cap, hq, hkv, d, rope_base=0.0)[0]
    u_gen, u_new, seq = 5, 50, 7
    x["gen_v"][0, u_gen, 0, :, 3] = value
    x["v_new"][0, u_new, :, 9] = value
    x["v"][0, seq * n + 11, :, 20] = value
    out, _, _, cu, q_pos = _run(x, lens, s2s, gen_len, cap, hq, hkv, d, rope_base=0.0)
    ref = _oracle(x, 0, cu, s2s, gen_len, q_pos, rope_base=0.0)[0]
    got = out[0].double().numpy()
    for kind in (np.isnan, np.isposinf, np.isneginf):
        np.testing.assert_array_equal(kind(got), kind(ref))
    touched = {u for u, s in enumerate(s2s) if s == seq} | {u_gen, u_new}
    others = [u for u in range(len(s2s)) if u not in touched]
    # (a wave that meets such a row takes its sums in another order)
    assert (out[0, others].float() - clean[0, others].float()).abs().max() <= 2.0 ** -7 * clean[0, others].float().abs().max()
