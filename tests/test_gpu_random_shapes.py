"""Seeded sweep over randomly drawn (valid) shapes: head counts and group sizes, both head dimensions, ragged caches
including empty ones, uneven beam counts (sequences without any stream included), ragged generated lengths, and
register counts.  Every case is checked against the fp64 oracle to the usual bars; the point is the shapes nobody
thought of when writing the targeted cases, so the draws are fixed by the seed and the case number names them.
"""
import numpy as np
import pytest
import torch

from oracle import earn_oracle as O
from paper_2507_00715_amd import workloads as W

from parity import check_attn as check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _B():
    from paper_2507_00715_amd import binding
    binding.lib()
    return binding


def draw_heads(rng):
    hkv = int(rng.choice([1, 2, 3, 4, 8]))
    gq = int(rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8]))
    return hkv * gq, hkv, int(rng.choice([64, 128]))


@pytest.mark.parametrize("case", range(24))
def test_decode_random_shape(case):
    B = _B()
    rng = np.random.default_rng(7000 + case)
    dtype = torch.float32 if case % 6 == 5 else torch.bfloat16
    hq, hkv, d = draw_heads(rng)
    batch = int(rng.integers(1, 6))
    slens = [int(x) for x in rng.choice([0, 1, 15, 64, 65, 127, 128, 129, 300, 700], size=batch)]
    beams_of = [int(x) for x in rng.choice([0, 1, 1, 2, 3, 9, 21], size=batch)]
    if sum(beams_of) == 0:
        beams_of[0] = 1
    s2s = [s for s in range(batch) for _ in range(beams_of[s])]
    S = len(s2s)
    gen_cap = int(rng.choice([1, 2, 5, 70]))
    glens = [int(x) for x in rng.integers(0, gen_cap, size=S)]
    gtor = torch.Generator().manual_seed(case)
    rnd = lambda *shape: torch.randn(*shape, generator=gtor).to(dtype)
    cu = np.concatenate([[0], np.cumsum(slens)]).astype(np.int32)
    T = int(cu[-1])
    sk, sv = rnd(max(T, 1), hkv, d)[:T], rnd(max(T, 1), hkv, d)[:T]
    q, kn, vn = rnd(S, hq, d), rnd(S, hkv, d), rnd(S, hkv, d)
    gk, gv = rnd(S, gen_cap, hkv, d), rnd(S, gen_cap, hkv, d)
    q_pos = [slens[s2s[u]] + glens[u] for u in range(S)]
    desc = B.make_desc(dtype, hq, hkv, d)
    dev = lambda x: x.contiguous().to(DEV)
    i32 = lambda x: torch.tensor(list(x), dtype=torch.int32, device=DEV)
    d_sk = dev(sk) if T else torch.zeros(1, hkv, d, dtype=dtype, device=DEV)
    d_sv = dev(sv) if T else torch.zeros(1, hkv, d, dtype=dtype, device=DEV)
    d_gk, d_gv = dev(gk), dev(gv)
    out = torch.full((S, hq, d), float("nan"), dtype=dtype, device=DEV)
    ws = torch.empty(max(B.earn_decode_workspace_bytes(desc, S, batch, max(slens), gen_cap), 1), dtype=torch.uint8,
                     device=DEV)
    print(f"case {case}: {dtype} hq={hq} hkv={hkv} d={d} slens={slens} beams={beams_of} gen_cap={gen_cap}", flush=True)
    B.earn_decode_attn(desc, dev(q), dev(kn), dev(vn), i32(q_pos), d_sk, d_sv, i32(cu), i32(s2s), d_gk, d_gv,
                       i32(glens), gen_cap, S, batch, max(slens), out, ws)
    torch.cuda.synchronize()
    o_gk, o_gv = W.to_f64(gk), W.to_f64(gv)
    ref = O.decode_attn(W.to_f64(q), W.to_f64(kn), W.to_f64(vn), q_pos, W.to_f64(sk), W.to_f64(sv), cu, s2s, o_gk, o_gv,
                        glens)
    for u in range(S):
        check(out[u], ref["out"][u], dtype, f"case {case} stream {u}")
        check(d_gk[u, glens[u]], o_gk[u, glens[u]], dtype, f"case {case} appended key of stream {u}")
        assert torch.equal(d_gv[u, glens[u]].cpu(), vn[u])
        keep = [j for j in range(gen_cap) if j != glens[u]]
        assert torch.equal(d_gk[u, keep].cpu(), gk[u, keep]) and torch.equal(d_gv[u, keep].cpu(), gv[u, keep])


@pytest.mark.parametrize("case", range(16))
def test_prefill_and_register_rows_random_shape(case):
    B = _B()
    rng = np.random.default_rng(9000 + case)
    dtype = torch.float32 if case % 8 == 7 else torch.bfloat16
    hq, hkv, d = draw_heads(rng)
    h, t = int(rng.choice([0, 1, 2, 8, 17, 32])), int(rng.choice([0, 1, 3, 8, 16, 33]))
    if h + t == 0:
        t = 1
    r = h + t
    batch = int(rng.integers(1, 5))
    lens = [r + int(x) for x in rng.choice([0, 1, 30, 63, 64, 200, 500, 1100], size=batch)]
    T = sum(lens)
    gtor = torch.Generator().manual_seed(100 + case)
    rnd = lambda *shape: torch.randn(*shape, generator=gtor).to(dtype)
    q, k, v = rnd(T, hq, d), rnd(T, hkv, d), rnd(T, hkv, d)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    d_cu = torch.from_numpy(cu).to(DEV)
    d_q, d_k, d_v = q.to(DEV), k.to(DEV), v.to(DEV)
    desc = B.make_desc(dtype, hq, hkv, d)
    print(f"case {case}: {dtype} hq={hq} hkv={hkv} d={d} h={h} t={t} lens={lens}", flush=True)

    # the whole layer
    out = torch.full((T, hq, d), float("nan"), dtype=dtype, device=DEV)
    k_rot = torch.empty_like(d_k)
    B.earn_prefill_attn(desc, d_q, d_k, d_v, d_cu, None, batch, T, max(lens), out, k_rot, None, None)
    torch.cuda.synchronize()
    ref = O.prefill_attn(W.to_f64(q), W.to_f64(k), W.to_f64(v), cu)
    for s in range(batch):
        check(out[cu[s]:cu[s + 1]], ref["out"][cu[s]:cu[s + 1]], dtype, f"case {case} prefill sequence {s}")
    check(k_rot, ref["k_rot"], dtype, f"case {case} rotated keys")

    # its register rows only
    q_rows = torch.empty(batch * r, hq, d, dtype=dtype, device=DEV)
    idx, pos = (torch.empty(batch * r, dtype=torch.int32, device=DEV) for _ in range(2))
    cu_c = torch.empty(batch + 1, dtype=torch.int32, device=DEV)
    B.earn_compact_registers([d_q], [q_rows], d_cu, batch, h, t, idx, pos, cu_c)
    out_rows = torch.full((batch * r, hq, d), float("nan"), dtype=dtype, device=DEV)
    k_rot2 = torch.empty_like(d_k)
    ws = torch.empty(max(B.earn_prefill_register_rows_workspace_bytes(desc, batch, max(lens), r), 256),
                     dtype=torch.uint8, device=DEV)
    B.earn_prefill_register_rows(desc, q_rows, d_k, d_v, d_cu, pos, batch, T, max(lens), r, out_rows, k_rot2, ws)
    torch.cuda.synchronize()
    ref_c = O.compact_registers(None, cu, h, t)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_c["idx"])
    want = ref["out"][ref_c["idx"]]
    for s in range(batch):
        check(out_rows[s * r:(s + 1) * r], want[s * r:(s + 1) * r], dtype, f"case {case} register rows of sequence {s}")
    assert torch.equal(k_rot2, k_rot)


@pytest.mark.parametrize("case", range(8))
def test_compaction_random_shape(case):
    """Random register counts, ragged lengths (sequences that are all registers included), 1 to 112 tensors of random
    row widths in one launch: bit-exact against the oracle's gather of the same bytes."""
    B = _B()
    rng = np.random.default_rng(11000 + case)
    h, t = int(rng.choice([0, 1, 3, 8, 32])), int(rng.choice([0, 1, 2, 16, 32]))
    if h + t == 0:
        h = 1
    r = h + t
    batch = int(rng.integers(1, 40))
    lens = [r + int(x) for x in rng.choice([0, 0, 1, 5, 64, 333, 2000], size=batch)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    n_tensors = int(rng.choice([1, 2, 7, 40, 112]))
    widths = [int(x) for x in rng.choice([16, 32, 48, 256, 512, 4096, 8208], size=n_tensors)]   # row bytes
    if n_tensors > 7:   # keep the byte volume of the many-tensor cases small
        widths = [min(wd, 512) for wd in widths]
    print(f"case {case}: h={h} t={t} batch={batch} T={T} tensors={n_tensors} widths={sorted(set(widths))}", flush=True)
    g = torch.Generator().manual_seed(case)
    srcs = [torch.randint(0, 256, (T, wd), dtype=torch.uint8, generator=g) for wd in widths]
    d_src = [s.to(DEV) for s in srcs]
    d_dst = [torch.full((batch * r, wd), 0xEE, dtype=torch.uint8, device=DEV) for wd in widths]
    d_cu = torch.from_numpy(cu).to(DEV)
    idx, pos = (torch.full((batch * r,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
    cu_c = torch.full((batch + 1,), -1, dtype=torch.int32, device=DEV)
    B.earn_compact_registers(d_src, d_dst, d_cu, batch, h, t, idx, pos, cu_c)
    torch.cuda.synchronize()
    ref = O.compact_registers(None, cu, h, t)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref["idx"])
    np.testing.assert_array_equal(pos.cpu().numpy(), ref["pos"])
    np.testing.assert_array_equal(cu_c.cpu().numpy(), ref["cu"])
    for s, dd in zip(srcs, d_dst):
        assert np.array_equal(dd.cpu().numpy(), O.compact_registers(s.numpy(), cu, h, t)["dst"])


@pytest.mark.parametrize("hq,hkv,d,lens", [(32, 8, 128, [64, 33]), (12, 2, 64, [128]), (4, 4, 128, [32, 7]), (32, 8, 128, [64] * 70)])
def test_prefill_short_sequences_rotate_keys_in_place(hq, hkv, d, lens):
    """k_rot_out may be k itself: one workgroup then reads and writes the keys of a (sequence, kv head), where small batches
    otherwise give several workgroups their own copy.  Same bits as with a cache of its own."""
    B = _B()
    T, batch = sum(lens), len(lens)
    g = torch.Generator().manual_seed(T + hq)
    q, k, v = (torch.randn(T, heads, d, generator=g).to(torch.bfloat16).to(DEV) for heads in (hq, hkv, hkv))
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    desc = B.make_desc(torch.bfloat16, hq, hkv, d)
    ws = torch.empty(max(B.earn_prefill_workspace_bytes(desc, batch, T, max(lens), True), 256), dtype=torch.uint8, device=DEV)
    out, k_rot = (torch.full((2, T, heads, d), float("nan"), dtype=torch.bfloat16, device=DEV) for heads in (hq, hkv))
    k_rot[1] = k
    for i in range(2):
        B.earn_prefill_attn(desc, q, k_rot[1] if i else k, v, cu, None, batch, T, max(lens), out[i], k_rot[i], None, ws)
    torch.cuda.synchronize()
    assert torch.equal(out[1], out[0]) and torch.equal(k_rot[1], k_rot[0])
    ref = O.prefill_attn(*(W.to_f64(x.cpu()) for x in (q, k, v)), cu.cpu().numpy())
    check(out[1], ref["out"], torch.bfloat16, "outputs")
    check(k_rot[1], ref["k_rot"], torch.bfloat16, "rotated keys")


# Short and medium key lists have a kernel of their own (blocks of 32 keys dealt to 2, 3, 4 or 8 waves); setting any launch
# shape of the general decode kernels sends the call to those.  Both against the oracle, at the edges of the blocks, of the
# wave counts and of the rule that chooses, with generated parts of one and several blocks, and through an ancestor table.
SHORT_CASES = [
    # hq, hkv, d, shared lengths, streams per sequence, gen_cap, generated lengths (cycled), ancestor table
    (4, 4, 128, [0, 1, 31, 32], 1, 1, [0], False),
    (12, 2, 128, [33, 63, 64, 2], 1, 34, [31, 32, 33, 0], False),
    (14, 2, 64, [65, 96, 97, 127], 1, 5, [4, 0, 3], False),
    (16, 2, 128, [128, 129, 255], 1, 3, [2, 1], False),
    (2, 1, 64, [256, 257, 1000, 955], 1, 24, [23, 0, 11], False),
    (8, 2, 64, [30, 33, 64], 5, 8, [7, 0, 3, 6], True),
    (3, 3, 128, [60, 257], 3, 70, [69, 32, 31, 64], True),
    (12, 2, 128, [16, 0, 5], 1, 500, [499, 0, 262], False),       # register rows and a long generated part, few workgroups
    (4, 4, 64, [16, 30], 1, 130, [129, 95], False),
    (8, 2, 64, [16] * 140, 1, 70, [69, 3, 33], False),            # more workgroups than CUs
]


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("hq,hkv,d,slens,beams,gen_cap,glens,table", SHORT_CASES)
def test_decode_short_key_lists(hq, hkv, d, slens, beams, gen_cap, glens, table, general):
    B = _B()
    batch, S = len(slens), len(slens) * beams
    g = torch.Generator().manual_seed(sum(slens) + hq)
    rnd = lambda *shape: torch.randn(*shape, generator=g).to(torch.bfloat16)
    s2s = [u // beams for u in range(S)]
    glens = [glens[u % len(glens)] for u in range(S)]
    cu = np.concatenate([[0], np.cumsum(slens)]).astype(np.int32)
    sk, sv, q, kn, vn = rnd(int(cu[-1]), hkv, d), rnd(int(cu[-1]), hkv, d), rnd(S, hq, d), rnd(S, hkv, d), rnd(S, hkv, d)
    gk, gv = rnd(S, gen_cap, hkv, d), rnd(S, gen_cap, hkv, d)
    q_pos = [slens[s2s[u]] + glens[u] for u in range(S)]
    o_gk, o_gv, src = W.to_f64(gk), W.to_f64(gv), None
    if table:   # the oracle's streams own copies of the rows that the table names
        # an ancestor's row must not be one that this call appends
        src = torch.tensor([[next(w for w in range((u * 7 + j) % S, 2 * S) if glens[w % S] != j) % S for j in range(gen_cap)]
                            for u in range(S)], dtype=torch.int32)
        o_gk, o_gv = (x[src.numpy(), np.arange(gen_cap)[None, :]].copy() for x in (o_gk, o_gv))
    ref = O.decode_attn(W.to_f64(q), W.to_f64(kn), W.to_f64(vn), q_pos, W.to_f64(sk), W.to_f64(sv), cu, s2s, o_gk, o_gv, glens)
    i32 = lambda x: torch.tensor(list(x), dtype=torch.int32, device=DEV)
    dev = lambda x: x.to(DEV)
    desc = B.make_desc(torch.bfloat16, hq, hkv, d)
    d_gk, d_gv, out = dev(gk), dev(gv), torch.full((S, hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(max(B.earn_decode_workspace_bytes(desc, S, batch, max(slens), gen_cap), 256), dtype=torch.uint8, device=DEV)
    args = (desc, dev(q), dev(kn), dev(vn), i32(q_pos), dev(sk), dev(sv), i32(cu), i32(s2s), d_gk, d_gv, i32(glens))
    if general:
        B.earn_set_tuning("decode_vec_wgs", 1024)   # the default, set: the general kernels
    try:
        if table:
            B.earn_decode_attn_beams(*args, dev(src), gen_cap, S, batch, max(slens), out, ws)
        else:
            B.earn_decode_attn(*args, gen_cap, S, batch, max(slens), out, ws)
        torch.cuda.synchronize()
    finally:
        if general:
            B.earn_set_tuning("decode_vec_wgs", 0)
    check(out, ref["out"], torch.bfloat16, "outputs")
    at = torch.arange(S)
    check(d_gk.cpu()[at, glens], o_gk[np.arange(S), glens], torch.bfloat16, "appended keys")
    expect_k, expect_v = gk.clone(), gv.clone()
    expect_k[at, glens], expect_v[at, glens] = d_gk.cpu()[at, glens], vn
    assert torch.equal(d_gk.cpu(), expect_k) and torch.equal(d_gv.cpu(), expect_v)


# Short sequences have a prefill kernel of their own (32, 64 or 128 rows; a pair's query rows in groups of 16 dealt to waves
# and, with few pairs, to several workgroups): the edges of the groups, of the 32-key blocks and of the row limits, sequences
# of one row and none, explicit positions, with and without rotation, a cache copy and the log-sum-exp.
@pytest.mark.parametrize("rope,keep_keys", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("hq,hkv,d,lens", [
    (4, 4, 128, [32, 1, 0, 17]), (12, 2, 128, [16, 15, 31]), (7, 1, 64, [33, 64, 63, 2]), (32, 8, 128, [64] * 70),
    (6, 2, 128, [65, 96, 97, 128]), (8, 4, 64, [127, 3, 128])])
def test_prefill_short_sequences(hq, hkv, d, lens, rope, keep_keys):
    B = _B()
    T, batch = sum(lens), len(lens)
    g = torch.Generator().manual_seed(T + hq)
    rnd = lambda heads: torch.randn(T, heads, d, generator=g).to(torch.bfloat16)
    q, k, v = rnd(hq), rnd(hkv), rnd(hkv)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pos = np.concatenate([np.sort(np.random.default_rng(n).choice(4000, n, replace=False)) for n in lens]).astype(np.int32)
    base = 10000.0 if rope else 0.0
    desc = B.make_desc(torch.bfloat16, hq, hkv, d, 0.0, base)
    out = torch.full((T, hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((T, hq), float("nan"), dtype=torch.float32, device=DEV)
    d_k = k.to(DEV)
    k_rot = torch.full_like(d_k, float("nan")) if keep_keys else None
    ws = torch.empty(max(B.earn_prefill_workspace_bytes(desc, batch, T, max(lens), keep_keys), 256), dtype=torch.uint8, device=DEV)
    B.earn_prefill_attn(desc, q.to(DEV), d_k, v.to(DEV), torch.from_numpy(cu).to(DEV), torch.from_numpy(pos).to(DEV), batch, T,
                        max(lens), out, k_rot, lse, ws)
    torch.cuda.synchronize()
    ref = O.prefill_attn(W.to_f64(q), W.to_f64(k), W.to_f64(v), cu, pos, rope_base=base)
    for s in range(batch):
        check(out[cu[s]:cu[s + 1]], ref["out"][cu[s]:cu[s + 1]], torch.bfloat16, f"sequence {s}")
    # q and k enter a score rounded to at most 2^-9 of their elements, evenly spread: the score of rows of N(0, 1) is wrong by
    # 2^-9 sqrt(2 / 3) = 1.6e-3 (standard deviation), a log-sum-exp by at most what its largest scores are.  2^-7 is five of
    # them, for a few ten thousand rows; 2^-6 leaves room for rows of twice the usual size.
    assert float((lse.cpu().double() - torch.from_numpy(ref["lse"])).abs().max()) <= 2.0 ** -6
    if keep_keys:
        check(k_rot, ref["k_rot"], torch.bfloat16, "rotated keys")
        assert rope or torch.equal(k_rot, d_k)
