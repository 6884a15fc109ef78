"""The launches' index arithmetic (csrc/work_order.h), compiled for the host: every workgroup of a launch, in dispatch order."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_00715_amd", "csrc")
SOURCE = r'''
#include "work_order.h"
using namespace earn;
extern "C" int takes(int longest, int mean, long long pairs, int in_place) { return short_prefill_takes(longest, mean, pairs, in_place); }
extern "C" int waves(int max_shared_len, int gen_cap, long long workgroups) { return short_decode_waves(max_shared_len, gen_cap, workgroups); }
extern "C" int groups(int n_streams, int batch, int gq, int (*out)[3]) {
  const BeamGroups g = beam_groups(n_streams, batch, gq);
  for (int i = 0; i < g.count; ++i) { const BeamGroup b = beam_group(g, i); out[i][0] = b.first; out[i][1] = b.count; out[i][2] = b.slot; }
  return g.count;
}
extern "C" int group_of(int n_streams, int batch, int gq, int u) { return beam_group_of(beam_groups(n_streams, batch, gq), u); }
extern "C" int runs_taken(int n_streams, int batch, int gq, int len) { return beam_runs(beam_groups(n_streams, batch, gq), n_streams, batch, len); }
extern "C" int beams_kernel(int n_streams, int batch, int hkv, int gq, int d, int len, int cap, int layers, int pass) {
  return (int)beam_kernel(n_streams, batch, hkv, gq, d, len, cap, layers, pass);
}
extern "C" void divide(unsigned d, const unsigned* n, unsigned* out, int count) {
  const FastDiv f = FastDiv::of(d);
  for (int i = 0; i < count; ++i) out[i] = f.div(n[i]);
}
extern "C" int fits(int n, int per, int threads) { return run_fits(n, per, threads); }
extern "C" long long runs(int n, int per, int even, int (*out)[3], long long limit) {
  const long long w = run_workgroups(n, per);
  for (long long i = 0; i < w && i < limit; ++i) {
    const RunItem r = run_item((unsigned)i, n, FastDiv::of(per), even);
    out[i][0] = r.item; out[i][1] = r.sub; out[i][2] = r.valid;
  }
  return w;
}
extern "C" long long backward(long long pairs, int max_seqlen, int rows, int heads, int* chunk, int (*out)[3], long long limit) {
  const BackwardPlan b = backward_plan(pairs, max_seqlen, rows, heads);
  const BackwardGrid g = backward_grid(b, heads);
  const long long n = (long long)g.x * g.y * g.z;
  *chunk = b.chunk;
  for (long long i = 0; i < n && i < limit; ++i) {
    const BackwardItem it = backward_item(b, heads, (int)(i / g.x), (int)(i % g.x));
    out[i][0] = (int)it.pair; out[i][1] = it.head; out[i][2] = it.step;
  }
  return n;
}
extern "C" void backward_grid_of(long long pairs, int max_seqlen, int rows, int heads, long long (*g)[3]) {
  const BackwardGrid b = backward_grid(backward_plan(pairs, max_seqlen, rows, heads), heads);
  (*g)[0] = b.x; (*g)[1] = b.y; (*g)[2] = b.z;
}
extern "C" int block_of(int keys, long long pairs, int max_seqlen, int rows, int heads, int blocks, int step) {
  return backward_block(keys ? Owned::kKeys : Owned::kQueries, backward_plan(pairs, max_seqlen, rows, heads), blocks, step);
}
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "order.so"), str(d / "order.cpp")],
                   check=True)
    so = ctypes.CDLL(str(d / "order.so"))
    so.runs.restype = ctypes.c_longlong
    so.runs.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_longlong]
    so.backward.restype = ctypes.c_longlong
    so.backward.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_longlong]
    so.block_of.argtypes = [ctypes.c_int, ctypes.c_longlong, *[ctypes.c_int] * 5]
    return so


@pytest.mark.parametrize("keys", [False, True])
@pytest.mark.parametrize("rows", [64, 128])
@pytest.mark.parametrize("batch,hkv,gq,lo,hi", [(16, 8, 4, 272, 1040), (1, 1, 1, 1, 64), (3, 2, 7, 0, 2080), (64, 8, 4, 68, 68),
                                                (5, 32, 1, 1, 300), (2, 8, 4, 4096, 4096)])
def test_backward_covers_every_block_longest_first(lib, batch, hkv, gq, lo, hi, rows, keys):
    rng = np.random.default_rng(batch + hi)
    lens = rng.integers(lo, hi + 1, batch)
    lens[batch // 2] = hi
    heads, pairs = (1 if keys else gq), batch * hkv
    chunk = ctypes.c_int()
    n = lib.backward(pairs, hi, rows, heads, ctypes.byref(chunk), None, 0)
    item = np.empty((n, 3), dtype=np.int32)
    assert lib.backward(pairs, hi, rows, heads, ctypes.byref(chunk), item.ctypes.data, n) == n
    seen, last = {}, {}
    for i, (pair, head, step) in enumerate(item.tolist()):
        if pair >= pairs:
            continue
        length = int(lens[pair // hkv])
        blocks = (length + rows - 1) // rows
        blk = lib.block_of(keys, pairs, hi, rows, heads, blocks, step)
        if not 0 <= blk < blocks:
            continue
        seen[pair, head, blk] = seen.get((pair, head, blk), 0) + 1
        # the XCD that a workgroup id goes to keeps the pair; within a chunk of its pairs the work does not grow
        assert pair % 8 == i % 8
        work = (blocks - blk) if keys else blk + 1
        group = (i % 8, pair // 8 // chunk.value)
        assert last.get(group, 1 << 30) >= work
        last[group] = work
    assert set(seen.values()) <= {1}
    assert len(seen) == sum((int(x) + rows - 1) // rows for x in lens) * hkv * heads


@pytest.mark.parametrize("rows,threads", [(128, 256), (64, 512)])
@pytest.mark.parametrize("batch,hkv,gq,longest", [(65535, 8, 4, 1040), (65535, 32, 1, 2080), (65535, 64, 1, 64), (1, 1, 8, 262144)])
def test_backward_grid_fits_a_launch(lib, batch, hkv, gq, longest, rows, threads):
    """Every batch that the entry point takes (up to 65535 sequences) is one launch: 2^32 threads in x, 65535 workgroups in y, z."""
    for heads in (1, gq):
        g = (ctypes.c_longlong * 3)()
        lib.backward_grid_of(ctypes.c_longlong(batch * hkv), longest, rows, heads, ctypes.byref(g))
        assert g[0] * threads < 2 ** 32 and g[1] <= 65535 and g[2] <= 65535
        assert g[0] * g[1] * g[2] >= batch * hkv * heads * ((longest + rows - 1) // rows)


@pytest.mark.parametrize("even", [True, False])
@pytest.mark.parametrize("per", [1, 2, 8, 24])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 10, 17, 20, 25, 64, 255, 1000])
def test_runs_cover_every_item_once(lib, n, per, even):
    w = lib.runs(n, per, even, None, 0)
    out = np.empty((w, 3), dtype=np.int32)
    lib.runs(n, per, even, out.ctypes.data, w)
    xcd = np.arange(w) % 8
    ok = out[:, 2] == 1
    assert sorted(map(tuple, out[ok, :2].tolist())) == [(i, s) for i in range(n) for s in range(per)]
    counts = np.bincount(xcd[ok], minlength=8)
    assert not even or counts.max() - counts.min() <= 1       # not five XCDs out of eight
    for x in range(8):                                         # consecutive items
        items = np.unique(out[ok & (xcd == x), 0])
        assert items.size == 0 or items[-1] - items[0] + 1 == items.size


@pytest.mark.parametrize("shared,gen_cap,workgroups,waves", [
    (0, 32, 8, 2), (32, 32, 10000, 2), (33, 16, 256, 3), (64, 16, 257, 3), (65, 1, 8, 4), (128, 32, 5000, 4), (129, 1, 8, 8),
    # generated rows count where a CU has one workgroup at most
    (16, 33, 256, 3), (16, 33, 257, 2), (16, 96, 256, 4), (16, 129, 256, 8), (16, 1000, 8, 8), (16, 1000, 2048, 2), (64, 1000, 2048, 3)])
def test_short_decode_waves(lib, shared, gen_cap, workgroups, waves):
    assert lib.waves(shared, gen_cap, ctypes.c_longlong(workgroups)) == waves


@pytest.mark.parametrize("n,per,threads,fits", [(8, 8, 512, True), ((1 << 20) - 8, 8, 512, True), (1 << 20, 8, 512, False),
                                                ((1 << 20) - 7, 8, 512, False), (1 << 24, 1, 256, False), ((1 << 31) - 1, 64, 256, False)])
def test_run_fits_a_grid_dimension(lib, n, per, threads, fits):
    assert bool(lib.fits(n, per, threads)) == fits


@pytest.mark.parametrize("longest,mean,pairs,in_place,short", [
    (64, 1, 260, True, True), (1, 1, 1, True, True), (128, 10, 512, True, True), (128, 10, 511, True, False),
    (96, 72, 128, True, True), (96, 71, 128, True, False), (97, 97, 128, True, False), (65, 65, 127, True, False), (65, 65, 257, True, False),
    (128, 32, 260, False, True), (128, 31, 260, False, False), (128, 10, 127, False, True), (128, 128, 40, False, True)])
def test_short_prefill_takes(lib, longest, mean, pairs, in_place, short):
    assert bool(lib.takes(longest, mean, ctypes.c_longlong(pairs), in_place)) == short


@pytest.mark.parametrize("d", [1, 2, 3, 5, 7, 12, 17, 32, 100, 1041, 65535, 65537, 524288, 2 ** 30 + 1, 2 ** 31 - 1])
def test_division_by_multiplication(lib, d):
    k = np.arange(1, 2000, dtype=np.uint64)
    n = np.concatenate([np.arange(2000, dtype=np.uint64), 2 ** 31 - k, k * d, k * d - 1, 2 ** 31 // d * d - np.array([0, 1], dtype=np.uint64),
                        np.random.default_rng(d).integers(0, 2 ** 31, 20000, dtype=np.uint64)])
    n = n[n < 2 ** 31].astype(np.uint32)
    out = np.empty_like(n)
    lib.divide(ctypes.c_uint(d), n.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p), len(n))
    assert np.array_equal(out, n // np.uint32(d))


@pytest.mark.parametrize("gq", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("n_streams,batch", [(10, 1), (160, 16), (161, 16), (320, 16), (7, 3), (2, 1), (1000, 7), (640, 64), (45, 44)])
def test_beam_groups_hold_every_stream_once(lib, n_streams, batch, gq):
    out = np.empty((n_streams, 3), dtype=np.int32)
    n = lib.groups(n_streams, batch, gq, out.ctypes.data_as(ctypes.c_void_p))
    first, count, slot = out[:n].T
    assert n <= n_streams and count.min() >= 1 and count.max() * gq <= max(16, gq)
    assert np.concatenate([np.arange(f, f + c) for f, c in zip(first, count)]).tolist() == list(range(n_streams))
    assert [lib.group_of(n_streams, batch, gq, u) for u in range(n_streams)] == np.repeat(np.arange(n), count).tolist()
    # streams in the order of their sequences, as many of each as can be, stay in their groups
    sequence = np.arange(n_streams) * batch // n_streams
    runs = [1 + int((np.diff(sequence[f:f + c]) != 0).sum()) for f, c in zip(first, count)]
    assert max(runs) <= lib.runs_taken(n_streams, batch, gq, 2048)
    if n_streams % batch == 0:                  # no group over two sequences of the usual layout
        w = n_streams // batch
        assert np.array_equal(slot, first // w) and np.array_equal(slot, (first + count - 1) // w)


GENERAL, PER_STREAM, GROUPED = range(3)


# The fastest kernel of each size as measured (us a layer: general, one workgroup per stream, groups), or one within a tenth of that
@pytest.mark.parametrize("streams,batch,hkv,gq,d,rows,cap,layers,n_pass,kernel", [
    (10, 1, 8, 4, 128, 64, 8, 1, 1, PER_STREAM),
    (160, 16, 8, 4, 128, 64, 8, 1, 1, GROUPED),              # 14.3  13.1   8.8
    (160, 16, 8, 4, 128, 32, 8, 1, 1, PER_STREAM),           # 15.4   8.9   8.2 (where the two cross)
    (160, 16, 8, 4, 128, 33, 8, 1, 1, GROUPED),              # 14.6  11.9   8.4
    (160, 16, 8, 4, 128, 100, 8, 1, 1, GROUPED),             # 15.2  17.7  11.3
    (160, 16, 8, 4, 128, 512, 8, 1, 1, GENERAL),             # 23.6  52.5  25.0
    (160, 16, 8, 4, 128, 16, 32, 1, 1, PER_STREAM),          # 25.6   9.3  11.5
    (160, 16, 8, 4, 128, 64, 200, 1, 1, PER_STREAM),         # 53.8  26.6  28.7
    (160, 16, 8, 4, 128, 64, 8, 24, 1, GROUPED),             #  6.7   7.3   5.0
    (80, 8, 2, 6, 128, 32, 8, 16, 1, PER_STREAM),            # 1.04  0.99  1.17
    (80, 8, 2, 6, 128, 200, 8, 16, 1, GENERAL),              # 1.23  3.43  2.46
    (320, 16, 8, 4, 128, 64, 8, 1, 2, GROUPED),              # 19.8  19.9  14.1
    (640, 64, 2, 7, 64, 256, 8, 1, 2, GENERAL),              # 14.1  19.1  18.8
    (640, 64, 2, 7, 64, 64, 8, 1, 2, PER_STREAM),            # 12.3   7.7   7.4
    (128, 32, 2, 7, 64, 512, 8, 1, 1, GROUPED),              # 14.3   9.2   9.7
    (64, 16, 4, 1, 64, 128, 16, 1, 1, PER_STREAM),           # 10.0   6.7   6.8
    (1400, 140, 2, 6, 128, 25, 16, 1, 1, PER_STREAM),        # 37.2  16.1  19.5
    (1400, 140, 2, 6, 128, 33, 16, 1, 1, PER_STREAM),        # 36.3  20.7  20.4
    (1400, 140, 2, 7, 64, 25, 16, 1, 2, PER_STREAM),         # 38.9  10.6  12.0
    (160, 16, 8, 4, 128, 2300, 8, 1, 1, GENERAL)])
def test_beam_kernel(lib, streams, batch, hkv, gq, d, rows, cap, layers, n_pass, kernel):
    assert lib.beams_kernel(streams, batch, hkv, gq, d, rows, cap, layers, n_pass) == kernel


def test_sizes_of_the_group_tests_are_grouped(lib):
    from test_gpu_beam_groups import ANY_ORDER, ANY_ORDER_ROOM, GROUPED as SIZES, STAY_AWAY, TIMED
    runs = [(x, 8, layers, more) for x in SIZES for layers in (1, 3) for more in (0, 1)]
    runs += [(x[:6], ANY_ORDER_ROOM, x[6], 0) for x in ANY_ORDER] + [(x, 8, 1, 0) for x in STAY_AWAY + TIMED]
    for (hq, hkv, d, batch, beams, rows), cap, layers, more in runs:
        n, gq = batch * beams + more, hq // hkv
        rows_bound, rows_mean = gq * (n - batch + 1), gq * ((n + batch - 1) // batch)
        n_pass = (rows_mean + 63) // 64 if rows_bound > 32 and rows_mean > 64 else 1
        assert lib.beams_kernel(n, batch, hkv, gq, d, rows, cap, layers, n_pass) == GROUPED, (hq, hkv, d, batch, beams, rows, layers, more)


def test_kernels_of_the_beam_search_tests(lib):
    from test_gpu_beams import BEAM_CASES
    kernels = [lib.beams_kernel(len(lens) * beams, len(lens), hkv, hq // hkv, d, max(lens), steps, 1, 2 if beams * hq // hkv > 64 else 1)
               for _, hq, hkv, d, lens, beams, steps, _ in BEAM_CASES[:3]]
    assert kernels == [GROUPED, PER_STREAM, PER_STREAM]
