// Which work a workgroup takes: index arithmetic of the launches and kernels, free of device code, so that it can be checked
// on the host for every workgroup of a launch.
#pragma once
#ifdef __HIPCC__
#define EARN_INDEX __host__ __device__ __forceinline__
#else
#define EARN_INDEX inline
#endif

namespace earn {

// Division of n < 2^31 by a divisor that the host knows: a multiplication in the kernel, where dividing a wave-uniform number
// takes some thirty vector instructions.  2^(31 + shift) <= mul d < 2^(31 + shift) + d with d <= 2^shift, so n mul / 2^(31 +
// shift) is less than 1 / d above n / d and rounds down to the same.
struct FastDiv {
  unsigned d, mul;
  int shift;
  static FastDiv of(unsigned d) {
    FastDiv f{d, 0, 0};
    while ((1ull << f.shift) < d) ++f.shift;
    f.mul = (unsigned)(((1ull << (31 + f.shift)) + d - 1) / d);
    return f;
  }
  EARN_INDEX unsigned div(unsigned n) const { return (unsigned)((unsigned long long)n * mul >> (31 + shift)); }
};

constexpr int kXcds = 8;  // accelerator complex dies, each with a private L2; consecutive workgroup ids go to them in turn

// ---- short decode and prefill: an XCD takes a run of consecutive units, `per` workgroups of each item (stream, sequence) ----
// Even runs: XCD x has units [x n per / 8, (x + 1) n per / 8), whichever items they belong to, so that a single item is spread
// over the XCDs too.  Whole runs: n / 8 items, rounded up, each, and what is left to the last ones (9 items keep 5 XCDs busy, 17
// six).
EARN_INDEX long long run_workgroups(int n, int per) { return ((long long)n + kXcds - 1) / kXcds * kXcds * per; }
// what one grid dimension takes: fewer than 2^32 threads
EARN_INDEX bool run_fits(int n, int per, int threads) { return run_workgroups(n, per) * threads < (1ll << 32); }
struct RunItem { int item, sub; bool valid; };   // sub: 0 .. per - 1
EARN_INDEX RunItem run_item(unsigned id, int n, const FastDiv& by_per, bool even) {
  const int per = (int)by_per.d, xcd = (int)(id % kXcds), at = (int)(id / kXcds), units = n * per;
  const int base = units / kXcds, extra = units % kXcds, whole = (n + kXcds - 1) / kXcds * per;
  const int first = even ? xcd * base + xcd * extra / kXcds : xcd * whole;
  const int count = even ? base + ((xcd + 1) * extra / kXcds - xcd * extra / kXcds) : whole;
  const int unit = first + at, item = (int)by_per.div((unsigned)unit);
  return RunItem{item, unit - item * per, at < count && unit < units};
}

// Does the short prefill kernel take a batch of grouped heads whose longest sequence has `longest` rows (up to 128) and its
// average one `mean`?  Up to 64 rows always.  Beyond, a pair is one 8-wave workgroup, one or two to a CU, and what counts is
// whether the pairs fill the GPU.  The medium kernel -> it, us a layer.  512 pairs and more: 64 sequences, 32 / 8 heads of 128,
// 96 rows 24.3 -> 17.1, lengths of 1-128 31.9 -> 30.6; 200, 12 / 2 heads, 128 rows 61 -> 57; at worst 400, 14 / 2 heads of 64,
// lengths of 1-128 39 -> 42.  Fewer pairs, keys read in place: even lengths up to 96 rows on 128 - 256 pairs gain (64, 14 / 2
// heads, 65 / 96 rows 14.1 -> 10.4, 16.0 -> 14.8), the rest lose (260 pairs, 128 rows 21.9 -> 30.0, ragged 17.4 -> 28; 66 pairs,
// 128 rows 1.25 times the time; 40 pairs, 12 / 2 heads 9.4 -> 11.7).  With keys to rotate or copy, a launch of its own for the
// medium kernel, it gains except where most sequences are much shorter than the longest (130, 14 / 2 heads, one of 128 rows
// among some of about 12: 18.6 -> 23.2; 8 / 1 heads 23.2 -> 32.5).
EARN_INDEX bool short_prefill_takes(int longest, int mean, long long pairs, bool keys_in_place) {
  if (longest <= 64 || pairs >= 512) return true;
  if (keys_in_place) return pairs >= 128 && pairs <= 256 && longest <= 96 && 4ll * mean >= 3ll * longest;
  return pairs < 128 || 4ll * mean >= longest;
}
// Medium and long prefill: workgroups of a (sequence, kv head) pair whose waves take units of 32 rows of one query head.
EARN_INDEX int unit_blocks(int rows, int heads, int waves) { return (int)(((rows + 31ll) / 32 * heads + waves - 1) / waves); }
// fp32 prefill: are there so few workgroups of 16 query rows (a CU holds one) that their chains, not the products, are what a
// launch costs: 512 of 64 elements, 256 of 128?  Then eight waves share a workgroup's keys and rotate them themselves, in one launch;
// else 32 rows share them, in four waves, behind a rotation pass.  The line lies where the two were measured to cross.  us,
// rotating / eight waves / four waves: 2 sequences of 132 rows, 4 heads of 64 (72 workgroups) 10.3 / 12.2 / 16.0; 8 of them (288) 16.0 /
// 17.6 / 17.2; 16 (576) 22.1 / 24.3 / 21.2; 2 of 64, 32 / 8 heads of 128 (256) 13.9 / 14.7 / 22.0; 3 of them (384) 25.6 / 23.7 / 22.6; one
// of 256, 16 / 4 heads of 128 (256), whose late rows rotate many keys, 22.8 / 20.3 / 31.9; one of 512, 12 / 2 (384) 67.9 / 47.3 / 43.8.
EARN_INDEX bool f32_few_workgroups(int rows, int hq, int d, long long sequences) { return (rows + 15ll) / 16 * hq * sequences * d <= 256 * 128; }
// Streams that share a workgroup of the short decode over beams: up to 16 / gq consecutive ones, whose query heads fill the 16
// columns of a product, in equal groups of the W = n_streams / batch streams that a sequence usually has side by side (`slot`;
// any other layout is served too, group by group).  No even number per sequence: all streams are one slot.
struct BeamGroups { int count, group, slot_streams; FastDiv per_slot; };
EARN_INDEX BeamGroups beam_groups(int n_streams, int batch, int gq) {
  BeamGroups g;
  g.slot_streams = n_streams % batch == 0 ? n_streams / batch : n_streams;
  const int most = 16 / gq < 1 ? 1 : 16 / gq;
  const int per_slot = (g.slot_streams + most - 1) / most;
  g.group = (g.slot_streams + per_slot - 1) / per_slot;
  g.per_slot = FastDiv::of((unsigned)((g.slot_streams + g.group - 1) / g.group));
  g.count = n_streams / g.slot_streams * (int)g.per_slot.d;
  return g;
}
struct BeamGroup { int first, count, slot; };
EARN_INDEX BeamGroup beam_group(const BeamGroups& g, int i) {
  BeamGroup b;
  b.slot = (int)g.per_slot.div((unsigned)i);
  const int at = (i - b.slot * (int)g.per_slot.d) * g.group, rest = g.slot_streams - at;
  b.first = b.slot * g.slot_streams + at;
  b.count = rest < g.group ? rest : g.group;
  return b;
}
EARN_INDEX int beam_group_of(const BeamGroups& g, int u) {
  const int slot = u / g.slot_streams;
  return slot * (int)g.per_slot.d + (u - slot * g.slot_streams) / g.group;
}
// Runs of streams of one sequence that a group takes as they come: those that streams in the order of their sequences give it, and
// as many more as are ten blocks of 32 rows to walk.  A group with more of them looks its streams up anew, about 3 us.  us, streams
// u of sequences u % batch, groups as they come -> anew: 16 x 20 streams, 32 / 8 heads, 16 rows 18.3 -> 23.3; 8 x 10, 8 / 8 heads of
// 64, 64 rows 15.1 -> 10.4; 16 x 10, 32 / 8 heads, 64 rows 9.9 either way, 256 rows 37.7 -> 33.2; 8 x 10, 32 / 32 heads, 256 rows 60
// -> 21.9.
EARN_INDEX int beam_runs(const BeamGroups& g, int n_streams, int batch, int shared_len) {
  const int per_sequence = n_streams / batch, blocks = (shared_len + 31) / 32;
  const int in_order = n_streams % batch == 0 ? 1 : (g.group + per_sequence - 1) / per_sequence + 1;
  return in_order + 10 / (blocks < 1 ? 1 : blocks);
}
// Waves of a short decode workgroup: one per block of 32 shared keys and one for the generated rows, eight for longer lists.
// With no more workgroups than CUs, nothing else hides a wave's round trips, so the blocks that the generated rows may come to
// count too.  us, 16 shared rows, waves by shared rows -> by all: one sequence, 32 / 8 heads, 249 / 999 generated rows 14.5 /
// 39.8 -> 9.5 / 18.8, 4 heads of 64 in 8 sequences, 499 / 739 rows 15.9 / 21.1 -> 9.3 / 10.7 (general kernels 10.6 / 11.0);
// place for 499 but 62 in use, 8.0 -> 6.8.  With more workgroups the fewer waves leave room for more of them: 256 sequences, 12
// / 2 heads, 31 of 250 rows in use 7.2 -> 11.8, all 249 19.8 -> 22.2.
EARN_INDEX int short_decode_waves(int max_shared_len, int gen_cap, long long workgroups) {
  const long long generated = workgroups <= 256 ? ((long long)gen_cap + 31) / 32 : 1;
  const long long blocks = ((long long)max_shared_len + 31) / 32 + generated;
  return blocks <= 2 ? 2 : blocks == 3 ? 3 : blocks <= 5 ? 4 : 8;
}
// ... and of a group's, four or eight
EARN_INDEX int beam_group_waves(const BeamGroups& g, int max_shared_len, int gen_cap) {
  return short_decode_waves(max_shared_len, g.group * gen_cap, 1) <= 4 ? 4 : 8;
}
// Streams that share caches: which kernel?  The one that a count of its time says is the fastest, in us, for rows of 128 elements (all
// but the first figures two thirds of that for 64); the generated part counts with half the rows that there is room for.
//   general     11.5 for each round on the XCD with the most workgroups, 0.85 for 64 rows of a split, and for each stream of a
//               sequence 0.45 and 1.8 for 32 generated rows, over the splits;
//   per stream  3.1 and 1.2 for each step of 32 rows of a workgroup's waves; beyond half a round 0.45 for 256 workgroups' 32 rows;
//   grouped     4.8 and 1.15 for each step; beyond half a round 1.7 for 256 workgroups and 0.4 for 32 rows of theirs;
//               workgroups of eight waves 0.5 / 0.8 more, and 3.1 / 4.5 for 256 of them (one or two fill a CU).
// Figures that put the three in the right order for 1996 sizes, most of them drawn at random: 1 to 160 sequences, 2 to 24 streams each,
// eleven head layouts, caches of 4 to 1500 rows, 4 to 200 generated rows, 1 to 24 layers in a launch.  The kernel named takes 1.011 times
// as long as the best of them on the geometric mean, more than 1.25 times at 0.8 %, at most 2.6 times (1.022 and 2.5 % on 600 of the
// sizes by figures from 906 others; thresholds that told the kernels apart by rows to read again: 1.090, 14 %, 12 times).  16 x 10 streams, 32 /
// 8 heads, general / per stream / grouped: 32 rows 15.4 / 8.9 / 8.2, 64 rows 14.3 / 13.1 / 8.8, 512 rows 23.6 / 52.5 / 25.0, 16 rows and 30
// generated 25.6 / 9.3 / 11.5; 140 x 10, 12 / 2 heads, 25 rows 37.2 / 16.1 / 19.5.
enum class BeamKernel { kGeneral, kPerStream, kGrouped };
EARN_INDEX BeamKernel beam_kernel(int n_streams, int batch, int hkv, int gq, int d, int shared_len, int gen_cap, int n_layers, int n_pass) {
  if ((long long)shared_len + gen_cap > 2304) return BeamKernel::kGeneral;   // beyond what was measured
  auto over = [](long long a, long long b) { return (a + b - 1) / b; };
  auto past_half_round = [](long long workgroups) { return workgroups > 128 ? (double)workgroups / 256. - 0.5 : 0.; };
  const double size = (d + 64) / 192.;
  const long long generated = gen_cap < 2 ? 1 : gen_cap / 2, blocks = over(shared_len, 32);

  const long long lists = (long long)batch * n_pass;
  long long splits = over(256, lists * hkv * n_layers);
  if (splits > over(shared_len, 256)) splits = over(shared_len, 256);
  if (splits < 1) splits = 1;
  const double t_general = (double)over(over(lists * splits, kXcds) * hkv * n_layers, 32) *
                           (11.5 + size * (0.85 * (double)over(over(shared_len, 64), splits) +
                                          (double)over(n_streams, batch) * (0.45 + 1.8 / 32. * (double)generated) / (double)splits));

  const long long pairs = (long long)n_streams * hkv * n_layers, stream_blocks = blocks + over(generated, 32);
  const int waves = short_decode_waves(shared_len, gen_cap, pairs);
  const double t_per_stream = (waves == 8 ? 3.6 : 3.1) + size * (1.2 * (double)over(stream_blocks, waves) +
                              past_half_round(pairs) * ((waves == 8 ? 3.1 : 0.) + 0.45 * (double)stream_blocks));

  const BeamGroups g = beam_groups(n_streams, batch, gq);
  const long long workgroups = (long long)g.count * hkv * n_layers;
  const long long caches = n_streams % batch == 0 ? 1 : over(g.group - 1, n_streams / batch) + 1;   // of streams in the order of their sequences
  const long long group_blocks = blocks * caches + over(g.group * generated, 32);
  const int group_waves = beam_group_waves(g, shared_len, gen_cap);
  const double t_grouped = (group_waves == 8 ? 5.6 : 4.8) + size * (1.15 * (double)over(group_blocks, group_waves) +
                           past_half_round(workgroups) * ((group_waves == 8 ? 6.2 : 1.7) + 0.4 * (double)group_blocks));
  if (t_general <= t_per_stream && t_general <= t_grouped) return BeamKernel::kGeneral;
  return t_per_stream <= t_grouped ? BeamKernel::kPerStream : BeamKernel::kGrouped;
}

// ---- attention backward (bf16): (sequence, kv head) pairs, blocks of owned rows, query heads of the group ----
// An XCD keeps its own pairs, whose rows its L2 then holds.  It takes them in chunks, within a chunk longest work first over
// ALL its pairs: a block's work is the number of rows it is paired with (keys up to a query, queries from a key on), so with
// few pairs no long block is left to start when the GPU is about to run dry.
struct BackwardPlan {
  int n_blk;      // row blocks of the longest sequence
  int chunk;      // pairs an XCD works on together: about four rounds of its 64 workgroup slots
  int per_xcd;    // pairs of an XCD
};
EARN_INDEX BackwardPlan backward_plan(long long pairs, int max_seqlen, int block_rows, int heads) {
  BackwardPlan b;
  b.per_xcd = (int)((pairs + kXcds - 1) / kXcds);
  b.n_blk = (max_seqlen + block_rows - 1) / block_rows;
  const int fit = 256 / (b.n_blk * heads);
  b.chunk = fit < 1 ? 1 : fit < b.per_xcd ? fit : b.per_xcd;
  return b;
}
// A chunk is a row of the grid: what all chunks hold together may be more than one grid dimension takes (65535 sequences, 32
// heads, 9 blocks are 19 million workgroups).
struct BackwardGrid { unsigned x, y, z; };
EARN_INDEX BackwardGrid backward_grid(const BackwardPlan& b, int heads) {
  const unsigned chunks = (unsigned)((b.per_xcd + b.chunk - 1) / b.chunk), y = chunks < 32768u ? chunks : 32768u;
  return BackwardGrid{(unsigned)b.chunk * b.n_blk * heads * kXcds, y, (chunks + y - 1) / y};
}
// Workgroup `id` of chunk `chunk`.  step: 0 = the longest work of a chunk, n_blk - 1 the shortest.  pair may lie past the last
// one.
struct BackwardItem { long long pair; int head, step; };
EARN_INDEX BackwardItem backward_item(const BackwardPlan& b, int heads, int chunk, int id) {
  const int xcd = id % kXcds, k = id / kXcds;
  return BackwardItem{((long long)chunk * b.chunk + k / heads % b.chunk) * kXcds + xcd, k % heads, k / (b.chunk * heads)};
}
// The block of a sequence of `blocks` blocks that is step `step`; outside [0, blocks): none.  Queries are paired with the
// keys before them, so the last block is the longest work; keys with the queries after them: the first.
enum class Owned { kQueries, kKeys };
EARN_INDEX int backward_block(Owned rows, const BackwardPlan& b, int blocks, int step) {
  return rows == Owned::kQueries ? b.n_blk - 1 - step : blocks - b.n_blk + step;
}

}  // namespace earn
