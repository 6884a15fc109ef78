// Beam-search bookkeeping around the decode step (paper Appendix, implementation details: inference uses beam search
// with beam size 20).  Three pieces, none of which touches a K/V byte:
//   beam_topk      per sequence, the W best of the W * V candidates  score(beam w) + logprob(w, token t), ordered by
//                  (score descending, candidate index ascending): each winner names its parent beam and its token;
//   beam_reorder   the new beams' ancestor table: which physical stream's cache slot holds each earlier generated row.
//                  The decode kernels read generated rows through this table (DecodeParams::gen_src), so a beam step
//                  moves W * step integers per sequence instead of copying W * step K/V rows in every layer;
// Selection is exact and deterministic: candidates are compared as (score, index) pairs in a total order.
#include "common.h"

namespace earn {

constexpr int kTopkThreads = 256;
constexpr int kTopkChunk = 8192;   // candidates of one workgroup, 32 per thread, in registers
constexpr int kTopkMaxBeams = 64;
constexpr int kTopkSlabs = kTopkChunk / (4 * kTopkThreads);  // a slab: 4 consecutive candidates per thread
// candidates that can be left after the exact threshold: fewer than k threads hold any above it, and at most k equal ones
// are kept
constexpr int kTopkList = kTopkMaxBeams * 4 * kTopkSlabs + kTopkMaxBeams;

struct TopkSmem {
  float best[kTopkThreads];   // largest candidate of every quad of threads, or of every thread
  float threshold;
  int n_list;                 // candidates appended to the list
  int ties[kTopkSlabs][kTopkThreads / kWave];
  __align__(16) float list_v[kTopkList];
  __align__(16) int list_i[kTopkList];
  float pick_v[kTopkMaxBeams];
  int pick_i[kTopkMaxBeams];
};

// number of entries of x[0 .. n) (n a multiple of 4) that come before entry `at` of value `v` in descending order
__device__ __forceinline__ int count_before(const float* x, int n, float v, int at) {
  int before = 0;
#pragma unroll 8
  for (int j = 0; j < n; j += 4) {
    const f32x4 y = *(const f32x4*)&x[j];
#pragma unroll
    for (int e = 0; e < 4; ++e) before += (int)(y[e] > v) | ((int)(y[e] == v) & (int)(j + e < at));
  }
  return before;
}

// A thread's 32 candidates: slab s holds positions s * 1024 + 4 * thread + (0..3); bit 4 s + e of a mask stands for v[s][e].
// What is done to few of them runs as a loop over the bits of a mask: these kernels execute their code once, so every 64
// bytes of it are a fetch from memory (unrolled over the candidates, 23 KB of it, they took half as long again).
typedef float TopkValues[kTopkSlabs][4];
__device__ __forceinline__ int position_of(int bit) { return (bit >> 2) * 4 * kTopkThreads + 4 * (int)threadIdx.x + (bit & 3); }
__device__ __forceinline__ float value_of(const TopkValues& v, int bit) {
  float x = v[0][0];
#pragma unroll
  for (int b = 1; b < 4 * kTopkSlabs; ++b) {
    x = bit == b ? v[b >> 2][b & 3] : x;
    asm("" : "+v"(x));   // stays a chain of selects: as an indexed array the candidates would live in scratch memory
  }
  return x;
}
template <typename Cmp>
__device__ __forceinline__ unsigned mask_of(const TopkValues& v, Cmp cmp) {
  unsigned m = 0;
#pragma unroll
  for (int b = 0; b < 4 * kTopkSlabs; ++b) m |= (cmp(v[b >> 2][b & 3]) ? 1u : 0u) << b;
  return m;
}
__device__ __forceinline__ void append(const TopkValues& v, unsigned mask, TopkSmem& sm) {
#pragma unroll 1
  for (; mask; mask &= mask - 1) {
    const int bit = __ffs(mask) - 1, at = atomicAdd(&sm.n_list, 1);
    if (at < kTopkList) { sm.list_v[at] = value_of(v, bit); sm.list_i[at] = position_of(bit); }
  }
}

// Fills the list from the exact threshold, the k-th largest of the 256 threads' own maxima: what exceeds it, then the
// first equal candidates in order of position, up to k.  Returns the number of entries.  (Called by all threads.)
template <typename Exists>
__device__ __forceinline__ int list_from_exact_threshold(const TopkValues& v, int k, float best, TopkSmem& sm, Exists exists) {
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  __syncthreads();
  sm.best[tid] = best;
  if (tid == 0) sm.n_list = 0;
  __syncthreads();
  if (count_before(sm.best, kTopkThreads, best, tid) == k - 1) sm.threshold = best;
  __syncthreads();
  const float t = sm.threshold;
  append(v, mask_of(v, [t](float x) { return x > t; }), sm);
  unsigned equal = mask_of(v, [t](float x) { return x == t; });
#pragma unroll 1
  for (unsigned m = equal; m; m &= m - 1)   // missing candidates hold -inf
    if (!exists(position_of(__ffs(m) - 1))) equal &= ~(m & (0u - m));
#pragma unroll 1
  for (int s = 0; s < kTopkSlabs; ++s) {
    int n_equal = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) n_equal += __popcll(__ballot((equal >> (4 * s + e)) & 1));
    if (lane == 0) sm.ties[s][wave] = n_equal;
  }
  __syncthreads();
  const int n_above = sm.n_list, need = k - n_above;
  if (need <= 0) return n_above;
  int at = 0;   // equal candidates in the slabs so far
#pragma unroll 1
  for (int s = 0; s < kTopkSlabs && at < need; ++s) {
    int mine = at;
#pragma unroll
    for (int w = 0; w < kTopkThreads / kWave; ++w) { const int c = sm.ties[s][w]; mine += w < wave ? c : 0; at += c; }
    const unsigned own = (equal >> (4 * s)) & 15u;
#pragma unroll
    for (int e = 0; e < 4; ++e) mine += __popcll(__ballot((own >> e) & 1) & ((1ull << lane) - 1ull));
#pragma unroll 1
    for (unsigned m = own; m; m &= m - 1, ++mine)
      if (mine < need) {   // its own value, not t: zeros of either sign are equal
        const int bit = 4 * s + __ffs(m) - 1;
        sm.list_v[n_above + mine] = value_of(v, bit);
        sm.list_i[n_above + mine] = position_of(bit);
      }
  }
  return n_above + min(at, need);
}

// The k best of the workgroup's candidates in selection order (larger score first, lower position first among equals) into
// sm.pick_v / sm.pick_i (position; -1 and -inf when there are fewer than k).  Candidates that do not exist hold -inf;
// exists(position) tells them from those that merely score -inf.
//
// The k-th largest of 64 quads of threads' maxima is a lower bound of the k-th best (at least k candidates reach it).  What
// reaches it goes into a list, a few more than k entries as a rule, and the place of an entry is the number of entries
// before it.  A list that overflows (many equal scores, winners crowded into few threads) or a bound of -inf (fewer than k
// quads hold a finite score) takes the exact threshold instead, whose list cannot overflow.  One pass over the candidates
// and a few barriers, where picking one candidate per round took k passes.
template <typename Exists>
__device__ __forceinline__ void select_topk(const TopkValues& v, int k, TopkSmem& sm, Exists exists) {
  const int tid = threadIdx.x;
  float best = -INFINITY;
#pragma unroll
  for (int s = 0; s < kTopkSlabs; ++s) best = fmaxf(best, fmaxf(fmaxf(v[s][0], v[s][1]), fmaxf(v[s][2], v[s][3])));
  float quad = fmaxf(best, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(best), 0xB1, 0xf, 0xf, true)));  // [1,0,3,2]
  quad = fmaxf(quad, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(quad), 0x4E, 0xf, 0xf, true)));        // [2,3,0,1]
  if (tid % 4 == 0) sm.best[tid / 4] = quad;
  if (tid == 0) sm.n_list = 0;
  if (tid < k) { sm.pick_v[tid] = -INFINITY; sm.pick_i[tid] = -1; }
  __syncthreads();
  if (tid < kTopkThreads / 4) {
    const float mine = sm.best[tid];
    if (count_before(sm.best, kTopkThreads / 4, mine, tid) == k - 1) sm.threshold = mine;
  }
  __syncthreads();
  const float t = sm.threshold;
  if (t > -INFINITY && best >= t) append(v, mask_of(v, [t](float x) { return x >= t; }), sm);
  __syncthreads();
  int n = sm.n_list;
  if (t == -INFINITY || n > kTopkList) n = list_from_exact_threshold(v, k, best, sm, exists);
  // pad the list to a whole quad with entries that come before none
  if (tid < 3 && n + tid < (n + 3) / 4 * 4) { sm.list_v[n + tid] = -INFINITY; sm.list_i[n + tid] = 0x7fffffff; }
  __syncthreads();
#pragma unroll 1
  for (int a = tid; a < n; a += kTopkThreads) {
    const float av = sm.list_v[a];
    const int ai = sm.list_i[a];
    int place = 0;
#pragma unroll 2
    for (int b = 0; b < n; b += 4) {
      const f32x4 bv = *(const f32x4*)&sm.list_v[b];
      const u32x4 bi = *(const u32x4*)&sm.list_i[b];
#pragma unroll
      for (int e = 0; e < 4; ++e) place += (int)(bv[e] > av) | ((int)(bv[e] == av) & (int)((int)bi[e] < ai));
    }
    if (place < k) { sm.pick_v[place] = av; sm.pick_i[place] = ai; }
  }
  __syncthreads();
}

typedef float f32x4_unaligned __attribute__((ext_vector_type(4), aligned(4)));
// the workgroup's n candidates at src; -inf past the end
__device__ __forceinline__ void load_candidates(const float* __restrict__ src, int n, TopkValues& v) {
  if (n == kTopkChunk) {
#pragma unroll
    for (int s = 0; s < kTopkSlabs; ++s) {
      const f32x4 w = *(const f32x4_unaligned*)(src + position_of(4 * s));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[s][e] = w[e];
    }
  } else {
#pragma unroll
    for (int s = 0; s < kTopkSlabs; ++s) {
      if (s * 4 * kTopkThreads >= n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[s][e] = -INFINITY;
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = position_of(4 * s + e);
        const float x = src[min(j, n - 1)];
        v[s][e] = j < n ? x : -INFINITY;
      }
    }
  }
}

// Phase 1: workgroup (chunk, sequence) selects the W best of its chunk of candidates.  With one chunk per sequence the
// picks are final (written as parent / token / score); otherwise they go to the workspace for phase 2.
// 16 sequences, beam width 20, 32000 tokens: 41 MB of log-probabilities; both phases 363 us with one pick per round,
// 27 us in this form (16 + 11).
__global__ __launch_bounds__(kTopkThreads) void beam_topk_kernel(const float* __restrict__ beam_scores,
                                                                 const float* __restrict__ logp, int beams, int vocab,
                                                                 int n_chunks, float* __restrict__ ws_v,
                                                                 int* __restrict__ ws_i, int32_t* __restrict__ parent,
                                                                 int32_t* __restrict__ token, float* __restrict__ score) {
  __shared__ TopkSmem sm;
  __shared__ float beam[kTopkMaxBeams];
  const int b = blockIdx.y, chunk = blockIdx.x;
  const int n_cand = beams * vocab, c0 = chunk * kTopkChunk;   // n_cand: at most 2^26 (beam_topk_limits)
  const int n = min(kTopkChunk, n_cand - c0);
  TopkValues v;
  load_candidates(logp + (long long)b * n_cand + c0, n, v);
  if ((int)threadIdx.x < beams) beam[threadIdx.x] = beam_scores ? beam_scores[b * beams + threadIdx.x] : 0.f;
  __syncthreads();
  // candidate score = beam score + log-probability; a NaN never wins.  (Past the end, -inf plus anything is -inf or NaN.)
  const int w0 = c0 / vocab;
  if ((w0 + 1) * (long long)vocab >= c0 + n) {   // the whole chunk belongs to one beam
    const float add = beam[w0];
#pragma unroll
    for (int s = 0; s < kTopkSlabs; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) { const float x = v[s][e] + add; v[s][e] = x == x ? x : -INFINITY; }
  } else {
    // one division, then steps of 1 inside a quad and of 1020 to the next slab
    int w = (c0 + 4 * (int)threadIdx.x) / vocab, rem = c0 + 4 * (int)threadIdx.x - w * vocab;
#pragma unroll
    for (int s = 0; s < kTopkSlabs; ++s) {
      if (s * 4 * kTopkThreads >= n) continue;
      if (s > 0) {
        rem += 4 * kTopkThreads - 4;
        while (rem >= vocab) { rem -= vocab; ++w; }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = v[s][e] + beam[min(w, beams - 1)];
        v[s][e] = x == x ? x : -INFINITY;
        if (++rem == vocab) { rem = 0; ++w; }
      }
    }
  }
  select_topk(v, beams, sm, [n](int position) { return position < n; });
  if ((int)threadIdx.x < beams) {
    const int r = threadIdx.x, i = sm.pick_i[r] >= 0 ? c0 + sm.pick_i[r] : -1;
    if (n_chunks == 1) {
      parent[b * beams + r] = i >= 0 ? b * beams + i / vocab : -1;
      token[b * beams + r] = i >= 0 ? i % vocab : -1;
      score[b * beams + r] = sm.pick_v[r];
    } else {
      ws_v[((long long)b * n_chunks + chunk) * beams + r] = sm.pick_v[r];
      ws_i[((long long)b * n_chunks + chunk) * beams + r] = i;
    }
  }
}

// Phase 2: the W best of the chunks' picks of one sequence (the top W of a union lie among the top W of its parts).  The
// picks lie chunk after chunk, best first: among equal scores their positions ascend with the candidate index.
__global__ __launch_bounds__(kTopkThreads) void beam_topk_merge_kernel(const float* __restrict__ ws_v,
                                                                       const int* __restrict__ ws_i, int beams,
                                                                       int vocab, int n_chunks,
                                                                       int32_t* __restrict__ parent,
                                                                       int32_t* __restrict__ token,
                                                                       float* __restrict__ score) {
  __shared__ TopkSmem sm;
  const int b = blockIdx.x, n = n_chunks * beams;
  ws_v += (long long)b * n;
  ws_i += (long long)b * n;
  TopkValues v;
  load_candidates(ws_v, n, v);
  // (a chunk with fewer candidates than beams leaves places without an index)
  select_topk(v, beams, sm, [=](int position) { return position < n && ws_i[position] >= 0; });
  if ((int)threadIdx.x < beams) {
    const int r = threadIdx.x, at = sm.pick_i[r], i = at >= 0 ? ws_i[at] : -1;
    parent[b * beams + r] = i >= 0 ? b * beams + i / vocab : -1;
    token[b * beams + r] = i >= 0 ? i % vocab : -1;
    score[b * beams + r] = sm.pick_v[r];
  }
}

// gen_src_out[u][g] = g < step ? gen_src_in[parent[u]][g] (parent's own id when gen_src_in is NULL) : parent[u] at g == step;
// slots past `step` are set to u (a stream's future appends go to its own slots).
__global__ __launch_bounds__(256) void beam_reorder_kernel(const int32_t* __restrict__ parent,
                                                           const int32_t* __restrict__ src_in,
                                                           int32_t* __restrict__ src_out, int n_streams, int gen_cap,
                                                           int step) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)n_streams * gen_cap) return;
  const int u = (int)(t / gen_cap), g = (int)(t % gen_cap);
  const int par = max(min(parent[u], n_streams - 1), 0);
  int v = u;
  if (g < step) v = src_in ? src_in[(long long)par * gen_cap + g] : par;
  else if (g == step) v = par;
  src_out[t] = v;
}

static int topk_chunks(int beams, int vocab) { return (int)(((long long)beams * vocab + kTopkChunk - 1) / kTopkChunk); }

size_t beam_topk_workspace_bytes(int batch, int beams, int vocab) {
  const int n_chunks = topk_chunks(beams, vocab);
  return n_chunks <= 1 ? 0 : (size_t)batch * n_chunks * beams * 8;
}

int launch_beam_topk(const float* beam_scores, const float* logp, int batch, int beams, int vocab, int32_t* parent,
                     int32_t* token, float* score, void* workspace, hipStream_t stream) {
  const int n_chunks = topk_chunks(beams, vocab);
  float* ws_v = (float*)workspace;
  int* ws_i = (int*)(ws_v + (size_t)batch * n_chunks * beams);
  hipLaunchKernelGGL(beam_topk_kernel, dim3(n_chunks, batch), dim3(kTopkThreads), 0, stream, beam_scores, logp, beams,
                     vocab, n_chunks, ws_v, ws_i, parent, token, score);
  if (n_chunks > 1)
    hipLaunchKernelGGL(beam_topk_merge_kernel, dim3(batch), dim3(kTopkThreads), 0, stream, ws_v, ws_i, beams, vocab,
                       n_chunks, parent, token, score);
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

int launch_beam_reorder(const int32_t* parent, const int32_t* src_in, int32_t* src_out, int n_streams, int gen_cap, int step,
                        hipStream_t stream) {
  const long long n = (long long)n_streams * gen_cap;
  hipLaunchKernelGGL(beam_reorder_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, parent, src_in, src_out,
                     n_streams, gen_cap, step);
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

int beam_topk_limits(int beams, int vocab, const char** why) {
  if (beams > kTopkMaxBeams) { *why = "more than 64 beams"; return 0; }
  if ((long long)topk_chunks(beams, vocab) * beams > kTopkChunk) { *why = "beams * vocab too large for the two-phase selection"; return 0; }
  return 1;
}

}  // namespace earn
