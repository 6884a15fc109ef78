// Backward of the causal attention (paper Section 3.2, Training: the model is trained through the same attention, full
// length for layers l <= k and over register + target tokens for l > k; Eq. 3).  Given the forward's inputs as the
// attention saw them (rotated queries and keys), its output O, the log-sum-exp of every softmax row and dO:
//   D_i  = sum_e dO_ie O_ie                    P_ij = exp(s_ij - lse_i),  s_ij = scale q_i . k_j   (j <= i)
//   dV_j = sum_i P_ij dO_i                     dP_ij = dO_i . v_j          dS_ij = P_ij (dP_ij - D_i)
//   dQ_i = scale sum_j dS_ij k_j               dK_j = scale sum_i dS_ij q_i
// (sums over the query heads of a kv head's group for dK, dV).  No atomics: one kernel owns query rows (D, dQ), one owns
// key rows (dK, dV); each recomputes the probabilities it needs from lse.
//   bf16  bwd_dq_mfma_kernel, bwd_dkv_mfma_kernel: the five products on the matrix cores.
//   fp32  bwd_dsum_kernel, bwd_dq_kernel, bwd_dkv_kernel: vector ALU, four lanes share a row and hold d/4 of its elements
//         each (the precise form for the small fp32 configuration; in bf16, of rows with infinities or NaN).
#include "common.h"
#include "mfma_tiles.h"

namespace earn {

struct BwdParams {
  const void* q; const void* k; const void* v; const void* out; const float* lse; const void* d_out;
  const int32_t* cu; float* dsum;  // D: [tokens, Hq] (fp32 kernels) or [Hq, tokens] (bf16 kernels)
  void* dq; void* dk; void* dv;
  int batch, hq, hkv, total, max_seqlen;
  BackwardPlan plan;   // of this launch (bf16 kernels)
  float scale, scale_log2;
  HeadMap heads;
};

template <typename T> struct B8;
template <> struct B8<float> {
  static __device__ __forceinline__ void load(const float* p, float* x) {
    f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
    x[0] = a[0]; x[1] = a[1]; x[2] = a[2]; x[3] = a[3]; x[4] = b[0]; x[5] = b[1]; x[6] = b[2]; x[7] = b[3];
  }
  static __device__ __forceinline__ void store(float* p, const float* x) {
    *(f32x4*)p = f32x4{x[0], x[1], x[2], x[3]};
    *(f32x4*)(p + 4) = f32x4{x[4], x[5], x[6], x[7]};
  }
};
template <> struct B8<__bf16> {
  static __device__ __forceinline__ void load(const __bf16* p, float* x) {
    u32x4 w = *(const u32x4*)p;
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[2 * i] = bf16_lo(w[i]); x[2 * i + 1] = bf16_hi(w[i]); }
  }
  static __device__ __forceinline__ void store(__bf16* p, const float* x) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack_bf16(x[2 * i], x[2 * i + 1]);
    *(u32x4*)p = w;
  }
};
// A row shared by L lanes (4, or 8 where registers are short): lane `part` holds pieces [part*E, +E) and [D/2 + part*E, +E),
// E = D / (2 L)
template <typename T, int D, int L>
__device__ __forceinline__ void load_part(const T* row, int part, float* x) {
  constexpr int E = D / 2 / L;
  static_assert(E % 8 == 0);
#pragma unroll
  for (int e = 0; e < E; e += 8) { B8<T>::load(row + part * E + e, x + e); B8<T>::load(row + D / 2 + part * E + e, x + E + e); }
}
template <typename T, int D, int L>
__device__ __forceinline__ void store_part(T* row, int part, const float* x) {
  constexpr int E = D / 2 / L;
#pragma unroll
  for (int e = 0; e < E; e += 8) { B8<T>::store(row + part * E + e, x + e); B8<T>::store(row + D / 2 + part * E + e, x + E + e); }
}
template <int L>
__device__ __forceinline__ float row_sum(float x) {
#pragma unroll
  for (int o = 1; o < L; o <<= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

// D_i = dO_i . O_i for every (token, query head): a quad per row
template <int D>
__global__ __launch_bounds__(256) void bwd_dsum_kernel(const float* __restrict__ out, const float* __restrict__ d_out,
                                                       float* __restrict__ dsum, long long rows) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long row = t >> 2;
  const int qt = (int)(t & 3);
  float acc = 0.f;
  if (row < rows) {
    float o[D / 4], g[D / 4];
    load_part<float, D, 4>(out + row * D, qt, o);
    load_part<float, D, 4>(d_out + row * D, qt, g);
#pragma unroll
    for (int e = 0; e < D / 4; ++e) acc = __builtin_fmaf(o[e], g[e], acc);
  }
  acc = row_sum<4>(acc);
  if (row < rows && qt == 0) dsum[row] = acc;
}

// dQ of query row i by the L lanes that own it; the rows of a wave walk the keys 0 .. wave_last together.  dsum: the row's D.
// Pairs that are masked are passed over, not multiplied by zero: a later key's or value's infinity stays its own.
template <typename T, int D, int L>
__device__ __forceinline__ void bwd_dq_row(const BwdParams& p, int b0, int n, int c, int a, int i, int wave_last, float dsum, int part) {
  constexpr int N = D / L;
  const bool row_ok = i < n;
  const int ic = row_ok ? i : n - 1;
  const long long io = ((long long)(b0 + ic) * p.hq + a);
  float q[N], g[N], dq[N];
  load_part<T, D, L>((const T*)p.q + io * D, part, q);
  load_part<T, D, L>((const T*)p.d_out + io * D, part, g);
#pragma unroll
  for (int e = 0; e < N; ++e) { q[e] *= p.scale_log2; dq[e] = 0.f; }
  const float lse2 = p.lse[io] * 1.4426950408889634f;
  const T* kbase = (const T*)p.k + ((long long)b0 * p.hkv + c) * D;
  const T* vbase = (const T*)p.v + ((long long)b0 * p.hkv + c) * D;
  const long long rs = (long long)p.hkv * D;
  for (int j = 0; j <= wave_last; ++j) {
    float kx[N], vx[N];
    load_part<T, D, L>(kbase + j * rs, part, kx);
    load_part<T, D, L>(vbase + j * rs, part, vx);
    float sc = 0.f, dp = 0.f;
#pragma unroll
    for (int e = 0; e < N; ++e) { sc = __builtin_fmaf(q[e], kx[e], sc); dp = __builtin_fmaf(g[e], vx[e], dp); }
    sc = row_sum<L>(sc);
    dp = row_sum<L>(dp);
    if (j > ic) continue;   // causal: keys 0 .. i
    const float ds = __builtin_amdgcn_exp2f(sc - lse2) * (dp - dsum);
#pragma unroll
    for (int e = 0; e < N; ++e) dq[e] = __builtin_fmaf(ds, kx[e], dq[e]);
  }
  if (!row_ok) return;
#pragma unroll
  for (int e = 0; e < N; ++e) dq[e] *= p.scale;
  store_part<T, D, L>((T*)p.dq + io * D, part, dq);
}
// dK and dV of key row j by the L lanes that own it: query rows j .. n-1 of every query head of the group, which the rows of a
// wave walk together from wave_first on.  (Masked pairs: as above.)
template <typename T, int D, int L>
__device__ __forceinline__ void bwd_dkv_row(const BwdParams& p, int b0, int n, int c, int j, int wave_first, int part) {
  constexpr int N = D / L;
  const int gq = p.hq / p.hkv;
  const bool key_ok = j < n;
  const int jc = key_ok ? j : n - 1;
  const long long jo = ((long long)(b0 + jc) * p.hkv + c);
  float kx[N], vx[N], dk[N], dv[N];
  load_part<T, D, L>((const T*)p.k + jo * D, part, kx);
  load_part<T, D, L>((const T*)p.v + jo * D, part, vx);
#pragma unroll
  for (int e = 0; e < N; ++e) { kx[e] *= p.scale_log2; dk[e] = 0.f; dv[e] = 0.f; }
  for (int ai = 0; ai < gq; ++ai) {
    const int a = head_of_slot(p.heads, c * gq + ai);
    for (int i = wave_first; i < n; ++i) {
      const long long io = ((long long)(b0 + i) * p.hq + a);
      float q[N], g[N];
      load_part<T, D, L>((const T*)p.q + io * D, part, q);
      load_part<T, D, L>((const T*)p.d_out + io * D, part, g);
      float sc = 0.f, dp = 0.f;
#pragma unroll
      for (int e = 0; e < N; ++e) { sc = __builtin_fmaf(q[e], kx[e], sc); dp = __builtin_fmaf(g[e], vx[e], dp); }
      sc = row_sum<L>(sc);
      dp = row_sum<L>(dp);
      if (jc > i) continue;   // query i sees keys 0 .. i
      const float pr = __builtin_amdgcn_exp2f(sc - p.lse[io] * 1.4426950408889634f);
      const float ds = pr * (dp - p.dsum[sizeof(T) == 2 ? (long long)a * p.total + b0 + i : io]);
#pragma unroll
      for (int e = 0; e < N; ++e) { dv[e] = __builtin_fmaf(pr, g[e], dv[e]); dk[e] = __builtin_fmaf(ds, q[e], dk[e]); }
    }
  }
  if (!key_ok) return;
#pragma unroll
  for (int e = 0; e < N; ++e) dk[e] *= p.scale;
  store_part<T, D, L>((T*)p.dk + jo * D, part, dk);
  store_part<T, D, L>((T*)p.dv + jo * D, part, dv);
}

// dQ: 64 query rows per workgroup (grid: row block, query-head slot, sequence)
template <int D>
__global__ __launch_bounds__(256) void bwd_dq_kernel(BwdParams p) {
  const int slot = blockIdx.y, s = blockIdx.z;
  const int a = head_of_slot(p.heads, slot), c = slot / (p.hq / p.hkv);
  int b0, n;
  clamped_bounds(p.cu, s, p.total, p.max_seqlen, b0, n);
  const int row0 = blockIdx.x * 64;
  if (row0 >= n) return;
  const int i = row0 + (threadIdx.x >> 2);
  const int wave_last = min(n - 1, row0 + (int)(threadIdx.x / kWave) * 16 + 15);
  bwd_dq_row<float, D, 4>(p, b0, n, c, a, i, wave_last, p.dsum[(long long)(b0 + min(i, n - 1)) * p.hq + a], threadIdx.x & 3);
}

// dK, dV: 64 key rows per workgroup (grid: key block, kv head, sequence)
template <int D>
__global__ __launch_bounds__(256) void bwd_dkv_kernel(BwdParams p) {
  int b0, n;
  clamped_bounds(p.cu, blockIdx.z, p.total, p.max_seqlen, b0, n);
  const int key0 = blockIdx.x * 64;
  if (key0 >= n) return;
  bwd_dkv_row<float, D, 4>(p, b0, n, blockIdx.y, key0 + (threadIdx.x >> 2), key0 + (int)(threadIdx.x / kWave) * 16, threadIdx.x & 3);
}

// ------------------------------------------------------------------------------------------------------------------
// bf16 on the matrix cores (v_mfma_f32_32x32x16_bf16; lane = (r32 = lane % 32, hf = lane / 32))
//
// Both kernels take the forward's register-level scheme: a score tile whose accumulator columns are the rows the wave
// OWNS (queries for dQ, keys for dK / dV) gives a lane one owned row and 16 of the 32 rows it is paired with; the
// accumulator registers, converted to bf16, are the B operand of the product that contracts over the paired rows, whose
// A operand is the paired tile read transposed from LDS (ds_read_b64_tr_b16).  A wave keeps its 32 owned rows (q and dO, or
// k and v) as B operands in registers; the paired rows stream through LDS in tiles shared by the workgroup:
//   dQ:      S^T = K Q^T   dP^T = V dO^T    dQ^T += K^T dS^T                       (paired: keys)
//   dK, dV:  S = Q K^T     dP = dO V^T      dV^T += dO^T P,  dK^T += Q^T dS        (paired: queries of every head of the group)
// (dK, dV: -lse_i / scale and -D_i are the start values of the S and dP accumulators.)  P and dS enter the last products as
// THREE bf16 operands, value, remainder and its remainder, 24 significant bits: the products are those of fp32 probabilities,
// at 32 of the 64 (dK, dV) and 16 of the 40 (dQ) matrix instructions per 32 x 32 tile and 128 dimensions.  (Two operands, 16
// bits: 604 -> 518 and 123 -> 115 us at the sizes below, and every term of a sum wrong by up to 2^-18 of itself.)
// Bound by the instruction chain of a wave (matrix products, exponentials and splits of one tile: about 2 us, 3 us when two
// waves share a SIMD) times the tiles it walks.  Measured, forward included, against the vector-ALU form that these kernels
// replaced: 16 sequences of 272-1040 rows, 32 / 8 heads of 128: 18.36 -> 0.60 ms; 64 sequences of 68 rows: 1.01 -> 0.12 ms.
// The gradients leave through LDS, whole rows at a time (32 stores of 8 bytes a lane, 32 rows each, before: backward alone 485 -> 476
// and 84.0 -> 81.3 us at those sizes, 151 sequences of 140-189 rows 529 -> 498).
// ------------------------------------------------------------------------------------------------------------------
struct BwdBlock { int c, a, b0, n, row0; bool valid; };
// Workgroup -> (sequence, kv head, block of owned rows, query head of the group)
template <Owned ROWS_ARE>
__device__ __forceinline__ BwdBlock bwd_map_block(const BwdParams& p, int block_rows, int heads) {
  BwdBlock b;
  b.valid = false;
  const BackwardItem it = backward_item(p.plan, heads, blockIdx.z * gridDim.y + blockIdx.y, blockIdx.x);
  if (it.pair >= (long long)p.batch * p.hkv) return b;
  b.c = (int)it.pair % p.hkv;
  b.a = head_of_slot(p.heads, b.c * (p.hq / p.hkv) + it.head);
  clamped_bounds(p.cu, (int)it.pair / p.hkv, p.total, p.max_seqlen, b.b0, b.n);
  const int blk = backward_block(ROWS_ARE, p.plan, (b.n + block_rows - 1) / block_rows, it.step);
  b.row0 = blk * block_rows;
  b.valid = blk >= 0 && b.row0 < b.n;
  return b;
}
// Tiles of ROWS rows of one head of a packed [rows, heads, D] tensor into LDS (the swizzled layout of mfma_tiles.h).  The
// descriptor is rebuilt per tile from a 64-bit base, so a sequence of any length can be addressed; rows past the end of
// the sequence read as zeros.
template <int D, int WAVES, int ROWS>
struct BwdStager {
  static constexpr int UPR = D / 8, NI = ROWS * UPR / kWave / WAVES, RPI = kWave / UPR;
  static_assert(NI >= 1 && NI * WAVES * kWave == ROWS * UPR);
  int voff[NI], row_bytes, wave;
  __device__ __forceinline__ void init(int heads, int wave_, int lane) {
    row_bytes = heads * D * 2;
    wave = wave_;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int row = RPI * (wave + WAVES * i) + lane / UPR;
      voff[i] = row * row_bytes + ((lane % UPR) ^ swz<D>(row)) * 16;
    }
  }
  // rows [0, rows) of the tile starting at `base` exist (rows >= 1)
  __device__ __forceinline__ void issue(const __bf16* base, int rows, unsigned lds_tile) const {
    const u32x4 rsrc = raw_buffer(base, (min(rows, ROWS) - 1) * row_bytes + D * 2);
#pragma unroll
    for (int i = 0; i < NI; ++i) dma16_to_lds(rsrc, lds_tile + (unsigned)((wave + WAVES * i) * 1024), voff[i]);
  }
};
// 32 owned rows as B operands: lane (r32, hf) holds, per k-step ks, elements 16 ks + 8 hf + (0..7) of row r32
template <int D>
__device__ __forceinline__ void bwd_load_rows(const __bf16* row /* + 8 hf */, bf16x8 (&f)[D / 16]) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) f[ks] = *(const bf16x8*)(row + 16 * ks);
}
// acc += (32 tile rows at `tile`) x (owned rows: from registers, or from LDS rows `own`).  Fragments are requested AHEAD
// products early; slot(ks) is vector work of the caller's that runs while product ks does.
template <int D, int AHEAD, typename Slot>
__device__ __forceinline__ void bwd_product(const __bf16* tile, const FragOffsets<D>& fo, const bf16x8 (&f)[D / 16], f32x16& acc, Slot&& slot) {
  constexpr int KS = D / 16, N = AHEAD + 1;
  bf16x8 r[N];
#pragma unroll
  for (int ks = 0; ks < AHEAD && ks < KS; ++ks) r[ks] = *(const bf16x8*)(tile + fo.k(ks));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + AHEAD < KS) r[(ks + AHEAD) % N] = *(const bf16x8*)(tile + fo.k(ks + AHEAD));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[ks % N], f[ks], acc, 0, 0, 0);
    slot(ks);
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int D, int AHEAD>
__device__ __forceinline__ void bwd_product(const __bf16* tile, const __bf16* own, const FragOffsets<D>& fo, f32x16& acc) {
  constexpr int KS = D / 16, N = AHEAD + 1;
  bf16x8 r[N], f[N];
#pragma unroll
  for (int ks = 0; ks < AHEAD && ks < KS; ++ks) { r[ks] = *(const bf16x8*)(tile + fo.k(ks)); f[ks] = *(const bf16x8*)(own + fo.k(ks)); }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + AHEAD < KS) {
      r[(ks + AHEAD) % N] = *(const bf16x8*)(tile + fo.k(ks + AHEAD));
      f[(ks + AHEAD) % N] = *(const bf16x8*)(own + fo.k(ks + AHEAD));
    }
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[ks % N], f[ks % N], acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
__device__ __forceinline__ int word_reg(int w) { return 8 * (w >> 2) + 2 * (w & 3); }  // first accumulator register of word w
// o^T += (32 tile rows, transposed) x the fp32 tile of which src(w, a, b) gives registers word_reg(w), + 1, as three bf16
// operands: the values rounded, the remainders rounded, and what is left.  The second half of the tile is split while the
// first half's products run.  A fragment is requested two blocks ahead, the first two by the caller (bwd_request), ahead of
// the vector work that produces the tile.  slot(i), i < 2 D / 32: the caller's vector work that runs while block i's
// products do.
struct TransposedPair { bf16x8 f[2]; };
template <int D>
__device__ __forceinline__ TransposedPair bwd_request(const __bf16* tile, const FragOffsets<D>& fo) {
  return TransposedPair{read_v_fragment<D>(tile, fo, 0, 0), read_v_fragment<D>(tile, fo, 1, 0)};
}
template <int D, typename Src, typename Slot>
__device__ __forceinline__ void bwd_accumulate(const __bf16* tile, const FragOffsets<D>& fo, const TransposedPair& first,
                                               Src&& src, f32x16 (&o)[D / 32], Slot&& slot) {
  constexpr int DB = D / 32;
  u32x4 x[2][3];   // [half][term]
  auto split = [&](int w) {
    float a, b;
    src(w, a, b);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const unsigned h = pack_bf16(a, b);
      x[w >> 2][i][w & 3] = h;
      a -= bf16_lo(h);
      b -= bf16_hi(h);
    }
  };
#pragma unroll
  for (int w = 0; w < 4; ++w) split(w);
  bf16x8 r[3] = {first.f[0], first.f[1]};
#pragma unroll
  for (int i = 0; i < 2 * DB; ++i) {
    const int kk = i / DB, db = i % DB;
    if (i + 2 < 2 * DB) r[(i + 2) % 3] = read_v_fragment<D>(tile, fo, (i + 2) % DB, (i + 2) / DB);
#pragma unroll
    for (int t = 2; t >= 0; --t) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[i % 3], __builtin_bit_cast(bf16x8, x[kk][t]), o[db], 0, 0, 0);
    if (kk == 0) {
#pragma unroll
      for (int w = 4 + db * (4 / DB); w < 4 + (db + 1) * (4 / DB); ++w) split(w);
    }
    slot(i);
    __builtin_amdgcn_sched_barrier(0);
  }
}
// keeps the products that write these registers in front of what follows (the compiler otherwise starts the next
// products early, at the price of registers)
template <int N>
__device__ __forceinline__ void pin(f32x16 (&o)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(o[i]));
}
// Is there a NaN in the wave's sums (or infinities of both signs)?  A masked pair enters the products with weight 0, which an
// infinity or NaN on its other side turns into NaN, and an infinity times an operand of three terms may be inf - inf: such
// rows are worked out again on the vector ALU, pair by pair.
template <int N>
__device__ __forceinline__ bool any_nan(const f32x16 (&o)[N]) {
  float x = 0.f;
#pragma unroll
  for (int i = 0; i < 16 * N; ++i) x += o[i / 16][i % 16];
  return __any(x != x);
}
// D and dQ of 32 * WAVES query rows of one head.  (Late queries, which see the most keys, are dispatched first: with early ones
// first, 2 sequences of 2080 rows, 32 / 8 heads of 128, took 442 us for 423, 8 of 500-1000 with 12 / 2 heads 197 for 184.)
template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void bwd_dq_mfma_kernel(BwdParams p) {
  constexpr int ROWS = 16 * WAVES, BLOCK = 32 * WAVES;   // keys per tile, query rows per workgroup
  __shared__ __bf16 smk[2][ROWS * D];
  __shared__ __bf16 smv[2][ROWS * D];
  const BwdBlock blk = bwd_map_block<Owned::kQueries>(p, BLOCK, p.hq / p.hkv);
  if (!blk.valid) return;
  const int b0 = blk.b0, n = blk.n;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int r32 = lane & 31, hf = lane >> 5;
  const int qw = blk.row0 + wave * 32;               // first query row of this wave
  const bool active = qw < n;
  const int n_tiles = (min(blk.row0 + BLOCK, n) + ROWS - 1) / ROWS;
  const __bf16* kg = (const __bf16*)p.k + ((long long)b0 * p.hkv + blk.c) * D;
  const __bf16* vg = (const __bf16*)p.v + ((long long)b0 * p.hkv + blk.c) * D;
  const long long tile_stride = (long long)ROWS * p.hkv * D;
  BwdStager<D, WAVES, ROWS> st;
  st.init(p.hkv, wave, lane);
  const unsigned lds_k = (unsigned)(size_t)(lds_void_ptr)&smk[0][0], lds_v = (unsigned)(size_t)(lds_void_ptr)&smv[0][0];
  auto issue = [&](int t) {
    const unsigned at = (unsigned)((t & 1) * ROWS * D * 2);
    st.issue(kg + t * tile_stride, n - t * ROWS, lds_k + at);
    st.issue(vg + t * tile_stride, n - t * ROWS, lds_v + at);
  };
  issue(0);

  const int qi = min(qw + r32, n - 1);
  const long long io = (long long)(b0 + qi) * p.hq + blk.a;
  bf16x8 qf[D / 16], gf[D / 16];
  bwd_load_rows<D>((const __bf16*)p.q + io * D + 8 * hf, qf);
  bwd_load_rows<D>((const __bf16*)p.d_out + io * D + 8 * hf, gf);
  float dsum = 0.f;
  {
    const __bf16* orow = (const __bf16*)p.out + io * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      float o[8], g[8];
      B8<__bf16>::load(orow + 16 * ks, o);
      const u32x4 w = __builtin_bit_cast(u32x4, gf[ks]);
#pragma unroll
      for (int j = 0; j < 4; ++j) { g[2 * j] = bf16_lo(w[j]); g[2 * j + 1] = bf16_hi(w[j]); }
#pragma unroll
      for (int j = 0; j < 8; ++j) dsum = __builtin_fmaf(o[j], g[j], dsum);
    }
    dsum = half_sum(dsum);
    if (active && hf == 0 && qw + r32 < n) p.dsum[(long long)blk.a * p.total + b0 + qi] = dsum;
  }
  const float lse2 = p.lse[io] * 1.4426950408889634f;
  FragOffsets<D> fo;
  fo.init(lane);
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;

  for (int t = 0; t < n_tiles; ++t) {
    drain_loads_and_barrier();
    if (t + 1 < n_tiles) issue(t + 1);
#pragma unroll
    for (int h = 0; h < ROWS / 32; ++h) {
      const int key0 = t * ROWS + 32 * h;
      if (!active || key0 > qw + 31) continue;
      const __bf16* tk = smk[t & 1] + h * 32 * D;
      f32x16 s, ds;
#pragma unroll
      for (int i = 0; i < 16; ++i) { s[i] = 0.f; ds[i] = -dsum; }
      bwd_product<D, 3>(tk, fo, qf, s, [](int) {});
      // the exponentials run while the matrix core forms dP
      constexpr int EPS = 16 / (D / 16);   // per slot
      bwd_product<D, 3>(smv[t & 1] + h * 32 * D, fo, gf, ds, [&](int ks) {
#pragma unroll
        for (int i = EPS * ks; i < EPS * (ks + 1); ++i) s[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.scale_log2, -lse2));
      });
      const TransposedPair tp = bwd_request<D>(tk, fo);
      if (key0 + 31 > qw) {   // the diagonal: query r32 sees keys up to its own index
        const int bound = qw + r32 - key0 - 4 * hf;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + (i & 3) > bound) s[i] = 0.f;
      }
      auto d_score = [&](int w, float& a, float& b) {
        a = s[word_reg(w)] * ds[word_reg(w)];
        b = s[word_reg(w) + 1] * ds[word_reg(w) + 1];
      };
      bwd_accumulate<D>(tk, fo, tp, d_score, o, [](int) {});
    }
  }
  if (!active) return;
  constexpr int L = D / 16;   // lanes per row of the vector form
  if (any_nan(o)) {
#pragma unroll 1
    for (int r = 0; r < 32 && qw + r < n; r += kWave / L) {
      const int i = r + lane / L;
      bwd_dq_row<__bf16, D, L>(p, b0, n, blk.c, blk.a, qw + i, min(n, qw + r + kWave / L) - 1, __shfl(dsum, i, kWave), lane % L);
    }
    return;
  }
  // through the stage that the last tile, behind the last barrier, is not in: half of the waves in its K tile, half in its V tile
  __bf16* own = (wave < WAVES / 2 ? smk[n_tiles & 1] : smv[n_tiles & 1]) + (wave % (WAVES / 2)) * 32 * D;
  store_rows<D>((__bf16*)p.dq + ((long long)(b0 + qw) * p.hq + blk.a) * D, n - qw, (long long)p.hq * D, own, o, p.scale, lane);
}

// dK and dV of 32 * KW key rows of one kv head: walks the (head of the group, query tile) pairs from the block's own rows
// to the end of the sequence.  G groups of KW waves take every G-th pair each; their sums are added through LDS at the end.
// The 128 accumulators and 64 registers of owned rows of d = 128 leave too few for the rest of two waves per SIMD (24
// registers spilled inside the loop, whose reloads wait for the tiles in flight), so the owned keys stay in LDS there.
template <int D, int KW, int G>
__global__ __launch_bounds__(64 * KW * G, 2) void bwd_dkv_mfma_kernel(BwdParams p) {
  constexpr int ROWS = 32, BLOCK = 32 * KW, DB = D / 32;   // ROWS queries per tile, BLOCK key rows per workgroup
  constexpr bool KEYS_IN_LDS = D == 128;
  struct Stage { __bf16 q[ROWS * D], g[ROWS * D]; };
  __shared__ Stage sm[G][2];                               // q and dO tiles; at the end, the merge buffer
  __shared__ __bf16 smk[KEYS_IN_LDS ? BLOCK * D : 8];
  __shared__ float sml[G][2][2 * ROWS];                    // -lse / scale, then -D, of a tile's queries: start values of S, dP
  static_assert(G == 1 || sizeof(sm) >= sizeof(f32x16) * DB * 64 * KW);
  const BwdBlock blk = bwd_map_block<Owned::kKeys>(p, BLOCK, 1);
  if (!blk.valid) return;
  const int b0 = blk.b0, n = blk.n, gq = p.hq / p.hkv;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave % KW);
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / (kWave * KW)), tid = threadIdx.x % (kWave * KW);
  const int r32 = lane & 31, hf = lane >> 5;
  const int kw = blk.row0 + wave * 32;                     // first key row of this wave
  const bool active = kw < n;
  const int q_first = blk.row0, tiles = (n - q_first + ROWS - 1) / ROWS, steps = tiles * gq;
  BwdStager<D, KW, ROWS> st;
  st.init(p.hq, wave, lane);
  const unsigned lds_tiles = (unsigned)(size_t)(lds_void_ptr)&sm[grp][0];
  // This thread's word of the next tile's statistics: row stat_row of lse (tid < ROWS) or D (the next ROWS threads).  It is
  // requested with the tile and not touched before the tile is due: any arithmetic on it would wait for it here.
  const bool is_lse = tid < ROWS;
  const float inv_scale = 1.f / p.scale;
  const int stat_row = tid % ROWS;
  float stat = 0.f;
  // query tile at q0 of head i of the group, into stage `buf`
  auto issue = [&](int i, int q0, int buf) {
    const int a = head_of_slot(p.heads, blk.c * gq + i);
    const long long at = ((long long)(b0 + q0) * p.hq + a) * D;
    if (tid < 2 * ROWS) {
      const long long q = b0 + min(q0 + stat_row, n - 1);
      const float* src = is_lse ? p.lse + q * p.hq + a : p.dsum + (long long)a * p.total + q;
      stat = *src;
    }
    const unsigned to = lds_tiles + (unsigned)(buf * sizeof(Stage));
    st.issue((const __bf16*)p.q + at, n - q0, to);
    st.issue((const __bf16*)p.d_out + at, n - q0, to + (unsigned)(ROWS * D * 2));
  };
  const long long jo = (long long)(b0 + min(kw + r32, n - 1)) * p.hkv + blk.c;
  bf16x8 kf[D / 16], vf[D / 16];
  if constexpr (KEYS_IN_LDS) {
    BwdStager<D, KW * G, BLOCK> sk;
    sk.init(p.hkv, wave + KW * grp, lane);
    sk.issue((const __bf16*)p.k + ((long long)(b0 + blk.row0) * p.hkv + blk.c) * D, n - blk.row0,
             (unsigned)(size_t)(lds_void_ptr)&smk[0]);
  } else {
    bwd_load_rows<D>((const __bf16*)p.k + jo * D + 8 * hf, kf);
  }
  bwd_load_rows<D>((const __bf16*)p.v + jo * D + 8 * hf, vf);
  // this group's next (head, tile) pair
  int head = grp / tiles, tile = grp % tiles;
  if (head < gq) issue(head, q_first + tile * ROWS, 0);
  FragOffsets<D> fo;
  fo.init(lane);
  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dk[db][i] = 0.f; dv[db][i] = 0.f; }

  int buf = 0;
  for (int step = 0; step < steps; step += G) {            // the same count in every group: they share the barrier
    const bool have = head < gq;
    const int q0 = q_first + tile * ROWS;
    // rows past the end of the sequence: q = dO = 0 there, any finite value will do
    if (tid < 2 * ROWS) sml[grp][buf][tid] = q0 + stat_row < n ? stat * (is_lse ? -inv_scale : -1.f) : 0.f;
    drain_loads_and_barrier();
    tile += G;
    while (tile >= tiles) { tile -= tiles; ++head; }
    if (head < gq) issue(head, q_first + tile * ROWS, buf ^ 1);
    if (have && active && q0 + 31 >= kw) {
      const __bf16* tq = sm[grp][buf].q;
      const __bf16* tg = sm[grp][buf].g;
      const float* stats = sml[grp][buf] + 4 * hf;
      // The fragment addresses are worked out again for every product (one instruction each): kept, they would hold 16
      // registers.
      auto forget = [&] { asm volatile("" : "+v"(fo.k_base), "+v"(fo.v_base[0]), "+v"(fo.v_base[1])); };
      forget();
      f32x16 s, ds;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 l4 = *(const f32x4*)(stats + 8 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[4 * j + e] = l4[e];
      }
      if constexpr (KEYS_IN_LDS) bwd_product<D, 3>(tq, smk + wave * 32 * D, fo, s);
      else bwd_product<D, 3>(tq, fo, kf, s, [](int) {});
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 d4 = *(const f32x4*)(stats + ROWS + 8 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) ds[4 * j + e] = d4[e];
      }
      forget();
      // the exponentials run while the matrix core forms dP
      constexpr int EPS = 16 / (D / 16);   // per slot
      bwd_product<D, 3>(tg, fo, vf, ds, [&](int ks) {
#pragma unroll
        for (int i = EPS * ks; i < EPS * (ks + 1); ++i) s[i] = __builtin_amdgcn_exp2f(s[i] * p.scale_log2);
      });
      TransposedPair tp = bwd_request<D>(tg, fo);
      if (q0 < kw + 31) {     // the diagonal: key r32 is seen by queries from its own index on
        const int bound = kw + r32 - q0 - 4 * hf;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + (i & 3) < bound) s[i] = 0.f;
      }
      auto words_of = [](const f32x16& x) { return [&x](int w, float& a, float& b) { a = x[word_reg(w)]; b = x[word_reg(w) + 1]; }; };
      // dS = P (dP - D) is formed while the matrix core takes dV
      constexpr int RPS = 16 / (2 * DB);   // registers per slot
      bwd_accumulate<D>(tg, fo, tp, words_of(s), dv, [&](int i) {
#pragma unroll
        for (int r = RPS * i; r < RPS * (i + 1); ++r) ds[r] *= s[r];
      });
      forget();
      tp = bwd_request<D>(tq, fo);
      bwd_accumulate<D>(tq, fo, tp, words_of(ds), dk, [](int) {});
      pin(dv);
      pin(dk);
    }
    buf ^= 1;
  }
  // the groups' sums, added in group order (lane-wise: the layouts are identical)
  float* merge = (float*)&sm[0][0] + (wave * kWave + lane) * 4;
  auto add_groups = [&](f32x16 (&o)[DB]) {
#pragma unroll
    for (int g = 1; g < G; ++g) {
      __syncthreads();
      if (grp == g) {
#pragma unroll
        for (int i = 0; i < 4 * DB; ++i)
          *(f32x4*)(merge + i * KW * kWave * 4) = f32x4{o[i / 4][4 * (i % 4)], o[i / 4][4 * (i % 4) + 1], o[i / 4][4 * (i % 4) + 2], o[i / 4][4 * (i % 4) + 3]};
      }
      __syncthreads();
      if (grp == 0) {
#pragma unroll
        for (int i = 0; i < 4 * DB; ++i) {
          const f32x4 x = *(const f32x4*)(merge + i * KW * kWave * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[i / 4][4 * (i % 4) + e] += x[e];
        }
      }
    }
  };
  add_groups(dv);
  add_groups(dk);
  __syncthreads();            // the tiles' LDS is free
  if (grp > 0 || !active) return;
  constexpr int L = D / 16;   // lanes per row of the vector form
  if (any_nan(dk) || any_nan(dv)) {
    int at = lane;
    asm volatile("" : "+v"(at));   // nothing of this branch is worked out ahead of the loop above, which has no register to spare
#pragma unroll 1
    for (int r = 0; r < 32 && kw + r < n; r += kWave / L) bwd_dkv_row<__bf16, D, L>(p, b0, n, blk.c, kw + r + at / L, kw + r, at % L);
    return;
  }
  static_assert(sizeof(sm) >= KW * 32 * D * sizeof(__bf16));
  __bf16* own = (__bf16*)&sm[0][0] + wave * 32 * D;
  const long long at = ((long long)(b0 + kw) * p.hkv + blk.c) * D, row = (long long)p.hkv * D;
  store_rows<D>((__bf16*)p.dk + at, n - kw, row, own, dk, p.scale, lane);
  asm volatile("" ::: "memory");
  store_rows<D>((__bf16*)p.dv + at, n - kw, row, own, dv, 1.f, lane);
}

size_t attn_backward_workspace_bytes(int hq, int total_tokens) { return ((size_t)total_tokens * hq * sizeof(float) + 255) / 256 * 256; }

template <int D>
static void launch_bwd_f32(const BwdParams& p, int total_tokens, int max_seqlen, hipStream_t stream) {
  const long long rows = (long long)total_tokens * p.hq;
  hipLaunchKernelGGL((bwd_dsum_kernel<D>), dim3((unsigned)((rows * 4 + 255) / 256)), dim3(256), 0, stream, (const float*)p.out,
                     (const float*)p.d_out, p.dsum, rows);
  const unsigned blocks = (unsigned)((max_seqlen + 63) / 64);
  hipLaunchKernelGGL((bwd_dq_kernel<D>), dim3(blocks, p.hq, p.batch), dim3(256), 0, stream, p);
  hipLaunchKernelGGL((bwd_dkv_kernel<D>), dim3(blocks, p.hkv, p.batch), dim3(256), 0, stream, p);
}

// Workgroups of 128 owned rows as long as there are 512 of them (two per CU).  Below that, 64-row ones, and for dK / dV,
// where an early block of a long sequence walks all its tiles once per grouped head, four groups of waves per workgroup:
// the launch then takes as long as its longest chain of tiles (2 sequences of 2080 rows, 32 / 8 heads of 128, whole step:
// 442 against 608 us in the 128-row form; 12 / 2 heads, 8 sequences of 500-1000: 190 against 333; where 736 workgroups have
// work, 16 sequences of 272-1040, it is 578 against 519, and 64 sequences of 68 rows 142 against 118).
template <int D>
static void launch_bwd_mfma(BwdParams& p, hipStream_t stream) {
  const long long pairs = (long long)p.batch * p.hkv;
  auto fills = [&](int heads) { return (pairs + kXcds - 1) / kXcds * kXcds * ((p.max_seqlen + 127) / 128) * heads >= 512; };
  auto plan = [&](int rows, int heads) {
    p.plan = backward_plan(pairs, p.max_seqlen, rows, heads);
    const BackwardGrid g = backward_grid(p.plan, heads);
    return dim3(g.x, g.y, g.z);
  };
  const int gq = p.hq / p.hkv;
  const bool dq_wide = p.max_seqlen > 64 && fills(gq), dkv_wide = fills(1);
  dim3 grid = plan(dq_wide ? 128 : 64, gq);
  if (dq_wide) hipLaunchKernelGGL((bwd_dq_mfma_kernel<D, 4>), grid, dim3(256), 0, stream, p);
  else hipLaunchKernelGGL((bwd_dq_mfma_kernel<D, 2>), grid, dim3(128), 0, stream, p);
  grid = plan(dkv_wide ? 128 : 64, 1);
  if (dkv_wide) hipLaunchKernelGGL((bwd_dkv_mfma_kernel<D, 4, 1>), grid, dim3(256), 0, stream, p);
  else hipLaunchKernelGGL((bwd_dkv_mfma_kernel<D, 2, 4>), grid, dim3(512), 0, stream, p);
}

int launch_attn_backward(const earn_attn_desc* desc, const void* q, const void* k, const void* v, const void* out,
                         const float* lse, const void* d_out, const int32_t* cu_seqlens, int batch, int total_tokens,
                         int max_seqlen, void* dq, void* dk, void* dv, void* workspace, hipStream_t stream) {
  BwdParams p;
  p.q = q; p.k = k; p.v = v; p.out = out; p.lse = lse; p.d_out = d_out; p.cu = cu_seqlens; p.dsum = (float*)workspace;
  p.dq = dq; p.dk = dk; p.dv = dv; p.batch = batch; p.hq = desc->n_q_heads; p.hkv = desc->n_kv_heads;
  p.total = total_tokens; p.max_seqlen = max_seqlen;
  const int d = desc->head_dim;
  p.scale = desc->softmax_scale > 0.f ? desc->softmax_scale : 1.0f / sqrtf((float)d);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  if (make_head_map(desc, &p.heads, "earn_attn_backward") != EARN_OK) return EARN_ERR_UNSUPPORTED;
  if (batch > 65535 || p.hq > 65535) { set_error("earn_attn_backward: batch or head count beyond 65535"); return EARN_ERR_UNSUPPORTED; }
  if (desc->dtype == EARN_F32) {
    if (d == 64) launch_bwd_f32<64>(p, total_tokens, max_seqlen, stream); else launch_bwd_f32<128>(p, total_tokens, max_seqlen, stream);
  } else {
    if (d == 64) launch_bwd_mfma<64>(p, stream); else launch_bwd_mfma<128>(p, stream);
  }
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

}  // namespace earn
