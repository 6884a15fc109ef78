// Causal prefill attention over a packed ragged batch (paper Section 2.2, Eq. 3; used at full length for the first
// k layers and on the compacted register rows, with their original positions, for the remaining N-k layers —
// Section 3.2, Inference).
//
// Kernels:
//   rope_k_kernel        rotates K once per layer into the buffer the KV cache keeps (k_rot_out); every query block
//                        then reads rotated keys, so the sin/cos work is O(T), not O(T * blocks).
//   prefill_pipe_kernel  bf16 flash-style attention on the matrix cores (v_mfma_f32_32x32x16_bf16), software pipelined:
//                        long sequences.
//   prefill_mfma_kernel  the same arithmetic in a plain per-tile schedule with smaller workgroups: medium sequences.
//   prefill_short_kernel rotation and attention of a whole (sequence, kv head) in one workgroup: the register-only layers.
//   prefill_f32_kernel   fp32 attention on fp32 matrix products, for the fp32 configuration, where the 1e-4 tolerance rules
//                        out bf16 operands.
//
// MFMA kernel layout (all shapes in the 32x32x16 tile of the instruction, 64 lanes, lane = (r32 = lane%32, hf = lane/32)):
//   The kernels compute the TRANSPOSED score tile S^T = K Q^T (keys x queries).  Its accumulator layout gives every lane
//   ONE query column (r32) and 16 of the 32 keys of a block, so the softmax row statistics are a private loop plus one
//   exchange with lane^32, and the rescaling of the output accumulator is lane-private as well.
//   The accumulator registers of S^T, converted to bf16, are exactly the B operand (keys x queries, 8 keys per lane)
//   of the second product O^T = V^T P^T, so P never leaves registers.  The 8 key slots of a lane are keys
//   {4hf..4hf+3, 8+4hf..8+4hf+3} of a 16-key step; the A operand V^T uses the same key order, which is what two
//   transposing LDS reads (ds_read_b64_tr_b16: 4 consecutive keys of one d column) deliver from a V tile kept in its
//   natural [key][d] layout.
//   Each wave owns 32 query rows; the 64-key K/V tile in LDS is shared by the waves of a workgroup.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "mfma_tiles.h"

namespace earn {

struct PrefillParams {
  const void* q; const void* k_rot; const void* v; const int32_t* cu; const int32_t* positions;
  const f32x4* cs;  // [d/4][tokens] (cos, sin) of two rotary pairs of every token, written by rope_k_kernel (bf16 paths)
  void* out; float* lse;
  int batch, hq, hkv, max_seqlen;
  int total;   // rows of the packed tensors
  int n_qblk;  // workgroups of the longest sequence's (sequence, kv head) pair
  FastDiv by_pair, by_group, by_kv;  // workgroups per (sequence, kv head), query heads per kv head, kv heads
  FastDiv by_run;                    // prefill_short_kernel: workgroups per sequence
  // chosen-rows mode of the fp32 kernel (rows_per_seq > 0): q and out hold rows_per_seq rows per sequence in
  // compacted order, row m of sequence s being token row_pos[s * rows_per_seq + m] (ascending) of the sequence
  const int32_t* row_pos;
  int rows_per_seq;
  float scale_log2;
  // byte strides between the layers of a layer-batched launch (one grid dimension indexes the layer); zero otherwise.
  // The sequence bounds, the positions and the cos/sin table are shared by the layers.
  long long ls_q, ls_k_rot, ls_v, ls_out, ls_lse;
  RopeTable rope;
  HeadMap heads;
};

// Bounds of sequence s as the kernels use them: whatever cu_seqlens holds, rows [b0, b0 + n) lie inside the packed
// tensors and n within the length the launch was sized (and its 32-bit offsets checked) for.  A corrupt or not yet
// written cu_seqlens then gives wrong values, never an access outside the tensors.
__device__ __forceinline__ void pf_seq_bounds(const PrefillParams& p, int s, int& b0, int& n) {
  b0 = min(max(p.cu[s], 0), p.total);
  n = min(min(max(p.cu[s + 1] - b0, 0), p.total - b0), p.max_seqlen);
}

template <typename P>
__device__ __forceinline__ P* pf_layer_ptr(P* base, long long stride, int layer) {
  return (P*)((const char*)base + stride * layer);
}
// The per-layer pointers of one layer, as a view beside the parameter block (a modified copy of the block would live
// in scratch memory: it holds arrays indexed at run time).
struct PfLayer { const void* q; const void* k_rot; const void* v; void* out; float* lse; };
__device__ __forceinline__ PfLayer pf_layer_view(const PrefillParams& p, int layer) {
  PfLayer v;
  v.q = pf_layer_ptr(p.q, p.ls_q, layer);
  v.k_rot = pf_layer_ptr(p.k_rot, p.ls_k_rot, layer);
  v.v = pf_layer_ptr(p.v, p.ls_v, layer);
  v.out = pf_layer_ptr(p.out, p.ls_out, layer);
  v.lse = p.lse ? pf_layer_ptr(p.lse, p.ls_lse, layer) : nullptr;
  return v;
}

// ------------------------------------------------------------------------------------------------------------------
// K rotation
// ------------------------------------------------------------------------------------------------------------------
template <typename T> struct Vec8;
template <> struct Vec8<float> {
  static __device__ __forceinline__ void load(const float* p, float* x) {
    f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
    x[0] = a[0]; x[1] = a[1]; x[2] = a[2]; x[3] = a[3]; x[4] = b[0]; x[5] = b[1]; x[6] = b[2]; x[7] = b[3];
  }
  static __device__ __forceinline__ void store(float* p, const float* x) {
    f32x4 a = {x[0], x[1], x[2], x[3]}, b = {x[4], x[5], x[6], x[7]};
    *(f32x4*)p = a; *(f32x4*)(p + 4) = b;
  }
};
template <> struct Vec8<__bf16> {
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

// One thread per (token, group of 8 rotary pairs): the sin/cos of the group are computed once and applied to every kv
// head of the token.  bf16 rows use the hardware sin/cos (error ~1e-6, far below bf16 resolution).
// cs_out (optional): the (cos, sin) pairs themselves, two at a time, [d/4][token].  The attention kernels rotate their query
// rows with them: a workgroup per query head would otherwise recompute the same angles once per head, and on short sequences
// that prologue costs as much as the attention itself.  (Tokens innermost: the lanes of a wave hold consecutive query rows, and
// 16 loads of one row per lane kept a workgroup's memory pipeline busy for longer than the rows take to arrive.)
template <typename T, int D>
__global__ __launch_bounds__(256) void rope_k_kernel(const T* __restrict__ k, T* __restrict__ k_rot,
                                                     const int32_t* __restrict__ cu,
                                                     const int32_t* __restrict__ positions, int batch, int total,
                                                     int hkv, RopeTable rope, f32x4* __restrict__ cs_out,
                                                     int heads_per_thread, long long ls_k, long long ls_k_rot) {
  constexpr int G = D / 16;  // groups of 8 pairs per head
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)total * G) return;
  k = pf_layer_ptr(k, ls_k, blockIdx.z);           // grid layer z = layer of a layer-batched launch
  k_rot = pf_layer_ptr(k_rot, ls_k_rot, blockIdx.z);
  const int g = (int)(t % G);
  const int token = (int)(t / G);
  float sn[8], cs[8];
  if (rope.enabled) {
    int pos;
    if (positions) pos = positions[token];
    else pos = token - cu[find_seq(cu, batch, token)];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float turns = rope_turns((float)pos, rope.hi[g * 8 + i], rope.lo[g * 8 + i]);
      if (sizeof(T) == 2) sincos_turns_fast(turns, &sn[i], &cs[i]);
      else sincos_turns_precise(turns, &sn[i], &cs[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) { sn[i] = 0.f; cs[i] = 1.f; }
  }
  if (cs_out && blockIdx.y == 0 && blockIdx.z == 0) {
#pragma unroll
    for (int i = 0; i < 8; i += 2) cs_out[(long long)(g * 4 + i / 2) * total + token] = f32x4{cs[i], sn[i], cs[i + 1], sn[i + 1]};
  }
  const T* src = k + (long long)token * hkv * D + g * 8;
  T* dst = k_rot + (long long)token * hkv * D + g * 8;
  // grid row y takes kv heads [y * heads_per_thread, + heads_per_thread): all of them when there are tokens enough to
  // fill the GPU, a few when there are not (the loop over heads is a chain of memory round trips)
  const int h_begin = blockIdx.y * heads_per_thread, h_end = min(hkv, h_begin + heads_per_thread);
  for (int h = h_begin; h < h_end; ++h) {
    float lo[8], hi[8];
    Vec8<T>::load(src + h * D, lo);
    Vec8<T>::load(src + h * D + D / 2, hi);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float a = lo[i], b = hi[i];
      lo[i] = a * cs[i] - b * sn[i];
      hi[i] = b * cs[i] + a * sn[i];
    }
    Vec8<T>::store(dst + h * D, lo);
    Vec8<T>::store(dst + h * D + D / 2, hi);
  }
}

// ------------------------------------------------------------------------------------------------------------------
// fp32 attention on fp32 matrix products (v_mfma_f32_16x16x4_f32: exact products, fp32 sums).  A workgroup takes 16 QB query
// rows of one head; its waves take the 16-key blocks in turn and merge their states through LDS at the end, so that a short
// sequence is a few steps of many waves instead of a walk of few waves over all its keys.
//   S^T = K Q^T    lane (r16, quad) holds elements [quad E, + E) and [D/2 + quad E, + E) of key / query r16 (E = D/8): both
//                  sides of its rotary pairs, and any order of the contraction will do as long as both operands have it
//   O^T = V^T P^T  register s of S^T is key 4 quad + s of query r16: the B operand of a product over keys {4 quad + s}.  A lane
//                  reads dimensions 64 h + 4 r16 + (0..3) of its key, whole rows per wave instruction, and ends up with
//                  16 consecutive dimensions of its query.
// Nothing but the merge goes through LDS: every fragment is a 16-byte load of the wave's own.
//
// ROTATE: the keys are rotated here, every workgroup for itself, and the workgroup whose queries are the same rows writes the
// cache copy: one launch instead of two where the launch, not the arithmetic, is what a layer costs.
//
// Before, 4 lanes shared a query row on the vector ALU and 64 rows walked all their keys together.  us, with the rotation of the
// keys: 2 sequences of 132 rows, 4 heads of 64 55.1 -> 10.9 (17 round trips to memory in a row, now at most two); 16 of 512, 32 / 8
// heads of 128 6770 -> 1270, 27 TFLOP/s: one 4-wave workgroup a CU, whose loads nothing covers.  Relative error against 64 bits
// 1.8e-7 -> 1.5e-7 and 2.8e-7 -> 1.9e-7.
// ------------------------------------------------------------------------------------------------------------------
template <int D, int QB, int WAVES, bool ROTATE>
__global__ __launch_bounds__(64 * WAVES, D == 64 || QB == 1 ? 2 : 1) void prefill_f32_kernel(PrefillParams p, const float* k_in, long long ls_k_in, float* k_out) {
  constexpr int E = D / 8, H = D / 64, ROWS = 16 * QB, BLK = 16, OP = D + 4;   // OP: row pitch of the merge buffer
  __shared__ float smo[WAVES][ROWS][OP];
  __shared__ float sml[WAVES][ROWS][2];
  const int slot = blockIdx.y, s = blockIdx.z % p.batch;  // slot: the query heads in kv-head order
  const PfLayer lv = pf_layer_view(p, blockIdx.z / p.batch);
  const int a = head_of_slot(p.heads, slot), gq = p.hq / p.hkv, c = slot / gq;
  int b0, n;
  pf_seq_bounds(p, s, b0, n);
  const int r = p.rows_per_seq;           // 0: every row of the sequence
  const int n_rows = r > 0 ? r : n;
  const int row0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * ROWS;   // late rows, which see the most keys, first
  if (row0 >= n_rows || n <= 0) return;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int r16 = lane & 15, quad = lane >> 4;
  const long long rs = (long long)p.hkv * D;
  const float* kbase = (ROTATE ? pf_layer_ptr(k_in, ls_k_in, blockIdx.z / p.batch) : (const float*)lv.k_rot) + ((long long)b0 * p.hkv + c) * D + quad * E;
  const float* vbase = (const float*)lv.v + ((long long)b0 * p.hkv + c) * D + 4 * r16;
  // row of the sequence's row list -> its token: it sees keys 0 .. token (a row_pos outside the sequence is held inside it: wrong
  // values, no stray access)
  auto token_of = [&](int row) {
    const int m = min(row, n_rows - 1);
    return r > 0 ? min(max(p.row_pos[(long long)s * r + m], 0), n - 1) : m;
  };
  const int last_key = token_of(row0 + ROWS - 1), first_token = token_of(row0);   // rows ascend
  const int n_blocks = last_key / BLK + 1;

  float kx[2 * E];
  f32x4 vx[4][H];
  auto load_block = [&](int blk) {
    const float* krow = kbase + min(blk * BLK + r16, n - 1) * rs;
#pragma unroll
    for (int e = 0; e < E; e += 8) { Vec8<float>::load(krow + e, kx + e); Vec8<float>::load(krow + D / 2 + e, kx + E + e); }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vrow = vbase + min(blk * BLK + 4 * quad + i, n - 1) * rs;
#pragma unroll
      for (int h = 0; h < H; ++h) vx[i][h] = *(const f32x4*)(vrow + 64 * h);
    }
  };
  auto rotate = [&](float* x, int token) {
    const int pos = (p.positions && r == 0) ? p.positions[b0 + token] : token;
    int at = quad * E;
    // The table is read again for every block: kept, its 32 registers had 17 others spilled.  us: one sequence of 128 rows, 32 / 8 heads
    // 18.1 -> 17.1, two of 64 14.5 -> 14.4; one of 60, 12 / 2 heads, a block to a wave, 12.8 -> 13.1.
    if (D == 128) asm volatile("" : "+v"(at));
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float sn, cs;
      sincos_turns_precise(rope_turns((float)pos, p.rope.hi[at + e], p.rope.lo[at + e]), &sn, &cs);
      const float lo = x[e], hi = x[E + e];
      x[e] = lo * cs - hi * sn;
      x[E + e] = hi * cs + lo * sn;
    }
  };
  // queries: rotated and scaled; row of q / out / lse
  int ic[QB];
  long long io[QB];
  float qx[QB][2 * E];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const int row = min(row0 + 16 * b + r16, n_rows - 1);
    ic[b] = token_of(row);
    io[b] = r > 0 ? (long long)s * r + row : (long long)b0 + row;
    const float* q = (const float*)lv.q + (io[b] * p.hq + a) * D + quad * E;
#pragma unroll
    for (int e = 0; e < E; e += 8) { Vec8<float>::load(q + e, qx[b] + e); Vec8<float>::load(q + D / 2 + e, qx[b] + E + e); }
  }
  if (wave < n_blocks) load_block(wave);
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    if (p.rope.enabled) rotate(qx[b], ic[b]);
#pragma unroll
    for (int e = 0; e < 2 * E; ++e) qx[b][e] *= p.scale_log2;
  }

  f32x4 o[QB][H][4];
  float mrow[QB], lrow[QB];    // lrow: of this lane's keys
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    mrow[b] = -INFINITY; lrow[b] = 0.f;
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[b][h][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int blk = wave; blk < n_blocks; blk += WAVES) {
    const int j0 = blk * BLK;
    if (blk != wave) load_block(blk);
    if constexpr (ROTATE) {
      const int key = min(j0 + r16, n - 1);
      rotate(kx, key);
      // this block's own rows, by the first head of the group
      if (k_out && j0 >= row0 && j0 < row0 + ROWS && slot % gq == 0 && j0 + r16 < n) {
        float* dst = pf_layer_ptr(k_out, p.ls_k_rot, blockIdx.z / p.batch) + ((long long)(b0 + key) * p.hkv + c) * D + quad * E;
#pragma unroll
        for (int e = 0; e < E; e += 8) { Vec8<float>::store(dst + e, kx + e); Vec8<float>::store(dst + D / 2 + e, kx + E + e); }
      }
    }
    // Four partial sums: one would round a score D times in a row, twice the error (D = 128) of four lanes' sums added up.
    f32x4 sc[QB], part[QB][4];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[b][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 2 * E; ++e)
#pragma unroll
      for (int b = 0; b < QB; ++b) part[b][e % 4] = __builtin_amdgcn_mfma_f32_16x16x4f32(kx[e], qx[b][e], part[b][e % 4], 0, 0, 0);
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[b][i] = (part[b][0][i] + part[b][1][i]) + (part[b][2][i] + part[b][3][i]);
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (j0 + 4 * quad + i > ic[b]) sc[b][i] = -INFINITY;
        m = fmaxf(m, sc[b][i]);
      }
      m = fmaxf(m, __shfl_xor(m, 16, kWave));
      m = half_max(m);
      const float mnew = fmaxf(mrow[b], m), ref = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(mrow[b] - ref);
      mrow[b] = mnew;
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) { sc[b][i] = __builtin_amdgcn_exp2f(sc[b][i] - ref); sum += sc[b][i]; }
      lrow[b] = lrow[b] * alpha + sum;
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[b][h][j][i] *= alpha;
    }
    // A masked key has weight 0, and 0 times an infinite or NaN value is NaN: such a block is weighed pair by pair, without the
    // keys that a query does not see.
    bool pairwise = false;
    if (j0 + BLK - 1 > first_token) {   // some query does not see all of the block
      float probe = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j) probe = __builtin_fmaf(vx[i][h][j], 0.f, probe);
      pairwise = __any(probe != probe);
    }
    if (!pairwise) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < QB; ++b)
              o[b][h][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx[i][h][j], sc[b][i], o[b][h][j], 0, 0, 0);
    } else {
#pragma unroll
      for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll 1
          for (int g = 0; g < 4; ++g) {
            const int key = j0 + 4 * g + i;
            const float w = __shfl(sc[b][i], 16 * g + r16, kWave);
            if (key > ic[b]) continue;
            const float* vrow = vbase - 4 * r16 + key * rs + 16 * quad;
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
              for (int x = 0; x < 4; ++x) {
                const f32x4 v = *(const f32x4*)(vrow + 64 * h + 4 * x);
#pragma unroll
                for (int j = 0; j < 4; ++j) o[b][h][j][x] = __builtin_fmaf(w, v[j], o[b][h][j][x]);
              }
          }
    }
  }
  const int n_waves = min(WAVES, n_blocks);
  if (wave < n_waves) {
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      lrow[b] += __shfl_xor(lrow[b], 16, kWave);
      lrow[b] = half_sum(lrow[b]);
      if (quad == 0) { sml[wave][16 * b + r16][0] = mrow[b]; sml[wave][16 * b + r16][1] = lrow[b]; }
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int x = 0; x < 4; ++x)
          *(f32x4*)&smo[wave][16 * b + r16][64 * h + 16 * quad + 4 * x] = f32x4{o[b][h][0][x], o[b][h][1][x], o[b][h][2][x], o[b][h][3][x]};
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < ROWS * (D / 4); i += 64 * WAVES) {
    const int row = i / (D / 4), e = i % (D / 4) * 4;
    if (row0 + row >= n_rows) break;     // rows ascend with i
    float m = -INFINITY, l = 0.f;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < n_waves; ++w) m = fmaxf(m, sml[w][row][0]);
    for (int w = 0; w < n_waves; ++w) {
      // a wave none of whose keys the row sees: its sums hold zeros
      const float f = sml[w][row][0] == -INFINITY && m != -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sml[w][row][0] - m);
      l = __builtin_fmaf(f, sml[w][row][1], l);
      const f32x4 y = *(const f32x4*)&smo[w][row][e];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = __builtin_fmaf(f, y[j], x[j]);
    }
    const float inv = 1.f / l;
    const long long at = r > 0 ? (long long)s * r + row0 + row : (long long)b0 + row0 + row;
    *(f32x4*)((float*)lv.out + (at * p.hq + a) * D + e) = f32x4{x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv};
    if (lv.lse && e == 0) lv.lse[at * p.hq + a] = (m + __builtin_log2f(l)) * 0.6931471805599453f;
  }
}
template <int D>
static void launch_prefill_f32(const PrefillParams& p, const void* k_in, long long ls_k_in, void* k_out, bool rotate, int rows, int n_layers,
                               hipStream_t stream) {
  auto launch = [&](auto kernel, int block_rows, int waves) {
    hipLaunchKernelGGL(kernel, dim3((rows + block_rows - 1) / block_rows, p.hq, p.batch * n_layers), dim3(64 * waves), 0, stream, p,
                       (const float*)k_in, ls_k_in, (float*)k_out);
  };
  const bool few = f32_few_workgroups(rows, p.hq, D, (long long)p.batch * n_layers);
  if (rotate) launch(prefill_f32_kernel<D, 1, 8, true>, 16, 8);
  else if (few) launch(prefill_f32_kernel<D, 1, 8, false>, 16, 8);
  else launch(prefill_f32_kernel<D, 2, 4, false>, 32, 4);
}

// ------------------------------------------------------------------------------------------------------------------
// bf16 MFMA flash attention
// ------------------------------------------------------------------------------------------------------------------

// ---- workgroup -> (sequence, kv head) and its waves' (32 query rows, head of the group), XCD aware ----
// Workgroups are handed to the 8 XCDs round-robin by linear id, and every XCD has its own L2.  Id (x, k) = the k-th
// workgroup of XCD x.  Each XCD walks its own list of (sequence, kv head) pairs (pair % 8 == x) one pair at a time:
// all query rows of the pair (long, late ones first) and all query heads of the group, so the workgroups that
// are resident on an XCD at any moment stream the SAME K/V rows and find them in that XCD's L2.
// The pair's units of 32 rows of one head, heads innermost, go to the waves one after the other: the waves of a workgroup then
// see about the same keys, so none waits at the diagonal for the others, and a sequence's end leaves less than a unit per head
// idle (against 128 rows of one head to a workgroup: 256 sequences of 80-1040 rows, 12 / 2 heads of 128, 325 -> 292
// us; 16 of 272-1040, 32 / 8 heads, 121 -> 113.  The same in the backward's dQ: 483 -> 505 us for the latter, not kept).  With one head per kv head the units of a workgroup are consecutive rows.
struct PfBlock {
  int c, a;     // kv head; this wave's query head
  int b0, n;    // first packed row and length of the sequence
  int qw;       // this wave's first query row inside the sequence
  int end;      // query rows of the workgroup end here (as far as the sequence has them)
  bool valid;
};
template <int WAVES>
__device__ __forceinline__ PfBlock pf_map_block(const PrefillParams& p, int wave) {
  PfBlock b;
  b.valid = false;
  const unsigned gq = p.by_group.d, k_in_xcd = blockIdx.x / kXcds;
  const unsigned nth = p.by_pair.div(k_in_xcd), pair = nth * kXcds + blockIdx.x % kXcds;
  if (pair >= (unsigned)(p.batch * p.hkv)) return b;
  const unsigned s = p.by_kv.div(pair);
  b.c = (int)(pair - s * p.by_kv.d);
  pf_seq_bounds(p, s, b.b0, b.n);
  const unsigned first = (unsigned)(p.n_qblk - 1 - (int)(k_in_xcd - nth * p.by_pair.d)) * WAVES, unit = first + (unsigned)wave;
  const unsigned rows32 = p.by_group.div(unit);
  b.a = head_of_slot(p.heads, b.c * (int)gq + (int)(unit - rows32 * gq));
  b.qw = (int)rows32 * 32;
  b.end = min((int)p.by_group.div(first + WAVES - 1) * 32 + 32, b.n);
  b.valid = (int)p.by_group.div(first) * 32 < b.n;
  return b;
}

// ---- Q fragments: rotate at the original position (tabulated cos/sin), fold in scale*log2(e), keep as bf16 B operands ----
// lane (r32, hf) holds, for k-step ks, dims 16 ks + 8 hf + (0..7) of query r32
// unit(ks): those 8 elements as they came; c: the lane's (cos, sin) pairs (no table: no rotation)
template <int D>
__device__ __forceinline__ void pf_load_cs(const PrefillParams& p, long long token, int hf, f32x4 (&c)[D / 8]) {
  const f32x4* cs = p.cs + (long long)(4 * hf) * p.total + token;
#pragma unroll
  for (int i = 0; i < D / 8; ++i)    // pairs 16 (i / 4) + 8 hf + 2 (i % 4), + 1
    c[i] = p.cs ? cs[(long long)(8 * (i / 4) + i % 4) * p.total] : f32x4{1.f, 0.f, 1.f, 0.f};
}
template <int D, typename Unit>
__device__ __forceinline__ void pf_rotate_q(const PrefillParams& p, Unit&& unit, const f32x4 (&c)[D / 8], bf16x8 (&qf)[D / 16]) {
  constexpr int KSTEPS = D / 16;
#pragma unroll
  for (int ks = 0; ks < KSTEPS / 2; ++ks) {
    float lo[8], hi[8];
    Vec8<__bf16>::load(unit(ks), lo);
    Vec8<__bf16>::load(unit(ks + KSTEPS / 2), hi);
    u32x4 wl, wh;
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      const f32x4 t = c[4 * ks + j / 2];
      const float x0 = (lo[j] * t[0] - hi[j] * t[1]) * p.scale_log2, y0 = (hi[j] * t[0] + lo[j] * t[1]) * p.scale_log2;
      const float x1 = (lo[j + 1] * t[2] - hi[j + 1] * t[3]) * p.scale_log2, y1 = (hi[j + 1] * t[2] + lo[j + 1] * t[3]) * p.scale_log2;
      wl[j / 2] = pack_bf16(x0, x1);
      wh[j / 2] = pack_bf16(y0, y1);
    }
    qf[ks] = __builtin_bit_cast(bf16x8, wl);
    qf[ks + KSTEPS / 2] = __builtin_bit_cast(bf16x8, wh);
  }
}

// 32 query rows of a wave, whole rows at a time, into its own 32 x D region of LDS (swizzled like a K tile); rows past the
// sequence's end are not used.  DIRECT: every row starts on 16 bytes.
template <int D, bool DIRECT>
__device__ __forceinline__ void pf_stage_q(const __bf16* q /* first row */, int rows, int row_bytes, __bf16* own, int lane) {
  constexpr int UPR = D / 8, RPI = kWave / UPR;
  if constexpr (!DIRECT) {   // loads into LDS are for whole 16-byte units: rows that start elsewhere pass through registers
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
      const int row = RPI * i + lane / UPR;
      const u32x4 x = *(const u32x4*)((const char*)q + (long long)min(row, min(rows, 32) - 1) * row_bytes + ((lane % UPR) ^ swz<D>(row)) * 16);
      *(u32x4*)(own + i * 512 + lane * 8) = x;
    }
    return;
  }
  const unsigned lds = (unsigned)(size_t)(lds_void_ptr)own;
  const u32x4 rsrc = raw_buffer(q, (min(rows, 32) - 1) * row_bytes + D * 2);
#pragma unroll
  for (int i = 0; i < 32 / RPI; ++i) {
    const int row = RPI * i + lane / UPR;
    dma16_to_lds(rsrc, lds + (unsigned)(i * 1024), row * row_bytes + ((lane % UPR) ^ swz<D>(row)) * 16);
  }
}
// S^T (+)= K Q^T for the K tile at smk: two 32-key blocks, K fragments requested AHEAD k-steps before the MFMAs that use
// them.  ZERO: start from 0, else from `init` in every register (the steady state starts at -m, which takes the
// subtraction of the reference maximum off the vector ALU).
template <int D, bool ZERO, int AHEAD = ZERO ? 1 : 2>  // the exact paths are short of registers, not of time
__device__ __forceinline__ void score_tile(const __bf16* smk, const FragOffsets<D>& fo, const bf16x8 (&qf)[D / 16],
                                           const f32x16& init, f32x16 (&sc)[2]) {
  constexpr int KSTEPS = D / 16;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 kf[2][KSTEPS];
#pragma unroll
  for (int ks = 0; ks < AHEAD; ++ks)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) kf[kb][ks] = *(const bf16x8*)(smk + fo.k(ks) + kb * 32 * D);
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    if (ks + AHEAD < KSTEPS) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) kf[kb][ks + AHEAD] = *(const bf16x8*)(smk + fo.k(ks + AHEAD) + kb * 32 * D);
    }
    __builtin_amdgcn_sched_barrier(0);  // the fragment requests stay ahead of the MFMAs that hide their latency
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][ks], qf[ks], ks == 0 ? (ZERO ? zero : init) : sc[kb], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
// causal mask of the wave's diagonal tile, in place: lane (r32, hf) holds keys 32 kb + 8 (i/4) + 4 hf + i%4 of query
// q_in_tile + r32 (keys beyond the sequence end are beyond every valid query too)
__device__ __forceinline__ void mask_diagonal(f32x16 (&sc)[2], int q_in_tile, int r32, int hf) {
  const int bound = q_in_tile + r32 - 4 * hf;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (32 * kb + 8 * (i >> 2) + (i & 3) > bound) sc[kb][i] = -INFINITY;
}
// Softmax unit u (0..15) of a score tile: two exponentials (the scores already carry -m), the bf16 word that holds
// them, and the word's contribution to the lane's row sum.  Word (kk, j) of the B operand P^T packs accumulator
// registers 8 (kk & 1) + 2 j, + 1 of key block kk >> 1; u = 4 kk + j.
__device__ __forceinline__ void softmax_unit(const f32x16 (&sc)[2], int u, u32x4 (&w)[4], float& s0, float& s1) {
  const int kk = u >> 2, j = u & 3, r = 8 * (kk & 1) + 2 * j;
  w[kk][j] = pack_bf16(__builtin_amdgcn_exp2f(sc[kk >> 1][r]), __builtin_amdgcn_exp2f(sc[kk >> 1][r + 1]));
  add_pair(j & 1 ? s1 : s0, w[kk][j]);
}
// normalise and store one query row's share: lane holds d = 32 db + 8 j + 4 hf + (0..3)
template <int D>
__device__ __forceinline__ void pf_store_row(__bf16* orow /* row + 4 hf */, const f32x16 (&o)[D / 32], float inv) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x2 w;
      w[0] = pack_bf16(o[db][4 * j] * inv, o[db][4 * j + 1] * inv);
      w[1] = pack_bf16(o[db][4 * j + 2] * inv, o[db][4 * j + 3] * inv);
      *(u32x2*)(orow + 32 * db + 8 * j) = w;
    }
}

// ------------------------------------------------------------------------------------------------------------------
// Plain schedule: per tile  barrier -> S^T -> exponentials -> O^T.  One 32-query column block per wave.
//   WAVES = 4: 128 query rows per workgroup, two workgroups per CU: less idle time on the causal diagonal of medium
//              sequences than 256-row workgroups, at the price of staging every K/V tile twice as often.  The two are at
//              1.4 PFLOP/s while both are inside their tiles; what counts is the rest of a workgroup's life.  Queries and
//              outputs therefore pass through the stage that is free at the time, whole rows at a time, the rotary table is
//              read along the tokens, and tile 0 rescales nothing (one row per lane and load: 32.3 us of life for 12.6
//              tiles, 5.1 of them waiting for rows, 4.3 in tile 0 and 2.3 storing; now 26.5, 3.3, 3.1, 1.8.  64 sequences
//              of 288-2080 rows, 32 heads of 128: 1.49 -> 1.37 ms; 256 of 80-1040, 12 / 2 heads: 404 -> 332 us).
//              The pipelined schedule below in 128-row workgroups, two per CU, is slower here: 1.49 -> 1.72 ms.
//   WAVES = 2, STAGES = 1: sequences of one K/V tile with a kv head per query head: there is nothing to double buffer, and
//              the small footprint lets 4 workgroups share a CU, which is what hides the load -> rotate -> multiply
//              latency chain of these tiny problems.
// ------------------------------------------------------------------------------------------------------------------
//
// Life-cycle timers, compiled in only with -DEARN_PF_TIMELINE (paper_2507_00715_amd/timeline.py builds that variant
// into a library of its own and prints where a workgroup's life goes).  Thread 0 of every workgroup stamps the 100 MHz
// wall clock into 8 words of a caller-provided buffer: 0 entry, 1 block known, 2 queries, cos/sin rows and first K/V
// tile arrived (this stamp waits for them, which the normal build does only at the first barrier), 3 first tile done,
// 4 all tiles done, 5 output stores issued; 6 the CU, 7 the block's tile count (0: block beyond its sequence).  In the
// normal build the macros are empty.
#ifdef EARN_PF_TIMELINE
__device__ long long* g_pf_timeline;
__device__ int g_pf_timeline_slots;
#define PF_TIMELINE(code) code
#define PF_STAMP(i)                                                                                    \
  do {                                                                                                 \
    const long long pf_wg = (long long)blockIdx.y * gridDim.x + blockIdx.x;                            \
    if (threadIdx.x == 0 && g_pf_timeline && pf_wg < g_pf_timeline_slots) g_pf_timeline[pf_wg * 8 + (i)] = wall_clock64(); \
  } while (0)
#else
#define PF_TIMELINE(code)
#define PF_STAMP(i)
#endif
// DIRECT_Q (two stages): the queries start on 16 bytes.  Those that do not have a form of their own, so that the others stay without
// its instructions (the choice inside the kernel: 0.4 % and less at the first of those sizes, no more than two runs differ by).
template <int D, int WAVES, int STAGES, bool DIRECT_Q = true>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 1 : 2) void prefill_mfma_kernel(PrefillParams p) {
  constexpr int DB = D / 32;             // 32-row blocks of O^T
  __shared__ __bf16 smk[STAGES][kTileKeys * D];  // tile t+1 arrives while tile t is read
  __shared__ __bf16 smv[STAGES][kTileKeys * D];
  PF_STAMP(0);

  // the wave index is the same in all 64 lanes: say so, and everything derived from it (the wave's query window, its
  // diagonal tile, the tile loop) lives in scalar registers and branches without touching the execution mask
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const PfBlock blk = pf_map_block<WAVES>(p, wave);
  PF_TIMELINE({
    const long long pf_wg = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    if (threadIdx.x == 0 && g_pf_timeline && pf_wg < g_pf_timeline_slots) {
      g_pf_timeline[pf_wg * 8 + 6] = __smid();
      g_pf_timeline[pf_wg * 8 + 7] = blk.valid ? (blk.end + kTileKeys - 1) / kTileKeys : 0;
    }
  })
  if (!blk.valid) return;
  PF_STAMP(1);
  const PfLayer lv = pf_layer_view(p, blockIdx.y);
  const int b0 = blk.b0, n = blk.n;
  const int r32 = lane & 31, hf = lane >> 5;
  const int qw = blk.qw;                         // first query row of this wave
  const bool wave_active = qw < n;
  const int t_diag = qw / kTileKeys;             // last (diagonal) tile of this wave
  const int q_in_tile = qw - t_diag * kTileKeys; // offset of the wave's first query inside that tile
  const int n_tiles = (blk.end + kTileKeys - 1) / kTileKeys;

  TileStager<D, WAVES> stager;
  stager.init((const __bf16*)lv.k_rot + ((long long)b0 * p.hkv + blk.c) * D, (const __bf16*)lv.v + ((long long)b0 * p.hkv + blk.c) * D,
              n, p.hkv, wave, lane);
  const unsigned lds_k = (unsigned)(size_t)(lds_void_ptr)&smk[0][0], lds_v = (unsigned)(size_t)(lds_void_ptr)&smv[0][0];
  auto issue_tile = [&](int t) {
    const unsigned at = (unsigned)((t % STAGES) * kTileKeys * D * 2);
    stager.issue(stager.k_rsrc, lds_k + at, t);
    stager.issue(stager.v_rsrc, lds_v + at, t);
  };
  // Barrier t: every wave has waited for its own part of tile t, so behind the barrier tile t is complete and visible;
  // the wave then starts its part of tile t+1 into the other buffer, which every wave has finished reading (tile t-1).
  auto sync_and_stage = [&](int t) {
    drain_loads_and_barrier();
    if constexpr (STAGES > 1) {
      if (t + 1 < n_tiles) issue_tile(t + 1);
    }
  };
  FragOffsets<D> fo;
  fo.init(lane);
  // The wave's own 32 x D region inside stage x (two stages only): waves 0, 1 in its K tile, 2, 3 in its V tile.
  auto own_region = [&](int x) { return (wave & 2 ? smv[x] : smk[x]) + (wave & 1) * 32 * D; };
  bf16x8 qf[D / 16];
  const int q_c = min(qw + r32, n - 1);
  f32x4 cs[D / 8];
  if constexpr (STAGES == 2) {
    // through the second stage, which nothing uses before the first barrier
    __bf16* own = own_region(1);
    if (wave_active) pf_stage_q<D, DIRECT_Q>((const __bf16*)lv.q + ((long long)(b0 + qw) * p.hq + blk.a) * D, n - qw, p.hq * D * 2, own, lane);
    issue_tile(0);
    pf_load_cs<D>(p, b0 + q_c, hf, cs);
    asm volatile("" ::: "memory");
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    pf_rotate_q<D>(p, [&](int ks) { return own + fo.k(ks); }, cs, qf);
  } else {
    pf_load_cs<D>(p, b0 + q_c, hf, cs);
    issue_tile(0);  // in flight while the queries are loaded and rotated
    const __bf16* qrow = (const __bf16*)lv.q + ((long long)(b0 + q_c) * p.hq + blk.a) * D + 8 * hf;
    pf_rotate_q<D>(p, [&](int ks) { return qrow + 16 * ks; }, cs, qf);
  }
  PF_TIMELINE(__builtin_amdgcn_s_waitcnt(0x0F70);)  // vmcnt(0)
  PF_STAMP(2);

  f32x16 o[DB], neg_m;  // neg_m: -m in every register, the start value of the steady-state score accumulators
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_m[i] = 0.f;
  float mrow = -INFINITY, lrow = 0.f;

  // exponentials of a whole score tile (already shifted by -m), packed, with the lane's row sum
  auto softmax_tile = [&](const f32x16 (&sc)[2], u32x4 (&w)[4], float& lsum) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) softmax_unit(sc, u, w, s0, s1);
    lsum = add_chains(s0, s1);
  };
  // O^T += V^T P^T; the V^T fragments are requested up front so that their latency hides behind whatever the caller
  // does between fetch and use
  auto fetch_v = [&](const __bf16* smv_t, bf16x8 (&vf)[4][DB]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int db = 0; db < DB; ++db) vf[kk][db] = read_v_fragment<D>(smv_t, fo, db, kk);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto accumulate = [&](const u32x4 (&w)[4], float lsum, const bf16x8 (&vf)[4][DB]) {
    lrow += lsum;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk][db], __builtin_bit_cast(bf16x8, w[kk]), o[db], 0, 0, 0);
  };
  // The exact path: raw scores, exact row maxima, rescale of everything accumulated so far.
  // Tile 0 has nothing to rescale yet; any other one fell out of the steady-state loop, which has passed its barrier already.
  auto exact_tile = [&](int t, auto first_c) {
    constexpr bool FIRST = decltype(first_c)::value;
    if (FIRST) sync_and_stage(t);
    f32x16 sc[2];
    bf16x8 vf[4][DB];
    u32x4 w[4];
    float lsum;
    score_tile<D, true, FIRST ? 3 : 1>(smk[t % STAGES], fo, qf, neg_m, sc);
    if (t == t_diag) mask_diagonal(sc, q_in_tile, r32, hf);
    float m = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, sc[kb][i]);
    const float mnew = fmaxf(mrow, half_max(m));  // finite: tile 0 holds key 0, visible to every query
    if (!FIRST) {
      const float alpha = __builtin_amdgcn_exp2f(mrow - mnew);
      lrow *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    mrow = mnew;
#pragma unroll
    for (int i = 0; i < 16; ++i) neg_m[i] = -mnew;
    fetch_v(smv[t % STAGES], vf);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[kb][i] -= mnew;
    softmax_tile(sc, w, lsum);
    accumulate(w, lsum, vf);
  };

  // Every wave passes exactly one barrier per tile, whichever path it takes.  The steady-state loop takes the
  // exponentials against the reference maxima it already has and never touches the output accumulators with the
  // vector ALU.  It does not even compute row maxima: a reference is stale exactly when some exponential is large, so
  // the (already needed) partial row sums are compared with kSumLimit instead.  A wave that fails leaves the loop,
  // recomputes the tile's scores, takes the exact maxima, rescales, finishes the tile and re-enters.  Tile 0 (no reference
  // yet) always takes the exact path; the wave's diagonal tile is the only one that needs the causal mask.
  int t = 0;
  if (wave_active) {
    exact_tile(0, std::true_type{});
    t = 1;
    PF_STAMP(3);
  }
  while (t < n_tiles) {
    bool exact = false;
    for (; t < n_tiles; ++t) {
      const bool work = wave_active && t <= t_diag;  // else rows past the sequence end or a tile past the diagonal: only stage
      sync_and_stage(t);
      if (work) {
        f32x16 sc[2];
        bf16x8 vf[4][DB];
        u32x4 w[4];
        float lsum;
        score_tile<D, false>(smk[t % STAGES], fo, qf, neg_m, sc);
        if (t == t_diag) mask_diagonal(sc, q_in_tile, r32, hf);  // masked scores give weight 0 on this path as well
        fetch_v(smv[t % STAGES], vf);
        softmax_tile(sc, w, lsum);
        if (__any(!(lsum <= kSumLimit))) { exact = true; break; }
        accumulate(w, lsum, vf);
      }
    }
    if (!exact) break;
    exact_tile(t, std::false_type{});
    ++t;
  }
  PF_STAMP(4);

  if (!wave_active) return;
  const int qi = qw + r32;
  const float ltot = half_sum(lrow), inv = 1.f / ltot;
  __bf16* out = (__bf16*)lv.out + ((long long)(b0 + qw) * p.hq + blk.a) * D;
  if (lv.lse && hf == 0 && qi < n) lv.lse[(long long)(b0 + qi) * p.hq + blk.a] = (mrow + __builtin_log2f(ltot)) * 0.6931471805599453f;
  if constexpr (STAGES == 2) {
    // through the stage that the last tile, behind the last barrier, is not in
    store_rows<D>(out, n - qw, (long long)p.hq * D, own_region(n_tiles & 1), o, inv, lane);
  } else if (qi < n) {
    pf_store_row<D>(out + (long long)r32 * p.hq * D + 4 * hf, o, inv);
  }
  PF_STAMP(5);
}

// ------------------------------------------------------------------------------------------------------------------
// Short sequences (up to NR rows): the register-only layers and short prompts.  One workgroup takes a whole (sequence, kv
// head): it rotates the keys once, keeps them in LDS (and writes the cache copy), and its waves then take the gq * n query
// rows of the group, packed head after head, 16 at a time, on v_mfma_f32_16x16x32_bf16:
//   S^T = K Q^T   (16 keys x 16 rows per product; K rows padded to spread the fragment reads over the banks)
//   O^T = V^T P^T (V in swizzled rows; the accumulators of two S^T tiles are the B operand, keys in the order 4 quad + i,
//                  16 + 4 quad + i, which is what two transposing reads deliver)
// All scores of a row fit the registers, so the softmax is exact and taken once.  What bounds these layers is the number of
// dependent steps, not arithmetic: a rotation pass of its own, one workgroup per query head and 32-row column blocks that a
// 16-row sequence half fills cost 24.2 + 5.3 us where this kernel takes 12 (256 sequences of 16 rows, 12 / 2
// heads of 128; one launch per layer 29.8 -> 13.4 us, 24 layers in one launch 18.9 -> 8.2 us each).
// ------------------------------------------------------------------------------------------------------------------
// LDS of a workgroup, and workgroups that a CU is given: as many as fit, by LDS and 16 waves (up to 128 registers); two at most
// where each of a pair's workgroups would rotate the keys again (256 sequences of 16 rows, 12 / 2 heads, in four a CU: whole
// path of 28 layers 1586 -> 1696 us)
constexpr int short_lds(int d, int nr, bool rope) { return nr * (d + 8) * 2 + nr * d * 2 + (rope ? nr * (d / 2 + 2) * 8 : 0); }
constexpr int short_per_cu(int d, int nr, int waves, bool rope) {
  const int by_lds = 160 * 1024 / short_lds(d, nr, rope), by_waves = 16 / waves;
  const int fit = by_lds < by_waves ? by_lds : by_waves;
  return rope && fit > 2 ? 2 : fit;
}
template <int D, int NR, int WAVES, bool ROPE>
__global__ __launch_bounds__(64 * WAVES, NR == 128 && (D == 64 || !ROPE) ? 4 : 1) void prefill_short_kernel(PrefillParams p, const void* k_in, long long ls_k_in, int store_k, int parts) {
  constexpr int KS = D / 32, DB = D / 16, UPR = D / 8, NB = NR / 32, THREADS = 64 * WAVES;
  constexpr int KI = NR * (D / 8) / THREADS, VI = NR * UPR / THREADS;   // K items (4 rotary pairs), V units per thread
  constexpr int KP = D + 8, CP = D / 2 + 2;                             // row pitches of the K tile and of the rotary table
  static_assert(KI >= 1 && KI * THREADS == NR * (D / 8) && VI >= 1 && THREADS % (D / 2) == 0);
  __shared__ __align__(16) __bf16 smk[NR * KP];
  __shared__ __align__(16) __bf16 smv[NR * D];
  __shared__ __align__(16) f32x2 smc[ROPE ? NR * CP : 1];
  // An XCD takes a run of consecutive workgroups of consecutive sequences, the kv heads of a sequence, whose rows are interleaved,
  // next to each other.  (Against runs of whole sequences, rounded up: 9 sequences of 128 rows, 32 / 8 heads of 128, 20.7 -> 14.7
  // us, 25 of 128 30.0 -> 23.3, 33 of 64 21.1 -> 20.5.)
  const RunItem run = run_item(blockIdx.x, p.batch, p.by_run, true);
  if (!run.valid) return;
  const int part = (int)p.by_kv.div((unsigned)run.sub), s = run.item, c = run.sub - part * p.hkv;
  int b0, n;
  pf_seq_bounds(p, s, b0, n);
  // this wave's first 16 query rows, and the rows to its next ones
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), m_first = 16 * (part * WAVES + wave), m_step = 16 * WAVES * parts;
  if (n <= 0 || (part > 0 && 16 * part * WAVES >= (int)p.by_group.d * n)) return;
  const PfLayer lv = pf_layer_view(p, blockIdx.y);
  const int gq = (int)p.by_group.d, rows = gq * n;
  const int lane = threadIdx.x % kWave, r16 = lane & 15, quad = lane >> 4;
  const __bf16* kg = (const __bf16*)pf_layer_ptr(k_in, ls_k_in, blockIdx.y) + ((long long)b0 * p.hkv + c) * D;
  const __bf16* vg = (const __bf16*)lv.v + ((long long)b0 * p.hkv + c) * D;
  const long long row_stride = (long long)p.hkv * D;
  // Everything that comes from memory is requested before anything is used, the positions ahead of the rest: the rotary table is
  // worked out while the rows are on their way.
  constexpr int RI = NR * (D / 2) / THREADS, RSTEP = THREADS / (D / 2);   // rows of the table per thread, and from one to the next
  int pos[RI];
  if constexpr (ROPE) {
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int row = threadIdx.x / (D / 2) + i * RSTEP;
      pos[i] = p.positions ? p.positions[b0 + min(row, n - 1)] : row;
    }
  }
  u32x2 k_lo[KI], k_hi[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int item = threadIdx.x + i * THREADS, row = item / (D / 8), e = item % (D / 8) * 4;
    if (row >= n) continue;
    k_lo[i] = *(const u32x2*)(kg + row * row_stride + e);
    k_hi[i] = *(const u32x2*)(kg + row * row_stride + e + D / 2);
  }
  u32x4 vr[VI];
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    const int unit = threadIdx.x + i * THREADS, row = unit / UPR;
    vr[i] = u32x4{0u, 0u, 0u, 0u};       // rows past the end: weight 0, so the values must be finite
    if (row < n) vr[i] = *(const u32x4*)(vg + row * row_stride + (unit % UPR) * 8);
  }
  // packed query row m is row m % n of the group's head m / n (n <= 128, m < 8 n up to the group: far inside what fp32 tells apart)
  u32x4 qr[KS];
  const float inv_n = 1.f / (float)n;
  auto head_of = [&](int m) { return (int)(((float)m + 0.5f) * inv_n); };
  auto q_index = [&](int m) { const int h = head_of(m); return (long long)(b0 + m - h * n) * p.hq + head_of_slot(p.heads, c * gq + h); };
  auto load_q = [&](int m) {
    const __bf16* q = (const __bf16*)lv.q + q_index(m) * D + 8 * quad;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qr[ks] = *(const u32x4*)(q + 32 * ks);
  };
  if (m_first < rows) load_q(min(m_first + r16, rows - 1));
  if constexpr (ROPE) {
    const int e = threadIdx.x % (D / 2);
    const float hi = p.rope.hi[e], lo = p.rope.lo[e];
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int row = threadIdx.x / (D / 2) + i * RSTEP;
      if (row >= n) continue;
      float sn, cs;
      sincos_turns_fast(rope_turns((float)pos[i], hi, lo), &sn, &cs);
      smc[row * CP + e] = f32x2{cs, sn};
    }
    __syncthreads();
  }
  auto v_swz = [](int row) { return D == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); };
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int item = threadIdx.x + i * THREADS, row = item / (D / 8), e = item % (D / 8) * 4;
    if (row >= n) continue;
    if constexpr (ROPE) {
      float x[4], y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x2 t = smc[row * CP + e + j];
        const float a = j & 1 ? bf16_hi(k_lo[i][j / 2]) : bf16_lo(k_lo[i][j / 2]);
        const float b = j & 1 ? bf16_hi(k_hi[i][j / 2]) : bf16_lo(k_hi[i][j / 2]);
        x[j] = __builtin_fmaf(a, t[0], -(b * t[1]));
        y[j] = __builtin_fmaf(b, t[0], a * t[1]);
      }
      k_lo[i] = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
      k_hi[i] = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
    }
    *(u32x2*)(smk + row * KP + e) = k_lo[i];
    *(u32x2*)(smk + row * KP + e + D / 2) = k_hi[i];
    if (store_k && part == 0) {
      __bf16* dst = (__bf16*)lv.k_rot + ((long long)(b0 + row) * p.hkv + c) * D + e;
      *(u32x2*)dst = k_lo[i];
      *(u32x2*)(dst + D / 2) = k_hi[i];
    }
  }
#pragma unroll
  for (int i = 0; i < VI; ++i) {
    const int unit = threadIdx.x + i * THREADS, row = unit / UPR;
    *(u32x4*)(smv + row * D + (((unit % UPR) ^ v_swz(row)) << 3)) = vr[i];
  }
  __syncthreads();

  for (int m0 = m_first; m0 < rows; m0 += m_step) {
    const int m = min(m0 + r16, rows - 1), qi = m - head_of(m) * n;   // this lane's query row sees keys 0 .. qi
    const long long io = q_index(m);
    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks) {
      u32x4 wl, wh;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x4 t = {1.f, 0.f, 1.f, 0.f};                    // (cos, sin) of pairs 32 ks + 8 quad + 2 j, + 1
        if constexpr (ROPE) t = *(const f32x4*)&smc[qi * CP + 32 * ks + 8 * quad + 2 * j];
        const float a0 = bf16_lo(qr[ks][j]), a1 = bf16_hi(qr[ks][j]);
        const float c0 = bf16_lo(qr[ks + KS / 2][j]), c1 = bf16_hi(qr[ks + KS / 2][j]);
        wl[j] = pack_bf16((a0 * t[0] - c0 * t[1]) * p.scale_log2, (a1 * t[2] - c1 * t[3]) * p.scale_log2);
        wh[j] = pack_bf16((c0 * t[0] + a0 * t[1]) * p.scale_log2, (c1 * t[2] + a1 * t[3]) * p.scale_log2);
      }
      qf[ks] = __builtin_bit_cast(bf16x8, wl);
      qf[ks + KS / 2] = __builtin_bit_cast(bf16x8, wh);
    }
    if (m0 + m_step < rows) load_q(min(m0 + m_step + r16, rows - 1));   // arrives while this one is worked on
    // key blocks that some row of the 16 sees: rows of one head run on, a second head starts again at 0
    const int m_end = min(m0 + 15, rows - 1), h_end = head_of(m_end), last = head_of(m0) == h_end ? m_end - h_end * n : n - 1;
    const int blocks = last / 32 + 1;
    f32x4 sc[2 * NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b >= blocks) continue;
#pragma unroll
      for (int t = 2 * b; t < 2 * b + 2; ++t) {
        sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)(smk + (16 * t + r16) * KP + 32 * ks + 8 * quad), qf[ks], sc[t], 0, 0, 0);
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2 * NB; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (t / 2 >= blocks || 16 * t + 4 * quad + i > qi) sc[t][i] = -INFINITY;
        mx = fmaxf(mx, sc[t][i]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = half_max(mx);                                     // finite: every row sees key 0
    f32x4 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float s0 = 0.f, s1 = 0.f;                              // row sums over the rounded weights
    auto weigh = [&](auto early_c) {
      constexpr bool EARLY = decltype(early_c)::value;
      f32x4 o_early[DB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b >= blocks) continue;
        if (EARLY && b == 2) {
#pragma unroll
          for (int db = 0; db < DB; ++db) o_early[db] = o[db];
        }
        u32x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4& x = sc[2 * b + j / 2];
          w[j] = pack_bf16(__builtin_amdgcn_exp2f(x[2 * (j & 1)] - mx), __builtin_amdgcn_exp2f(x[2 * (j & 1) + 1] - mx));
          add_pair(j & 1 ? s1 : s0, w[j]);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          typedef short s16x8 __attribute__((ext_vector_type(8)));
          const int row = 32 * b + 4 * quad + (r16 >> 2), chunk = 2 * db + ((r16 & 3) >> 1);
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(smv + row * D + ((chunk ^ v_swz(row)) << 3) + 4 * (r16 & 1)));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(smv + (row + 16) * D + ((chunk ^ v_swz(row + 16)) << 3) + 4 * (r16 & 1)));
          const bf16x8 vf = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
          o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, w), o[db], 0, 0, 0);
        }
      }
      if (EARLY) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[db][i] = qi < 64 ? o_early[db][i] : o[db][i];
      }
    };
    // Rows of the first 64 among later ones (a group that spans two heads, or row 64) are done with the first 64 keys: the
    // weights of later ones are 0 for them, but 0 times an infinite value is NaN.
    if (NB > 2 && blocks > 2 && __any(qi < 64)) weigh(std::true_type{}); else weigh(std::false_type{});
    float sum = add_chains(s0, s1);
    sum += __shfl_xor(sum, 16, kWave);
    sum = half_sum(sum);
    if (m0 + r16 >= rows) continue;
    const float inv = 1.f / sum;
    __bf16* orow = (__bf16*)lv.out + io * D + 4 * quad;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *(u32x2*)(orow + 16 * db) = u32x2{pack_bf16(o[db][0] * inv, o[db][1] * inv), pack_bf16(o[db][2] * inv, o[db][3] * inv)};
    if (lv.lse && quad == 0) lv.lse[io] = (mx + __builtin_log2f(sum)) * 0.6931471805599453f;
  }
}

// ------------------------------------------------------------------------------------------------------------------
// Software-pipelined schedule for long sequences (instantiated with 8 waves: 256 query rows per workgroup, one
// workgroup per CU, two waves per SIMD).
//
// A single wave cannot hide its exponentials behind its own matrix products when the two alternate, and two waves of a
// SIMD that meet at a barrier every tile fall into step, so they do not hide them for each other either.  Here every
// wave overlaps them itself: while the matrix core accumulates the scores of tile t+1, the vector ALU takes the
// exponentials of tile t, instruction by instruction in one stream; then O^T += V^T P^T of tile t follows at once.  The
// matrix core always has the next product queued.
//
//   iteration t:  barrier t (K(t+1) and V(t) have landed; start K(t+2), V(t+1))
//                 S(t+1) = K(t+1) Q^T - m   interleaved with   P(t) = exp2(S(t)), row sums
//                 [sums too large -> reference stale: recompute S(t) exactly from K(t), which is still in LDS]
//                 O += V(t) P(t)
//
// K tiles live in a ring of 3 (t: kept for the exact path, t+1: being multiplied, t+2: in flight), V tiles in a ring
// of 2 (t: being multiplied, t+1: in flight).  The two score tiles swap roles every iteration; the loop is unrolled by
// two so that the swap costs no register moves.
// ------------------------------------------------------------------------------------------------------------------
template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 1 : 2) void prefill_pipe_kernel(PrefillParams p) {
  constexpr int KSTEPS = D / 16, DB = D / 32;
  constexpr int UPM = 16 / (2 * KSTEPS);  // softmax units per score MFMA: 1 (D = 128) or 2 (D = 64)
  __shared__ __bf16 smk[3][kTileKeys * D];
  __shared__ __bf16 smv[2][kTileKeys * D];

  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const PfBlock blk = pf_map_block<WAVES>(p, wave);
  if (!blk.valid) return;
  const PfLayer lv = pf_layer_view(p, blockIdx.y);
  const int b0 = blk.b0, n = blk.n;
  const int r32 = lane & 31, hf = lane >> 5;
  const int qw = blk.qw;
  const bool wave_active = qw < n;
  const int t_diag = qw / kTileKeys;
  const int q_in_tile = qw - t_diag * kTileKeys;
  const int n_tiles = (blk.end + kTileKeys - 1) / kTileKeys;

  TileStager<D, WAVES> stager;
  stager.init((const __bf16*)lv.k_rot + ((long long)b0 * p.hkv + blk.c) * D, (const __bf16*)lv.v + ((long long)b0 * p.hkv + blk.c) * D,
              n, p.hkv, wave, lane);
  const unsigned lds_k = (unsigned)(size_t)(lds_void_ptr)&smk[0][0], lds_v = (unsigned)(size_t)(lds_void_ptr)&smv[0][0];
  auto issue_k = [&](int t) { stager.issue(stager.k_rsrc, lds_k + (unsigned)((t % 3) * kTileKeys * D * 2), t); };
  auto issue_v = [&](int t) { stager.issue(stager.v_rsrc, lds_v + (unsigned)((t & 1) * kTileKeys * D * 2), t); };
  // Barrier t.  Before it every wave has waited for its own loads, i.e. its parts of K(t+1) and V(t), issued behind
  // barrier t-1.  Behind it nobody reads K(t-1) (last use: the exact path of iteration t-1) or V(t-1) any more, which is
  // where K(t+2) and V(t+1) go.
  auto sync_and_stage = [&](int t) {
    drain_loads_and_barrier();
    if (t + 2 < n_tiles) issue_k(t + 2);
    if (t + 1 < n_tiles) issue_v(t + 1);
  };
  issue_k(0);
  issue_v(0);
  if (n_tiles > 1) issue_k(1);

  bf16x8 qf[KSTEPS];
  {
    const int qi = min(qw + r32, n - 1);
    const __bf16* qrow = (const __bf16*)lv.q + ((long long)(b0 + qi) * p.hq + blk.a) * D + 8 * hf;
    f32x4 cs[D / 8];
    pf_load_cs<D>(p, b0 + qi, hf, cs);
    pf_rotate_q<D>(p, [&](int ks) { return qrow + 16 * ks; }, cs, qf);
  }
  FragOffsets<D> fo;
  fo.init(lane);

  f32x16 o[DB], neg_m;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_m[i] = 0.f;
  float mrow = 0.f, lrow = 0.f;
  f32x16 sa[2], sb[2];  // score tiles (minus m): one has its exponentials taken while the other is accumulated

  // ---- tile 0: exact maxima, so that the pipeline starts from a finite reference ----
  drain_loads_and_barrier();  // K(0), V(0), K(1)
  if (wave_active) {
    score_tile<D, true>(smk[0], fo, qf, neg_m, sa);
    if (t_diag == 0) mask_diagonal(sa, q_in_tile, r32, hf);
    float m = sa[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, sa[kb][i]);
    mrow = half_max(m);  // finite: key 0 is visible to every query
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) sa[kb][i] -= mrow;
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_m[i] = -mrow;

  // The reference of tile t turned out stale (or its sums overflowed): redo the tile exactly.  K(t) is still in LDS.
  // The next tile's scores were started from the old reference and move with it.
  auto exact_redo = [&](int t, f32x16 (&nxt)[2], bool have_next, u32x4 (&w)[4], float& lsum, bf16x8 (&vf0)[DB]) {
    f32x16 sc[2];
    score_tile<D, true>(smk[t % 3], fo, qf, neg_m, sc);
    if (t == t_diag) mask_diagonal(sc, q_in_tile, r32, hf);
    float m = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, sc[kb][i]);
    const float mnew = fmaxf(mrow, half_max(m));
    const float shift = mrow - mnew;  // <= 0
    const float alpha = __builtin_amdgcn_exp2f(shift);
    mrow = mnew;
    lrow *= alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) neg_m[i] = -mnew;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    if (have_next) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) nxt[kb][i] += shift;
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[kb][i] -= mnew;
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) softmax_unit(sc, u, w, s0, s1);
    lsum = add_chains(s0, s1);
    // requested again rather than kept: this path is short of registers, not of time
#pragma unroll
    for (int db = 0; db < DB; ++db) vf0[db] = read_v_fragment<D>(smv[t & 1], fo, db, 0);
  };

  // one iteration; cur = S(t) - m (consumed), nxt = S(t+1) - m (produced)
  auto iteration = [&](int t, f32x16 (&cur)[2], f32x16 (&nxt)[2]) {
    sync_and_stage(t);
    if (!(wave_active && t <= t_diag)) return;  // rows past the sequence end, tiles past the diagonal: only stage
    const bool have_next = t < t_diag;
    const __bf16* smv_t = smv[t & 1];
    u32x4 w[4];
    bf16x8 vf[2][DB];  // V^T fragments of two 16-key steps: one feeding the MFMAs, one arriving
    float lsum, s0 = 0.f, s1 = 0.f;
    if (have_next) {
      // S(t+1) on the matrix core, exponentials of S(t) on the vector ALU, in ONE instruction stream laid out by hand:
      // slot i = [K fragment requests two k-steps ahead] + MFMA i + exponentials of softmax unit(s) i + packing and row
      // sum of unit(s) i-1 (whose exponentials have had a slot's time to finish).  The scheduling barriers keep the
      // compiler from regrouping the slots; the last slots also request the first V^T fragments of the second product.
      const __bf16* smk_n = smk[(t + 1) % 3];
      constexpr int AHEAD = 2 < KSTEPS ? 2 : KSTEPS;
      constexpr int SLOTS = 2 * KSTEPS;
      bf16x8 kf[2][KSTEPS];
      float e[2][UPM][2];  // exponentials of the units of slot i (parity i & 1)
#pragma unroll
      for (int ks = 0; ks < AHEAD; ++ks)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) kf[kb][ks] = *(const bf16x8*)(smk_n + fo.k(ks) + kb * 32 * D);
#pragma unroll
      for (int i = 0; i <= SLOTS; ++i) {
        const int ks = i >> 1, kb = i & 1;
        if (i < SLOTS) {
          if (kb == 0 && ks + AHEAD < KSTEPS) {
#pragma unroll
            for (int b = 0; b < 2; ++b) kf[b][ks + AHEAD] = *(const bf16x8*)(smk_n + fo.k(ks + AHEAD) + b * 32 * D);
          }
          if (i >= SLOTS - DB) vf[0][i - (SLOTS - DB)] = read_v_fragment<D>(smv_t, fo, i - (SLOTS - DB), 0);
          nxt[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][ks], qf[ks], ks == 0 ? neg_m : nxt[kb], 0, 0, 0);
#pragma unroll
          for (int x = 0; x < UPM; ++x) {
            const int u = i * UPM + x, kk = u >> 2, j = u & 3, r = 8 * (kk & 1) + 2 * j;
            e[i & 1][x][0] = __builtin_amdgcn_exp2f(cur[kk >> 1][r]);
            e[i & 1][x][1] = __builtin_amdgcn_exp2f(cur[kk >> 1][r + 1]);
          }
        }
        if (i > 0) {
#pragma unroll
          for (int x = 0; x < UPM; ++x) {
            const int u = (i - 1) * UPM + x, kk = u >> 2, j = u & 3;
            w[kk][j] = pack_bf16(e[(i - 1) & 1][x][0], e[(i - 1) & 1][x][1]);
            add_pair(j & 1 ? s1 : s0, w[kk][j]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (t + 1 == t_diag) {
        asm volatile("" ::: "memory");  // keeps this a branch: only one tile per wave needs the mask
        mask_diagonal(nxt, q_in_tile, r32, hf);
      }
    } else {
      // the wave's last tile: nothing to overlap with
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int kk = u >> 2, j = u & 3, r = 8 * (kk & 1) + 2 * j;
        float x0 = cur[kk >> 1][r], x1 = cur[kk >> 1][r + 1];
        asm("" : "+v"(x0), "+v"(x1));  // keeps these exponentials apart from the ones in the other branch, which must stay in their slots
        w[kk][j] = pack_bf16(__builtin_amdgcn_exp2f(x0), __builtin_amdgcn_exp2f(x1));
        add_pair(j & 1 ? s1 : s0, w[kk][j]);
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) vf[0][db] = read_v_fragment<D>(smv_t, fo, db, 0);
    }
    lsum = add_chains(s0, s1);
    if (__any(!(lsum <= kSumLimit))) exact_redo(t, nxt, have_next, w, lsum, vf[0]);
    lrow += lsum;
    // O^T += V^T P^T, the fragments of the next 16-key step requested while this step's MFMAs run
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        if (kk + 1 < 4) vf[(kk + 1) & 1][db] = read_v_fragment<D>(smv_t, fo, db, kk + 1);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kk & 1][db], __builtin_bit_cast(bf16x8, w[kk]), o[db], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  // unrolled by two; an odd tile count ends in an iteration past the last tile, which only meets the barrier
  for (int t = 0; t < n_tiles; t += 2) {
    iteration(t, sa, sb);
    iteration(t + 1, sb, sa);
  }

  if (!wave_active) return;
  const int qi = qw + r32;
  const float ltot = half_sum(lrow);
  if (qi >= n) return;
  pf_store_row<D>((__bf16*)lv.out + ((long long)(b0 + qi) * p.hq + blk.a) * D + 4 * hf, o, 1.f / ltot);
  if (lv.lse && hf == 0) lv.lse[(long long)(b0 + qi) * p.hq + blk.a] = (mrow + __builtin_log2f(ltot)) * 0.6931471805599453f;
}

// ------------------------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------------------------
// rotated keys when the caller keeps none
static size_t k_rot_bytes(const earn_attn_desc* desc, int total_tokens) {
  const size_t e = desc->dtype == EARN_F32 ? 4 : 2;
  return ((size_t)total_tokens * desc->n_kv_heads * desc->head_dim * e + 255) / 256 * 256;
}
// (cos, sin) table of the bf16 paths: [d/4][tokens] of four floats, two pairs
static size_t cs_table_bytes(const earn_attn_desc* desc, int total_tokens) {
  if (desc->dtype == EARN_F32) return 0;
  return ((size_t)total_tokens * (desc->head_dim / 2) * sizeof(f32x2) + 255) / 256 * 256;
}
// workspace layout: [rotated keys, unless the caller passes k_rot_out][cos/sin table]
// Without rotation and without k_rot_out nothing is staged at all: the keys are read in place.
size_t prefill_workspace_bytes(const earn_attn_desc* desc, int total_tokens, int have_k_rot_out) {
  if (!(desc->rope_base > 0.f) && !have_k_rot_out) return 0;
  return (have_k_rot_out ? 0 : k_rot_bytes(desc, total_tokens)) + cs_table_bytes(desc, total_tokens);
}

template <typename T, int D>
static void launch_rope_k(const void* k, void* k_rot, const int32_t* cu, const int32_t* positions, int batch, int total,
                          int hkv, const RopeTable& rope, f32x4* cs_out, hipStream_t stream, int n_layers = 1,
                          long long ls_k = 0, long long ls_k_rot = 0) {
  long long threads = (long long)total * (D / 16);
  const unsigned gx = (unsigned)((threads + 255) / 256);
  // fewer than about two workgroups per CU: split the heads over grid rows as well
  const int hpt = (long long)gx * n_layers >= 512 ? hkv : (hkv + 7) / 8;
  hipLaunchKernelGGL((rope_k_kernel<T, D>), dim3(gx, (unsigned)((hkv + hpt - 1) / hpt), n_layers), dim3(256), 0, stream,
                     (const T*)k, (T*)k_rot, cu, positions, batch, total, hkv, rope, cs_out, hpt, ls_k, ls_k_rot);
}

// fp32: the chosen rows of every sequence (q_rows, out_rows: [batch * r, Hq, d]) against the rotated keys
int launch_prefill_rows_f32(const earn_attn_desc* desc, const void* q_rows, const void* k_rot, const void* v,
                            const int32_t* cu_seqlens, const int32_t* row_pos, int batch, int total_tokens,
                            int max_seqlen, int rows_per_seq, void* out_rows, hipStream_t stream) {
  const int d = desc->head_dim;
  PrefillParams p;
  p.cs = nullptr; p.row_pos = row_pos; p.rows_per_seq = rows_per_seq;
  p.q = q_rows; p.k_rot = k_rot; p.v = v; p.cu = cu_seqlens; p.positions = nullptr; p.out = out_rows; p.lse = nullptr;
  p.batch = batch; p.hq = desc->n_q_heads; p.hkv = desc->n_kv_heads; p.max_seqlen = max_seqlen; p.n_qblk = 1;
  p.total = total_tokens;
  p.ls_q = p.ls_k_rot = p.ls_v = p.ls_out = p.ls_lse = 0;
  const float scale = desc->softmax_scale > 0.f ? desc->softmax_scale : 1.0f / sqrtf((float)d);
  p.scale_log2 = scale * 1.4426950408889634f;
  p.rope = make_rope_table(desc->rope_base, d);
  if (make_head_map(desc, &p.heads, "earn_prefill_register_rows") != EARN_OK) return EARN_ERR_UNSUPPORTED;
  if (d == 64) launch_prefill_f32<64>(p, nullptr, 0, nullptr, false, rows_per_seq, 1, stream);
  else launch_prefill_f32<128>(p, nullptr, 0, nullptr, false, rows_per_seq, 1, stream);
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

// K rotation on its own (for callers that run the attention with another kernel)
int launch_rope_keys(const earn_attn_desc* desc, const void* k, void* k_rot, const int32_t* cu_seqlens,
                     const int32_t* positions, int batch, int total_tokens, hipStream_t stream) {
  const RopeTable rope = make_rope_table(desc->rope_base, desc->head_dim);
  const int hkv = desc->n_kv_heads;
  if (desc->dtype == EARN_F32) {
    if (desc->head_dim == 64) launch_rope_k<float, 64>(k, k_rot, cu_seqlens, positions, batch, total_tokens, hkv, rope, nullptr, stream);
    else launch_rope_k<float, 128>(k, k_rot, cu_seqlens, positions, batch, total_tokens, hkv, rope, nullptr, stream);
  } else {
    if (desc->head_dim == 64) launch_rope_k<__bf16, 64>(k, k_rot, cu_seqlens, positions, batch, total_tokens, hkv, rope, nullptr, stream);
    else launch_rope_k<__bf16, 128>(k, k_rot, cu_seqlens, positions, batch, total_tokens, hkv, rope, nullptr, stream);
  }
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

int launch_prefill(const earn_attn_desc* desc, const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                   const int32_t* positions, int batch, int total_tokens, int max_seqlen, void* out, void* k_rot_out,
                   float* lse_out, void* workspace, size_t workspace_bytes, hipStream_t stream,
                   const PrefillLayers* layers) {
  const int d = desc->head_dim;
  const int n_layers = layers ? layers->n_layers : 1;
  const long long ls_k = layers ? layers->kv : 0, ls_kr = layers ? layers->k_rot : 0;
  if ((long long)batch * n_layers > 65535 && desc->dtype == EARN_F32) {
    set_error("earn_prefill_attn_layers: batch * n_layers = %lld exceeds 65535 (fp32 launch shape)", (long long)batch * n_layers);
    return EARN_ERR_UNSUPPORTED;
  }
  const size_t need = prefill_workspace_bytes(desc, total_tokens, k_rot_out != nullptr);
  if (need > workspace_bytes || (need > 0 && !workspace)) {
    set_error("earn_prefill_attn: workspace too small (%zu bytes given, %zu needed)", workspace_bytes, need);
    return EARN_ERR_WORKSPACE_TOO_SMALL;
  }
  // the matrix-core kernels address the K/V rows of ONE sequence with 32-bit byte offsets
  if (desc->dtype == EARN_BF16 && (long long)(max_seqlen + 256) * desc->n_kv_heads * d * 2 >= (1ll << 31)) {
    set_error("earn_prefill_attn: a sequence of %d rows exceeds the 2 GiB addressing range of one sequence", max_seqlen);
    return EARN_ERR_UNSUPPORTED;
  }
  // no rotation and no cache copy asked for: the keys (already rotated by their producer) are read where they are
  const bool in_place = !(desc->rope_base > 0.f) && !k_rot_out;
  const void* k_rot = in_place ? k : (k_rot_out ? k_rot_out : workspace);
  f32x4* cs = !in_place && cs_table_bytes(desc, total_tokens) ? (f32x4*)((char*)workspace + (k_rot_out ? 0 : k_rot_bytes(desc, total_tokens))) : nullptr;
  PrefillParams p;
  p.cs = cs; p.row_pos = nullptr; p.rows_per_seq = 0;
  p.q = q; p.k_rot = k_rot; p.v = v; p.cu = cu_seqlens; p.positions = positions; p.out = out; p.lse = lse_out;
  p.batch = batch; p.hq = desc->n_q_heads; p.hkv = desc->n_kv_heads; p.max_seqlen = max_seqlen;
  p.total = total_tokens;
  p.ls_q = layers ? layers->q : 0; p.ls_k_rot = in_place ? ls_k : ls_kr; p.ls_v = ls_k; p.ls_out = layers ? layers->out : 0;
  p.ls_lse = layers ? layers->lse : 0;
  const float scale = desc->softmax_scale > 0.f ? desc->softmax_scale : 1.0f / sqrtf((float)d);
  p.scale_log2 = scale * 1.4426950408889634f;
  p.rope = make_rope_table(desc->rope_base, d);
  if (make_head_map(desc, &p.heads, "earn_prefill_attn") != EARN_OK) return EARN_ERR_UNSUPPORTED;
  const bool f32 = desc->dtype == EARN_F32;
  auto set_query_blocks = [&p](int rows, int waves) {
    const unsigned gq = (unsigned)(p.hq / p.hkv);
    p.n_qblk = unit_blocks(rows, (int)gq, waves);
    p.by_pair = FastDiv::of((unsigned)p.n_qblk); p.by_group = FastDiv::of(gq); p.by_kv = FastDiv::of((unsigned)p.hkv);
  };
  // prefill_short_kernel: grouped heads up to 128 rows (beyond 64: short_prefill_takes), single heads up to 32.  us per layer
  // with rotation, one launch per layer / 24 layers in one launch, the kernels of longer sequences (and a rotation pass) -> this one:
  //   256 sequences, 12 / 2 heads of 128: 16 rows 29.8 / 18.9 -> 13.4 / 8.2, 64 rows 60.0 / 44.7 -> 41.0 / 32.4, 128 rows
  //   105.9 / 90.5 -> 81.2 / 71.0; 64 sequences, 32 / 8 heads: 64 rows 43.2 / 31.3 -> 29.0 / 23.4, 128 rows 75.7 / 63.0 ->
  //   61.0 / 49.9; 32 sequences, 14 / 2 heads of 64: 16 rows 9.4 / 1.6 -> 6.6 / 0.7, 128 rows 16.2 / 7.2 -> 12.5 / 5.1.
  //   64 sequences, 32 / 32 heads, where every workgroup has keys of its own to stage and little to multiply: 32 rows
  //   34.4 / 27.4 -> 29.5 / 21.8, 64 rows 57.6 / 53.4 -> 60.6 / 46.6 (without rotation 38.7 -> 40.4), 96 rows 85 / 75 ->
  //   95 / 80.
  // (and as many pairs as its grid takes: single heads have twice the room in the other kernel's smaller workgroups)
  const bool few_rows = max_seqlen <= (p.hq > p.hkv ? 128 : 32) && run_fits(batch, p.hkv, max_seqlen <= 64 ? 256 : 512) &&
                        short_prefill_takes(max_seqlen, total_tokens / batch, (long long)batch * p.hkv * n_layers, in_place);
  if (f32) {
    // (the bound given may be far above any sequence; none is longer than all of them together)
    const int longest = std::min(max_seqlen, total_tokens);
    // the keys are rotated by the attention kernel where there are few workgroups (and not in place: others read them)
    const bool rotate = !in_place && k != k_rot_out && f32_few_workgroups(longest, p.hq, d, (long long)batch * n_layers);
    if (!in_place && !rotate) {
      if (d == 64) launch_rope_k<float, 64>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
      else launch_rope_k<float, 128>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
    }
    if (d == 64) launch_prefill_f32<64>(p, k, ls_k, k_rot_out, rotate, longest, n_layers, stream);
    else launch_prefill_f32<128>(p, k, ls_k, k_rot_out, rotate, longest, n_layers, stream);
  } else if (few_rows) {
    auto launch = [&](auto kernel, int waves, int per_cu) {
      // Few (sequence, kv head) pairs: several workgroups per pair, each with its own copy of the keys, as many as an XCD
      // holds at a time, per_cu on each of its 32 CUs (2 sequences, 32 / 8 heads, 64 rows: 17.0 -> 10.2 us).
      // groups: of 16 query rows, in a pair.  (Keys rotated in place have one reader: the others would race with its stores.)
      const long long groups = ((long long)(p.hq / p.hkv) * max_seqlen + 15) / 16;
      const long long on_xcd = ((long long)batch * p.hkv * n_layers + kXcds - 1) / kXcds;
      const int parts = k == k_rot_out ? 1 : (int)std::max<long long>(1, std::min<long long>((groups + waves - 1) / waves, 32 * per_cu / on_xcd));
      set_query_blocks(max_seqlen, waves);
      p.by_run = FastDiv::of((unsigned)(p.hkv * parts));
      const dim3 grid((unsigned)run_workgroups(batch, p.hkv * parts), n_layers, 1);
      hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, stream, p, k, ls_k, k_rot_out ? 1 : 0, parts);
    };
    auto launch_d = [&](auto rope_c) {
      constexpr bool ROPE = decltype(rope_c)::value;
      if (max_seqlen <= 32) {
        if (d == 64) launch(prefill_short_kernel<64, 32, 4, ROPE>, 4, short_per_cu(64, 32, 4, ROPE)); else launch(prefill_short_kernel<128, 32, 4, ROPE>, 4, short_per_cu(128, 32, 4, ROPE));
      } else if (max_seqlen <= 64) {
        if (d == 64) launch(prefill_short_kernel<64, 64, 4, ROPE>, 4, short_per_cu(64, 64, 4, ROPE)); else launch(prefill_short_kernel<128, 64, 4, ROPE>, 4, short_per_cu(128, 64, 4, ROPE));
      } else {
        if (d == 64) launch(prefill_short_kernel<64, 128, 8, ROPE>, 8, short_per_cu(64, 128, 8, ROPE)); else launch(prefill_short_kernel<128, 128, 8, ROPE>, 8, short_per_cu(128, 128, 8, ROPE));
      }
    };
    if (p.rope.enabled) launch_d(std::true_type{}); else launch_d(std::false_type{});
  } else if (max_seqlen <= kTileKeys) {
    // single heads, one K/V tile
    if (!in_place) {
      if (d == 64) launch_rope_k<__bf16, 64>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
      else launch_rope_k<__bf16, 128>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
    }
    set_query_blocks(max_seqlen, 2);
    const long long pairs8 = ((long long)batch * p.hkv + kXcds - 1) / kXcds * kXcds;
    dim3 grid((unsigned)(pairs8 * p.n_qblk), n_layers, 1);
    if (d == 64) hipLaunchKernelGGL((prefill_mfma_kernel<64, 2, 1>), grid, dim3(128), 0, stream, p);
    else hipLaunchKernelGGL((prefill_mfma_kernel<128, 2, 1>), grid, dim3(128), 0, stream, p);
  } else {
    if (!in_place) {
      if (d == 64) launch_rope_k<__bf16, 64>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
      else launch_rope_k<__bf16, 128>(k, (void*)k_rot, cu_seqlens, positions, batch, total_tokens, p.hkv, p.rope, cs, stream, n_layers, ls_k, ls_kr);
    }
    // 128-row workgroups (two per CU) in the plain schedule up to medium lengths, where the ends of a workgroup's
    // life (first tile's latency, output store) and the causal diagonal weigh most; the pipelined 256-row kernel beyond.
    // What counts is the length of most sequences, not of the longest: a ragged batch whose mean length is medium
    // takes the 128-row form whatever its longest sequence (lengths spread over 269-4018, mean 1411: 1.18 against
    // 1.27 ms per layer).
    const int rows_set = tuning(kTunePrefillBlockRows, 0);
    const bool medium = max_seqlen <= 3072 || total_tokens / batch <= 2048;
    const int block_rows = rows_set == 128 || rows_set == 256 ? rows_set : (medium ? 128 : 256);
    set_query_blocks(max_seqlen, block_rows / 32);
    const long long pairs8 = ((long long)batch * p.hkv + kXcds - 1) / kXcds * kXcds;
    dim3 grid((unsigned)(pairs8 * p.n_qblk), n_layers, 1);
    if (block_rows == 128) {
      auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, p); };
      const bool direct_q = (((unsigned long long)q | (unsigned long long)p.ls_q) & 15) == 0;
      if (d == 64) direct_q ? launch(prefill_mfma_kernel<64, 4, 2>) : launch(prefill_mfma_kernel<64, 4, 2, false>);
      else direct_q ? launch(prefill_mfma_kernel<128, 4, 2>) : launch(prefill_mfma_kernel<128, 4, 2, false>);
    } else {
      if (d == 64) hipLaunchKernelGGL((prefill_pipe_kernel<64, 8>), grid, dim3(512), 0, stream, p);
      else hipLaunchKernelGGL((prefill_pipe_kernel<128, 8>), grid, dim3(512), 0, stream, p);
    }
  }
  return hipGetLastError() == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}

}  // namespace earn

#ifdef EARN_PF_TIMELINE
// buf: device memory of slots * 8 64-bit words, zeroed by the caller; NULL switches the timers off
extern "C" int earn_debug_set_timeline(void* buf, int slots) {
  if (hipMemcpyToSymbol(HIP_SYMBOL(earn::g_pf_timeline_slots), &slots, sizeof(slots)) != hipSuccess) return EARN_ERR_HIP;
  return hipMemcpyToSymbol(HIP_SYMBOL(earn::g_pf_timeline), &buf, sizeof(buf)) == hipSuccess ? EARN_OK : EARN_ERR_HIP;
}
#endif
