// Decode attention over the INT2 paged cache (Alg. 1 DecodeStep; Sec. 4
// "Decoding Attention Kernel"), in three kernels:
//   prepare : q~ = q R_k * (sm_scale * log2 e)                    [B*Hq, 128] fp32
//             (in append.hip, where it can share a launch with the cache update)
//   split   : online softmax over page ranges in the rotated basis, unnormalized
//             o~ and (m, l) per piece (decode_mfma.hip)
//   reduce  : log-sum-exp merge of the pieces, o = o~ R_v^T, bf16/fp32 store
//             (this file)
//
// Rotated-basis identities used (Sec. 2, K^ = Q(K~) R^T with R orthogonal):
//   q k^T = (q R_k) Q(k~)^T,   sum_t p_t v^_t = (sum_t p_t Q(v~_t)) R_v^T,
// and per group g of 32 channels, with Q(x~)_c = s_g (code_c - z_g):
//   q~ . Q(k~) = sum_g s_g (sum_{c in g} q~_c code_c - z_g sum_{c in g} q~_c).
// Scores are kept in log2 units (q~ carries log2 e) so the softmax uses exp2.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "internal.h"

namespace oscar {
namespace {

__device__ inline uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}


// ---------------------------------------------------------------------------
// reduce: RB (sequence, head) rows per block of 8 waves, 512 / RB threads a row: 32
// float4 columns x SG = 16 / RB groups of slots.
//   1. thread (row, slot group, column): M = max_s m_s, L = sum_s 2^(m_s - M) l_s
//      over the row's splits (empty splits have m_s = -inf and only follow live
//      ones), then o~[c] = sum_s 2^(m_s - M) part_o[s][c] / L over the group's live
//      splits (s = group, group + SG, ..), with independent loads over s; the
//      groups are added in LDS;
//   2. o = o~ R_v^T on the fp32 matrix cores: wave w computes column tile w of the
//      rows (a 16-row tile; rows RB.. of it are zero) as 32 chained 16x16x4 MFMAs,
//      step s taking channel c = 32k + s in k-slot k (A: lane (row lo, k-slot hi)
//      reads o~[lo][32hi + s] from LDS; B: lane (column lo, k-slot hi) holds
//      R_v[16w + lo][32hi + s], 128 contiguous bytes of a row of R_v read from L2
//      at the start, before the loads of the partial states).  D lane (column
//      lo, hi): rows 4hi + i.
// Bound: latency (the slots' maxima, then their states, then the products).  Few rows
// are spread over more blocks, with the slots of a row read by more threads at once:
// 40 slots of 64 rows took three dependent rounds of loads at 8 rows per block of
// 256 threads (10.4 us; 7.1 us now).  Eight slots a round: sixteen, of which a short
// sequence fills one or two, took 13.8 us instead of 10.4 at 8192 rows of one slot and
// 93 instead of 58 at 65536.
// ---------------------------------------------------------------------------
constexpr int kOmPitch = kD + 4;  // LDS row pitch of o~ (floats)

constexpr int kRedThreads = 512;

typedef float red_f4 __attribute__((ext_vector_type(4)));

// MIXED: a row has num_splits + 1 slots; the last holds the bf16 tokens' state
// in the original basis, o = (sum_s e_s o~_s R_v^T + e_b o_b) / L.
// Rows are taken RB per block in the natural order, or (rph: one R_v per KV
// head) RB rows of one KV head per block.
template <bool MIXED, int RB>
__global__ __launch_bounds__(kRedThreads) void reduce_kernel(int rows, int num_splits,
                                                     const float* __restrict__ part_o,
                                                     const float* __restrict__ part_ml,
                                                     const float* __restrict__ Rv,
                                                     void* __restrict__ out, int out_f32, int rph,
                                                     int Hq, int Hkv) {
  constexpr int kRedRows = RB;
  constexpr int TPR = kRedThreads / RB;  // threads per row in the merge
  constexpr int SG = TPR / 32;           // groups of slots
  constexpr int SR = 8;                  // slots of a group whose loads are issued together
  __shared__ float om[16 * kOmPitch];
  __shared__ float4 og[SG > 1 ? RB * (SG - 1) : 1][kD / 4];  // sums of groups 1..
  __shared__ float mx[kRedThreads / 64][2];                   // per wave: maximum, live slots
  __shared__ float lg[RB * SG];                               // per group: sum of the weights
  __shared__ float eb_il[16];  // MIXED: e_b / L per row
  const int stride = MIXED ? num_splits + 1 : num_splits;
  const int t = threadIdx.x, w = t >> 6, lo = t & 15, hi = (t >> 4) & 3;
  int kvh;
  query_row(blockIdx.x, 0, kRedRows, rows, Hq, Hkv, rph, kvh);
  if (Rv && rph) Rv += (size_t)kvh * kD * kD;
  auto row_of = [&](int r) {  // the block's r-th row, or rows (past the end)
    int kv_;
    const int x = query_row(blockIdx.x, r, kRedRows, rows, Hq, Hkv, rph, kv_);
    return x < 0 ? rows : x;
  };
  // R_v operands of the wave's column tile, issued first (L2)
  float4 rb[8];
  if (Rv) {
    const float4* src = reinterpret_cast<const float4*>(Rv + (size_t)(16 * w + lo) * kD + 32 * hi);
#pragma unroll
    for (int k = 0; k < 8; ++k) rb[k] = src[k];
  }
  if (RB < 16)  // rows RB..15 of the MFMA tile
    for (int i = t; i < (16 - RB) * kOmPitch; i += kRedThreads) om[RB * kOmPitch + i] = 0.0f;
  {  // RB rows x SG slot groups x 32 columns
    const int rr = t / TPR, tr = t % TPR, c8 = tr % 32, sg = tr / 32, r = row_of(rr);
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const float2* ml = reinterpret_cast<const float2*>(part_ml + (size_t)r * stride * 2);
    // live slots lead (empty ones only follow the end of a sequence): n_live is
    // one past the last live slot.  Slot s is read by thread s % TPR of the row;
    // maximum and last live slot are then reduced over the row's threads.
    float M = -INFINITY;
    int n_live = 0;
    if (r < rows)
      for (int s = tr; s < num_splits; s += TPR) {
        const float m = ml[s].x;
        M = fmaxf(M, m);
        n_live = (m != -INFINITY) ? s + 1 : n_live;
      }
    constexpr int kIn = TPR < 64 ? TPR : 64;  // threads of the row in a wave
#pragma unroll
    for (int off = kIn / 2; off >= 1; off >>= 1) {
      M = fmaxf(M, __shfl_xor(M, off, 64));
      n_live = max(n_live, __shfl_xor(n_live, off, 64));
    }
    if (TPR > 64) {  // a row's waves
      if ((t & 63) == 0) {
        mx[w][0] = M;
        mx[w][1] = __int_as_float(n_live);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < TPR / 64; ++k) {
        M = fmaxf(M, mx[rr * (TPR / 64) + k][0]);
        n_live = max(n_live, __float_as_int(mx[rr * (TPR / 64) + k][1]));
      }
    }
    float2 mb = make_float2(-INFINITY, 0.0f);
    if (MIXED && r < rows) mb = ml[num_splits];
    if (MIXED) M = fmaxf(M, mb.x);
    float L = 0.0f;
    if (r < rows && M != -INFINITY) {
      const float4* po = reinterpret_cast<const float4*>(part_o + (size_t)r * stride * kD) + c8;
      // up to SR slots of the group per round, loads issued together (indices
      // clamped to the live range, weights of the clamped repeats set to 0)
      for (int s0 = sg; s0 < n_live; s0 += SR * SG) {
        float2 m[SR];
        float4 x[SR];
#pragma unroll
        for (int k = 0; k < SR; ++k) {
          const int s = min(s0 + SG * k, n_live - 1);
          m[k] = ml[s];
          x[k] = po[(size_t)s * (kD / 4)];
        }
#pragma unroll
        for (int k = 0; k < SR; ++k) {
          const bool use = s0 + SG * k < n_live && m[k].x != -INFINITY;  // empty slots add nothing
          const float e = use ? exp2f(m[k].x - M) : 0.0f;
          L = fmaf(e, use ? m[k].y : 0.0f, L);
          o.x = fmaf(e, use ? x[k].x : 0.0f, o.x);
          o.y = fmaf(e, use ? x[k].y : 0.0f, o.y);
          o.z = fmaf(e, use ? x[k].z : 0.0f, o.z);
          o.w = fmaf(e, use ? x[k].w : 0.0f, o.w);
        }
      }
    }
    if (SG > 1) {
      __syncthreads();  // mx has been read
      if (sg > 0) og[rr * (SG - 1) + sg - 1][c8] = o;
      if (c8 == 0) lg[rr * SG + sg] = L;
      __syncthreads();
    }
    if (sg == 0) {
#pragma unroll
      for (int k = 1; k < SG; ++k) {
        const float4 v = og[rr * (SG - 1) + k - 1][c8];
        o.x += v.x;
        o.y += v.y;
        o.z += v.z;
        o.w += v.w;
        L += lg[rr * SG + k];
      }
      float eb = 0.0f;
      if (MIXED && mb.x != -INFINITY) {
        eb = exp2f(mb.x - M);
        L = fmaf(eb, mb.y, L);
      }
      const float il = L > 0.0f ? 1.0f / L : 0.0f;
      o.x *= il; o.y *= il; o.z *= il; o.w *= il;
      *reinterpret_cast<float4*>(&om[rr * kOmPitch + 4 * c8]) = o;
      if (MIXED && c8 == 0) eb_il[rr] = eb * il;
    }
  }
  __syncthreads();
  // lane (column lo, hi): out[row 4hi + i][16 w + lo]
  auto store = [&](int i, float v) {
    const int rr = 4 * hi + i, col = 16 * w + lo;
    if (rr >= RB) return;
    const int r = row_of(rr);
    if (r >= rows) return;
    if (MIXED) {  // the bf16 tokens' part, already in the original basis
      const float e = eb_il[rr];
      if (e != 0.0f) v = fmaf(e, part_o[((size_t)r * stride + num_splits) * kD + col], v);
    }
    if (out_f32) static_cast<float*>(out)[(size_t)r * kD + col] = v;
    else static_cast<uint16_t*>(out)[(size_t)r * kD + col] = f32_to_bf16_rne(v);
  };
  if (!Rv) {  // R = I (bf16 baseline)
#pragma unroll
    for (int i = 0; i < 4; ++i) store(i, om[(4 * hi + i) * kOmPitch + 16 * w + lo]);
    return;
  }
  // The products first, then the stores, on a path no other branch joins: with the
  // identity case as the other arm of an if/else whose join read the MFMA results,
  // the compiler put no wait states between the last MFMA and the first read of its
  // result (wrong values in one result register).
  red_f4 d = red_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float4 a = *reinterpret_cast<const float4*>(&om[lo * kOmPitch + 32 * hi + 4 * k]);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, rb[k].x, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, rb[k].y, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, rb[k].z, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, rb[k].w, d, 0, 0, 0);
  }
  float res[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) res[i] = d[i];
#pragma unroll
  for (int i = 0; i < 4; ++i) store(i, res[i]);
}

}  // namespace

hipError_t launch_decode_split(const uint8_t* pages, int Hkv, int B, int Hq,
                               const int32_t* block_table, int max_pages,
                               const int32_t* seq_lens, int num_splits, const float* qt,
                               float* part_o, float* part_ml, hipStream_t st, int meta_bf16,
                               int ng, const MixedSpec* mixed) {
  // (with more splits the grid does not grow with the sequences)
  return by_seqs(B, num_splits == 1 ? launch_seqs(Hq) : B, [&](int b0, int nb) {
    const size_t row = (size_t)b0 * Hq, part = row * (mixed ? mixed->row_stride : num_splits);
    return launch_decode_split_mfma(pages, Hkv, nb, Hq, block_table + (size_t)b0 * max_pages, max_pages,
                                    seq_lens + b0, num_splits, device_cus(), qt + row * kD,
                                    part_o + part * kD, part_ml + part * 2, st, meta_bf16, ng, mixed);
  });
}

hipError_t launch_decode_reduce(int B, int Hq, int num_splits, const float* part_o,
                                const float* part_ml, const float* Rv, void* out, int out_f32,
                                hipStream_t st, const MixedSpec* mixed, int rph, int Hkv) {
  if (const int most = launch_seqs(Hq); B > most)
    return by_seqs(B, most, [&](int b0, int nb) {
      const size_t row = (size_t)b0 * Hq, part = row * (mixed ? num_splits + 1 : num_splits);
      return launch_decode_reduce(nb, Hq, num_splits, part_o + part * kD, part_ml + part * 2, Rv,
                                  static_cast<char*>(out) + row * kD * (out_f32 ? 4 : 2), out_f32, st,
                                  mixed, rph, Hkv);
    });
  const int rows = B * Hq;
  // As many rows per block as leave a block for every CU, or every other one.  1024 rows
  // (128 blocks of 8): 7.0 us, 8.0 with 17 slots; 256 blocks of 4: 7.2 to 7.6 and 7.7,
  // and the split kernel of the next call is slower after them (16 sequences x 4096
  // tokens, 64/8 heads: 21.6 us, 20.0 after the 128).
  const int cus = device_cus();
  const int rb = rows >= 16 * cus ? 16 : rows >= 4 * cus ? 8 : rows >= 2 * cus ? 4 : 2;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(query_blocks(B, Hq, Hkv, rph, rb)), dim3(kRedThreads), 0, st, rows,
                       num_splits, part_o, part_ml, Rv, out, out_f32, rph, Hq, Hkv);
  };
  auto by_rows = [&](auto mixed_c) {
    constexpr bool M = decltype(mixed_c)::value;
    if (rb == 16) go(reduce_kernel<M, 16>);
    else if (rb == 8) go(reduce_kernel<M, 8>);
    else if (rb == 4) go(reduce_kernel<M, 4>);
    else go(reduce_kernel<M, 2>);
  };
  if (mixed) by_rows(std::true_type{});
  else by_rows(std::false_type{});
  return hipGetLastError();
}

}  // namespace oscar
