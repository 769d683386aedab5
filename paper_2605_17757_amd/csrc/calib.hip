// Offline calibration of the rotations (Sec. 3 "Algorithm Design: Offline
// Calibration and Justification"; App. "Hadamard transform" and "P_K"; Alg. 1
// Calibrate), on the GPU:
//
//   C_Q = (1/Hkv) sum_h (1/(T g)) sum_{i in group h} sum_t q_{t,i}^T q_{t,i}
//                                   -> gram_kernel + gram_reduce_kernel
//   O   = softmax_row(Q K^T / sqrt(d) + M) V per query head   -> attn_kernel
//   C_S = the same GQA average of o^T o (= V^T S^T S V / N)   -> gram kernels on O
//   C   = U diag(lam) U^T, lam descending, each eigenvector's largest-magnitude
//         entry positive                                      -> jacobi_kernel,
//                                                                jacobi_vectors_kernel,
//                                                                eig_finish_kernel
//   R   = U H_Had P_br                                         -> compose_kernel
//
// Equal group sizes make the GQA average the plain mean over all T * Hq rows.
//
// This file is compiled with -ffp-contract=off: the composition's sums are
// separate IEEE multiplies and adds in ascending order, so that for a given U the
// rotation is the same bit pattern as the plain definition evaluated in fp64.
#include <math.h>

#include "internal.h"

namespace oscar {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Second-moment matrix X^T X of rows X [n][128] (bf16 or fp32) on fp32 MFMAs.
// A block stages 64 rows at a time in LDS as fp32 and accumulates the 10 upper
// 32x32 tiles of the 128x128 result (2 per wave, 5 waves) with
// v_mfma_f32_32x32x2_f32: per step the two rows 2s + h (h = lane / 32) feed
// lane l as A[i = l % 32][k = h] = x[32 ti + i] and B[k = h][j = l % 32] = x[32 tj + j].
// Products of bf16 inputs are exact in fp32; the block's fp32 partial tiles are
// summed in fp64, in block order, by gram_reduce_kernel.
// ---------------------------------------------------------------------------
constexpr int kGramRows = 64;
constexpr int kGramWaves = 5;
constexpr int kGramTiles = 10;
constexpr int kGramPitch = kD + 32;  // floats: rows 2s and 2s + 1 use different bank halves

__device__ inline void gram_tile(int t, int& ti, int& tj) {
  // (0,0) (0,1) (0,2) (0,3) (1,1) (1,2) (1,3) (2,2) (2,3) (3,3)
  ti = t < 4 ? 0 : t < 7 ? 1 : t < 9 ? 2 : 3;
  const int first = ti == 0 ? 0 : ti == 1 ? 4 : ti == 2 ? 7 : 9;
  tj = ti + (t - first);
}

// Row r of X is at element (r / rpt) * tok_stride + (r % rpt) * 128: rpt
// consecutive rows per token (one KV head's query heads), tokens tok_stride apart.
__device__ inline int64_t gram_row(int64_t r, int64_t rpt, int64_t tok_stride) {
  return (r / rpt) * tok_stride + (r % rpt) * kD;
}

template <bool BF16>
__global__ __launch_bounds__(kGramWaves * 64) void gram_kernel(const void* __restrict__ X,
                                                              int64_t n_rows,
                                                              int64_t rows_per_block,
                                                              int64_t rpt, int64_t tok_stride,
                                                              float* __restrict__ partial) {
  __shared__ float xs[kGramRows * kGramPitch];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, h = l >> 5, li = l & 31;
  int ti0, tj0, ti1, tj1;
  gram_tile(2 * w, ti0, tj0);
  gram_tile(2 * w + 1, ti1, tj1);
  f32x16 acc0 = {}, acc1 = {};
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = min(n_rows, r0 + rows_per_block);
  for (int64_t base = r0; base < r1; base += kGramRows) {
    __syncthreads();
    if (BF16) {  // 64 rows x 16 pieces of 8 bf16
      const uint16_t* x = static_cast<const uint16_t*>(X);
      for (int idx = tid; idx < kGramRows * 16; idx += kGramWaves * 64) {
        const int row = idx >> 4, c8 = idx & 15;
        uint4 u = make_uint4(0, 0, 0, 0);
        if (base + row < r1)
          u = *reinterpret_cast<const uint4*>(x + gram_row(base + row, rpt, tok_stride) + c8 * 8);
        float* dst = xs + row * kGramPitch + c8 * 8;
        const uint32_t wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dst[2 * e] = __uint_as_float(wd[e] << 16);
          dst[2 * e + 1] = __uint_as_float(wd[e] & 0xffff0000u);
        }
      }
    } else {  // 64 rows x 32 float4
      const float* x = static_cast<const float*>(X);
      for (int idx = tid; idx < kGramRows * 32; idx += kGramWaves * 64) {
        const int row = idx >> 5, c4 = idx & 31;
        float4 f = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (base + row < r1)
          f = *reinterpret_cast<const float4*>(x + gram_row(base + row, rpt, tok_stride) + c4 * 4);
        *reinterpret_cast<float4*>(xs + row * kGramPitch + c4 * 4) = f;
      }
    }
    __syncthreads();
#pragma unroll 4
    for (int s = 0; s < kGramRows / 2; ++s) {
      const float* rp = xs + (2 * s + h) * kGramPitch + li;
      const float a0 = rp[32 * ti0], b0 = rp[32 * tj0];
      const float a1 = rp[32 * ti1], b1 = rp[32 * tj1];
      acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc1, 0, 0, 0);
    }
  }
  // result element of register r: row 8 (r / 4) + 4 h + r % 4, column l % 32
  float* p0 = partial + ((size_t)blockIdx.x * kGramTiles + 2 * w) * 1024;
  float* p1 = p0 + 1024;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * h + (r & 3);
    p0[i * 32 + li] = acc0[r];
    p1[i * 32 + li] = acc1[r];
  }
}

// C[i][j] = C[j][i] = (sum over the blocks' partial tiles, in fp64) * inv_n.  A
// block takes 32 elements; thread (element e, part p) adds blocks p, p + 8, ...
// in order, then part 0 adds the 8 sums in order (a fixed order: deterministic).
constexpr int kRedParts = 8;

__global__ __launch_bounds__(256) void gram_reduce_kernel(const float* __restrict__ partial,
                                                          int n_blocks, double inv_n,
                                                          double* __restrict__ C) {
  __shared__ double sums[kRedParts][32];
  const int el = threadIdx.x & 31, part = threadIdx.x >> 5;
  const int e = blockIdx.x * 32 + el;  // tile * 1024 + element
  double acc = 0.0;
#pragma unroll 16
  for (int b = part; b < n_blocks; b += kRedParts)
    acc += (double)partial[((size_t)b * kGramTiles) * 1024 + e];
  sums[part][el] = acc;
  __syncthreads();
  if (part != 0) return;
  double tot = 0.0;
#pragma unroll
  for (int p = 0; p < kRedParts; ++p) tot += sums[p][el];
  const int t = e >> 10, ij = e & 1023;
  int ti, tj;
  gram_tile(t, ti, tj);
  const int i = 32 * ti + (ij >> 5), j = 32 * tj + (ij & 31);
  const double c = tot * inv_n;
  C[i * kD + j] = c;
  C[j * kD + i] = c;
}

// ---------------------------------------------------------------------------
// Calibration attention, O = softmax_row(Q K^T / sqrt(d) + M) V, M causal or 0.
// A block of kCalibAttnWaves (8) waves covers one KV head's key/value tiles for hc
// of its query heads and 32 * 8 / hc queries; wave w takes head (w % hc) and 32
// queries (blocks of 4 waves, two per CU, measured 1.34x slower: each K/V tile then
// serves half as many waves; a double-buffered version that issues the next tile's
// score MFMAs before the current tile's softmax needs more than 256 registers per
// lane and spills: 1.16x slower; K and V tiles in two LDS buffers, with one barrier
// per tile instead of two: 2 % faster (0.5 % of a layer's calibration), not kept).  Bound: the matrix
// cores, 48 MFMAs per wave and tile: 0.97 ms at 8878 tokens x 32 heads, 1.0 PFLOP/s of
// products, P's two parts among them, where a large bf16 product reaches 1.2.
// Per 64-key tile the wave computes S^T = K Q^T (v_mfma_f32_32x32x16_bf16,
// A = K rows from LDS, B = the wave's queries held in registers), so that a lane
// owns one query and 32 of the tile's keys: the row maximum is a lane maximum and
// one cross-half exchange.  Those scores, exponentiated, are already the B
// operand of O^T += V^T P^T, the key order inside an MFMA step being free as long
// as A and B agree; V^T comes from LDS (staged transposed).  P enters the bf16
// MFMA as a sum of two bf16 parts, p = hi + lo (16 significant bits), so that
// the product with the bf16 values is kept to ~2^-17 relative; Q K^T of bf16
// inputs is exact up to the fp32 accumulation.  Online softmax in base 2; the
// running maximum is raised (and O^T, l rescaled) only when a tile's maximum
// exceeds it by more than 8, the result being the same up to rounding; O^T is kept
// in the accumulators and normalized at the end.
// ---------------------------------------------------------------------------
constexpr int kAttnWaves = kCalibAttnWaves;
constexpr int kKPitch = kD + 8;  // bf16: 272-byte K rows (conflict-free 16-byte reads)
constexpr int kVPitch = 64 + 4;  // bf16: 136-byte V^T rows (conflict-free 8-byte reads)

__global__ __launch_bounds__(kAttnWaves * 64) void attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    int T, int Hq, int Hkv, int hc, int causal, float scale_log2, int n_qtiles,
    float* __restrict__ out) {
  __shared__ __align__(16) uint16_t Ks[64 * kKPitch];
  __shared__ __align__(16) uint16_t Vt[kD * kVPitch];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, h = l >> 5, li = l & 31;
  const int g = Hq / Hkv;
  const int span = 32 * (kAttnWaves / hc);
  const int qt = n_qtiles - 1 - (int)blockIdx.y;  // longest causal rows first
  const int head = blockIdx.x * hc + (w % hc);
  const int kvh = (blockIdx.x * hc) / g;
  const int qw0 = qt * span + 32 * (w / hc);
  const int qblock_last = min(T - 1, qt * span + span - 1);
  const int n_kt = causal ? qblock_last / 64 + 1 : (T + 63) / 64;
  const bool active = qw0 < T;
  const int wave_kt = causal ? min(T - 1, qw0 + 31) / 64 + 1 : n_kt;
  const int qrow = qw0 + li;

  // the wave's queries: lane l holds q[qrow][16 ks + 8 h + 0..7], ks = 0..7
  bf16x8 qf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
    uint4 u = make_uint4(0, 0, 0, 0);
    if (qrow < T) u = *reinterpret_cast<const uint4*>(q + ((size_t)qrow * Hq + head) * kD + 16 * ks + 8 * h);
    qf[ks] = __builtin_bit_cast(bf16x8, u);
  }

  f32x16 o[4] = {};
  float m = -INFINITY, lsum = 0.0f;

  // tile staging: K as 16-byte pieces (64 rows x 16) spread over the threads; V as
  // items (key pair kp: keys 2 kp, 2 kp + 1; dims 8 dq .. 8 dq + 7), written
  // transposed (key pairs per dword)
  constexpr int kNT = kAttnWaves * 64;
  constexpr int kKPer = 1024 / kNT, kVPer = 512 / kNT;
  uint4 kr[kKPer], vr[kVPer][2];
  auto load_tile = [&](int kt) {
#pragma unroll
    for (int i = 0; i < kKPer; ++i) {
      const int idx = tid + kNT * i, row = idx >> 4, c8 = idx & 15;
      const int key = 64 * kt + row;
      kr[i] = key < T ? *reinterpret_cast<const uint4*>(k + ((size_t)key * Hkv + kvh) * kD + c8 * 8)
                      : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < kVPer; ++j) {
      const int item = tid + kNT * j, kp = item & 31, dq = item >> 5;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int vkey = 64 * kt + 2 * kp + e;
        vr[j][e] = vkey < T ? *reinterpret_cast<const uint4*>(v + ((size_t)vkey * Hkv + kvh) * kD + dq * 8)
                            : make_uint4(0, 0, 0, 0);
      }
    }
  };
  load_tile(0);

  for (int kt = 0; kt < n_kt; ++kt) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kKPer; ++i) {
      const int idx = tid + kNT * i, row = idx >> 4, c8 = idx & 15;
      *reinterpret_cast<uint4*>(Ks + row * kKPitch + c8 * 8) = kr[i];
    }
#pragma unroll
    for (int j = 0; j < kVPer; ++j) {
      const int item = tid + kNT * j, kp = item & 31, dq = item >> 5;
      const uint32_t a[4] = {vr[j][0].x, vr[j][0].y, vr[j][0].z, vr[j][0].w};
      const uint32_t b[4] = {vr[j][1].x, vr[j][1].y, vr[j][1].z, vr[j][1].w};
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const uint32_t word = __builtin_amdgcn_perm(b[c >> 1], a[c >> 1], (c & 1) ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<uint32_t*>(Vt + (8 * dq + c) * kVPitch + 2 * kp) = word;
      }
    }
    __syncthreads();
    if (kt + 1 < n_kt) load_tile(kt + 1);
    if (!active || kt >= wave_kt) continue;

    // issue priority: high while a wave feeds the matrix cores, low in its softmax,
    // so that a SIMD's other wave fills the gaps
    __builtin_amdgcn_s_setprio(1);
    // S^T: lane holds query qrow, keys 64 kt + 32 kk + 8 (r / 4) + 4 h + r % 4
    // the two 32-key halves as two interleaved MFMA chains; each step's K pieces
    // are read from LDS one step ahead
    f32x16 s[2] = {};
    const uint16_t* kb = Ks + li * kKPitch + 8 * h;
    uint4 ka0 = *reinterpret_cast<const uint4*>(kb);
    uint4 ka1 = *reinterpret_cast<const uint4*>(kb + 32 * kKPitch);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      uint4 kn0 = ka0, kn1 = ka1;
      if (ks + 1 < 8) {
        kn0 = *reinterpret_cast<const uint4*>(kb + 16 * (ks + 1));
        kn1 = *reinterpret_cast<const uint4*>(kb + 32 * kKPitch + 16 * (ks + 1));
      }
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka0), qf[ks], s[0], 0, 0, 0);
      s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka1), qf[ks], s[1], 0, 0, 0);
      ka0 = kn0;
      ka1 = kn1;
    }
    // keep the LDS reads one step ahead of the MFMAs that consume them
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int ks = 0; ks < 7; ++ks) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      if (ks < 6) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_s_setprio(0);
    const bool edge = (causal && 64 * kt + 63 > qw0) || 64 * kt + 64 > T;
    float mt = -INFINITY;
    if (edge) {  // keys >= limit are masked
      const int limit = causal ? min(T, qrow + 1) : T;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = 64 * kt + 32 * kk + 8 * (r >> 2) + 4 * h + (r & 3);
          s[kk][r] = key < limit ? s[kk][r] : -INFINITY;
        }
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int r = 0; r < 16; ++r) mt = fmaxf(mt, s[kk][r]);
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64)) * scale_log2;  // finite: key 0 is visible to every query
    // The running maximum m (base-2 units) is raised only when a score exceeds it
    // by more than 8, so most tiles skip the rescale; probabilities stay <= 2^8.
    if (__ballot(mt > m + 8.0f)) {
      const float m_new = fmaxf(m, mt);
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    __builtin_amdgcn_s_setprio(1);
    float tsum = 0.0f;  // the tile's probabilities, added to the running sum once
    // V^T pieces for step (kk, u): dims 32 dt + l % 32, keys 32 kk + 16 u + 4 h + 0..3
    // and + 8; read one step ahead
    auto vload = [&](int kk, int u, uint4 (&va)[4]) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const uint16_t* vp = Vt + (32 * dt + li) * kVPitch + 32 * kk + 16 * u + 4 * h;
        const uint2 v0 = *reinterpret_cast<const uint2*>(vp);
        const uint2 v1 = *reinterpret_cast<const uint2*>(vp + 8);
        va[dt] = make_uint4(v0.x, v0.y, v1.x, v1.y);
      }
    };
    uint4 vcur[4], vnext[4];
    vload(0, 0, vcur);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int step = 2 * kk + u;
        if (step + 1 < 4) vload((step + 1) >> 1, (step + 1) & 1, vnext);
        uint32_t hw[4], lw[4];
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kk][8 * u + 2 * t2], scale_log2, -m));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kk][8 * u + 2 * t2 + 1], scale_log2, -m));
          tsum += p0;
          tsum += p1;
          const bf16x2 hb = {(__bf16)p0, (__bf16)p1};
          hw[t2] = __builtin_bit_cast(uint32_t, hb);
          const bf16x2 lb = {(__bf16)(p0 - __uint_as_float(hw[t2] << 16)),
                             (__bf16)(p1 - __uint_as_float(hw[t2] & 0xffff0000u))};
          lw[t2] = __builtin_bit_cast(uint32_t, lb);
        }
        const bf16x8 phi = __builtin_bit_cast(bf16x8, make_uint4(hw[0], hw[1], hw[2], hw[3]));
        const bf16x8 plo = __builtin_bit_cast(bf16x8, make_uint4(lw[0], lw[1], lw[2], lw[3]));
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vcur[dt]), phi, o[dt], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vcur[dt]), plo, o[dt], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) vcur[dt] = vnext[dt];
      }
    lsum += tsum;
    __builtin_amdgcn_s_setprio(0);
  }

  if (!active || qrow >= T) return;
  const float ltot = lsum + __shfl_xor(lsum, 32, 64);
  const float inv = 1.0f / ltot;
  float* orow = out + ((size_t)qrow * Hq + head) * kD;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int dim = 32 * dt + 8 * r4 + 4 * h;
      *reinterpret_cast<float4*>(orow + dim) =
          make_float4(o[dt][4 * r4] * inv, o[dt][4 * r4 + 1] * inv, o[dt][4 * r4 + 2] * inv,
                      o[dt][4 * r4 + 3] * inv);
    }
}

// ---------------------------------------------------------------------------
// Symmetric eigen-decomposition by cyclic Jacobi (round-robin ordering), fp64.
// A sweep is 127 rounds of 64 disjoint pairs (circle method: in round r pair 0 is
// (127, r) and pair k is (a, b) = ((r + k) mod 127, (r - k) mod 127), k = 1..63), so
// every off-diagonal entry is visited once per sweep.  For each pair, p = min(a, b),
// q = max(a, b), the rotation J (J_pp = J_qq = c, J_pq = s, J_qp = -s) with
// tau = (a_qq - a_pp) / (2 a_pq), t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
// c = 1 / sqrt(1 + t^2), s = t c zeroes a_pq (Golub and Van Loan, symmetric Schur
// decomposition); the round applies A <- J^T A J as independent 2x2 block updates.
// A pair is skipped when |a_pq| <= 1e-15 sqrt(|a_pp a_qq|); the sweeps stop when a
// sweep skips every pair (info = sweeps run, or -1 if max_sweeps did not converge).
//
// One block of 16 waves per matrix.  The rounds are a dependent chain (some 1,800 of
// them), so a round has to be short; the matrix is kept in pair space to that end:
// block (k1, k2), k1 < k2, holds the entries of pairs k1 and k2 of the current
// round, and from one round to the next the indices move by one pair,
//   a'_0 = a_0, a'_k = a_(k+1) (k = 1..62), a'_63 = b_63,
//   b'_0 = a_1, b'_k = b_(k-1) (k = 1..63),
// the same in every round.  So a thread's blocks read their four entries from four
// fixed places of the last round's buffer and write them to one of the other buffer
// (one barrier per round, each entry read and written once, no index arithmetic).  Lane k of wave 0 holds pair k's diagonal block, takes the block
// whose entries become the pair's next off-diagonal entry, and forms the next
// round's rotation while the other waves update.  Its 64 blocks are those whose
// entry comes from within a pair, which therefore never leaves the lane.
// Rotations are kept as (c, s~), s~ = s if a < b, -s otherwise: a' = c a - s~ b and
// b' = s~ a + c b are then the two rows of J^T, in either order.  They are recorded
// for jacobi_vectors_kernel.  Bound: the chain of a round, 0.95 us of LDS accesses and
// fp64 VALU work of 16 waves (1,250 and 340 instructions; VALU 48 % busy on the block's
// CU, 40 % of the waves' time at waits and the barrier); 1700 us for two matrices of 14
// and 10 sweeps (the whole matrix in index order, with the rotations formed between two
// barriers: 2.0 us a round, 3593 us).
// ---------------------------------------------------------------------------
constexpr int kJacRounds = kD - 1;
constexpr int kJacPairs = kD / 2;
constexpr int kJacWaves = 16;
constexpr int kJacThreads = kJacWaves * 64;
// A buffer holds the blocks in 32 rows of 64 (padded: fewer bank conflicts), block
// rows k1 and 62 - k1 (63 - k1 and k1 + 1 blocks) end to end, so that a wave takes a
// row and most of its accesses are consecutive; element (t1, t2) in plane 2 t1 + t2.
constexpr int kJacRows = kJacPairs / 2;
constexpr int kJacPitch = kJacPairs + 1;
constexpr int kJacPlane = kJacRows * kJacPitch;
constexpr int kJacPerThread = (kJacRows + kJacWaves - 2) / (kJacWaves - 1);  // of the waves other than wave 0
constexpr double kJacTol = 1e-15;

// Indices of pair k in round 0.
__device__ inline int jac_a(int k) { return k == 0 ? kD - 1 : k; }
__device__ inline int jac_b(int k) { return k == 0 ? 0 : kJacRounds - k; }
// Place of element (t1, t2) (0: a, 1: b) of pairs k1 != k2 in a buffer.
__device__ inline int jac_place(int k1, int t1, int k2, int t2) {
  if (k1 > k2) {
    const int k = k1, t = t1;
    k1 = k2;
    t1 = t2;
    k2 = k;
    t2 = t;
  }
  const int row = min(k1, kJacPairs - 2 - k1), col = k1 < kJacRows ? k2 - k1 - 1 : k2;
  return (2 * t1 + t2) * kJacPlane + row * kJacPitch + col;
}
// Pair and side that index t of pair k had one round before.
__device__ inline void jac_from(int k, int t, int& kf, int& tf) {
  if (t == 0) {
    kf = k == 0 ? 0 : k == kJacPairs - 1 ? k : k + 1;
    tf = k == kJacPairs - 1 ? 1 : 0;
  } else {
    kf = k == 0 ? 1 : k - 1;
    tf = k == 0 ? 0 : 1;
  }
}
// Block at lane l of a row, if it is one of the waves other than wave 0 (which takes
// (0, 1), (62, 63) and those with k2 = k1 + 2).
__device__ inline bool jac_block(int row, int l, int& k1, int& k2) {
  k1 = l < kJacPairs - 1 - row ? row : kJacPairs - 2 - row;
  k2 = k1 == row ? row + 1 + l : l;
  if (row == kJacRows - 1 && l >= kJacRows) return false;  // the middle row is half a row
  return k2 != k1 + 2 && !(k1 == 0 && k2 == 1) && k1 != kJacPairs - 2;
}

// Rotation of a pair with diagonal entries daa, dbb and off-diagonal entry dab: (c,
// s~); any: whether it is one (not skipped).
__device__ inline double2 jac_rotation(double daa, double dbb, double dab, bool a_first, bool& any) {
  const double app = a_first ? daa : dbb, aqq = a_first ? dbb : daa;
  double c = 1.0, s = 0.0;
  any = dab != 0.0 && fabs(dab) > kJacTol * sqrt(fabs(app * aqq));
  if (any) {
    const double tau = (aqq - app) / (2.0 * dab);
    const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
    c = 1.0 / sqrt(1.0 + t * t);
    s = t * c;
  }
  return make_double2(c, a_first ? s : -s);
}

// Entries (aa, ab, ba, bb) of a block under the rotations of its two pairs.
__device__ inline void jac_update(double (&m)[4], double2 r1, double2 r2) {
  const double t00 = r1.x * m[0] - r1.y * m[2], t01 = r1.x * m[1] - r1.y * m[3];
  const double t10 = r1.y * m[0] + r1.x * m[2], t11 = r1.y * m[1] + r1.x * m[3];
  m[0] = t00 * r2.x - t01 * r2.y;
  m[1] = t00 * r2.y + t01 * r2.x;
  m[2] = t10 * r2.x - t11 * r2.y;
  m[3] = t10 * r2.y + t11 * r2.x;
}

// Lane i's value of lane i + 1 (UP) or i - 1; `edge` in the lane that has none.
template <bool UP>
__device__ inline double lane_shift(double edge, double v) {
  constexpr int kCtrl = UP ? 0x130 : 0x138;  // wave_shl:1, wave_shr:1
  const uint64_t e = (uint64_t)__double_as_longlong(edge), u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)e, (int)(uint32_t)u, kCtrl, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(e >> 32), (int)(uint32_t)(u >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// One round's move of values held per pair (a, b in lane k).
__device__ inline void jac_move(double& a, double& b, int l) {
  const double up = lane_shift<true>(b, a);  // a_(k+1); lane 63: b_63
  b = lane_shift<false>(up, b);              // b_(k-1); lane 0: a_1
  a = l == 0 ? a : up;
}

struct JacSmem {
  double buf[2][4 * kJacPlane];  // 130 KB
  double2 cs[2][kJacPairs];      // by round parity
  int rotated[2];                // by sweep parity
};

// A thread's block: pairs k1 < k2, its place in a buffer and those of its entries
// one round before.
struct JacBlock {
  int k1, k2, own, from[4];
};
// The places of block (k1, k2), and its entries of round 0 into them; returns the
// entry that comes from within a pair (at most one), or -1, and its value in v.
__device__ inline int jac_place_block(JacBlock& blk, double* buf, const double* __restrict__ Cm,
                                      int k1, int k2, double& v) {
  auto index = [](int k, int t) { return t == 0 ? jac_a(k) : jac_b(k); };
  int inner = -1;
  blk.k1 = k1;
  blk.k2 = k2;
  blk.own = jac_place(k1, 0, k2, 0);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int ka, ta, kb, tb;
    jac_from(k1, e >> 1, ka, ta);
    jac_from(k2, e & 1, kb, tb);
    const double x = Cm[index(k1, e >> 1) * kD + index(k2, e & 1)];
    if (ka == kb) {
      inner = e;
      v = x;
      blk.from[e] = 0;
    } else {
      blk.from[e] = jac_place(ka, ta, kb, tb);
      buf[blk.from[e]] = x;
    }
  }
  return inner;
}

// Wave 0: the pairs' diagonal blocks (lane l: pair l), the rotations, and the block
// that holds the pair's next off-diagonal entry.
__device__ inline void jac_lead(JacSmem& sm, const double* __restrict__ Cm, int max_sweeps,
                                double2* __restrict__ rm, double* __restrict__ diag,
                                int* __restrict__ n_rounds, int* __restrict__ info) {
  __builtin_amdgcn_s_setprio(3);  // the round waits for this wave
  const int l = threadIdx.x;
  JacBlock blk;
  double dab_old = 0.0;
  const int inner = jac_place_block(blk, sm.buf[0], Cm, l == 0 ? 0 : l - 1,
                                    l == 0 ? 1 : l == kJacPairs - 1 ? l : l + 1, dab_old);
  const int ia = jac_a(l), ib = jac_b(l);
  double daa = Cm[ia * kD + ia], dbb = Cm[ib * kD + ib], dab = Cm[ia * kD + ib];
  bool any, af = ia < ib;  // any rotation in the sweep so far; a < b in this round
  double2 mine = jac_rotation(daa, dbb, dab, af, any);
  sm.cs[0][l] = mine;
  rm[l] = mine;
  rm += kJacPairs;
  __syncthreads();
  int sweeps = 0, converged = 0, cur = 0;
  for (int sw = 0; sw < max_sweeps; ++sw) {
    for (int r = 0; r < kJacRounds; ++r, cur ^= 1) {
      const double* src = sm.buf[cur];
      double m[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = src[blk.from[e]];
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = e == inner ? dab_old : m[e];
      // rotations of pairs l - 1 (lane 0: 0) and l + 1 (lane 63: 63), the block's two
      const double2 r1 = make_double2(lane_shift<false>(mine.x, mine.x), lane_shift<false>(mine.y, mine.y));
      const double2 r2 = make_double2(lane_shift<true>(mine.x, mine.x), lane_shift<true>(mine.y, mine.y));
      jac_update(m, r1, r2);
      if (mine.y != 0.0) {  // the pair's own block; its off-diagonal entry is zero by construction
        const double app = af ? daa : dbb, aqq = af ? dbb : daa, c = mine.x, s = af ? mine.y : -mine.y;
        const double t00 = c * app - s * dab, t01 = c * dab - s * aqq;
        const double t10 = s * app + c * dab, t11 = s * dab + c * aqq;
        const double npp = t00 * c - t01 * s, nqq = t10 * s + t11 * c;
        daa = af ? npp : nqq;
        dbb = af ? nqq : npp;
        dab = 0.0;
      }
      dab_old = dab;
      dab = l == 0 ? m[0] : l == kJacPairs - 1 ? m[3] : m[2];
      jac_move(daa, dbb, l);
      const bool last = r == kJacRounds - 1;
      if (last) {
        const bool sweep_any = __any(any);
        if (l == 0) sm.rotated[sw & 1] = sweep_any;
        any = false;
      }
      const int rn = last ? 0 : r + 1;
      const int a = rn + l, b = rn - l;
      af = l != 0 && (a >= kJacRounds ? a - kJacRounds : a) < (b < 0 ? b + kJacRounds : b);
      bool now;
      mine = jac_rotation(daa, dbb, dab, af, now);
      any |= now;
      sm.cs[cur ^ 1][l] = mine;
      if (!last || sw + 1 < max_sweeps) rm[l] = mine;
      rm += kJacPairs;
      double* dst = sm.buf[cur ^ 1] + blk.own;
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[e * kJacPlane] = m[e];
      __syncthreads();
    }
    if (!sm.rotated[sw & 1]) {  // a sweep without rotations: converged (its identity rounds are not kept)
      converged = 1;
      break;
    }
    sweeps = sw + 1;
  }
  diag[ia] = daa;  // the pairs are back at round 0
  diag[ib] = dbb;
  if (l == 0) {
    *n_rounds = sweeps * kJacRounds;
    *info = converged ? sweeps + 1 : -1;
  }
}

// The other waves: the other blocks, two or three per thread.
__device__ inline void jac_follow(JacSmem& sm, const double* __restrict__ Cm, int max_sweeps) {
  JacBlock blk[kJacPerThread];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
#pragma unroll
  for (int n = 0; n < kJacPerThread; ++n) {
    const int row = w - 1 + (kJacWaves - 1) * n;
    int k1, k2;
    double none;
    blk[n].k1 = -1;
    if (row < kJacRows && jac_block(row, l, k1, k2))
      jac_place_block(blk[n], sm.buf[0], Cm, k1, k2, none);
  }
  __syncthreads();
  int cur = 0;
  for (int sw = 0; sw < max_sweeps; ++sw) {
    for (int r = 0; r < kJacRounds; ++r, cur ^= 1) {
      const double* src = sm.buf[cur];
#pragma unroll
      for (int n = 0; n < kJacPerThread; ++n) {
        if (blk[n].k1 < 0) continue;
        double m[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = src[blk[n].from[e]];
        jac_update(m, sm.cs[cur][blk[n].k1], sm.cs[cur][blk[n].k2]);
        double* dst = sm.buf[cur ^ 1] + blk[n].own;
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e * kJacPlane] = m[e];
      }
      __syncthreads();
    }
    if (!sm.rotated[sw & 1]) break;
  }
}

__global__ __launch_bounds__(kJacThreads) void jacobi_kernel(const double* __restrict__ C, int max_sweeps,
                                                     double* __restrict__ diag,
                                                     double2* __restrict__ rot,
                                                     int* __restrict__ n_rounds,
                                                     int* __restrict__ info) {
  __shared__ JacSmem sm;
  const int mtx = blockIdx.x;
  const double* Cm = C + (size_t)mtx * kD * kD;
  // both sides run the same barriers: one at the start and one per round
  if (__builtin_amdgcn_readfirstlane(threadIdx.x) < 64)
    jac_lead(sm, Cm, max_sweeps, rot + (size_t)mtx * max_sweeps * kJacRounds * kJacPairs,
             diag + (size_t)mtx * kD, n_rounds + mtx, info + mtx);
  else
    jac_follow(sm, Cm, max_sweeps);
}

// V = J_1 J_2 ... J_R: each row of V evolves on its own (v <- v J), so one wave
// per row applies the recorded rounds in registers: lane k holds the row's entries
// of pair k, which move between lanes as in jacobi_kernel.  The rounds' (c, s~) are
// loaded 16 rounds ahead.  Bound: the dependent chain of a round, 56 ns (two
// matrices, 14 sweeps: 99 us; 300 us with the row in LDS, indexed).
constexpr int kVecWaves = 4;
constexpr int kVecAhead = 16;

__global__ __launch_bounds__(kVecWaves * 64) void jacobi_vectors_kernel(
    const double2* __restrict__ rot, const int* __restrict__ n_rounds, int max_sweeps,
    int n_mats, double* __restrict__ V) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int grow = blockIdx.x * kVecWaves + w;  // matrix * 128 + row
  if (grow >= n_mats * kD) return;            // whole wave
  const int mtx = grow / kD, row = grow % kD;
  double a = jac_a(l) == row ? 1.0 : 0.0, b = jac_b(l) == row ? 1.0 : 0.0;
  const int R = __builtin_amdgcn_readfirstlane(n_rounds[mtx]);  // whole sweeps: the pairs end as they begin
  const double2* rm = rot + (size_t)mtx * max_sweeps * kJacRounds * kJacPairs + l;
  auto turn = [&](double2 c) {
    const double na = c.x * a - c.y * b;
    b = c.y * a + c.x * b;
    a = na;
    jac_move(a, b, l);
  };
  // whole groups of rounds without branches (the loads past the end repeat the last
  // round's), so that no wait drains the loads ahead
  const int whole = R / kVecAhead * kVecAhead;
  if (whole > 0) {
    double2 buf[kVecAhead];
#pragma unroll
    for (int i = 0; i < kVecAhead; ++i) buf[i] = rm[(size_t)i * kJacPairs];
    for (int t0 = 0; t0 < whole; t0 += kVecAhead) {
#pragma unroll
      for (int i = 0; i < kVecAhead; ++i) {
        const double2 c = buf[i];
        buf[i] = rm[(size_t)min(t0 + kVecAhead + i, R - 1) * kJacPairs];
        turn(c);
      }
    }
  }
  for (int t = whole; t < R; ++t) turn(rm[(size_t)t * kJacPairs]);
  double* vo = V + ((size_t)mtx * kD + row) * kD;
  vo[jac_a(l)] = a;
  vo[jac_b(l)] = b;
}

// Sort the eigenpairs by descending eigenvalue (ties: lower index first) and fix
// each eigenvector's sign so that its largest-magnitude entry (the first such)
// is positive.  One block of 1024 threads per matrix; thread (column i, part p) looks
// for the largest of the column's rows 16p .. 16p + 15 (loads issued together) and
// moves them.  (One thread per column, row after row: 25 us; latency only.)
constexpr int kFinParts = 8;

__global__ __launch_bounds__(kD * kFinParts) void eig_finish_kernel(const double* __restrict__ diag,
                                                        const double* __restrict__ V,
                                                        double* __restrict__ lam,
                                                        double* __restrict__ U) {
  constexpr int kRows = kD / kFinParts;
  __shared__ double ls[kD];
  __shared__ double top[kFinParts][kD];  // a part's largest-magnitude entry, with its sign
  const int mtx = blockIdx.x, i = threadIdx.x % kD, p = threadIdx.x / kD;
  const double* Vm = V + (size_t)mtx * kD * kD;
  double x[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) x[r] = Vm[(kRows * p + r) * kD + i];
  const double li = diag[(size_t)mtx * kD + i];
  if (p == 0) ls[i] = li;
  double best = x[0];
#pragma unroll
  for (int r = 1; r < kRows; ++r)
    if (fabs(x[r]) > fabs(best)) best = x[r];
  top[p][i] = best;
  __syncthreads();
  int rank = 0;
#pragma unroll 16
  for (int j = 0; j < kD; ++j) {
    const double lj = ls[j];
    rank += (lj > li || (lj == li && j < i)) ? 1 : 0;
  }
  if (p == 0) lam[(size_t)mtx * kD + rank] = li;
  best = top[0][i];
#pragma unroll
  for (int k = 1; k < kFinParts; ++k)
    if (fabs(top[k][i]) > fabs(best)) best = top[k][i];
  const double sgn = best < 0.0 ? -1.0 : 1.0;
  double* Um = U + (size_t)mtx * kD * kD;
#pragma unroll
  for (int r = 0; r < kRows; ++r) Um[(kRows * p + r) * kD + rank] = sgn * x[r];
}

// R = U H_Had P_br: R[i][j] = sum_c U[i][c] H[c][bitrev(j)] (P_br moves column k
// to bitrev(k); bit reversal is its own inverse), summed in ascending c with
// H[c][k] = (-1)^popcount(c & k) h, h = 1 divided by sqrt 2 seven times (the
// Sylvester recursion's normalization).  One thread per entry.
__global__ __launch_bounds__(256) void compose_kernel(const double* __restrict__ U,
                                                      double* __restrict__ R64,
                                                      float* __restrict__ R32) {
  const int mtx = blockIdx.y;
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int i = e >> 7, j = e & (kD - 1);
  const int k = (int)(__brev((unsigned)j) >> 25);  // 7-bit reversal
  double hmag = 1.0;
  for (int lev = 1; lev < kD; lev <<= 1) hmag = hmag / sqrt(2.0);
  const double* Ui = U + ((size_t)mtx * kD + i) * kD;
  double acc = 0.0;
  for (int c = 0; c < kD; ++c) {
    const double hc = (__popc((unsigned)(c & k)) & 1) ? -hmag : hmag;
    acc = acc + Ui[c] * hc;
  }
  if (R64) R64[((size_t)mtx * kD + i) * kD + j] = acc;
  if (R32) R32[((size_t)mtx * kD + i) * kD + j] = (float)acc;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

int64_t gram_blocks(int64_t n_rows) {
  int64_t nb = (n_rows + kGramRows - 1) / kGramRows;
  const int64_t cap = 2 * (int64_t)device_cus();
  return nb < 1 ? 1 : nb > cap ? cap : nb;
}

size_t gram_partial_bytes(int64_t n_rows) {
  return (size_t)gram_blocks(n_rows) * kGramTiles * 1024 * sizeof(float);
}

hipError_t launch_gram(const void* X, int x_bf16, int64_t n_rows, double inv_n, float* partial,
                       double* C, hipStream_t st, int64_t rpt, int64_t tok_stride) {
  const int64_t nb = gram_blocks(n_rows);
  int64_t per = (n_rows + nb - 1) / nb;
  per = (per + kGramRows - 1) / kGramRows * kGramRows;
  if (x_bf16)
    hipLaunchKernelGGL(gram_kernel<true>, dim3((unsigned)nb), dim3(kGramWaves * 64), 0, st, X,
                       n_rows, per, rpt, tok_stride, partial);
  else
    hipLaunchKernelGGL(gram_kernel<false>, dim3((unsigned)nb), dim3(kGramWaves * 64), 0, st, X,
                       n_rows, per, rpt, tok_stride, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(kGramTiles * 1024 / 32), dim3(256), 0, st,
                     partial, (int)nb, inv_n, C);
  return hipGetLastError();
}

hipError_t launch_calib_attn(const uint16_t* q, const uint16_t* k, const uint16_t* v, int T,
                             int Hq, int Hkv, int causal, float* out, hipStream_t st) {
  const int g = Hq / Hkv;
  const int hc = g % 4 == 0 ? 4 : g % 2 == 0 ? 2 : 1;
  const int span = 32 * (kAttnWaves / hc);
  const int n_qtiles = (T + span - 1) / span;
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)kD));
  hipLaunchKernelGGL(attn_kernel, dim3((unsigned)(Hq / hc), (unsigned)n_qtiles),
                     dim3(kAttnWaves * 64), 0, st, q, k, v, T, Hq, Hkv, hc, causal, scale_log2,
                     n_qtiles, out);
  return hipGetLastError();
}

size_t eig_rot_bytes(int n_mats, int max_sweeps) {
  return (size_t)n_mats * max_sweeps * kJacRounds * kJacPairs * sizeof(double2);
}

hipError_t launch_eig(const double* C, int n_mats, int max_sweeps, double* diag, double2* rot,
                      int* n_rounds, double* V, double* lam, double* U, int* info,
                      hipStream_t st) {
  hipLaunchKernelGGL(jacobi_kernel, dim3((unsigned)n_mats), dim3(kJacThreads), 0, st, C, max_sweeps,
                     diag, rot, n_rounds, info);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(jacobi_vectors_kernel, dim3((unsigned)((n_mats * kD + kVecWaves - 1) / kVecWaves)),
                     dim3(kVecWaves * 64), 0, st, rot, n_rounds, max_sweeps, n_mats, V);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(eig_finish_kernel, dim3((unsigned)n_mats), dim3(kD * kFinParts), 0, st, diag, V, lam, U);
  return hipGetLastError();
}

hipError_t launch_compose(const double* U, int n_mats, double* R64, float* R32, hipStream_t st) {
  hipLaunchKernelGGL(compose_kernel, dim3(kD * kD / 256, (unsigned)n_mats), dim3(256), 0, st, U,
                     R64, R32);
  return hipGetLastError();
}

}  // namespace oscar
