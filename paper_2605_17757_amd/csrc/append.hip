// Cache update: rotate -> clip -> asymmetric INT2 per 32-channel group -> pack.
// (Sec. 4 "KV Cache Update"; App. "Scale Determination and Per-token Clipping
// Details"; Alg. 1 QuantizeAndWrite.)
//
// This file is compiled with -ffp-contract=off: every fp32 step below is one
// IEEE operation (no fused multiply-add unless written).  The rotation is summed
// in fp64 in ascending channel order.  Because each product of a bf16 input and an
// fp32 matrix entry is exact in fp64, that sum is the same whether it is built of
// fused or separate operations, bit for bit.
#include <float.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "seg_partial.h"

namespace oscar {
namespace {

constexpr int kMaxClipCands = 32;  // candidate clip ratios per calibration call

__device__ inline float f16_bits_to_f32(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// binary16 with saturation to +-65504 (round to nearest even).
__device__ inline uint16_t f16_sat_bits(float f) {
  f = fminf(fmaxf(f, -65504.0f), 65504.0f);
  return __half_as_ushort(__float2half_rn(f));
}

// A zero point of zero is stored as +0.  This is done on the binary16 bits: the
// compiler may drop an "x + 0.0f" whose result only feeds fmaxf/fminf.
__device__ inline uint16_t plus_zero(uint16_t h) { return (h & 0x7fffu) ? h : (uint16_t)0; }

// bfloat16 with saturation to +-(largest finite) (round to nearest even on the
// binary32 bits; finite inputs).
__device__ inline uint16_t bf16_sat_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  uint16_t h = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  if ((h & 0x7fffu) == 0x7f80u) h = (uint16_t)((h & 0x8000u) | 0x7f7fu);
  return h;
}

using QFmt = QuantFmt;  // storage format of scale and zero, and the clip rule
__device__ inline uint16_t meta_store(const QFmt& q, float f) {
  return q.bf16 ? bf16_sat_bits(f) : f16_sat_bits(f);
}
__device__ inline float meta_load(const QFmt& q, uint16_t h) {
  return q.bf16 ? __uint_as_float((uint32_t)h << 16) : f16_bits_to_f32(h);
}

// Scale and zero point of a group with (clipped) minimum a and maximum b, as
// stored (s16, z16) and as used for the codes (sf, zf); a group whose stored
// scale is 0 stores s = 1, z = M(-a) and codes 0 (deg).
struct QParams {
  uint16_t s16, z16;
  float sf, zf;
  bool deg;
};
__device__ inline QParams quant_params(float a, float b, const QFmt& fmt) {
  QParams p;
  const float s = __fdiv_rn(__fsub_rn(b, a), 3.0f);
  p.s16 = meta_store(fmt, s);
  p.deg = (p.s16 & 0x7fffu) == 0;
  if (p.deg) {
    p.s16 = fmt.bf16 ? 0x3f80u : 0x3c00u;  // 1.0
    p.z16 = plus_zero(meta_store(fmt, -a));
    p.sf = p.zf = 0.0f;
  } else {
    p.sf = meta_load(fmt, p.s16);
    p.z16 = plus_zero(meta_store(fmt, __fdiv_rn(-a, p.sf)));
    p.zf = meta_load(fmt, p.z16);
  }
  return p;
}
// Code of one clipped channel value y: clamp(round_half_even(y / s + z), 0, 3).
__device__ inline uint32_t quant_code(float y, const QParams& p) {
  if (p.deg) return 0u;
  const float r = rintf(__fadd_rn(__fdiv_rn(y, p.sf), p.zf));
  return (uint32_t)fminf(fmaxf(r, 0.0f), 3.0f);
}

// Token-wise clip threshold (App. "Scale Determination and Per-token Clipping
// Details"): the rho-quantile of |x~| over the row, a_k + f (a_{k+1} - a_k) with
// pos = rho (d - 1), k = floor(pos), f = pos - k, in fp32 steps.  (Candidate ratios are
// read on the device, unchecked: those below 0 are taken as 0, so that k is an index.)
__device__ inline void quantile_pos(float rho, int& k, float& f) {
  const float pos = fmaxf(__fmul_rn(rho, (float)(kD - 1)), 0.0f);
  k = min((int)floorf(pos), kD - 1);
  f = __fsub_rn(pos, (float)k);
}
__device__ inline float lerp_tau(float ak, float ak1, float f) {
  return __fadd_rn(ak, __fmul_rn(f, __fsub_rn(ak1, ak)));
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// ---------------------------------------------------------------------------
// prepare: q~ = q R_k (times the logit scale) on the fp32 matrix cores, 16 query
// rows per block of 8 waves.  Wave w computes column tile w (16 channels) of the
// block's rows as 32 chained 16x16x4 MFMAs: step s takes channels c = 32k + s in
// k-slot k, so lane (row lo, k-slot hi) holds q[row][32hi + s] (one 64-byte run of
// the row) and lane (column lo, k-slot hi) R_k[32hi + s][16w + lo] (16 lanes read 64
// contiguous bytes of a row of R_k).  R_k is read straight from L2 (no LDS copy, no
// barrier); all loads of a wave are issued before its MFMAs.  D lane (column lo,
// hi): rows 4hi + i.
// ---------------------------------------------------------------------------
constexpr int kPrepRows = 16;
constexpr int kRotWaves = 8;  // waves of a rotating block: one 16-channel tile each

typedef float prep_f4 __attribute__((ext_vector_type(4)));

__device__ inline void prepare_body(int bx, const uint16_t* __restrict__ q, int rows,
                                    const float* __restrict__ Rk, float qscale,
                                    float* __restrict__ qt, int rph, int Hq, int Hkv) {
  const int t = threadIdx.x, w = t >> 6, lo = t & 15, hi = (t >> 4) & 3;
  int kvh;
  query_row(bx, 0, kPrepRows, rows, Hq, Hkv, rph, kvh);
  if (Rk && rph) Rk += (size_t)kvh * kD * kD;  // the block's rows share a KV head
  int kv_;
  const int arow = query_row(bx, lo, kPrepRows, rows, Hq, Hkv, rph, kv_);
  if (!Rk) {  // R = I (bf16 baseline): a scaled copy, rows 2w, 2w + 1, lane: 2 channels
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = query_row(bx, 2 * w + i, kPrepRows, rows, Hq, Hkv, rph, kv_);
      if (row < 0) continue;
      const int c = 2 * (t & 63);
      const uint32_t v = *reinterpret_cast<const uint32_t*>(q + (size_t)row * kD + c);
      qt[(size_t)row * kD + c] = bf16_to_f32((uint16_t)(v & 0xffffu)) * qscale;
      qt[(size_t)row * kD + c + 1] = bf16_to_f32((uint16_t)(v >> 16)) * qscale;
    }
    return;
  }
  float a[32];
  if (arow >= 0) {
    const uint4* src = reinterpret_cast<const uint4*>(q + (size_t)arow * kD + 32 * hi);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 v = src[k];
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[8 * k + 2 * e] = bf16_to_f32((uint16_t)(u[e] & 0xffffu));
        a[8 * k + 2 * e + 1] = bf16_to_f32((uint16_t)(u[e] >> 16));
      }
    }
  } else {
#pragma unroll
    for (int s = 0; s < 32; ++s) a[s] = 0.0f;
  }
  float b[32];
#pragma unroll
  for (int s = 0; s < 32; ++s) b[s] = Rk[(size_t)(32 * hi + s) * kD + 16 * w + lo];
  prep_f4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < 32; ++s) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], d, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = query_row(bx, 4 * hi + i, kPrepRows, rows, Hq, Hkv, rph, kv_);
    if (row >= 0) qt[(size_t)row * kD + 16 * w + lo] = d[i] * qscale;
  }
}

// ---------------------------------------------------------------------------
// Row routing.  A cache update takes rows (token, kv-head h) of K or V (is_v);
// 32 consecutive lanes hold a row, lane c its channels 4c .. 4c + 3.  A policy gives
// the lane's part of a row in three steps, so that a loop can issue the loads of
// later rows without waiting for them:
//   key(tok)               loads that lead to other addresses;
//   load(tok, h, .., key)  the row's values and what else its destination needs;
//   route(raw, ..)         no loads (StepRows apart): x, the bf16 values to rotate
//                          and quantize, slot, the pool slot that receives them
//                          (< 0: none), and the bf16 values cp to copy to dst in the
//                          mixed cache's segment store (null: none).
// The lane that read x writes cp, after it: a row may be demoted from the place
// that its copy takes.
// ---------------------------------------------------------------------------
typedef uint32_t u2a4 __attribute__((ext_vector_type(2), aligned(4)));  // rows are 4-byte aligned

struct Key {
  int32_t b;
  int64_t p;
};
struct Raw {
  u2a4 x;
  int64_t p;        // slot (PlainRows) or position
  int32_t b, len, page;
};
struct Routed {
  u2a4 x, cp;
  int64_t slot;
  u2a4* dst;
};

struct PlainRows {  // oscar_kv_append: token i -> slot_mapping[i]
  const uint16_t* k;
  const uint16_t* v;
  const int64_t* slots;
  int n_tok, Hkv;
  __device__ Key key(int) const { return Key{0, 0}; }
  __device__ Raw load(int tok, int h, int is_v, int c, const Key&) const {
    Raw w{u2a4{0, 0}, -1, 0, 0, 0};
    if (tok < n_tok) {
      w.x = reinterpret_cast<const u2a4*>((is_v ? v : k) + ((size_t)tok * Hkv + h) * kD)[c];
      w.p = slots[tok];
    }
    return w;
  }
  __device__ Routed route(const Raw& w, int, int, int) const {
    return Routed{w.x, w.x, w.p, nullptr};
  }
};

// Segment store of the mixed cache: [B][Hkv][K, V][S0 + W][d] bf16; position p
// of a sequence has segment slot p (p < S0) or S0 + (p - S0) mod W (window).
__device__ inline u2a4* seg_row(uint16_t* seg, int Hkv, int S0, int W, int b, int h, int is_v,
                                int slot) {
  return reinterpret_cast<u2a4*>(
      seg + ((((size_t)b * Hkv + h) * 2 + is_v) * (size_t)(S0 + W) + slot) * kD);
}
__device__ inline int seg_slot(int S0, int W, int p) { return p < S0 ? p : S0 + (p - S0) % W; }

// oscar_mixed_append: token i of sequence seq_idx[i] at position pos[i] goes
// where a cache of length seq_lens[b] keeps it: INT2 for the history [lo, hi)
// (pool slot from the block table), bf16 segment slot otherwise; positions
// outside [0, seq_lens[b]) are skipped.
struct PrefillRows {
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* seg;
  const int32_t* seq_idx;
  const int64_t* pos;
  const int32_t* seq_lens;
  const int32_t* block_table;
  int n_tok, Hkv, max_pages, S0, W;
  __device__ Key key(int tok) const {
    return tok < n_tok ? Key{seq_idx[tok], pos[tok]} : Key{-1, 0};
  }
  __device__ Raw load(int tok, int h, int is_v, int c, const Key& key) const {
    Raw w{u2a4{0, 0}, key.p, key.b, 0, 0};
    if (key.b >= 0) {  // the page of any position: in range, whether it is used or not
      const int pg = key.p <= 0 ? 0 : (int)min(key.p / kP, (int64_t)max_pages - 1);
      w.x = reinterpret_cast<const u2a4*>((is_v ? v : k) + ((size_t)tok * Hkv + h) * kD)[c];
      w.len = seq_lens[key.b];
      w.page = block_table[(size_t)key.b * max_pages + pg];
    }
    return w;
  }
  __device__ Routed route(const Raw& w, int h, int is_v, int c) const {
    Routed f{w.x, w.x, -1, nullptr};
    const int len = min(max(w.len, 0), max_pages * kP);
    if (w.b < 0 || w.p < 0 || w.p >= len) return f;
    const int p = (int)w.p, lo = min(S0, len), hi = max(lo, len - W);
    if (p >= lo && p < hi) f.slot = (int64_t)w.page * kP + p % kP;
    else f.dst = seg_row(seg, Hkv, S0, W, w.b, h, is_v, seg_slot(S0, W, p)) + c;
    return f;
  }
};

// Decode step over the mixed cache: one new token per sequence b at position
// p = seq_lens[b] - 1 (Alg. 1 DecodeStep):
//   p < S0          -> bf16 sink slot p;
//   p >= S0, W = 0  -> INT2 at position p;
//   otherwise       -> bf16 window slot of p; when p - W >= S0 the token at
//                      p - W, which holds that slot, is first quantized into
//                      INT2 at position p - W (read before the slot is reused).
struct StepRows {
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* seg;
  const int32_t* seq_lens;
  const int32_t* block_table;
  int n_tok, Hkv, max_pages, S0, W;
  __device__ Key key(int b) const { return b < n_tok ? Key{b, seq_lens[b]} : Key{-1, 0}; }
  __device__ Raw load(int b, int h, int is_v, int c, const Key& key) const {
    Raw w{u2a4{0, 0}, key.p, key.b, 0, 0};
    if (key.b >= 0)
      w.x = reinterpret_cast<const u2a4*>((is_v ? v : k) + ((size_t)b * Hkv + h) * kD)[c];
    return w;
  }
  __device__ Routed route(const Raw& w, int h, int is_v, int c) const {
    Routed f{u2a4{0, 0}, w.x, -1, nullptr};
    const int p = min(max((int)w.p, 0), max_pages * kP) - 1;
    if (w.b < 0 || p < 0) return f;
    int qp = -1;  // position quantized into INT2 by this step
    if (p >= S0 && W == 0) {
      qp = p;
      f.x = w.x;
    } else {
      f.dst = seg_row(seg, Hkv, S0, W, w.b, h, is_v, seg_slot(S0, W, p)) + c;
      if (p - W >= S0) {
        qp = p - W;
        f.x = *f.dst;
      }
    }
    if (qp >= 0) f.slot = (int64_t)block_table[(size_t)w.b * max_pages + qp / kP] * kP + qp % kP;
    return f;
  }
};

// DEF: the default format (binary16 metadata, group-absmax clip, 32-channel
// groups) as compile-time constants, so that its code has no format branches.
__device__ inline QFmt pick(bool def, const QFmt& fmt) { return def ? QFmt{0, 0, 4, 0} : fmt; }

// ---------------------------------------------------------------------------
// Rotation of 16 rows by one block on the fp64 matrix cores: a 16 x 128 x 128
// product of v_mfma_f64_16x16x4_f64 steps.  Wave w owns columns 16w .. 16w + 15 and
// keeps its columns of R as fp64 in 64 registers for all of the block's items.  Step
// s takes channels 4s .. 4s + 3, A = the rows' values of those channels (lane l: row
// l % 16, channel 4s + l / 16) from LDS, where they are stored as fp64, B = rows
// 4s .. 4s + 3 of R.  A step adds its four products to the running fp64 sum one
// after another in channel order (lane group l / 16 = position in that order) and
// the steps run s = 0..31 in turn, so each x~ is the fp64 sum of the 128 exact
// products in ascending channel order rounded once to fp32.  Output lane l, register
// i holds row l / 16 + 4i, column l % 16; the rows go to LDS in fp32 for the
// quantizer.
//
// For a decode step's few rows, where latency counts: all columns at once on 8 waves
// (32 products deep), R straight from L2 into registers, nothing converted between
// the products.  Larger updates use the bulk kernel below.
// ---------------------------------------------------------------------------
constexpr int kItemRows = 16;
// A operand in LDS: channel 4s + k of a row at double 48 k + s of its 177 (reads of
// 16 rows and writes of 32 neighbouring lanes each hit all banks once; with channels
// in order the reads met four to a bank and kept the LDS busy 68 % of the time).
constexpr int kAPitch = 177;
__device__ inline int a_col(int ch) { return 48 * (ch & 3) + (ch >> 2); }
constexpr int kXtPitch = 144;  // floats per x~ row: 4 rows x 16 columns are written to 64 banks

typedef double d4v __attribute__((ext_vector_type(4)));

struct RotSmem {
  double a[kItemRows][kAPitch];
  float xt[kItemRows][kXtPitch];
};

// The wave's columns of R (lane l: R[4s + l / 16][16w + l % 16]).
__device__ inline void load_rot(const float* __restrict__ R, int w, int l, double (&b)[32]) {
#pragma unroll
  for (int s = 0; s < 32; ++s) b[s] = (double)R[(4 * s + (l >> 4)) * kD + 16 * w + (l & 15)];
}
// The lane's 4 channels (4c ..) of row r into the A operand.
__device__ inline void stage_row(RotSmem& sm, int r, int c, u2a4 x) {
  double* d = sm.a[r];
  d[a_col(4 * c)] = (double)__uint_as_float(x[0] << 16);
  d[a_col(4 * c + 1)] = (double)__uint_as_float(x[0] & 0xffff0000u);
  d[a_col(4 * c + 2)] = (double)__uint_as_float(x[1] << 16);
  d[a_col(4 * c + 3)] = (double)__uint_as_float(x[1] & 0xffff0000u);
}
// x~ of the staged rows' columns 16w .. 16w + 15, to sm.xt.
__device__ inline void rotate16(RotSmem& sm, int w, int l, const double (&b)[32]) {
  const int kq = l >> 4, j = l & 15;
  d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 32; ++s)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sm.a[j][48 * kq + s], b[s], acc, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) sm.xt[kq + 4 * i][16 * w + j] = __double2float_rn(acc[i]);
}

// Reductions over the lanes of a group in the quantizer's layout (32 lanes per row,
// 4 channels per lane; a group of G channels is G / 4 lanes): quad swaps and the
// mirror of 8 lanes, then by 16 and 32 lanes for the larger groups.
template <bool MAX>
__device__ inline float lanes_reduce(float x, int ng) {
  auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : fminf(a, b); };
  auto dpp = [](float v, auto ctrl) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false));
  };
  x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));   // lane ^ 1
  x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));   // lane ^ 2
  x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));  // mirror of 8 lanes
  if (ng <= 2) x = op(x, dpp(x, std::integral_constant<int, 0x128>{}));  // rotation by 8 of 16
  if (ng == 1) {
    const uint32_t u = __float_as_uint(x);
    const auto sw = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = op(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  }
  return x;
}

// Token quantile of a wave's two rows (rmax: the row's largest |x~|).  Bisection
// over the bit patterns of |x~| (positive floats order like their bits) for a
// threshold t with exactly k + 1 values at or below it, which ends as soon as t
// separates a_k from a_{k+1} (about 17 of the 31 halvings on Gaussian rows); equal
// values run it down to the smallest t with at least k + 1.  Counts are scalar
// work (ballots of both rows).
__device__ inline float token_quantile2(const float (&x)[4], float rmax, float rho, int half) {
  int k;
  float f;
  quantile_pos(rho, k, f);
  if (k >= kD - 1) return rmax;
  auto count_le = [&](uint32_t t0, uint32_t t1, int& c0, int& c1) {
    const float t = __uint_as_float(half ? t1 : t0);
    c0 = c1 = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint64_t m = __ballot(fabsf(x[e]) <= t);
      c0 += __popc((uint32_t)m);
      c1 += __popc((uint32_t)(m >> 32));
    }
  };
  uint32_t lo0 = 0, hi0 = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(rmax), 0);
  uint32_t lo1 = 0, hi1 = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(rmax), 32);
  int n0 = kD, n1 = kD;  // counts at hi0, hi1
  auto step = [&](uint32_t& lo, uint32_t& hi, int& n, uint32_t mid, int c) {
    if (lo >= hi || n == k + 1) return;
    if (c >= k + 1) {
      hi = mid;
      n = c;
    } else {
      lo = mid + 1;
    }
  };
  while ((lo0 < hi0 && n0 != k + 1) || (lo1 < hi1 && n1 != k + 1)) {
    const uint32_t m0 = lo0 + ((hi0 - lo0) >> 1), m1 = lo1 + ((hi1 - lo1) >> 1);
    int c0, c1;
    count_le(m0, m1, c0, c1);
    step(lo0, hi0, n0, m0, c0);
    step(lo1, hi1, n1, m1, c1);
  }
  const float t = __uint_as_float(half ? hi1 : hi0);
  float ak = 0.0f, ak1 = INFINITY;  // largest value at or below t, smallest above
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float v = fabsf(x[e]);
    ak = fmaxf(ak, v <= t ? v : 0.0f);
    ak1 = fminf(ak1, v <= t ? INFINITY : v);
  }
  ak = lanes_reduce<true>(ak, 1);
  ak1 = lanes_reduce<false>(ak1, 1);
  return lerp_tau(ak, (half ? n1 : n0) > k + 1 ? ak : ak1, f);
}

// y / s for a group's stored scale s (at most 11 significant bits), correctly
// rounded as an IEEE division, in three operations from r = 1 / s rounded to
// nearest: one residual correction of y r.  Equal to y / s for every pair of an
// 11-bit and a 24-bit significand (all 2^33: tests/test_scale_division.py), as long as r
// and the residual are not subnormal; see fast_scale.
__device__ inline float div_by_scale(float y, float s, float r) {
  const float q = __fmul_rn(y, r);
  return __fmaf_rn(__fmaf_rn(-q, s, y), r, q);
}
// Whether div_by_scale may replace the division for codes: always with binary16
// scales (2^-24 <= s; where the residual underflows, |y / s| < 2^-100 and the code
// follows from the zero point either way), and within these bounds with bfloat16.
__device__ inline bool fast_scale(float s) { return s >= 0x1p-60f && s <= 0x1p60f; }
// Clip bound of the values given to div_by_scale: finite, since a residual against an
// infinite y is NaN.  Finite rows can rotate to an fp32 infinity; a binary16 scale is
// then saturated, |s| = 65504 >= |z|, and y = +-FLT_MAX has the code of +-infinity.
// (A bfloat16 scale is past fast_scale's bounds there.)
__device__ inline float finite_bound(float tau) { return fminf(tau, FLT_MAX); }

// Clip, quantize, pack and write the wave's two rows (half-wave each, lane c of a
// half: channels 4c .. 4c + 3 in x) to pool slot `slot` (< 0: the row only takes
// part in the cross-lane steps).  Clipping is monotone, so the clipped extremes are
// the clipped values' extremes; a code is rint(clamp(y / s + z, 0, 3)), taken from
// the low mantissa bits after adding 2^23.
__device__ inline void store_rows(uint8_t* __restrict__ pages, int Hkv, int h, int64_t slot,
                                  int is_v, float clip, const QFmt& fmt, const float (&x)[4],
                                  int c, int half) {
  float mn = fminf(fminf(x[0], x[1]), fminf(x[2], x[3]));
  float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
  float tau;
  if (fmt.quantile) tau = token_quantile2(x, lanes_reduce<true>(fmaxf(-mn, mx), 1), clip, half);
  mn = lanes_reduce<false>(mn, fmt.ng);
  mx = lanes_reduce<true>(mx, fmt.ng);
  if (!fmt.quantile) tau = __fmul_rn(clip, fmaxf(fmaxf(-mn, mx), 0.0f));
  auto clamp = [](float v, float lo, float hi) { return __builtin_amdgcn_fmed3f(v, lo, hi); };
  const QParams p = quant_params(clamp(mn, -tau, tau), clamp(mx, -tau, tau), fmt);
  uint32_t byte = 0;
  if (fmt.bf16 && __any(!p.deg && !fast_scale(p.sf))) {
#pragma unroll
    for (int e = 0; e < 4; ++e) byte |= quant_code(clamp(x[e], -tau, tau), p) << (2 * e);
  } else {
    const float s = p.deg ? 1.0f : p.sf, r = p.deg ? 0.0f : __fdiv_rn(1.0f, p.sf);  // deg: y / s = 0
    tau = finite_bound(tau);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float d = div_by_scale(clamp(x[e], -tau, tau), s, r);
      byte += __float_as_uint(__fadd_rn(clamp(__fadd_rn(d, p.zf), 0.0f, 3.0f), 8388608.0f)) << (2 * e);
    }
  }
  if (slot < 0) return;  // uniform across the half wave
  const int64_t page = slot / kP;
  const int t = (int)(slot - page * kP);
  uint8_t* blk = pages + ((size_t)page * Hkv + h) * block_bytes(fmt.ng);
  if (is_v) blk[kOffVCodes + c * kP + t] = (uint8_t)byte;
  else blk[kOffKCodes + t * (kD / 4) + c] = (uint8_t)byte;
  const int lanes = 32 / fmt.ng;  // per group
  if ((c & (lanes - 1)) == 0)
    *reinterpret_cast<uint32_t*>(blk + (is_v ? off_vsz(fmt.ng) : kOffKSz) +
                                 ((c / lanes) * kP + t) * 4) =
        (uint32_t)p.s16 | ((uint32_t)p.z16 << 16);
}

// x~ of the thread's 4 channels: rotated (from LDS), or the row itself.
__device__ inline void xt_of(const RotSmem& sm, int r, int c, float (&x)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(&sm.xt[r][4 * c]);
  x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
}
__device__ inline void xt_of(u2a4 w, float (&x)[4]) {
  x[0] = __uint_as_float(w[0] << 16);
  x[1] = __uint_as_float(w[0] & 0xffff0000u);
  x[2] = __uint_as_float(w[1] << 16);
  x[3] = __uint_as_float(w[1] & 0xffff0000u);
}

// Items of a cache update: 16 consecutive tokens (group g) of one kv-head h (their
// bytes of a page's token-minor regions are adjacent), item = g Hkv + h.
struct Items {
  int groups, Hkv, step, g, h;
  __device__ Items(int n_tok, int Hkv_, int first, int step_)
      : groups((n_tok + kItemRows - 1) / kItemRows), Hkv(Hkv_), step(step_), g(first / Hkv_),
        h(first % Hkv_) {}
  __device__ bool valid() const { return g < groups; }
  __device__ void advance() {
    g += step / Hkv;
    h += step % Hkv;
    if (h >= Hkv) {
      h -= Hkv;
      ++g;
    }
  }
};

// One item per block of 8 waves (a decode step's tokens; more than one in turn past
// two blocks per CU).
// bx of gx: the block's items; rph: of head bx % Hkv (gx is a multiple of Hkv).
template <class Rows>
__device__ inline void append_body(RotSmem& sm, int is_v, int bx, int gx,
                                   uint8_t* __restrict__ pages, const Rows& rows,
                                   const float* __restrict__ Rk, const float* __restrict__ Rv,
                                   float clip_k, float clip_v, const QFmt& fmt) {
  const float* __restrict__ R = is_v ? Rv : Rk;  // nullptr: identity
  const float clip = is_v ? clip_v : clip_k;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, half = l >> 5;
  const int r = t >> 5, c = t & 31;  // the thread's row of an item, and lane in it
  if (R && fmt.rph) R += (size_t)(bx % rows.Hkv) * kD * kD;
  Items it(rows.n_tok, rows.Hkv, bx, gx);
  if (!it.valid()) return;
  int tok = it.g * kItemRows + r;
  Raw raw = rows.load(tok, it.h, is_v, c, rows.key(tok));
  double b[32];
  if (R) load_rot(R, w, l, b);
  for (;;) {
    const Routed cur = rows.route(raw, it.h, is_v, c);
    if (cur.dst) *cur.dst = cur.cp;
    float x[4];
    if (R) {
      stage_row(sm, r, c, cur.x);
      __syncthreads();
      rotate16(sm, w, l, b);
      __syncthreads();
      xt_of(sm, r, c, x);
    } else {
      xt_of(cur.x, x);
    }
    store_rows(pages, rows.Hkv, it.h, cur.slot, is_v, clip, fmt, x, c, half);
    it.advance();
    if (!it.valid()) break;
    tok = it.g * kItemRows + r;
    raw = rows.load(tok, it.h, is_v, c, rows.key(tok));
  }
}

// ---------------------------------------------------------------------------
// Bulk cache update (more items than teams of 8 waves fit on the GPU): one
// persistent block of 16 independent waves per CU, half of the blocks per tensor.  A
// wave takes an item at a time from the block's list (a counter in LDS: the oldest
// wave of a SIMD issues first and would be done early with a fixed share), stages
// its rows as bf16, rotates them over all eight column tiles and quantizes them in
// the quad-lane layout.  The products are as in rotate16; tile t holds channels
// 64 (t / 4) + 4 j + t % 4 (j = column), so that a lane's B values are two 16-byte
// reads of the fp32 R in LDS, and x~ goes through the wave's 4 KB area one channel
// half at a time.
//
// Bound: the fp64 matrix core, 16,384 of a SIMD's cycles per item: 74 % busy over a
// prompt of 131072 tokens, 37 % where a wave has 1.6 items in the token-quantile format.
// With four waves per SIMD at different points of their items, the rest of an item (980
// vector instructions beside its 256 products, 2,570 with the token quantile, and the
// dependent loads that route its rows) runs while other waves' products do.  At the 128
// registers of 16 waves the instances keep 12 to 44 bytes per lane in scratch.  The quantizer has the most
// work per lane here (32 channels), which costs the fewest instructions; 32 lanes a
// row, as in store_rows, took 1,700 and 7,000.  131072 tokens x 8 heads: 1474 us with
// two waves per SIMD, IEEE divisions per code and the routing loads in front of each
// item's products, 1156 us now (1092 without the stores); 6408 tokens x 8 heads in the
// token-quantile format: 288 -> 89 us.
// ---------------------------------------------------------------------------
constexpr int kBulkWaves = 16;
constexpr int kStagePitch = 66;  // dwords per staged bf16 row (8-byte reads of 16 rows: all banks)
constexpr int kHalfPitch = 68;   // floats per half row of x~

// Quad-lane layout of the bulk kernels: lane l takes row l / 4 of an item's 16
// rows, channels 32 q .. 32 q + 31 (q = l % 4); a group of G channels is the G / 32
// lanes of a row with equal q / (G / 32).
__device__ inline float quad_swap1(float v) {  // lane ^ 1
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}
__device__ inline float quad_swap2(float v) {  // lane ^ 2
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
}
__device__ inline float quad_group_max(float v, int ng) {
  if (ng <= 2) v = fmaxf(v, quad_swap1(v));
  if (ng == 1) v = fmaxf(v, quad_swap2(v));
  return v;
}
__device__ inline float quad_group_min(float v, int ng) {
  if (ng <= 2) v = fminf(v, quad_swap1(v));
  if (ng == 1) v = fminf(v, quad_swap2(v));
  return v;
}
__device__ inline int quad_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
  return v + __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
}

// Token quantile of 16 rows at once in the quad-lane layout; rmax: the row's
// largest |x~|.  Bisection over the bit patterns of |x~| (positive floats order
// like their bits) for a threshold t with exactly k + 1 values at or below it,
// which ends as soon as t separates a_k from a_{k+1} (about 17 of the 31 halvings
// on Gaussian rows); equal values run it down to the smallest t with at least k + 1.
__device__ inline float token_quantile_quad(const float (&x)[32], float rmax, float rho) {
  int k;
  float f;
  quantile_pos(rho, k, f);
  if (k >= kD - 1) return rmax;
  auto count_le = [&](uint32_t t) {
    const float tf = __uint_as_float(t);
    int c = 0;
#pragma unroll
    for (int i = 0; i < 32; ++i) c += fabsf(x[i]) <= tf ? 1 : 0;
    return quad_sum(c);
  };
  // smallest t with count >= k + 1 in [lo, hi]; n = count at hi
  uint32_t lo = 0, hi = __float_as_uint(rmax);
  int n = kD;
  while (__any(lo < hi && n != k + 1)) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    const int c = count_le(mid);
    const bool open = lo < hi && n != k + 1;
    const bool up = open && c < k + 1, down = open && c >= k + 1;
    lo = up ? mid + 1 : lo;
    hi = down ? mid : hi;
    n = down ? c : n;
  }
  const float t = __uint_as_float(hi);
  float ak = 0.0f, ak1 = INFINITY;  // largest value at or below t, smallest above
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const float v = fabsf(x[i]);
    ak = fmaxf(ak, v <= t ? v : 0.0f);
    ak1 = fminf(ak1, v <= t ? INFINITY : v);
  }
  ak = quad_group_max(ak, 1);
  ak1 = quad_group_min(ak1, 1);
  return lerp_tau(ak, n > k + 1 ? ak : ak1, f);
}

// Clip, quantize, pack and write a bulk item's 16 rows (quad-lane layout); same
// steps as store_rows.
__device__ inline void store_slice32(uint8_t* __restrict__ pages, int Hkv, int h, int64_t slot,
                                     int is_v, float clip, const QFmt& fmt, const float (&x)[32],
                                     int q) {
  float mn = x[0], mx = x[0];
#pragma unroll
  for (int i = 1; i < 32; ++i) {
    mn = fminf(mn, x[i]);
    mx = fmaxf(mx, x[i]);
  }
  float tau;
  if (fmt.quantile) {
    tau = token_quantile_quad(x, quad_group_max(fmaxf(-mn, mx), 1), clip);
    mn = quad_group_min(mn, fmt.ng);
    mx = quad_group_max(mx, fmt.ng);
  } else {
    mn = quad_group_min(mn, fmt.ng);
    mx = quad_group_max(mx, fmt.ng);
    tau = __fmul_rn(clip, fmaxf(fmaxf(-mn, mx), 0.0f));
  }
  auto clamp = [](float v, float lo, float hi) { return __builtin_amdgcn_fmed3f(v, lo, hi); };
  const QParams p = quant_params(clamp(mn, -tau, tau), clamp(mx, -tau, tau), fmt);
  uint32_t w[8];
  if (fmt.bf16 && __any(!p.deg && !fast_scale(p.sf))) {
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) {
      w[jb] = 0;
#pragma unroll 1
      for (int e = 0; e < 4; ++e) {
        float v = x[0];
#pragma unroll
        for (int i = 1; i < 32; ++i) v = i == 4 * jb + e ? x[i] : v;
        w[jb] |= quant_code(clamp(v, -tau, tau), p) << (2 * e);
      }
    }
  } else {
    const float s = p.deg ? 1.0f : p.sf, r = p.deg ? 0.0f : __fdiv_rn(1.0f, p.sf);  // deg: y / s = 0
    tau = finite_bound(tau);
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) {
      uint32_t c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = div_by_scale(clamp(x[4 * jb + e], -tau, tau), s, r);
        c[e] = __float_as_uint(__fadd_rn(clamp(__fadd_rn(d, p.zf), 0.0f, 3.0f), 8388608.0f));
      }
      w[jb] = c[0] + (c[1] << 2) + (c[2] << 4) + (c[3] << 6);  // the low byte
    }
  }
  if (slot < 0) return;
  const int64_t page = slot / kP;
  const int t = (int)(slot - page * kP);
  uint8_t* blk = pages + ((size_t)page * Hkv + h) * block_bytes(fmt.ng);
  if (is_v) {
#pragma unroll
    for (int jb = 0; jb < 8; ++jb) blk[kOffVCodes + (8 * q + jb) * kP + t] = (uint8_t)w[jb];
  } else {
    auto join = [](uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
      return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400u),
                                   __builtin_amdgcn_perm(b, a, 0x0c0c0400u), 0x05040100u);
    };
    *reinterpret_cast<uint2*>(blk + kOffKCodes + t * (kD / 4) + 8 * q) =
        make_uint2(join(w[0], w[1], w[2], w[3]), join(w[4], w[5], w[6], w[7]));
  }
  const int per = 4 / fmt.ng;  // slices per group
  if (q % per == 0) {
    const uint32_t sz_base = is_v ? off_vsz(fmt.ng) : kOffKSz;
    *reinterpret_cast<uint32_t*>(blk + sz_base + ((q / per) * kP + t) * 4) =
        (uint32_t)p.s16 | ((uint32_t)p.z16 << 16);
  }
}

// 64-bit value of lane src (any source lane, per-lane index).  The halves are
// moved as 32-bit ints and widened as unsigned (a sign-extended low half would
// set every bit of the high half).
__device__ inline int64_t shfl64(int64_t v, int src) {
  const int lo = __shfl((int)(uint32_t)v, src, 64), hi = __shfl((int)(v >> 32), src, 64);
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
// 64-bit value of lane `lane` (wave-uniform index), widened the same way.
__device__ inline uint64_t readlane64(uint64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// R to LDS by a block of WAVES waves (loads issued before the stores).
template <int WAVES>
__device__ inline void stage_rot(float4 (&Rs)[kD][kD / 4], const float* __restrict__ R, int t) {
  constexpr int kN = kD * kD / 4 / (WAVES * 64);
  float4 r4[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) r4[i] = reinterpret_cast<const float4*>(R)[t + WAVES * 64 * i];
#pragma unroll
  for (int i = 0; i < kN; ++i) (&Rs[0][0])[t + WAVES * 64 * i] = r4[i];
}
// One wave's product of the 16 bf16 rows staged in its area and R: column j of tile t
// is channel 64 (t / 4) + 4 j + t % 4.
__device__ inline void rotate_wave(const float4 (&Rs)[kD][kD / 4], const uint32_t* area, int l,
                                   d4v (&acc)[8]) {
  const int kq = l >> 4, j = l & 15;
  // v_perm selector: the bf16 of channel 4 s + kq (of the 8 bytes read) into the
  // high half of a dword, zeros below: an fp32 with the same value
  const uint32_t asel = 0x01000C0Cu + 0x02020000u * (uint32_t)kq;
#pragma unroll
  for (int tt = 0; tt < 8; ++tt) acc[tt] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int s = 0; s < kD / 4; ++s) {
    const uint2 xa = *reinterpret_cast<const uint2*>(&area[j * kStagePitch + 2 * s]);
    const double a = (double)__uint_as_float(__builtin_amdgcn_perm(xa.y, xa.x, asel));
    const float4 r0 = Rs[4 * s + kq][j], r1 = Rs[4 * s + kq][16 + j];
    const float rb[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
    for (int tt = 0; tt < 8; ++tt)
      acc[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)rb[tt], acc[tt], 0, 0, 0);
  }
}

template <class Rows, bool DEF>
__global__ __launch_bounds__(kBulkWaves * 64) void append_bulk_kernel(
    uint8_t* __restrict__ pages, Rows rows, const float* __restrict__ Rk,
    const float* __restrict__ Rv, float clip_k, float clip_v, QFmt fmt_arg) {
  __shared__ float4 Rs[kD][kD / 4];                                  // 64 KB
  __shared__ uint32_t area_all[kBulkWaves][kItemRows * kHalfPitch];  // 68 KB
  __shared__ int taken;
  const QFmt fmt = pick(DEF, fmt_arg);
  const int is_v = blockIdx.y, bx = blockIdx.x, gx = gridDim.x, Hkv = rows.Hkv;
  const float* __restrict__ R = is_v ? Rv : Rk;  // nullptr: identity
  const float clip = is_v ? clip_v : clip_k;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, kq = l >> 4, j = l & 15;
  if (R) stage_rot<kBulkWaves>(Rs, R + (fmt.rph ? (size_t)(bx % Hkv) * kD * kD : 0), t);  // gx: a multiple of Hkv
  if (t == 0) taken = 0;
  __syncthreads();
  uint32_t* area = area_all[w];
  float* xt = reinterpret_cast<float*>(area);
  const int groups = (rows.n_tok + kItemRows - 1) / kItemRows;
  const int n_items = groups * Hkv, n_mine = (n_items - bx + gx - 1) / gx;
  for (;;) {
    int n = 0;
    if (l == 0) n = atomicAdd(&taken, 1);
    n = __builtin_amdgcn_readfirstlane(n);
    if (n >= n_mine) break;
    const int item = bx + n * gx, tok0 = item / Hkv * kItemRows, h = item % Hkv;
    // rows of the item: lane l their channels 2 l, 2 l + 1; destination of row l % 16
    uint32_t row[kItemRows];
    const uint16_t* src = (is_v ? rows.v : rows.k) + ((size_t)tok0 * Hkv + h) * kD;
#pragma unroll
    for (int r = 0; r < kItemRows; ++r)
      row[r] = tok0 + r < rows.n_tok
                   ? reinterpret_cast<const uint32_t*>(src + (size_t)r * Hkv * kD)[l] : 0u;
    const int tok = tok0 + j;
    const Routed to = rows.route(rows.load(tok, h, is_v, 0, rows.key(tok)), h, is_v, 0);
    lane_exchange();  // the previous item's reads of the wave's area come first
#pragma unroll
    for (int r = 0; r < kItemRows; ++r) area[r * kStagePitch + l] = row[r];
    if (__any(to.dst != nullptr)) {
#pragma unroll
      for (int r = 0; r < kItemRows; ++r) {
        uint32_t* d = reinterpret_cast<uint32_t*>(
            (uintptr_t)readlane64((uint64_t)reinterpret_cast<uintptr_t>(to.dst), r));
        if (d) d[l] = row[r];
      }
    }
    lane_exchange();
    const int rr = l >> 2, q = l & 3;  // quantizer: row, channels 32 q .. + 31
    float x[32];
    if (R) {
      d4v acc[8];
      rotate_wave(Rs, area, l, acc);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        lane_exchange();  // earlier reads of the area come first
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<float4*>(xt + (kq + 4 * i) * kHalfPitch + 4 * j) =
              make_float4(__double2float_rn(acc[4 * hf][i]), __double2float_rn(acc[4 * hf + 1][i]),
                          __double2float_rn(acc[4 * hf + 2][i]), __double2float_rn(acc[4 * hf + 3][i]));
        lane_exchange();
        if ((q >> 1) == hf) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(xt + rr * kHalfPitch + 32 * (q & 1) + 4 * i);
            x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
          }
        }
      }
    } else {  // x~ = x: the staged bf16 values
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t pr = area[rr * kStagePitch + 16 * q + i];
        x[2 * i] = __uint_as_float(pr << 16);
        x[2 * i + 1] = __uint_as_float(pr & 0xffff0000u);
      }
    }
    store_slice32(pages, Hkv, h, shfl64(to.slot, rr), is_v, clip, fmt, x, q);
  }
}

template <class Rows, bool DEF>
__global__ __launch_bounds__(kRotWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void append_kernel(
    uint8_t* __restrict__ pages, Rows rows, const float* __restrict__ Rk,
    const float* __restrict__ Rv, float clip_k, float clip_v, QFmt fmt) {
  __shared__ RotSmem sm;
  append_body(sm, blockIdx.y, blockIdx.x, gridDim.x, pages, rows, Rk, Rv, clip_k, clip_v,
              pick(DEF, fmt));
}

__global__ __launch_bounds__(kRotWaves * 64) void prepare_kernel(const uint16_t* __restrict__ q, int rows,
                                                      const float* __restrict__ Rk, float qscale,
                                                      float* __restrict__ qt, int rph, int Hq,
                                                      int Hkv) {
  prepare_body(blockIdx.x, q, rows, Rk, qscale, qt, rph, Hq, Hkv);
}

// One launch for a decode step's prologue: append_blocks blocks of the K update, as
// many of the V update, then the query rotation's.  The parts are independent; the
// split kernel that follows needs them all.
template <class Rows, bool DEF>
__global__ __launch_bounds__(kRotWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void prologue_kernel(
    uint8_t* __restrict__ pages, Rows rows, const float* __restrict__ Rk,
    const float* __restrict__ Rv, float clip_k, float clip_v, QFmt fmt_arg, int append_blocks,
    const uint16_t* __restrict__ q, int q_rows, int Hq, float qscale, float* __restrict__ qt) {
  __shared__ RotSmem sm;
  const int bx = blockIdx.x;
  if (bx < 2 * append_blocks) {
    const int is_v = bx >= append_blocks;
    append_body(sm, is_v, is_v ? bx - append_blocks : bx, append_blocks, pages, rows,
                Rk, Rv, clip_k, clip_v, pick(DEF, fmt_arg));
  } else {
    prepare_body(bx - 2 * append_blocks, q, q_rows, Rk, qscale, qt, fmt_arg.rph, Hq, rows.Hkv);
  }
}

// The prologue of a decode step over the mixed cache, and the bf16 tokens' partial
// states, which need nothing of it but the newest token (taken from k_new and v_new;
// the slot that the update overwrites meanwhile is not used).  The partial's blocks
// come first: they are the longer ones (one wave per 64 slots of a (sequence,
// kv-head); 5 of the 8 waves at S0 + W = 320).  In a launch of their own between the
// split kernel and the reduce they took 21.8 us at 64 sequences x 8 KV heads, after a
// prologue of 14 us, and 10 us after 9 at 8 sequences.
template <int NH, bool DEF>
__global__ __launch_bounds__(kRotWaves * 64)
__attribute__((amdgpu_waves_per_eu(NH > 8 ? 2 : 4, NH > 8 ? 2 : 4))) void mixed_prologue_kernel(
    uint8_t* __restrict__ pages, StepRows rows, const float* __restrict__ Rk,
    const float* __restrict__ Rv, float clip_k, float clip_v, QFmt fmt_arg, int append_blocks,
    const uint16_t* __restrict__ q, int q_rows, int Hq, float qscale, float* __restrict__ qt,
    SegArgs seg, int seg_blocks) {
  __shared__ union {
    RotSmem rot;
    SegSmem<NH> seg;
  } sm;
  int bx = blockIdx.x;
  if (bx < seg_blocks) {
    seg_partial_body<NH>(sm.seg, bx, kRotWaves, seg);
    return;
  }
  bx -= seg_blocks;
  if (bx < 2 * append_blocks) {
    const int is_v = bx >= append_blocks;
    append_body(sm.rot, is_v, is_v ? bx - append_blocks : bx, append_blocks, pages, rows, Rk, Rv,
                clip_k, clip_v, pick(DEF, fmt_arg));
  } else {
    prepare_body(bx - 2 * append_blocks, q, q_rows, Rk, qscale, qt, fmt_arg.rph, Hq, rows.Hkv);
  }
}

// ---------------------------------------------------------------------------
// Clip calibration (Alg. 1 CalibrateClip).  The paper leaves the procedure open;
// it is read here as: the candidate ratio whose quantization of the rotated
// calibration rows has the smallest squared error.  Independent waves take items
// (16 tokens of a head; a fixed share, so that sums have a fixed order) and rotate
// them as the bulk cache update does, in its quad-lane layout (lane: 32 channels of a row); for every
// candidate a lane clips and quantizes its channels with the cache update's steps
// and adds (x~_c - s (code_c - z))^2 in fp64, s and z read back from their stored
// format.  What does not depend on the candidate is done once per item: the groups'
// extremes (clipping is monotone), and for the token quantile the row's |x~| sorted
// (a bitonic network over the quad, kept in LDS), of which a candidate reads a_k and
// a_{k+1}.  Sums are added in a fixed order: over the lanes per item and candidate
// (lane n keeps candidate n), then the waves, then (clip_reduce_kernel) the blocks.
//
// Bound: VALU issue, 67 % busy at two waves per SIMD, the matrix cores 22 %: 12,500
// instructions per item with 21 candidates, its sort and 256 products among them.  One wave per row, with cross-lane reductions, three divisions per value and
// the group's parameters formed by every lane for every candidate, took 1112 us per
// tensor (8878 tokens x 8 heads, 21 candidates, groups of 128 with the quantile).
// ---------------------------------------------------------------------------
constexpr int kClipWaves = 8;
constexpr int kRowPitch = kD + 4;  // floats per x~ row in LDS

// Sum over the wave, the same in every lane: DPP inside rows of 16 lanes, then the
// row swaps across 16 and 32 lanes.
__device__ inline double wave_sum_f64(double x) {
  auto dpp = [](double v, auto ctrl) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, decltype(ctrl)::value, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), decltype(ctrl)::value, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
  };
  x += dpp(x, std::integral_constant<int, 0xB1>{});
  x += dpp(x, std::integral_constant<int, 0x4E>{});
  x += dpp(x, std::integral_constant<int, 0x124>{});
  x += dpp(x, std::integral_constant<int, 0x128>{});
  double tot = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    tot += __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(x), 16 * k));
  return tot;
}

// Ascending sort of a row's 128 values in the quad-lane layout (element 32 q + i in
// v[i] of lane q): each lane's 32 by a bitonic network, then two merges over lanes.
__device__ inline void quad_sort128(float (&v)[32], int q) {
  auto order = [&](int a, int b) {  // v[a] <= v[b]
    const float lo = fminf(v[a], v[b]), hi = fmaxf(v[a], v[b]);
    v[a] = lo;
    v[b] = hi;
  };
  // compare with the elements `mirror`ed or in place of lane q ^ x
  auto across = [&](auto ctrl, bool mirror, bool low) {
    float o[32];
#pragma unroll
    for (int i = 0; i < 32; ++i)
      o[i] = __int_as_float(__builtin_amdgcn_update_dpp(
          0, __float_as_int(v[mirror ? 31 - i : i]), decltype(ctrl)::value, 0xF, 0xF, false));
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = low ? fminf(v[i], o[i]) : fmaxf(v[i], o[i]);
  };
  auto merge32 = [&]() {
#pragma unroll
    for (int d = 16; d >= 1; d >>= 1)
#pragma unroll
      for (int i = 0; i < 32; ++i)
        if (!(i & d)) order(i, i + d);
  };
#pragma unroll
  for (int k = 2; k <= 32; k <<= 1) {
#pragma unroll
    for (int i = 0; i < 32; ++i)  // first step of a merge against the mirrored half
      if ((i & (k - 1)) < k / 2) order(i, (i & ~(k - 1)) + (k - 1 - (i & (k - 1))));
#pragma unroll
    for (int d = k >> 2; d >= 1; d >>= 1)
#pragma unroll
      for (int i = 0; i < 32; ++i)
        if (!(i & d)) order(i, i + d);
  }
  across(std::integral_constant<int, 0xB1>{}, true, (q & 1) == 0);  // 64: lane ^ 1, mirrored
  merge32();
  across(std::integral_constant<int, 0x1B>{}, true, q < 2);         // 128: lane 3 - q, mirrored
  across(std::integral_constant<int, 0xB1>{}, false, (q & 1) == 0); // distance 32
  merge32();
}

// Up to two tensors (K and V of a layer) in one launch: blockIdx.y.
struct ClipJobs {
  const uint16_t* x[2];
  const float* R[2];
  double* partial[2];
  double* err[2];
  float* best[2];
};

// FEW: blocks have at most two items each, see `share`.
template <bool FEW>
__global__ __launch_bounds__(kClipWaves * 64) void clip_err_kernel(
    ClipJobs jobs, int n_tok, const float* __restrict__ cands, int n_cands, QFmt fmt, int Hkv) {
  __shared__ float4 Rs[kD][kD / 4];                                   // 64 KB
  __shared__ uint32_t area_all[kClipWaves][kItemRows * kRowPitch];    // 66 KB
  __shared__ double werr[kClipWaves][kMaxClipCands];
  const uint16_t* __restrict__ x_all = jobs.x[blockIdx.y];
  const float* __restrict__ R = jobs.R[blockIdx.y];
  const int bx = blockIdx.x, gx = gridDim.x;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, kq = l >> 4, j = l & 15;
  if (R) stage_rot<kClipWaves>(Rs, R + (fmt.rph ? (size_t)(bx % Hkv) * kD * kD : 0), t);  // gx: a multiple of Hkv
  __syncthreads();
  uint32_t* area = area_all[w];
  float* xt = reinterpret_cast<float*>(area);
  const int n_items = (n_tok + kItemRows - 1) / kItemRows * Hkv, n_mine = (n_items - bx + gx - 1) / gx;
  const int rr = l >> 2, q = l & 3;
  double mine = 0.0;  // lane n: the wave's error of candidate n
  auto clamp = [](float v, float lo, float hi) { return __builtin_amdgcn_fmed3f(v, lo, hi); };
  // One or two items: `share` waves take the same item and every share-th candidate (the
  // sums have the same terms in the same order), at most a wave per SIMD, whose products
  // would wait for each other.  300 tokens of one head: 37.9 -> 23.0 us.
  const int share = !FEW ? 1 : n_mine == 1 ? 4 : 2;
  const int first = !FEW ? 0 : __builtin_amdgcn_readfirstlane(w % share);
  for (int n = w / share; n < n_mine; n += kClipWaves / share) {
    const int item = bx + n * gx, tok0 = item / Hkv * kItemRows, h = item % Hkv;
    const uint16_t* src = x_all + ((size_t)tok0 * Hkv + h) * kD;
    uint32_t row[kItemRows];
#pragma unroll
    for (int r = 0; r < kItemRows; ++r)
      row[r] = tok0 + r < n_tok ? reinterpret_cast<const uint32_t*>(src + (size_t)r * Hkv * kD)[l] : 0u;
    lane_exchange();  // the previous item's reads of the wave's area come first
#pragma unroll
    for (int r = 0; r < kItemRows; ++r) area[r * kStagePitch + l] = row[r];
    lane_exchange();
    float x[32];
    if (R) {
      d4v acc[8];
      rotate_wave(Rs, area, l, acc);
      lane_exchange();
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
          *reinterpret_cast<float4*>(xt + (kq + 4 * i) * kRowPitch + 64 * hf + 4 * j) =
              make_float4(__double2float_rn(acc[4 * hf][i]), __double2float_rn(acc[4 * hf + 1][i]),
                          __double2float_rn(acc[4 * hf + 2][i]), __double2float_rn(acc[4 * hf + 3][i]));
      lane_exchange();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(xt + rr * kRowPitch + 32 * q + 4 * i);
        x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t pr = area[rr * kStagePitch + 16 * q + i];
        x[2 * i] = __uint_as_float(pr << 16);
        x[2 * i + 1] = __uint_as_float(pr & 0xffff0000u);
      }
    }
    float mn = x[0], mx = x[0];
#pragma unroll
    for (int i = 1; i < 32; ++i) {
      mn = fminf(mn, x[i]);
      mx = fmaxf(mx, x[i]);
    }
    mn = quad_group_min(mn, fmt.ng);
    mx = quad_group_max(mx, fmt.ng);
    if (fmt.quantile) {
      float v[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = fabsf(x[i]);
      quad_sort128(v, q);
      lane_exchange();  // every lane's reads of the area come first
#pragma unroll
      for (int i = 0; i < 8; ++i)
        *reinterpret_cast<float4*>(xt + rr * kRowPitch + 32 * q + 4 * i) =
            make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
      lane_exchange();
    }
    const bool live = tok0 + rr < n_tok;
    double x64[32];  // (an infinite one has an infinite error whatever its code: no finite_bound)
#pragma unroll
    for (int i = 0; i < 32; ++i) x64[i] = (double)x[i];
#pragma unroll 1
    for (int n_c = first; n_c < n_cands; n_c += share) {
      const float clip = cands[n_c];
      float tau;
      if (fmt.quantile) {
        int k;
        float f;
        quantile_pos(clip, k, f);
        const float ak = xt[rr * kRowPitch + k], ak1 = xt[rr * kRowPitch + min(k + 1, kD - 1)];
        tau = k >= kD - 1 ? ak : lerp_tau(ak, ak1, f);
      } else {
        tau = __fmul_rn(clip, fmaxf(fmaxf(-mn, mx), 0.0f));
      }
      const QParams p = quant_params(clamp(mn, -tau, tau), clamp(mx, -tau, tau), fmt);
      const double s64 = (double)meta_load(fmt, p.s16), z64 = (double)meta_load(fmt, p.z16);
      double e0 = 0.0, e1 = 0.0;
      if (fmt.bf16 && __any(!p.deg && !fast_scale(p.sf))) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const double d = __fma_rn(-s64, (double)quant_code(clamp(x[i], -tau, tau), p) - z64, x64[i]);
          e0 = __fma_rn(d, d, e0);
        }
      } else {
        const float s = p.deg ? 1.0f : p.sf, r = p.deg ? 0.0f : __fdiv_rn(1.0f, p.sf);  // deg: y / s = 0
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const float d = div_by_scale(clamp(x[i], -tau, tau), s, r);
          const float code = rintf(clamp(__fadd_rn(d, p.zf), 0.0f, 3.0f));
          const double u = __fma_rn(-s64, (double)code - z64, x64[i]);
          if (i & 1) e1 = __fma_rn(u, u, e1);
          else e0 = __fma_rn(u, u, e0);
        }
      }
      const double tot = wave_sum_f64(live ? e0 + e1 : 0.0);
      if (l == n_c) mine += tot;
    }
  }
  if (l < kMaxClipCands) werr[w][l] = mine;
  __syncthreads();
  if (t < n_cands) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < kClipWaves; ++k) tot += werr[k][t];
    jobs.partial[blockIdx.y][(size_t)bx * n_cands + t] = tot;
  }
}

// err[n] = (sum of the blocks' partials) / (n_rows d); best = the candidate of the
// first minimum.  Thread (candidate n, part p) adds blocks p, p + 8, ... in order,
// then the 8 part sums are added in order (a fixed order: deterministic).
constexpr int kClipParts = 8;

__global__ __launch_bounds__(kClipParts * kMaxClipCands) void clip_reduce_kernel(
    ClipJobs jobs, int n_blocks, int n_cands, const float* __restrict__ cands, double inv_n) {
  const double* __restrict__ partial = jobs.partial[blockIdx.x];
  double* __restrict__ err = jobs.err[blockIdx.x];
  float* __restrict__ best = jobs.best[blockIdx.x];
  __shared__ double ps[kClipParts][kMaxClipCands];
  __shared__ double es[kMaxClipCands];
  const int n = threadIdx.x % kMaxClipCands, part = threadIdx.x / kMaxClipCands;
  double acc = 0.0;
  if (n < n_cands)
    for (int b = part; b < n_blocks; b += kClipParts) acc += partial[(size_t)b * n_cands + n];
  ps[part][n] = acc;
  __syncthreads();
  if (part == 0 && n < n_cands) {
    double tot = 0.0;
#pragma unroll
    for (int p = 0; p < kClipParts; ++p) tot += ps[p][n];
    es[n] = tot * inv_n;
    err[n] = es[n];
  }
  __syncthreads();
  if (threadIdx.x == 0 && best) {
    int arg = 0;
    for (int i = 1; i < n_cands; ++i)
      if (es[i] < es[arg]) arg = i;
    best[0] = cands[arg];
  }
}

}  // namespace

namespace {
// Items of a cache update per tensor (16 tokens of a head each), and the blocks that
// take them: one per item up to `most`; with one rotation per KV head a multiple of
// Hkv, a block then keeps to one head.
int64_t append_items(int n_tok, int Hkv) {
  return ((int64_t)n_tok + kItemRows - 1) / kItemRows * Hkv;
}
int append_blocks(int64_t items, int Hkv, int rph, int64_t most) {
  return (int)std::min(items, rph ? std::max<int64_t>(1, most / Hkv) * Hkv : most);
}

bool is_default(const QFmt& f) { return f.bf16 == 0 && f.quantile == 0 && f.ng == 4 && f.rph == 0; }

template <class Rows>
hipError_t launch_rows(void* pages, const Rows& rows, const float* Rk, const float* Rv,
                       float clip_k, float clip_v, QFmt fmt, hipStream_t st) {
  auto go = [&](auto kernel, int blocks, int waves) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, 2), dim3(waves * 64), 0, st,
                       static_cast<uint8_t*>(pages), rows, Rk, Rv, clip_k, clip_v, fmt);
  };
  const bool def = is_default(fmt);
  const int64_t items = append_items(rows.n_tok, rows.Hkv);
  if (items <= device_cus()) {
    if (def) go(append_kernel<Rows, true>, (int)items, kRotWaves);
    else go(append_kernel<Rows, false>, (int)items, kRotWaves);
  } else {
    const int blocks = append_blocks(items, rows.Hkv, fmt.rph, device_cus() / 2);
    if (def) go(append_bulk_kernel<Rows, true>, blocks, kBulkWaves);
    else go(append_bulk_kernel<Rows, false>, blocks, kBulkWaves);
  }
  return hipGetLastError();
}

template <class Rows>
hipError_t launch_prologue(void* pages, const Rows& rows, const float* Rk, const float* Rv,
                           float clip_k, float clip_v, QFmt fmt, const uint16_t* q, int B, int Hq,
                           float qscale, float* qt, hipStream_t st) {
  const int ab = append_blocks(append_items(rows.n_tok, rows.Hkv), rows.Hkv, fmt.rph, device_cus());
  const int B1 = std::min(B, launch_seqs(Hq));
  const int pb = query_blocks(B1, Hq, rows.Hkv, fmt.rph, kPrepRows);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(2 * ab + pb)), dim3(kRotWaves * 64), 0, st,
                       static_cast<uint8_t*>(pages), rows, Rk, Rv, clip_k, clip_v, fmt, ab, q,
                       B1 * Hq, Hq, qscale, qt);
  };
  if (is_default(fmt)) go(prologue_kernel<Rows, true>);
  else go(prologue_kernel<Rows, false>);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || B1 == B) return e;
  const size_t o = (size_t)B1 * Hq * kD;  // the other sequences' queries
  return launch_decode_prepare(q + o, B - B1, Hq, Rk, qscale, qt + o, st, fmt.rph, rows.Hkv);
}
}  // namespace

hipError_t launch_append(void* pages, int64_t Hkv, const uint16_t* k, const uint16_t* v,
                         const int64_t* slots, int n_tok, const float* Rk, const float* Rv,
                         float clip_k, float clip_v, QuantFmt fmt, hipStream_t st) {
  const PlainRows rows{k, v, slots, n_tok, (int)Hkv};
  return launch_rows(pages, rows, Rk, Rv, clip_k, clip_v, fmt, st);
}

hipError_t launch_mixed_append(void* pages, uint16_t* seg, int64_t Hkv, int S0, int W,
                               const uint16_t* k, const uint16_t* v, const int32_t* seq_idx,
                               const int64_t* pos, int n_tok, const int32_t* seq_lens,
                               const int32_t* block_table, int max_pages, const float* Rk,
                               const float* Rv, float clip_k, float clip_v, QuantFmt fmt,
                               hipStream_t st) {
  const PrefillRows rows{k, v, seg, seq_idx, pos, seq_lens, block_table, n_tok, (int)Hkv,
                         max_pages, S0, W};
  return launch_rows(pages, rows, Rk, Rv, clip_k, clip_v, fmt, st);
}

hipError_t launch_decode_prepare(const uint16_t* q, int B, int Hq, const float* Rk,
                                 float qscale, float* qt, hipStream_t st, int rph, int Hkv) {
  return by_seqs(B, launch_seqs(Hq), [&](int b0, int nb) {
    const size_t o = (size_t)b0 * Hq * kD;
    hipLaunchKernelGGL(prepare_kernel, dim3(query_blocks(nb, Hq, Hkv, rph, kPrepRows)),
                       dim3(kRotWaves * 64), 0, st, q + o, nb * Hq, Rk, qscale, qt + o, rph, Hq, Hkv);
    return hipGetLastError();
  });
}

hipError_t launch_step_prologue(void* pages, int64_t Hkv, const uint16_t* k, const uint16_t* v,
                                const int64_t* slots, int n_tok, const float* Rk,
                                const float* Rv, float clip_k, float clip_v, QuantFmt fmt,
                                const uint16_t* q, int B, int Hq, float qscale, float* qt,
                                hipStream_t st) {
  const PlainRows rows{k, v, slots, n_tok, (int)Hkv};
  return launch_prologue(pages, rows, Rk, Rv, clip_k, clip_v, fmt, q, B, Hq, qscale, qt, st);
}

hipError_t launch_mixed_step_prologue(void* pages, uint16_t* seg, int64_t Hkv, int S0, int W,
                                      const uint16_t* k, const uint16_t* v,
                                      const int32_t* seq_lens, const int32_t* block_table,
                                      int max_pages, const float* Rk, const float* Rv,
                                      float clip_k, float clip_v, QuantFmt fmt, const uint16_t* q,
                                      int B, int Hq, float qscale, float* qt, int num_splits,
                                      float* part_o, float* part_ml, hipStream_t st) {
  if (const int most = launch_seqs(Hq); B > most)
    return by_seqs(B, most, [&](int b0, int nb) {
      const size_t kv = (size_t)b0 * Hkv * kD, row = (size_t)b0 * Hq, part = row * (num_splits + 1);
      return launch_mixed_step_prologue(
          pages, seg ? seg + kv * 2 * (S0 + W) : nullptr, Hkv, S0, W, k + kv, v + kv, seq_lens + b0,
          block_table + (size_t)b0 * max_pages, max_pages, Rk, Rv, clip_k, clip_v, fmt, q + row * kD,
          nb, Hq, qscale, qt + row * kD, num_splits, part_o + part * kD, part_ml + part * 2, st);
    });
  const StepRows rows{k, v, seg, seq_lens, block_table, B, (int)Hkv, max_pages, S0, W};
  // Past 8 heads per KV head a CU holds one block of 8 waves, or two of at most 4.  With
  // no more than 4 chunks of 64 slots the partial's blocks then run in a launch of their
  // own, of as many waves as there are chunks, if a CU gets more than one.  A step of
  // 16/1 heads per KV head, S0 + W = 128, one launch / two: 32 sequences of 8 KV heads 66.4 /
  // 73.3 us, 48: 104.6 / 102.4, 64: 122.2 / 111.2, 256: 409 / 342; S0 + W = 320: 64
  // sequences 126.3 / 135.4.  Up to 8 heads one launch is faster at every size.
  if (Hq / (int)Hkv > 8 && S0 + W <= 4 * kP && (int64_t)B * Hkv > device_cus()) {
    const hipError_t e = launch_prologue(pages, rows, Rk, Rv, clip_k, clip_v, fmt, q, B, Hq, qscale, qt, st);
    if (e != hipSuccess) return e;
    return launch_seg_partial(seg, (int)Hkv, S0, W, B, Hq, seq_lens, max_pages, q, qscale, num_splits,
                              part_o, part_ml, st);
  }
  const SegArgs sa{seg, k, v, (int)Hkv, S0, W, Hq, seq_lens, max_pages, q, qscale, num_splits,
                   part_o, part_ml};
  const int ab = append_blocks(append_items(B, (int)Hkv), (int)Hkv, fmt.rph, device_cus());
  const int pb = query_blocks(B, Hq, (int)Hkv, fmt.rph, kPrepRows), sb = B * (int)Hkv;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)sb + (unsigned)(2 * ab + pb)), dim3(kRotWaves * 64), 0,
                       st, static_cast<uint8_t*>(pages), rows, Rk, Rv, clip_k, clip_v, fmt, ab, q,
                       B * Hq, Hq, qscale, qt, sa, sb);
  };
  const int g = Hq / (int)Hkv;
  if (is_default(fmt)) {
    if (g <= 4) go(mixed_prologue_kernel<4, true>);
    else if (g <= 8) go(mixed_prologue_kernel<8, true>);
    else go(mixed_prologue_kernel<16, true>);
  } else {
    if (g <= 4) go(mixed_prologue_kernel<4, false>);
    else if (g <= 8) go(mixed_prologue_kernel<8, false>);
    else go(mixed_prologue_kernel<16, false>);
  }
  return hipGetLastError();
}

hipError_t launch_clip_errors(const ClipTensor* tensors, int n_tensors, int64_t n_tok,
                              const float* cands, int n_cands, QuantFmt fmt, int Hkv,
                              hipStream_t st) {
  ClipJobs jobs{};
  for (int i = 0; i < n_tensors; ++i) {
    jobs.x[i] = tensors[i].x;
    jobs.R[i] = tensors[i].R;
    jobs.partial[i] = tensors[i].partial;
    jobs.err[i] = tensors[i].err;
    jobs.best[i] = tensors[i].best;
  }
  // one block per CU over all tensors, and no more than each has room for
  int64_t room = append_blocks(append_items((int)n_tok, Hkv), Hkv, fmt.rph, device_cus() / n_tensors);
  for (int i = 0; i < n_tensors; ++i) room = std::min(room, tensors[i].blocks);
  const int nb = (int)(fmt.rph ? room / Hkv * Hkv : room);
  if (nb < 1) return hipErrorInvalidValue;
  const bool few = append_items((int)n_tok, Hkv) <= 2 * (int64_t)nb;
  hipLaunchKernelGGL(few ? clip_err_kernel<true> : clip_err_kernel<false>,
                     dim3((unsigned)nb, (unsigned)n_tensors), dim3(kClipWaves * 64), 0, st, jobs,
                     (int)n_tok, cands, n_cands, fmt, Hkv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(clip_reduce_kernel, dim3((unsigned)n_tensors), dim3(kClipParts * kMaxClipCands),
                     0, st, jobs, nb, n_cands, cands, 1.0 / ((double)(n_tok * Hkv) * kD));
  return hipGetLastError();
}

int clip_blocks(int64_t n_rows, int Hkv, int rph) {
  const int64_t heads = rph ? Hkv : 1;  // rph: blocks per head, times Hkv
  const int64_t items = (n_rows / heads + 3) / 4;
  const int64_t cap = std::max<int64_t>(1, 4 * (int64_t)device_cus() / heads);
  return (int)(std::max<int64_t>(1, std::min(items, cap)) * heads);
}

}  // namespace oscar
