// fp32 products on the bf16 matrix cores of gfx950.
//
// An fp32 value is the sum of three bf16 terms, x = hi + mid + lo with
//   hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid),
// each rounded to nearest even: 8 significant bits a term, |mid| <= 2^-8 |x|,
// |lo| <= 2^-17 |x|, so the three terms hold all 24 bits (exactly, while lo is
// not subnormal: |x| above about 2e-34; below, the sum is off by at most half
// the smallest bf16 subnormal, 4.6e-41; above 3.39e38 hi overflows, and an
// infinite operand gives NaN where a plain fp32 product would give an infinity).
// Products of two bf16 values are exact in fp32, and of the nine term products
// of x y the three smallest (mid lo, lo mid, lo lo) are together at most
// 2^-24 |x y|, 2^-27.5 in the mean square over all mantissas: no more than the
// rounding of one fp32 product (2^-24, 2^-25.2).  Six products of
// v_mfma_f32_32x32x16_bf16, accumulated in fp32, therefore replace one fp32
// product at the accuracy of fp32 accumulation, at 16/6 of the rate of the
// fp32 matrix instructions (2,517 against 157 TFLOP/s dense).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sagips {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef unsigned short u16;

constexpr int kTerms = 3;

// Raw buffer resource over [base, base + bytes): reads past the end give 0.
__device__ __forceinline__ Rsrc split_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ bf16x8 split_load(Rsrc r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

// Two fp32 values -> packed bf16 pair (a in the low half), round to nearest even.
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// The three terms of a and b, packed in pairs.  The subtractions are exact; no
// contraction with whatever formed a or b.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&t)[kTerms]) {
#pragma clang fp contract(off)
  t[0] = pk_bf16(a, b);
  const float a1 = a - bf16_lo(t[0]), b1 = b - bf16_hi(t[0]);
  t[1] = pk_bf16(a1, b1);
  const float a2 = a1 - bf16_lo(t[1]), b2 = b1 - bf16_hi(t[1]);
  t[2] = pk_bf16(a2, b2);
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// c += A B over one K step of 16 for two accumulators that share the operand B:
// the five corrections, smallest first, into d (which may be c), then the hi hi
// products into c.  The two chains alternate, so that no product waits for the one
// just before it.
__device__ __forceinline__ void split_mfma2(const bf16x8 (&a0)[kTerms], const bf16x8 (&a1)[kTerms],
                                            const bf16x8 (&b)[kTerms], f32x16& c0, f32x16& c1, f32x16& d0, f32x16& d1) {
  constexpr int ta[5] = {2, 0, 1, 1, 0}, tb[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    d0 = mfma32(b[tb[p]], a0[ta[p]], d0);
    d1 = mfma32(b[tb[p]], a1[ta[p]], d1);
  }
  c0 = mfma32(b[0], a0[0], c0);
  c1 = mfma32(b[0], a1[0], c1);
}

// The same for MT accumulators, with the hi hi products in accumulators of their
// own (c), the five corrections in d: the full-size sum is then rounded once per
// K step instead of six times.  M comes from a, N from b; kSwap: the other way
// round.  kInit: the first step.
template <bool kInit, bool kSwap, int MT>
__device__ __forceinline__ void split_mfma_apart(const bf16x8 (&a)[MT][kTerms], const bf16x8 (&b)[kTerms],
                                                 f32x16 (&c)[MT], f32x16 (&d)[MT]) {
  constexpr int ta[5] = {2, 0, 1, 1, 0}, tb[5] = {0, 2, 1, 0, 1};
  const f32x16 zero = {};
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const f32x16 i = kInit ? zero : c[m];
    c[m] = kSwap ? mfma32(b[0], a[m][0], i) : mfma32(a[m][0], b[0], i);
  }
#pragma unroll
  for (int p = 0; p < 5; ++p)
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const f32x16 i = kInit && p == 0 ? zero : d[m];
      d[m] = kSwap ? mfma32(b[tb[p]], a[m][ta[p]], i) : mfma32(a[m][ta[p]], b[tb[p]], i);
    }
}

// Instruction order of a step of N products with other work beside them: a
// product occupies the matrix core for 32 cycles, in which the wave can issue
// seven more instructions.
template <int kVmem, int kValu, int N = 12>
__device__ __forceinline__ void interleave() {
  if (kVmem) __builtin_amdgcn_sched_group_barrier(0x20, kVmem, 0);    // vector memory reads
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                  // a product
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                // an LDS read
    __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);              // vector ALU
    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);                // an LDS write
  }
}

// Weight fragments.  Layer copies of an H x H matrix B[n][k] (n = output
// index): piece (nb, ks, term, lane) holds term `term` of B[32 nb + lane % 32]
// [16 ks + 8 (lane / 32) .. + 7], so that a wave reads one contiguous kilobyte
// per fragment.  The forward copy has B = W (n = out, k = in), the backward
// copy B = W^T.
constexpr size_t split_copy_bytes(int H) { return (size_t)H * H * 2 * kTerms; }

// One piece of 8 values, all three terms.
__device__ __forceinline__ void split_piece(const float (&v)[8], u16* out, int nb, int ks, int KS, int lane) {
  uint32_t t[4][kTerms];
#pragma unroll
  for (int q = 0; q < 4; ++q) split_pair(v[2 * q], v[2 * q + 1], t[q]);
#pragma unroll
  for (int s = 0; s < kTerms; ++s)
    *reinterpret_cast<uint4*>(out + ((size_t)((nb * KS + ks) * kTerms + s) * 64 + lane) * 8) =
        make_uint4(t[0][s], t[1][s], t[2][s], t[3][s]);
}

// Split activations in LDS: [term][feature][event] bf16, T events a row (a
// multiple of 64).  Of a 32 x 32 product with M = event, N = feature, a lane (half
// lh, column lr) holds one feature of events 8 g + 4 lh + 0..3.  A 16-byte unit of
// a row holds the 8 events that one lane half has of a 16-event step s (events
// 16 s + 4 lh + 0..3 and + 8..11), so that two accumulator groups are one store,
// and the K = events fragment of a weight gradient is one read in the order of the
// accumulators.  Unit u of feature f sits at u ^ swz(f): the 8 lanes (features)
// of a 16-byte access and the 4 x 4 lanes (features x half units) of a
// transposed read (K = features) hit distinct banks.
template <int H, int T>
struct SplitLds {
  static constexpr int RB = 2 * T;             // bytes of one feature's row of one term
  static constexpr int PL = H * RB;            // bytes of one term of a buffer
  static constexpr int BUF = kTerms * PL;

  struct Lane {
    int lane, lr, lh, wf, ew;                  // wave (wf, ew): features 32 wf .., events 64 ew ..
    uint32_t w[4];                             // unit 2 s + lh of row lr
    uint32_t tr[2][2];                         // [mt][j]: transposed read of events 32 mt .., features 8 lh + 4 j ..
  };
  static __device__ __forceinline__ uint32_t swz(int f) { return (uint32_t)(2 * (f & 3) + ((f >> 2) & 1)); }
  static __device__ __forceinline__ Lane make_lane(int wf, int ew) {
    Lane L;
    L.lane = threadIdx.x & 63;
    L.lr = L.lane & 31;
    L.lh = L.lane >> 5;
    L.wf = wf;
    L.ew = ew;
    const uint32_t erow = 128u * ew;           // the wave's events within a row
#pragma unroll
    for (int q = 0; q < 4; ++q) L.w[q] = (uint32_t)L.lr * RB + erow + (((uint32_t)(2 * q + L.lh) ^ swz(L.lr)) << 4);
    // transposed reads: lane i of 16-lane group g addresses feature row
    // 8 (g / 2) + 4 j + i / 4, events 32 mt + 16 (g % 2) + 4 (i % 4) .. + 3, which
    // are half i % 4 / 2 of unit 2 (2 mt + g % 2) + i % 2
    const int g = L.lane >> 4, i = L.lane & 15;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int f = 8 * (g >> 1) + 4 * j + (i >> 2);
        const uint32_t u = 2 * (2 * mt + (g & 1)) + (i & 1);
        L.tr[mt][j] = (uint32_t)f * RB + erow + ((u ^ swz(f)) << 4) + 8 * ((i >> 1) & 1);
      }
    return L;
  }

  // Terms of the K = features operand of one 32-event block and K step.
  static __device__ __forceinline__ void read_tr(const char* buf, const Lane& L, int mt, int ks, bf16x8 (&a)[kTerms]) {
#pragma unroll
    for (int t = 0; t < kTerms; ++t) {
      const int o = t * PL + ks * 16 * RB;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(buf + L.tr[mt][0] + o));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(buf + L.tr[mt][1] + o));
      a[t] = bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
  }
  // Terms of the K = events operand: columns 32 kb + lr, step s.
  static __device__ __forceinline__ void read_ev(const char* buf, const Lane& L, int kb, int s, bf16x8 (&b)[kTerms]) {
#pragma unroll
    for (int t = 0; t < kTerms; ++t) b[t] = *reinterpret_cast<const bf16x8*>(buf + L.w[s] + t * PL + kb * 32 * RB);
  }

  // Terms of a step (16 events) of the lane's feature: packed pairs of events.
  typedef uint32_t Step[kTerms][4];
  // Half u of a step: 4 events.
  static __device__ __forceinline__ void split4(const float (&v)[4], int u, Step& d) {
    uint32_t t0[kTerms], t1[kTerms];
    split_pair(v[0], v[1], t0);
    split_pair(v[2], v[3], t1);
#pragma unroll
    for (int t = 0; t < kTerms; ++t) {
      d[t][2 * u] = t0[t];
      d[t][2 * u + 1] = t1[t];
    }
  }
  // A step of the wave's features into a buffer.
  static __device__ __forceinline__ void store_step(char* buf, const Lane& L, int s, const Step& d) {
#pragma unroll
    for (int t = 0; t < kTerms; ++t)
      *reinterpret_cast<uint4*>(buf + L.w[s] + t * PL + L.wf * 32 * RB) = make_uint4(d[t][0], d[t][1], d[t][2], d[t][3]);
  }
};

// Cross-lane sums without LDS traffic (DPP within a row of 16 lanes, then the
// permlane swaps).  kCtrl: 0xB1 = quad_perm xor 1, 0x1B = quad_perm xor 3,
// 0x141 = row_half_mirror (xor 7), 0x140 = row_mirror (xor 15).
template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
// Sum over the 16 lanes of a row, in every lane.
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x1B>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  return v;
}
// v + (the value of the lane 16 away within a half) / (32 away).
__device__ __forceinline__ float add_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sums of 32 values over the 32 lanes of a wave half, halving the values a
// lane keeps at each step: lane lr of the half gets the total of v[lr].
__device__ __forceinline__ float half_scatter_sum(float (&v)[32], int lr) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 16]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool up = lr & 8;
    v[i] = (up ? v[i + 8] : v[i]) + dpp_move<0x140>(up ? v[i] : v[i + 8]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool up = lr & 4;
    v[i] = (up ? v[i + 4] : v[i]) + dpp_move<0x141>(up ? v[i] : v[i + 4]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool up = lr & 2;
    v[i] = (up ? v[i + 2] : v[i]) + dpp_move<0x1B>(up ? v[i] : v[i + 2]);
  }
  const bool up = lr & 1;
  return (up ? v[1] : v[0]) + dpp_move<0xB1>(up ? v[0] : v[1]);
}
// Sum over the wave, in every lane; the same order on every call.
__device__ __forceinline__ float wave_total(float v) { return add_xor32(add_xor16(row_sum(v))); }

// Sums of four values over the wave: lanes 0..15 get the total of v0, 16..31 of
// v1, 32..47 of v2, 48..63 of v3.
__device__ __forceinline__ float wave_scatter_sum4(float v0, float v1, float v2, float v3) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v2), false, false);
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v1), __float_as_uint(v3), false, false);
  const float a = __uint_as_float(r[0]) + __uint_as_float(r[1]), b = __uint_as_float(t[0]) + __uint_as_float(t[1]);
  const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return row_sum(__uint_as_float(u[0]) + __uint_as_float(u[1]));
}

}  // namespace sagips
