// The GAN generator (noise -> parameters) of Sec. III, for a stack of M
// members of the same shape, and the ensemble response of Sec. VI-A.
//
// Network: IN -> H -> (H -> H) x NH -> OUT, LeakyReLU on the hidden layers,
// theta = 1 + softplus(last layer), so that every shape parameter is above 1.
// The paper's generator (51,206 parameters) is 6 -> 128 x 4 -> 6, i.e.
// H = 128, NH = 3.  Member m's parameters sit at W[l] + m * |W[l]|.
//
// Row tiles: T = 64 rows of the noise batch, or 16 when 64-row tiles of all
// members would leave most CUs idle (a single generator on 1,024 rows).
//
// Forward, 64-row tiles: one workgroup of 4 waves per (tile, member); the H x H
// products run on the bf16 matrix cores from split operands (split_bf16.hpp; see
// GenFwd).  16-row tiles take the forward pass below instead: with few tiles the
// time is one tile's latency, which splitting the weights lengthens (1,024 rows,
// one member: 12.9 us on 64 workgroups, 14.9 us split on 32).
//
// Backward (and the 16-row forward): one workgroup of 8 waves per (tile, member).
// The backward kernel recomputes the tile's forward pass (cheaper than storing it): the
// activations A_1 .. A_{NH+1} live in LDS as [T][H+4] fp32; the H x H products run on the fp32
// matrix cores (v_mfma_f32_16x16x4_f32) as out^T = W * in^T, each wave owning 16
// output features of all T rows.  The first layer (K = IN) and the last (N = OUT)
// are VALU work.  Then the backward pass from dL/dtheta: each backward signal
// overwrites the activation it replaces.  Weight gradients of the tile go to a
// per-tile partial; a second kernel sums the partials over tiles in a fixed
// order, so results are deterministic.
#include "device_math.hpp"
#include "kernels.hpp"
#include "split_bf16.hpp"

#include <string.h>

namespace sagips {
namespace {

constexpr int kGThreads = 512;   // 8 waves
constexpr int kGMaxIO = 8;       // largest IN / OUT

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float g_leaky(float v, float s) { return v > 0.0f ? v : s * v; }
__device__ __forceinline__ float g_leaky_grad(float h, float s) { return h > 0.0f ? 1.0f : s; }
__device__ __forceinline__ float g_softplus(float t) { return fmaxf(t, 0.0f) + log1pf(expf(-fabsf(t))); }
__device__ __forceinline__ float g_sigmoid(float t) { return 1.0f / (1.0f + expf(-t)); }

// Workgroups are numbered L = x + y * gridDim.x and dealt to the 8 XCDs in
// turn (XCD = L mod 8); each XCD has its own L2.  The first 8 * floor(M / 8)
// members are placed so that all tiles of a member run on one XCD (member =
// 8 (j / tiles) + L mod 8, tile = j mod tiles, j = L / 8), so its weights are
// fetched into one L2 only; the remaining members are laid out in order.
__device__ __forceinline__ void gen_block(int tiles, int members, int& m, int& tile) {
  const int L = blockIdx.x + blockIdx.y * gridDim.x;
  const int m8 = members - members % 8;
  if (L < tiles * m8) {
    const int j = L >> 3;
    m = 8 * (j / tiles) + (L & 7);
    tile = j % tiles;
  } else {
    const int r = L - tiles * m8;
    m = m8 + r / tiles;
    tile = r % tiles;
  }
}

struct GenParams {
  const float* W[kMaxGenLayers];   // layer l of member 0; member m at + m * wsz[l]
  const float* b[kMaxGenLayers];
  int64_t wsz[kMaxGenLayers], bsz[kMaxGenLayers];
  int in, out;
  int64_t k;                       // rows of the noise batch
  float slope;
  const float* noise;              // [k][in], shared by every member
  float* theta;                    // forward: [M][k][out]
  const float* dtheta;             // backward: [M][k][out]
  float* part;                     // backward: [M][tiles][P]
  int64_t P;                       // floats per partial (all parameters of one member)
  int64_t poff_w[kMaxGenLayers], poff_b[kMaxGenLayers];
};

template <int H, int NH, int kGT>
struct Gen {
  static constexpr int LD = H + 4;
  static constexpr int WAVES = kGThreads / 64;
  static constexpr int KB = H / 16;
  static constexpr int CB = kGT / 16;
  static_assert(kGT == 16 || kGT == 64, "row tile");
  static constexpr int PPO = kGThreads / H;     // threads per feature in the VALU loops
  static_assert(H == 16 * WAVES, "one wave per 16 features");

  struct Smem {
    float act[NH + 1][kGT][LD];
    float n[kGT][kGMaxIO];
    float o[kGT][kGMaxIO];     // last-layer pre-activation
    float dout[kGT][kGMaxIO];  // dL/d(pre-activation of the last layer)
  };

  // out^T (16 features of this wave x 64 rows) = W[o][k] in[ev][k]; W row-major [H][H].
  static __device__ __forceinline__ void gemm_fwd(const float* __restrict__ W, const float* in, f32x4 (&acc)[CB],
                                                  int o0, int lr, int lg) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* wrow = W + (o0 + lr) * H + 4 * lg;
#pragma unroll 2
    for (int kb = 0; kb < KB; ++kb) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(wrow + 16 * kb);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const f32x4 bv = *reinterpret_cast<const f32x4*>(in + (16 * cb + lr) * LD + 16 * kb + 4 * lg);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[cb] = mfma4(a[s], bv[s], acc[cb]);
      }
    }
  }

  // out^T (16 input features k of this wave x 64 rows) = sum_o W[o][k] dl[ev][o]:
  // the backward-data product, reading W column-wise.
  static __device__ __forceinline__ void gemm_bwd(const float* __restrict__ W, const float* dl, f32x4 (&acc)[CB],
                                                  int k0, int lr, int lg) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int kb = 0; kb < KB; ++kb) {
      const int o = 16 * kb + 4 * lg;
      f32x4 a;
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = W[(o + s) * H + k0 + lr];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const f32x4 bv = *reinterpret_cast<const f32x4*>(dl + (16 * cb + lr) * LD + o);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[cb] = mfma4(a[s], bv[s], acc[cb]);
      }
    }
  }

  // Forward pass of member m on rows [row0, row0 + 64) into LDS; rows past k
  // carry zero noise.  Leaves A_1..A_{NH+1} in act and the last layer's
  // pre-activation in o.
  static __device__ void forward(const GenParams& p, Smem& sm, int m, int64_t row0) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const float slope = p.slope;
    for (int i = tid; i < kGT * kGMaxIO; i += kGThreads) {
      const int ev = i / kGMaxIO, j = i % kGMaxIO;
      const int64_t r = row0 + ev;
      sm.n[ev][j] = (j < p.in && r < p.k) ? p.noise[r * p.in + j] : 0.0f;
    }
    __syncthreads();
    {   // first layer: thread (feature o, part) over rows part, part + PPO, ...
      const int o = tid % H, part = tid / H;
      const float* W0 = p.W[0] + m * p.wsz[0];
      float w[kGMaxIO];
#pragma unroll
      for (int j = 0; j < kGMaxIO; ++j) w[j] = j < p.in ? W0[o * p.in + j] : 0.0f;
      const float bias = p.b[0][m * p.bsz[0] + o];
      for (int ev = part; ev < kGT; ev += PPO) {
        float v = bias;
#pragma unroll
        for (int j = 0; j < kGMaxIO; ++j) v = fmaf(w[j], sm.n[ev][j], v);
        sm.act[0][ev][o] = g_leaky(v, slope);
      }
    }
    __syncthreads();
    const int o0 = 16 * wave;
#pragma unroll
    for (int l = 0; l < NH; ++l) {
      f32x4 acc[CB];
      gemm_fwd(p.W[1 + l] + m * p.wsz[1 + l], &sm.act[l][0][0], acc, o0, lr, lg);
      const int o = o0 + 4 * lg;
      const f32x4 bias = *reinterpret_cast<const f32x4*>(p.b[1 + l] + m * p.bsz[1 + l] + o);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        f32x4 v = acc[cb] + bias;
        v.x = g_leaky(v.x, slope); v.y = g_leaky(v.y, slope);
        v.z = g_leaky(v.z, slope); v.w = g_leaky(v.w, slope);
        *reinterpret_cast<f32x4*>(&sm.act[l + 1][16 * cb + lr][o]) = v;
      }
      __syncthreads();
    }
    if ((tid >> 3) < kGT) {   // last layer: thread (row ev, part) sums features 4 part + 32 c (c < H / 32)
      const int ev = tid >> 3, part = tid & 7;
      const float* Wl = p.W[NH + 1] + m * p.wsz[NH + 1];
      const float* hrow = &sm.act[NH][ev][0];
      for (int j = 0; j < p.out; ++j) {
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < H / 32; ++c) {
          const int f = 4 * part + 32 * c;
          const f32x4 hv = *reinterpret_cast<const f32x4*>(hrow + f);
          const f32x4 wv = *reinterpret_cast<const f32x4*>(Wl + j * H + f);
          z = fmaf(hv.x, wv.x, z); z = fmaf(hv.y, wv.y, z);
          z = fmaf(hv.z, wv.z, z); z = fmaf(hv.w, wv.w, z);
        }
#pragma unroll
        for (int s = 1; s < 8; s <<= 1) z += __shfl_xor(z, s, 64);
        if (part == 0) sm.o[ev][j] = z + p.b[NH + 1][m * p.bsz[NH + 1] + j];
      }
    }
    __syncthreads();
  }

  static __device__ void run_forward(const GenParams& p) {
    __shared__ Smem sm;
    int m, tile;
    gen_block(gridDim.x, gridDim.y, m, tile);
    const int64_t row0 = (int64_t)tile * kGT;
    forward(p, sm, m, row0);
    for (int i = threadIdx.x; i < kGT * p.out; i += kGThreads) {
      const int ev = i / p.out, j = i % p.out;
      const int64_t r = row0 + ev;
      if (r < p.k) p.theta[((int64_t)m * p.k + r) * p.out + j] = 1.0f + g_softplus(sm.o[ev][j]);
    }
  }

  static __device__ void run_backward(const GenParams& p) {
    __shared__ Smem sm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    int m, tile;
    gen_block(gridDim.x, gridDim.y, m, tile);
    const int64_t row0 = (int64_t)tile * kGT;
    const float slope = p.slope;
    forward(p, sm, m, row0);
    float* part = p.part + ((int64_t)m * gridDim.x + tile) * p.P;

    // dL/d(last pre-activation) = dL/dtheta * sigmoid(o); zero on rows past k
    for (int i = tid; i < kGT * kGMaxIO; i += kGThreads) {
      const int ev = i / kGMaxIO, j = i % kGMaxIO;
      const int64_t r = row0 + ev;
      float d = 0.f;
      if (j < p.out && r < p.k) d = p.dtheta[((int64_t)m * p.k + r) * p.out + j] * g_sigmoid(sm.o[ev][j]);
      sm.dout[ev][j] = d;
    }
    __syncthreads();
    const int L = NH + 1;   // index of the last layer
    const float* WL = p.W[L] + m * p.wsz[L];
    {   // last layer: dW[j][k] = sum_ev dout[ev][j] A_{NH+1}[ev][k]; db[j] = sum_ev dout[ev][j]
      const int k = tid % H, g = tid / H;
      for (int j = g; j < p.out; j += PPO) {
        float s = 0.f;
        for (int ev = 0; ev < kGT; ++ev) s = fmaf(sm.dout[ev][j], sm.act[NH][ev][k], s);
        part[p.poff_w[L] + j * H + k] = s;
      }
      if (tid < p.out) {
        float s = 0.f;
        for (int ev = 0; ev < kGT; ++ev) s += sm.dout[ev][tid];
        part[p.poff_b[L] + tid] = s;
      }
    }
    __syncthreads();
    {   // delta_{NH+1} = (dout W_L) * leaky'(A_{NH+1}), in place
      const int k = tid % H, g = tid / H;
      float w[kGMaxIO];
#pragma unroll
      for (int j = 0; j < kGMaxIO; ++j) w[j] = j < p.out ? WL[j * H + k] : 0.0f;
      for (int ev = g; ev < kGT; ev += PPO) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < kGMaxIO; ++j) s = fmaf(sm.dout[ev][j], w[j], s);
        float& h = sm.act[NH][ev][k];
        h = s * g_leaky_grad(h, slope);
      }
    }
    __syncthreads();
    const int o0 = 16 * wave;
#pragma unroll
    for (int l = NH - 1; l >= 0; --l) {
      // layer 1 + l maps A_{l+1} (act[l]) -> A_{l+2}; its output signal delta_{l+2} is in act[l+1]
      const float* dl = &sm.act[l + 1][0][0];
      float* A = &sm.act[l][0][0];
      {   // dW[o][k] = sum_ev delta[ev][o] A[ev][k]: rows o0.., 8 column blocks, K = 64 rows
        f32x4 acc[KB];
#pragma unroll
        for (int nb = 0; nb < KB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int q = 0; q < kGT / 4; ++q) {
          const int ev = 4 * q + lg;
          const float a = dl[ev * LD + o0 + lr];
#pragma unroll
          for (int nb = 0; nb < KB; ++nb) acc[nb] = mfma4(a, A[ev * LD + 16 * nb + lr], acc[nb]);
        }
        float* dW = part + p.poff_w[1 + l];
#pragma unroll
        for (int nb = 0; nb < KB; ++nb)
#pragma unroll
          for (int r = 0; r < 4; ++r) dW[(o0 + 4 * lg + r) * H + 16 * nb + lr] = acc[nb][r];
        if (tid < H) {
          float s = 0.f;
          for (int ev = 0; ev < kGT; ++ev) s += dl[ev * LD + tid];
          part[p.poff_b[1 + l] + tid] = s;
        }
      }
      __syncthreads();   // delta_{l+1} overwrites A_{l+1}, which every wave just read
      f32x4 acc[CB];
      gemm_bwd(p.W[1 + l] + m * p.wsz[1 + l], dl, acc, o0, lr, lg);
      const int k = o0 + 4 * lg;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int ev = 16 * cb + lr;
        f32x4 h = *reinterpret_cast<const f32x4*>(A + ev * LD + k);
        f32x4 v = acc[cb];
        v.x *= g_leaky_grad(h.x, slope); v.y *= g_leaky_grad(h.y, slope);
        v.z *= g_leaky_grad(h.z, slope); v.w *= g_leaky_grad(h.w, slope);
        *reinterpret_cast<f32x4*>(A + ev * LD + k) = v;
      }
      __syncthreads();
    }
    {   // first layer: dW[o][j] = sum_ev delta_1[ev][o] n[ev][j]; db[o] = sum_ev delta_1[ev][o]
      const int o = tid % H, g = tid / H;
      for (int j = g; j < p.in; j += PPO) {
        float s = 0.f;
        for (int ev = 0; ev < kGT; ++ev) s = fmaf(sm.act[0][ev][o], sm.n[ev][j], s);
        part[p.poff_w[0] + o * p.in + j] = s;
      }
      if (g == 0) {
        float s = 0.f;
        for (int ev = 0; ev < kGT; ++ev) s += sm.act[0][ev][o];
        part[p.poff_b[0] + o] = s;
      }
    }
  }
};

template <int H, int NH, int T>
__global__ __launch_bounds__(kGThreads, 1) void k_gen_backward(GenParams p) {
  Gen<H, NH, T>::run_backward(p);
}

template <int H, int NH>
__global__ __launch_bounds__(kGThreads, 1) void k_gen_forward16(GenParams p) {
  Gen<H, NH, 16>::run_forward(p);
}

// Forward pass on the bf16 matrix cores, H = 128.  Wave w owns features [32 w,
// 32 w + 32) of every layer for all 64 rows of the tile.  The activations live
// in LDS split (SplitLds) and are overwritten layer by layer, two barriers a
// layer; 52 KB, so three workgroups share a CU and the vector work of one runs
// beside the products of the others.  A member's weights are split as they are read: 8 values per
// lane and K step, between the products of the step before (44 instructions
// against 12 products of 32 cycles), which saves the pass over all members that
// a split copy would need.  The last hidden layer is formed with M = feature, so
// that a lane holds 16 features of its own rows and the output layer (N = OUT)
// needs only one exchange between the wave's halves and one between the waves.
// Bound by the matrix cores and the vector ALU together.  100 members x 1,024
// rows: 138 us with fp32 matrix instructions, 74 us now.
constexpr int kFwdThreads = 256;

template <int NH>
struct GenFwd : SplitLds<128, 64> {
  static constexpr int H = 128, KS = H / 16, MT = 2, R = 32 * MT, WAVES = 4, PD = 2;
  static_assert(WAVES * 32 == H && WAVES * 64 == kFwdThreads, "one wave per 32 features");

  struct Smem {
    union {
      char act[BUF];
      float op[WAVES][kGMaxIO][64];    // last layer: partials over a wave's features
    };
    union {
      float n[kGMaxIO][64];            // noise, transposed
      float wl[kGMaxIO][H];            // last layer's weights
    };
  };

  // 8 weights of row 32 wf + lr, columns 16 ks + 8 lh .. + 7.
  typedef f32x4 Raw[2];
  static __device__ __forceinline__ void split_raw(const Raw& r, bf16x8 (&w)[kTerms]) {
    uint32_t t[4][kTerms];
#pragma unroll
    for (int q = 0; q < 4; ++q) split_pair(r[q >> 1][2 * (q & 1)], r[q >> 1][2 * (q & 1) + 1], t[q]);
#pragma unroll
    for (int k = 0; k < kTerms; ++k) w[k] = __builtin_bit_cast(bf16x8, make_uint4(t[0][k], t[1][k], t[2][k], t[3][k]));
  }

  // acc[m] = act W^T for the wave's features and rows 32 m .. (kSwap: M = feature,
  // N = row).
  template <bool kSwap>
  static __device__ __forceinline__ void product(const float* __restrict__ W, const char* buf, const Lane& L,
                                                 f32x16 (&acc)[MT]) {
    const float* wrow = W + (32 * L.wf + L.lr) * H + 8 * L.lh;
    f32x16 corr[MT];
    Raw raw[PD + 1];
    bf16x8 w[2][kTerms], a[2][MT][kTerms];
    auto load = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2; ++q) raw[ks % (PD + 1)][q] = *reinterpret_cast<const f32x4*>(wrow + 16 * ks + 4 * q);
    };
#pragma unroll
    for (int q = 0; q < PD; ++q) load(q);
#pragma unroll
    for (int m = 0; m < MT; ++m) read_tr(buf, L, m, 0, a[0][m]);
    split_raw(raw[0], w[0]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      __builtin_amdgcn_sched_barrier(0);
      if (ks + PD < KS) load(ks + PD);
      if (ks + 1 < KS) {
#pragma unroll
        for (int m = 0; m < MT; ++m) read_tr(buf, L, m, ks + 1, a[(ks + 1) & 1][m]);
        split_raw(raw[(ks + 1) % (PD + 1)], w[(ks + 1) & 1]);
      }
      if (ks == 0) split_mfma_apart<true, kSwap>(a[0], w[0], acc, corr);
      else split_mfma_apart<false, kSwap>(a[ks & 1], w[ks & 1], acc, corr);
      interleave<2, 8 / MT, 6 * MT>();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] += corr[m];
  }

  // A_1 of the wave's features (in <= J).
  template <int J>
  static __device__ __forceinline__ void first_layer(const GenParams& p, Smem& sm, int m, const Lane& L) {
    const int fo = 32 * L.wf + L.lr;
    const float* W0 = p.W[0] + m * p.wsz[0];
    float w[J];
#pragma unroll
    for (int j = 0; j < J; ++j) w[j] = j < p.in ? W0[fo * p.in + j] : 0.0f;
    const float bias = p.b[0][m * p.bsz[0] + fo];
#pragma unroll
    for (int s = 0; s < 2 * MT; ++s) {
      Step d;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x4 v = {bias, bias, bias, bias};
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(&sm.n[j][16 * s + 8 * u + 4 * L.lh]);
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = fmaf(w[j], x[q], v[q]);
        }
        const float h[4] = {g_leaky(v.x, p.slope), g_leaky(v.y, p.slope), g_leaky(v.z, p.slope), g_leaky(v.w, p.slope)};
        split4(h, u, d);
      }
      store_step(sm.act, L, s, d);
    }
  }

  static __device__ void run(const GenParams& p) {
    __shared__ __attribute__((aligned(1024))) Smem sm;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Lane L = make_lane(wave, 0);
    int m, tile;
    gen_block(gridDim.x, gridDim.y, m, tile);
    const int64_t row0 = (int64_t)tile * R;
    const float slope = p.slope;
    for (int i = tid; i < R * kGMaxIO; i += kFwdThreads) {
      const int ev = i % R, j = i / R;
      const int64_t r = row0 + ev;
      sm.n[j][ev] = (j < p.in && r < p.k) ? p.noise[r * p.in + j] : 0.0f;
    }
    __syncthreads();
    if (p.in <= 6) first_layer<6>(p, sm, m, L);
    else first_layer<kGMaxIO>(p, sm, m, L);
    __syncthreads();
    const float* WL = p.W[NH + 1] + m * p.wsz[NH + 1];
    for (int i = tid; i < p.out * H; i += kFwdThreads) sm.wl[i / H][i % H] = WL[i];
    f32x16 acc[MT];
#pragma unroll 1
    for (int l = 0; l < NH - 1; ++l) {
      const float bias = p.b[1 + l][m * p.bsz[1 + l] + 32 * L.wf + L.lr];
      product<false>(p.W[1 + l] + m * p.wsz[1 + l], sm.act, L, acc);
      __syncthreads();                           // every wave is done reading this layer's input
#pragma unroll
      for (int s = 0; s < 2 * MT; ++s) {
        Step d;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float h[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) h[q] = g_leaky(acc[s >> 1][8 * (s & 1) + 4 * u + q] + bias, slope);
          split4(h, u, d);
        }
        store_step(sm.act, L, s, d);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    }
    // last hidden layer: lane = row 32 m + lr, register i = feature 32 wf + 8 (i / 4) + 4 lh + i % 4
    product<true>(p.W[NH] + m * p.wsz[NH], sm.act, L, acc);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 bias = *reinterpret_cast<const f32x4*>(p.b[NH] + m * p.bsz[NH] + 32 * L.wf + 8 * g + 4 * L.lh);
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][4 * g + q] = g_leaky(acc[t][4 * g + q] + bias[q], slope);
    }
    __syncthreads();                             // act is read, wl staged
    for (int j = 0; j < p.out; ++j) {
      float z[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) z[t] = 0.f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 wv = *reinterpret_cast<const f32x4*>(&sm.wl[j][32 * L.wf + 8 * g + 4 * L.lh]);
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q) z[t] = fmaf(acc[t][4 * g + q], wv[q], z[t]);
      }
      // both halves' features; lanes 0..31 keep rows 0..31
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[0]), __float_as_uint(z[1]), false, false);
      sm.op[wave][j][L.lane] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    __syncthreads();
    for (int i = tid; i < R * p.out; i += kFwdThreads) {
      const int ev = i / p.out, j = i % p.out;
      const int64_t r = row0 + ev;
      float o = p.b[NH + 1][m * p.bsz[NH + 1] + j];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) o += sm.op[w][j][ev];
      if (r < p.k) p.theta[((int64_t)m * p.k + r) * p.out + j] = 1.0f + g_softplus(o);
    }
  }
};

template <int NH>
__global__ __launch_bounds__(kFwdThreads, 3) void k_gen_forward(GenParams p) {
  GenFwd<NH>::run(p);
}

// Sum of the per-tile partials of member blockIdx.y in a fixed order, scattered
// to the caller's gradient arrays.
struct GenReduceArgs {
  const float* part;
  int64_t P;
  int tiles;
  int n_layers;
  int64_t poff_w[kMaxGenLayers], poff_b[kMaxGenLayers], wsz[kMaxGenLayers], bsz[kMaxGenLayers];
  float* dW[kMaxGenLayers];
  float* db[kMaxGenLayers];
};

// s += the values of tiles t, t + S, ..., up to N of them, loaded together.
template <int S, int N>
__device__ __forceinline__ void add_tiles(const float* src, int t, int tiles, int64_t P, float& s) {
  float x[N];
#pragma unroll
  for (int u = 0; u < N; ++u) x[u] = src[(int64_t)min(t + u * S, tiles - 1) * P];
#pragma unroll
  for (int u = 0; u < N; ++u) s += t + u * S < tiles ? x[u] : 0.f;
}

// S tile slices summed side by side, then combined in order: four, or one where there are
// no more tiles than that (the same sum; four slices then are blocks of mostly idle waves:
// 300 members of one tile 134 us against 69, 100 members 47 against 25).  Eight tiles'
// loads in flight (one by one, 16 tiles a slice are 16 round trips), and fewer for a last
// group that is shorter; a slice is a whole number of waves, so that no branch diverges.
template <int S>
__global__ __launch_bounds__(256) void k_gen_reduce(GenReduceArgs r) {
  constexpr int C = 256 / S;
  const int m = blockIdx.y;
  const int le = threadIdx.x % C, sl = threadIdx.x / C;
  const int64_t e = (int64_t)blockIdx.x * C + le;
  float v = 0.f;
  if (e < r.P) {
    const float* src = r.part + (int64_t)m * r.tiles * r.P + e;
    int t = sl;
    for (; t + 4 * S < r.tiles; t += 8 * S) add_tiles<S, 8>(src, t, r.tiles, r.P, v);
    if (t + 2 * S < r.tiles) add_tiles<S, 4>(src, t, r.tiles, r.P, v);
    else if (t < r.tiles) add_tiles<S, 2>(src, t, r.tiles, r.P, v);
  }
  if constexpr (S > 1) {
    __shared__ float red[S][C];
    red[sl][le] = v;
    __syncthreads();
    if (sl != 0) return;
    v = 0.f;
#pragma unroll
    for (int q = 0; q < S; ++q) v += red[q][le];
  }
  if (e >= r.P) return;
  for (int l = 0; l < r.n_layers; ++l) {
    if (e >= r.poff_w[l] && e < r.poff_w[l] + r.wsz[l]) { r.dW[l][m * r.wsz[l] + (e - r.poff_w[l])] = v; return; }
    if (e >= r.poff_b[l] && e < r.poff_b[l] + r.bsz[l]) { r.db[l][m * r.bsz[l] + (e - r.poff_b[l])] = v; return; }
  }
}

// Ensemble statistics of theta[M][k][out]: per (row, component) the member
// mean and the population standard deviation about it; rowstat[0][r][c] = mean,
// rowstat[1][r][c] = sigma.  A block has 16 (row, component) pairs side by side,
// so that a load is 64 contiguous bytes of a member, and 16 slices of the members:
// slice j takes members j, j + 16, ..., and the sixteen partial sums are added in
// a fixed tree.  A slice's first kEnsKeep members are loaded together and kept for
// the second pass, so that up to 128 members are one round trip to memory (100
// members on 1,024 rows, with k_ens_final's 1,024 threads: 79.7 -> 76.3 us a call
// of the ensemble response).
constexpr int kEnsCols = 16, kEnsSlices = 16, kEnsKeep = 8;

__global__ __launch_bounds__(256) void k_ens_rows(const float* __restrict__ theta, int M, int64_t k, int out,
                                                  float* __restrict__ rowstat) {
  __shared__ float red[2][4][kEnsCols];
  const int il = threadIdx.x % kEnsCols, j = threadIdx.x / kEnsCols, wave = threadIdx.x >> 6;
  const int64_t stride = k * out;
  const int64_t i = (int64_t)blockIdx.x * kEnsCols + il;
  const float* src = theta + min(i, stride - 1);
  // over the slices: 2 bits within a wave, 2 across the waves
  auto total = [&](float v, int pass) __attribute__((always_inline)) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if ((threadIdx.x & 63) < kEnsCols) red[pass][wave][il] = v;
    __syncthreads();
    return (red[pass][0][il] + red[pass][1][il]) + (red[pass][2][il] + red[pass][3][il]);
  };
  float x[kEnsKeep];
#pragma unroll
  for (int u = 0; u < kEnsKeep; ++u) x[u] = src[min(j + u * kEnsSlices, M - 1) * stride];
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < kEnsKeep; ++u) s += j + u * kEnsSlices < M ? x[u] : 0.f;
#pragma unroll 4
  for (int m = j + kEnsKeep * kEnsSlices; m < M; m += kEnsSlices) s += src[m * stride];
  const float mean = total(s, 0) / (float)M;
  float q = 0.f;
#pragma unroll
  for (int u = 0; u < kEnsKeep; ++u) {
    const float dv = j + u * kEnsSlices < M ? x[u] - mean : 0.f;
    q = fmaf(dv, dv, q);
  }
#pragma unroll 4
  for (int m = j + kEnsKeep * kEnsSlices; m < M; m += kEnsSlices) {
    const float dv = src[m * stride] - mean;
    q = fmaf(dv, dv, q);
  }
  q = total(q, 1);
  if (i < stride && j == 0) {
    rowstat[i] = mean;
    rowstat[stride + i] = sqrtf(q / (float)M);
  }
}

// Batch averages of the row statistics (one workgroup): thread (component
// c, slice q) sums rows q, q + 128, ... of component c (out <= 8); the 128
// slices of a component are then added in a fixed tree.
constexpr int kEnsFinal = 1024;

__global__ __launch_bounds__(kEnsFinal) void k_ens_final(const float* __restrict__ rowstat, int64_t k, int out,
                                                   const float* __restrict__ p_true, float* __restrict__ p_hat,
                                                   float* __restrict__ sigma, float* __restrict__ r_hat) {
  constexpr int kSlices = kEnsFinal / kGMaxIO;   // 128
  __shared__ float red[2][kSlices][kGMaxIO];
  const int c = threadIdx.x % kGMaxIO, q = threadIdx.x / kGMaxIO;
  float a = 0.f, b = 0.f;
  if (c < out) {
    // unrolled so that eight rows' loads are in flight at once (the adds keep
    // their order)
#pragma unroll 8
    for (int64_t r = q; r < k; r += kSlices) {
      a += rowstat[r * out + c];
      b += rowstat[k * out + r * out + c];
    }
  }
  red[0][q][c] = a;
  red[1][q][c] = b;
  __syncthreads();
  for (int w = kSlices / 2; w > 0; w >>= 1) {
    if (q < w) {
      red[0][q][c] += red[0][q + w][c];
      red[1][q][c] += red[1][q + w][c];
    }
    __syncthreads();
  }
  if (q == 0 && c < out) {
    const float ph = red[0][0][c] / (float)k;
    p_hat[c] = ph;
    sigma[c] = red[1][0][c] / (float)k;
    if (r_hat) r_hat[c] = (p_true[c] - ph) / p_true[c];
  }
}

struct GenVariant {
  int H, NH;
  void (*fwd[2])(GenParams);   // 64-row, 16-row tiles
  void (*bwd[2])(GenParams);
};

#define SAGIPS_GEN_VARIANT(H_, NH_)                                               \
  {                                                                              \
    H_, NH_, {k_gen_forward<NH_>, k_gen_forward16<H_, NH_>},                     \
        {k_gen_backward<H_, NH_, 64>, k_gen_backward<H_, NH_, 16> }              \
  }

const GenVariant kGenVariants[] = {SAGIPS_GEN_VARIANT(128, 1), SAGIPS_GEN_VARIANT(128, 2), SAGIPS_GEN_VARIANT(128, 3)};

const GenVariant* find_gen(const sagips_gen& G) {
  const int H = G.width[1], NH = G.n_layers - 2;
  for (const GenVariant& v : kGenVariants)
    if (v.H == H && v.NH == NH) return &v;
  return nullptr;
}

GenParams gen_params(const sagips_gen& G, const float* noise, int64_t k) {
  GenParams p;
  memset(&p, 0, sizeof(p));
  int64_t off = 0;
  for (int l = 0; l < G.n_layers; ++l) {
    p.W[l] = G.W[l];
    p.b[l] = G.b[l];
    p.wsz[l] = (int64_t)G.width[l + 1] * G.width[l];
    p.bsz[l] = G.width[l + 1];
    p.poff_w[l] = off;
    off += p.wsz[l];
    p.poff_b[l] = off;
    off += p.bsz[l];
  }
  p.P = off;
  p.in = G.width[0];
  p.out = G.width[G.n_layers];
  p.k = k;
  p.slope = G.leaky_slope;
  p.noise = noise;
  return p;
}

// Row tile: 64, unless 64-row tiles of all members would not cover the CUs.
inline int gen_rows(const sagips_gen& G, int64_t k, int n_cu) {
  return ((k + 63) / 64) * G.n_members >= n_cu ? 64 : 16;
}
inline int gen_tiles(int64_t k, int T) { return (int)((k + T - 1) / T); }

}  // namespace

bool gen_supported(const sagips_gen& G, const char** why) {
  if (G.n_layers < 3 || G.n_layers > kMaxGenLayers) { *why = "generator needs 3 to 5 layers"; return false; }
  if (G.width[0] < 1 || G.width[0] > kGMaxIO || G.width[G.n_layers] < 1 || G.width[G.n_layers] > kGMaxIO) {
    *why = "generator input and output widths must be in [1, 8]";
    return false;
  }
  for (int l = 1; l < G.n_layers; ++l)
    if (G.width[l] != G.width[1]) { *why = "all hidden widths must be equal"; return false; }
  if (!find_gen(G)) { *why = "unsupported generator shape (hidden width 128 with 1-3 hidden-to-hidden layers)"; return false; }
  return true;
}

size_t gen_backward_workspace(const sagips_gen& G, int64_t k, int n_cu) {
  const GenParams p = gen_params(G, nullptr, k);
  return sizeof(float) * (size_t)p.P * gen_tiles(k, gen_rows(G, k, n_cu)) * G.n_members;
}

size_t ensemble_workspace(const sagips_gen& G, int64_t k) {
  const size_t th = (sizeof(float) * (size_t)G.n_members * k * G.width[G.n_layers] + 255) & ~(size_t)255;
  return th + sizeof(float) * 2 * (size_t)k * G.width[G.n_layers];
}

hipError_t launch_gen_forward(const sagips_gen& G, const float* noise, int64_t k, float* theta, int n_cu,
                              hipStream_t st, Timer* tm) {
  GenParams p = gen_params(G, noise, k);
  p.theta = theta;
  const GenVariant* v = find_gen(G);
  const int T = gen_rows(G, k, n_cu);
  if (tm) tm->begin("gen_forward");
  hipLaunchKernelGGL(v->fwd[T == 64 ? 0 : 1], dim3(gen_tiles(k, T), G.n_members), dim3(T == 64 ? kFwdThreads : kGThreads),
                     0, st, p);
  if (tm) tm->end();
  return hipGetLastError();
}

hipError_t launch_gen_backward(const sagips_gen& G, const float* noise, int64_t k, const float* dtheta,
                               float* const* dW, float* const* db, void* ws, int n_cu, hipStream_t st, Timer* tm) {
  GenParams p = gen_params(G, noise, k);
  p.dtheta = dtheta;
  p.part = static_cast<float*>(ws);
  const GenVariant* v = find_gen(G);
  const int T = gen_rows(G, k, n_cu);
  const int tiles = gen_tiles(k, T);
  if (tm) tm->begin("gen_backward");
  hipLaunchKernelGGL(v->bwd[T == 64 ? 0 : 1], dim3(tiles, G.n_members), dim3(kGThreads), 0, st, p);
  if (tm) tm->end();
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  GenReduceArgs r;
  memset(&r, 0, sizeof(r));
  r.part = p.part;
  r.P = p.P;
  r.tiles = tiles;
  r.n_layers = G.n_layers;
  for (int l = 0; l < G.n_layers; ++l) {
    r.poff_w[l] = p.poff_w[l];
    r.poff_b[l] = p.poff_b[l];
    r.wsz[l] = p.wsz[l];
    r.bsz[l] = p.bsz[l];
    r.dW[l] = dW[l];
    r.db[l] = db[l];
  }
  if (tm) tm->begin("gen_reduce");
  if (tiles <= 4) hipLaunchKernelGGL(k_gen_reduce<1>, dim3((unsigned)((p.P + 255) / 256), G.n_members), dim3(256), 0, st, r);
  else hipLaunchKernelGGL(k_gen_reduce<4>, dim3((unsigned)((p.P + 63) / 64), G.n_members), dim3(256), 0, st, r);
  if (tm) tm->end();
  return hipGetLastError();
}

hipError_t launch_ensemble(const sagips_gen& G, const float* noise, int64_t k, const float* p_true, float* p_hat,
                           float* sigma, float* r_hat, void* ws, int n_cu, hipStream_t st, Timer* tm) {
  const int out = G.width[G.n_layers];
  float* theta = static_cast<float*>(ws);
  const size_t th = (sizeof(float) * (size_t)G.n_members * k * out + 255) & ~(size_t)255;
  float* rowstat = reinterpret_cast<float*>(static_cast<char*>(ws) + th);
  hipError_t e = launch_gen_forward(G, noise, k, theta, n_cu, st, tm);
  if (e != hipSuccess) return e;
  if (tm) tm->begin("ensemble_rows");
  hipLaunchKernelGGL(k_ens_rows, dim3((unsigned)((k * out + kEnsCols - 1) / kEnsCols)), dim3(256), 0, st, theta,
                     G.n_members, k, out, rowstat);
  if (tm) tm->end();
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (tm) tm->begin("ensemble_final");
  hipLaunchKernelGGL(k_ens_final, dim3(1), dim3(kEnsFinal), 0, st, rowstat, k, out, p_true, p_hat, sigma, r_hat);
  if (tm) tm->end();
  return hipGetLastError();
}

}  // namespace sagips
