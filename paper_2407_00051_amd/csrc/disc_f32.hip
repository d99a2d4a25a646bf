// Fused fp32 discriminator step on gfx950: forward on fake and real events,
// BCE loss, backward to the weights (dL_D) and to the fake events (dL_G),
// and, when the fake events come from a source, the sampler and the
// per-parameter reduction as well -- one persistent kernel per call.
//
// Network: F -> H -> (H -> H) x NH -> 1, LeakyReLU on the hidden layers
// (paper Sec. V-A), weights in torch.nn.Linear layout.  Events have DX
// coordinates; the network sees F features of them: the coordinates
// themselves (F = DX), or the two observables y0 = x1 + x3, y1 = x2 + x3 of
// the six-parameter, two-observable pipeline (DX = 3, F = 2; Sec. V).
//
// The H x H products run on the bf16 matrix cores with every fp32 operand
// split into its three bf16 terms (split_bf16.hpp): six bf16 products in the
// place of one fp32 product, at 16 times the fp32 matrix rate.
//
// Work decomposition
//   * One persistent workgroup of 4 waves (one per SIMD, so that each has 512
//     registers) per CU loops over tiles of T events; a tile is all fake or all
//     real.  The waves form a grid of WF x WE: wave (wf, ew) owns output
//     features [32 wf, 32 wf + 32) of every product for events [64 ew, 64 ew + 64)
//     of the tile.  H = 128: 4 x 1 waves, T = 64; H = 64: 2 x 2 waves, T = 128.
//     Two 32 x 32 accumulators per wave share each weight fragment: a CU's
//     weight loads (L2) and LDS reads then stay near half of what they deliver at
//     full matrix rate; with eight waves of one accumulator each, the weight
//     loads alone would need all of it.
//   * Activations and backward signals live in LDS, split, feature-major:
//     [term][feature][event] bf16.  Products have M = event, N = output feature,
//     so that a lane's accumulators are one feature of 4 consecutive events at a
//     time, and the same registers are the next weight gradient's
//     operand (K = events) without another pass through LDS.  The products read
//     their K = features operand with the transposing ds_read_b64_tr_b16.
//     (SplitLds has the arrangement.)
//   * Sums over features (the logit, dL/dx) go across the 32 lanes of a wave half
//     by DPP and permlane swaps, then over the waves through LDS.
//   * Weight gradients dW = sum_events (e delta)^T A accumulate in registers
//     across all of the workgroup's tiles, written once per workgroup and summed
//     over workgroups in a fixed order afterwards.
//   * One backward chain with a unit seed per event serves both losses: the
//     signals are linear in the seed, so dL_D terms are scaled by
//     e_D = dL_D/dz and the fake-input gradient by e_G = dL_G/dz.
//   * Three LDS buffers hold A_1 .. A_NH and the top signal; a backward signal
//     overwrites the activation it replaces, one barrier per layer.  With
//     NH = 3 the top signal takes A_1's buffer and A_1 is formed again (two
//     inputs a feature) before its weight gradient.
//   * Sampled fake events: the next tile's events are sampled while the seeds of
//     this one are formed; event i takes parameter row i / E, so a 64-event
//     block may straddle two rows (E >= 64) and its per-parameter partials keep
//     one slot per row.
//
// What bounds it: with one wave per SIMD, the vector ALU work that is not
// placed between products adds to the products' own time (six bf16 products:
// 0.25 ms of the 262,144 + 262,144-event, 2-128-128-128-1 step at 2.5 PFLOP/s).
// Measured on that step: 0.95 ms with fp32 matrix instructions (8 waves, 0.69 of
// their peak), 0.55 ms now (0.62 to 0.73 in the first launches from idle), matrix cores
// 0.5 busy at 2.0 GHz; the paper's 2-128-128-128-128-1 network on 102,400 + 102,400
// events 0.62 -> 0.35 ms.  Error
// against float64, same inputs: logits 0.5 times the fp32 instructions' (one
// rounding per 8 products and per K step of the full-size sum, not one per 4).
#include "device_math.hpp"
#include "kernels.hpp"
#include "split_bf16.hpp"

#include <string.h>

#include <algorithm>

namespace sagips {
namespace {

constexpr int kThreads = 256;  // 4 waves, one per SIMD
constexpr int kSub = 64;       // events per wave and tile, and per loss / parameter partial
constexpr int kMaxNH = 3;
constexpr int padded(int P) { return (P + 3) & ~3; }   // partial rows: a multiple of 16 bytes

struct F32Params {
  // network
  const float* W1;             // [H][F]
  const float* b1;             // [H]
  const u16* Wf;               // [NH] split forward copies, then [NH] split backward copies
  const float* bh[kMaxNH];     // [H]
  const float* Wo;             // [H]
  const float* bo;             // [1]
  float slope;
  // inputs
  const float* fake_x;         // [n_fake][DX] or NULL (then sampled)
  const float* real_x;         // [n_real][DX]
  SourceArgs src;              // valid when fake_x == NULL
  int64_t n_fake, n_real;
  int n_fake_tiles, n_tiles;
  int fake_rem;                // n_fake_tiles modulo the grid
  int64_t E;                   // events per parameter row (source path)
  float inv_nf, inv_nr;
  // outputs
  float* logits_fake;
  float* logits_real;
  float* dLg_dx;               // [n_fake][DX] or NULL
  // workspace
  float* wg_part;              // [gridDim.x][P], rows padded to 16 bytes
  float* loss_part;            // [n_tiles WE][2]
  float* theta_part;           // [n_fake_tiles WE][2][2 DX] (source path): slot 0 = row of the
                               // block's first event, slot 1 = the next row
};

// softplus(t) = max(t, 0) + ln(1 + e^-|t|) on the hardware units (exp2 and
// log2 within 1 ulp; Kahan's log1p keeps the small-argument accuracy).
__device__ __forceinline__ float softplus(float t) { return fmaxf(t, 0.0f) + log1p_k(fast_exp(-fabsf(t))); }

// Events of a tile: 64 per wave along the events.
constexpr int tile_events(int H) { return kSub * (kThreads / 64) / (H / 32); }

template <int H, int NH, int DX, int F, int FEAT>
struct Fused : SplitLds<H, tile_events(H)> {
  static_assert(FEAT == SAGIPS_FEAT_IDENTITY ? DX == F : (FEAT == SAGIPS_FEAT_PROXY2 && DX == 3 && F == 2),
                "feature map");
  static constexpr int WAVES = kThreads / 64;
  static constexpr int WF = H / 32;            // waves along the features
  static constexpr int WE = WAVES / WF;        // waves along the events
  static constexpr int T = tile_events(H);
  static constexpr int KS = H / 16;            // K steps of a product over features
  static constexpr int KB = H / 32;            // 32-column blocks of a weight gradient
  static constexpr int SE = kSub / 16;         // K steps of a weight gradient (events)
  using Lds = SplitLds<H, T>;
  using typename Lds::Lane;
  using typename Lds::Step;
  using Lds::BUF;
  using Lds::read_ev;
  using Lds::read_tr;
  using Lds::split4;
  using Lds::store_step;
  static constexpr int NBUF = NH + 1 < 3 ? NH + 1 : 3;
  static constexpr int kTop = NH < 3 ? NH : 0; // buffer of the top signal
  static constexpr bool kRemakeA1 = kTop == 0;
  static constexpr int EU = (DX + WF - 1) / WF;   // coordinates per wave
  // Weight gradients' correction products in accumulators of their own, as in product().
  // Width 64 has the registers, and needs them where a workgroup has one tile, all fake or
  // all real (2-64-64-1 on 16,384 + 16,384 events: error of dW_2 against float64 7.0e-8 ->
  // 6.1e-8; before the split products 7.5e-8).  At width 128 the tiles' order suffices; there
  // they cost 2% with one hidden-to-hidden layer and spill 4 to 21 registers with two, 371
  // with three.
  static constexpr bool kApart = H == 64;
  static constexpr int PD = NH < 3 ? 3 : 2;   // weight-fragment prefetch distance (K steps)
  static_assert(WF * WE == WAVES && (H == 64 || H == 128), "wave decomposition");
  // per-workgroup partial layout (floats)
  static constexpr int P_DWH = H * H + H;      // dW + db of one hidden layer
  static constexpr int OFF_W1 = NH * P_DWH;    // dW1 [H][F], then db1 [H]
  static constexpr int OFF_WO = OFF_W1 + H * F + H;  // dWo [H], then dbo
  static constexpr int P = OFF_WO + H + 1;

  struct Smem {
    char act[NBUF * BUF];
    float xs[2][DX][T];        // coordinates of this tile and the next
    float zp[WAVES][kSub];     // logit partials over a wave's features
    float es[WAVES][kSub];     // e_D of a wave's events
    float gp[WAVES][F][kSub];  // dL/d(feature) partials over a wave's features
  };
  static_assert(WE == 1 || WE * padded(P) * 4 <= NBUF * BUF, "staging of the partials");

  // Weight steps of the next product, loaded during the tail of the current one.
  struct Prefetch {
    bf16x8 w[PD][kTerms];
  };

  static __device__ __forceinline__ void load_w(Rsrc W, uint32_t woff, int ks, bf16x8 (&w)[kTerms]) {
#pragma unroll
    for (int t = 0; t < kTerms; ++t) w[t] = split_load(W, woff, (uint32_t)(ks * kTerms + t) * 1024u);
  }
  static __device__ __forceinline__ Rsrc weight(const u16* Wf, int copy) {
    return split_rsrc(Wf + (size_t)copy * (split_copy_bytes(H) / 2), (uint32_t)split_copy_bytes(H));
  }

  // acc[mt] = in W + bias for the wave's 32 features and event blocks mt.  pf holds the
  // first PD weight steps on entry and, with kNext, those of Wn (the next
  // product's weights) on exit.  side(ks) is other work of step ks, issued
  // between its products (kValu instructions after each).
  template <bool kNext, int kValu, typename Side>
  static __device__ __forceinline__ void product(Rsrc W, Rsrc Wn, uint32_t woff, Prefetch& pf, const char* buf, const Lane& L,
                                                 float bias, f32x16 (&acc)[2], Side side) {
    f32x16 corr[2];
    bf16x8 w[PD + 1][kTerms];
    bf16x8 a[2][2][kTerms];
#pragma unroll
    for (int q = 0; q < PD; ++q)
#pragma unroll
      for (int t = 0; t < kTerms; ++t) w[q][t] = pf.w[q][t];
    read_tr(buf, L, 0, 0, a[0][0]);
    read_tr(buf, L, 1, 0, a[0][1]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      __builtin_amdgcn_sched_barrier(0);
      if (ks + PD < KS) load_w(W, woff, ks + PD, w[(ks + PD) % (PD + 1)]);
      else if (kNext) load_w(Wn, woff, ks + PD - KS, pf.w[ks + PD - KS]);
      if (ks + 1 < KS) {
        read_tr(buf, L, 0, ks + 1, a[(ks + 1) & 1][0]);
        read_tr(buf, L, 1, ks + 1, a[(ks + 1) & 1][1]);
      }
      // without side work the loads stay above the products of this step
      if (kValu == 0) __builtin_amdgcn_sched_barrier(0);
      side(ks);
      if (ks == 0) split_mfma_apart<true, false>(a[0], w[0], acc, corr);
      else split_mfma_apart<false, false>(a[ks & 1], w[ks % (PD + 1)], acc, corr);
      if (kValu) interleave<kTerms, kValu>();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      acc[0][i] = (acc[0][i] + corr[0][i]) + bias;
      acc[1][i] = (acc[1][i] + corr[1][i]) + bias;
    }
  }

  // accW[kb] += sum over the wave's events of (e delta)[o] A[k], rows o = the
  // wave's features.  signal(s, u, d, ed) forms half u of step s of the signal
  // (d, stored in dst for the next product) and of e_D times it (ed); those of
  // step s + 1 are formed between the products of step s.  The next product's
  // first weight steps are loaded in the last steps.
  template <typename Signal>
  static __device__ __forceinline__ void wgrad(const char* A, const Lane& L, f32x16 (&accW)[KB], f32x16 (&corW)[kApart ? KB : 1], char* dst, Rsrc Wn,
                                               uint32_t woff, Prefetch& pf, Signal signal) {
    Step d, ed[2];
    auto form = [&](int s, int u) __attribute__((always_inline)) {
      signal(s, u, d, ed[s & 1]);
      if (u == 1) store_step(dst, L, s, d);
    };
    bf16x8 b[2][2][kTerms];
    read_ev(A, L, 0, 0, b[0][0]);
    read_ev(A, L, 1, 0, b[0][1]);
    form(0, 0);
    form(0, 1);
    constexpr int N = SE * KB / 2;             // steps: K step s, column blocks kb, kb + 1
#pragma unroll
    for (int q = 0; q < N; ++q) {
      __builtin_amdgcn_sched_barrier(0);
      const int s = q / (KB / 2), kb = 2 * (q % (KB / 2));
      if (q + 1 < N) {
        const int s1 = (q + 1) / (KB / 2), kb1 = 2 * ((q + 1) % (KB / 2));
        read_ev(A, L, kb1, s1, b[(q + 1) & 1][0]);
        read_ev(A, L, kb1 + 1, s1, b[(q + 1) & 1][1]);
      }
      if (q >= N - PD) load_w(Wn, woff, q - (N - PD), pf.w[q - (N - PD)]);
      bf16x8 a[kTerms];
#pragma unroll
      for (int t = 0; t < kTerms; ++t)
        a[t] = __builtin_bit_cast(bf16x8, make_uint4(ed[s & 1][t][0], ed[s & 1][t][1], ed[s & 1][t][2], ed[s & 1][t][3]));
      if (s + 1 < SE) {
#pragma unroll
        for (int u = 0; u < 4 / KB; ++u) form(s + 1, 4 / KB * (kb / 2) + u);
      }
      if constexpr (kApart) split_mfma2(b[q & 1][0], b[q & 1][1], a, accW[kb], accW[kb + 1], corW[kb], corW[kb + 1]);
      else split_mfma2(b[q & 1][0], b[q & 1][1], a, accW[kb], accW[kb + 1], accW[kb], accW[kb + 1]);
      interleave<kTerms, 12 / KB * 2>();
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Features of 4 consecutive events from the coordinate rows.
  static __device__ __forceinline__ void features4(const float (&xs)[DX][T], int ev, f32x4 (&x)[F]) {
    f32x4 c[DX];
#pragma unroll
    for (int j = 0; j < DX; ++j) c[j] = *reinterpret_cast<const f32x4*>(&xs[j][ev]);
    if constexpr (FEAT == SAGIPS_FEAT_PROXY2) {
      x[0] = c[0] + c[2];
      x[1] = c[1] + c[2];
    } else {
#pragma unroll
      for (int j = 0; j < F; ++j) x[j] = c[j];
    }
  }

  // A copy of an LDS offset that the compiler cannot merge with another: what is
  // read through it is read again, not kept in registers from an earlier read.
  static __device__ __forceinline__ int fresh(int o) {
    asm volatile("" : "+v"(o));
    return o;
  }

  // First layer (VALU): A_1 = leaky(x W_1^T + b_1) of the wave's features, half u of
  // step s of its events (evo = 64 ew + 4 lh), into d; stored with the second half.
  static __device__ __forceinline__ void first_layer(const float (&xs)[DX][T], int evo, int s, int u,
                                                     const float (&w1r)[F], float b1r, float slope, Step& d, char* buf,
                                                     const Lane& L) {
    f32x4 x[F];
    features4(xs, evo + 16 * s + 8 * u, x);
    float h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v = b1r;
#pragma unroll
      for (int j = F - 1; j >= 0; --j) v = fmaf(w1r[j], x[j][q], v);
      h[q] = v > 0.0f ? v : slope * v;
    }
    split4(h, u, d);
    if (u == 1) store_step(buf, L, s, d);
  }

  // What a wave keeps of a tile's 64-event block until the block's input gradient is
  // complete: the sampled coordinates' pathwise terms and e_G, lane = event.
  struct Block {
    int64_t i0;             // first event
    int64_t sub;            // index among the fake batch's blocks
    int fake, sampled, split;
    float eG;
    float da[EU], db[EU];
  };

  // The tiles of a workgroup: tile blockIdx.x and every gridDim.x-th from there, fake and
  // real ones in turn, in the ratio of their numbers: next is the one after which less of
  // its batch is done.  The two batches' gradients nearly cancel, so the accumulators then
  // never hold much more than a tile's share, and the roundings of their sums are relative
  // to that and not to a whole batch's.  2-128-128-128-1 on 262,144 + 262,144 events: error
  // of dW_3 against float64 1.2e-7, 3.2e-7 with all fake tiles first (2.2e-7 on the fp32
  // matrix instructions, which rounded a sum four times per 16 events where these round it
  // twelve times); the step takes 0.3% longer for it.  The tiles of a batch that has fewer
  // than the grid come last: each is a large share of the sum, and tiles after it would be
  // rounded at its size (80,000 + 100 events: dW_2 5.3e-7, 1.1e-6 with such a tile first).
  struct Tiles {
    int f, r;               // the next fake and the next real tile
    __device__ __forceinline__ explicit Tiles(const F32Params& p) {
      f = blockIdx.x;
      r = p.n_fake_tiles - p.fake_rem + (f < p.fake_rem ? f + (int)gridDim.x : f);
    }
    // The next tile, -1 past the last one.
    __device__ __forceinline__ int take(const F32Params& p) {
      const int nf = p.n_fake_tiles, n = p.n_tiles, step = gridDim.x;
      const bool fake = f < nf && (r >= n || (int64_t)(f + step) * (n - nf) <= (int64_t)(r + step - nf) * nf);
      const int t = fake ? f : (r < n ? r : -1);
      f += fake ? step : 0;
      r += fake ? 0 : step;
      return t;
    }
  };

  // Events of block ew of a tile: lane = event, coordinate j = wf + u WF (waves
  // without one of their own repeat the last).  fetch() loads what they need:
  // theta (a, b) of the event's parameter row for sampled events, the coordinate
  // for buffer ones.  form(piece) does the arithmetic in four pieces without a
  // branch, so that they fit between the products of a step; for buffer events
  // its results are dropped.
  struct Sampler {
    float a[EU], b[EU], x[EU];
    Words w;
    Shape sh[EU];
    Quantile q[EU];
    int valid;
  };
  static __device__ __forceinline__ int coord(const Lane& L, int u) { return min(L.wf + u * WF, DX - 1); }

  static __device__ __forceinline__ void fetch(const F32Params& p, int tile, const Lane& L, Block& b, Sampler& S) {
    b.fake = tile < p.n_fake_tiles;
    const int64_t n = b.fake ? p.n_fake : p.n_real;
    const int t = b.fake ? tile : tile - p.n_fake_tiles;
    b.i0 = (int64_t)t * T + kSub * L.ew;
    b.sub = (int64_t)t * WE + L.ew;
    b.sampled = b.fake && p.fake_x == nullptr;
    b.split = kSub;
    const int here = (int)max<int64_t>(0, min<int64_t>(kSub, n - b.i0));   // events of the block
    S.valid = L.lane < here;
    // the parameter row of the block's first event, and the first event of the next row
    // (E >= 64: at most these two); n_fake < 2^30 keeps this in 32 bits
    uint32_t row = 0;
    if (b.sampled) {
      row = (uint32_t)b.i0 / (uint32_t)p.E;
      b.split = (int)min<int64_t>((int64_t)(row + 1) * p.E - b.i0, kSub);
    }
    // loads past the records read 0: no theta for buffer events, no coordinates for
    // sampled ones; the rows of a block are row and, past the split, row + 1
    const Rsrc rt = split_rsrc(p.src.theta + (size_t)row * 2 * DX,
                               b.sampled && here > 0 ? (b.split < here ? 16u : 8u) * DX : 0u);
    const float* xin = b.fake ? p.fake_x : p.real_x;
    const Rsrc rx = split_rsrc(xin + b.i0 * DX, b.sampled ? 0u : (uint32_t)here * DX * 4u);
#pragma unroll
    for (int u = 0; u < EU; ++u) {
      const int j = coord(L, u);
      const uint32_t ot = (uint32_t)((L.lane >= b.split ? 2 * DX : 0) + 2 * j) * 4u;
      S.a[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, (int)ot, 0, 0));
      S.b[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, (int)ot, 4, 0));
      S.x[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (L.lane * DX + j) * 4, 0, 0));
    }
  }

  static __device__ __forceinline__ void form(const F32Params& p, int piece, float (&xs)[DX][T], const Lane& L, Block& b,
                                              Sampler& S) {
    if (piece == 0) {
      // opaque key words: their schedule is formed here, not kept in 20 scalar registers
      // across the tile loop
      uint32_t k0 = p.src.k0, k1 = p.src.k1;
      asm volatile("" : "+s"(k0), "+s"(k1));
      S.w = event_words(p.src.base + (uint64_t)(b.i0 + L.lane), p.src.stream, k0, k1);
    }
#pragma unroll
    for (int u = 0; u < EU; ++u) {
      const int j = coord(L, u);
      if (piece == 1) S.sh[u] = make_shape(S.a[u], S.b[u]);
      if (piece == 2) S.q[u] = kumaraswamy_w<true>(j == 0 ? S.w.w[0] : (j == 1 ? S.w.w[1] : S.w.w[2]), S.sh[u]);
      if (piece == 3) {
        float da, db;
        pathwise(S.q[u], S.sh[u], da, db);
        const bool on = b.sampled && S.valid;
        b.da[u] = on ? da : 0.f;
        b.db[u] = on ? db : 0.f;
        xs[j][kSub * L.ew + L.lane] = S.valid ? (b.sampled ? S.q[u].x : S.x[u]) : 0.5f;
      }
    }
  }

  // dL_G/dx and the per-parameter partials of a fake block, once every wave's
  // feature partials are in gp: lane = event, coordinate j = wf + u WF.
  static __device__ __forceinline__ void finish(const F32Params& p, const Smem& sm, const Lane& L, const Block& b) {
    if (!b.fake) return;
#pragma unroll
    for (int u = 0; u < EU; ++u) {
      const int j = L.wf + u * WF;
      if (j < DX) {
        auto total = [&](int f) __attribute__((always_inline)) {
          float s = 0.f;
#pragma unroll
          for (int w = 0; w < WF; ++w) s += sm.gp[L.ew * WF + w][f][L.lane];
          return s * b.eG;
        };
        // through the feature map's Jacobian
        float gx;
        if constexpr (FEAT == SAGIPS_FEAT_PROXY2) gx = j == 2 ? total(0) + total(1) : total(j);
        else gx = total(j);
        const int64_t i = b.i0 + L.lane;
        if (p.dLg_dx && i < p.n_fake) p.dLg_dx[i * DX + j] = gx;
        if (b.sampled) {
          const bool lo = L.lane < b.split;
          const float ta = gx * b.da[u], tb = gx * b.db[u];
          // lane 0, 16, 32, 48 of the wave: totals of slot 0 a, b, slot 1 a, b
          const float s = wave_scatter_sum4(lo ? ta : 0.f, lo ? tb : 0.f, lo ? 0.f : ta, lo ? 0.f : tb);
          if ((L.lane & 15) == 0)
            p.theta_part[(b.sub * 2 + (L.lane >> 5)) * 2 * DX + 2 * j + ((L.lane >> 4) & 1)] = s;
        }
      }
    }
  }

  static __device__ void run(const F32Params& p) {
    __shared__ __attribute__((aligned(1024))) Smem sm;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Lane L = Lds::make_lane(wave % WF, wave / WF);
    const int lr = L.lr, lh = L.lh;
    const uint32_t woff = (uint32_t)(L.wf * KS * kTerms * 64 + L.lane) * 16u;   // weight fragment (wf, 0, 0)
    const int fo = 32 * L.wf + lr;               // the lane's feature where N = features
    const float slope = p.slope;
    // event of accumulator value i = lr (the one whose sum over features a lane gets)
    const int ev_of_lane = 32 * (lr >> 4) + 8 * ((lr >> 2) & 3) + 4 * lh + (lr & 3);
    auto buf = [&](int i) __attribute__((always_inline)) { return &sm.act[i * BUF]; };

    f32x16 accW[NH][KB], corW[NH][kApart ? KB : 1];
    float dbacc[NH];
#pragma unroll
    for (int l = 0; l < NH; ++l) {
      dbacc[l] = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        accW[l][kb] = f32x16{};
        if (kApart) corW[l][kb] = f32x16{};
      }
    }
    float aw1[F + 1];                            // dW_1 and db_1 of feature fo over the lane's events
#pragma unroll
    for (int j = 0; j <= F; ++j) aw1[j] = 0.f;
    float dwo = 0.f, dbo = 0.f;
    float w1r[F];
#pragma unroll
    for (int j = 0; j < F; ++j) w1r[j] = p.W1[fo * F + j];
    const float b1r = p.b1[fo];
    const float wor = p.Wo[fo], wos = wor * slope;
    float bhr[NH];
#pragma unroll
    for (int l = 0; l < NH; ++l) bhr[l] = p.bh[l][fo];
    const float bo = p.bo[0];
    Prefetch pf;
#pragma unroll
    for (int q = 0; q < PD; ++q) load_w(weight(p.Wf, 0), woff, q, pf.w[q]);

    Block cur, prev, next;
    prev.fake = 0;
    int par = 0;
    Sampler S;
    Tiles order(p);                              // gridDim.x <= n_tiles: at least one
    int tile = order.take(p);
    fetch(p, tile, L, cur, S);
#pragma unroll
    for (int i = 0; i < 4; ++i) form(p, i, sm.xs[0], L, cur, S);
    __syncthreads();
    const int evo = kSub * L.ew + 4 * lh;        // the lane's first event in the tile
    Step a1;
#pragma unroll
    for (int i = 0; i < 2 * SE; ++i) {
      first_layer(sm.xs[0], evo, i / 2, i % 2, w1r, b1r, slope, a1, buf(0), L);
      __builtin_amdgcn_sched_barrier(0);
    }
    auto nothing = [](int) {};

    // A tile starts with its A_1 in buffer 0 (formed during the last product of the tile before).
    for (int following; tile >= 0; tile = following, par ^= 1) {
      // ---- forward ---------------------------------------------------------------
      // (past the last tile its events are formed once more and not used)
      following = order.take(p);
      fetch(p, following >= 0 ? following : tile, L, next, S);
      __syncthreads();
      // the weight-gradient accumulators stay in the accumulation registers (left to
      // itself the compiler carries half of them round the loop in the others)
#pragma unroll
      for (int l = 0; l < NH; ++l)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          asm volatile("" : "+a"(accW[l][kb]));
          if (kApart) asm volatile("" : "+a"(corW[l][kb]));
        }
      uint32_t mask[NH];                         // bit 31 - i: output i of A_{l+2} positive
      f32x16 acc[2];
#pragma unroll
      for (int l = 0; l < NH - 1; ++l) {
        product<true, 0>(weight(p.Wf, l), weight(p.Wf, l + 1), woff, pf, buf(l), L, bhr[l], acc, nothing);
        uint32_t m = 0u;
#pragma unroll
        for (int q = 0; q < SE; ++q) {
          Step d;
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float v = acc[q >> 1][8 * (q & 1) + 4 * u + i];
              m = __builtin_amdgcn_alignbit(m, __float_as_uint(0.0f - v), 31);
              h[i] = v > 0.0f ? v : slope * v;
            }
            split4(h, u, d);
          }
          store_step(buf(l + 1), L, q, d);
          __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" : "+v"(m));              // packed here, not where it is used
        mask[l] = m;
        __syncthreads();
      }
      // ---- top layer and logit partials; meanwhile the next tile's events ----------
      product<false, 6>(weight(p.Wf, NH - 1), weight(p.Wf, 0), woff, pf, buf(NH - 1), L, bhr[NH - 1], acc,
                        [&](int ks) __attribute__((always_inline)) {
                          if (ks % (KS / 4) == 0) form(p, ks / (KS / 4), sm.xs[par ^ 1], L, next, S);
                        });
      float h[32];
      {
        float z[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
          const float v = acc[i >> 4][i & 15];
          h[i] = v > 0.0f ? v : slope * v;
          z[i] = h[i] * wor;
        }
        sm.zp[wave][ev_of_lane] = half_scatter_sum(z, lr);
      }
      __syncthreads();

      // ---- logits, BCE seeds (lane = event) -----------------------------------------
      {
        float z = bo;
#pragma unroll
        for (int w = 0; w < WF; ++w) z += sm.zp[L.ew * WF + w][L.lane];
        const int64_t i = cur.i0 + L.lane;
        const bool valid = i < (cur.fake ? p.n_fake : p.n_real);
        float eD = 0.f, eG = 0.f;
        if (valid) {
          const float sig_neg = fast_rcp(1.0f + fast_exp(z));   // sigmoid(-z)
          if (cur.fake) {
            eD = (1.0f - sig_neg) * p.inv_nf;                // dL_D/dz = sigmoid(z)/N_f
            eG = -sig_neg * p.inv_nf;                        // dL_G/dz = (sigmoid(z)-1)/N_f
          } else {
            eD = -sig_neg * p.inv_nr;                        // (sigmoid(z)-1)/N_r
          }
        }
        sm.es[wave][L.lane] = eD;
        cur.eG = eG;
        if (L.wf == 0) dbo += eD;
        if (L.wf == WF - 1) {
          float l0 = 0.f, l1 = 0.f;
          if (valid) {
            l0 = softplus(cur.fake ? z : -z);
            if (cur.fake) l1 = softplus(-z);
            float* lg = cur.fake ? p.logits_fake : p.logits_real;
            if (lg) lg[i] = z;
          }
          l0 = wave_total(l0);
          l1 = wave_total(l1);
          if (L.lane == 0) {
            const int64_t sub = (int64_t)tile * WE + L.ew;
            *reinterpret_cast<float2*>(p.loss_part + 2 * sub) = make_float2(l0, l1);
          }
        }
      }
      finish(p, sm, L, prev);        // the input gradient of the block before
      prev = cur;
      cur = next;

      // ---- hidden layers backward -----------------------------------------------------
      // Layer l maps A_{l+1} (buffer l) -> A_{l+2}.  Its weight gradient forms the
      // signal at A_{l+2} on the way (the top one from the logit weights, with the
      // logit layer's own gradient) and stores it, split, in buffer l + 1 (the top
      // one in kTop) for the product that follows.
#pragma unroll
      for (int l = NH - 1; l >= 0; --l) {
        if (kRemakeA1 && l == 0) __syncthreads();         // A_1 formed again by every wave
        const uint32_t m = l < NH - 1 ? mask[l] : 0u;
        const float* es = &sm.es[wave][fresh(4 * lh)];
        wgrad(buf(l), L, accW[l], corW[l], buf(l == NH - 1 ? kTop : l + 1), weight(p.Wf, NH + l), woff, pf,
              [&](int s, int u, Step& dt, Step& edt) __attribute__((always_inline)) {
                const f32x4 e = *reinterpret_cast<const f32x4*>(es + 16 * s + 8 * u);
                float d[4], ed[4], eh = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  const int i = 8 * s + 4 * u + q;
                  if (l == NH - 1) {
                    eh = q ? fmaf(e[q], h[i], eh) : e[q] * h[i];
                    d[q] = h[i] > 0.0f ? wor : wos;
                  } else {
                    const float v = acc[i >> 4][i & 15];
                    const uint32_t pos = (uint32_t)__builtin_amdgcn_sbfe((int)m, 31 - i, 1);
                    d[q] = __uint_as_float(
                        __builtin_amdgcn_bitop3_b32(pos, __float_as_uint(v), __float_as_uint(slope * v), 0xCA));
                  }
                  ed[q] = e[q] * d[q];
                }
                // four events first, so that the running sum is rounded once for all of them
                if (l == NH - 1) dwo += eh;
                dbacc[l] += (ed[0] + ed[1]) + (ed[2] + ed[3]);
                // accumulated here and now: the compiler would otherwise move the sums to the
                // end of the tile and keep their terms in registers until then
                asm volatile("" : "+v"(dbacc[l]), "+v"(dwo));
                split4(d, u, dt);
                split4(ed, u, edt);
              });
        __syncthreads();             // the signal is visible; every wave is done with buffer l
        if (l == 0) break;
        if constexpr (kRemakeA1) {
          // the top signal's buffer is free once the top product is through
          if (l == NH - 2) {
#pragma unroll
            for (int i = 0; i < 2 * SE; ++i) {
              first_layer(sm.xs[par], fresh(evo), i / 2, i % 2, w1r, b1r, slope, a1, buf(0), L);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        product<false, 0>(weight(p.Wf, NH + l), weight(p.Wf, 0), woff, pf, buf(l == NH - 1 ? kTop : l + 1), L, 0.f, acc,
                                 nothing);
      }

      // ---- first layer: delta_1, dW_1, db_1 and dL/dx; meanwhile the next tile's A_1 ------
      const int evn = fresh(evo), evp = fresh(evo), evs = fresh(4 * lh);
      product<true, 5>(weight(p.Wf, NH), weight(p.Wf, 0), woff, pf, buf(NH == 1 ? kTop : 1), L, 0.f, acc,
                       [&](int ks) __attribute__((always_inline)) {
#pragma unroll
                         for (int i = 2 * SE / KS * ks; i < 2 * SE / KS * (ks + 1); ++i)
                           first_layer(sm.xs[par ^ 1], evn, i / 2, i % 2, w1r, b1r, slope, a1, buf(0), L);
                       });
      {
        f32x4 x[2][F], e[2];                     // one group ahead
        auto get = [&](int k) __attribute__((always_inline)) {
          features4(sm.xs[par], evp + 8 * k, x[k & 1]);
          e[k & 1] = *reinterpret_cast<const f32x4*>(&sm.es[wave][evs + 8 * k]);
        };
        get(0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (k + 1 < 8) get(k + 1);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v = b1r;                       // the pre-activation, as in first_layer
#pragma unroll
            for (int j = F - 1; j >= 0; --j) v = fmaf(w1r[j], x[k & 1][j][q], v);
            const float a = acc[k >> 2][4 * (k & 3) + q];
            const float d = v > 0.0f ? a : slope * a;
            acc[k >> 2][4 * (k & 3) + q] = d;
            const float ed = e[k & 1][q] * d;
#pragma unroll
            for (int j = 0; j < F; ++j) aw1[j] = fmaf(ed, x[k & 1][j][q], aw1[j]);
            aw1[F] += ed;
          }
#pragma unroll
          for (int j = 0; j <= F; ++j) asm volatile("" : "+v"(aw1[j]));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (prev.fake) {
#pragma unroll
        for (int j = 0; j < F; ++j) {
          float g[32];
#pragma unroll
          for (int i = 0; i < 32; ++i) g[i] = acc[i >> 4][i & 15] * w1r[j];
          sm.gp[wave][j][ev_of_lane] = half_scatter_sum(g, lr);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __syncthreads();                             // the last tile's feature partials are in gp
    finish(p, sm, L, prev);

    // ---- per-workgroup partials ---------------------------------------------------
    // With two event groups both go through LDS and are added on the way out, in 16-byte
    // stores.  One copy of the code that empties the accumulators serves both groups: a
    // workgroup of one tile runs all of it once, at the rate at which it is fetched
    // (2-64-64-64-64-1 on 64 + 64 events: 49.9 KB of code and 32.1 us a call; 53.0 KB and
    // 33.5 us with a copy for each group).
    float* out = p.wg_part + (int64_t)blockIdx.x * padded(P);
    float* stage = reinterpret_cast<float*>(&sm.act[0]);
    float* dst = WE > 1 ? stage + L.ew * padded(P) : out;
#pragma unroll
    for (int l = 0; l < NH; ++l) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          dst[l * P_DWH + (32 * L.wf + 8 * (i / 4) + 4 * lh + i % 4) * H + 32 * kb + lr] =
              kApart ? accW[l][kb][i] + corW[l][kApart ? kb : 0][i] : accW[l][kb][i];
      const float v = add_xor32(dbacc[l]);
      if (lh == 0) dst[l * P_DWH + H * H + fo] = v;
    }
#pragma unroll
    for (int j = 0; j <= F; ++j) {
      const float v = add_xor32(aw1[j]);
      if (lh == 0) dst[j < F ? OFF_W1 + fo * F + j : OFF_W1 + H * F + fo] = v;
    }
    const float v = add_xor32(dwo);
    if (lh == 0) dst[OFF_WO + fo] = v;
    if (L.wf == 0) {
      const float s = wave_total(dbo);
      if (L.lane == 0) dst[OFF_WO + H] = s;
    }
    if constexpr (WE > 1) {
      static_assert(WE == 2, "two event groups");
      __syncthreads();
      for (int o = 4 * tid; o < P; o += 4 * kThreads)
        *reinterpret_cast<f32x4*>(out + o) =
            *reinterpret_cast<const f32x4*>(stage + o) + *reinterpret_cast<const f32x4*>(stage + padded(P) + o);
    }
  }
};

template <int H, int NH, int DX, int F, int FEAT>
__global__ __launch_bounds__(kThreads, 1) void k_disc_f32(F32Params p) {
  Fused<H, NH, DX, F, FEAT>::run(p);
}

// Split copies of the hidden layers (split_bf16.hpp): blockIdx.z = layer,
// blockIdx.y = 0 for W, 1 for its transpose; one thread per piece of 8 values.
struct SplitArgs {
  const float* W[kMaxNH];
  u16* out;
};

__global__ __launch_bounds__(256) void k_split_weights(SplitArgs a, int H, int NH) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int KS = H / 16;
  const int lane = t % 64, ks = t / 64 % KS, nb = t / (64 * KS);
  const float* W = a.W[blockIdx.z];
  const int n = 32 * nb + (lane & 31), k0 = 16 * ks + 8 * (lane >> 5);
  float v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = blockIdx.y ? W[(k0 + q) * H + n] : W[n * H + k0 + q];
  split_piece(v, a.out + (size_t)(blockIdx.y * NH + blockIdx.z) * (split_copy_bytes(H) / 2), nb, ks, KS, lane);
}

// All fixed-order reductions after the fused kernel, in one launch:
//   blocks [0, wg_blocks)        sum over workgroups of every gradient partial,
//                                scattered to the caller's arrays (segment table);
//   block  wg_blocks             the two losses from the per-block sums;
//   block  wg_blocks + 1 + q     dL_G/dtheta of parameter row q from the slots of the
//                                64-event blocks that hold its events.
struct Segments {
  int n;
  int off[2 * kMaxNH + 4];
  int len[2 * kMaxNH + 4];
  float* dst[2 * kMaxNH + 4];
};

struct ReduceArgs {
  const float* wg_part;             // [n_wg][PS]
  int n_wg, P, PS, wg_blocks;
  Segments sg;
  const float* loss_part;
  int n_fake_blocks, n_blocks;      // 64-event blocks of the fake batch, of both
  float inv_nf, inv_nr;
  float* loss_d;
  float* loss_g;
  const float* theta_part;
  int64_t E;
  int C, n_theta;
  float* dLg_dtheta;
};

// What bounds it: the bytes of the partials (P floats from each of n_wg workgroups,
// 34 MB at P = 33,537), if enough of them are in flight.  A block takes 32 values
// in 32 slices of workgroups, so that a thread adds 8 of 256 partials, four values
// each, all eight 16-byte loads in flight (rows are padded to 16 bytes); the losses'
// per-block sums are also loaded eight at a time.  Workgroups are added in pairs
// (g, n_wg - 1 - g): in a short step the first half of them have only fake events and
// the rest only real ones, whose gradients nearly cancel (2-64-64-1 on 16,384 + 16,384
// events: error of dW_2 against float64 7.0e-8; 7.8e-8 with the workgroups of a slice in
// turn, 2e-7 with contiguous ranges of them).  Against one 4-byte load after another that
// step is 1.5 us shorter a call (23.4 us) and the GAN training step at the paper's shape 2 us
// (412); 12.2 us at P = 33,537, 16.3 us at 50,049.
constexpr int kRedElems = 32;                       // values per block
constexpr int kRedLanes = kRedElems / 4;            // threads along the values
constexpr int kRedSlices = 256 / kRedLanes;         // slices of workgroups
constexpr int kRedGroups = 4;                       // slices combined eight to a group, then the groups
constexpr int kRedAhead = 8;                        // loads in flight

__global__ __launch_bounds__(256) void k_reduce_all(ReduceArgs r) {
  __shared__ __attribute__((aligned(16))) float red[kRedSlices][kRedElems];
  __shared__ float grp[kRedGroups][kRedElems];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < r.wg_blocks) {
    const int le = tid % kRedLanes, sl = tid / kRedLanes;
    const int e0 = blockIdx.x * kRedElems + 4 * le;
    f32x4 s = {};
    if (e0 < r.PS) {
      const float* src = r.wg_part + e0;
      const int half = (r.n_wg + 1) / 2;             // pairs (g, n_wg - 1 - g); an odd middle one is alone
      for (int g = sl; g < half; g += kRedAhead / 2 * kRedSlices) {
        f32x4 x[kRedAhead / 2], y[kRedAhead / 2];
#pragma unroll
        for (int u = 0; u < kRedAhead / 2; ++u) {
          const int a = min(g + kRedSlices * u, half - 1);
          x[u] = *reinterpret_cast<const f32x4*>(src + (int64_t)a * r.PS);
          y[u] = *reinterpret_cast<const f32x4*>(src + (int64_t)(r.n_wg - 1 - a) * r.PS);
        }
#pragma unroll
        for (int u = 0; u < kRedAhead / 2; ++u) {
          const int a = g + kRedSlices * u;
          if (2 * a + 1 < r.n_wg) s += x[u] + y[u];
          else if (a < half) s += x[u];
        }
      }
    }
    *reinterpret_cast<f32x4*>(&red[sl][4 * le]) = s;
    __syncthreads();
    const int le1 = tid % kRedElems, q = tid / kRedElems;
    if (q < kRedGroups) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < kRedSlices / kRedGroups; ++i) t += red[kRedSlices / kRedGroups * q + i][le1];
      grp[q][le1] = t;
    }
    __syncthreads();
    const int e = blockIdx.x * kRedElems + tid;
    if (tid >= kRedElems || e >= r.P) return;
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kRedGroups; ++i) t += grp[i][tid];
    for (int i = 0; i < r.sg.n; ++i)
      if (e >= r.sg.off[i] && e < r.sg.off[i] + r.sg.len[i]) {
        if (r.sg.dst[i]) r.sg.dst[i][e - r.sg.off[i]] = t;
        break;
      }
    return;
  }
  float* sums = &red[0][0];
  if ((int)blockIdx.x == r.wg_blocks) {
    float sf = 0.f, sgg = 0.f, sr = 0.f;
    const float2* part = reinterpret_cast<const float2*>(r.loss_part);
    for (int t = tid; t < r.n_blocks; t += 256 * kRedAhead) {
      float2 x[kRedAhead];
#pragma unroll
      for (int u = 0; u < kRedAhead; ++u) x[u] = part[min(t + 256 * u, r.n_blocks - 1)];
#pragma unroll
      for (int u = 0; u < kRedAhead; ++u) {
        const int i = t + 256 * u;
        sf = i < r.n_fake_blocks ? sf + x[u].x : sf;
        sgg = i < r.n_fake_blocks ? sgg + x[u].y : sgg;
        sr = i >= r.n_fake_blocks && i < r.n_blocks ? sr + x[u].x : sr;
      }
    }
    sf = wave_sum(sf); sgg = wave_sum(sgg); sr = wave_sum(sr);
    if ((tid & 63) == 0) { sums[3 * (tid >> 6)] = sf; sums[3 * (tid >> 6) + 1] = sgg; sums[3 * (tid >> 6) + 2] = sr; }
    __syncthreads();
    if (tid == 0) {
      float a = 0.f, b = 0.f, c = 0.f;
      for (int w = 0; w < 4; ++w) { a += sums[3 * w]; b += sums[3 * w + 1]; c += sums[3 * w + 2]; }
      if (r.loss_d) *r.loss_d = c * r.inv_nr + a * r.inv_nf;
      if (r.loss_g) *r.loss_g = b * r.inv_nf;
    }
    return;
  }
  // one parameter row: its events fill blocks t0..t1; a block holds the row in
  // slot 0 if the row starts at or before the block, else in slot 1.  Thread
  // (component c, slice s) sums blocks t0 + s, t0 + s + S, ...; slices combined in order.
  const int row = blockIdx.x - r.wg_blocks - 1;
  const int S = 256 / r.C;
  const int c = tid % r.C, sl = tid / r.C;
  float s = 0.f;
  if (sl < S) {
    const int64_t t0 = (int64_t)row * r.E / kSub, t1 = ((int64_t)row * r.E + r.E - 1) / kSub;
    for (int64_t t = t0 + sl; t <= t1; t += S) {
      const int slot = (t * kSub) / r.E == row ? 0 : 1;
      s += r.theta_part[(t * 2 + slot) * r.C + c];
    }
  }
  sums[tid] = s;
  __syncthreads();
  if (tid < r.C) {
    float t = 0.f;
    for (int q = 0; q < S; ++q) t += sums[q * r.C + tid];
    r.dLg_dtheta[row * r.C + tid] = t;
  }
}

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct Layout {
  int n_wg;              // workgroups: one per CU, at most one per tile
  int n_fake_tiles, n_tiles, blocks_per_tile;
  size_t off_wt, off_wg, off_loss, off_theta, total;
  size_t counted;        // what counts against the no-allocation call's limit
};

template <int H, int NH, int DX, int F, int FEAT>
Layout layout_for(const DiscArgs& a, int n_cu) {
  using K = Fused<H, NH, DX, F, FEAT>;
  Layout L;
  L.n_fake_tiles = (int)((a.n_fake + K::T - 1) / K::T);
  L.n_tiles = L.n_fake_tiles + (int)((a.n_real + K::T - 1) / K::T);
  L.blocks_per_tile = K::WE;
  L.n_wg = std::min(n_cu, L.n_tiles);
  size_t o = 0;
  L.off_wt = o; o += align256(2 * NH * split_copy_bytes(H));
  L.off_wg = o; o += align256(sizeof(float) * (size_t)L.n_wg * padded(K::P));
  L.off_loss = o; o += align256(sizeof(float) * 2 * (size_t)L.n_tiles * K::WE);
  L.off_theta = o; o += align256(sizeof(float) * 2 * 2 * DX * (size_t)L.n_fake_tiles * K::WE);
  L.total = o;
  // The no-allocation call's limit depends on what a call sums, not on how operands are
  // laid out: one fp32 copy of the hidden weights, a row of P values per CU, and the
  // partials of each 64 events.  The rest lies in kNoallocReserve.
  const size_t fake = (size_t)((a.n_fake + kSub - 1) / kSub), real = (size_t)((a.n_real + kSub - 1) / kSub);
  L.counted = align256(sizeof(float) * NH * H * H) + align256(sizeof(float) * (size_t)n_cu * K::P) +
              align256(sizeof(float) * 2 * (fake + real)) + align256(sizeof(float) * 2 * 2 * DX * fake);
  static_assert(2 * NH * split_copy_bytes(H) - sizeof(float) * NH * H * H + 4096 * sizeof(float) < kNoallocReserve,
                "split copies beyond the weights' own size, and up to 3 floats of padding a row of up to 1,024 CUs");
  return L;
}

typedef void (*KernelFn)(F32Params);

struct Variant {
  int H, NH, DX, F, FEAT;
  KernelFn fn;
  Layout (*layout)(const DiscArgs&, int);
  int P;
};

#define SAGIPS_F32_VARIANT(H_, NH_, DX_, F_, FEAT_)                                          \
  { H_, NH_, DX_, F_, FEAT_, k_disc_f32<H_, NH_, DX_, F_, FEAT_>, layout_for<H_, NH_, DX_, F_, FEAT_>, \
    Fused<H_, NH_, DX_, F_, FEAT_>::P }
#define SAGIPS_F32_ID(H_, NH_, D_) SAGIPS_F32_VARIANT(H_, NH_, D_, D_, SAGIPS_FEAT_IDENTITY)

const Variant kVariants[] = {
    SAGIPS_F32_ID(64, 1, 2),  SAGIPS_F32_ID(64, 2, 2),  SAGIPS_F32_ID(64, 3, 2),
    SAGIPS_F32_ID(128, 1, 2), SAGIPS_F32_ID(128, 2, 2),
    SAGIPS_F32_ID(64, 1, 3),  SAGIPS_F32_ID(64, 2, 3),  SAGIPS_F32_ID(128, 2, 3),
    // the paper's discriminator, 2 -> 128 -> 128 -> 128 -> 128 -> 1, on the two observables
    SAGIPS_F32_VARIANT(128, 3, 3, 2, SAGIPS_FEAT_PROXY2),
};

const Variant* find_variant(const sagips_mlp& D, int d) {
  const int H = D.width[1];
  const int NH = D.n_layers - 2;
  const int F = D.width[0];
  for (const Variant& v : kVariants)
    if (v.H == H && v.NH == NH && v.DX == d && v.F == F && v.FEAT == D.features) return &v;
  return nullptr;
}

}  // namespace

int disc_f32_block() { return kSub; }

bool disc_f32_supported(const sagips_mlp& D, int d, const char** why) {
  if (D.features == SAGIPS_FEAT_HD8) { *why = "fp32 discriminator supports IDENTITY and PROXY2 features"; return false; }
  if (D.features == SAGIPS_FEAT_IDENTITY && D.width[0] != d) { *why = "width[0] must equal d for IDENTITY features"; return false; }
  if (D.n_layers < 3) { *why = "fp32 discriminator needs at least one hidden-to-hidden layer"; return false; }
  for (int l = 1; l < D.n_layers; ++l)
    if (D.width[l] != D.width[1]) { *why = "all hidden widths must be equal"; return false; }
  if (D.width[D.n_layers] != 1) { *why = "last layer must have width 1"; return false; }
  if (!find_variant(D, d)) {
    *why = "unsupported fp32 shape (IDENTITY: hidden width 64 with 1-3 or 128 with 1-2 hidden-to-hidden layers, "
           "d 2, or 3 with fewer layers; PROXY2: hidden width 128 with 3 hidden-to-hidden layers)";
    return false;
  }
  return true;
}

size_t disc_f32_workspace(const DiscArgs& a, int n_cu, size_t* counted) {
  const Layout L = find_variant(*a.D, a.d)->layout(a, n_cu);
  *counted = L.counted;
  return L.total;
}

hipError_t launch_disc_f32(const DiscArgs& a, void* ws, int n_cu, hipStream_t st, Timer* tm) {
  const Variant* v = find_variant(*a.D, a.d);
  const sagips_mlp& D = *a.D;
  const Layout L = v->layout(a, n_cu);
  char* base = static_cast<char*>(ws);
  u16* Wf = reinterpret_cast<u16*>(base + L.off_wt);
  const int H = v->H, NH = v->NH, F = v->F, DX = v->DX;

  F32Params p;
  memset(&p, 0, sizeof(p));
  p.W1 = D.W[0];
  p.b1 = D.b[0];
  p.Wf = Wf;
  for (int l = 0; l < NH; ++l) p.bh[l] = D.b[1 + l];
  p.Wo = D.W[NH + 1];
  p.bo = D.b[NH + 1];
  p.slope = D.leaky_slope;
  p.fake_x = a.fake_x;
  p.real_x = a.real_x;
  if (a.fake_src) p.src = *a.fake_src;
  p.n_fake = a.n_fake;
  p.n_real = a.n_real;
  p.n_fake_tiles = L.n_fake_tiles;
  p.n_tiles = L.n_tiles;
  p.fake_rem = L.n_fake_tiles % L.n_wg;
  p.E = a.fake_src ? a.fake_src->E : 1;
  p.inv_nf = 1.0f / (float)a.n_fake;
  p.inv_nr = 1.0f / (float)a.n_real;
  p.logits_fake = a.out->logits_fake;
  p.logits_real = a.out->logits_real;
  p.dLg_dx = a.out->dLg_dx;
  p.wg_part = reinterpret_cast<float*>(base + L.off_wg);
  p.loss_part = reinterpret_cast<float*>(base + L.off_loss);
  p.theta_part = reinterpret_cast<float*>(base + L.off_theta);

  if (tm) tm->begin("disc_f32_split");
  {
    SplitArgs sa;
    memset(&sa, 0, sizeof(sa));
    for (int l = 0; l < NH; ++l) sa.W[l] = D.W[1 + l];
    sa.out = Wf;
    hipLaunchKernelGGL(k_split_weights, dim3(H * H / 8 / 256, 2, NH), dim3(256), 0, st, sa, H, NH);
  }
  if (tm) tm->end();
  if (tm) tm->begin("disc_f32_fused");
  hipLaunchKernelGGL(v->fn, dim3(L.n_wg), dim3(kThreads), 0, st, p);
  if (tm) tm->end();
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;

  ReduceArgs r;
  memset(&r, 0, sizeof(r));
  r.wg_part = p.wg_part;
  r.n_wg = L.n_wg;
  r.P = v->P;
  r.PS = padded(v->P);
  if (a.out->dW[0]) {
    Segments& sg = r.sg;
    int n = 0;
    for (int l = 0; l < NH; ++l) {
      sg.off[n] = l * (H * H + H); sg.len[n] = H * H; sg.dst[n++] = a.out->dW[1 + l];
      sg.off[n] = l * (H * H + H) + H * H; sg.len[n] = H; sg.dst[n++] = a.out->db[1 + l];
    }
    const int offw1 = NH * (H * H + H);
    sg.off[n] = offw1; sg.len[n] = H * F; sg.dst[n++] = a.out->dW[0];
    sg.off[n] = offw1 + H * F; sg.len[n] = H; sg.dst[n++] = a.out->db[0];
    const int offwo = offw1 + H * F + H;
    sg.off[n] = offwo; sg.len[n] = H; sg.dst[n++] = a.out->dW[NH + 1];
    sg.off[n] = offwo + H; sg.len[n] = 1; sg.dst[n++] = a.out->db[NH + 1];
    sg.n = n;
    r.wg_blocks = (v->P + kRedElems - 1) / kRedElems;
  }
  r.loss_part = p.loss_part;
  r.n_fake_blocks = L.n_fake_tiles * L.blocks_per_tile;
  r.n_blocks = L.n_tiles * L.blocks_per_tile;
  r.inv_nf = p.inv_nf;
  r.inv_nr = p.inv_nr;
  r.loss_d = a.out->loss_d;
  r.loss_g = a.out->loss_g;
  r.theta_part = p.theta_part;
  r.E = p.E;
  r.C = 2 * DX;
  r.n_theta = a.fake_src ? a.fake_src->n_theta : 0;
  r.dLg_dtheta = a.out->dLg_dtheta;
  const int rows = (a.fake_src && a.out->dLg_dtheta) ? a.fake_src->n_theta : 0;
  if (tm) tm->begin("disc_f32_reduce");
  hipLaunchKernelGGL(k_reduce_all, dim3(r.wg_blocks + 1 + rows), dim3(256), 0, st, r);
  if (tm) tm->end();
  return hipGetLastError();
}

}  // namespace sagips
