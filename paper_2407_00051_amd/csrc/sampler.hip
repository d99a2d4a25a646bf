// Event sampler and per-parameter gradient reduction on gfx950.
//
// Both kernels run on a 2D grid: blockIdx.y is the parameter row (so theta
// and its reciprocals are wave-uniform scalars) and blockIdx.x a chunk of
// kEPB consecutive events of that row.  Thread t of a chunk handles events
// chunk*kEPB + t + j*256, j < kEPT, so every store is coalesced.
#include "device_math.hpp"
#include "kernels.hpp"

#include <algorithm>

namespace sagips {
namespace {

constexpr int kThreads = 256;
constexpr int kEPT = 8;
constexpr int kEPB = kThreads * kEPT;

template <int D>
__global__ __launch_bounds__(kThreads) void k_sample(SourceArgs s, float* __restrict__ x,
                                                     uint32_t* __restrict__ words) {
  const int row = blockIdx.y;
  Shape sh[D];
#pragma unroll
  for (int j = 0; j < D; ++j) sh[j] = make_shape(s.theta[row * 2 * D + 2 * j], s.theta[row * 2 * D + 2 * j + 1]);
  const int64_t k_first = (int64_t)blockIdx.x * kEPB + threadIdx.x;
  const int64_t row_base = (int64_t)row * s.E;
#pragma unroll 2
  for (int e = 0; e < kEPT; ++e) {
    const int64_t k = k_first + e * kThreads;
    if (k >= s.E) break;
    const int64_t i = row_base + k;
    const Words w = event_words(s.base + (uint64_t)i, s.stream, s.k0, s.k1);
    if (words) {
      uint4 v;
      v.x = w.w[0]; v.y = w.w[1]; v.z = w.w[2]; v.w = w.w[3];
      reinterpret_cast<uint4*>(words)[i] = v;
    }
    if (x) {
      float xv[D];
#pragma unroll
      for (int j = 0; j < D; ++j) xv[j] = kumaraswamy_w(w.w[j], sh[j]).x;
      if constexpr (D == 2) {
        reinterpret_cast<float2*>(x)[i] = make_float2(xv[0], xv[1]);
      } else {
#pragma unroll
        for (int j = 0; j < D; ++j) x[i * D + j] = xv[j];
      }
    }
  }
}

// Per-chunk partial sums of dL/dtheta (2D values) and, for the quadratic
// critic, of the loss: partial[(row * chunks + chunk) * stride + c], stride =
// 2D + 1, or 2D without the loss where a row is one chunk and the partials are
// dL/dtheta itself.
template <int D, bool kQuadratic>
__global__ __launch_bounds__(kThreads) void k_param_grad(SourceArgs s, const float* __restrict__ dLdx,
                                                         float* __restrict__ partial, int stride) {
  constexpr int C = 2 * D + 1;
  __shared__ float red[kThreads / 64][C];
  const int row = blockIdx.y;
  Shape sh[D];
#pragma unroll
  for (int j = 0; j < D; ++j) sh[j] = make_shape(s.theta[row * 2 * D + 2 * j], s.theta[row * 2 * D + 2 * j + 1]);
  float acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0f;
  const int64_t k_first = (int64_t)blockIdx.x * kEPB + threadIdx.x;
  const int64_t row_base = (int64_t)row * s.E;
#pragma unroll 2
  for (int e = 0; e < kEPT; ++e) {
    const int64_t k = k_first + e * kThreads;
    if (k >= s.E) break;
    const int64_t i = row_base + k;
    const Words w = event_words(s.base + (uint64_t)i, s.stream, s.k0, s.k1);
    float gx[D];
    if constexpr (!kQuadratic) {
      if constexpr (D == 2) {
        const float2 v = reinterpret_cast<const float2*>(dLdx)[i];
        gx[0] = v.x; gx[1] = v.y;
      } else {
#pragma unroll
        for (int j = 0; j < D; ++j) gx[j] = dLdx[i * D + j];
      }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const Quantile q = kumaraswamy_w(w.w[j], sh[j]);
      float da, db;
      pathwise(q, sh[j], da, db);
      float g;
      if constexpr (kQuadratic) {
        const float r = q.x - 0.5f;
        g = 2.0f * r;
        acc[2 * D] = fmaf(r, r, acc[2 * D]);
      } else {
        g = gx[j];
      }
      acc[2 * j] = fmaf(g, da, acc[2 * j]);
      acc[2 * j + 1] = fmaf(g, db, acc[2 * j + 1]);
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float v = wave_sum(acc[c]);
    if (lane == 0) red[wave][c] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < stride) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) v += red[w][threadIdx.x];
    partial[((int64_t)row * gridDim.x + blockIdx.x) * stride + threadIdx.x] = v;
  }
}

// One block per row: fixed-order sum of the row's chunk partials.
__global__ __launch_bounds__(kThreads) void k_reduce_rows(const float* __restrict__ partial, int chunks, int C,
                                                          float* __restrict__ dLdtheta, float* __restrict__ row_loss,
                                                          int has_loss) {
  __shared__ float red[kThreads / 64];
  const int row = blockIdx.x;
  const float* p = partial + (int64_t)row * chunks * C;
  for (int c = 0; c < C; ++c) {
    if (c == C - 1 && !has_loss) break;
    float v = 0.0f;
    for (int k = threadIdx.x; k < chunks; k += kThreads) v += p[(int64_t)k * C + c];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = 0.0f;
      for (int w = 0; w < kThreads / 64; ++w) t += red[w];
      if (c < C - 1) dLdtheta[row * (C - 1) + c] = t;
      else row_loss[row] = t;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kThreads) void k_reduce_loss(const float* __restrict__ row_loss, int n,
                                                          float* __restrict__ loss) {
  __shared__ float red[kThreads / 64];
  float v = 0.0f;
  for (int k = threadIdx.x; k < n; k += kThreads) v += row_loss[k];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < kThreads / 64; ++w) t += red[w];
    *loss = t;
  }
}

inline int chunks_per_row(const SourceArgs& s) { return (int)((s.E + kEPB - 1) / kEPB); }

// Bootstrap draws, one per thread (grid-stride): draw i takes row
// floor(w0 * n_data / 2^32), w0 the first Philox word of counter
// (i lo, i hi, stream, step).  The rows are gathered (8 or 12 bytes each) and
// written back contiguously.
template <int D>
__global__ __launch_bounds__(kThreads) void k_bootstrap(const float* __restrict__ data, uint64_t n_data, uint32_t k0,
                                                        uint32_t k1, uint32_t step, int64_t n_out,
                                                        float* __restrict__ out, int64_t* __restrict__ idx_out) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_out; i += stride) {
    const Words w = philox4x32_10((uint32_t)i, (uint32_t)((uint64_t)i >> 32), SAGIPS_STREAM_BOOTSTRAP, step, k0, k1);
    const uint64_t r = ((uint64_t)w.w[0] * n_data) >> 32;    // < n_data <= 2^32: the product fits in 64 bits
    if (idx_out) idx_out[i] = (int64_t)r;
    if constexpr (D == 2) {
      reinterpret_cast<float2*>(out)[i] = reinterpret_cast<const float2*>(data)[r];
    } else {
#pragma unroll
      for (int j = 0; j < D; ++j) out[i * D + j] = data[r * D + j];
    }
  }
}

// The same draws listed in ascending row order, by a counting sort over
// slabs of 2^kSlabBits consecutive rows of the reference data:
//   k_boot_count    each chunk of draws: its rows (kept for the scatter) and a
//                   per-slab count, [slab][chunk]
//   k_boot_scan     per slab, the exclusive scan of its chunk counts, and the
//                   slab's total
//   k_boot_scatter  the chunk's draws sorted by slab in LDS, then each slab's run
//                   of row offsets within it (16 bits) written to the slab's
//                   segment, at the chunk's place (the segments start at the
//                   exclusive scan of the totals)
//                   (k_boot_scatter_few: without the sort, where a chunk has few
//                   draws of a slab)
//   k_boot_expand   per slab: a histogram of the offsets in LDS, its scan, then
//                   every drawn row listed at its output positions; rows are read
//                   nearly in order and written in order.
// Placement within a (slab, chunk) segment follows LDS atomics, but the final
// output is the unique ascending listing of the drawn rows.
constexpr int kSlabBits = 14;
constexpr int kSlabRows = 1 << kSlabBits;
constexpr int kBootBig = 1024;     // threads of the count, scatter and expand kernels

__global__ __launch_bounds__(kBootBig) void k_boot_count(uint64_t n_data, uint32_t k0, uint32_t k1, uint32_t step,
                                                         int64_t n_out, int64_t per_chunk, int n_slabs, int n_chunks,
                                                         uint32_t* __restrict__ rows, uint32_t* __restrict__ cnt) {
  extern __shared__ uint32_t hist[];   // [n_slabs]
  for (int s = threadIdx.x; s < n_slabs; s += kBootBig) hist[s] = 0u;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * per_chunk, i1 = min(n_out, i0 + per_chunk);
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kBootBig) {
    const Words w = philox4x32_10((uint32_t)i, (uint32_t)((uint64_t)i >> 32), SAGIPS_STREAM_BOOTSTRAP, step, k0, k1);
    const uint32_t r = (uint32_t)(((uint64_t)w.w[0] * n_data) >> 32);
    rows[i] = r;
    atomicAdd(&hist[r >> kSlabBits], 1u);
  }
  __syncthreads();
  for (int s = threadIdx.x; s < n_slabs; s += kBootBig) cnt[(int64_t)s * n_chunks + blockIdx.x] = hist[s];
}

// One wave per slab: exclusive scan of cnt[slab][0 .. n_chunks) in place, and
// the slab's total.
__global__ __launch_bounds__(64) void k_boot_scan(uint32_t* __restrict__ cnt, int n_chunks,
                                                  uint32_t* __restrict__ total) {
  uint32_t* c = cnt + (int64_t)blockIdx.x * n_chunks;
  const int lane = threadIdx.x;
  uint32_t carry = 0u;
  for (int b = 0; b < n_chunks; b += 64) {
    const int j = b + lane;
    const uint32_t v = j < n_chunks ? c[j] : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (j < n_chunks) c[j] = carry + incl - v;
    carry += __shfl(incl, 63, 64);
  }
  if (lane == 0) total[blockIdx.x] = carry;
}

// Exclusive prefix of v over the kBootBig threads of a workgroup, and the total
// in *sum; part holds one word per wave and one more.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* part, uint32_t* sum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  uint32_t off = 0u, all = 0u;
#pragma unroll
  for (int w = 0; w < kBootBig / 64; ++w) {
    const uint32_t t = part[w];
    off += w < wave ? t : 0u;
    all += t;
  }
  __syncthreads();                 // part may be used again
  *sum = all;
  return off + incl - v;
}

// Largest v of the threads before this one (0 for the first).
__device__ __forceinline__ uint32_t block_max_before(uint32_t v, uint32_t* part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl = max(incl, t);
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  uint32_t m = __shfl_up(incl, 1, 64);
  if (lane == 0) m = 0u;
#pragma unroll
  for (int w = 0; w < kBootBig / 64; ++w)
    if (w < wave) m = max(m, part[w]);
  return m;
}

// The draws of a chunk, at most kBootBatch at a time.  Writing each draw's 16-bit
// offset straight to its slab's segment reached HBM as partial lines (405 MB for
// 33.5 MB of offsets at 16.8M draws from 2,048 slabs, 164 us): the lines a
// workgroup is filling do not fit its share of L2.  Sorted in LDS first, a slab's
// run (16 to 64 draws) leaves as one contiguous store.
constexpr int kBootBatch = 40960;            // 80 KB of offsets
constexpr int kMaxSlabs = 1 << 13;           // n_data <= 2^27

__global__ __launch_bounds__(kBootBig) void k_boot_scatter(const uint32_t* __restrict__ rows, int64_t n_out,
                                                           int64_t per_chunk, int n_slabs, int n_chunks,
                                                           const uint32_t* __restrict__ cnt,
                                                           const uint32_t* __restrict__ total,
                                                           uint32_t* __restrict__ base, uint16_t* __restrict__ keys) {
  __shared__ uint16_t sorted[kBootBatch];
  __shared__ uint32_t loc[kMaxSlabs];        // the batch's count, then its place, per slab
  __shared__ uint32_t gcur[kMaxSlabs];       // where the slab's next run goes
  __shared__ uint32_t part[kBootBig / 64 + 1];
  const int t = threadIdx.x, chunk = blockIdx.x;
  const int per = (n_slabs + kBootBig - 1) / kBootBig, s0 = min(n_slabs, t * per), s1 = min(n_slabs, s0 + per);
  const int64_t i0 = (int64_t)chunk * per_chunk, i1 = min(n_out, i0 + per_chunk);
  const bool single = per_chunk <= kBootBatch;   // then the chunk's counts are the table's
  {   // segment starts: exclusive scan of the totals (kept for the expansion by workgroup 0)
    uint32_t v = 0u, all;
    for (int s = s0; s < s1; ++s) v += total[s];
    uint32_t run = block_scan(v, part, &all);
    for (int s = s0; s < s1; ++s) {
      const uint32_t c = cnt[(int64_t)s * n_chunks + chunk], tot = total[s];
      gcur[s] = run + c;
      if (single) loc[s] = (chunk + 1 < n_chunks ? cnt[(int64_t)s * n_chunks + chunk + 1] : tot) - c;
      if (chunk == 0) base[s] = run;
      run += tot;
    }
    if (chunk == 0 && t == 0) base[n_slabs] = all;
  }
  for (int64_t b0 = i0; b0 < i1; b0 += kBootBatch) {
    const int64_t b1 = min(i1, b0 + kBootBatch);
    if (!single) {
      __syncthreads();
      for (int s = t; s < n_slabs; s += kBootBig) loc[s] = 0u;
      __syncthreads();
      for (int64_t i = b0 + t; i < b1; i += kBootBig) atomicAdd(&loc[rows[i] >> kSlabBits], 1u);
      __syncthreads();
    }
    uint32_t v = 0u, all;
    for (int s = s0; s < s1; ++s) v += loc[s];
    uint32_t run = block_scan(v, part, &all);
    for (int s = s0; s < s1; ++s) {
      const uint32_t c = loc[s];
      loc[s] = run;
      run += c;
    }
    __syncthreads();
    for (int64_t i = b0 + t; i < b1; i += kBootBig) {
      const uint32_t r = rows[i];
      sorted[atomicAdd(&loc[r >> kSlabBits], 1u)] = (uint16_t)(r & (kSlabRows - 1));
    }
    __syncthreads();               // loc[s] is now the end of slab s's run
    // half a wave per slab
    for (int s = t >> 5; s < n_slabs; s += kBootBig / 32) {
      const uint32_t a = s ? loc[s - 1] : 0u, e = loc[s], g = gcur[s];
      for (uint32_t q = a + (t & 31); q < e; q += 32) keys[g + (q - a)] = sorted[q];
      if (!single && (t & 31) == 0) gcur[s] = g + (e - a);
    }
  }
}

// The same without the sort, for tables of so many slabs that a chunk has only a few draws
// of each (min_run): each draw straight to its slab's segment.
__global__ __launch_bounds__(kBootBig) void k_boot_scatter_few(const uint32_t* __restrict__ rows, int64_t n_out,
                                                               int64_t per_chunk, int n_slabs, int n_chunks,
                                                               const uint32_t* __restrict__ cnt,
                                                               const uint32_t* __restrict__ total,
                                                               uint32_t* __restrict__ base, uint16_t* __restrict__ keys) {
  __shared__ uint32_t cursor[kMaxSlabs];
  __shared__ uint32_t part[kBootBig / 64 + 1];
  const int t = threadIdx.x, chunk = blockIdx.x;
  const int per = (n_slabs + kBootBig - 1) / kBootBig, s0 = min(n_slabs, t * per), s1 = min(n_slabs, s0 + per);
  for (int s = t; s < n_slabs; s += kBootBig) cursor[s] = total[s];
  __syncthreads();
  uint32_t v = 0u, all;
  for (int s = s0; s < s1; ++s) v += cursor[s];
  uint32_t run = block_scan(v, part, &all);
  for (int s = s0; s < s1; ++s) {
    const uint32_t tot = cursor[s];
    cursor[s] = run;
    run += tot;
  }
  __syncthreads();
  for (int s = t; s < n_slabs; s += kBootBig) {
    const uint32_t b = cursor[s];
    cursor[s] = b + cnt[(int64_t)s * n_chunks + chunk];
    if (chunk == 0) base[s] = b;
  }
  if (chunk == 0 && t == 0) base[n_slabs] = all;
  __syncthreads();
  const int64_t i0 = (int64_t)chunk * per_chunk, i1 = min(n_out, i0 + per_chunk);
  for (int64_t i = i0 + t; i < i1; i += kBootBig) {
    const uint32_t r = rows[i];
    keys[atomicAdd(&cursor[r >> kSlabBits], 1u)] = (uint16_t)(r & (kSlabRows - 1));
  }
}

template <int D>
__global__ __launch_bounds__(kBootBig) void k_boot_expand(const float* __restrict__ data, const uint16_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ base, float* __restrict__ out,
                                                          int64_t* __restrict__ idx_out) {
  __shared__ __attribute__((aligned(16))) uint32_t h[kSlabRows];
  __shared__ uint32_t part[kBootBig / 64 + 1];
  constexpr int PER = kSlabRows / kBootBig;   // 16 histogram entries per thread
  constexpr uint32_t kWin = 16 * kBootBig;    // output positions listed at a time, in h's place
  const int t = threadIdx.x;
  const uint32_t b0 = base[blockIdx.x], b1 = base[blockIdx.x + 1];
  for (int j = t; j < kSlabRows; j += kBootBig) h[j] = 0u;
  __syncthreads();
  for (uint32_t p = b0 + t; p < b1; p += kBootBig) atomicAdd(&h[keys[p]], 1u);
  __syncthreads();
  uint32_t c[PER], s = 0u, all;
#pragma unroll
  for (int j = 0; j < PER; j += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(&h[t * PER + j]);
    c[j] = v.x; c[j + 1] = v.y; c[j + 2] = v.z; c[j + 3] = v.w;
    s += v.x + v.y + v.z + v.w;
  }
  const uint32_t off = block_scan(s, part, &all);   // (every count is read before the list overwrites h)
  // list[x - w]: row of output position x, for a window of positions at a time.
  // Every drawn row marks its first position in the window; a running maximum over
  // the positions (16 per thread) then fills the others, at a cost that does not
  // depend on how often a row is drawn.
  uint16_t* list = reinterpret_cast<uint16_t*>(h);
  uint4* list4 = reinterpret_cast<uint4*>(h) + 2 * t;
  const uint64_t row0 = (uint64_t)blockIdx.x << kSlabBits;
  for (uint32_t w = 0; w < all; w += kWin) {
    const uint32_t end = min(all, w + kWin);
    list4[0] = list4[1] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint32_t q = off;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint32_t e = q + c[j], x = max(q, w);
      if (x < min(e, end)) list[x - w] = (uint16_t)(t * PER + j);
      q = e;
    }
    __syncthreads();
    uint32_t v[8], m = 0u;
    *reinterpret_cast<uint4*>(&v[0]) = list4[0];
    *reinterpret_cast<uint4*>(&v[4]) = list4[1];
#pragma unroll
    for (int k = 0; k < 8; ++k) m = max(m, max(v[k] & 0xffffu, v[k] >> 16));
    m = block_max_before(m, part);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t lo = max(m, v[k] & 0xffffu);
      m = max(lo, v[k] >> 16);
      v[k] = lo | (m << 16);
    }
    list4[0] = *reinterpret_cast<uint4*>(&v[0]);
    list4[1] = *reinterpret_cast<uint4*>(&v[4]);
    __syncthreads();
    for (uint32_t x = w + t; x < end; x += kBootBig) {
      const uint64_t r = row0 + list[x - w];
      const int64_t p = (int64_t)b0 + x;
      if (idx_out) idx_out[p] = (int64_t)r;
      if constexpr (D == 2) {
        reinterpret_cast<float2*>(out)[p] = reinterpret_cast<const float2*>(data)[r];
      } else {
#pragma unroll
        for (int j = 0; j < D; ++j) out[p * D + j] = data[r * D + j];
      }
    }
    __syncthreads();               // the list is read before the next window overwrites it
  }
}

}  // namespace

hipError_t launch_bootstrap(const float* data, uint64_t n_data, int d, uint32_t k0, uint32_t k1, uint32_t step,
                            int64_t n_out, float* out, int64_t* idx_out, int n_cu, hipStream_t st, Timer* tm) {
  const int64_t want = (n_out + kThreads - 1) / kThreads;
  const int blocks = (int)std::min<int64_t>(want, (int64_t)n_cu * 32);
  if (tm) tm->begin("bootstrap");
  if (d == 2) hipLaunchKernelGGL(k_bootstrap<2>, dim3(blocks), dim3(kThreads), 0, st, data, n_data, k0, k1, step, n_out, out, idx_out);
  else hipLaunchKernelGGL(k_bootstrap<3>, dim3(blocks), dim3(kThreads), 0, st, data, n_data, k0, k1, step, n_out, out, idx_out);
  if (tm) tm->end();
  return hipGetLastError();
}

namespace {

struct RowsPlan {
  int n_slabs, n_chunks;
  int64_t per_chunk;       // draws
  bool sorted;             // k_boot_scatter, else k_boot_scatter_few
};

// Draws of a slab in a chunk (its run) from which sorting the chunk first pays.  The sort
// costs each chunk a pass over the slabs; without it the lines that the draws are filling
// are written to HBM partly filled, the more chunks run side by side, the more of them.
// So 16 for one chunk down to 3.5 for one per CU; beyond, where the last round of sorting
// workgroups may be nearly empty, 4.  us a call, unsorted and sorted (n_data up to 2^27):
// 1M draws (62 chunks) in runs of 16, 11, 8, 4, 2: 53 51, 61 62, 70 75, 102 123, 168 223;
// 3M (184) in runs of 16, 8, 5, 4: 68 64, 94 91, 118 116, 140 145; 6M (256) in runs of 4, 3:
// 257 239, 287 291; 10M (306) in runs of 8, 5, 4: 283 270, 328 346, 382 439; 16.8M (512) in
// runs of 16, 8, 4: 299 201, 380 299, 495 487.
double min_run(int n_chunks) { return n_chunks <= 256 ? 16.0 - 12.5 * n_chunks / 256 : 4.0; }

RowsPlan rows_plan(uint64_t n_data, int64_t n_out) {
  RowsPlan p;
  p.n_slabs = (int)((n_data + kSlabRows - 1) / kSlabRows);
  const auto chunks = [&](int64_t n) {
    p.n_chunks = (int)std::min<int64_t>(1024, std::max<int64_t>(1, n));
    p.per_chunk = (n_out + p.n_chunks - 1) / p.n_chunks;
  };
  // one chunk per CU from 16,384 draws each; sorted, one batch of the scatter per chunk
  // where that takes at most 1,024 chunks
  const int64_t by_batch = (n_out + 32767) / 32768, by_cu = std::min<int64_t>(256, (n_out + 16383) / 16384);
  chunks(std::max(by_batch, by_cu));
  p.sorted = (double)std::min<int64_t>(p.per_chunk, kBootBatch) >= min_run(p.n_chunks) * p.n_slabs;
  if (!p.sorted) chunks(by_cu);
  return p;
}

inline size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t bootstrap_rows_workspace(uint64_t n_data, int64_t n_out) {
  const RowsPlan p = rows_plan(n_data, n_out);
  return al256(4 * (size_t)n_out) + al256(2 * (size_t)n_out) + al256(4 * (size_t)p.n_slabs * p.n_chunks) +
         al256(4 * (size_t)p.n_slabs) + al256(4 * ((size_t)p.n_slabs + 1));
}

hipError_t launch_bootstrap_rows(const float* data, uint64_t n_data, int d, uint32_t k0, uint32_t k1, uint32_t step,
                                 int64_t n_out, float* out, int64_t* idx_out, void* ws, hipStream_t st, Timer* tm) {
  const RowsPlan p = rows_plan(n_data, n_out);
  const int n_slabs = p.n_slabs, n_chunks = p.n_chunks;
  const int64_t per_chunk = p.per_chunk;
  char* w = static_cast<char*>(ws);
  uint32_t* rows = reinterpret_cast<uint32_t*>(w);
  w += al256(4 * (size_t)n_out);
  uint16_t* keys = reinterpret_cast<uint16_t*>(w);
  w += al256(2 * (size_t)n_out);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(w);
  w += al256(4 * (size_t)n_slabs * n_chunks);
  uint32_t* total = reinterpret_cast<uint32_t*>(w);
  w += al256(4 * (size_t)n_slabs);
  uint32_t* base = reinterpret_cast<uint32_t*>(w);
  const size_t lds = sizeof(uint32_t) * (size_t)n_slabs;
  if (tm) tm->begin("bootstrap_rows");
  hipLaunchKernelGGL(k_boot_count, dim3(n_chunks), dim3(kBootBig), lds, st, n_data, k0, k1, step, n_out, per_chunk,
                     n_slabs, n_chunks, rows, cnt);
  hipLaunchKernelGGL(k_boot_scan, dim3(n_slabs), dim3(64), 0, st, cnt, n_chunks, total);
  hipLaunchKernelGGL(p.sorted ? k_boot_scatter : k_boot_scatter_few, dim3(n_chunks), dim3(kBootBig), 0, st, rows, n_out,
                     per_chunk, n_slabs, n_chunks, cnt, total, base, keys);
  if (d == 2) hipLaunchKernelGGL(k_boot_expand<2>, dim3(n_slabs), dim3(kBootBig), 0, st, data, keys, base, out, idx_out);
  else hipLaunchKernelGGL(k_boot_expand<3>, dim3(n_slabs), dim3(kBootBig), 0, st, data, keys, base, out, idx_out);
  if (tm) tm->end();
  return hipGetLastError();
}

hipError_t launch_sample(const SourceArgs& s, float* x, uint32_t* words, hipStream_t st, Timer* tm) {
  const dim3 grid(chunks_per_row(s), s.n_theta);
  if (tm) tm->begin("sample_events");
  if (s.d == 2) hipLaunchKernelGGL(k_sample<2>, grid, dim3(kThreads), 0, st, s, x, words);
  else hipLaunchKernelGGL(k_sample<3>, grid, dim3(kThreads), 0, st, s, x, words);
  if (tm) tm->end();
  return hipGetLastError();
}

size_t param_grad_workspace(const SourceArgs& s) {
  const size_t C = 2 * s.d + 1;
  return ((size_t)s.n_theta * chunks_per_row(s) * C + s.n_theta) * sizeof(float);
}

hipError_t launch_param_grad(const SourceArgs& s, const float* dLdx, float* dLdtheta, float* loss, void* ws,
                             hipStream_t st, Timer* tm) {
  const int chunks = chunks_per_row(s);
  const int C = 2 * s.d + 1;
  float* partial = static_cast<float*>(ws);
  float* row_loss = partial + (size_t)s.n_theta * chunks * C;
  const dim3 grid(chunks, s.n_theta);
  const bool quad = (dLdx == nullptr);
  // One chunk a row and no loss: the kernel's sums are the result (E <= 2,048;
  // 3 rows of 1,000 events: 5 us without the 3 us reduction and its launch).
  const bool direct = chunks == 1 && !quad;
  float* dst = direct ? dLdtheta : partial;
  const int stride = direct ? 2 * s.d : C;
  if (tm) tm->begin("param_grad");
  if (s.d == 2) {
    if (quad) hipLaunchKernelGGL((k_param_grad<2, true>), grid, dim3(kThreads), 0, st, s, dLdx, dst, stride);
    else hipLaunchKernelGGL((k_param_grad<2, false>), grid, dim3(kThreads), 0, st, s, dLdx, dst, stride);
  } else {
    if (quad) hipLaunchKernelGGL((k_param_grad<3, true>), grid, dim3(kThreads), 0, st, s, dLdx, dst, stride);
    else hipLaunchKernelGGL((k_param_grad<3, false>), grid, dim3(kThreads), 0, st, s, dLdx, dst, stride);
  }
  if (tm) tm->end();
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || direct) return e;
  if (tm) tm->begin("param_grad_reduce");
  hipLaunchKernelGGL(k_reduce_rows, dim3(s.n_theta), dim3(kThreads), 0, st, partial, chunks, C, dLdtheta, row_loss,
                     quad ? 1 : 0);
  if (quad && loss) hipLaunchKernelGGL(k_reduce_loss, dim3(1), dim3(kThreads), 0, st, row_loss, s.n_theta, loss);
  if (tm) tm->end();
  return hipGetLastError();
}

}  // namespace sagips
