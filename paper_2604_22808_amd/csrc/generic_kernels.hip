// Small helper kernels both paths share: pooling, summaries, band energy, copies, conversions.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {

struct SkipBits { uint64_t w[NBMAX][4]; };   // per band: slices whose summaries of that band are not pooled here (unused, or summed from the untransformed V)
struct BandGeom { int64_t off[NBMAX], n[NBMAX]; int m[NBMAX]; int nb; };   // first row, rows and summary tokens per band; nb bands

// row of band `band`'s token u among the tokens band b != band looks at
__device__ __forceinline__ int summary_pos(const BandGeom& g, int band, int b, int u) {
  int pos = u;
  for (int o = 0; o < band; ++o)
    if (o != b) pos += g.m[o];
  return pos;
}

struct PoolKernelArgs {
  const void* spec[3]; void* low[3]; const int32_t* low_list; int64_t n_low, nbar; int c; int64_t low_vecs; unsigned low_blocks;
  const void* Y; const void* V; void* C; const int32_t* masks; BandGeom g; int m2rows; SkipBits skip; int nsplit, mmax; float* part;
  int64_t N; int d;
};

// The two poolings of band-major rows in one launch (they read the same fresh spectral rows and neither fills the chip):
//  - workgroups [0, low_blocks): low-band compression (section 3.3), mean of c consecutive band rows of Q~, K~ and V~;
//  - the rest: summary tokens (section 3.6, U = I): chunk u of band l covers band rows [floor(u n / m), floor((u+1) n / m)).
//    One workgroup per (slice, band, chunk[, part of the chunk]); thread = VW adjacent channels (16 bytes) of every
//    `groups`-th row, eight rows in flight; partial sums are added in a fixed order, so results do not depend on
//    scheduling.  The mean goes to the C rows of the other bands (ascending band index).
// What bounds it: at ordinary sizes the latency of one chunk (16 waves per workgroup: a chunk of 115 KB takes seven loads
// per thread); chunks above 1 MB are cut into parts that meet in k_summaries_finish.  Compression (3 launches), pooling
// (1-2) and the low band's expansion (1; groups of up to 16 rows are now written by the band operator) took 34 us at 16K tokens x 8 heads x 64, 136 us at
// 256K x 24 x 128 and 78 + 19 us in fp32 at 12,150 x 4 x 64; this launch takes 11, 65 and 8 us.
template <typename T, int VW, int NT>
__global__ void __launch_bounds__(NT) k_band_pools(PoolKernelArgs a) {
  typedef T vec __attribute__((ext_vector_type(VW)));
  __shared__ float part[NT * VW];
  const int d = a.d, tid = threadIdx.x, tpr = d / VW;   // threads per row
  if (blockIdx.x < a.low_blocks) {
    const int64_t idx = (int64_t)blockIdx.x * NT + tid;
    if (idx >= a.low_vecs) return;
    const int cv = (int)(idx % tpr);
    const int64_t r = idx / tpr, j = r % a.nbar;
    const int64_t li = r / a.nbar;
    const int tensor = (int)(li % 3), slice = a.low_list[li / 3];
    const int64_t r0 = j * a.c, r1 = r0 + a.c < a.n_low ? r0 + a.c : a.n_low;
    const T* src = (const T*)a.spec[tensor] + (int64_t)slice * a.N * d + cv * VW;
    float s[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) s[k] = 0.f;
    for (int64_t q = r0; q < r1; ++q) {
      const vec x = *(const vec*)(src + q * d);
#pragma unroll
      for (int k = 0; k < VW; ++k) s[k] += (float)x[k];
    }
    vec o;
#pragma unroll
    for (int k = 0; k < VW; ++k) o[k] = (T)(s[k] / (float)(r1 - r0));
    *(vec*)((T*)a.low[tensor] + ((int64_t)slice * a.nbar + j) * d + cv * VW) = o;
    return;
  }
  unsigned b = blockIdx.x - a.low_blocks;
  const int sp = b % a.nsplit; b /= a.nsplit;
  const int u = b % a.mmax; b /= a.mmax;
  const int band = b % a.g.nb, slice = b / a.g.nb;
  if (slice < 256 && ((a.skip.w[band][slice >> 6] >> (slice & 63)) & 1)) return;
  const int64_t off = a.g.off[band], n = a.g.n[band];
  const int me = a.g.m[band];
  if (u >= me) return;
  const T* src = (const T*)(((a.masks[slice] >> band) & 1) ? a.Y : a.V) + ((int64_t)slice * a.N + off) * d;
  const int64_t c0 = ((int64_t)u * n) / me, c1 = ((int64_t)(u + 1) * n) / me;   // the chunk
  const int64_t r0 = c0 + ((c1 - c0) * sp) / a.nsplit, r1 = c0 + ((c1 - c0) * (sp + 1)) / a.nsplit;
  const int groups = NT / tpr, cv = tid % tpr, grp = tid / tpr;
  float acc[VW];
#pragma unroll
  for (int k = 0; k < VW; ++k) acc[k] = 0.f;
  if (grp < groups) {
    int64_t r = r0 + grp;
    constexpr int INF = 8;   // rows in flight per thread
    for (; r + (INF - 1) * (int64_t)groups < r1; r += INF * (int64_t)groups) {
      vec x[INF];
#pragma unroll
      for (int q = 0; q < INF; ++q) x[q] = *(const vec*)(src + (r + (int64_t)q * groups) * d + cv * VW);
#pragma unroll
      for (int q = 0; q < INF; ++q)
#pragma unroll
        for (int k = 0; k < VW; ++k) acc[k] += (float)x[q][k];
    }
    for (; r < r1; r += groups) {
      const vec x = *(const vec*)(src + r * d + cv * VW);
#pragma unroll
      for (int k = 0; k < VW; ++k) acc[k] += (float)x[k];
    }
#pragma unroll
    for (int k = 0; k < VW; ++k) part[(size_t)grp * d + cv * VW + k] = acc[k];
  }
  __syncthreads();
  for (int ch = tid; ch < d; ch += NT) {
    float t4[4] = {0.f, 0.f, 0.f, 0.f};
    int q = 0;
    for (; q + 3 < groups; q += 4)
#pragma unroll
      for (int k = 0; k < 4; ++k) t4[k] += part[(size_t)(q + k) * d + ch];
    for (; q < groups; ++q) t4[0] += part[(size_t)q * d + ch];
    const float t = (t4[0] + t4[1]) + (t4[2] + t4[3]);
    if (a.nsplit > 1) {   // [slice][band][u][part][d]
      a.part[((((int64_t)slice * a.g.nb + band) * a.mmax + u) * a.nsplit + sp) * d + ch] = t;
      continue;
    }
    const T mean = (T)(t / (float)(c1 - c0));
    for (int o = 0; o < a.g.nb; ++o)
      if (o != band) ((T*)a.C)[(((int64_t)slice * a.g.nb + o) * a.m2rows + summary_pos(a.g, band, o, u)) * d + ch] = mean;
  }
}

// Second stage of pooled chunks that were cut: adds the parts' sums in order and writes the mean rows.
template <typename T>
__global__ void __launch_bounds__(256) k_summaries_finish(PoolKernelArgs a) {
  const int slice = blockIdx.z, band = blockIdx.y, u = blockIdx.x, ch = threadIdx.x, d = a.d;
  if (slice < 256 && ((a.skip.w[band][slice >> 6] >> (slice & 63)) & 1)) return;
  const int64_t n = a.g.n[band];
  const int me = a.g.m[band];
  if (u >= me || ch >= d) return;
  const int64_t c0 = ((int64_t)u * n) / me, c1 = ((int64_t)(u + 1) * n) / me;
  const float* src = a.part + ((((int64_t)slice * a.g.nb + band) * a.mmax + u) * a.nsplit) * d + ch;
  float t = 0.f;
  for (int sp = 0; sp < a.nsplit; ++sp) t += src[(int64_t)sp * d];
  const T mean = (T)(t / (float)(c1 - c0));
  for (int o = 0; o < a.g.nb; ++o)
    if (o != band) ((T*)a.C)[(((int64_t)slice * a.g.nb + o) * a.m2rows + summary_pos(a.g, band, o, u)) * d + ch] = mean;
}

template <typename T, int VW, int NT>
static hipError_t launch_pools_v(PoolKernelArgs& k, int n_low_slices, int slices, hipStream_t st) {
  k.low_vecs = (int64_t)n_low_slices * 3 * k.nbar * (k.d / VW);
  const int64_t low_blocks = (k.low_vecs + NT - 1) / NT;
  const int64_t blocks = low_blocks + (int64_t)slices * k.g.nb * k.mmax * k.nsplit;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  k.low_blocks = (unsigned)low_blocks;
  hipLaunchKernelGGL((k_band_pools<T, VW, NT>), dim3((unsigned)blocks), dim3(NT), 0, st, k);
  if (k.nsplit > 1 && k.mmax > 0)
    hipLaunchKernelGGL(k_summaries_finish<T>, dim3((unsigned)k.mmax, (unsigned)k.g.nb, (unsigned)slices), dim3(256), 0, st, k);
  return hipGetLastError();
}

hipError_t launch_band_pools(const PoolArgs& p, hipStream_t st) {
  PoolKernelArgs k{};
  for (int i = 0; i < 3; ++i) { k.spec[i] = p.spec[i]; k.low[i] = p.low[i]; }
  k.low_list = p.low_list; k.n_low = p.n_low; k.nbar = p.nbar; k.c = p.c;
  k.Y = p.Y; k.V = p.V; k.C = p.C; k.masks = p.masks; k.m2rows = p.m2rows; k.N = p.N; k.d = p.d; k.part = p.part;
  k.nsplit = 1;
  k.g.nb = p.nb;
  int64_t longest = 0;   // rows of the longest chunk that some slice pools
  for (int l = 0; l < NBMAX; ++l) {
    for (int i = 0; i < 4; ++i) k.skip.w[l][i] = p.skip_bits ? p.skip_bits[l * 4 + i] : 0;
    k.g.off[l] = p.band_off[l]; k.g.n[l] = l < p.nb ? p.band_n[l] : 0; k.g.m[l] = l < p.nb ? p.m_eff[l] : 0;
    if (!p.pool) k.g.m[l] = 0;
    k.mmax = std::max(k.mmax, k.g.m[l]);
    if (k.g.m[l] > 0 && (p.pooled_bands >> l & 1)) longest = std::max(longest, (k.g.n[l] + k.g.m[l] - 1) / k.g.m[l]);
  }
  const int slices = k.mmax > 0 ? p.slices : 0;
  const int es = p.is_half ? 2 : 4;
  if (slices > 0 && longest * p.d * es > (1 << 20)) {
    const int64_t fit = p.part_floats / ((int64_t)slices * p.nb * k.mmax * p.d);
    k.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>((longest * p.d * es + (1 << 19) - 1) >> 19, std::min<int64_t>(fit, 64)));
  }
  // Threads per workgroup: sixteen waves on a chunk where there are at most two chunks per compute unit, four otherwise (a
  // workgroup of 1024 has a unit to itself, and its start and end are then exposed: 105 against 65 us with 1,300 chunks).
  const bool wide = (int64_t)p.n_pooled * k.mmax * k.nsplit <= 2 * p.num_cu;
  if (p.is_half) {
    if (p.d % 8 != 0) return hipErrorInvalidValue;
    return wide ? launch_pools_v<half_t, 8, 1024>(k, p.n_low_slices, slices, st) : launch_pools_v<half_t, 8, 256>(k, p.n_low_slices, slices, st);
  }
  if (p.d % 4 == 0) return wide ? launch_pools_v<float, 4, 1024>(k, p.n_low_slices, slices, st) : launch_pools_v<float, 4, 256>(k, p.n_low_slices, slices, st);
  return launch_pools_v<float, 1, 1024>(k, p.n_low_slices, slices, st);
}

// Rows of a low-band group behind its first one, which holds the band operator's output.  One thread per VEC and row.
template <typename VEC>
__global__ void __launch_bounds__(256) k_expand_low(VEC* Y, const int32_t* slice_list, int64_t slice_vecs, int64_t n_low, int c,
                                                    int row_vecs, int64_t total) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int64_t r = idx / row_vecs, i = r % n_low, first = i - i % c;
  if (i == first) return;
  VEC* Ys = Y + slice_list[r / n_low] * slice_vecs + idx % row_vecs;
  Ys[i * row_vecs] = Ys[first * row_vecs];
}
hipError_t launch_expand_low(void* Y, const int32_t* slice_list, int n_slices, int64_t N, int64_t n_low, int c, int64_t row_bytes,
                             hipStream_t st) {
  const int vec = row_bytes % 16 == 0 ? 16 : 4;
  const int64_t row_vecs = row_bytes / vec, total = n_slices * n_low * row_vecs, blocks = (total + 255) / 256;
  if (total == 0) return hipSuccess;
  if (row_bytes % 4 != 0 || blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (vec == 16) hipLaunchKernelGGL(k_expand_low<uint4>, dim3((unsigned)blocks), dim3(256), 0, st, (uint4*)Y, slice_list, N * row_vecs, n_low, c, (int)row_vecs, total);
  else hipLaunchKernelGGL(k_expand_low<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, st, (uint32_t*)Y, slice_list, N * row_vecs, n_low, c, (int)row_vecs, total);
  return hipGetLastError();
}

// Summary tokens of the projected forward (sections 3.1 + 3.6): the mean over a chunk of band rows commutes with the
// value projection, so the rows of the transformed model-width input X~ are pooled once per batch entry -
// P[b][band][u][:] = mean of X~ rows of chunk u (the chunk rule of the kernels above) - and every head's summary tokens
// of a band it passes through are P times its W_V.  Workgroup = (chunk, band, batch entry) x a block of 256 columns:
// 32 threads across the columns (8 each), 8 row phases, eight rows in flight per thread; fixed summation order.
__global__ void __launch_bounds__(256) k_pool_wide(const half_t* __restrict__ X, half_t* __restrict__ P, int64_t N, int dm,
                                                   BandGeom g, int mrows) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  __shared__ float part[8][32][8];
  const int u = blockIdx.x, band = blockIdx.y % g.nb, b = blockIdx.y / g.nb, cb = blockIdx.z;
  const int64_t off = g.off[band];
  const int64_t n = g.n[band];
  const int me = g.m[band];
  const int tid = threadIdx.x, cg = tid & 31, ph = tid >> 5;
  const int col = cb * 256 + cg * 8;
  half_t* dst = P + (((int64_t)b * g.nb + band) * mrows + u) * dm + col;
  const bool live = col < dm;   // (dm is a multiple of 8: a thread's 8 columns are all inside or all outside)
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int64_t c0 = 0, c1 = 0;
  if (u < me && live) {
    c0 = ((int64_t)u * n) / me; c1 = ((int64_t)(u + 1) * n) / me;
    const half_t* src = X + ((int64_t)b * N + off) * dm + col;
    int64_t r = c0 + ph;
    constexpr int INF = 8;
    for (; r + (INF - 1) * 8 < c1; r += INF * 8) {
      h8 x[INF];
#pragma unroll
      for (int k = 0; k < INF; ++k) x[k] = *(const h8*)(src + (r + k * 8) * dm);
#pragma unroll
      for (int k = 0; k < INF; ++k)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += (float)x[k][j];
    }
    for (; r < c1; r += 8) {
      const h8 x = *(const h8*)(src + r * dm);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += (float)x[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) part[ph][cg][j] = acc[j];
  __syncthreads();
  if (ph == 0 && live) {
    const float inv = c1 > c0 ? 1.f / (float)(c1 - c0) : 0.f;   // rows beyond the band's chunk count are zero
    h8 mean;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float t = 0.f;
      for (int q = 0; q < 8; ++q) t += part[q][cg][j];
      mean[j] = (_Float16)(t * inv);
    }
    *(h8*)dst = mean;
  }
}
static BandGeom band_geom(int nb, const int64_t band_off[NBMAX], const int64_t band_n[NBMAX], const int m_eff[NBMAX]) {
  BandGeom g;
  g.nb = nb;
  for (int l = 0; l < NBMAX; ++l) {
    g.off[l] = band_off[l]; g.n[l] = l < nb ? band_n[l] : 0; g.m[l] = l < nb ? m_eff[l] : 0;
  }
  return g;
}
hipError_t launch_pool_wide(const void* X, void* P, int batch, int64_t N, int dm, int nb, const int64_t band_off[NBMAX],
                            const int64_t band_n[NBMAX], const int m_eff[NBMAX], int mrows, hipStream_t st) {
  if (mrows <= 0 || batch <= 0) return hipSuccess;
  if (dm % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pool_wide, dim3((unsigned)mrows, (unsigned)(nb * batch), (unsigned)((dm + 255) / 256)), dim3(256), 0, st,
                     (const half_t*)X, (half_t*)P, N, dm, band_geom(nb, band_off, band_n, m_eff), mrows);
  return hipGetLastError();
}

// T[slice][band][u][:] (the projected pooled rows, mrows per band) -> the slots of C where the other bands of the slice
// look for band `band`'s summary tokens, for every band the slice passes through while it runs another one.
__global__ void __launch_bounds__(256) k_place_summaries(const half_t* __restrict__ T, half_t* __restrict__ C,
                                                         const int32_t* __restrict__ masks, int d, BandGeom g,
                                                         int mrows, int m2rows) {
  const int u = blockIdx.x, band = blockIdx.y, slice = blockIdx.z;
  const int me = g.m[band];
  const int mask = masks[slice] & ((1 << g.nb) - 1);
  if (u >= me || ((mask >> band) & 1) || (mask & ~(1 << band)) == 0) return;
  const half_t* src = T + (((int64_t)slice * g.nb + band) * mrows + u) * d;
  for (int b = 0; b < g.nb; ++b) {
    if (b == band) continue;
    const int pos = summary_pos(g, band, b, u);
    half_t* dst = C + (((int64_t)slice * g.nb + b) * m2rows + pos) * d;
    for (int ch = threadIdx.x; ch < d; ch += 256) dst[ch] = src[ch];
  }
}
hipError_t launch_place_summaries(const void* T, void* C, const int32_t* masks, int slices, int d, int nb, const int m_eff[NBMAX],
                                  int mrows, int m2rows, hipStream_t st) {
  if (mrows <= 0 || slices <= 0) return hipSuccess;
  const int64_t none[NBMAX] = {0, 0, 0, 0};
  hipLaunchKernelGGL(k_place_summaries, dim3((unsigned)mrows, (unsigned)nb, (unsigned)slices), dim3(256), 0, st, (const half_t*)T,
                     (half_t*)C, masks, d, band_geom(nb, none, none, m_eff), mrows, m2rows);
  return hipGetLastError();
}

// Router statistics (section 3.5): per band and channel, the sum of squared coefficients over all slices and the
// three spectral tensors.  Workgroup (chunk, band) adds its rows in a fixed order into part[chunk][band][d]; the
// second kernel adds the chunks in order.  No floating-point atomics, so the result is reproducible.
#define BE_CHUNKS 64
template <typename T>
__global__ void __launch_bounds__(256) k_band_energy(const T* sq, const T* sk, const T* sv, float* part, int slices,
                                                     int64_t N, int d, int64_t off0, int64_t off1, int64_t off2,
                                                     int64_t n0, int64_t n1, int64_t n2) {
  __shared__ float red[256];
  const int chunk = blockIdx.x, band = blockIdx.y;
  const int64_t off = band == 0 ? off0 : band == 1 ? off1 : off2;
  const int64_t n = band == 0 ? n0 : band == 1 ? n1 : n2;
  const int64_t rows = n * slices;  // virtual row index: slice-major
  const int64_t r0 = (chunk * rows) / BE_CHUNKS, r1 = ((chunk + 1) * rows) / BE_CHUNKS;
  const int tid = threadIdx.x;
  const int groups = 256 / d, ch = tid % d, grp = tid / d;
  float s = 0.f;
  if (grp < groups)
    for (int64_t r = r0 + grp; r < r1; r += groups) {
      const int64_t slice = r / n, row = r % n;
      const int64_t e = ((int64_t)slice * N + off + row) * d + ch;
      const float a = (float)sq[e], b = (float)sk[e], c = (float)sv[e];
      s += a * a + b * b + c * c;
    }
  red[tid] = s;
  __syncthreads();
  if (grp == 0) {
    float t = 0.f;
    for (int g2 = 0; g2 < groups; ++g2) t += red[g2 * d + ch];
    part[((int64_t)chunk * 3 + band) * d + ch] = t;
  }
}
__global__ void k_band_energy_final(const float* part, float* stats, int d) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= 3 * d) return;
  float t = 0.f;
  for (int c = 0; c < BE_CHUNKS; ++c) t += part[(int64_t)c * 3 * d + idx];
  stats[idx] = t;
}

hipError_t launch_band_energy(const void* sq, const void* sk, const void* sv, float* stats, int slices, int64_t N, int d,
                              const int64_t band_off[3], const int64_t band_n[3], int is_half, hipStream_t st) {
  // stats holds [3][d] results followed by BE_CHUNKS*3*d partial sums
  float* part = stats + 3 * d;
  dim3 grid(BE_CHUNKS, 3);
  if (is_half)
    hipLaunchKernelGGL(k_band_energy<half_t>, grid, dim3(256), 0, st, (const half_t*)sq, (const half_t*)sk,
                       (const half_t*)sv, part, slices, N, d, band_off[0], band_off[1], band_off[2], band_n[0],
                       band_n[1], band_n[2]);
  else
    hipLaunchKernelGGL(k_band_energy<float>, grid, dim3(256), 0, st, (const float*)sq, (const float*)sk,
                       (const float*)sv, part, slices, N, d, band_off[0], band_off[1], band_off[2], band_n[0], band_n[1],
                       band_n[2]);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_band_energy_final, dim3((3 * d + 255) / 256), dim3(256), 0, st, part, stats, d);
  return hipGetLastError();
}

__global__ void k_fill_zero(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}
hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

// Plain streaming copy, 16 bytes per thread and step: the machine's achievable HBM read+write rate, measured next
// to the transform passes (which are read-once / write-once kernels of the same kind).
__global__ void __launch_bounds__(256) k_probe_copy(const uint4* __restrict__ in, uint4* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) out[i] = in[i];
}
hipError_t launch_probe_copy(const void* in, void* out, int64_t bytes, int num_cu, hipStream_t st) {
  if (bytes < 16) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_probe_copy, dim3((unsigned)(num_cu * 16)), dim3(256), 0, st, (const uint4*)in, (uint4*)out, bytes / 16);
  return hipGetLastError();
}

__global__ void k_copy_slices(const uint4* in, uint4* out, const int32_t* slice_list, int64_t vec_per_slice) {
  const int64_t base = (int64_t)slice_list[blockIdx.y] * vec_per_slice;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < vec_per_slice; i += (int64_t)gridDim.x * blockDim.x)
    out[base + i] = in[base + i];
}
hipError_t launch_copy_slices(const void* in, void* out, const int32_t* slice_list, int n_slices, int64_t slice_bytes,
                              hipStream_t st) {
  if (n_slices <= 0 || slice_bytes <= 0) return hipSuccess;
  if (slice_bytes % 16) return hipErrorInvalidValue;
  const int64_t vec = slice_bytes / 16;
  const unsigned gx = (unsigned)std::min<int64_t>((vec + 255) / 256, 2048);
  hipLaunchKernelGGL(k_copy_slices, dim3(gx, (unsigned)n_slices), dim3(256), 0, st, (const uint4*)in, (uint4*)out,
                     slice_list, vec);
  return hipGetLastError();
}

// Element-wise conversions between the caller's bf16 tensors and fp16 scratch (n a multiple of 8): the dense comparison
// runs the attention kernel's direct-to-LDS path, which needs its operands in fp16 in memory.
__global__ void k_bf16_to_f16(const uint4* in, uint4* out, int64_t nvec) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * blockDim.x) {
    const uint4 v = in[i];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const half_t lo = (half_t)__uint_as_float(w[j] << 16), hi = (half_t)__uint_as_float(w[j] & 0xffff0000u);
      o[j] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    out[i] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}
__global__ void k_f16_to_bf16(const uint4* in, uint4* out, int64_t nvec) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * blockDim.x) {
    const uint4 v = in[i];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t r[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float f = (float)__builtin_bit_cast(half_t, (uint16_t)(h ? (w[j] >> 16) : (w[j] & 0xffffu)));
        uint32_t u = __float_as_uint(f);
        u = (u & 0x7f800000u) == 0x7f800000u ? u : u + 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
        r[h] = u >> 16;
      }
      o[j] = r[0] | (r[1] << 16);
    }
    out[i] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}
hipError_t launch_convert_16(const void* in, void* out, int64_t n, int to_bf16, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (n % 8) return hipErrorInvalidValue;
  const int64_t nvec = n / 8;
  const unsigned gx = (unsigned)std::min<int64_t>((nvec + 255) / 256, 8192);
  if (to_bf16) hipLaunchKernelGGL(k_f16_to_bf16, dim3(gx), dim3(256), 0, st, (const uint4*)in, (uint4*)out, nvec);
  else hipLaunchKernelGGL(k_bf16_to_f16, dim3(gx), dim3(256), 0, st, (const uint4*)in, (uint4*)out, nvec);
  return hipGetLastError();
}

// Fixed-order sum of the per-wave partial statistics written by the fused forward passes of Q, K and V.
// Wave w of a launch worked on column chunk w % (d/64) only, and left [3 bands][64 columns] floats behind (768 bytes).
// Two stages.  Stage 1: ENERGY_PARTS workgroups of 4 x 192 threads (thread = band, column); workgroup b takes the waves
// w = b, b + ENERGY_PARTS, ... of every slot, shared among its four groups of threads (ENERGY_PARTS is a multiple of
// d/64, so all of them belong to chunk b % (d/64)), and reads their 768 bytes whole.  Stage 2: a workgroup per band and
// chunk; 16 threads per channel add the stage-1 sums of every 16th workgroup of the chunk each, then their sums in order.
// With tot_part set, the tensors in slots 0..2 were only computed on the low+mid box: their high-band energy is the
// energy of the input (Parseval, the transform is orthonormal) minus their low and mid energies.
// What bounds the two stages is latency: stage 1 has a few MB of slots to read, so it is spread over the whole chip (one
// workgroup per channel took 13 us of the routed forward at 64K tokens and 41 at 1M, now 6 and 23), and stage 2 shares the
// sums of a channel among 16 threads (one thread walking through them took 16 us, now 5).
#define ENERGY_PARTS 256   // stage-1 workgroups (a multiple of the channel chunks of a token)
__global__ void __launch_bounds__(768) k_energy_reduce1(const float* __restrict__ part, const float* __restrict__ tot_part,
                                                        float* __restrict__ part1 /*[ENERGY_PARTS][3][64]*/, EnergyWaves nw) {
  // four groups of 192 threads share a workgroup's waves (group q takes every fourth of them), four loads in flight each
  __shared__ float red[4][192];
  const int b = blockIdx.x, q = threadIdx.x / 192, tid = threadIdx.x % 192, band = tid >> 6, col = tid & 63;
  const bool parseval = tot_part != nullptr && band == 2;
  const int first = b + q * ENERGY_PARTS, step = 4 * ENERGY_PARTS;
  float t[4] = {0.f, 0.f, 0.f, 0.f};
  for (int tensor = 0; tensor < 6; ++tensor) {   // slots: Q, K, V on the box (Parseval for the high band), Q, K, V on the whole grid
    const float* base = part + (size_t)tensor * DCT_MAX_WAVES * 192;
    const int n = nw.en[tensor];
    if (parseval && tensor < 3) {
      for (int w = first; w < n; w += 4 * step)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (w + u * step < n) t[u] -= base[(size_t)(w + u * step) * 192 + col] + base[(size_t)(w + u * step) * 192 + 64 + col];
    } else {
      for (int w = first; w < n; w += 4 * step)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (w + u * step < n) t[u] += base[(size_t)(w + u * step) * 192 + tid];
    }
  }
  if (parseval)
    for (int tensor = 0; tensor < 3; ++tensor) {
      const int n = nw.tot[tensor];
      for (int w = first; w < n; w += 4 * step)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (w + u * step < n) t[u] += tot_part[((size_t)tensor * DCT_MAX_WAVES + w + u * step) * 64 + col];
    }
  red[q][tid] = (t[0] + t[1]) + (t[2] + t[3]);
  __syncthreads();
  if (q == 0) part1[(size_t)b * 192 + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// One workgroup per band and channel chunk: 16 rows of 64 threads share the chunk's partial sums.  `host` ([3][d] + 1, pinned): the
// sums and the range flag once more, where the host reads them after waiting for the stream (two copies less in front of it).
__global__ void __launch_bounds__(1024) k_energy_reduce2(const float* __restrict__ part1, float* __restrict__ stats, int d, int parseval,
                                                         float* __restrict__ host, const int32_t* __restrict__ range_flag) {
  __shared__ float red[16][64];
  const int chunks = d / 64, band = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int row = threadIdx.x >> 6, col = threadIdx.x & 63;
  float t = 0.f;
#pragma unroll 4
  for (int b = chunk + row * chunks; b < ENERGY_PARTS; b += 16 * chunks) t += part1[(size_t)b * 192 + band * 64 + col];
  red[row][col] = t;
  __syncthreads();
  if (row != 0) return;
  for (int r = 1; r < 16; ++r) t += red[r][col];
  // The Parseval difference of a band that holds (almost) no energy can come out slightly negative (the low and mid
  // sums carry the rounding of the fp16 transform): an energy is never below zero.
  t = (parseval && band == 2 && t < 0.f) ? 0.f : t;   // (a NaN stays a NaN: the host reports it)
  stats[band * d + chunk * 64 + col] = t;
  host[band * d + chunk * 64 + col] = t;
  if (blockIdx.x == 0 && col == 0) host[3 * d] = __int_as_float(*range_flag);
}

// stats: [3][d] results followed by ENERGY_PART_FLOATS of scratch (the stage-1 sums)
hipError_t launch_energy_reduce(const float* energy_part, const float* tot_part, float* stats, int d, const EnergyWaves& nw,
                                float* host, const int32_t* range_flag, hipStream_t st) {
  if (d <= 0 || d % 64 != 0 || ENERGY_PARTS % (d / 64) != 0) return hipErrorInvalidValue;
  static_assert(ENERGY_PARTS * 192 == ENERGY_PART_FLOATS, "scratch of the stage-1 sums");
  float* part1 = stats + 3 * d;
  hipLaunchKernelGGL(k_energy_reduce1, dim3(ENERGY_PARTS), dim3(768), 0, st, energy_part, tot_part, part1, nw);
  hipLaunchKernelGGL(k_energy_reduce2, dim3(3 * (d / 64)), dim3(1024), 0, st, part1, stats, d, tot_part != nullptr ? 1 : 0, host, range_flag);
  return hipGetLastError();
}

}  // namespace fa
