// One axis of the separable transform on the generic fp32 path (sections 3.2, 3.7), any axis length and head_dim:
//   out[s, k, i] = sum_j M[k][j] in[s, j, i],   fp32 operands and accumulation, fp32 or bf16 tensors at the ends.
//
// A wave owns 64 columns (s, i) - neighbours in i, across slabs where a slab has fewer - and up to 64 output rows, on
// v_mfma_f32_16x16x4_f32.  Lane (n, g) of 16 x 4 holds columns 4 n .. 4 n + 3, one per column tile, so an input row is
// read as 256 contiguous bytes per 16 lanes and an output row written the same way; its four input rows per step of 16
// are j = 16 jc + 4 g + r, which is also how it reads 16 bytes of a matrix row (the matrix is stored with rows and
// columns padded to multiples of 16 by zeros, so nothing is tested there).  No LDS, no barrier.  Q, K and V go through
// one launch (blockIdx.y).
//
// What bounds it: memory (one read and one write per pass; 3.9-5 TB/s) and, for small tensors, the launch.  The kernel
// before it computed one output per thread with n strided loads, one tensor per launch.  12 passes over 12,150 tokens x 4
// heads x 64 in fp32: 1.03 ms before (12 launches), 98 us now (6 launches); 6,160 tokens x 6 heads x 128, bf16 in and out:
// 1.23 ms before, 146 us now.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t gx_bf16(float f) {   // round to nearest even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// IN / OUT: 0 fp32, 1 bf16.  VEC: head_dim is a multiple of 4 and the tensors start at a multiple of four elements, so four
// columns are adjacent, aligned and of one slab.
template <int KT, int IN, int OUT, bool VEC>
__global__ void __launch_bounds__(256) k_gaxis(AxisPassArgs a, int64_t ncols) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int kgroups = (a.n_out + 16 * KT - 1) / (16 * KT);
  const int tensor = blockIdx.y / kgroups, k0 = (blockIdx.y % kgroups) * 16 * KT;
  const int64_t c0 = ((int64_t)blockIdx.x * 4 + wave) * 64;
  if (c0 >= ncols) return;
  const char* in = (const char*)a.in[tensor];
  char* out = (char*)a.out[tensor];
  constexpr int IE = IN ? 2 : 4, OE = OUT ? 2 : 4;

  // this lane's four columns: element offset of input row 0 / output row 0, and what the looked-up rows need
  constexpr int NC = VEC ? 1 : 4;   // columns with an address of their own
  int64_t in_off[NC], out_off[NC], slice_off[NC];
  int32_t pbase[NC], mask[NC];
  bool live[NC];
#pragma unroll
  for (int t = 0; t < NC; ++t) {
    const int64_t col = c0 + 4 * n + t;
    live[t] = col < ncols;
    const uint64_t cc = live[t] ? (uint64_t)col : 0u;
    int64_t s, i;
    if (ncols <= 0x7fffffff) { s = (uint32_t)cc / (uint32_t)a.inner; i = (uint32_t)cc % (uint32_t)a.inner; }
    else { s = cc / (uint64_t)a.inner; i = cc % (uint64_t)a.inner; }
    in_off[t] = s * a.n * a.inner + i;
    out_off[t] = s * a.n_out * a.inner + i;
    slice_off[t] = 0; pbase[t] = 0; mask[t] = 0;
    if (a.perm_in || a.perm_out) {
      const int64_t slice = s / a.outer, o = s - slice * a.outer;
      slice_off[t] = slice * a.Ntok * a.inner + i;
      pbase[t] = (int32_t)(o * (a.perm_in ? a.n : a.n_out));
      if (a.masks) mask[t] = a.masks[slice];
    }
  }
  auto load = [&](int j) -> float4v {
    float4v v = {0.f, 0.f, 0.f, 0.f};
    if (j >= a.n) return v;
#pragma unroll
    for (int t = 0; t < NC; ++t) {
      if (!live[t]) continue;
      const char* src = in;
      int64_t e;
      if (a.perm_in) {
        const int32_t row = a.perm_in[pbase[t] + j];
        if (a.masks) {
          const int band = row < a.band_off1 ? 0 : (row < a.band_off2 ? 1 : (row < a.band_off3 ? 2 : 3));
          if (!((mask[t] >> band) & 1)) src = (const char*)a.in_alt;
        }
        e = slice_off[t] + (int64_t)row * a.inner;
      } else {
        e = in_off[t] + (int64_t)j * a.inner;
      }
      src += e * IE;
      if (VEC && IN) {
        const uint2 u = *(const uint2*)src;
        v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
        v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
      } else if (VEC) {
        v = *(const float4v*)src;
      } else {
        v[t] = IN ? __uint_as_float((uint32_t)*(const uint16_t*)src << 16) : *(const float*)src;
      }
    }
    return v;
  };

  float4v acc[KT][4];   // [row tile][column tile]: rows 4 g + r, column 4 n + tile
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[kt][t] = float4v{0.f, 0.f, 0.f, 0.f};
  const int nc = (a.n + 15) / 16;
  float4v B[4], Bn[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) B[r] = load(4 * g + r);
  for (int jc = 0; jc < nc; ++jc) {
    float4v A[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const int k = k0 + 16 * kt + n;
      A[kt] = float4v{0.f, 0.f, 0.f, 0.f};
      if (k < a.ldm) A[kt] = *(const float4v*)(a.M + (int64_t)k * a.ldm + 16 * jc + 4 * g);
    }
    if (jc + 1 < nc) {
#pragma unroll
      for (int r = 0; r < 4; ++r) Bn[r] = load(16 * (jc + 1) + 4 * g + r);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[kt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[kt][r], B[r][t], acc[kt][t], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) B[r] = Bn[r];
  }
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = k0 + 16 * kt + 4 * g + r;
      if (k >= a.n_out) continue;
#pragma unroll
      for (int t = 0; t < NC; ++t) {
        if (!live[t]) continue;
        const int64_t e = a.perm_out ? slice_off[t] + (int64_t)a.perm_out[pbase[t] + k] * a.inner : out_off[t] + (int64_t)k * a.inner;
        char* dst = out + e * OE;
        if (VEC && OUT) {
          uint2 u;
          u.x = gx_bf16(acc[kt][0][r]) | (gx_bf16(acc[kt][1][r]) << 16);
          u.y = gx_bf16(acc[kt][2][r]) | (gx_bf16(acc[kt][3][r]) << 16);
          *(uint2*)dst = u;
        } else if (VEC) {
          *(float4v*)dst = float4v{acc[kt][0][r], acc[kt][1][r], acc[kt][2][r], acc[kt][3][r]};
        } else if (OUT) {
          *(uint16_t*)dst = (uint16_t)gx_bf16(acc[kt][t][r]);
        } else {
          *(float*)dst = acc[kt][t][r];
        }
      }
    }
}

template <int KT, int IN, int OUT>
hipError_t launch_io(const AxisPassArgs& a, int64_t ncols, bool vec, hipStream_t st) {
  const int64_t bx = (ncols + 255) / 256;
  const int64_t by = (int64_t)a.n_tensors * ((a.n_out + 16 * KT - 1) / (16 * KT));
  if (bx > 0x7fffffff || by > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)bx, (unsigned)by);
  if (vec) hipLaunchKernelGGL((k_gaxis<KT, IN, OUT, true>), grid, dim3(256), 0, st, a, ncols);
  else hipLaunchKernelGGL((k_gaxis<KT, IN, OUT, false>), grid, dim3(256), 0, st, a, ncols);
  return hipGetLastError();
}
template <int KT>
hipError_t launch_kt(const AxisPassArgs& a, int64_t ncols, bool vec, hipStream_t st) {
  if (a.in_bf16 && a.out_bf16) return hipErrorInvalidValue;   // (a transform is at least two passes long)
  if (a.in_bf16) return launch_io<KT, 1, 0>(a, ncols, vec, st);
  if (a.out_bf16) return launch_io<KT, 0, 1>(a, ncols, vec, st);
  return launch_io<KT, 0, 0>(a, ncols, vec, st);
}

}  // namespace

hipError_t launch_generic_axis_pass(const AxisPassArgs& a, hipStream_t st) {
  const int64_t ncols = a.nslab * a.inner;
  if (ncols == 0 || a.n_tensors == 0) return hipSuccess;
  if (a.ldm < a.n || a.ldm % 16 != 0 || (a.perm_in && a.perm_out)) return hipErrorInvalidValue;
  bool vec = a.d % 4 == 0;
  for (int i = 0; i < a.n_tensors; ++i)   // (a caller's tensor may be a view that starts anywhere)
    vec = vec && (uintptr_t)a.in[i] % (a.in_bf16 ? 8 : 16) == 0 && (uintptr_t)a.out[i] % (a.out_bf16 ? 8 : 16) == 0;
  switch ((std::min(a.n_out, 64) + 15) / 16) {
    case 1: return launch_kt<1>(a, ncols, vec, st);
    case 2: return launch_kt<2>(a, ncols, vec, st);
    case 3: return launch_kt<3>(a, ncols, vec, st);
    default: return launch_kt<4>(a, ncols, vec, st);
  }
}

}  // namespace fa
