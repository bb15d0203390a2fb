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

// Coefficients of axis `ax` that tensor `tensor` of a slice is made for.
__device__ __forceinline__ int gx_extent(const AxisBoxes& b, int tensor, int mask, int ax) {
  if (tensor >= b.n || (mask & 12)) return b.full[ax];   // (the high band and the second mid band lie outside the boxes)
  return mask & 2 ? b.mid[ax] : mask & 1 ? b.low[ax] : 0;
}

// IN / OUT: 0 fp32, 1 bf16.  VEC: head_dim is a multiple of 4 and the tensors start at a multiple of four elements, so four
// columns are adjacent, aligned and of one slab.  BOX: some tensors are only made on a box (a variant of its own: the test of every output row
// costs passes that make everything 1-2 %).
template <int KT, int IN, int OUT, bool VEC, bool BOX>
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
  int32_t pbase[NC], mask[NC], kend[NC];   // (kend: output rows made)
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
    slice_off[t] = 0; pbase[t] = 0; mask[t] = 0; kend[t] = a.n_out;
    if (a.perm_in || a.perm_out) {
      const int64_t slice = s / a.outer, o = s - slice * a.outer;
      slice_off[t] = slice * a.Ntok * a.inner + i;
      pbase[t] = (int32_t)(o * (a.perm_in ? a.n : a.n_out));
      if (a.masks) mask[t] = a.masks[slice];
      if (BOX && tensor < a.box.n) {
        const int m = a.box.masks[slice], h = (int)(o % a.box.full[1]), z = (int)(o / a.box.full[1]);
        live[t] = live[t] && z < gx_extent(a.box, tensor, m, 0) && h < gx_extent(a.box, tensor, m, 1);
        kend[t] = gx_extent(a.box, tensor, m, 2);
      }
    }
  }
  if (BOX && tensor < a.box.n) {   // nothing of this wave is needed
    bool any = false;
#pragma unroll
    for (int t = 0; t < NC; ++t) any = any || (live[t] && k0 < kend[t]);
    if (__builtin_amdgcn_ballot_w64(any) == 0) return;
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
        if (!live[t] || (BOX && k >= kend[t])) continue;
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
  constexpr bool BOXES = !IN && !OUT;   // (the last pass of a forward transform is fp32 on both sides)
  if (a.box.n > 0 && !BOXES) return hipErrorInvalidValue;
  void (*const k)(AxisPassArgs, int64_t) = BOXES && a.box.n > 0 ? (vec ? k_gaxis<KT, IN, OUT, true, BOXES> : k_gaxis<KT, IN, OUT, false, BOXES>)
                                                                : (vec ? k_gaxis<KT, IN, OUT, true, false> : k_gaxis<KT, IN, OUT, false, false>);
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, a, ncols);
  return hipGetLastError();
}
template <int KT>
hipError_t launch_kt(const AxisPassArgs& a, int64_t ncols, bool vec, hipStream_t st) {
  if (a.in_bf16 && a.out_bf16) return hipErrorInvalidValue;   // (a transform is at least two passes long)
  if (a.in_bf16) return launch_io<KT, 1, 0>(a, ncols, vec, st);
  if (a.out_bf16) return launch_io<KT, 0, 1>(a, ncols, vec, st);
  return launch_io<KT, 0, 0>(a, ncols, vec, st);
}

// T and H axes in one pass:  out[s, kt, kh, i] = sum_h Mh[kh][h] sum_t Mt[kt][t] in[s, t, h, i],  the tensor between the axes in LDS.
// A workgroup of up to 8 waves owns 64 columns i of one slice, all T H rows of them: a wave takes the T axis of one row h after the other
// from memory (lane (n, g) holds columns 4 n .. 4 n + 3 of its rows), leaves the results in LDS as [kt][h][64], and takes
// the H axis of (kt, 16 output rows) one after the other from there.  Product r of R = ceil(n / 4) takes rows j = g R + r, so an axis of n
// takes R products and not whole steps of 16.  (Against 64 bits both orders come out the same: mean over
// eight inputs of 256 tokens 1.42e-7 in two passes, 1.43e-7 here, of 504 x 64 1.72e-7 and 1.71e-7, of 2,592 x 64 1.878e-7 and 1.879e-7.)
//
// What bounds it: memory, read once and written once for two axes, and at the sizes it is used at the chain load - products - LDS -
// products - store of a workgroup.  Two passes / this, Q, K and V: 12,150 tokens (9 x 30 x 45) x 4 heads x 64 in fp32 42 / 25 us, 6,160
// (7 x 22 x 40) x 6 x 128 from bf16 62 / 34 us; 256 tokens x 2 x 32 8.5 / 5 us; the inverse 18 / 12, 27 / 14 and 8.5 / 4.5 us.
// Q~ and K~ made only on the box a slice's bands live in, forwards, whole / boxes: 125 / 120 us (two of four heads without the high band),
// 193 / 174 (four of six); nothing at 256 tokens.
template <int IN, int OUT, bool VEC>
__global__ void __launch_bounds__(512) k_gaxis_th(AxisPairArgs a) {
  extern __shared__ __attribute__((aligned(16))) float th_smem[];
  constexpr int IE = IN ? 2 : 4, OE = OUT ? 2 : 4;
  const int n_waves = (int)blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int T = a.T, H = a.H, mstr = a.ldh + 4, rt = (T + 3) / 4, rh = (H + 3) / 4;
  float* Y = th_smem;                       // [T][H][64]
  float* Mh = th_smem + T * H * 64;         // [ldh][mstr]
  const int tensor = blockIdx.z, slice = blockIdx.y;
  const int64_t col = (int64_t)blockIdx.x * 64 + 4 * n;
  const int mask = tensor < a.box.n ? a.box.masks[slice] : 0;
  const int KT = tensor < a.box.n ? gx_extent(a.box, tensor, mask, 0) : T, KH = tensor < a.box.n ? gx_extent(a.box, tensor, mask, 1) : H;   // coefficients made
  const int t_rows = th_rows(T, H, KT);   // rows kt that the H axis reads
  const int nlive = (int)(a.inner - col < 4 ? a.inner - col : 4);   // columns of this lane's four that exist (VEC: all or none)
  const int64_t base = (int64_t)slice * T * H * a.inner + col;
  const char* in = (const char*)a.in[tensor] + base * IE;
  char* out = (char*)a.out[tensor] + base * OE;
  const int64_t t_stride = (int64_t)H * a.inner;

  auto load = [&](int h, float4v (&x)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x[r] = float4v{0.f, 0.f, 0.f, 0.f};
      const int t = g * rt + r;
      if (r >= rt || t >= T || nlive <= 0) continue;
      const char* src = in + (t * t_stride + (int64_t)h * a.inner) * IE;
      if (!VEC) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nlive) x[r][c] = IN ? __uint_as_float((uint32_t)*(const uint16_t*)(src + c * IE) << 16) : *(const float*)(src + c * IE);
      } else if (IN) {
        const uint2 u = *(const uint2*)src;
        x[r][0] = __uint_as_float(u.x << 16); x[r][1] = __uint_as_float(u.x & 0xffff0000u);
        x[r][2] = __uint_as_float(u.y << 16); x[r][3] = __uint_as_float(u.y & 0xffff0000u);
      } else {
        x[r] = *(const float4v*)src;
      }
    }
  };
  float4v x[2][4];
  if (wave < H) load(wave, x[0]);
  if (wave + n_waves < H) load(wave + n_waves, x[1]);
  if (KT == 0) return;   // (uniform over the workgroup; behind the loads, which need not wait for the mask)
  float At[4];   // operand of the T matrix (padded with zeros to 16 x 16)
#pragma unroll
  for (int r = 0; r < 4; ++r) At[r] = r < rt ? a.Mt[n * a.ldt + g * rt + r] : 0.f;
  for (int e = tid; e < a.ldh * (mstr / 4); e += (int)blockDim.x) {   // (the padding too: the last rows' products below reach into it)
    const int row = e / (mstr / 4), c4 = e % (mstr / 4) * 4;
    float4v m = {0.f, 0.f, 0.f, 0.f};
    if (c4 < a.ldh) m = *(const float4v*)(a.Mh + row * a.ldh + c4);
    *(float4v*)(Mh + row * mstr + c4) = m;
  }
  for (int h = wave; h < H; h += 2 * n_waves)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int hb = h + b * n_waves;
      if (hb >= H) break;   // (uniform)
      float4v acc[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < rt)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(At[r], x[b][r][c], acc[c], 0, 0, 0);
      if (hb + 2 * n_waves < H) load(hb + 2 * n_waves, x[b]);
#pragma unroll
      for (int r = 0; r < 4; ++r)   // result row 4 g + r
        if (4 * g + r < t_rows) *(float4v*)(Y + ((4 * g + r) * H + hb) * 64 + 4 * n) = float4v{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
    }
  __syncthreads();
  const int tiles = (KH + 15) / 16;
  for (int u = wave; u < KT * tiles; u += n_waves) {
    const int kt = u / tiles, tile = u - kt * tiles;
    float4v acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = float4v{0.f, 0.f, 0.f, 0.f};
    const float* y = Y + (kt * H + g * rh) * 64 + 4 * n;
    const float* m = Mh + (16 * tile + n) * mstr + g * rh;
#pragma unroll 4
    for (int r = 0; r < rh; ++r) {
      // (rows past the axis: the matrix is zero there, and what lies behind is a row of a later kt - made for this if it is not needed
      // itself, see th_rows - or of the matrix)
      const float A = m[r];
      const float4v b = *(const float4v*)(y + r * 64);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(A, b[c], acc[c], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kh = 16 * tile + 4 * g + r;
      if (kh >= KH || nlive <= 0) continue;
      char* dst = out + (kt * t_stride + (int64_t)kh * a.inner) * OE;
      if (!VEC) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nlive) {
            if (OUT) *(uint16_t*)(dst + c * OE) = (uint16_t)gx_bf16(acc[c][r]);
            else *(float*)(dst + c * OE) = acc[c][r];
          }
      } else if (OUT) {
        uint2 w;
        w.x = gx_bf16(acc[0][r]) | (gx_bf16(acc[1][r]) << 16);
        w.y = gx_bf16(acc[2][r]) | (gx_bf16(acc[3][r]) << 16);
        *(uint2*)dst = w;
      } else {
        *(float4v*)dst = float4v{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
      }
    }
  }
}

// Four columns are adjacent, aligned and of one row.
bool gx_aligned(int d, const void* const* in, void* const* out, int n, bool in_bf16, bool out_bf16) {
  bool vec = d % 4 == 0;
  for (int i = 0; i < n; ++i)   // (a caller's tensor may be a view that starts anywhere)
    vec = vec && (uintptr_t)in[i] % (in_bf16 ? 8 : 16) == 0 && (uintptr_t)out[i] % (out_bf16 ? 8 : 16) == 0;
  return vec;
}

typedef void (*ThKernel)(AxisPairArgs);
// [in bf16, out bf16, neither][VEC]
const ThKernel th_kernel[3][2] = {{k_gaxis_th<1, 0, false>, k_gaxis_th<1, 0, true>},
                                  {k_gaxis_th<0, 1, false>, k_gaxis_th<0, 1, true>},
                                  {k_gaxis_th<0, 0, false>, k_gaxis_th<0, 0, true>}};

}  // namespace

// By sizes alone: the two forms sum in another order, and the bits must not depend on where a tensor starts.  The tensor between the
// axes takes 256 bytes of LDS for each of the T H rows, at most 440 here; with more than 300 a compute unit holds one workgroup and the pass is
// still the faster way (whole forwards, two passes / this: 8,184 tokens of 11 x 31 x 24 x 4 heads x 32 70.5 / 64.3 us).
bool generic_pair_fits(const AxisPairArgs& a) {
  return a.T <= 16 && a.H <= 64 && a.slices <= 65535 && a.inner <= (int64_t)64 * 0x7fffffff && (a.T * a.H * 64 + a.ldh * (a.ldh + 4)) * 4 <= 112 * 1024;
}
hipError_t allow_generic_axis_pair() {
  static OncePerDevice limit[3][2];
  hipError_t e = hipSuccess;
  for (int i = 0; i < 6 && e == hipSuccess; ++i) e = allow_lds(limit[i / 2][i % 2], (const void*)th_kernel[i / 2][i % 2], 160 * 1024);
  return e;
}
hipError_t launch_generic_axis_pair(const AxisPairArgs& a, hipStream_t st) {
  if (a.slices == 0 || a.n_tensors == 0) return hipSuccess;
  if (!generic_pair_fits(a) || a.ldt < 16 || a.ldh < a.H || a.ldh % 16 != 0 || (a.in_bf16 && a.out_bf16)) return hipErrorInvalidValue;
  const int lds = (a.T * a.H * 64 + a.ldh * (a.ldh + 4)) * 4;
  const ThKernel k = th_kernel[a.in_bf16 ? 0 : a.out_bf16 ? 1 : 2][gx_aligned(a.d, a.in, a.out, a.n_tensors, a.in_bf16, a.out_bf16)];
  // No more waves than there are rows or row tiles, and four rows for each: 1 x 1 x 1000 x 4 heads x 64 with eight waves 409 us a forward, with one 360 (an
  // axis at a time 373); 2 x 4 x 1000 475 / 432 (470), 16 x 1 x 1000 594 / 549 (634), 1 x 16 x 64 59 / 58 (72).
  const int waves = std::min({8, std::max(a.H, a.T * (a.ldh / 16)), (a.T * a.H + 3) / 4});
  hipLaunchKernelGGL(k, dim3((unsigned)((a.inner + 63) / 64), (unsigned)a.slices, (unsigned)a.n_tensors), dim3(64 * waves), (size_t)lds, st, a);
  return hipGetLastError();
}

hipError_t launch_generic_axis_pass(const AxisPassArgs& a, hipStream_t st) {
  const int64_t ncols = a.nslab * a.inner;
  if (ncols == 0 || a.n_tensors == 0) return hipSuccess;
  if (a.ldm < a.n || a.ldm % 16 != 0 || (a.perm_in && a.perm_out)) return hipErrorInvalidValue;
  const bool vec = gx_aligned(a.d, a.in, a.out, a.n_tensors, a.in_bf16, a.out_bf16);
  switch ((std::min(a.n_out, 64) + 15) / 16) {
    case 1: return launch_kt<1>(a, ncols, vec, st);
    case 2: return launch_kt<2>(a, ncols, vec, st);
    case 3: return launch_kt<3>(a, ncols, vec, st);
    default: return launch_kt<4>(a, ncols, vec, st);
  }
}

}  // namespace fa
