#pragma once
// The H and W axes of the inverse transform (paper section 3.7) in one pass, for slices whose spectral box is small:
//   out[t, h, w, c] = (v[t, h, w, c] +) fp16( sum_kw Fw[w][kw] * fp16( sum_kh Fh[h][kh] * y[kh, t, kw, c] ) )
// A workgroup of four waves takes 64 channels of one (slice, t) plane, all of its rows h or a part of them.  The plane's kh x kw coefficients are read once into
// registers, as operands that hold 4 consecutive kh of one channel (through LDS, transposing reads); 16 rows h at a time are
// expanded along H (v_mfma_f32_16x16x16_f16, h as rows, channels as columns), rounded to fp16, exchanged between the
// lane groups so that an operand holds 4 consecutive kw of one h, and expanded along W (channels as rows, w as columns).  A
// row of the output goes through LDS, where the four waves put their channels together, and is added to the row of V that
// was requested some rows earlier.  The tensor between the axes never reaches memory.
//
// Bound by HBM: it reads V and writes the output, the coefficients are a small part of that.  16 slices of 64^3 x 128 from the
// 16 x 16 box 507 (two passes) -> 412 us, 16 slices of 16 x 64 x 64 x 64 from the 16 x 16 box 68 -> 51 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef __fp16 fp16x4 __attribute__((__vector_size__(4 * sizeof(__fp16))));

__device__ __forceinline__ uint32_t iwh_pack_f16(float lo, float hi) {
  const _Float16 l = (_Float16)lo, h = (_Float16)hi;
  return (uint32_t)__builtin_bit_cast(uint16_t, l) | ((uint32_t)__builtin_bit_cast(uint16_t, h) << 16);
}
__device__ __forceinline__ uint32_t iwh_bf16(float f) {   // round to nearest even, NaN stays NaN
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

// Waves per SIMD, and workgroups per compute unit: the plane takes 32 registers per 256 coefficients.
template <int KHS, int KWT> constexpr int iwh_waves() { return KHS * KWT == 1 ? 3 : 2; }
constexpr int IWH_ROW = 144;   // bytes per staged row of 64 channels (128 + 16: rows side by side take all LDS banks once)

// (RESID is a template argument: with the branch inside, between a product and the first use of its result, a draft of the forward
// kernel gave wrong sums; see there.)
template <int NW16, int KHS, int KWT, bool RESID>   // W / 16, kh / 16, kw / 16
__global__ void __launch_bounds__(256, (iwh_waves<KHS, KWT>())) k_iwh_pass(IwhPassArgs a) {
  constexpr int W = 16 * NW16, KH = 16 * KHS, KW = 16 * KWT;
  constexpr int NP = (NW16 + 1) / 2;    // 16-byte pieces of an output row per thread
  constexpr int SKW = 4;                // kw per slice of the plane on its way into registers
  constexpr int NS = KH * SKW * 8 / 256;   // 16-byte pieces of a slice per thread
  constexpr int VD = 2;   // rows of V requested ahead
  constexpr int ROWS = 2 * W > SKW * KH ? 2 * W : SKW * KH;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  char* stage = smem;                                       // [ROWS][IWH_ROW]
  constexpr int MSTR = KH + 8;
  half_t* Fh = (half_t*)(smem + ROWS * IWH_ROW);            // [H][MSTR]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wc = __builtin_amdgcn_readfirstlane(tid >> 6);   // this wave's 16 channels
  const int l16 = lane & 15, q = lane >> 4;

  for (int e = tid; e < a.H * (KH / 8); e += 256) {
    const int row = e / (KH / 8), c8 = e % (KH / 8);
    *(uint4v*)(Fh + row * MSTR + c8 * 8) = *(const uint4v*)(a.Fh + (size_t)row * a.H + c8 * 8);
  }
  // W matrix operands: lane = w, 4 consecutive kw
  half4 Bw[NW16][KWT];
#pragma unroll
  for (int n = 0; n < NW16; ++n)
#pragma unroll
    for (int u = 0; u < KWT; ++u) Bw[n][u] = *(const half4*)(a.Fw + (size_t)(16 * n + l16) * W + 16 * u + 4 * q);

  const int cpt = a.d >> 6;
  const int n_items = a.n_slices * a.T * cpt * a.parts;
  const int64_t kh_stride = (int64_t)a.T * KW * a.d;
  // slice pieces: piece p of a slice is channels 8 (p % 8) .. of (kh, kw) = (p / 8 / SKW, p / 8 % SKW)
  uint32_t s_src[NS], s_dst[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int p = tid + 256 * i, kwl = p / 8 % SKW, kh = p / 8 / SKW;
    s_src[i] = (uint32_t)((int64_t)kh * kh_stride + kwl * a.d + (p % 8) * 8) * 2u;
    s_dst[i] = (uint32_t)((kwl * KH + kh) * IWH_ROW + (p % 8) * 16);
  }
  // output pieces: piece p of a row is channels 8 (p % 8) .. of w = p / 8
  uint32_t o_off[NP], o_lds[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = tid + 256 * i;
    o_off[i] = (uint32_t)((p / 8) * a.d + (p % 8) * 8) * 2u;
    o_lds[i] = (uint32_t)((p / 8) * IWH_ROW + (p % 8) * 16);
  }
  const bool last_piece = NW16 % 2 == 0 || wc < 2;   // with an odd NW16 the last piece exists for half the threads
  const int tr = (4 * q + (l16 >> 2)) * IWH_ROW + wc * 32 + (lane & 3) * 8;   // transposing reads: row kh, 4 channels

  for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int part = item % a.parts, pl = item / a.parts, chunk = pl % cpt, t = pl / cpt % a.T, sl = pl / cpt / a.T;
    const int h_lo = a.H / 16 * part / a.parts * 16, h_hi = a.H / 16 * (part + 1) / a.parts * 16;   // rows h of this item
    const int64_t slice = a.slice_list[sl];
    const char* in = (const char*)((const half_t*)a.in + ((int64_t)sl * KH * a.T + t) * KW * a.d + chunk * 64);
    const int64_t plane = (slice * a.T + t) * a.H * (int64_t)W * a.d + chunk * 64;
    const char* vin = (const char*)((const uint16_t*)a.resid + plane);
    char* out = (char*)((uint16_t*)a.out + plane);
    const int64_t h_bytes = (int64_t)W * a.d * 2;

    // ---- the plane's coefficients, SKW columns kw at a time
    uint2v Y[KW][KHS];
    uint4v piece[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) piece[i] = *(const uint4v*)(in + s_src[i]);
#pragma unroll
    for (int k = 0; k < KW; k += SKW) {
      __syncthreads();   // everybody has read what the rows held before
#pragma unroll
      for (int i = 0; i < NS; ++i) *(uint4v*)(stage + s_dst[i]) = piece[i];
      if (k + SKW < KW)
#pragma unroll
        for (int i = 0; i < NS; ++i) piece[i] = *(const uint4v*)(in + (size_t)(k + SKW) * a.d * 2 + s_src[i]);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < SKW; ++kk)
#pragma unroll
        for (int s = 0; s < KHS; ++s) {
          const char* ptr = stage + (kk * KH + 16 * s) * IWH_ROW + tr;
          const fp16x4 t4 = __builtin_amdgcn_ds_read_tr16_b64_v4f16((fp16x4 __attribute__((address_space(3)))*)ptr);
          Y[k + kk][s] = __builtin_bit_cast(uint2v, t4);
        }
    }
    // rows of V, VD ahead of their use
    uint4v vr[VD][NP];
    auto request_v = [&](int h, int to) {
      const char* row = vin + (h < h_hi ? h : h_hi - 1) * h_bytes;
#pragma unroll
      for (int i = 0; i < NP; ++i)
        if (i + 1 < NP || last_piece) vr[to][i] = *(const uint4v*)(row + o_off[i]);
    };
    if (RESID)
#pragma unroll
      for (int i = 0; i < VD; ++i) request_v(h_lo + i, i);
    __syncthreads();   // the slices have been read: the rows take output from here on

    for (int h0 = h_lo; h0 < h_hi; h0 += 16) {
      half4 Ah[KHS];
#pragma unroll
      for (int s = 0; s < KHS; ++s) Ah[s] = *(const half4*)(Fh + (h0 + l16) * MSTR + 16 * s + 4 * q);
      uint32_t st[KWT][4][4][2];   // [16 kw][h 4 q + r][4 kw][pair]
#pragma unroll
      for (int u = 0; u < KWT; ++u)
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          float4v z[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            z[j] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KHS; ++s)
              z[j] = __builtin_amdgcn_mfma_f32_16x16x16f16(Ah[s], __builtin_bit_cast(half4, Y[16 * u + k + j][s]), z[j], 0, 0, 0);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            uint32_t pk = iwh_pack_f16(z[0][r], z[1][r]);
            asm volatile("" : "+v"(pk));   // (rounded here: postponed, it would keep twice the registers alive)
            st[u][r][k >> 2][(k >> 1) & 1] = pk;
          }
        }
      // block b of lane group g: 4 kw of h 4 g + r  ->  block g of h 4 b + r
#pragma unroll
      for (int u = 0; u < KWT; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            auto s0 = __builtin_amdgcn_permlane32_swap(st[u][r][0][j], st[u][r][2][j], false, false);
            auto s1 = __builtin_amdgcn_permlane32_swap(st[u][r][1][j], st[u][r][3][j], false, false);
            auto t0 = __builtin_amdgcn_permlane16_swap(s0[0], s1[0], false, false);
            auto t1 = __builtin_amdgcn_permlane16_swap(s0[1], s1[1], false, false);
            st[u][r][0][j] = t0[0]; st[u][r][1][j] = t0[1]; st[u][r][2][j] = t1[0]; st[u][r][3][j] = t1[1];
          }
#pragma unroll
      for (int hh = 0; hh < 16; ++hh) {
        const int b = hh >> 2, r = hh & 3;
        char* buf = stage + (hh & 1) * (W * IWH_ROW);
#pragma unroll
        for (int n = 0; n < NW16; ++n) {
          float4v x = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int u = 0; u < KWT; ++u)
            x = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4, uint2v{st[u][r][b][0], st[u][r][b][1]}), Bw[n][u], x, 0, 0, 0);
          uint2v p;
          if (RESID) {   // (fp16 until V is added)
            p[0] = iwh_pack_f16(x[0], x[1]); p[1] = iwh_pack_f16(x[2], x[3]);
          } else {
            p[0] = iwh_bf16(x[0]) | (iwh_bf16(x[1]) << 16); p[1] = iwh_bf16(x[2]) | (iwh_bf16(x[3]) << 16);
          }
          *(uint2v*)(buf + (16 * n + l16) * IWH_ROW + wc * 32 + q * 8) = p;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int h = h0 + hh;
        char* row = out + h * h_bytes;
#pragma unroll
        for (int i = 0; i < NP; ++i)
          if (i + 1 < NP || last_piece) {
            uint4v v = *(const uint4v*)(buf + o_lds[i]);
            if (RESID) {
              const uint4v rs = vr[hh % VD][i];
              const half8 f = __builtin_bit_cast(half8, v);
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const float lo = __uint_as_float(rs[j] << 16) + (float)f[2 * j];
                const float hi = __uint_as_float(rs[j] & 0xffff0000u) + (float)f[2 * j + 1];
                v[j] = iwh_bf16(lo) | (iwh_bf16(hi) << 16);
              }
            }
            *(uint4v*)(row + o_off[i]) = v;
          }
        if (RESID) request_v(h + VD, hh % VD);
      }
    }
  }
}

template <int NW16, int KHS, int KWT>
static hipError_t iwh_launch(IwhPassArgs a, int num_cu, hipStream_t st) {
  constexpr int ROWS = 32 * NW16 > 64 * KHS ? 32 * NW16 : 64 * KHS;
  const int lds = ROWS * IWH_ROW + a.H * (16 * KHS + 8) * 2;
  const int64_t planes = (int64_t)a.n_slices * a.T * (a.d / 64), cap = (int64_t)num_cu * iwh_waves<KHS, KWT>();
  if (planes <= 0) return hipSuccess;
  // a plane's rows are shared among workgroups until there are four items for each place on the chip
  a.parts = (int)std::max<int64_t>(1, std::min<int64_t>(a.H / 16, (4 * cap + planes - 1) / planes));
  // per-lane byte offsets are unsigned 32-bit numbers
  if (planes * a.parts > 0x3fffffff || (int64_t)16 * KHS * a.T * 16 * KWT * a.d * 2 > 0xffffffffLL || (int64_t)16 * NW16 * a.d * 2 > 0xffffffffLL)
    return hipErrorInvalidValue;
  const int grid = (int)std::min<int64_t>(planes * a.parts, cap);
  if (a.resid) hipLaunchKernelGGL((k_iwh_pass<NW16, KHS, KWT, true>), dim3((unsigned)grid), dim3(256), (size_t)lds, st, a);
  else hipLaunchKernelGGL((k_iwh_pass<NW16, KHS, KWT, false>), dim3((unsigned)grid), dim3(256), (size_t)lds, st, a);
  return hipGetLastError();
}

template <int NW16>
static hipError_t iwh_dispatch(const IwhPassArgs& a, int num_cu, hipStream_t st) {
  const int s = a.kh / 16, u = a.kw / 16;
  if (s == 1 && u == 1) return iwh_launch<NW16, 1, 1>(a, num_cu, st);
  if constexpr (NW16 >= 2) {
    if (s == 1 && u == 2) return iwh_launch<NW16, 1, 2>(a, num_cu, st);
  }
  if (s == 2 && u == 1) return iwh_launch<NW16, 2, 1>(a, num_cu, st);
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace fa
