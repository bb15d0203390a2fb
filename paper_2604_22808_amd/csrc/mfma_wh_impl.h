#pragma once
// The W and H axes of the forward transform (paper section 3.2) in one pass over the input:
//   out[kh, t, kw, c] = sum_h Mh[kh][h] * fp16( sum_w Mw[kw][w] * x[t, h, w, c] )
// for up to three tensors (Q, K, V) per launch.  The plane between the two axes never reaches memory.
//
// A work item is 64 channels of one (tensor, slice, t) plane and KT tiles of 16 W coefficients, all H coefficients of
// them kept as accumulators for as long as the plane's rows stream by:
//   rows      x[t, h, :, 64 channels] (W pieces of 128 bytes) are copied straight into a ring of LDS slots, several groups
//             of rows ahead, across items too; the 32-byte column groups of a piece are permuted through the source
//             address so that the transposing reads below are free of bank conflicts
//   W axis    per row, a wave multiplies its 16 channels: v_mfma_f32_16x16x32_bf16 on the bf16 input as it is, the fp16
//             matrix split exactly into two bf16 terms (11 significant bits = 8 + 3), so nothing is converted and
//             nothing is rounded that an fp16 product would not round
//   between   rounded to fp16; a lane collects 16 rows h of its 4 kw x 1 channel, then a 4 x 4 exchange of lane groups
//             (v_permlane32_swap, v_permlane16_swap) turns them into operands that hold 16 consecutive h per kw
//   H axis    v_mfma_f32_16x16x16_f16, channels as rows, kh as columns: a lane ends up with 4 consecutive channels
// The accumulators (64 KHT registers per wave) bound the tile: KHT <= 2, two waves per SIMD.  A workgroup is KT x HT sets of
// four waves, a set for each W tile and each half of the H coefficients.  A plane is read by ceil(kw / (16 KT)) workgroups,
// which run side by side on one XCD: the first of them fetches the rows into its L2.
//
// What bounds it and what it measured (one tensor, against the two passes it replaces): HBM where few workgroups share a
// plane - 22 slices of 64^3 x 128 on the 32 x 32 box 631 -> 378 us (4.9 TB/s); LDS traffic, matrix instructions and the
// barrier per two rows, one after the other, where four do - 17 slices of 64^3 x 128 with 64 x 64 kept 838 -> 710 us.  Stores
// of 8 bytes per lane straight from the accumulators made that 844 us: hence the trip through LDS.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef __fp16 fp16x4 __attribute__((__vector_size__(4 * sizeof(__fp16))));

// One wave-wide copy of 16 bytes per lane from global memory into LDS: base (wave-uniform) + this lane's byte offset, lane l's
// piece at LDS byte dst + 16 l (issued as assembly: the kernel does its own waiting, see k_attn).
__device__ __forceinline__ void wh_dma16(const void* base, uint32_t lane_off, unsigned dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(dst) : "memory", "m0");
}

constexpr int WH_EROW = 144;   // bytes per staged output row (128 + 16: the 16 rows a wave writes side by side take all banks once)
template <int NW16> constexpr int wh_out_buffers() { return (NW16 + 1) / 2 % 2 == 0 ? 1 : 2; }   // (what LDS has room for beside the ring)
constexpr int WH_GR = 2;   // rows h per ring slot (a group)
// Ring slots (8 or 4: slots are numbered by their place in a block of 16 rows).  Up to W = 64, workgroups of four waves leave
// room for a second one on the compute unit; from W = 80 on the ring alone is 96 or 128 KB of its 160.
template <int NW16, int SETS> constexpr int wh_slots() {
  return 8 * WH_GR * ((NW16 + 1) / 2) * 4096 <= (SETS == 1 ? 64 : 128) * 1024 ? 8 : 4;
}

// The lane's number, worked out where it is used: addresses formed from it ahead of the main loop cost registers the loop needs.
// A spilled one is reloaded there, and the wait for it, which counts in order, takes the copies in flight along.  (Only the
// variants at the register limit do this: 12 slices of 32 x 32 x 128 x 128 on the whole grid, forward transforms 1199 us with three
// registers spilled, 1155 with none; the others are 0.5 % faster with the addresses kept.)
__device__ __forceinline__ int wh_lane() {
  unsigned all = ~0u;
  asm volatile("" : "+s"(all));
  return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

template <int NW16, int KHT, int KT, int HT>
__global__ void __launch_bounds__(256 * KT * HT, 2) k_wh_pass(WhPassArgs a) {
  constexpr int W = 16 * NW16;
  constexpr int KW = (NW16 + 1) / 2;           // 32-deep steps over w
  constexpr int SROWS = 32 * KW;               // LDS rows per h (rows beyond W stay zero)
  constexpr int GR = WH_GR, SETS = KT * HT;
  constexpr int SLOTS = wh_slots<NW16, SETS>();
  constexpr int NI = GR * NW16 * 2;            // copy instructions (8 rows of 128 bytes each) per group
  constexpr int NWV = 4 * SETS;                // waves
  constexpr int NPW = (NI + NWV - 1) / NWV;    // copies per wave and group
  constexpr bool TIGHT = KHT == 2 && NW16 > 6;   // (would spill registers)
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  uint16_t* ring = smem;                                        // [SLOTS][GR][SROWS][64]
  const int mstr = a.H + 8;                                 // row stride of the H matrix in LDS
  half_t* Mh = (half_t*)(smem + SLOTS * GR * SROWS * 64);   // [16 KHT HT][mstr]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave & 3, set = wave >> 2;    // this wave's 16 channels and set
  const int kt = set % KT, ht = set / KT;      // W tile of the workgroup, half of the H coefficients
  const int l16 = lane & 15, q = lane >> 4;
  constexpr int EB = wh_out_buffers<NW16>();
  char* stage = (char*)(Mh + 16 * KHT * HT * mstr) + set * (EB * 32 * WH_EROW);   // output rows on their way out

  for (int e = tid; e < 16 * KHT * HT * (a.H / 8); e += 64 * NWV) {
    const int row = e / (a.H / 8), c8 = e % (a.H / 8);
    uint4v v = {0u, 0u, 0u, 0u};
    if (row < a.kh) v = *(const uint4v*)(a.Mh + (size_t)row * a.H + c8 * 8);
    *(uint4v*)(Mh + row * mstr + c8 * 8) = v;
  }
  if constexpr (W < SROWS)
    for (int e = tid; e < SLOTS * GR * (SROWS - W) * 8; e += 64 * NWV) {
      const int r = e / 8, hr = r / (SROWS - W), w = W + r % (SROWS - W);
      *(uint4v*)(ring + ((size_t)hr * SROWS + w) * 64 + (e % 8) * 8) = uint4v{0u, 0u, 0u, 0u};
    }

  // Items of this workgroup.  Planes are dealt to the XCDs by their index mod 8 (workgroups are dealt round-robin by
  // blockIdx); the R workgroups of a plane have neighbouring places in their XCD's list.  With 64 or 128 channels per
  // token the channel chunk (plane index mod channels / 64) is then the same for all items of a workgroup.
  const int cpt = a.d >> 6, R = a.members;
  const int xcd = blockIdx.x & 7, J = gridDim.x >> 3;
  const int n_planes = a.seg_end[2] * a.T * cpt;
  const int n_items = n_planes > xcd ? ((n_planes - xcd + 7) >> 3) * R : 0;
  const int64_t row_stride = (int64_t)W * a.d;   // elements between rows h
  struct Item { const uint16_t* in; half_t* out; int r; };
  auto decode = [&](int l) -> Item {
    Item it;
    it.r = l % R;
    int p = (l / R) * 8 + xcd;
    const int chunk = p % cpt; p /= cpt;
    const int t = p % a.T; p /= a.T;
    const int seg = p < a.seg_end[0] ? 0 : p < a.seg_end[1] ? 1 : 2;
    const int sl = p - (seg == 0 ? 0 : seg == 1 ? a.seg_end[0] : a.seg_end[1]);
    const int32_t* list = seg == 0 ? a.slice_list[0] : seg == 1 ? a.slice_list[1] : a.slice_list[2];
    const int64_t slice = list ? list[sl] : sl;
    it.in = (const uint16_t*)(seg == 0 ? a.in[0] : seg == 1 ? a.in[1] : a.in[2]) + (slice * a.T + t) * a.H * row_stride + chunk * 64;
    it.out = (half_t*)(seg == 0 ? a.out[0] : seg == 1 ? a.out[1] : a.out[2]) + ((int64_t)sl * a.kh * a.T + t) * a.kw * a.d + chunk * 64;
    return it;
  };

  // Copies: instruction i of a group fills rows w = 8 (i % (W / 8)) .. + 7 of row h = i / (W / 8); a lane's 16-byte piece
  // comes from the column group its place stands for.  Column group of place p in row w: p ^ f(w), f from bits 1 and 3 of w.
  // (instruction i is copied by wave i mod the number of waves, which fixes bit 3 of w per wave)
  const uint32_t src = ((uint32_t)((lane >> 3) * a.d + (((lane & 7) ^ (((lane >> 4) & 1) << 1)) << 3)) * 2u) ^ ((wave & 1) << 6);
  const unsigned ring_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)ring;
  uint32_t c_src[NPW], c_dst[NPW];   // bytes from the group's first row / from the slot's start
#pragma unroll
  for (int n = 0; n < NPW; ++n) {
    int i = wave + n * NWV;
    if (NI % NWV != 0) i %= NI;   // (the same bytes twice; NI is even, so bit 3 of w stays the wave's)
    const int hr = i / (2 * NW16), w8 = i - hr * (2 * NW16);
    c_src[n] = (uint32_t)(hr * W + w8 * 8) * (uint32_t)a.d * 2u;
    c_dst[n] = ring_at + (uint32_t)(hr * SROWS + w8 * 8) * 128u;
  }
  auto copy_group = [&](const uint16_t* base, int slot) {
#pragma unroll
    for (int n = 0; n < NPW; ++n) wh_dma16((const char*)base + c_src[n], src, c_dst[n] + slot * (GR * SROWS * 128));
  };

  if ((int)(blockIdx.x >> 3) >= n_items) {   // nothing to do: zero sums
    if (a.tot_part && tid < 64 * SETS) a.tot_part[((size_t)(tid >> 6) * gridDim.x + blockIdx.x) * 64 + (tid & 63)] = 0.f;
    return;
  }

  // Rows are requested SLOTS - 1 groups ahead of their use: `pf` is the group requested next, `pnext` the first group of
  // the item after the one `pf` is in (of the last item: its own last group again and again, so that the count of copies
  // in flight stays what the waits assume).
  const int64_t group_stride = GR * row_stride;
  const int n_groups = a.H / GR;   // at least SLOTS (H is at least 16)
  const uint16_t* pf = decode(blockIdx.x >> 3).in;
#pragma unroll
  for (int s = 0; s < SLOTS - 1; ++s) { copy_group(pf, s); pf += group_stride; }

  // transposing reads: lane j of a group of 16 names row j / 4, columns 4 (j % 4) .. + 3 of the wave's 16 channels
  const int trow = 8 * q + (l16 >> 2);                                       // + 4 for the second half of an operand
  const int fz = ((trow >> 1) & 1) | (((trow >> 3) & 1) << 1);               // (the same for trow + 4, and + 32 s)
  const int boff = trow * 64 + ((wc ^ fz) << 4) + ((lane & 3) << 2);         // halfs

  // (one address register per 64 KB of the ring: what an LDS instruction's own offset reaches)
  constexpr int RING = SLOTS * GR * SROWS * 128, NBASE = (RING + 65535) / 65536;
  uint32_t rbase[NBASE];
#pragma unroll
  for (int i = 0; i < NBASE; ++i) {
    rbase[i] = ring_at + (uint32_t)boff * 2u + 65536u * i;
    asm volatile("" : "+v"(rbase[i]));
  }
  auto operand = [&](int lds_row, int s) -> uint4v {   // w = 32 s + 8 q .. + 7 of one channel
    uint4v b;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int at = (lds_row * SROWS + 32 * s + 4 * hh) * 128;
      typedef fp16x4 __attribute__((address_space(3))) * lds_ptr;
      const fp16x4 t4 = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_ptr)(uintptr_t)(rbase[at >> 16] + (uint32_t)(at & 65535)));
      const uint2v u2 = __builtin_bit_cast(uint2v, t4);
      b[2 * hh] = u2[0]; b[2 * hh + 1] = u2[1];
    }
    return b;
  };
  bf16x8 Ah[KW], Al[KW];   // matrix terms of the W tile: rows kw, k = w
  int a_tile = -1;
  float tot = 0.f;
  ushort2v amax = {0, 0};
  // the first row's operands (and everybody's part of the H matrix and the zero rows)
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((SLOTS - 2) * NPW) : "memory");
  uint4v b[2][KW];   // operands of two rows
#pragma unroll
  for (int s = 0; s < KW; ++s) b[0][s] = operand(0, s);
  for (int l = blockIdx.x >> 3; l < n_items; l += J) {
    const Item it = decode(l);
    const int kw0 = (it.r * KT + kt) * 16;     // first W coefficient of this wave
    if (kw0 != a_tile) {
      a_tile = kw0;
#pragma unroll
      for (int s = 0; s < KW; ++s) {
        const int ln = TIGHT ? wh_lane() : lane, k = 32 * s + 8 * (ln >> 4);
        half8 m = {0, 0, 0, 0, 0, 0, 0, 0};
        if (kw0 < a.kw && k < W) m = *(const half8*)((const char*)(a.Mw + (size_t)kw0 * W) + (uint32_t)((ln & 15) * W + k) * 2u);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float f = (float)m[j];
          const float hi = __uint_as_float(__float_as_uint(f) & 0xffff0000u);
          Ah[s][j] = (__bf16)hi;
          Al[s][j] = (__bf16)(f - hi);
        }
      }
    }
    // The sets of waves that read a plane share the sums and the range check of its rows: a set takes every nm-th group.
    const int nm = R * SETS, me = it.r * SETS + set;
    int turn = 0;   // group of the plane mod nm
    const bool more = l + J < n_items;
    const uint16_t* pnext = more ? decode(l + J).in : nullptr;
    int left = n_groups - (SLOTS - 1);   // groups of this item still to be requested

    float4v acc[16][KHT];
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
      for (int n = 0; n < KHT; ++n) acc[k][n] = float4v{0.f, 0.f, 0.f, 0.f};

    float te[2] = {0.f, 0.f};
    for (int h0 = 0; h0 < a.H; h0 += 16) {
      uint32_t st[4][4][2];   // [kw 4 q + r][4 rows h][pair of rows]
#pragma unroll
      for (int p = 0; p < 8; ++p) {   // pairs of rows = groups
        uint32_t first[4];   // the first row's results
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float4v y[2];
          // The operands of a row are requested while the row before it is multiplied: the second row of the group, then
          // the first row of the next group, behind the barrier that says it has arrived - and that everybody has done
          // with the slot of the group before this one (its operands have been multiplied), which the next copies go into.
          if (u == 1) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((SLOTS - 3) * NPW) : "memory");
            if (left == 0 && more) pf = pnext;
            if (left <= 0 && !more) pf -= group_stride;
            copy_group(pf, (p + SLOTS - 1) % SLOTS);
            pf += group_stride;
            --left;
          }
#pragma unroll
          for (int s = 0; s < KW; ++s) b[u ^ 1][s] = operand(((p + u) % SLOTS) * GR + (u ^ 1), s);
          __builtin_amdgcn_sched_barrier(0);
          // (In front of the products: a draft with this branch behind them gave wrong sums.  Its cause was not shown - the
          // compiler keeps the wait states between a product and the first use of its result on both ways of a branch, 8 here
          // as in that form - so the order stays.)
          if (turn == me) {
#pragma unroll
            for (int s = 0; s < KW; ++s)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const uint32_t x = b[u][s][j];
                const uint32_t m = x & 0x7fff7fffu;
                amax = __builtin_elementwise_max(amax, __builtin_bit_cast(ushort2v, m));
                te[j & 1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, x), te[j & 1], false);
              }
          }
          y[0] = y[1] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < KW; ++s) {
            y[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al[s], __builtin_bit_cast(bf16x8, b[u][s]), y[0], 0, 0, 0);
            y[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah[s], __builtin_bit_cast(bf16x8, b[u][s]), y[1], 0, 0, 0);
          }
          // (pinned here: postponed to the exchange below, the rounding would keep twice the registers alive)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const _Float16 h = (_Float16)(y[0][r] + y[1][r]);
            const uint32_t bits = __builtin_bit_cast(uint16_t, h);
            if (u == 0) {
              first[r] = bits;
              asm volatile("" : "+v"(first[r]));
            } else {
              uint32_t pk = first[r] | (bits << 16);
              asm volatile("" : "+v"(pk));
              st[r][p >> 1][p & 1] = pk;
            }
          }
        }
        if (++turn == nm) turn = 0;
      }
      half4 B[KHT];
      const int ln = TIGHT ? wh_lane() : lane;
#pragma unroll
      for (int n = 0; n < KHT; ++n) B[n] = *(const half4*)(Mh + (16 * (ht * KHT + n) + (ln & 15)) * mstr + h0 + 4 * (ln >> 4));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // block b of lane group g: rows 4 b .. of kw 4 g + r  ->  block g of kw 4 b + r
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          auto s0 = __builtin_amdgcn_permlane32_swap(st[r][0][j], st[r][2][j], false, false);
          auto s1 = __builtin_amdgcn_permlane32_swap(st[r][1][j], st[r][3][j], false, false);
          auto t0 = __builtin_amdgcn_permlane16_swap(s0[0], s1[0], false, false);
          auto t1 = __builtin_amdgcn_permlane16_swap(s0[1], s1[1], false, false);
          st[r][0][j] = t0[0]; st[r][1][j] = t0[1]; st[r][2][j] = t1[0]; st[r][3][j] = t1[1];
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const half4 A = __builtin_bit_cast(half4, uint2v{st[r][b][0], st[r][b][1]});
#pragma unroll
          for (int n = 0; n < KHT; ++n) acc[4 * b + r][n] = __builtin_amdgcn_mfma_f32_16x16x16f16(A, B[n], acc[4 * b + r][n], 0, 0, 0);
        }
      }
    }
    // (wait states between the last products and the first use of their accumulators, whatever way leads there)
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    tot += te[0] + te[1];

    // A lane holds channels 4 q .. + 3 of the wave's 16 at kh = 16 (ht KHT + n) + l16.  Two kw at a time go through LDS, where the
    // four waves of a set put their channels together: whole 128-byte rows are stored.
    {
      const bool mine = kw0 < a.kw;
      const int64_t kh_stride = (int64_t)a.T * a.kw * a.d;
      const int ln = TIGHT ? wh_lane() : lane, l16 = ln & 15, q = ln >> 4;
      const int row = wc * 8 + (ln >> 3);   // kw = row / 16, kh = row % 16
      const uint32_t lane_out = ((uint32_t)(row & 15) * (uint32_t)kh_stride + (uint32_t)((row >> 4) * a.d + (ln & 7) * 8)) * 2u;
#pragma unroll
      for (int n = 0; n < KHT; ++n) {
        const bool store = mine && 16 * (ht * KHT + n) < a.kh;
        char* dst = (char*)(it.out + 16 * (ht * KHT + n) * kh_stride + (int64_t)kw0 * a.d);
#pragma unroll
        for (int k = 0; k < 16; k += 2) {
          char* sb = stage + ((k >> 1) % EB) * (32 * WH_EROW);
          if (EB == 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
          for (int kk = 0; kk < 2; ++kk) {
            uint2v v;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const _Float16 lo = (_Float16)acc[k + kk][n][2 * j], hi = (_Float16)acc[k + kk][n][2 * j + 1];
              v[j] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
            }
            *(uint2v*)(sb + (kk * 16 + l16) * WH_EROW + wc * 32 + q * 8) = v;
          }
          asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
          const uint4v v = *(const uint4v*)(sb + row * WH_EROW + (ln & 7) * 16);
          if (store) *(uint4v*)(dst + lane_out) = v;
          dst += (size_t)a.d * 4;
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may land in LDS that another workgroup owns by then
  // an input that fp16 cannot hold (the spectral buffers' range contract), infinities and NaN included
  if (a.range_flag && (amax[0] >= 0x4780 || amax[1] >= 0x4780)) *a.range_flag = 1;
  if (a.tot_part) {   // per channel of the workgroup's chunk, this wave's rows
    tot += __shfl_xor(tot, 16);
    tot += __shfl_xor(tot, 32);
    if (q == 0) a.tot_part[((size_t)set * gridDim.x + blockIdx.x) * 64 + wc * 16 + l16] = tot;
  }
}

template <int NW16, int KHT, int KT, int HT>
static hipError_t wh_launch(WhPassArgs a, int num_cu, hipStream_t st, int* slots_out) {
  constexpr int RING = wh_slots<NW16, KT * HT>() * WH_GR * ((NW16 + 1) / 2) * 4096;
  constexpr int STAGE = KT * HT * wh_out_buffers<NW16>() * 32 * WH_EROW;
  static_assert(RING + STAGE + 16 * KHT * HT * (128 + 8) * 2 <= 160 * 1024, "LDS of one compute unit");
  const int lds = RING + STAGE + 16 * KHT * HT * (a.H + 8) * 2;
  a.members = (a.kw / 16 + KT - 1) / KT;
  const int64_t planes = (int64_t)a.seg_end[2] * a.T * (a.d / 64);
  if (planes <= 0) return hipSuccess;
  if (planes * a.members > 0x3fffffff) return hipErrorInvalidValue;
  // per-lane byte offsets are unsigned 32-bit numbers: 16 rows kh of the output, the rows of a group of the input
  if ((int64_t)a.T * a.kw * a.d * 2 * 16 > 0xffffffffLL || (int64_t)WH_GR * 16 * NW16 * a.d * 2 > 0xffffffffLL) return hipErrorInvalidValue;
  const int per_cu = std::min(2 / (KT * HT), 160 * 1024 / lds);
  const int64_t per_xcd = (planes + 7) / 8 * a.members;   // items of the fullest XCD
  const int grid = 8 * (int)std::min<int64_t>(per_xcd, std::max(1, num_cu / 8) * per_cu);
  static OncePerDevice limit;
  hipError_t e = allow_lds(limit, (const void*)k_wh_pass<NW16, KHT, KT, HT>, 160 * 1024);
  if (e != hipSuccess) return e;
  if (slots_out) *slots_out = grid * KT * HT;
  hipLaunchKernelGGL((k_wh_pass<NW16, KHT, KT, HT>), dim3((unsigned)grid), dim3(256 * KT * HT), (size_t)lds, st, a);
  return hipGetLastError();
}

template <int NW16>
static hipError_t wh_dispatch(const WhPassArgs& a, int num_cu, hipStream_t st, int* slots_out) {
  const int kht = a.kh / 16;
  // A single W tile: the whole axis of 16, or the box of an axis that can be cut that far (a power of two).
  if constexpr ((NW16 & (NW16 - 1)) == 0) {
    if (a.kw == 16 && kht == 1) return wh_launch<NW16, 1, 1, 1>(a, num_cu, st, slots_out);
    if (a.kw == 16 && kht == 2) return wh_launch<NW16, 2, 1, 1>(a, num_cu, st, slots_out);
  }
  if constexpr (NW16 > 1) {
    if (a.kw > 16 && kht == 1) return wh_launch<NW16, 1, 2, 1>(a, num_cu, st, slots_out);
    if (a.kw > 16 && kht == 2) return wh_launch<NW16, 2, 2, 1>(a, num_cu, st, slots_out);
  }
  if (kht == 3 || kht == 4) return wh_launch<NW16, 2, 1, 2>(a, num_cu, st, slots_out);
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace fa
