#pragma once
// The W and H axes of the forward transform (paper section 3.2) in one pass over the input:
//   out[kh, t, kw, c] = sum_h Mh[kh][h] * fp16( sum_w Mw[kw][w] * x[t, h, w, c] )
// for up to three tensors (Q, K, V) per launch.  The plane between the two axes never reaches memory.  And (INV) those of the
// inverse transform (section 3.7), the same contraction from fp16 coefficients to bf16 values:
//   out[t, h, w, c] = (v[t, h, w, c] +) fp16( sum_kh Fh[h][kh] * fp16( sum_kw Fw[w][kw] * y[kh, t, kw, c] ) )
// where the comments below say coefficients for the output's rows and columns, positions for the input's.
//
// A work item is 64 channels of one (tensor, slice, t) plane and KT tiles of 16 W coefficients, all 16 KH H coefficients of
// them kept as accumulators (32 KT KH registers per wave) for as long as the plane's rows stream by, 16 rows per round:
//   W axis    a wave takes two rows h of the round by itself, 32 positions w at a time, straight from memory into registers: 8 lanes
//             hold a position's 128 bytes.  Lanes 8 apart exchange halves of what they hold (a lane then has 4 channels of twice the
//             positions, one DPP move per register), and pairing the positions' halfwords (v_perm_b32, one per register) makes
//             operands of v_mfma_f32_16x16x32_bf16 for 4 x 16 channels.  Positions within a step go in the order the loads leave
//             them in; the matrix, in LDS, has its columns in the same order.  The bf16 input is multiplied as it is, the
//             fp16 matrix split exactly into two bf16 terms (11 significant bits = 8 + 3), so nothing is converted and nothing
//             is rounded that an fp16 product would not round
//   between   rounded to fp16 and left in LDS, [h][kw][channel], for everybody (two buffers, one barrier per round)
//   H axis    a wave takes 2 KT of the W coefficients, 64 channels and all H coefficients: transposing LDS reads,
//             v_mfma_f32_16x16x16_f16 with channels as rows, kh as columns
// The next steps' rows (up to 4 steps of 4 KB per wave) are always on their way, across rounds and items.  A plane is read by
// ceil(kw / (16 KT)) workgroups, which run side by side on one XCD: the first of them fetches the rows into its L2.
//
// What bounds it: where one or two workgroups share a plane, memory (22 slices of 64^3 x 128 on the 32 x 32 box: 5.0 TB/s); where
// four and more do, what a compute unit takes in from its L2.  Copying the rows through LDS and reading operands from
// there moved 48 KB of LDS per row of 128 x 64, with a barrier every two rows; this moves 14.  One tensor's share of a launch, rows
// through LDS -> this: 12 slices of 64 x 128 x 128 x 128 on the 64 x 64 box 1.33 -> 0.98 ms; 17 of 64^3 x 128 whole 0.70 -> 0.54; 12 of
// 32 x 48 x 80 x 128 whole 0.27 -> 0.18.  On the way there (first / second of these): 8 bytes per lane and load, which the L1 serves at
// 36 bytes per cycle instead of 64, 1.18 / 0.68; stores as the products leave them (16 bytes per lane, neighbouring lanes in different
// rows) 1.01 / 0.60; all workgroups of a plane taking its rows in the same order (all wait for memory at once) +10 / +3 %.
// Inverse, against two passes: 17 slices of 64^3 x 128 whole 0.82 -> 0.56 ms; 6 of 64 x 128 x 128 x 128 from the 64 x 64 box 1.18 -> 1.02, from
// the 32 x 32 box 1.00 -> 0.72; 24 of 32 x 48 x 80 x 128 whole 0.66 -> 0.48.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef __fp16 fp16x4 __attribute__((__vector_size__(4 * sizeof(__fp16))));

constexpr int WH_WAVES = 8;
// Steps requested ahead (the inverse's rows come from the L2 more often than from memory, and V's take registers in between).  They live in registers (16 each) beside the accumulators; the number divides the steps of a round.
template <int KW, int KT, int KH, bool INV> constexpr int wh_depth() {
  if (KT * KH == 1 || KT * KT * KH > 4 || (INV && KH == 4)) return 2;
  return KW == 1 ? 2 : KW == 3 ? 3 : 4;
}
constexpr int wh_row_bytes(int KT) { return KT * 2048 + 64; }   // a row between the axes: [16 KT][64] fp16, and 64 bytes against bank conflicts
constexpr int wh_waves_per_simd(int KW, int KT, int KH) { return KT * KH == 1 && KW <= 2 ? 4 : 2; }

// `own`, but lanes of the banks (4 lanes of each 16) in the mask take `other` of the lane 8 places on in their 16.
__device__ __forceinline__ uint32_t wh_from_other(uint32_t own, uint32_t other, int banks) {
  return banks == 0xc ? __builtin_amdgcn_update_dpp((int)own, (int)other, 0x128, 0xf, 0xc, false)
                      : __builtin_amdgcn_update_dpp((int)own, (int)other, 0x128, 0xf, 0x3, false);
}

// One launch: up to three passes (the slices that keep different boxes), workgroups [first[i], first[i + 1]) run the i-th.
struct WhLaunch { WhPassArgs sub[3]; int first[4]; };

// Workgroup `block` of the `blocks` of a pass.
template <int NW16, int KT, int KH, bool INV>
__device__ __forceinline__ void wh_pass(const WhPassArgs& a, const int block, const int blocks, const int tid = threadIdx.x) {
  constexpr int W = 16 * NW16;                 // positions (inverse: coefficients) of an input row
  constexpr int TERMS = INV ? 1 : 2;           // terms the W matrix is split into
  constexpr int KW = (NW16 + 1) / 2;           // steps of 32 positions w per row (the last one of 16 when NW16 is odd)
  constexpr int U = 2 * KW;                    // steps of a wave per round
  constexpr int D = wh_depth<KW, KT, KH, INV>();
  static_assert(U % D == 0, "a step's registers are known at compile time");
  constexpr int RB = wh_row_bytes(KT);
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  char* Ys = smem;                                              // [2][16] rows between the axes
  uint4v* Aw = (uint4v*)(Ys + 2 * 16 * RB);                     // [KT][KW][hi, lo][lane]: matrix operands of the W axis
  float* tot = (float*)(Aw + KT * KW * TERMS * 64);             // [wave][64]: sums of squares of the rows a wave has taken
  half_t* Mh = (half_t*)(tot + WH_WAVES * 64);                  // [16 KH][mstr]
  const int mstr = a.rows + 8;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4;

  // Items of this workgroup.  Planes are dealt to the XCDs by their index mod 8 (workgroups are dealt round-robin by
  // blockIdx); the R workgroups of a plane have neighbouring places in their XCD's list.  With 64, 128, 256 or 512 channels per
  // token the channel chunk (plane index mod channels / 64) is then the same for all items of a workgroup.
  const int cpt = a.d >> 6, R = a.members;
  const int xcd = block & 7, J = blocks >> 3;
  const int n_planes = a.seg_end[2] * a.T * cpt;
  const int n_items = n_planes > xcd ? ((n_planes - xcd + 7) >> 3) * R : 0;
  // Rows of the caller's tensors are [slice][t][h][w], rows of the other side [segment's slice][kh][t][kw].
  const int64_t row_bytes = (INV ? (int64_t)a.T : 1) * W * a.d * 2;                    // between input rows
  const int64_t out_stride = (INV ? 1 : (int64_t)a.T) * a.out_cols * a.d;              // between output rows, elements
  struct Item { const char* in; uint16_t* out; int r; };
  auto decode = [&](int l) -> Item {
    Item it;
    it.r = l % R;
    int p = (l / R) * 8 + xcd;
    const int chunk = p % cpt; p /= cpt;
    const int t = p % a.T; p /= a.T;
    const int seg = p < a.seg_end[0] ? 0 : p < a.seg_end[1] ? 1 : 2;
    const int sl = p - (seg == 0 ? 0 : seg == 1 ? a.seg_end[0] : a.seg_end[1]);
    const int32_t* list = seg == 0 ? a.slice_list[0] : seg == 1 ? a.slice_list[1] : a.slice_list[2];
    const int64_t slice = __builtin_amdgcn_readfirstlane(list ? list[sl] : sl);   // (addresses stay in scalar registers)
    const int64_t whole = (slice * a.T + t) * (INV ? a.out_rows : a.rows) * (int64_t)((INV ? a.out_cols : W) * a.d);
    const int64_t compact = ((int64_t)sl * (INV ? a.rows : a.out_rows) * a.T + t) * (int64_t)((INV ? W : a.out_cols) * a.d);
    it.in = (const char*)((const uint16_t*)(seg == 0 ? a.in[0] : seg == 1 ? a.in[1] : a.in[2]) + (INV ? compact : whole) + chunk * 64);
    it.out = (uint16_t*)(seg == 0 ? a.out[0] : seg == 1 ? a.out[1] : a.out[2]) + (INV ? whole : compact) + chunk * 64;
    return it;
  };
  // Workgroup r of a plane: column part r % Rc (KT tiles of 16), row part r / Rc (KH tiles of 16; forward passes have one)
  const int Rc = a.col_parts;
  if ((block >> 3) >= n_items) {   // nothing to do: zero sums
    if (a.tot_part) a.tot_part[((size_t)wave * blocks + block) * 64 + lane] = 0.f;
    return;
  }

  // Step u of a round: the wave's row u / KW, positions 32 (u % KW) + 16 hh + 4 q + 2 j + l16 / 8, channels 8 (l16 % 8) .. + 7.
  const int late8 = l16 >> 3, piece = 2 * (l16 & 7) + late8;   // the lane's operand column: channels 4 piece .. + 3
  const uint32_t src = (uint32_t)((4 * q + late8) * a.d + 8 * (l16 & 7)) * 2u;   // this lane's bytes of its first position
  // The workgroups of a plane go through a round's rows in different orders, so that each is the first one to ask memory for
  // a part of them and finds the rest in the L2: half of them take the second eight rows first (nothing else depends on
  // it), and for every other pair of W tiles the halves of a row change places (the order of the sum, so it goes by the tile
  // and not by the workgroup: the same coefficient may come from another grouping of tiles).
  const uint32_t step16 = (uint32_t)a.d * 32u;   // bytes of 16 positions
  uint4v x[D][2][2];
  struct Order { int64_t second; int32_t lo, hi; int first; };   // bytes from the first row of a round to the second, of the changes; the first row
  auto order = [&](int member) -> Order {
    Order o;
    const int r = INV ? member % Rc : member;
    const int late = (KT == 1 ? r : r >> 1) & 1, turned = KW % 2 == 0 && NW16 % 2 == 0 ? (KT == 1 ? r >> 1 : r) & 1 : 0;
    o.first = wave + 8 * late;
    o.second = (late ? -8 : 8) * row_bytes;
    o.lo = turned * (W / 2) * a.d * 2;
    o.hi = -o.lo;
    return o;
  };
  auto request = [&](const char* rows, const Order& o, int u) {
    uint32_t at = src;
    asm("" : "+v"(at));   // (a 32-bit offset to the compiler, which the load itself adds to a base in scalar registers)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
      if (32 * (u % KW) + 16 * hh < W)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          typedef const char __attribute__((address_space(1))) * ptr;
          ptr p = (ptr)(rows + (u / KW ? o.second : 0) + (KW % 2 ? 0 : 2 * (u % KW) < KW ? o.lo : o.hi) + (size_t)(2 * (u % KW) + hh) * step16 + j * (step16 >> 3));
          asm("" : "+s"(p));
          x[u % D][hh][j] = *(const uint4v __attribute__((address_space(1)))*)(p + at);
        }
  };

  // between the axes: piece of 4 channels p4 of (row h, coefficient k) sits at h RB + (k ^ (k / 4 & 1)) 128 + (p4 ^ (h / 4 & 1)) 8,
  // which spreads what half a wave writes (two groups of 4 coefficients) and reads (8 rows) over all banks
  const unsigned ys_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)Ys;
  uint32_t put[2];   // (coefficients 4 q and 4 q + 1 of a tile)
#pragma unroll
  for (int r = 0; r < 2; ++r) put[r] = (uint32_t)(wave * RB + ((4 * q + r) ^ (q & 1)) * 128 + ((piece ^ ((wave >> 2) & 1)) * 8));
  // (transposing read: lane 4 k + c of a group of 16 names row k, piece c of the four; row 4 q + k, pieces 8 p + 2 c + b)
  const uint32_t get0 = ys_at + (uint32_t)((4 * q + (l16 >> 2)) * RB + ((2 * (l16 & 3) + (q & 1)) * 8));
  const uint32_t get1 = get0 ^ 8u;   // (b = 1)

  int l = block >> 3;
  Item it = decode(l);
  Order ord = order(it.r);
  const char* rows = it.in + ord.first * row_bytes;   // this wave's first row of the round
#pragma unroll
  for (int u = 0; u < D; ++u) request(rows, ord, u);

  tot[tid] = 0.f;   // (a wave's own)
  ushort2v amax = {0, 0};
  int a_r = -1, buf = 0;
  for (;;) {
    if (it.r != a_r) {   // (everybody's last reads of the operands that go: behind the barrier of the last round)
      a_r = it.r;
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      for (int e = tid; e < KT * KW * 64; e += 64 * WH_WAVES) {
        const int ln = e & 63, s = (e >> 6) % KW, kt = (e >> 6) / KW;
        const int c0 = ((INV ? it.r % Rc : it.r) * KT + kt) * 16;   // first output column of the tile
        half8 m8;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const int w = 32 * s + (KW % 2 ? 0 : 2 * s < KW ? ord.lo : ord.hi) / (2 * a.d) + 16 * hh + 4 * (ln >> 4);
          half4 m = {0, 0, 0, 0};
          if (c0 < a.out_cols && w < W) m = *(const half4*)(a.Mw + (size_t)(c0 + (ln & 15)) * a.ldw + w);
#pragma unroll
          for (int j = 0; j < 4; ++j) m8[4 * hh + j] = m[j];
        }
        if constexpr (INV) {
          Aw[(kt * KW + s) * 64 + ln] = __builtin_bit_cast(uint4v, m8);
        } else {
          bf16x8 hi, lo;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float f = (float)m8[j];
            const float h = __uint_as_float(__float_as_uint(f) & 0xffff0000u);
            hi[j] = (__bf16)h;
            lo[j] = (__bf16)(f - h);
          }
          Aw[((kt * KW + s) * 2 + 0) * 64 + ln] = __builtin_bit_cast(uint4v, hi);
          Aw[((kt * KW + s) * 2 + 1) * 64 + ln] = __builtin_bit_cast(uint4v, lo);
        }
      }
      const int row0 = INV ? it.r / Rc * 16 * KH : 0;
      for (int e = tid; e < 16 * KH * (a.rows / 8); e += 64 * WH_WAVES) {
        const int row = e / (a.rows / 8), c8 = e % (a.rows / 8);
        uint4v v = {0u, 0u, 0u, 0u};
        if (row0 + row < a.out_rows) v = *(const uint4v*)(a.Mh + (size_t)(row0 + row) * a.ldh + c8 * 8);
        *(uint4v*)(Mh + row * mstr + c8 * 8) = v;
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    const bool more = l + J < n_items;
    Item next = it;
    if (more) next = decode(l + J);
    const Order ord_next = order(next.r);

    float4v acc[2 * KT][4][KH];
#pragma unroll
    for (int k = 0; k < 2 * KT; ++k)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int n = 0; n < KH; ++n) acc[k][c][n] = float4v{0.f, 0.f, 0.f, 0.f};
    float te[4] = {0.f, 0.f, 0.f, 0.f};
    int turn = it.r;   // the workgroups of a plane share the sums and the range check of its rows, round by round
    for (int h0 = 0; h0 < a.rows; h0 += 16) {
      // (behind the last item its rows once more, so that the code does not depend on it)
      const char* rows_next = h0 + 16 < a.rows ? rows + 16 * row_bytes : next.in + ord_next.first * row_bytes;
      const bool mine = turn == 0;
      turn = turn == 0 ? R - 1 : turn - 1;
      float4v y[KT][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = u % KW;
        constexpr int LAST = NW16 & 1;   // the last step of a row has 16 positions
        const bool half = LAST && s == KW - 1;
        if (s == 0)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int c = 0; c < 4; ++c) y[kt][c] = float4v{0.f, 0.f, 0.f, 0.f};
        uint4v A[KT][2];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) A[kt][TERMS - 1] = Aw[((kt * KW + s) * TERMS + TERMS - 1) * 64 + lane];
        uint4v B[4];   // channels 4 piece + c
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // positions 4 q + 2 (i % 2), + 1 of 16
          if (half && i >= 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) B[c][i] = 0u;
            continue;
          }
          const uint4v v = x[u % D][i >> 1][i & 1];
#pragma unroll
          for (int w = 0; w < 2; ++w) {   // words of the lane's 4 channels: of the even and of the odd position
            const uint32_t lo = v[w], hi = v[2 + w];
            const uint32_t even = wh_from_other(lo, hi, 0xc), odd = wh_from_other(hi, lo, 0x3);
            B[2 * w][i] = __builtin_amdgcn_perm(odd, even, 0x05040100u);
            B[2 * w + 1][i] = __builtin_amdgcn_perm(odd, even, 0x07060302u);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!INV && mine) {
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < (half ? 2 : 4); ++i) {
              const uint32_t xx = B[c][i], m = xx & 0x7fff7fffu;
              amax = __builtin_elementwise_max(amax, __builtin_bit_cast(ushort2v, m));
              te[c] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xx), __builtin_bit_cast(bf16x2, xx), te[c], false);
            }
        }
        if constexpr (!INV)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt) A[kt][0] = Aw[((kt * KW + s) * 2 + 0) * 64 + lane];
#pragma unroll
        for (int t = TERMS - 1; t >= 0; --t)   // the small terms first
#pragma unroll
          for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              if constexpr (INV) {
                if (half) {
                  const half4 Ah = __builtin_bit_cast(half4, uint2v{A[kt][0][0], A[kt][0][1]}), Bh = __builtin_bit_cast(half4, uint2v{B[c][0], B[c][1]});
                  y[kt][c] = __builtin_amdgcn_mfma_f32_16x16x16f16(Ah, Bh, y[kt][c], 0, 0, 0);
                } else {
                  y[kt][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, A[kt][0]), __builtin_bit_cast(half8, B[c]), y[kt][c], 0, 0, 0);
                }
              } else if (half) {
                const short4v Ah = __builtin_bit_cast(short4v, uint2v{A[kt][t][0], A[kt][t][1]}), Bh = __builtin_bit_cast(short4v, uint2v{B[c][0], B[c][1]});
                y[kt][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Ah, Bh, y[kt][c], 0, 0, 0);
              } else {
                y[kt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[kt][t]), __builtin_bit_cast(bf16x8, B[c]), y[kt][c], 0, 0, 0);
              }
            }
        __builtin_amdgcn_sched_barrier(0);
        request(u + D < U ? rows : rows_next, u + D < U || h0 + 16 < a.rows ? ord : ord_next, (u + D) % U);   // (here its registers are free)
        if (s == KW - 1)
#pragma unroll
          for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              half4 v;
#pragma unroll
              for (int c = 0; c < 4; ++c) v[c] = (_Float16)y[kt][c][r];
              *(half4*)(Ys + (buf * 16 + 8 * ((u / KW) ^ (ord.first >> 3))) * RB + kt * 2048 + (r >> 1) * 256 + put[r & 1]) = v;
            }
        __builtin_amdgcn_sched_barrier(0);
      }
      rows = rows_next;
      // Rows are there; and whoever is past this has read the buffer the next round writes into.
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      half4 Bm[KH];
#pragma unroll
      for (int n = 0; n < KH; ++n) Bm[n] = *(const half4*)(Mh + (16 * n + l16) * mstr + h0 + 4 * q);
#pragma unroll
      for (int k = 0; k < 2 * KT; ++k) {
        const int kw = wave * 2 * KT + k;
        const uint32_t at = (uint32_t)(buf * 16 * RB + (kw ^ ((kw >> 2) & 1)) * 128);
#pragma unroll
        for (int c = 0; c < 4; ++c) {   // 16 channels 32 (c / 2) + 8 (i / 4) + 4 (c % 2) + i % 4
          typedef fp16x4 __attribute__((address_space(3))) * lds_ptr;
          const fp16x4 t4 = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_ptr)(uintptr_t)((c & 1 ? get1 : get0) + at + 64u * (c >> 1)));
          const half4 Ay = __builtin_bit_cast(half4, t4);
#pragma unroll
          for (int n = 0; n < KH; ++n) acc[k][c][n] = __builtin_amdgcn_mfma_f32_16x16x16f16(Ay, Bm[n], acc[k][c][n], 0, 0, 0);
        }
      }
      buf ^= 1;
    }
    if (!INV && a.tot_part) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        te[c] += __shfl_xor(te[c], 16);
        te[c] += __shfl_xor(te[c], 32);
      }
      if (q == 0) *(float4v*)(tot + wave * 64 + 4 * piece) += float4v{te[0], te[1], te[2], te[3]};
    }
    {
      // A lane holds channels 32 p + 8 q .. + 7 of row 16 n + l16.  Sixteen rows at a time go through LDS, so that eight neighbouring
      // lanes store a row's 128 bytes.
      // The place is the wave's own: the row it writes first in the next round.
      char* stage = Ys + (buf * 16 + wave) * RB;
      int ln = lane;   // (addresses formed from it here: kept through the rounds they would cost registers that the rounds need)
      asm volatile("" : "+v"(ln));
      char* const put_at = stage + (ln & 15) * 128;
      const char* const get_at = stage + (ln >> 3) * 128 + ((ln & 7) ^ (ln >> 3)) * 16;
      const uint32_t lane_out = ((uint32_t)(ln >> 3) * (uint32_t)out_stride + 8u * (uint32_t)(ln & 7)) * 2u;
      const int col0 = (INV ? it.r % Rc : it.r) * 16 * KT + wave * 2 * KT, row0 = INV ? it.r / Rc * 16 * KH : 0;
      uint16_t* const first = it.out + row0 * out_stride + (int64_t)col0 * a.d;
      // (V where the output goes, requested one group of 16 rows ahead)
      const bool add = INV && a.resid;
      uint4v rs[2][2];
      auto request_v = [&](int i) {
        const int k = i / KH, n = i % KH;
        if (row0 + 16 * n < a.out_rows)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            typedef const char __attribute__((address_space(1))) * ptr;
            ptr at = (ptr)((const uint16_t*)a.resid + (first - (const uint16_t*)a.out[0]) + (16 * n + 8 * p) * out_stride + k * a.d);
            asm("" : "+s"(at));
            rs[i & 1][p] = *(const uint4v __attribute__((address_space(1)))*)(at + lane_out);
          }
      };
      if (col0 < a.out_cols) {
        if (INV && add) request_v(0);
#pragma unroll
        for (int i = 0; i < 2 * KT * KH; ++i) {
          const int k = i / KH, n = i % KH;
          if (INV && add && i + 1 < 2 * KT * KH) request_v(i + 1);
          if (row0 + 16 * n >= a.out_rows || (!INV && col0 + k >= a.out_cols)) continue;
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            if (INV && !add) {
              bf16x8 v;
#pragma unroll
              for (int j = 0; j < 8; ++j) v[j] = (__bf16)acc[k][2 * p + (j >> 2)][n][j & 3];
              *(bf16x8*)(put_at + (((4 * p + (ln >> 4)) ^ (ln & 7)) * 16)) = v;
            } else {
              half8 v;
#pragma unroll
              for (int j = 0; j < 8; ++j) v[j] = (_Float16)acc[k][2 * p + (j >> 2)][n][j & 3];
              *(half8*)(put_at + (((4 * p + (ln >> 4)) ^ (ln & 7)) * 16)) = v;
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            uint4v v = *(const uint4v*)(get_at + p * 1024);
            if (INV && add) {   // out = resid + result, both bf16 in memory, the sum formed in fp32
              const half8 h = __builtin_bit_cast(half8, v);
              bf16x8 b;
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const uint32_t w = rs[i & 1][p][j];
                b[2 * j] = (__bf16)(__uint_as_float(w << 16) + (float)h[2 * j]);
                b[2 * j + 1] = (__bf16)(__uint_as_float(w & 0xffff0000u) + (float)h[2 * j + 1]);
              }
              v = __builtin_bit_cast(uint4v, b);
            }
            typedef char __attribute__((address_space(1))) * ptr;
            ptr at = (ptr)(first + (16 * n + 8 * p) * out_stride + k * a.d);
            asm("" : "+s"(at));
            if (INV || row0 + 16 * n + 8 * p + (ln >> 3) < a.out_rows) *(uint4v __attribute__((address_space(1)))*)(at + lane_out) = v;
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    if (!more) break;
    l += J;
    it = next;
    ord = ord_next;
  }
  if constexpr (INV) return;
  // an input that fp16 cannot hold (the spectral buffers' range contract), infinities and NaN included
  if (a.range_flag && (amax[0] >= 0x4780 || amax[1] >= 0x4780)) *a.range_flag = 1;
  if (a.tot_part) a.tot_part[((size_t)wave * blocks + block) * 64 + lane] = tot[tid];   // per channel of the workgroup's chunk
}

template <int NW16, int KT, int KH, bool INV>
__global__ void __launch_bounds__(64 * WH_WAVES, wh_waves_per_simd((NW16 + 1) / 2, KT, KH)) k_wh_pass(WhLaunch m) {
  const int i = ((int)blockIdx.x >= m.first[1]) + ((int)blockIdx.x >= m.first[2]);
  wh_pass<NW16, KT, KH, INV>(m.sub[i], (int)blockIdx.x - m.first[i], m.first[i + 1] - m.first[i]);
}

// Inverse passes from boxes of different widths (16, 32, 64) to planes of one size.
template <int KT, int KH>
__global__ void __launch_bounds__(64 * WH_WAVES, 2) k_hw_mixed(WhLaunch m) {
  const int i = ((int)blockIdx.x >= m.first[1]) + ((int)blockIdx.x >= m.first[2]);
  const int block = (int)blockIdx.x - m.first[i], blocks = m.first[i + 1] - m.first[i];
  switch (m.sub[i].cols >> 4) {   // (uniform)
    case 1: wh_pass<1, KT, KH, true>(m.sub[i], block, blocks); break;
    case 2: wh_pass<2, KT, KH, true>(m.sub[i], block, blocks); break;
    case 4: wh_pass<4, KT, KH, true>(m.sub[i], block, blocks); break;
  }
}

// Fills in a launch of `n` passes with tiles of KT x KH; NW16: of the widest.
template <int NW16, int KT, int KH, bool INV>
static hipError_t wh_size(const WhPassArgs* subs, int n, int num_cu, int per_simd, WhLaunch* m, int* lds_out, int* slots_out) {
  constexpr int FIXED = 2 * 16 * wh_row_bytes(KT) + KT * ((NW16 + 1) / 2) * (INV ? 1024 : 2048) + WH_WAVES * 64 * 4;
  static_assert(FIXED + 16 * KH * (128 + 8) * 2 <= 160 * 1024, "LDS of one compute unit");
  *m = WhLaunch{};
  int rows = 0;
  for (int i = 0; i < n; ++i) rows = std::max(rows, subs[i].rows);
  const int lds = FIXED + 16 * KH * (rows + 8) * 2;
  const int per_cu = std::min(per_simd / 2, 160 * 1024 / lds);
  for (int i = 0; i < 3; ++i) {
    m->first[i + 1] = m->first[i];
    if (i >= n) continue;
    WhPassArgs& a = m->sub[i];
    a = subs[i];
    if (a.rows % 16 || a.cols % 16 || (INV && (a.out_rows % 16 || a.out_cols % 16))) return hipErrorInvalidValue;
    a.col_parts = ((a.out_cols + 15) / 16 + KT - 1) / KT;
    a.members = a.col_parts * (((a.out_rows + 15) / 16 + KH - 1) / KH);
    if (!INV && (a.members != a.col_parts || a.out_rows > a.rows || a.out_cols > a.cols)) return hipErrorInvalidValue;
    // a workgroup's sums of squares are of one chunk of channels only if the planes of an XCD are
    if (a.tot_part && 8 % (a.d / 64) != 0) return hipErrorInvalidValue;
    // a lane reaches 8 rows of the output; and 16 positions of the input, which is less (wh_fits and hw_fits ask for the same)
    if (!eight_rows_fit((INV ? 1 : (int64_t)a.T) * a.out_cols * a.d)) return hipErrorInvalidValue;
    const int64_t planes = (int64_t)a.seg_end[2] * a.T * (a.d / 64);
    if (planes <= 0) continue;
    if (planes * a.members > 0x3fffffff) return hipErrorInvalidValue;
    const int64_t per_xcd = (planes + 7) / 8 * a.members;   // items of the fullest XCD
    const int grid = 8 * (int)std::min<int64_t>(per_xcd, std::max(1, num_cu / 8) * per_cu);
    if (slots_out) slots_out[i] = grid * WH_WAVES;
    m->first[i + 1] += grid;   // (a multiple of 8: every pass deals its planes to the XCDs the same way)
  }
  *lds_out = lds;
  return hipSuccess;
}

template <int NW16, int KT, int KH, bool INV>
static hipError_t wh_launch(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out) {
  WhLaunch m;
  int lds;
  hipError_t e = wh_size<NW16, KT, KH, INV>(subs, n, num_cu, wh_waves_per_simd((NW16 + 1) / 2, KT, KH), &m, &lds, slots_out);
  if (e != hipSuccess || m.first[3] == 0) return e;
  static OncePerDevice limit;
  e = allow_lds(limit, (const void*)k_wh_pass<NW16, KT, KH, INV>, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_wh_pass<NW16, KT, KH, INV>), dim3((unsigned)m.first[3]), dim3(64 * WH_WAVES), (size_t)lds, st, m);
  return hipGetLastError();
}

template <int KT, int KH>
static hipError_t hw_mixed_launch(const WhPassArgs* subs, int n, int num_cu, hipStream_t st) {
  WhLaunch m;
  int lds;
  hipError_t e = wh_size<4, KT, KH, true>(subs, n, num_cu, 2, &m, &lds, nullptr);
  if (e != hipSuccess || m.first[3] == 0) return e;
  static OncePerDevice limit;
  e = allow_lds(limit, (const void*)k_hw_mixed<KT, KH>, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_hw_mixed<KT, KH>), dim3((unsigned)m.first[3]), dim3(64 * WH_WAVES), (size_t)lds, st, m);
  return hipGetLastError();
}

// Tiles of output rows and columns (16 each) of a workgroup: as many as the accumulators take, the rows first; rows beyond four
// tiles are cut into equal parts (the inverse only: the forward pass keeps at most 64 rows).
static inline void wh_tiles(const WhPassArgs& a, int* kt, int* kh, int* members) {
  const int tiles = (a.out_rows + 15) / 16, parts = (tiles + 3) / 4, h = (tiles + parts - 1) / parts;
  const int t = h <= 2 && a.out_cols > 16 ? 2 : 1;
  if (kt) *kt = t;
  if (kh) *kh = h;
  if (members) *members = ((a.out_cols + 15) / 16 + t - 1) / t * ((tiles + h - 1) / h);
}

// The passes have input rows of the same width; the tiles are those of the first pass.
template <int NW16, bool INV>
static hipError_t wh_dispatch(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out) {
  int kt, kh;
  wh_tiles(subs[0], &kt, &kh, nullptr);
  for (int i = 0; i < n; ++i)
    if (subs[i].cols != 16 * NW16 || (!INV && subs[i].out_rows > 16 * kh)) return hipErrorInvalidValue;
  // A single W tile: the whole axis of 16, or (forward) the box of any axis.
  if constexpr (!INV || NW16 == 1) {
    if (kt == 1 && kh == 1) return wh_launch<NW16, 1, 1, INV>(subs, n, num_cu, st, slots_out);
    if (kt == 1 && kh == 2) return wh_launch<NW16, 1, 2, INV>(subs, n, num_cu, st, slots_out);
  }
  if constexpr (INV || NW16 > 1) {
    if (kt == 2 && kh == 1) return wh_launch<NW16, 2, 1, INV>(subs, n, num_cu, st, slots_out);
    if (kt == 2 && kh == 2) return wh_launch<NW16, 2, 2, INV>(subs, n, num_cu, st, slots_out);
  }
  if (kh == 3) return wh_launch<NW16, 1, 3, INV>(subs, n, num_cu, st, slots_out);
  if (kh == 4) return wh_launch<NW16, 1, 4, INV>(subs, n, num_cu, st, slots_out);
  return hipErrorInvalidValue;
}

// Two passes, one after the other in every workgroup: the first with tiles of 2 x 2, the second with 1 x KH.
//
// What it saves is the last round of each.  A workgroup holds a compute unit for whole items, and those of a pass seldom come out even:
// 66 tensors of 16 x 64 x 64 x 64 on the low+mid box are 1,056 on 256 workgroups, five rounds for four and an eighth; the whole of
// six more 384 smaller ones, two rounds for one and a half.  The second pass is dealt to the workgroups from the other end, and not to those
// with one item more of the first where that costs it no round: 168 + 42 us apart, 178 together (the forward 580 -> 556).
template <int NW16, int KH>
__global__ void __launch_bounds__(64 * WH_WAVES, 2) k_wh_two(WhLaunch m) {
  const int blocks = m.first[1];
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    int i = pass, tid = threadIdx.x;
    asm volatile("" : "+s"(i), "+v"(tid));   // (what a pass needs is made in it, and not kept for both)
    if (pass == 0) {
      wh_pass<NW16, 2, 2, false>(m.sub[i], (int)blockIdx.x, blocks, tid);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (before the second one writes where others still read)
    } else {
      const int block = ((blocks >> 3) - 1 - (int)(blockIdx.x >> 3)) * 8 + (int)(blockIdx.x & 7);   // (of the same XCD)
      if (block < m.first[2]) wh_pass<NW16, 1, KH, false>(m.sub[i], block, m.first[2], tid);
    }
  }
}

template <int NW16, int KH>
static hipError_t wh_two_launch(const WhPassArgs& a, const WhPassArgs& b, int num_cu, hipStream_t st, int slots_out[2]) {
  WhLaunch ma, mb;
  int lds_a, lds_b;
  hipError_t e = wh_size<NW16, 2, 2, false>(&a, 1, num_cu, 2, &ma, &lds_a, &slots_out[0]);
  if (e == hipSuccess) e = wh_size<NW16, 1, KH, false>(&b, 1, num_cu, 2, &mb, &lds_b, &slots_out[1]);
  if (e != hipSuccess) return e;
  const int blocks = ma.first[3];
  if (blocks == 0 || mb.first[3] != blocks) return hipErrorInvalidValue;   // (wh_two_fits: both fill the chip)
  const int per = blocks / 8;   // workgroups of an XCD
  auto items = [](const WhPassArgs& x) { return (((int64_t)x.seg_end[2] * x.T * (x.d / 64) + 7) / 8) * x.members; };   // (of the fullest)
  const int64_t over = items(ma.sub[0]) % per, n_b = items(mb.sub[0]);
  int blocks_b = blocks;
  if (over > 0 && (n_b + per - over - 1) / (per - over) == (n_b + per - 1) / per) blocks_b = 8 * (int)(per - over);
  slots_out[1] = blocks_b * WH_WAVES;
  ma.sub[1] = mb.sub[0];
  ma.first[2] = blocks_b;   // (here: workgroups of the second pass)
  static OncePerDevice limit;
  e = allow_lds(limit, (const void*)k_wh_two<NW16, KH>, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_wh_two<NW16, KH>), dim3((unsigned)blocks), dim3(64 * WH_WAVES), (size_t)std::max(lds_a, lds_b), st, ma);
  return hipGetLastError();
}

}  // namespace
}  // namespace fa
