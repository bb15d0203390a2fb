// Channel-mixing products around the spectral transform (paper sections 3.1 and 3.7: Q = X W_Q, K = X W_K, V = X W_V,
// concatenated heads times W_O).  The transform acts on the token axes and the projections on the channel axis, so
// they commute: F(X W) = F(X) W.  This file holds the matrix-core kernel those products run on once X itself has been
// transformed:
//
//   C[i][j] = sum over segments s, sum over k < K_s:  A_s[i][k] * B_s[j][k]
//
// with every operand K-contiguous (A_s [m][K_s], row stride lda; B_s [n][K_s], row stride ldb), fp16 in, fp32
// accumulation, fp16 out.  Segments let one product take its K range from several tensors (the output projection sums
// over heads whose rows live in per-head buffers, and picks per head the band output or the passed-through V~).
//
// Tile: 128 rows of C x 128 columns per workgroup of four waves, K in steps of 64.  Both operand tiles are copied from
// global memory straight into LDS (16 bytes per lane, rows of 128 bytes, the 16-byte chunks of a row permuted through
// the source address so that the 16-byte operand reads of 16 consecutive rows hit 16 different bank groups), double
// buffered, one barrier per step.  A wave owns 32 rows and all 128 columns: C^T = B A^T, so that a lane owns one row
// of C and its accumulator registers run over columns - the same register layout as the attention kernel's output.
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "ctx.h"

namespace fa {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ unsigned gemm_lds(const half_t* p) {   // byte address within LDS of a wave-uniform place
  return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(const __attribute__((address_space(3))) half_t*)p);
}
__device__ __forceinline__ void gemm_dma16(const void* src, unsigned base) {
  // one wave-wide copy of 16 bytes per lane into LDS at byte base + 16 * lane (base wave-uniform); issued as assembly so that the
  // compiler does not order every later LDS read behind it - the kernel waits for its copies itself
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ uint32_t gemm_pack_h2(float a, float b) {
  const _Float16 ha = (_Float16)a, hb = (_Float16)b;
  return (uint32_t)__builtin_bit_cast(uint16_t, ha) | ((uint32_t)__builtin_bit_cast(uint16_t, hb) << 16);
}

constexpr int GM = 128, GN = 128, GK = 64;   // tile of C and K step

// A launch runs `per` problems that share m, n and - in the callers here - their A rows (the same spectral rows
// projected with different heads' weights).  Workgroups are dealt to the 8 XCDs round-robin by blockIdx and each XCD has
// its own L2: XCD x takes the row tiles x, x + 8, ... and walks, for each of them, all column tiles of all problems
// back to back, so that a row tile of A is fetched into one L2 once and reused tiles_n * per times.
__global__ void __launch_bounds__(256, 2) k_gemm_nt(const GemmProblem* __restrict__ probs, const GemmSeg* __restrict__ segs,
                                                    int per, int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(16))) half_t As[2][GM * GK];
  __shared__ __attribute__((aligned(16))) half_t Bs[2][GN * GK];
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int inner_n = tiles_n * per;
  const int mt = (seq / inner_n) * 8 + xcd, inner = seq % inner_n;
  if (mt >= tiles_m) return;   // (uniform over the workgroup: the grid is padded to whole rounds of 8 row tiles)
  const GemmProblem pr = probs[inner / tiles_n];
  const int m0 = mt * GM, n0 = (inner % tiles_n) * GN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nn = lane & 31, g = lane >> 5;
  auto fK = [](int r) -> int { return (r >> 1) & 7; };

  // this lane's rows of the copies: instruction i of this wave moves rows (wave*4 + i)*8 + lane/8, chunk lane%8
  const int lr = lane >> 3, lc = lane & 7;
  int a_row[4], b_row[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 8 + lr;
    a_row[i] = m0 + r < pr.m ? m0 + r : pr.m - 1;   // rows past the end repeat the last row; their results are not stored
    b_row[i] = n0 + r < pr.n ? n0 + r : pr.n - 1;
  }
  auto stage = [&](const GemmSeg& sg, int k0, int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (wave * 4 + i) * 8 + lr;
      const int chunk = (lc ^ fK(r)) << 3;
      gemm_dma16(sg.A + (int64_t)a_row[i] * sg.lda + k0 + chunk, gemm_lds(As[buf] + (wave * 4 + i) * 8 * GK));
      gemm_dma16(sg.B + (int64_t)b_row[i] * sg.ldb + k0 + chunk, gemm_lds(Bs[buf] + (wave * 4 + i) * 8 * GK));
    }
  };

  float16v acc[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;

  // flattened (segment, k) iteration; the copy of step i+1 is in flight while step i is multiplied
  int seg_i = 0, k_i = 0;               // position of the step being staged next
  GemmSeg sg = segs[pr.seg0];
  int total_steps = 0;
  for (int s = 0; s < pr.nseg; ++s) total_steps += segs[pr.seg0 + s].K / GK;
  auto advance = [&]() {
    k_i += GK;
    if (k_i >= sg.K) {
      k_i = 0;
      ++seg_i;
      if (seg_i < pr.nseg) sg = segs[pr.seg0 + seg_i];
    }
  };
  if (total_steps > 0) { stage(sg, k_i, 0); advance(); }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int step = 0; step < total_steps; ++step) {
    const int buf = step & 1;
    if (step + 1 < total_steps) { stage(sg, k_i, buf ^ 1); advance(); }
    const half_t* Ab = As[buf] + (32 * wave + nn) * GK;
    const half_t* Bb = Bs[buf] + nn * GK;
#pragma unroll
    for (int ks = 0; ks < GK / 16; ++ks) {
      const int pos = ((2 * ks + g) ^ fK(nn)) << 3;        // fK(32 w + nn) = fK(32 t + nn) = fK(nn)
      const half8 rows = *(const half8*)(Ab + pos);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const half8 cols = *(const half8*)(Bb + nt * 32 * GK + pos);
        acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cols, rows, acc[nt], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }

  // store: lane = row of C, registers = columns; a register swap with the partner lane (lane ^ 32, same row) leaves
  // every lane with 8 consecutive columns, i.e. 16-byte stores
  const int row = m0 + 32 * wave + nn;
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float o[8];   // columns nt*32 + j*16 + g*8 + 0..7
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t lo = __float_as_uint(acc[nt][(2 * j) * 4 + b]);
        const uint32_t hi = __float_as_uint(acc[nt][(2 * j + 1) * 4 + b]);
        const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        o[b] = __uint_as_float(sw[0]);
        o[4 + b] = __uint_as_float(sw[1]);
      }
      const int col = n0 + nt * 32 + j * 16 + g * 8;
      if (row < pr.m && col < pr.n) {   // (n is a multiple of 8)
        uint4v st4;
#pragma unroll
        for (int b = 0; b < 4; ++b) st4[b] = gemm_pack_h2(o[2 * b], o[2 * b + 1]);
        *(uint4v*)(pr.C + (int64_t)row * pr.ldc + col) = st4;
      }
    }
}

// The same product with a 256 x 256 tile per workgroup of eight waves, one workgroup per compute unit, K in steps of 64.
//
// The tiles of A and B of a step are halves of 128 rows, 16 KB each in LDS, two copies of everything (128 KB).  A wave owns 32 rows of
// either half of A and 64 columns of either half of B, and a step is four phases of 8 MFMAs, one per pair of halves, in an order
// in which every phase changes one half only: A0 B0, A0 B1, A1 B1, A1 B0, then (next step) A0 B1, A0 B0, A1 B0, A1 B1.  So half number j
// of the sequence A0 B0 B1 A1 | A0 B1 B0 A1 | A0 B0 .. is, in phase
//   j - 9   copied from memory into the place of half j - 8, which every wave has read in phase j - 10,
//   j - 2   read into registers by every wave, beside the MFMAs of that phase,
//   j - 1 .. j + 2   multiplied.
// A copy has seven phases to arrive, six of them are always in flight (96 KB per compute unit), and no wait in the loop is for the
// latest ones; a phase starts with its operands in registers.
//
// What bounds it: power.  262,144 rows, d_model 2048, 16 heads of 128, Q~ / K~ / V~ products and output product: one step ahead and a wait for all
// of it at every step 1.70 and 2.78 ms (0.97 PFLOP/s, matrix cores busy 53 % of the cycles at 1.9 GHz), this 1.57 and 2.53 (1.07 PFLOP/s, busy
// 63 % at 1.7 GHz); a loop of products alone, busy all the time, is held to 1.93 GHz.  The copies are no limit of the machine: it takes 137
// bytes per ns and compute unit from L2 into LDS or into registers, the loop 35.
//
// The columns of a launch run over all its problems back to back (problem p owns columns [p n, (p + 1) n), n a
// multiple of 32), so that a tile can span several narrow problems - the per-head projections are 64 or 128 columns
// wide.  All problems of a launch must have the same A segments (pointers, strides and K); B and C are the problem's own.
constexpr int WM = 256, WN = 256, WK = 64;
constexpr int HALF = 128 * WK;   // elements of half a tile


// Stores a wave's part of a 256 x 256 tile: 2 x 32 columns from gc_first and from gc_first + gc_step of the launch's, rows row_first and row_first + row_step
// of this lane.  Lane = row of C, registers = columns; a register swap with the partner lane (lane ^ 32, same row) leaves
// every lane with 8 consecutive columns, i.e. 16-byte stores.  Every 32-column tile looks up its own problem.
__device__ __forceinline__ void store_wide(const GemmProblem* __restrict__ probs, const float16v (&acc)[4][2], int n, int n_total, int gc_first,
                                           int gc_step, int row_first, int row_step, int g) {
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const int gc = gc_first + gc_step * (ct >> 1) + 32 * (ct & 1);
    if (gc >= n_total) continue;
    const int pc = gc / n;
    const GemmProblem pr = probs[pc];
    const int col0 = gc - pc * n;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int row = row_first + row_step * rt;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float o[8];   // columns col0 + j*16 + g*8 + 0..7
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const uint32_t lo = __float_as_uint(acc[ct][rt][(2 * j) * 4 + b]);
          const uint32_t hi = __float_as_uint(acc[ct][rt][(2 * j + 1) * 4 + b]);
          const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
          o[b] = __uint_as_float(sw[0]);
          o[4 + b] = __uint_as_float(sw[1]);
        }
        if (row < pr.m) {
          uint4v st4;
#pragma unroll
          for (int b = 0; b < 4; ++b) st4[b] = gemm_pack_h2(o[2 * b], o[2 * b + 1]);
          *(uint4v*)(pr.C + (int64_t)row * pr.ldc + col0 + j * 16 + g * 8) = st4;
        }
      }
    }
  }
}

__global__ void __launch_bounds__(512, 2) k_gemm_nt_wide(const GemmProblem* __restrict__ probs, const GemmSeg* __restrict__ segs,
                                                         int per, int n, int tiles_m, int tiles_n) {
  static_assert(8 * HALF * 2 <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(16))) half_t lds[4][2][HALF];   // [A0, A1, B0, B1][step & 1]
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int mt = (seq / tiles_n) * 8 + xcd;
  if (mt >= tiles_m) return;   // (uniform over the workgroup: the grid is padded to whole rounds of 8 row tiles)
  const int m0 = mt * WM, gc0 = (seq % tiles_n) * WN;   // first row / first column (over all problems) of the tile
  const int n_total = per * n;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nn = lane & 31, g = lane >> 5;
  const int wm = wave & 3, wn = wave >> 2;              // this wave's 32 rows and 64 columns of every half
  // Rows are WK halfs in LDS; the 16-byte chunks of row r are permuted through the source address so that the operand
  // reads of 16 consecutive rows fall on 16 different 16-byte bank groups
  auto fK = [](int r) -> int { return (r >> 1) & 7; };

  // the copies: wave w moves rows [16 w, 16 w + 16) of a half, 8 per instruction
  int lr = lane >> 3, chunk = ((lane & 7) ^ fK(lane >> 3)) << 3;   // this lane's row and (even instructions) its chunk
  int pb[2];   // problem of the wave's rows of B0 and B1 (16 rows are one problem's)
#pragma unroll
  for (int h = 0; h < 2; ++h) pb[h] = min(gc0 + 128 * h + 16 * wave, n_total - 1) / n;
  const int m = probs[pb[0]].m, nseg = probs[pb[0]].nseg;
  const int seg0[2] = {probs[pb[0]].seg0, probs[pb[1]].seg0};
  int seg_i = 0, k_i = 0, total_steps = 0;   // position of the step that is copied next
  for (int s = 0; s < nseg; ++s) total_steps += segs[seg0[0] + s].K / WK;
  GemmSeg sg = segs[seg0[0]];
  const half_t* bp[2] = {sg.B, segs[seg0[1]].B};
  const unsigned copy_at = gemm_lds(lds[0][0] + 16 * wave * WK);
  auto copy = [&](int buf, int which) {   // 0, 1: A0, A1; 2, 3: B0, B1
    const int h = which & 1;
    const bool b = which >= 2;
    const half_t* base = b ? bp[h] + k_i : sg.A + (int64_t)m0 * sg.lda + k_i;   // wave-uniform
    const int last = b ? n_total - 1 - pb[h] * n : m - 1 - m0, first = 128 * h + 16 * wave + (b ? gc0 - pb[h] * n : 0);   // (rows clamped to what exists)
    asm volatile("" : "+v"(lr), "+v"(chunk));   // (addresses formed here: kept for the whole loop they would take the operands' registers)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      gemm_dma16(base + (uint32_t)(min(first + 8 * i + lr, last) * (b ? sg.ldb : sg.lda) + (chunk ^ (i * 32))), copy_at + ((which * 2 + buf) * HALF + 8 * i * WK) * 2);
  };
  auto advance = [&]() {   // (behind the last step: that step again, into places that nobody reads)
    if (k_i + WK < sg.K) {
      k_i += WK;
    } else if (seg_i + 1 < nseg) {
      k_i = 0;
      ++seg_i;
      sg = segs[seg0[0] + seg_i];
      bp[0] = sg.B; bp[1] = segs[seg0[1] + seg_i].B;
    }
  };

  float16v acc[4][2];   // [column tile: half of B, 32 columns][row tile: half of A]
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ct][rt][r] = 0.f;

  constexpr int NKS = WK / 16;
  half8 ra[2][NKS], rb[2][NKS][2];   // operands: halves of A and of B
  const half_t* const a_at = lds[0][0] + (32 * wm + nn) * WK;
  const half_t* const b_at = lds[2][0] + (64 * wn + nn) * WK;
  auto read = [&](int buf, int which) {
    const int h = which & 1;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int pos = ((2 * ks + g) ^ fK(nn)) << 3;        // fK(32 t + nn) = fK(nn)
      if (which < 2) {
        ra[h][ks] = *(const half8*)(a_at + (2 * h + buf) * HALF + pos);
      } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) rb[h][ks][c] = *(const half8*)(b_at + (2 * h + buf) * HALF + c * 32 * WK + pos);
      }
    }
  };
  // One phase: half of A `a`, half of B `b` multiplied; the half `rd` read; the half `cp` copied.
  auto phase = [&](int a, int b, int rd_buf, int rd, int cp_buf, int cp) {
    // The half to be read has landed (this wave's part; with the barrier, everybody's), and everybody has the half that was read last.
    asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    copy(cp_buf, cp);
    read(rd_buf, rd);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        acc[2 * b + c][a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rb[b][ks][c], ra[a][ks], acc[2 * b + c][a], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  if (total_steps > 0) {
    copy(0, 0); copy(0, 2); copy(0, 3); copy(0, 1); advance();   // halves 0 .. 3
    copy(1, 0); copy(1, 3); copy(1, 2); copy(1, 1); advance();   // 4 .. 7
    asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::: "memory");
    read(0, 0); read(0, 2);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    copy(0, 0);                                                   // 8
    for (int step = 0; step < total_steps; step += 2) {
      phase(0, 0, 0, 3, 0, 2);
      phase(0, 1, 0, 1, 0, 3);
      phase(1, 1, 1, 0, 0, 1); advance();
      phase(1, 0, 1, 3, 1, 0);
      if (step + 1 == total_steps) break;
      phase(0, 1, 1, 2, 1, 3);
      phase(0, 0, 1, 1, 1, 2);
      phase(1, 0, 0, 0, 1, 1); advance();
      phase(1, 1, 0, 2, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (copies into this workgroup's LDS)
  }

  store_wide(probs, acc, n, n_total, gc0 + 64 * wn, 128, m0 + 32 * wm + nn, 128, g);
}

// The same for products of few steps of K (the same sums, the same bits): one step copied ahead, a wait for all of it at every step, a wave's 64 rows
// and 128 columns side by side.  Such tiles come and go, and a tile waits longer for its first copies where every compute unit has six halves in flight.
// Forwards of 262,144 tokens, copies seven phases ahead / one step, us: d_model 256 (products of 4 to 7 steps) 1121 / 1094, 384 (6 to 9) 1512 / 1465,
// 512 (8 heads of 64, 8 to 12) 1921 / 1881, 640 (10 to 14) 2227 / 2190, 768 (12 to 18) 2648 / 2640, 1024 (16 to 24) 3682 / 3725; of 16,384 tokens,
// 256 208 / 204, 512 262 / 264, 768 344 / 354.
__global__ void __launch_bounds__(512, 1) k_gemm_nt_wide_few(const GemmProblem* __restrict__ probs, const GemmSeg* __restrict__ segs,
                                                             int per, int n, int tiles_m, int tiles_n) {
  static_assert((WM + WN) * WK * 2 * 2 <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(16))) half_t As[2][WM * WK];
  __shared__ __attribute__((aligned(16))) half_t Bs[2][WN * WK];
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int mt = (seq / tiles_n) * 8 + xcd;
  if (mt >= tiles_m) return;   // (uniform over the workgroup: the grid is padded to whole rounds of 8 row tiles)
  const int m0 = mt * WM, gc0 = (seq % tiles_n) * WN;   // first row / first column (over all problems) of the tile
  const int n_total = per * n;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nn = lane & 31, g = lane >> 5;
  const int wm = wave & 3, wn = wave >> 2;              // this wave's 64 rows and 128 columns of the tile
  // Rows are WK halfs in LDS; the 16-byte chunks of row r are permuted through the source address so that the operand
  // reads of 16 consecutive rows fall on 16 different 16-byte bank groups
  constexpr int CPR = WK / 8;                           // chunks per row
  constexpr int RPI = 64 / CPR;                         // rows per copy instruction (64 lanes x 16 bytes)
  constexpr int IPW = 32 / RPI;                         // copy instructions per wave, step and matrix
  auto fK = [](int r) -> int { return (r >> 1) & 7; };
  const int lr = lane / CPR, lc = lane % CPR;

  // the copies: wave w moves rows [32 w, 32 w + 32) of the A tile and of the B tile
  const int bcol0 = gc0 + 32 * wave;                                    // first B row (= column of C) this wave copies
  const int pb = min(bcol0, n_total - 1) / n;                           // its problem (n % 32 == 0: one problem per wave)
  const GemmProblem prb = probs[pb];
  const int m = prb.m;
  int a_row[IPW], b_row[IPW];   // row within the tile's A rows / within the problem's B rows, clamped to what exists
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r = 32 * wave + RPI * i + lr;
    a_row[i] = min(m0 + r, m - 1) - m0;
    b_row[i] = min(bcol0 + RPI * i + lr, n_total - 1) - pb * n;
  }
  auto stage = [&](const GemmSeg& sg, int k0, int buf) {
    const half_t* abase = sg.A + (int64_t)m0 * sg.lda + k0;   // wave-uniform
    const half_t* bbase = sg.B + k0;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int r = 32 * wave + RPI * i + lr;
      const int chunk = (lc ^ fK(r)) << 3;
      gemm_dma16(abase + (uint32_t)(a_row[i] * sg.lda + chunk), gemm_lds(As[buf] + (32 * wave + RPI * i) * WK));
      gemm_dma16(bbase + (uint32_t)(b_row[i] * sg.ldb + chunk), gemm_lds(Bs[buf] + (32 * wave + RPI * i) * WK));
    }
  };

  float16v acc[4][2];   // [column tile][row tile]
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ct][rt][r] = 0.f;

  int seg_i = 0, k_i = 0;   // position of the step that is copied next
  GemmSeg sg = segs[prb.seg0];
  int total_steps = 0;
  for (int s2 = 0; s2 < prb.nseg; ++s2) total_steps += segs[prb.seg0 + s2].K / WK;
  auto advance = [&]() {
    k_i += WK;
    if (k_i >= sg.K) {
      k_i = 0;
      ++seg_i;
      if (seg_i < prb.nseg) sg = segs[prb.seg0 + seg_i];
    }
  };
  if (total_steps > 0) { stage(sg, k_i, 0); advance(); }
  for (int step = 0; step < total_steps; ++step) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of step `step` has landed
    __syncthreads();   // step `step` is in LDS for every wave, and nobody reads the buffer of step - 1 any more
    if (step + 1 < total_steps) { stage(sg, k_i, (step + 1) & 1); advance(); }
    const int buf = step & 1;
    const half_t* Ab = As[buf] + (64 * wm + nn) * WK;
    const half_t* Bb = Bs[buf] + (128 * wn + nn) * WK;
    constexpr int NKS = WK / 16;
    half8 rows[2][2], cols[2][4];
    auto operands = [&](int ks, int set) {
      const int pos = ((2 * ks + g) ^ fK(nn)) << 3;        // fK(32 t + nn) = fK(nn)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) rows[set][rt] = *(const half8*)(Ab + rt * 32 * WK + pos);
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) cols[set][ct] = *(const half8*)(Bb + ct * 32 * WK + pos);
    };
    operands(0, 0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if (ks + 1 < NKS) operands(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          acc[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cols[ks & 1][ct], rows[ks & 1][rt], acc[ct][rt], 0, 0, 0);
    }
  }

  store_wide(probs, acc, n, n_total, gc0 + 128 * wn, 64, m0 + 64 * wm + nn, 32, g);
}

// out[c][r] = (fp16) in[r][c] for a bf16 matrix [R][Cc]: the weights arrive [k][n] (n contiguous) and the product wants
// them K-contiguous.  32 x 32 tiles through LDS.
__global__ void __launch_bounds__(256) k_transpose_bf16_to_f16(const uint16_t* __restrict__ in, half_t* __restrict__ out, int R, int Cc) {
  __shared__ half_t tile[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int i = ty; i < 32; i += 8) {
    const int r = r0 + i, c = c0 + tx;
    float v = 0.f;
    if (r < R && c < Cc) v = __uint_as_float((uint32_t)in[(int64_t)r * Cc + c] << 16);
    tile[i][tx] = (half_t)v;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int c = c0 + i, r = r0 + tx;
    if (r < R && c < Cc) out[(int64_t)c * R + r] = tile[tx][i];
  }
}

}  // namespace

// `per` problems d_probs[0 .. per) of identical m and n (host-checked by the caller).
// `steps`: steps of 64 of the sum over all segments; `call_steps`: of d_model, which nearly all of a call's work has at least.
// Below 12 steps a product copies one step ahead (k_gemm_nt_wide_few has both sides), and in calls of a d_model below 14 steps so do the large launches,
// of four rounds of the chip and more, whatever their own steps: the seven phases gain nothing there on any machine and lose up to 4 % on some,
// and products of both kinds in one call are no better.  12 heads of 64, 262,144 tokens, forwards with one step / seven phases / by 12 steps of
// the product, us, on four machines: d_model 576 1912 / 1987 / 1973, 1947 / - / 1998, 1992 / 2020 / 2014, 2031 / - / 2025; 704 2142 / 2207 / 2209, 2170 / - / 2242,
// 2200 / 2250 / 2265, 2255 / - / 2275; 768 2291 / 2338 / 2335, 2303 / - / 2358, 2351 / 2393 / 2396, 2410 / - / 2409; 14 heads, 896 2793 / - / 2831,
// 2835 / 2859 / 2869, 2913 / - / 2884; 16 heads, 1024 3323 / - / 3347, 3399 / 3394 / 3410, 3490 / - / 3432.  Of 16,384 tokens, where launches are a
// round and less: 704 333 / 322 / 326, 768 345 / 332 / 334.
hipError_t launch_gemm_nt(const GemmProblem* d_probs, const GemmSeg* d_segs, int per, int m, int n, int steps, int call_steps, int num_cu, hipStream_t st) {
  if (per <= 0 || m <= 0 || n <= 0) return hipSuccess;
  static int wide = -1;
  if (wide < 0) { const char* e = getenv("FREQATTN_GEMM_WIDE"); wide = e ? atoi(e) : 1; }
  if (wide && n % 32 == 0 && m >= WM && (int64_t)per * n >= WN) {
    // (the callers' launches share their A segments between problems, which the wide kernel relies on)
    const int tiles_m = (m + WM - 1) / WM, tiles_n = (int)(((int64_t)per * n + WN - 1) / WN);
    const int64_t blocks = (int64_t)((tiles_m + 7) / 8) * 8 * tiles_n;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const bool few = steps < 12 || (call_steps < 14 && blocks >= 4 * (int64_t)num_cu);
    hipLaunchKernelGGL(few ? k_gemm_nt_wide_few : k_gemm_nt_wide, dim3((unsigned)blocks), dim3(512), 0, st, d_probs, d_segs, per, n, tiles_m, tiles_n);
    return hipGetLastError();
  }
  const int tiles_m = (m + GM - 1) / GM, tiles_n = (n + GN - 1) / GN;
  const int64_t blocks = (int64_t)((tiles_m + 7) / 8) * 8 * tiles_n * per;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gemm_nt, dim3((unsigned)blocks), dim3(256), 0, st, d_probs, d_segs, per, tiles_m, tiles_n);
  return hipGetLastError();
}

hipError_t launch_transpose_bf16_to_f16(const void* in, void* out, int R, int Cc, hipStream_t st) {
  if (R <= 0 || Cc <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_transpose_bf16_to_f16, dim3((unsigned)((Cc + 31) / 32), (unsigned)((R + 31) / 32)), dim3(256), 0, st,
                     (const uint16_t*)in, (half_t*)out, R, Cc);
  return hipGetLastError();
}

}  // namespace fa
