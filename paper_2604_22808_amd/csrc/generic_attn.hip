// Attention of the generic fp32 path (sections 3.4.1-3.4.3, 3.6): any head_dim up to 256, any block size, any window, fp32
// operands and accumulation throughout, on the fp32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// One launch serves up to four branches (segments) of a forward.  A workgroup owns 16 or 32 query rows of one slice; its
// four waves take the key tiles (16 keys) of those rows in turn and their partial results meet in LDS at the end, so
// that a small problem still puts four waves on every query tile.  Per key tile and wave, scores are kept transposed
// (S^T = K Q^T: lane = query, registers = keys 4 g + r of a 16-key group, g = lane / 16), which makes the probabilities the B
// operand of O^T += V^T P^T as they stand.  Operands come straight from global memory: a lane reads 16 bytes of its own key
// row (K; the four channels feed four MFMA steps, the channel order of a contraction being free) and DC adjacent
// channels of four value rows per 16-lane group (V; channel n DC + dc belongs to output tile dc), i.e. whole row segments
// of 64 to 512 bytes, and no LDS traffic or barrier is left in the key loop.
//
// What bounds it: at small sizes, where it is used, the latency of a wave's few dependent tiles - leaving out the loads or the
// products of either half changes less than a quarter of the time.  Band operators and exchange together, 12,150 tokens
// x 4 heads x 64 in fp32 (window +-128, 16-row blocks): 59 us with tiles of 32 keys, expf, a mask on every score and a division per
// key of a block list, 39 us now (tiles of 16 keys leave registers for another wave per SIMD; masks on edge tiles only); 6,160
// tokens x 6 heads x 128 with several bands per head: 109 -> 72 us.  Key rows loaded whole and turned into operands in LDS measured
// the same, and 16 query rows per workgroup at 12,150 tokens 42 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.h"

namespace fa {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));

// channels ch .. ch + 3 of a row; with !EXACT only those below d exist (and rows need not be 16-byte aligned)
template <bool EXACT>
__device__ __forceinline__ float4v row4(const float* row, int ch, int d) {
  if (EXACT) return *(const float4v*)(row + ch);
  float4v v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = ch + i < d ? row[ch + i] : 0.f;
  return v;
}

// XCHG: some segments have summary tokens to attend to as well.
template <int DC, int NQ, bool EXACT, bool XCHG>
__device__ __forceinline__ void gattn_body(const GAttnSeg& s, int d, float scale, int tile, int sl, float* lds) {
  constexpr int ROWS = 16 * NQ, DP = 16 * DC, LROW = DP + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int slice = s.slice_list ? s.slice_list[sl] : sl;
  const float* Q = s.Q + (int64_t)slice * s.slice_stride;
  const float* K = s.K + (int64_t)slice * s.kv_slice_stride;
  const float* V = s.V + (int64_t)slice * s.kv_slice_stride;
  float* O = s.O + (int64_t)slice * s.o_slice_stride;

  // With C the rows attend to the other bands' summary tokens as well (section 3.6), in a second phase with the first one's result as
  // the query and the residual.
  const int n_phases = XCHG && s.C ? 2 : 1;
  int mode = s.mode, nk = s.nk;

  // query rows [q0, qend), keys j = 0 .. nkeys - 1 of the rows' own numbering
  int q0, qend, e0 = 0, k0 = 0, nkeys;
  if (s.mode == 1) {
    const int tpb = (s.block + ROWS - 1) / ROWS, I = tile / tpb;
    q0 = I * s.block + (tile - I * tpb) * ROWS;
    qend = min(min(q0 + ROWS, (I + 1) * s.block), s.nq);
    if (q0 >= qend) return;   // (uniform over the workgroup)
    e0 = s.row_ptr[I];
    const int e1 = s.row_ptr[I + 1];   // (columns ascend: only the last block of the list can be the band's short one)
    nkeys = e1 > e0 ? (e1 - 1 - e0) * s.block + min(s.block, s.nk - s.col_idx[e1 - 1] * s.block) : 0;
  } else {
    q0 = tile * ROWS;
    qend = min(q0 + ROWS, s.nq);
    if (q0 >= qend) return;
    nkeys = s.nk;
    if (s.mode == 2) {
      k0 = max(q0 - s.window, 0);
      nkeys = (int)min((int64_t)s.nk, (int64_t)qend + s.window) - k0;
    }
  }
  // key row of list position j: the identity plus k0, or through the block list
  auto key_of = [&](int j) -> int {
    if (mode != 1) return k0 + j;
    const int jj = min(j, nkeys - 1), b = jj / s.block;
    return s.col_idx[e0 + b] * s.block + (jj - b * s.block);
  };

  float4v Qr[NQ][DC];
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const float* row = Q + (int64_t)min(q0 + 16 * u + n, qend - 1) * d;
#pragma unroll
    for (int c = 0; c < DC; ++c) Qr[u][c] = row4<EXACT>(row, 16 * c + 4 * g, d);
  }
  for (int phase = 0;; ++phase) {
  float4v acc[NQ][DC];
  const float scale2 = scale * 1.44269504088896341f;
  float m_run[NQ], l_run[NQ];   // maximum over the tiles of this wave (an exponent of two); sum of this lane's keys only
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    m_run[u] = -INFINITY; l_run[u] = 0.f;
#pragma unroll
    for (int c = 0; c < DC; ++c) acc[u][c] = float4v{0.f, 0.f, 0.f, 0.f};
  }

  // A tile of 16 keys per wave and step, the four waves' tiles side by side.  Its rows follow one another, from a row that all
  // lanes share, unless the blocks of a list are no multiples of 16.
  constexpr int TK = 16, STEP = 4 * TK;
  const bool scattered = mode == 1 && s.block % TK != 0;
  // first key row of the tile at list position jt (for tiles whose rows follow one another)
  auto base_of = [&](int jt) -> int {
    if (mode != 1) return k0 + jt;
    const int b = jt / s.block;
    return s.col_idx[e0 + b] * s.block + (jt - b * s.block);
  };
  float4v Kr[DC];
  int kb = 0;   // (tile whose keys are in Kr)
  auto load_k = [&](int jt) {
    const float* row;
    if (scattered) {
      row = K + (int64_t)min(key_of(jt + n), nk - 1) * d;
    } else {
      kb = base_of(jt);
      row = K + (int64_t)kb * d + min(n, nk - 1 - kb) * d;
    }
#pragma unroll
    for (int c = 0; c < DC; ++c) Kr[c] = row4<EXACT>(row, 16 * c + 4 * g, d);
  };
  if (TK * wave < nkeys) load_k(TK * wave);
  for (int jt = TK * wave; jt < nkeys; jt += STEP) {
    // value rows of this lane's four keys: requested first, used after the softmax
    float Vr[4][DC];
    int key[4];
    const int kt = kb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      key[r] = scattered ? key_of(jt + 4 * g + r) : kt + 4 * g + r;
      const float* row = scattered ? V + (int64_t)min(key[r], nk - 1) * d : V + (int64_t)kt * d + min(4 * g + r, nk - 1 - kt) * d;
      if (EXACT && DC % 4 == 0) {
#pragma unroll
        for (int c = 0; c < DC; c += 4) *(float4v*)&Vr[r][c] = *(const float4v*)(row + n * DC + c);
      } else {
#pragma unroll
        for (int c = 0; c < DC; ++c) Vr[r][c] = (EXACT || n * DC + c < d) ? row[n * DC + c] : 0.f;
      }
    }
    float4v S[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) S[u] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < DC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < NQ; ++u)
          S[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(Kr[c][r], Qr[u][c][r], S[u], 0, 0, 0);
    if (jt + STEP < nkeys) load_k(jt + STEP);
    // (tiles inside the list and inside every row's window need no masks)
    const bool inside = jt + TK <= nkeys && !scattered && kt + TK <= nk &&
                        (mode != 2 || (kt + s.window >= qend - 1 && kt + TK - 1 - s.window <= q0));
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
      const int q = q0 + 16 * u + n;
      if (!inside)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          bool ok = jt + 4 * g + r < nkeys && key[r] < nk;
          if (mode == 2) ok = ok && key[r] >= q - s.window && key[r] - s.window <= q;
          S[u][r] = ok ? S[u][r] : -INFINITY;
        }
      // Scores times scale2 are exponents of two; the product and the difference to the running maximum are one rounding.
      float mx = fmaxf(fmaxf(S[u][0], S[u][1]), fmaxf(S[u][2], S[u][3]));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(m_run[u], fmaxf(mx, __shfl_xor(mx, 32)) * scale2);
      const float ref = mx == -INFINITY ? 0.f : mx;   // (no valid key for this query yet: every probability below is 0)
      const float alpha = __builtin_amdgcn_exp2f(m_run[u] - ref);
#pragma unroll
      for (int r = 0; r < 4; ++r) S[u][r] = __builtin_amdgcn_exp2f(fmaf(S[u][r], scale2, -ref));
      l_run[u] = l_run[u] * alpha + ((S[u][0] + S[u][1]) + (S[u][2] + S[u][3]));
      m_run[u] = mx;
#pragma unroll
      for (int c = 0; c < DC; ++c) acc[u][c] *= alpha;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < DC; ++c)
#pragma unroll
        for (int u = 0; u < NQ; ++u)
          acc[u][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(Vr[r][c], S[u][r], acc[u][c], 0, 0, 0);
  }

  // the four waves' results -> LDS (lane: query n, channels (4 g + r) DC + c), then every thread combines 4 channels
  float* ml = lds + 4 * ROWS * LROW;   // [wave][row][2]: maximum, sum
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    float l = l_run[u];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const int row = wave * ROWS + 16 * u + n;
    if (g == 0) { ml[row * 2] = m_run[u]; ml[row * 2 + 1] = l; }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < DC; ++c) lds[row * LROW + (4 * g + r) * DC + c] = acc[u][c][r];
  }
  __syncthreads();
  const bool last = !XCHG || phase + 1 == n_phases;
  for (int e = tid; e < ROWS * (DP / 4); e += 256) {
    const int row = e / (DP / 4), ch = (e % (DP / 4)) * 4;
    if (q0 + row >= qend || ch >= d) continue;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) m = fmaxf(m, ml[(w * ROWS + row) * 2]);
    float l = 0.f;
    float4v o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml[(w * ROWS + row) * 2] - m);
      l += f * ml[(w * ROWS + row) * 2 + 1];
      o += f * *(const float4v*)(lds + (w * ROWS + row) * LROW + ch);
    }
    o *= 1.f / l;
    const int64_t q = q0 + row;
    if (s.residual) o += row4<EXACT>(Q + q * d, ch, d);
    if (XCHG && phase > 0) o += row4<EXACT>(O + q * s.rep * d, ch, d);   // (the first phase's result, stored by this thread)
    if (!last) *(float4v*)(lds + row * LROW + ch) = o;           // (where only this thread has read: the second phase's queries)
    for (int64_t r = q * s.rep; r < min(q * s.rep + (last ? s.fill : 1), (int64_t)s.n_out); ++r) {
      float* dst = O + r * d + ch;
      if (EXACT) {
        *(float4v*)dst = o;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (ch + j < d) dst[j] = o[j];
      }
    }
  }
  if (!XCHG || last) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NQ; ++u) {
    const float* row = lds + min(16 * u + n, qend - 1 - q0) * LROW;
#pragma unroll
    for (int c = 0; c < DC; ++c) Qr[u][c] = row4<EXACT>(row, 16 * c + 4 * g, d);
  }
  __syncthreads();   // (before the results of the second phase take the place)
  mode = 0; k0 = 0; nk = nkeys = s.nc;
  K = V = s.C + (int64_t)slice * s.c_slice_stride;
  }
}

template <int DC, bool EXACT, bool XCHG>
__global__ void __launch_bounds__(256, DC <= 4 ? 3 : DC <= 8 ? 2 : 1) k_gattn(GAttnArgs a) {
  constexpr int NQMAX = DC <= 8 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float lds[4 * 16 * NQMAX * (16 * DC + 4) + 4 * 16 * NQMAX * 2];
  int k = 0;
  while (k + 1 < a.nseg && (int)blockIdx.x >= a.seg[k + 1].first_block) ++k;
  const GAttnSeg& s = a.seg[k];
  const int b = blockIdx.x - s.first_block, sl = b / s.tiles, tile = b - sl * s.tiles;
  if (NQMAX == 2 && s.rows == 32) gattn_body<DC, NQMAX, EXACT, XCHG>(s, a.d, a.scale, tile, sl, lds);
  else gattn_body<DC, 1, EXACT, XCHG>(s, a.d, a.scale, tile, sl, lds);
}

// (Variants without the second phase: its loop costs the first one registers, and launches that have none up to 3 %.)
template <int DC>
hipError_t launch_dc(const GAttnArgs& a, int blocks, hipStream_t st) {
  bool xchg = false;
  for (int i = 0; i < a.nseg; ++i) xchg = xchg || a.seg[i].C;
  const bool exact = a.d == 16 * DC;
  void (*const k)(GAttnArgs) = exact ? (xchg ? k_gattn<DC, true, true> : k_gattn<DC, true, false>)
                                     : (xchg ? k_gattn<DC, false, true> : k_gattn<DC, false, false>);
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_generic_attn(GAttnArgs a, int num_cu, hipStream_t st, int first, int count) {
  // Query rows per workgroup.  32 rows load every key and value once for twice the queries, but a block list with at most
  // 16 rows per query block would leave half of them empty, and a launch that does not fill the compute units twice over
  // gains more from twice the workgroups.  (head_dim > 128: the registers hold 16 rows only.)
  int64_t blocks32 = 0;
  int n = 0;
  for (int i = 0; i < a.nseg; ++i) {
    if (a.seg[i].nq <= 0 || a.seg[i].nk <= 0 || a.seg[i].n_slices <= 0) continue;
    blocks32 += (int64_t)((a.seg[i].nq + 31) / 32) * a.seg[i].n_slices;
    if (i >= first && i < first + count) a.seg[n++] = a.seg[i];
  }
  a.nseg = n;
  if (n == 0) return hipSuccess;
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) {
    GAttnSeg& s = a.seg[i];
    if (s.mode == 1) s.block = std::min(s.block, s.nq);   // (one block longer than the band is one block of the band's length)
    s.rows = (a.d > 128 || (s.mode == 1 && s.block <= 16) || blocks32 < 2 * num_cu) ? 16 : 32;
    int64_t tiles = ((int64_t)s.nq + s.rows - 1) / s.rows;
    if (s.mode == 1) tiles = (((int64_t)s.nq + s.block - 1) / s.block) * ((s.block + s.rows - 1) / s.rows);
    if (tiles * s.n_slices + blocks > 0x7fffffff) return hipErrorInvalidValue;
    s.tiles = (int)tiles;
    s.first_block = (int)blocks;
    blocks += tiles * s.n_slices;
  }
  if (a.d <= 32) return launch_dc<2>(a, (int)blocks, st);
  if (a.d <= 64) return launch_dc<4>(a, (int)blocks, st);
  if (a.d <= 128) return launch_dc<8>(a, (int)blocks, st);
  return launch_dc<16>(a, (int)blocks, st);
}

}  // namespace fa
