// Internal definitions shared by the host side and the kernel launchers of libfreqattn.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "freqattn.h"
#include "per_device.h"

namespace fa {

typedef _Float16 half_t;

enum { LOW = 0, MID = 1, HIGH = 2, MID2 = 3 };   // MID2: the second block-sparse band of a four-band layout (its rows follow the high band's)
enum { NBMAX = 4 };

// Work item of the attention kernels: a tile of query rows of one branch of one (batch*heads) slice.
// kind: 0 low (compressed tokens), 1 mid (block list), 2 high (window), 3 exchange on band `band`, 4 dense baseline.
struct AttnItem {
  int32_t kind_band;  // kind | band << 8
  int32_t slice;      // batch*heads index
  int32_t q0;         // first query row of the tile, in band order
  int32_t cost;       // key tiles the item visits (used for ordering only)
};

// Everything the attention kernels need besides the item list (device pointers into context-owned memory).
struct AttnParams {
  const void* specQ;  // [slices][N][d] band-major, band l starts at row band_off[l]
  const void* specK;
  const void* specV;
  void* Y;            // [slices][N][d] band-major band outputs
  const void* lowQ;   // [slices][nbar][d] compressed low band
  const void* lowK;
  const void* lowV;
  const void* C;      // [slices][nb][(nb-1) m][d] summary tokens seen by band l
  const int32_t* mid_row_ptr;
  const int32_t* mid_col_idx;
  const int32_t* mid2_row_ptr;   // block list of band MID2
  const int32_t* mid2_col_idx;
  int32_t band_off[NBMAX];
  int32_t band_n[NBMAX];
  int32_t n_c[NBMAX]; // valid rows of C per band
  int32_t nb;         // bands: 3 or 4
  int32_t low_c;      // compression factor c: group i's output belongs to low-band rows i c .. i c + c - 1
  int32_t low_fill;   // rows of a group the band operator writes itself: c, or 1 when launch_expand_low fills the rest
  int32_t N, d, nbar, m2;  // m2 = (nb-1) m = rows reserved per band in C
  int32_t mid_block, high_window;   // (high_window at most band_n[HIGH])
  float scale;
  // dense baseline
  const void* denseQ; const void* denseK; const void* denseV; void* denseO;   // fp16
};

// Matrix products of the projected forward (mfma_gemm.hip): C[i][j] = sum_s sum_k A_s[i][k] B_s[j][k], fp16, K-contiguous.
struct GemmSeg { const half_t* A; const half_t* B; int32_t lda, ldb, K, pad; };
struct GemmProblem { half_t* C; int32_t ldc, m, n, seg0, nseg, pad; };

struct Ctx {
  freqattn_shape shape;
  freqattn_band_cfg cfg;
  int path;         // resolved freqattn_path
  int launch_mode;
  int exchange_fusion = 1;   // band items of single-band slices carry the exchange (section 3.6) themselves
  int slices;       // batch*heads
  int64_t N;
  int d;
  int nb = 3;       // bands: 3, or 4 with cfg.mid2_num > 0
  int64_t band_n[NBMAX] = {0, 0, 0, 0}, band_off[NBMAX] = {0, 0, 0, 0};
  int64_t nbar, nb_mid, nb_mid2 = 0;
  int m_eff[NBMAX] = {0, 0, 0, 0}, n_c[NBMAX] = {0, 0, 0, 0};
  std::string err;

  // host tables
  std::vector<int32_t> h_band_index[NBMAX];
  std::vector<int32_t> h_perm;       // flat coefficient index -> band-major row
  std::vector<int32_t> h_row_ptr, h_col_idx;
  std::vector<int32_t> h_row_ptr2, h_col_idx2;   // block list of band MID2
  std::vector<double> h_F[3];        // per-axis DCT matrices as rounded for the device, [n][n]
  std::vector<int32_t> h_alloc;      // last head_alloc seen (size heads), empty before the first forward
  bool alloc_valid = false;

  // device tables
  int32_t* d_perm = nullptr;
  int32_t* d_perm_t = nullptr;   // the same map stored [kh*W + kw][kt]: the 64..128 rows a T-axis tile looks up are adjacent (MFMA path)
  int32_t* d_row_ptr = nullptr;
  int32_t* d_col_idx = nullptr;
  int32_t* d_row_ptr2 = nullptr;
  int32_t* d_col_idx2 = nullptr;
  float* d_F32[3] = {nullptr, nullptr, nullptr};    // F fp32 (generic path), rows and columns padded to multiples of 16 with zeros
  float* d_Ft32[3] = {nullptr, nullptr, nullptr};   // F^T
  half_t* d_F16[3] = {nullptr, nullptr, nullptr};   // F  fp16 (MFMA path)
  half_t* d_Ft16[3] = {nullptr, nullptr, nullptr};  // F^T fp16

  // device scratch (element type float on the generic path, fp16 on the MFMA path)
  void* specQ = nullptr; void* specK = nullptr; void* specV = nullptr; void* Y = nullptr;
  void* tmp0 = nullptr; void* tmp1 = nullptr;     // transform ping-pong, 3*slices*N*d
  void* lowQ = nullptr; void* lowK = nullptr; void* lowV = nullptr;
  void* Cbuf = nullptr;
  int32_t* d_range_flag = nullptr;                // set by the scattering transform passes when a coefficient leaves the fp16 range (sticky)
  float* d_stats = nullptr;                       // router statistics [3][d] (+ partial sums of the generic kernel)
  float* d_energy_part = nullptr;                 // per-wave partial sums of the fused statistics (MFMA path)
  float* d_tot_part = nullptr;                    // per-wave partial sums of the inputs' squares (Q, K), MFMA path
  int tot_waves[3] = {0, 0, 0};                   // waves that stored sums of squares in the last W-axis pass, per statistics slot
  bool keep_outputs = false;                      // transforms leave Y alone (routing without a forward: the last forward's Y^ stays readable)
  bool qk_on_mid_box = false;                     // the last routed transforms left Q~, K~ on the low+mid box only
  bool qk_boxed = false;                          // generic path: the last transforms made Q~, K~ on the box of a slice's bands only
  int energy_waves[6] = {0, 0, 0, 0, 0, 0};       // waves that stored band statistics in the last T-axis pass, per statistics slot
  int low_box[3] = {0, 0, 0}, mid_box[3] = {0, 0, 0};  // extent of the low / low+mid box per axis
  float* h_stats = nullptr;                       // pinned mirror and the range flag behind it
  float* h_stats_dev = nullptr;                   // the same where the device writes it (MFMA path)

  // per-forward lists (device + pinned host mirror)
  int32_t* d_lists = nullptr; int32_t* h_lists = nullptr; size_t lists_bytes = 0;
  // layout inside lists (int32 units)
  size_t off_masks = 0;               // [slices] band mask per slice
  size_t off_list[NBMAX] = {0, 0, 0, 0};     // [slices] slices with band l active
  int n_list[NBMAX] = {0, 0, 0, 0};
  size_t off_cls[4] = {0, 0, 0, 0};   // [slices] slices by class: 0 low only, 1 mid (no high, no second mid band), 2 high or second mid band, 3 nothing active
  int n_cls[4] = {0, 0, 0, 0};
  size_t off_nonhigh = 0;             // [slices] classes 0, 1 and 3 together (every slice that does not run the high band)
  int n_nonhigh = 0;
  size_t off_fix = 0;                 // [slices] routed forward: slices whose Q~/K~ have to be completed after routing
  int predict_alloc = 1;              // routed forward: transform Q/K of the last allocation's high slices in full at once
  std::vector<char> qk_full;          // routed forward: slices whose Q~/K~ (and V~) the first phase computed on the whole grid
  // V~ on the low+mid box only for slices that do not run the high band (MFMA path): their high-band summary tokens
  // come from the untransformed V through the weights d_wsum (mfma_vsum.hip)
  bool v_box_ok = false;              // the context can do it: summary weights built, or no summaries configured
  uint16_t* d_wsum = nullptr;         // bf16 [N/64][64][64]
  float* d_vsum_part = nullptr;       // [slices][vsum_parts][d][64] partial sums
  int vsum_nsplit = 0;
  std::vector<char> v_full;           // per slice: the current forward computed V~ on the whole grid
  size_t off_items = 0;               // AttnItem array (fused order: all branches), then exchange items
  int n_items_branch = 0;             // low+mid+high items in cost order
  int n_items_kind[3] = {0, 0, 0};    // per-branch sub-lists follow at off_items_kind
  size_t off_items_kind[3] = {0, 0, 0};
  size_t off_items_xchg = 0; int n_items_xchg = 0;
  size_t off_items_dense = 0; int n_items_dense = 0;
  size_t cap_items_kind = 0, cap_items_xchg = 0;   // AttnItem capacity of each branch / fused region and of the exchange / dense regions
  int attn_rows = 0;                  // query rows per attention item on the MFMA path
  int num_cu = 256;

  // stage timing
  bool timing = false;
  static const int MAX_STAGES = 16;
  static const int MAX_TIMED = 64;                // forwards whose events are kept (ring)
  hipEvent_t ev[MAX_TIMED][MAX_STAGES + 1];
  const char* stage_name[MAX_STAGES];
  int n_stages = 0;                               // stages of the last timed forward
  int64_t timed_steps = 0;                        // timed forwards since timing was switched on
  bool ev_created = false;

  // Projected forward (freqattn_forward_projected): buffers allocated at its first call for a model width
  int proj_d_model = 0;
  void* projX = nullptr; void* projZ = nullptr;           // X~ and the projected spectral output, [batch][N][d_model] fp16, band-major rows
  half_t* projWq = nullptr; half_t* projWk = nullptr; half_t* projWv = nullptr;   // [heads*d][d_model]: W^T, K-contiguous
  half_t* projWo = nullptr;                               // [d_model][heads*d]: W_O^T
  // Pass-through folding: on a band a head does not run, its V~ only feeds the output projection and the summary
  // tokens; both are taken from X~ directly (X~ (W_V,h W_O,h) summed over the passing heads; pooled X~ times W_V,h)
  bool proj_fold = false;                                 // this call's tables use the folding (decided per call)
  half_t* projWvN = nullptr;                              // [d_model][heads*d]: W_V as given, fp16
  half_t* projM = nullptr;                                // [3][d_model][d_model]: (sum over passing heads of W_V,h W_O,h)^T per band
  half_t* projPool = nullptr;                             // [batch][3][m][d_model]: chunk means of X~
  half_t* projCtmp = nullptr;                             // [slices][3][m][d]: the same projected with every head's W_V
  int32_t* proj_ones = nullptr;                           // [batch] band masks "every band from the first source" of the wide inverse
  GemmProblem* d_gemm_prob = nullptr; GemmProblem* h_gemm_prob = nullptr;   // device table + pinned mirror
  GemmSeg* d_gemm_seg = nullptr; GemmSeg* h_gemm_seg = nullptr;
  int gemm_cap_prob = 0, gemm_cap_seg = 0;
  struct GemmGroup { int first, per, m, n, steps, stage; };   // one launch: problems [first, first + per) of equal m, n and A rows; steps of 64 along K
  std::vector<GemmGroup> gemm_groups;                     // stage 0: Q~/K~ and V~ projections, stage 1: output projection
  bool gemm_tables_valid = false;                         // built for the current allocation (h_alloc)

  int64_t dev_bytes = 0;
  uint64_t uid = 0;                 // distinct for every context of the process
  // A context whose device memory is carved out of a caller-provided arena instead of hipMalloc (static scratch)
  char* arena_base = nullptr; size_t arena_cap = 0, arena_need = 0;
};

// ---- host tables (tables.cpp) --------------------------------------------------------------------------------
void build_dct_matrix(int n, std::vector<double>& F);  // [n][n], row = frequency
void build_haar_matrix(int n, std::vector<double>& F); // [n][n], row = scale (coarse to fine), n a power of two
void build_bands(Ctx& c);
void build_mid_blocks(Ctx& c);   // both block-sparse bands
void build_summary_weights(const Ctx& c, int band, std::vector<float>& out);   // [m_eff[band]][N]
void pack_vsum_weights(const std::vector<float>& w, int m, int64_t N, std::vector<uint16_t>& out);  // bf16 [N/64][64][64], see mfma_vsum.hip

// ---- generic fp32 kernels (generic_kernels.hip) -----------------------------------------------------------------
// The box of coefficients a slice's bands live in, by its band mask (T, H, W): the first n tensors of a launch (Q and K) are only made there.
struct AxisBoxes { const int32_t* masks; int n; int low[3], mid[3], full[3]; };
struct AxisPassArgs {      // (generic_axis.hip)
  const void* in[3]; void* out[3]; int n_tensors;   // Q, K, V go through one launch
  const float* M;           // [ldm][ldm], zero outside [n_out][n]: out[k] = sum_j M[k][j] in[j]
  int n, n_out, ldm;        // ldm a multiple of 16, >= n and n_out
  int64_t inner, outer;     // element index ((s*n + j)*inner + i), s in [0, nslab), slab s belongs to slice s/outer
  int64_t nslab;
  const int32_t* perm_in;   // when set (axis W only, inner == d): input row of token (s%outer)*n + j is perm[token]
  const int32_t* perm_out;  // same for output rows
  int64_t Ntok;
  int d;
  // input source selection per band for the first inverse pass (perm_in set): rows of band l of slice hb come from
  // `in` when bit l of masks[hb] is set, else from `in_alt`.
  const void* in_alt; const int32_t* masks; int32_t band_off1, band_off2, band_off3;   // first rows of bands 1, 2, 3 (band_off3 = Ntok without a fourth band)
  int in_bf16, out_bf16;    // element type: bf16 when set, else fp32
  AxisBoxes box;            // (W axis, forward)
};
hipError_t launch_generic_axis_pass(const AxisPassArgs& a, hipStream_t st);
// T and H axes of [slices][T][H][inner] tensors in one pass, in the forward or (with the transposed matrices) the inverse direction.
struct AxisPairArgs {
  const void* in[3]; void* out[3]; int n_tensors;
  const float* Mt; const float* Mh; int ldt, ldh;   // as in AxisPassArgs
  int T, H, slices; int64_t inner; int d;
  int in_bf16, out_bf16;
  AxisBoxes box;            // (forward)
};
// Rows kt of the T axis that the pass keeps in LDS when KT of them are wanted.  The products along H take rows in fours, so those of the last
// kt read up to row 4 ceil(H / 4) - 1 from its first: up to three rows on, which are as many kt where H is 1 and one kt where it is more.  (The
// matrix is zero there, but zero times what another kernel left in LDS is not if that is no number.)  Behind row T lies the H matrix.
constexpr int th_rows(int T, int H, int KT) {
  const int last = (KT - 1) * H + (H + 3) / 4 * 4 - 1;   // last row (kt, h) that is read
  return KT <= 0 ? 0 : last / H + 1 < T ? last / H + 1 : T;
}
bool generic_pair_fits(const AxisPairArgs& a);   // whether the pass takes these sizes and is the faster way
hipError_t allow_generic_axis_pair();            // lets its kernels ask for their LDS (when a context is set up: its calls may be captured)
hipError_t launch_generic_axis_pair(const AxisPairArgs& a, hipStream_t st);

// One branch of a generic attention launch (generic_attn.hip): query rows [0, nq) of every listed slice.
struct GAttnSeg {
  const float* Q; const float* K; const float* V; float* O;
  const int32_t* slice_list; int n_slices;
  int64_t slice_stride, o_slice_stride;   // elements between slices for Q / O
  int64_t kv_slice_stride;  // elements between slices for K/V (differs from Q for the exchange)
  int nq, nk;
  int mode;                 // 0 dense, 1 block list, 2 window
  const int32_t* row_ptr; const int32_t* col_idx; int block; int window;   // (window at most nk)
  int residual;             // O = Q + attention (exchange)
  const float* C; int64_t c_slice_stride; int nc;   // summary tokens the rows attend to after the band's keys (the exchange in the same launch), or NULL
  int rep, fill, n_out;     // query row i is written to output rows i rep .. i rep + fill - 1 below n_out (low band: its group)
  int rows, tiles, first_block;   // filled in by the launcher: query rows per workgroup, workgroups per slice, first workgroup
};
struct GAttnArgs { GAttnSeg seg[NBMAX]; int nseg; int d; float scale; };
// Launches the branches [first, first + count) of `a`; how their rows are split is decided for all of them together, so a branch
// gives the same bits alone.
hipError_t launch_generic_attn(GAttnArgs a, int num_cu, hipStream_t st, int first = 0, int count = NBMAX);

// Low-band compression of Q~, K~ and V~ for the slices in low_list, and summary tokens of the bands of all slices, written
// into the C slots of the other bands: one launch (pool = false: the compression alone, n_low_slices = 0: the
// summaries alone).
struct PoolArgs {
  const void* spec[3]; void* low[3];
  const int32_t* low_list; int n_low_slices;
  int64_t n_low, nbar; int c;
  bool pool;
  const void* Y; const void* V; void* C;
  const int32_t* masks; int slices, nb;
  const int64_t* band_off; const int64_t* band_n; const int* m_eff;
  int m2rows;
  // [NBMAX][4]: bit s of row l set = band l of slice s is not pooled here (no active band of the slice looks at it, or -
  // high band only - its V~ rows do not exist and launch_vsum supplies it); NULL: every band of every slice
  const uint64_t* skip_bits;
  float* part; int64_t part_floats;   // scratch for chunks that are cut into parts
  int n_pooled, pooled_bands;         // (slice, band) pairs pooled here, the bands among them (bits)
  int64_t N; int d, is_half, num_cu;
};
hipError_t launch_band_pools(const PoolArgs& p, hipStream_t st);
// Rows of the low band that the band operator left out (low_fill = 1): rows i c + 1 .. i c + c - 1 take row i c.
hipError_t launch_expand_low(void* Y, const int32_t* slice_list, int n_slices, int64_t N, int64_t n_low, int c, int64_t row_bytes,
                             hipStream_t st);
// High-band summary tokens of the slices in `sel` (bit set, nsel of them) from the untransformed bf16 V.
hipError_t launch_vsum(const void* V, const void* Wsum, float* part, void* C, const uint64_t sel[4], int nsel, int64_t N,
                       int d, int nsplit, int64_t n_high, const int m_eff[NBMAX], int m2rows, hipStream_t st);   // (three-band contexts only)
// Projected forward: P[batch][nb][mrows][dm] = per-chunk means of the band rows of X~ [batch][N][dm] (fp16), and the
// placement of the projected pooled rows T[slices][nb][mrows][d] into the C slots of the bands a slice passes through.
hipError_t launch_pool_wide(const void* X, void* P, int batch, int64_t N, int dm, int nb, const int64_t band_off[NBMAX],
                            const int64_t band_n[NBMAX], const int m_eff[NBMAX], int mrows, hipStream_t st);
hipError_t launch_place_summaries(const void* T, void* C, const int32_t* masks, int slices, int d, int nb, const int m_eff[NBMAX],
                                  int mrows, int m2rows, hipStream_t st);
// Router statistics: per band and channel, sum of squares over slices and the three spectral buffers.
hipError_t launch_band_energy(const void* sq, const void* sk, const void* sv, float* stats /*[3][d], zeroed inside*/,
                              int slices, int64_t N, int d, const int64_t band_off[3], const int64_t band_n[3],
                              int is_half, hipStream_t st);
hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t st);
hipError_t launch_probe_copy(const void* in, void* out, int64_t bytes, int num_cu, hipStream_t st);
hipError_t launch_probe_mfma(float* out, int blocks, int iters, hipStream_t st);
// out[slice] = in[slice] for the listed slices (slice_bytes each, a multiple of 16).
// out[i] = in[i] converted bf16 -> fp16 (to_bf16 = 0) or fp16 -> bf16 (round to nearest even), n elements, n % 8 == 0.
hipError_t launch_convert_16(const void* in, void* out, int64_t n, int to_bf16, hipStream_t st);
hipError_t launch_copy_slices(const void* in, void* out, const int32_t* slice_list, int n_slices, int64_t slice_bytes,
                              hipStream_t st);
#define ENERGY_PART_FLOATS 49152
struct EnergyWaves { int en[6]; int tot[3]; };   // waves whose slots hold this forward's partial sums, per statistics slot
hipError_t launch_energy_reduce(const float* energy_part /*[6][DCT_MAX_WAVES][3][64]: Q, K, V (box), Q, K, V (whole grid)*/,
                                const float* tot_part /*[3][DCT_MAX_WAVES][64] or NULL*/, float* stats /*[3][d] + ENERGY_PART_FLOATS of scratch*/, int d,
                                const EnergyWaves& nw, float* host /*[3][d] + 1, pinned*/, const int32_t* range_flag, hipStream_t st);

// Lets `kernel` ask for `bytes` of dynamic LDS on the current device.
inline hipError_t allow_lds(OncePerDevice& limit, const void* kernel, int bytes) {
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return (hipError_t)limit.run(dev, [&] { return (int)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}

// ---- MFMA kernels (mfma_dct.hip, mfma_attn.hip) -------------------------------------------------------------------
// The transform passes add what a lane's place within 8 rows takes to a wave-uniform 64-bit address, as an unsigned 32-bit number of
// bytes: whether rows `stride` 16-bit elements apart leave room for that.
inline bool eight_rows_fit(int64_t stride) { return stride * 8 * 2 + 128 <= 0xffffffffLL; }
struct DctPassArgs {
  const void* in; void* out;
  const half_t* M;          // fp16, row stride ldm: out[k] = sum_{j < n} M[k*ldm + j] in[j], k < n_out
  int n, n_out, ldm;        // rows contracted (multiple of 16, <= 128), rows produced (<= 128)
  // Slices of the caller's tensors: with slice_list set, slice sl of this launch is slice_list[sl] of q/k/v/out, of the
  // band-major buffers and of masks; list_in / list_out make the regular-layout input / output use it too
  // (element offset slice*slice_elems + slab_in_slice*rows*inner), otherwise those are compact scratch.
  const int32_t* slice_list; int list_in, list_out; int64_t slice_elems;
  // Scatter passes: up to three tensors per launch, segment i is slices [seg_end[i-1], seg_end[i]) of the launch with its own
  // input, output and slice list (instead of in, out, slice_list).
  const void* in_seg[3]; void* out_seg[3]; const int32_t* list_seg[3]; int seg_end[3];
  int delta;                // gather side: read (in - in_alt) on active bands and zero elsewhere instead of selecting
  const void* resid;        // bf16, addressed like out: out = resid + result (the sum is formed in fp32)
  float* tot_part;          // [global wave][64]: sum of squares of the input per column (pass with inner == d only)
  int64_t inner, outer, nslab;
  // Band-major side (section 3.3): with perm_in / perm_out set, row j (k) of the tile at slab s = slice*outer + o and
  // first column col0 is the band-major row perm[j*perm_k + o*perm_o + col0/d] of slice `slice`.
  const int32_t* perm_in; const int32_t* perm_out; int64_t Ntok, perm_k, perm_o;
  int32_t perm_scale;       // 0/1: index = k*perm_k + tile index; otherwise k*perm_k + tile index*perm_scale (transposed table)
  const void* in_alt; const int32_t* masks; int32_t band_off1, band_off2, band_off3;
  int in_bf16, out_bf16;    // element type of in / out: bf16 when set, else fp16
  int d;
  // Swapped scratch layout: with out_swap (in_swap) set, slab s = a*sw + b writes (reads) row k at
  // (((a*n + k)*sw_total) + b + sw_off)*inner instead of (s*n + k)*inner, i.e. the slab index b becomes the inner of the
  // two row indices.  The H-axis pass uses it to leave [h][t] order behind so that the T-axis pass finds its rows
  // W*d elements apart instead of H*W*d.
  int in_swap, out_swap, sw, sw_total, sw_off;
  // Router statistics fused into the forward pass that scatters into the band-major buffer (perm_out set): every
  // wave adds the squares of its fp32 results per band and column to energy_part[global wave][3][64].  With (u, v) the
  // coordinates of the tile on the two axes the pass does not transform (flat index = u*en_div + v), rows [0, t1) are
  // low, [t1, t2) mid and the rest high, t1 = low_a if u < low_u and v < low_v else 0, t2 likewise from the mid box.
  float* energy_part;
  // Scatter passes (perm_out set): a lane whose result leaves the fp16 range (or is not finite) stores 1 here.
  int32_t* range_flag;
  int en_omul, en_div, low_u, low_v, low_a, mid_u, mid_v, mid_a;  // flat index of the tile = o*en_omul + col0/d
};
#define DCT_MAX_WAVES 65536   // upper bound of waves in one launch of the DCT pass (sizes energy_part)
int mfma_dct_tiles(int n_in, int n_out);   // output tiles of 32 of the variant a pass takes
// `n` passes (at most three) of one variant - rows contracted, output tiles (at least as many as each keeps), kind of input and output - in one launch; waves_out[i]: waves
// of the i-th that store partial sums.
hipError_t launch_mfma_dct_pass(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out = nullptr);
inline hipError_t launch_mfma_dct_pass(const DctPassArgs& a, int num_cu, hipStream_t st, int* waves_out = nullptr) {
  return launch_mfma_dct_pass(&a, 1, num_cu, st, waves_out);
}
bool mfma_dct_supported(int n_in, int n_out);
// Whether the T pass of a class joins the launch of the class that keeps the most (`lead`).  It has to be small (fewer than four tiles per wave
// of a chip with two workgroups on every compute unit); and so has the lead on long axes, whose kernels pay for arguments that depend on
// the workgroup (k_dct_passes) more than a small launch takes.  Forward transforms apart / together, us, low heads beside two high
// ones: 16 x 64 x 64 x 64, 4 tiles per compute unit (2 heads) 100 / 93, 24 (12) 184 / 175; beyond the line 48 (24) 272 / 261, 256 (32 mid heads)
// 346 / 341; 32 x 64 x 64 x 128, 128 (32) 1051 / 1023.  Beside one high head of 64^3 x 128, where the lead is large, 4 to 32 heads:
// 451 / 447, 658 / 652, 1467 / 1456, 1870 / 1853 (mid heads: the same).  So the line is on the safe side; the gain beyond it is 1-4 %.
// The class goes through the lead's tiles and rows, of which it may keep and read fewer: tiles that it does not keep are dropped, and what a
// delta gathers beyond its box is zero (the same sums, the same bits).  Forwards, passes of unequal boxes apart / together, us: heads low, mid and
// high of 64, 64 x 16 x 16 101 / 81, 112 x 16 x 16 142 / 100, 128 x 32 x 64 502 / 466, 32 x 32 x 32 99 / 94; two low, mid and high
// each and more of 96 x 16 x 16 377 / 352, 128 x 32 x 64 x 128 (4 heads) 926 / 910.  Beside a large lead the gather is slower together: 16 heads of
// 32 x 128 x 128 x 128, 14 of them high, 12590 / 12745.
inline bool dct_passes_share(const DctPassArgs& lead, const DctPassArgs& a, int num_cu) {
  auto tiles = [](const DctPassArgs& x) { return x.nslab * (x.inner / 64); };
  if (a.n > lead.n || (a.n < lead.n && !(a.perm_in && a.delta)) || mfma_dct_tiles(lead.n, a.n_out) > mfma_dct_tiles(lead.n, lead.n_out)) return false;
  return tiles(a) < 32 * (int64_t)num_cu && ((lead.n <= 32 && a.n == lead.n) || tiles(lead) < 32 * (int64_t)num_cu);
}
// W and H axes of the forward transform in one pass, or those of the inverse (mfma_wh_impl.h): input rows of `cols` values
// through the W matrix, `rows` of them through the H matrix.
struct WhPassArgs {
  // up to three tensors: segment i is slices [seg_end[i-1], seg_end[i]) of the launch, slice sl of a segment is slice_list[i][sl]
  // (NULL: sl itself) of the caller's tensor and slice sl of the compact one
  // forward: in (caller's) bf16 [slices][T][rows][cols][d], out (compact) fp16 [segment's slices][out_rows][T][out_cols][d]
  // inverse: in (compact) fp16 [segment's slices][rows][T][cols][d], out (caller's) bf16 [slices][T][out_rows][out_cols][d]
  const void* in[3]; void* out[3];
  const int32_t* slice_list[3]; int seg_end[3];
  int T, d, rows, cols, out_rows, out_cols;         // d: channels per token (a multiple of 64); rows and cols multiples of 16, inverse: all four
  const half_t* Mh; const half_t* Mw; int ldh, ldw; // fp16 [out_rows][>= rows], [out_cols, to whole tiles of 16][>= cols] with their row strides
  const void* resid;                                // inverse: bf16, addressed like out, added, or NULL
  float* tot_part;                                  // forward: [slot][64]: sum of squares of the inputs per channel, or NULL
  int32_t* range_flag;                              // forward: set when an input value leaves the fp16 range
  int members, col_parts;                           // (filled in by the launcher) workgroups that share a plane
};
// Whether the pass takes kh x kw coefficients of T planes of H x W with d channels per token.
bool wh_fits(int T, int d, int H, int W, int kh, int kw);
int wh_items(const WhPassArgs& a);   // workgroups' worth of work in it
// `n` passes (at most three) over planes of the same width in one launch, with the tiles that suit the first, which keeps the most rows
// (inverse: over planes of one size, from boxes 16, 32 or 64 wide if there are several); slots_out[i]: slots of tot_part of the i-th.
hipError_t launch_wh_pass_0(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out);   // W <= 64
hipError_t launch_wh_pass_1(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out);   // W > 64
inline hipError_t launch_wh_pass(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out) {
  return subs[0].cols <= 64 ? launch_wh_pass_0(subs, n, num_cu, st, slots_out) : launch_wh_pass_1(subs, n, num_cu, st, slots_out);
}
// Two forward passes one after the other in one launch, the first on a box of at most 32 rows, the second keeping more than 32.
bool wh_two_fits(const WhPassArgs& a, const WhPassArgs& b, int num_cu);
hipError_t launch_wh_two(const WhPassArgs& a, const WhPassArgs& b, int num_cu, hipStream_t st, int slots_out[2]);
bool hw_fits(const WhPassArgs& a);   // whether the inverse takes these sizes and is faster than an axis at a time
hipError_t launch_hw_inverse(const WhPassArgs* subs, int n, int num_cu, hipStream_t st);
// H and W axes of the inverse transform in one pass (mfma_iwh_impl.h).
struct IwhPassArgs {
  const void* in; void* out; const void* resid;     // in: fp16 [n_slices][kh][T][kw][d]; out: bf16 [slices][T][H][W][d]; resid: like out, added, or NULL
  const int32_t* slice_list; int n_slices;          // slices of out and resid
  int T, H, W, d, kh, kw;                           // d: channels per token; kh, kw: coefficients (multiples of 16)
  const half_t* Fh; const half_t* Fw;               // fp16 [H][H], [W][W]: rows are positions
  int parts;                                        // (filled in by the launcher) workgroups that share a plane
};
bool iwh_fits(const IwhPassArgs& a, int num_cu);   // whether the pass takes these sizes and is the faster way
hipError_t launch_iwh_pass(const IwhPassArgs& a, int num_cu, hipStream_t st);
hipError_t launch_gemm_nt(const GemmProblem* d_probs, const GemmSeg* d_segs, int per, int m, int n, int steps, int call_steps, int num_cu, hipStream_t st);
hipError_t launch_transpose_bf16_to_f16(const void* in /*[R][Cc] bf16*/, void* out /*[Cc][R] fp16*/, int R, int Cc, hipStream_t st);
hipError_t launch_mfma_attn(const AttnParams& p, const AttnItem* items, int n_items, int rows_per_item, int num_cu,
                            hipStream_t st);

}  // namespace fa
