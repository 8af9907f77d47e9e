// Launchers of the gfx950 kernels of the HDF hot path (host-callable).
#pragma once
#include <hip/hip_runtime_api.h>
#include <cstdint>

namespace hdf {

// Device geometry record written by the prep pass (binary64).
struct GeoDev {
  double c[8];
  double R2, R, Reff, inv_unused;
  double nu2_sum;
  double rho2_min, rho2_max;
  double nonfinite;
};

constexpr int kPrepBlocks = 512;
constexpr int kNuPairs = 65536;
constexpr uint64_t kNuSeed = 0x48444600ull;

// Geometry: SoA copy of the points, bounding-box centre, radius, rho^2 range
// and the ||K||_F sample.  dtype 0 = float32, 1 = float64.
hipError_t launch_prep(const void* pts, int dtype, int64_t n, int d, int64_t ld, void* x_soa,
                       int64_t ldx, int kernel, double l, double* partials, GeoDev* geo,
                       hipStream_t s);

// Geometry of two sets (X u Y) with the cross-pair ||K(X, Y)||_F sample.
// partials: at least 2 * kPrepBlocks * 18 doubles.
hipError_t launch_prep_cross(const void* ptsx, int64_t nx, int64_t ldx, const void* ptsy, int64_t ny,
                             int64_t ldy, int dtype, int d, void* soax, int64_t ldsx, void* soay,
                             int64_t ldsy, int kernel, double l, double* partials, GeoDev* geo,
                             hipStream_t s);

// Sampled pairs of the tighter degree and rank rules: pair t uses SplitMix64
// outputs 2t+1 and 2t+2 of the stream `seed` (a = out >> 11 mod n, likewise
// b).  out[0..M) = ||x_a - x_b||, out[M..2M) = rho_a^2, out[2M..3M) = rho_b^2,
// out[3M..4M) = dot of the normalised points (x - c) / Reff; idx[0..M) = a,
// idx[M..2M) = b.  Needs the geometry of launch_prep.
constexpr uint64_t kPairSeed = 0x48444601ull;
hipError_t launch_pairs(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                        uint64_t seed, int M, double* out, int32_t* idx, hipStream_t s);

// Weighted Chebyshev moments mu[k][c] = sum_i rho_i^{2k} T_c(t_i), k <= K,
// c <= 2K, written to `moments` (rows 16*nrt x cols 16*nct, binary64).
// mode 0: binary64 MFMA; 1: binary32 MFMA; 2: binary32 hi/lo split MFMA.
int gram_blocks(int64_t n);
hipError_t launch_gram(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                       const GeoDev* geo, double u0, double u1, int K, int mode,
                       double* partials, double* moments, hipStream_t s);

// Refinement Gram: G2_k = (Y_k T1_k)^T (Y_k T1_k) for the selected degrees
// k = sel[0..n_sel) (binary64), written to out[i][32][32]; T1 packed per degree
// at t1_off[k] (L_k x L_k).
int gram2_blocks(int64_t n, int n_sel);
hipError_t launch_gram2(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                        const GeoDev* geo, double u0, double u1, int K, const double* T1,
                        const int32_t* t1_off, const int32_t* sel, int n_sel, double* partials,
                        double* out, hipStream_t s);

// Tables of the factor-evaluation kernel.
struct BuildTables {
  const int32_t* col_of;     // loop-order iteration -> harmonic row (or -1)
  const void* chain;         // (level, b, n) -> (A, B) pairs, storage type
  const int32_t* q_len;      // per radial row: L
  const int32_t* q_off;      // per radial row: offset into q_coef
  const void* q_coef;        // radial coefficients, storage type
  int K;                     // largest kept degree: depth of the harmonic recurrences
  int S;                     // radial rows
  const int32_t* leaves;     // (level, b) -> harmonics below a chain loop of that level and base, level 0..d-2
  int n_loop;                // harmonics evaluated (loop order), kept or not
};
// rows of phi and q get their n values and zeros up to the next multiple of 64 plus 64
hipError_t launch_build(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                        const GeoDev* geo, double u0, double u1, const BuildTables& tb,
                        int prec, void* phi, int64_t ld_phi, void* q, int64_t ld_q,
                        hipStream_t s);

// Per-degree description for the contraction kernels.
struct DegDev {
  int32_t hoff;   // first harmonic row of the degree in phi
  int32_t nh;     // |H_k|
  int32_t qoff;   // first radial row in q
  int32_t s;      // s_k
  int32_t roff;   // first rank row (k, h=0, l=0)
  int32_t boff;   // first block of the degree in pass 2's block-ordered copy of D W
  int32_t pad[2];
};
// Contraction launchers: prec is the factor's storage and arithmetic type (1 = binary32,
// 0 = binary64), io the type of V and KV (0 = float32, 1 = float64).  Supported pairs:
// (1, 0), (0, 1) and (0, 0), the last for a binary64 factor of binary32 data.

// Pass 1: partial[split][row][c] = sum_{i in split} U[i,row] V[i,c] (row = (k,h,l), c < m16, rows of mo
// entries, binary64); with n_slabs > 1 the m columns are n_slabs slabs of m16.
// Pass 1, tile-major (m16 <= 64).  A wave item is one 16-row tile of one
// degree's harmonics with a range of nl <= matvec_tile_nl(prec, NCT) of its
// radial functions and the column tiles [ct0, ct0 + nct) (NCT = 1, 2 or 4
// column tiles per launch); one load of the tile's harmonic values feeds the
// MFMAs of all its (l, column) slots.  A workgroup runs one group (up to kMvtWavesPerGroup wave items whose
// radial rows lie in [q_lo, q_lo + nq), nq <= kMvtMaxNq) over one split of
// split_len points (a multiple of 32; n_splits * split_len >= n >
// (n_splits - 1) * split_len) and writes partial[split][row][c] (binary64)
// for the rank rows of its wave items, every row once per split.
struct MvtWave {
  int32_t row0;   // first harmonic row of the tile (harmonic offset of the degree + h0)
  int32_t nr;     // harmonic rows in the tile (<= 16)
  int32_t qrow;   // radial row of the first radial function
  int32_t nl;     // radial functions
  int32_t ct0;    // first column tile
  int32_t nct;    // column tiles (<= 4)
  int32_t out0;   // rank row of (h0, first radial function)
  int32_t s;      // s_k: rank-row stride between consecutive harmonics
};
// A wave item with qrow < 0 is a rank-row item (nl = 1): its rows are the rank rows
// [row0, row0 + nr) of the rank-row table (nr <= 16), each a (harmonic row, radial row, output
// row) triple, so rows of different degrees and radial functions share one tile.  Row r of its
// tile is phi_{hrow}(x) q_{qrow}(x), its output row out.
struct MvtRankRow {
  int32_t hrow;   // harmonic row in phi
  int32_t qrow;   // radial row in q
  int32_t out;    // rank row of the result
  int32_t pad;
};
constexpr int kMvtWavesPerGroup = 8;   // wavefronts per workgroup
struct MvtGroup {
  int32_t w0, nw;     // wave items [w0, w0 + nw), nw <= kMvtWavesPerGroup
  int32_t q_lo, nq;   // radial rows staged in LDS
};
// radial functions per wave item for column-tile count nct (1, 2 or 4) of the launch
int matvec_tile_nl(int prec, int nct);
constexpr int kMvtMaxNq = 32;      // staged radial rows per workgroup
size_t matvec_tile_lds_bytes(int m16, int prec);
hipError_t launch_matvec_t_tile(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q,
                                const MvtWave* waves, const MvtRankRow* rank_rows, const MvtGroup* groups,
                                int n_groups, int n_splits,
                                int64_t split_len, const void* V, int64_t ldv, int64_t n, int m, int m16,
                                int n_slabs, int mo, int64_t rank, double* partials, int prec, int io, hipStream_t s);
// Pass 2 takes D W in blocks of 16 harmonics x one radial function, batch after batch of a degree and
// degree after degree (n_blocks = sum over degrees of ceil(nh / 16) s; the degrees' first blocks in
// DegDev::boff), 16 m16 values per block.  launch_matvec_reduce sums the pass-1 partials over the
// splits and writes W[row][c] (binary64), Wd[row][c] = lambda_row * W (storage type) and Wb, the same
// values in block order; any of them may be NULL.  src: the rank row of every row of the blocks, -1
// past a degree's harmonics.
hipError_t launch_matvec_reduce(const double* partials, int n_splits, int64_t rank, int m16, const int32_t* src,
                                int64_t n_blocks, const double* lam_row, double* W, void* Wd, void* Wb, int prec,
                                hipStream_t s);
// column tiles per wavefront of pass 2 over n points for cpl = m16 / 16
int matvec_n_tiles(int64_t n, int cpl);
// Pass 2: KV[i][c] = sum_rows U[i,row] (D W)[row][c], D W in block order.
// z_blocks > 0: the blocks are split into shares of z_blocks, each share's KV in part (shares x n x m,
// storage type), summed in order into KV
hipError_t launch_matvec_n(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q,
                           const DegDev* degs, int n_deg, const void* Wb, int64_t n_blocks, int m16,
                           void* KV, int64_t ldkv, int64_t n, int m, int prec, int io, int z_blocks,
                           void* part, hipStream_t s);

// Narrow products: 1 <= m <= kNwMax right-hand sides, on the vector units.  Pass 1 runs n_items (row
// blocks) x n_splits wavefronts and leaves Wn[row][c] = lambda_row W (storage type, stride m) and, where
// wanted, W (binary64, stride w_ld), by way of part (n_splits x rank x m) when there are several splits.
// Pass 2 forms KV from Wn; z_rows > 0 splits the n_rows harmonics into shares (shares x n x m values).
constexpr int kNwMax = 4;
int narrow_items(const DegDev* degs_host, int n_deg, int prec, int m);
void narrow_splits(int64_t n, int n_items, int prec, int64_t per_split_bytes, int64_t most_bytes, int* n_splits,
                   int64_t* split_len);
hipError_t launch_narrow_t(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q, const DegDev* degs, int n_deg,
                           int n_items, int n_splits, int64_t split_len, const void* V, int64_t ldv, int64_t n, int m,
                           int64_t rank, const double* lam, void* Wn, double* W, int64_t w_ld, double* part, int prec,
                           int io, hipStream_t s);
hipError_t launch_narrow_n(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q, const DegDev* degs, int n_deg,
                           const void* Wn, void* KV, int64_t ldkv, int64_t n, int m, int n_rows, int z_rows,
                           void* shares, int prec, int io, hipStream_t s);

// Products of several binary64 factors, one right-hand side each (entries [pos, pos + n) of v and out).
struct MvBatch {
  const double *phi, *q;
  int64_t ld, n, pos, rank, split_len;
  const DegDev* degs;
  const double* lam;
  double *part, *Wn, *shares;
  int32_t n_items, n_splits, n_deg, z_rows, nz, pad;
};
struct MvBatchGrid {
  int factors;      // descriptors
  int t_blocks;     // largest number of pass-1 workgroups, ...
  int r_blocks;     // ... of 64-row groups of the reduction (0: no factor has several splits),
  int n_blocks;     // ... of 64-point groups
  int shares;       // ... and of shares of pass 2
};
hipError_t launch_matvec_batch(const MvBatch* batch_dev, const MvBatchGrid& g, const double* v, double* out,
                               hipStream_t s);

// Coefficients of the adjoint's products: c2 (c2_rows x c2_cols; blocks of pass 2 in block order, or
// rank rows), cs (shift_blocks blocks of cs_cols columns, block order; n_shifted = 0: none).
hipError_t launch_adj_coefficients(const double* gv, const double* gw, int64_t gstride, int m, int d,
                                   const double* lam, const DegDev* degs, const int32_t* src, int64_t c2_rows,
                                   int c2_cols, int c2_block_order, void* c2, const DegDev* shifted, int n_shifted,
                                   const int32_t* map, const int32_t* map_h, const double* map_v,
                                   int64_t shift_blocks, int cs_cols, void* cs, int prec, hipStream_t s);

// Adjoint by contractions (see hdf_backward).  launch_radial evaluates S
// Chebyshev series of t(rho^2) at every point: out[row][i] = scale * sum_a
// coef[q_off[row] + a] T_a(t_i), a < q_len[row], zeros past n (rows as
// long as launch_build's).  launch_adj_combine
// forms dX[i][j] = (1/R) [sum_c w_ic KS[i][2mj + c] + v_ic KS[i][2mj + m + c]
// + 2 xt_ij (sum_c w_ic K2[i][c] + v_ic K2[i][m + c])], KS zeros if NULL.  prec: factor type
// (1 binary32, 0 binary64); dtype: points, W, V and dX (0 float32, 1 float64).
hipError_t launch_radial(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                         double u0, double u1, const int32_t* q_len, const int32_t* q_off, const void* coef,
                         int S, double scale, int prec, void* out, int64_t ld_out, hipStream_t s);
hipError_t launch_adj_combine(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                              const void* KS, int64_t ldks, const void* K2, int64_t ldk2, const void* Wm,
                              const void* Vm, int64_t ld, int m, void* dX, int64_t lddx, int prec, hipStream_t s);

// Fused matrix-free passes (mf_kernels.hip).  A workgroup of kMfWaves
// wavefronts takes kMfP points at a time: it evaluates their harmonics (the
// factor-evaluation recurrences, split into subtrees run by 16-lane groups)
// and radial functions into LDS and contracts them there with MFMA, so no
// factor value reaches HBM.
constexpr int kMfP = 16;                 // points per chunk
constexpr int kMfWaves = 8;              // wavefronts per workgroup
// One evaluation job of a wavefront.  A subtree of the harmonic recursion
// fixes the azimuthal index m (cosine or sine branch) and, for d >= 4, the
// index of chain level d - 2; its base b is their sum.  Subtrees of one base
// share every value below their prefixes, so a job runs the shared levels of
// base b once per point (lane = point) and writes the harmonics of a list of
// its subtrees (16-lane group g takes every fourth).  For d >= 5 a job covers
// the level d - 3 indices [n_lo, n_hi] only.
struct MfJob {
  int32_t b;        // base
  int32_t n_lo, n_hi;
  int32_t off;      // loop-order offset of the job's first harmonic within each of its subtrees
  int32_t task0;    // first entry of the job's subtrees in the per-base list (btab)
  int32_t ntask;    // subtrees of the job
  int32_t pad[2];
};
// Pass 1: one accumulator tile of a wavefront, 16 harmonics of one degree with one radial function
// (slot i: loop-order rows rows[17 i .. 17 i + 15], radial row rows[17 i + 16]): rank rows
// out0 + j s for j < nr.
struct MfSlot1 {
  int32_t row0, qrow, out0, s, nr;
  int32_t pad[3];
};
// Pass 2: one MFMA step of a wavefront, harmonics j < nv <= 4 of one degree with one radial function
// (slot i: loop-order rows rows[5 i .. 5 i + 3], radial row rows[5 i + 4]): rank rows rank0 + j s.
struct MfSlot2 {
  int32_t row0, qrow, rank0, s, nv;
  int32_t pad[3];
};
// LDS layout (byte offsets) of a fused pass: harmonic rows in loop order ((n_loop + 1) x kMfP,
// the last row zero), radial rows, V^T of the chunk (pass 1) or the per-wavefront partial
// products (pass 2), the slots' row table (n_rows 16-bit indices), the radial coefficients, the
// level d-2 recurrence pairs, two buffers of subtree prefixes (n_tasks x kMfP each) and the
// per-base subtree list.
struct MfLayout {
  int32_t phc, qc, aux, rtab, qcoef, ctop, ptab, ptab_len, btab, total;
  int32_t phc_len, qc_len, aux_len;   // values per buffer of the chunk data (two buffers when spec)
};
// spec: the wavefront-specialised kernels (2 kMfWaves wavefronts, the chunk data double-buffered)
MfLayout mf_layout(int64_t n_loop, int S, int64_t n_rows, int64_t n_qcoef, int64_t n_tasks, int d, int K, int prec,
                   int pass, bool spec);
// Pass-1 accumulator tiles and pass-2 steps per wavefront (the D W operands of the steps stay in
// registers).  Ranks beyond a workgroup's slots take several slot groups, each of which evaluates the
// factor again.  The plain binary32 kernels run where two buffers of the harmonics exceed LDS, so one
// workgroup has a CU and half the wavefronts per SIMD: they take the registers for half as many again.
// Products with 16 and 64 before, and so: 1e6 points in d = 5 of rank 2142 x 16 columns 7.9 and 4.6 ms; 200,003
// of rank 2212 x 16 1.68 and 1.01, x 64 6.5 and 3.8, of rank 3618 x 16 2.68 and 1.97; in d = 4 of rank 2666 x 16
// 1.48 and 1.20; 20,011 of rank 3048, where the number of groups stays, 0.258 both.
constexpr int mf_slots(bool f32, bool spec, int pass) { return (f32 && !spec ? 3 : 2) * (pass == 1 ? 8 : 32); }
// A wavefront's slot list is padded to whole blocks (pass 1: padding slots have out0 = -1; pass 2:
// nv = 0) so that the kernels test the list length once per block.
constexpr int kMfBlock1 = 4;
constexpr int kMfBlock2 = 8;
constexpr int kMfMaxKs = 8;              // radial coefficients per row <= 4 kMfMaxKs (p / 2 + 1 <= 31)
struct MfArgs {
  const void* x_soa; int64_t ldx; int64_t n; int dtype; int d;
  const GeoDev* geo; double u0, u1;
  const MfJob* jobs; const int32_t* job_off;          // jobs of wavefront w: [job_off[w], job_off[w + 1])
  const int32_t* btab; int n_tasks;                   // subtrees by base: (subtree index, first harmonic)
  int64_t n_loop;                                     // harmonics of the recursion (degrees <= K)
  const void* chain; int K;                           // recurrence pairs, as for the factor evaluation
  const void* qmat; int S, S_pad, L_pad; int64_t H;   // radial coefficients, S_pad x L_pad (factor type)
  int prec;                                           // factor type: 1 binary32, 0 binary64
};
// Workgroups of one fused pass that fit on a CU at once (occupancy of the kernel with its LDS).
int mf_blocks_per_cu(const MfArgs& a, int pass, const MfLayout& lay, bool spec);
// Pass 1: partial[split][row][c] for splits of split_len points (a multiple of kMfP), rank rows of
// slot group g (slots of wavefront w: [slot_off[9 g + w], slot_off[9 g + w + 1])), columns of tile ct;
// grid n_splits x (n_groups cpl).  rows: the slots' loop-order rows (n_rows entries).
hipError_t launch_mf_t(const MfArgs& a, const MfLayout& lay, bool spec, const MfSlot1* slots, const int32_t* slot_off,
                       const int32_t* rows, int n_rows, int n_groups, int cpl, int n_splits, int64_t split_len,
                       const void* V, int64_t ldv, int m, int m16, int64_t rank, double* partials, hipStream_t s);
// Pass 2: KV = U Wd over ranges of range_len points; with n_groups > 1 each slot group writes its
// share to part (n_groups x n x m, factor type), summed in group order into KV.
hipError_t launch_mf_n(const MfArgs& a, const MfLayout& lay, bool spec, const MfSlot2* slots, const int32_t* slot_off,
                       const int32_t* rows, int n_rows, int n_groups, int cpl, int n_ranges, int64_t range_len,
                       const void* Wd, int m16, void* KV, int64_t ldkv, int m, void* part, hipStream_t s);

// Scratch of hdf_matvec_noalloc: a fixed device array per GPU (scratch.hip).
// scratch_address returns its device address on the current device (resolved
// once per device); hipErrorInvalidDevice for device ordinals >= 64.
constexpr size_t kScratchBytes = (size_t)32 << 20;
hipError_t scratch_address(void** p);

}  // namespace hdf
