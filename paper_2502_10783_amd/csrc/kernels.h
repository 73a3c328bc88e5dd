// Kernel declarations of libipp (definitions in k_*.hip).
#pragma once

#include "ipp_internal.h"

namespace ipp {

template <int PPT>
__global__ void k_mesh_stats(Work wk, ipp_params p);
template <int PPL>
__global__ void k_mesh_stats_w(Work wk, ipp_params p);
__global__ void k_mesh_fill(Work wk, ipp_params p);
template <int F>
__global__ void k_mesh_filter(Work wk, ipp_params p);
template <int PASS>
__global__ void k_mesh_spline(Work wk, ipp_params p, int lines);

template <int TH, int TW>
__global__ void k_bkg_maps(Work wk, ipp_params p);
// k_aperture, k_refine, k_kron, k_source_moments (four rows) and k_mesh_stats_w
// take a wavefront per row or region, each in a workgroup of its own: rows
// differ (a refinement of no steps or of ten, one window or another), and a
// workgroup of four kept its registers and LDS until the last was done (a
// refinement of 1.0e5 rows held 72 % of the wavefront slots).  Against 4 and 2
// wavefronts a workgroup: k_refine 8095 and 7727 to 7119 us, k_aperture of
// 1.3e5 rows 864 and 848 to 839, k_kron of four 4096^2 frames 312 and 276 to
// 268; against 4, k_mesh_stats_w of sixteen 4096^2 frames 609 to 590 and
// k_source_moments 98 to 92; k_aperture_bwd, whose rows are alike, loses 3 %
// and keeps four.  Grids: as many rows as a launch deals out at no cost (half
// and twice as many: k_aperture 852 and 838 to 829 us; k_refine 7080 at half,
// 6993 at twice to 6945).
constexpr int kRowThreads = 64;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kRowGrid = 65536;
constexpr int kRefineGrid = 131072;
// threads per detection tile (4096 pixels: 8 per thread)
constexpr int kTileThreads = 512;
template <int TH, int TW, bool FUSED, bool CONN8, int NT>
__global__ void k_tile_ccl(Work wk, ipp_params p, int write_rms);
// threads of k_border: one per right-border and bottom-border pixel of a
// tile, in whole waves
template <int TH, int TW>
constexpr int border_threads() { return (TH + TW + 63) / 64 * 64; }
template <int TH, int TW>
__global__ void k_border(Work wk, ipp_params p);
template <int TH, int TW>
__global__ void k_relabel(Work wk, ipp_params p);

__global__ void k_fill_i64(int64_t* a, int64_t n, int64_t v);
__global__ void k_resolve(Work wk, ipp_params p);
__global__ void k_heads(Work wk, ipp_params p);
__global__ void k_scan_blocks(const int32_t* in, int32_t* blocks, int n);
__global__ void k_scan_top(int32_t* blocks, int nblocks, int64_t* total);
__global__ void k_scan_apply(const int32_t* in, const int32_t* blocks,
                             int32_t* out, int n);
__global__ void k_clear(Work wk);
__global__ void k_frame_offsets(Work wk, ipp_sources src, int64_t* diag);
constexpr int kScanThreads = 1024;  // threads of the one-workgroup kernels
constexpr int kScanRows = 16384;    // rows k_scan_rows takes
constexpr int kSmallTiles = 96;     // detection tiles k_number_small takes
__global__ void k_scan_rows(Work wk, ipp_sources src, int64_t* diag);
__global__ void k_number_small(Work wk, ipp_params p, ipp_sources src,
                               int64_t* diag);
__global__ void k_scatter(Work wk, ipp_params p);
__global__ void k_rank(Work wk, ipp_params p, ipp_sources src);
__global__ void k_reclabel(Work wk);
__global__ void k_source_stats(Work wk, ipp_sources src);
__global__ void k_source_moments(Work wk, ipp_sources src, double* mom);

template <int NS>
__global__ void k_aperture_t(Work wk, ipp_params p, ipp_sources src,
                             double* sky_lohi);

template <int NS>
__global__ void k_aperture_bwd_t(Work wk, ipp_params p, ipp_sources src,
                                 const double* sky_lohi, const double* gF,
                                 double* dxy);

// Centroid refinement, every step of a row in one wavefront: xo, yo get
// the refined centres; PHOT: the photometry columns of the first
// evaluation as well.  Rows: min(capacity, *n_total).
template <int NS, bool PHOT>
__global__ void k_refine_t(Work wk, ipp_params p, double r_c, double eta,
                           int steps, ipp_sources src, double* xo,
                           double* yo);

// ab (nullable): device (a, b) used in place of the value arguments
__global__ void k_asinh_fwd(const float* v, float* y, int64_t n, float inv_a,
                            float b, const double* ab);
__global__ void k_asinh_bwd(const float* v, const float* dy, float* dv,
                            int64_t n, double a, double b, const double* ab,
                            double* partial);
__global__ void k_asinh_bwd_final(const double* partial, int nb,
                                  double* out);
// Device address of the file-scope scratch of the asinh backward on
// `device` (2 * kAsinhMaxBlocks doubles), looked up on first use with that
// device current and kept per device.  hipSuccess or the lookup's error.
hipError_t asinh_scratch(int device, double** ptr);

// Deblending (k_deblend.hip): see that file for the sequence.
// need: scratch units per row; big / nbig: the rows of the workgroup
// kernels, k_db_large's from the front (nbig[0]), k_db_mid's from the back
// (nbig[1]); nbig zeroed by the caller.  queue: k_db_small's counters,
// cleared if they are several (the caller clears a single one).
__global__ void k_db_need(ipp_sources cand, int64_t* need, int32_t* big,
                          int64_t* nbig, int64_t* queue);
__global__ void k_scan64_blocks(const int64_t* in, int64_t* blocks,
                                int64_t n);
__global__ void k_scan64_top(int64_t* blocks, int64_t nblocks,
                             int64_t* total);
__global__ void k_scan64_apply(const int64_t* in, const int64_t* blocks,
                               int64_t* out, int64_t n);
// Bounding boxes up to kDbSmallBox pixels take a wavefront, up to kDbMidBox
// a workgroup of four, larger ones one of eight, in LDS up to kDbBigBox.
constexpr int kDbSmallBox = 512, kDbMidBox = 2048, kDbBigBox = 6144;
// Resident workgroups per compute unit of the three kernels (by their LDS);
// queue: a zeroed counter of taken rows (k_db_small: db_queues(capacity) of
// them, kDbQueueStep words apart).  The several counters lie where the object
// offsets go once the candidates are done, if those take so many words; short
// tables have one counter.
constexpr int kDbQueues = 16, kDbQueueStep = 16;
__host__ __device__ inline int db_queues(int64_t capacity) {
  return capacity + 1 >= kDbQueues * kDbQueueStep ? kDbQueues : 1;
}
constexpr int kDbSmallPerCu = 11, kDbMidPerCu = 3, kDbLargePerCu = 1;
#define IPP_DB_DECLARE(NAME)                                                  \
  __global__ void NAME(Work wk, ipp_sources cand, const int64_t* off,         \
                       const int64_t* tot, char* pool, int64_t pool_units,    \
                       double nsigma, int conn, int nthresh, int clean,       \
                       double mincont, double kc, int64_t* cnt,               \
                       int64_t* queue, const int32_t* big,                    \
                       const int64_t* nbig);
IPP_DB_DECLARE(k_db_small)
IPP_DB_DECLARE(k_db_mid)
IPP_DB_DECLARE(k_db_large)
#undef IPP_DB_DECLARE
// All three in one, for tables of at most kDbAllRows rows.
constexpr int kDbAllRows = 2048;
__global__ void k_db_all(Work wk, ipp_sources cand, const int64_t* off,
                         const int64_t* tot, char* pool, int64_t pool_units,
                         double nsigma, int conn, int nthresh, int clean,
                         double mincont, double kc, int64_t* cnt,
                         int64_t* queue2, int64_t* queue1, int64_t* queue0,
                         const int32_t* big, const int64_t* nbig);
__global__ void k_db_zero(Work wk);
constexpr int kDbWriteThreads = 256;
__global__ void k_db_write(Work wk, ipp_sources cand, const int64_t* off,
                           const int64_t* tot, const char* pool,
                           int64_t pool_units, const int64_t* cnt,
                           const int64_t* ooff, ipp_sources obj,
                           int32_t* parent);
__global__ void k_db_offsets(Work wk, ipp_sources cand, const int64_t* ooff,
                             const int64_t* total, ipp_sources obj);
__global__ void k_db_flags(ipp_sources cand, const int64_t* cnt,
                           const int64_t* total, ipp_sources obj,
                           const int32_t* parent);
__global__ void k_db_diag(const int64_t* tot, int64_t pool_units,
                          const int64_t* counters, int64_t* diag);

// AUTO (Kron) photometry: one wavefront per row (k_kron.hip); windows of
// more than kKronBigPx pixels go in parts of kKronPart pixels: k_kron lists
// them, then k_kron_parts<1> (pass 1 of the rows whose search window is
// large) and k_kron_parts<2>.
constexpr int kKronBigPx = 4096;
constexpr int kKronPart = 2048;
struct KronPart {
  int64_t row;           // -1: not used
  int32_t k, done;       // part of the row; of its first: parts summed
  double s0, s1;         // the part's two sums
};
struct KronTable {
  int64_t* count;        // parts asked for (may exceed cap)
  KronPart* part;
  int64_t cap;
};
__global__ void k_kron(Work wk, ipp_sources src, const double* mom,
                       double kfac, double rmin, double search, KronTable t1,
                       KronTable t2, double* kron, double* flux, double* area,
                       uint32_t* flags);
template <int PASS>
__global__ void k_kron_parts(Work wk, ipp_sources src, const double* mom,
                             double kfac, double rmin, double search,
                             KronTable tb, KronTable next, double* kron,
                             double* flux, double* area, uint32_t* flags);

// Stamp convolution and subtraction of the batch's `stamps` stamps (the
// descriptors already on the device).
hipError_t launch_subtract(const SubFrame* frames, int nframes,
                           const SubBasis& bs, int64_t stamps,
                           hipStream_t s);

__global__ void k_zscale(const GrayFrame* frames, double contrast,
                         double krej, int max_iter, double* z1z2,
                         double* info);
__global__ void k_gray_map(const GrayFrame* frames, int nframes,
                           int total_rows, int kind, float a, float c,
                           float lna, const double* lohi);
__global__ void k_eq_clear(uint32_t* mm, int n, uint32_t* counts, int64_t nc);
__global__ void k_eq_minmax(const GrayFrame* frames, int nframes,
                            int total_rows, uint32_t* mm);
__global__ void k_eq_hist(const GrayFrame* frames, int nframes,
                          int total_rows, int nbins, const uint32_t* mm,
                          uint32_t* counts);
__global__ void k_eq_map(const GrayFrame* frames, int nframes, int total_rows,
                         int nbins, const uint32_t* mm,
                         const uint32_t* counts);

}  // namespace ipp
