// Host-side interfaces between the C ABI layer and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/vup.h"
#include "vup_device.hpp"

namespace vup {

constexpr uint64_t kMagic = 0x5655504d4d763031ull;  // "VUPMMv01"

// LDS layout of a sweep kernel (offsets in floats from the start of dynamic LDS)
struct SweepLayout {
  int tab_off[4];
  int cap[4];
  int row_off;      // row table: [rrows] / [kBwdRowChunk] entries in the run forms, [kRowChunk] in the cell forms
  int rrows;        // rows per row-table pass of the propagation (run and cell forms)
  int trow_off;     // float4[kRowChunk] (backward only, else -1)
  int hist_off;     // histogram copies (propagate) or v table (backward)
  int hist_stride;  // floats per histogram copy (run form); words of all copies (cell form)
  int cpw;          // histogram copies (cell form: interleaved by bin, a power of two)
  int cshift;       // log2(cpw) (cell form)
  int ncls;         // magnitude classes (1 in the cell form, 3 in the run form)
  int red_off;      // double scratch
  int g_off;        // FP64 prefix sums of the fastest-axis factors (run form)
  size_t bytes;
};

enum SweepKind {
  kSweepPropagate = 0,
  kSweepMoments = 1,
  kSweepBackward = 2,
  kSweepRuns = 3,
  kSweepBwdRuns = 4
};

// run_rows: rows per row-table pass of the run-form propagation (0: the
// default, kRunRowChunk)
bool sweep_layout(const vup_grid& g, int B, SweepKind kind, SweepLayout* out, int run_rows = 0);
GridDev make_grid_dev(const vup_mm& mm);
DistsDev make_dists_dev(const vup_dists& d);

// launches (return hipError_t of the launch)
hipError_t launch_eval_grid(const vup_grid& g, const vup_model& m, double* f, hipStream_t s);
hipError_t launch_uniform_edges(const double* f, int64_t N, int B, double* edges, hipStream_t s);
hipError_t launch_bin(const vup_mm& mm, const double* f, const double* edges, int32_t* bin,
                      hipStream_t s);
hipError_t launch_windows(const vup_grid& g, const vup_dists& d, int32_t* win, hipStream_t s);
hipError_t launch_propagate(const vup_mm& mm, const vup_dists& d, int prec, float* P, double* Z,
                            hipStream_t s);
// FP32 propagation of many single-component pdfs on a 2-D grid by tiles, one
// pdf per lane (model matrices in the run form that tiles_pay). From 16 384
// pdfs on it was faster than the per-pdf kernel at nearly every size, spread
// and deviation measured (sin/cos model, 16 384 and 65 536 pdfs, deviations of 4
// to 8 cells: 256^2 cells 87 -> 55 and 308 -> 117 us, 1024^2 86 -> 75 and 322 ->
// 165, 4096^2 287 -> 110 and 1144 -> 319; of 8.5 to 85 cells: 1024^2 346 -> 218
// and 1232 -> 719; of a tenth to half a cell: 65 536 pdfs 282 -> 181; models
// rising evenly 1.04 to 2.3 times as fast, but for 0.96 and 0.99 where 100
// columns leave a second column of tiles a third full). Fewer pdfs were not
// measured against this form: narrow ones fill fewer batches than the chip
// takes at once.
constexpr long long kPtMinK = VUP_TILED_MIN_K;
// vup_mm.reserved once vup_set_sweep_mode(AUTO) has looked: the tiled
// propagation pays for the model matrix, or not (0: not looked, the device
// decides on each call)
constexpr int kTilesPay = 1, kTilesNot = 2;
// tiles of a 2-D grid, and bytes of the tiled propagation's entries of its model
// matrix
long long tile_count(const vup_grid& g);
void tile_entry_sizes(const vup_grid& g, size_t* ents, size_t* chunks, size_t* blocks);
bool propagate_tiled_applies(const vup_mm& mm, const vup_dists& d, int prec);
size_t propagate_tiled_ws_bytes(const vup_mm& mm, long long K);
// workspace for the fewest passes, and the pdfs of a pass that ws_bytes allow
// (0: too few for the tiles to pay)
size_t propagate_tiled_full_bytes(const vup_mm& mm, long long K);
long long propagate_tiled_pass(const vup_mm& mm, long long K, size_t ws_bytes);
hipError_t launch_propagate_tiled(const vup_mm& mm, const vup_dists& d, long long kg, void* ws,
                                  float* P, double* Z, hipStream_t s);
// the run form for the *kcount distributions klist[0 .. *kcount) (device)
hipError_t launch_propagate_list(const vup_mm& mm, const vup_dists& d, const int* klist,
                                 const int* kcount, float* P, double* Z, hipStream_t s);
hipError_t launch_moments(const vup_mm& mm, const vup_dists& d, const vup_model* model,
                          double* mean, double* var, double* delta2, hipStream_t s);
// moments by tiles of the model values on the matrix cores (2-D grids,
// single-component pdfs, at most 256 tiles of 64 cells per axis)
bool moments_tiled_applies(const vup_mm& mm, const vup_dists& d);
size_t moments_tiled_ws_bytes(const vup_mm& mm, long long K);
hipError_t launch_moments_tiled(const vup_mm& mm, const vup_dists& d, const vup_model* model,
                                void* ws, double* mean, double* var, double* delta2,
                                hipStream_t s);
hipError_t launch_backward(const vup_mm& mm, const vup_dists& d, const float* P,
                           const double* mean_hist, const double* g_var, const double* g_ent,
                           double* g_mu, double* g_sigma, double* g_weight, hipStream_t s);

hipError_t launch_set_mode(const vup_mm& mm, int mode, hipStream_t s);
// the run form of the FP32 propagation applies to this model matrix
bool runs_allowed(const vup_mm& mm);
size_t sep_workspace_bytes(const vup_grid& g, int B, int Mx, int My);
hipError_t launch_separable(const vup_mm& mm, int Mx, int My, const double* mu_x,
                            const double* mu_y, const double* sg_x, const double* sg_y,
                            double ns, int prec, void* ws, float* P, double* Z, hipStream_t s);

// workspace sizing shared by vup_bin_workspace_bytes and vup_bin
struct WsLayout {
  int pitch;
  int64_t rows;
  int64_t nblk;  // chunks of the bin sort
  int chunk;     // padded positions per chunk
  int nseg;      // segments of a row, in the construction of the runs
  size_t off_edges, off_binmap, off_f32, off_counts, off_offsets, off_perm, off_scratch,
      off_counters, off_runs, off_rowptr, off_runidx, off_tsum, off_segs, off_tents, off_tchunks, off_tblocks,
      bytes;
};
bool ws_layout(const vup_grid& g, int B, WsLayout* out);
// exclusive prefix sum of n ints in place; tsum: scan_tiles(n) int64 scratch;
// total (device int) may be null
long long scan_tiles(long long n);
hipError_t launch_scan_excl(int* v, long long n, long long* tsum, int* total, hipStream_t s);

}  // namespace vup
