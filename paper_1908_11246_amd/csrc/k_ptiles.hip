// Propagation (eq. VUP) of many single-component pdfs over a 2-D grid, by
// tiles of the model matrix with one pdf per lane.
//
// The per-pdf run form (k_propagate_runs) gives a workgroup one pdf and its
// lanes the runs of a row: every run costs two random prefix-sum reads and one
// random LDS atomic, and the window, factor tables and row tables are set up
// once per pdf. Here a workgroup takes a batch of 64 pdfs whose windows meet
// one tile of 128 x 64 cells, one pdf per lane. The tile's runs are then the
// same for all lanes: their boundaries are uniform values, and every LDS
// access is at (uniform offset) + 4 lane, free of bank conflicts.
//
// Boundary sweep. Along a row of the tile a run ends where the next begins, so
// with G[c] the prefix sum of a pdf's column factors the mass of the runs
// needs one new prefix sum per run. Four consecutive rows (a chunk) advance
// together: an entry names a bin and the four columns the rows stand at after
// their run of that bin (rows not at that bin stay where they are and add
// nothing); with q = sum_i gx_i G[c_i] after each entry, the bin's mass is the
// step of q. tile_entries (k_ptiles.hpp, part of vup_bin) builds the entries
// of every chunk, once per model matrix: the next bin is the lowest, the
// highest, or that of the row furthest behind, whichever rule gives the chunk
// the fewest entries (rising, falling, other model values along the row). On the sin/cos model at 1024^2 cells and
// 256 bins that is 1.045 row steps per run; eight rows per entry would take
// 1.13 and sixteen 1.26. k_pt_scan lists the pdfs that meet each tile, so a
// batch is full except the last of a list and any order of the pdfs will do.
//
// Numbers. Column factors are formed by the FP64 recurrence g' = g r,
// r' = r q (q = exp(-(h/sigma)^2)), rounded to integers in units of 2^-26 of
// the Gaussian's peak and summed exactly in 32 bits. A row step is one FP64
// FMA: an LDS word read into the low half of a register pair whose high half
// holds the exponent of 2^52 is the double 2^52 + G, without a conversion; the
// 2^52 cancels from the step of q, whose rounding (a few units of gx 2^-26 of
// the peak) is far below the run's mass. The row factors stay FP64 and carry
// the fixed-point scale that makes the pdf's whole mass just below 2^32. An
// entry's step is rounded to an integer and added to its slot with an integer
// LDS atomic, and a tile's slots are added to the row of P, as integers, with
// integer global atomics: exact, so the result does not depend on any order.
// k_pt_final normalises each row by its own total, as the other forms do.
// Column L1 against FP64 at 1024^2 cells: 1.5e-7 (per-pdf form 5.5e-7).
//
// Measured, 65 536 pdfs on 1024^2 cells, 256 bins, deviations of 8.5 to 85
// cells: 1.36 ms per-pdf form, 0.58 ms here (k_pt_main 0.56; k_pt_prep, which
// clears P, k_pt_scan and k_pt_final 0.013, 0.015 and 0.028). k_pt_main issues
// VALU on 0.65 of the cycles and keeps the LDS pipe busy on about half (per
// entry and wave 13 VALU instructions, four 4-byte reads and one atomic);
// lanes whose window covers only part of the tile take 0.33 of the row steps.
// Integer sums with conversions and FP32 FMAs took 24 VALU instructions per
// entry (0.74 ms); one wave per workgroup with its own tables left two waves
// per SIMD (2.2 ms); entries through scalar loads 0.75 ms (the wait for a
// scalar load is a wait for the LDS too); looking for the tile's pdfs inside
// the sweep 0.87 ms; eight columns more per batch or pdfs sorted by deviation
// within 256 no change.
#include <hip/hip_runtime.h>

#include "k_ptiles.hpp"
#include "vup_device.hpp"
#include "vup_internal.hpp"

namespace vup {

namespace {

constexpr int kPY = 128;           // tile rows: two blocks of entries
constexpr unsigned long long kPNoTile = 1ull;  // tile range of a pdf not in the tiles: meets none
constexpr int kPPart = 16384;      // pdfs a list covers (16-bit positions)
constexpr long long kPMaxList = 1ll << 27;  // entries of the lists (16 bits each)
constexpr long long kPMaxBlocks = 65536;
// narrowest pdf, in cells: below it the mass bound is loose (fewer bits left
// for the fixed point); such pdfs are left to the per-pdf kernels
constexpr double kPMinSigma = 0.5;
// factors in units of 2^-26 of the peak: 64 of them stay below 2^32
constexpr double kPUnit = 67108863.0;

struct PtRec {
  uint16_t lo[2], hi[2];  // window
  int k;                  // pdf
  uint32_t pad;
  double t0[2];           // (x of cell 0 - mu) / sigma
  double dt[2];           // h / sigma
  double qq[2];           // exp(-dt^2)
  double scale;           // fixed-point units per unit of gx gy; 0: not in the tiles
};
static_assert(sizeof(PtRec) == 72, "record layout");

struct PtArgs {
  int n[2];
  double lo[2], hi[2];
  const unsigned long long* counters;
  long long K;
  double ns;
  const double* __restrict__ mu;
  const double* __restrict__ sigma;
  int B;
  int ntx, nty;               // tiles
  int nly;                    // blocks of entries along the rows (ntx along the columns)
  const uint2* __restrict__ entries;
  const PtChunk* __restrict__ chunks;
  const PtBlock* __restrict__ blocks;
  PtRec* rec;                 // [K], in the order of k_pt_prep
  unsigned long long* bbox;   // [K] tile range of each record's window
  int parts;                  // lists per tile
  uint16_t* lists;            // [tiles][parts][kPPart] records whose windows meet the tile
  int* counts;                // [tiles][parts] records in each list
  uint32_t* batches;          // list << 8 | batch of the list
  int* state;                 // [0] batches, [1] batches taken by k_pt_main
  uint32_t* none;             // [K] mass in cells without a bin
  int* klist;                 // pdfs left to the per-pdf kernel; [K] holds their number
  float* P;
  double* Z;
};

// exp(a) in FP64 for a up to 700 (0 for very negative a): a = n ln 2 + r, ln 2
// split in a head and a tail (Cody and Waite's argument reduction), and the
// Taylor series of exp(r), |r| <= ln 2 / 2, to degree 11 (truncation below
// 1e-14)
__device__ __forceinline__ double pt_exp(double a) {
  if (a < -745.0) return 0.0;
  const double n = rint(a * 1.4426950408889634);
  double r = fma(-n, 0.6931471805599453, a);
  r = fma(-n, 2.3190468138462996e-17, r);
  double p = 1.0 / 39916800.0;
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, (int)n);
}

// ---------------------------------------------------------------------------
// per pdf: window, fixed-point scale; clears the rows of P
// ---------------------------------------------------------------------------
// upper bound of the sum of the factors of window cells lo .. hi, in cells: a
// unimodal function's sum is at most its integral plus its largest value
__device__ __forceinline__ double mass_bound(double lo, double h, int jlo, int jhi, double mu,
                                             double sigma) {
  const double rs = 0.7071067811865476 / sigma;
  const float ta = (float)((lo + (jlo + 0.5) * h - mu) * rs);
  const float tb = (float)((lo + (jhi + 0.5) * h - mu) * rs);
  // (a pdf so wide that its factors differ by less than the bound's margin: the
  // cells themselves; further out ta and tb would lose their digits)
  if (!(tb - ta > 1e-4f)) return (double)(jhi - jlo + 1);
  const double area = 1.2533141373155003 * sigma / h * (double)(erff(tb) - erff(ta));
  return area * (1.0 + 1e-5) + 1.0;
}

__global__ __launch_bounds__(256) void k_pt_prep(PtArgs a) {
  const long long t0 = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t0 == 0) a.klist[a.K] = a.state[0] = a.state[1] = 0;
  // the rows of P hold integers until k_pt_final; rows of pdfs that are not
  // in the tiles are written whole by the per-pdf kernel
  const long long words = a.K * a.B, step = (long long)gridDim.x * 256;
  uint32_t* Pu = reinterpret_cast<uint32_t*>(a.P);
  if (((uintptr_t)a.P & 15) == 0) {
    uint4* P4 = reinterpret_cast<uint4*>(Pu);
    for (long long i = t0; i < words / 4; i += step) P4[i] = make_uint4(0u, 0u, 0u, 0u);
    for (long long i = words / 4 * 4 + t0; i < words; i += step) Pu[i] = 0u;
  } else {
    for (long long i = t0; i < words; i += step) Pu[i] = 0u;
  }
  const long long k = t0;
  PtRec r = {};
  unsigned long long bb = kPNoTile;
  if (k < a.K) {
    const double mu0 = a.mu[2 * k], mu1 = a.mu[2 * k + 1];
    const double s0 = a.sigma[2 * k], s1 = a.sigma[2 * k + 1];
    int lo0, hi0, lo1, hi1;
    const bool ok0 = axis_window(a.lo[0], a.hi[0], a.n[0], mu0, s0, a.ns, lo0, hi0);
    const bool ok1 = axis_window(a.lo[1], a.hi[1], a.n[1], mu1, s1, a.ns, lo1, hi1);
    const double h0 = (a.hi[0] - a.lo[0]) / a.n[0], h1 = (a.hi[1] - a.lo[1]) / a.n[1];
    // in the tiles: valid pdfs with the mean inside the grid and a deviation
    // of at least kPMinSigma cells (so the mass bound is within a small factor
    // of the mass; invalid, empty and very narrow ones take the per-pdf kernel)
    const bool in = ok0 && ok1 && lo0 <= hi0 && lo1 <= hi1 && mu0 >= a.lo[0] &&
                    mu0 <= a.hi[0] && mu1 >= a.lo[1] && mu1 <= a.hi[1] &&
                    s0 >= kPMinSigma * h0 && s1 >= kPMinSigma * h1;
    r.k = (int)k;
    if (in) {
      r.lo[0] = (uint16_t)lo0;
      r.lo[1] = (uint16_t)lo1;
      r.hi[0] = (uint16_t)hi0;
      r.hi[1] = (uint16_t)hi1;
      const double rs0 = 1.0 / s0, rs1 = 1.0 / s1;
      r.t0[0] = (cell_centre(a.lo[0], a.hi[0], a.n[0], 0) - mu0) * rs0;
      r.t0[1] = (cell_centre(a.lo[1], a.hi[1], a.n[1], 0) - mu1) * rs1;
      r.dt[0] = h0 * rs0;
      r.dt[1] = h1 * rs1;
      r.qq[0] = pt_exp(-r.dt[0] * r.dt[0]);
      r.qq[1] = pt_exp(-r.dt[1] * r.dt[1]);
      const double m = mass_bound(a.lo[0], h0, lo0, hi0, mu0, s0) *
                       mass_bound(a.lo[1], h1, lo1, hi1, mu1, s1);
      // every entry of the tiles it meets rounds by at most half a unit
      const double ent = (double)((lo1 / kPX - hi1 / kPX - 1) * (lo0 / kPY - hi0 / kPY - 1)) *
                         (2 * kPCh * kPEnt);
      r.scale = (4294967296.0 - 1048576.0 - ent) / (m * (1.0 + 1.0 / 65536));
      bb = (unsigned long long)(lo1 / kPX) | ((unsigned long long)(hi1 / kPX) << 16) |
           ((unsigned long long)(lo0 / kPY) << 32) | ((unsigned long long)(hi0 / kPY) << 48);
    }
    a.none[k] = 0u;
    a.rec[k] = r;
    a.bbox[k] = bb;
  }
}

// ---------------------------------------------------------------------------
// per (tile, part of the records): the records whose windows meet the tile
// ---------------------------------------------------------------------------
constexpr int kPScan = 512;  // threads

__global__ __launch_bounds__(kPScan) void k_pt_scan(PtArgs a) {
  __shared__ int wcnt[2][kPScan / 64];
  __shared__ int first;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int part = blockIdx.x % a.parts, tile = blockIdx.x / a.parts;
  const int tx = tile % a.ntx, ty = tile / a.ntx;
  const int kbeg = part * kPPart, kend = (int)min((long long)kbeg + kPPart, a.K);
  // the entries are used when they fit and their row steps are at most three
  // times the model matrix's runs; otherwise the per-pdf kernel takes all pdfs
  const bool use = tiles_pay(a.counters[kCntTiles], a.counters[kCntRuns]);
  if (tile == 0 && !use) {
    for (int k = kbeg + threadIdx.x; k < kend; k += kPScan) {
      a.rec[k].scale = 0.0;
      a.klist[k] = k;
    }
    if (part == 0 && threadIdx.x == 0) a.klist[a.K] = (int)a.K;
  }
  int n = 0;
  if (use) {
    uint16_t* list = a.lists + (long long)blockIdx.x * kPPart;
    // four records per thread and step, the next step's in flight
    auto range = [&](int k) { return k < kend ? a.bbox[k] : kPNoTile; };
    unsigned long long nx[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) nx[u] = range(kbeg + u * kPScan + threadIdx.x);
    for (int k0 = kbeg, odd = 0; k0 < kend; k0 += 4 * kPScan, odd ^= 1) {
      unsigned long long m[4];
      bool hit[4];
      int c = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned long long bb = nx[u];
        hit[u] = tx >= (int)(bb & 0xFFFFu) && tx <= (int)((bb >> 16) & 0xFFFFu) &&
                 ty >= (int)((bb >> 32) & 0xFFFFu) && ty <= (int)(bb >> 48);
        m[u] = __ballot(hit[u]);
        c += __popcll(m[u]);
        const int k = k0 + u * kPScan + (int)threadIdx.x;
        if (tile == 0 && bb == kPNoTile && k < kend)
          a.klist[atomicAdd(&a.klist[a.K], 1)] = k;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) nx[u] = range(k0 + (4 + u) * kPScan + threadIdx.x);
      if (lane == 0) wcnt[odd][w] = c;
      __syncthreads();
      int off = n;
#pragma unroll
      for (int v = 0; v < kPScan / 64; ++v) {
        if (v < w) off += wcnt[odd][v];
        n += wcnt[odd][v];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (hit[u])
          list[off + __popcll(m[u] & ((1ull << lane) - 1ull))] =
              (uint16_t)(k0 - kbeg + u * kPScan + threadIdx.x);
        off += __popcll(m[u]);
      }
    }
  }
  // its batches of 64 records, wherever they fall among the others'
  const int nb = (n + 63) / 64;
  if (threadIdx.x == 0) {
    a.counts[blockIdx.x] = n;
    first = nb > 0 ? atomicAdd(&a.state[0], nb) : 0;
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += kPScan)
    a.batches[first + b] = (uint32_t)blockIdx.x << 8 | (uint32_t)b;
}

// ---------------------------------------------------------------------------
// per batch (64 pdfs of a tile's lists, one per lane): four waves; wave w forms the prefix sums of columns 16 w .. 16 w + 15 and sweeps
// rows 16 w .. 16 w + 15
// ---------------------------------------------------------------------------
// bit j of a lane's mask as 0 or -1
__device__ __forceinline__ uint32_t bit_mask(uint32_t m, int j) {
  return (uint32_t)__builtin_amdgcn_sbfe((int)m, j, 1);
}

constexpr int kPWaves = 4;
constexpr int kPWCols = kPX / kPWaves;            // columns of a wave
constexpr int kPWRows = kPY / kPWaves;            // rows of a wave
constexpr int kPWCh = kPWRows / kPR;              // chunks of a wave
static_assert(kPWCh * kPWaves == 2 * kPCh && kPWRows == 32, "a wave's rows lie in one block");

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(256, 4) void k_pt_main(PtArgs a) {
  __shared__ uint32_t sG[(kPX + 1) * 64];        // [column][lane] prefix sums
  // [slot][lane xor slot] sums; slot kPSlots: cells without a bin, then a
  // slot for bins outside the pass
  __shared__ uint32_t sH[(kPSlots + 2) * 64];
  __shared__ uint32_t sOff[64];                  // rows of P of the batch (element offsets)
  __shared__ uint32_t wtot[kPWaves][64];
  __shared__ int snext;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane4 = 4u * (uint32_t)lane;
  // byte n of a word over the lane's byte offset: v_perm_b32 selectors, kept
  // in vector registers (an instruction reads one scalar register)
  uint32_t sel0 = 0x0c0c0400u, sel1 = 0x0c0c0500u, sel2 = 0x0c0c0600u, sel3 = 0x0c0c0700u;
  asm("" : "+v"(sel0), "+v"(sel1), "+v"(sel2), "+v"(sel3));
  uint32_t two52 = 0x43300000u;  // high word of 2^52 (kept from the optimiser)
  asm("" : "+v"(two52));
  if (w == 0) sG[lane] = 0u;
  for (int i = threadIdx.x; i < (kPSlots + 2) * 64; i += 256) sH[i] = 0u;
  uint32_t* Pu = reinterpret_cast<uint32_t*>(a.P);
  // workgroups take batches until none is left: the first by their index, the
  // next ones from a counter
  const int nbatches = a.state[0];
  int id = blockIdx.x;
  while (id < nbatches) {
  const uint32_t desc = a.batches[id];
  const int list = (int)(desc >> 8), tile = list / a.parts;
  const int tx = tile % a.ntx, ty = tile / a.ntx;
  const int c0 = tx * kPX + kPWCols * w, r0 = ty * kPY + kPWRows * w;  // of the wave
  // the wave's chunks and the tile's bins (its two blocks of lists)
  const int ly = 2 * ty + w / 2;
  const long long blk = (long long)ly * a.ntx + tx;
  const bool have = ly < a.nly;
  const PtChunk* cs = a.chunks + blk * kPCh + kPWCh * (w & 1);
  int tmn, tmx, tnone;
  {
    const PtBlock b0 = a.blocks[(long long)(2 * ty) * a.ntx + tx];
    tmn = b0.mn;
    tmx = b0.mx;
    tnone = b0.none;
    if (2 * ty + 1 < a.nly) {
      const PtBlock b1 = a.blocks[(long long)(2 * ty + 1) * a.ntx + tx];
      tmn = min(tmn, b1.mn);
      tmx = max(tmx, b1.mx);
      tnone |= b1.none;
    }
  }
  // passes over the tile's bins, kPSlots at a time (nearly always one)
  const int passes = tmx >= tmn ? (tmx - tmn) / kPSlots + 1 : 1;

  {
    PtRec r;
    {
      const int at = (int)(desc & 0xFFu) * 64 + lane;
      const bool in = at < a.counts[list];
      r = a.rec[(list % a.parts) * kPPart + (in ? a.lists[(long long)list * kPPart + at] : 0)];
      if (!in) r.k = -1;
    }
    const int k = r.k;
    const bool valid = k >= 0;
    int after = 0;
    if (threadIdx.x == 0) after = (int)gridDim.x + atomicAdd(&a.state[1], 1);
    uint32_t cmask = 0u, rmask = 0u;  // of the wave's columns and rows
    if (valid) {
      // bits of j in [lo, hi] among first .. first + len - 1
      auto bits = [](int lo, int hi, int first, int len) {
        const int x = max(lo - first, 0), y = min(hi - first, len - 1);
        return x <= y ? (0xFFFFFFFFu >> (31 - y)) & (0xFFFFFFFFu << x) : 0u;
      };
      cmask = bits(r.lo[1], r.hi[1], c0, kPWCols);
      rmask = bits(r.lo[0], r.hi[0], r0, kPWRows);
    }
    const double dt0 = r.dt[0], dt1 = r.dt[1];
    const double ty0 = fma((double)r0, dt0, r.t0[0]), tx0 = fma((double)c0, dt1, r.t0[1]);
    const double S0 = r.scale * (1.0 / kPUnit);  // row factors carry the fixed-point scale
    // The recurrences start at the wave's first row and column, which may lie
    // outside the window, n dt deviations further out (n = 15 columns, 31
    // rows). A start beyond t = 37 is 0 in FP64 and stays 0; that loses nothing
    // while n dt <= 30, since factors beyond t = 7 are below the units used.
    // dt <= 2 (kPMinSigma), so the columns are safe, and the rows when they
    // start again half way.
    static_assert((kPWCols - 1) / kPMinSigma <= 30 && (kPWRows / 2 - 1) / kPMinSigma <= 30, "range");
    const bool restart = __any(valid && (kPWRows - 1) * dt0 > 30.0);
    uint32_t G[kPWCols], sum = 0u;
    {
      double g = kPUnit * pt_exp(-0.5 * tx0 * tx0);
      double q = pt_exp(fmin(-(tx0 + 0.5 * dt1) * dt1, 700.0));
      const double qq = r.qq[1];
#pragma unroll
      for (int c = 0; c < kPWCols; ++c) {
        // + 2^52: the low word is g rounded to an integer
        const uint32_t u = (uint32_t)__double_as_longlong(g + 4503599627370496.0);
        sum += u & bit_mask(cmask, c);
        G[c] = sum;
        g *= q;
        q *= qq;
      }
    }
    wtot[w][lane] = sum;
    __syncthreads();  // the last batch's readers of sG, sH, sOff and snext are done
    if (threadIdx.x == 0) snext = after;
    uint32_t before = 0u;
#pragma unroll
    for (int v = 0; v < kPWaves - 1; ++v) before += v < w ? wtot[v][lane] : 0u;
#pragma unroll
    for (int c = 0; c < kPWCols; ++c) sG[(kPWCols * w + c + 1) * 64 + lane] = before + G[c];
    if (w == 0) sOff[lane] = (uint32_t)(valid ? k : 0) * (uint32_t)a.B;
    __syncthreads();
    for (int ps = 0; ps < passes; ++ps) {
      const int base = tmn + ps * kPSlots;
      if (have) {
        double g = S0 * pt_exp(-0.5 * ty0 * ty0);
        double q = pt_exp(fmin(-(ty0 + 0.5 * dt0) * dt0, 700.0));
        const double qq = r.qq[0];
        uint32_t rm = rmask;
        // buffers of prefix sums as doubles 2^52 + G: only the low words change
        u32x2 A[2 * kPR], Bf[2 * kPR];
#pragma unroll
        for (int j = 0; j < 2 * kPR; ++j) {
          A[j][0] = Bf[j][0] = 0u;
          A[j][1] = Bf[j][1] = two52;
        }
        int cn = __builtin_amdgcn_readfirstlane(cs[0].n);
        const uint2* ev = a.entries + __builtin_amdgcn_readfirstlane(cs[0].first);
        uint2 ent = ev[lane];  // (there are 64 entries more than the model matrix has)
#pragma unroll 1
        for (int ch = 0; ch < kPWCh; ++ch) {
          if (restart && ch == kPWCh / 2) {
            const double t = fma((double)(kPWRows / 2), dt0, ty0);
            g = S0 * pt_exp(-0.5 * t * t);
            q = pt_exp(fmin(-(t + 0.5 * dt0) * dt0, 700.0));
          }
          double gx[kPR];
#pragma unroll
          for (int i = 0; i < kPR; ++i) {
            const long long b = __double_as_longlong(g);
            const uint32_t on = bit_mask(rm, i);
            gx[i] = __hiloint2double((int)((uint32_t)(b >> 32) & on), (int)((uint32_t)b & on));
            g *= q;
            q *= qq;
          }
          const bool any = __any((rm & 15u) != 0u);
          rm >>= kPR;
          const int n = cn;
          const uint2* here = ev;
          const uint2 first = ent;
          if (ch + 1 < kPWCh) {  // the next chunk's
            cn = __builtin_amdgcn_readfirstlane(cs[ch + 1].n);
            ev = a.entries + __builtin_amdgcn_readfirstlane(cs[ch + 1].first);
            ent = ev[lane];
          }
          if (!any) continue;  // no pdf of the batch has these rows
          // the sum at G = 0, by add()'s operations in add()'s order: an entry
          // that moves no row over mass then gives exactly 0
          double last = gx[0] * 4503599627370496.0;
#pragma unroll
          for (int j = 1; j < kPR; ++j) last = __builtin_fma(gx[j], 4503599627370496.0, last);
          for (int f = 0; f < n; f += 64) {
            const int m = min(64, n - f);  // even
            uint2 e = first;
            if (f) e = here[f + min(lane, m - 1)];
            uint32_t slot = e.y >> 16;
            if (passes > 1) {  // bins outside the pass go to the last slot
              const uint32_t b = e.y & 0xFFFFu;
              if (b == (uint32_t)kPNoBin ? ps > 0 : b - (uint32_t)base >= (uint32_t)kPSlots)
                slot = slot_code(kPSlots + 1);
            }
            auto load = [&](int i, u32x2 (&o)[2 * kPR]) {
              const uint32_t cols[2] = {(uint32_t)__builtin_amdgcn_readlane((int)e.x, i),
                                        (uint32_t)__builtin_amdgcn_readlane((int)e.x, i + 1)};
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const uint32_t c = cols[u];
                const char* p = reinterpret_cast<const char*>(sG);
                o[4 * u][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel0));
                o[4 * u + 1][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel1));
                o[4 * u + 2][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel2));
                o[4 * u + 3][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel3));
              }
            };
            auto add = [&](int i, const u32x2 (&o)[2 * kPR]) {
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                double sum = gx[0] * __builtin_bit_cast(double, o[4 * u]);
#pragma unroll
                for (int j = 1; j < kPR; ++j)
                  sum = __builtin_fma(gx[j], __builtin_bit_cast(double, o[4 * u + j]), sum);
                const uint32_t v =
                    (uint32_t)__double_as_longlong((sum - last) + 6755399441055744.0);
                last = sum;
                const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)slot, i + u);
                uint32_t* h = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(sH) + (at ^ lane4));
                __hip_atomic_fetch_add(h, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              }
            };
            // two entries at a time, the reads of the next two in flight
            load(0, A);
            for (int i = 0;; i += 4) {
              const bool more = i + 2 < m, more2 = i + 4 < m;
              if (more) load(i + 2, Bf);
              __builtin_amdgcn_sched_barrier(0);
              add(i, A);
              if (!more) break;
              if (more2) load(i + 4, A);
              __builtin_amdgcn_sched_barrier(0);
              add(i + 2, Bf);
              if (!more2) break;
            }
          }
        }
      }
      __syncthreads();
      if (ps == 0) id = __builtin_amdgcn_readfirstlane(snext);
      // add the slots of bins base .. to the rows of P and clear them: 32 (or
      // 64) lanes a pdf, so a pdf's bins are contiguous. Lanes without a pdf
      // hold zeros.
      const int span = min(tmx - base + 1, kPSlots);
      const int b0 = base % kPSlots;  // slot of the pass's first bin
      auto give = [&](int b, int p) {  // bin base + b of pdf p
        const int s = b0 + b < kPSlots ? b0 + b : b0 + b - kPSlots;
        const int at = s * 64 + (p ^ (s & 63));
        const uint32_t v = sH[at], o = sOff[p] + (uint32_t)(base + b);
        sH[at] = 0u;
        // (a slot without mass may hold a few units of negative rounding noise)
        if (v - 1u < 0xFFF80000u && b < span) __hip_atomic_fetch_add(&Pu[o], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      if (span > 32) {
#pragma unroll 4
        for (int i = 0; i < 16; ++i) give(lane, 4 * i + w);
        if (span > 64) {
          // the last slots: 16 lanes a pdf
          static_assert(kPSlots <= 80, "16 slots after the first 64");
          if (64 + (lane & 15) < span)
#pragma unroll
            for (int i = 0; i < 4; ++i) give(64 + (lane & 15), 16 * i + 4 * w + (lane >> 4));
        }
      } else {
#pragma unroll 4
        for (int i = 0; i < 8; ++i) give(lane & 31, 8 * i + 2 * w + (lane >> 5));
      }
      if (ps + 1 < passes) __syncthreads();
    }
    if (tnone && w == 0) {
      const int at = kPSlots * 64 + (lane ^ (kPSlots & 63));
      const uint32_t v = sH[at];
      sH[at] = 0u;
      if (valid && v - 1u < 0xFFF80000u)
        __hip_atomic_fetch_add(&a.none[k], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  }
}

// ---------------------------------------------------------------------------
// per pdf: normalise the row of integers by its total; a wave per row
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pt_final(PtArgs a) {
  const int lane = threadIdx.x & 63;
  const long long at = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (at >= a.K) return;
  const double scale = a.rec[at].scale;
  const long long k = a.rec[at].k;
  if (!(scale > 0.0)) return;  // the per-pdf kernel's row
  const uint32_t* u = reinterpret_cast<const uint32_t*>(a.P) + k * a.B;
  float* p = a.P + k * a.B;
  double sum = 0.0;
  if (a.B <= 256) {
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = lane + 64 * i < a.B ? u[lane + 64 * i] : 0u;
      sum += (double)v[i];
    }
    const double tot = wave_sum(sum) + (double)a.none[k];
    const double f = 1.0 / tot;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (lane + 64 * i < a.B) p[lane + 64 * i] = (float)((double)v[i] * f);
    if (a.Z && lane == 0) a.Z[k] = tot / scale;
    return;
  }
  for (int b = lane; b < a.B; b += 64) sum += (double)u[b];
  const double tot = wave_sum(sum) + (double)a.none[k];
  const double f = 1.0 / tot;
  for (int b = lane; b < a.B; b += 64) p[b] = (float)((double)u[b] * f);
  if (a.Z && lane == 0) a.Z[k] = tot / scale;
}

constexpr size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct PtLayout {
  size_t rec, bbox, lists, counts, batches, state, none, klist, bytes;
};

PtLayout pt_layout(long long ntiles, long long K) {
  const long long nlists = ntiles * ((K + kPPart - 1) / kPPart);
  PtLayout L;
  L.rec = 0;
  L.bbox = L.rec + al256((size_t)K * sizeof(PtRec));
  L.lists = L.bbox + al256((size_t)K * 8);
  L.counts = L.lists + al256((size_t)nlists * kPPart * 2);
  L.batches = L.counts + al256((size_t)nlists * 4);
  L.state = L.batches + al256((size_t)nlists * (kPPart / 64) * 4);
  L.none = L.state + 256;
  L.klist = L.none + al256((size_t)K * 4);
  L.bytes = L.klist + al256((size_t)(K + 1) * 4);
  return L;
}

int pt_div(int n, int m) { return (n + m - 1) / m; }

// blocks of lists of a grid
long long pt_blocks(const vup_mm& mm) {
  return (long long)pt_div(mm.grid.n[1], kPX) * pt_div(mm.grid.n[0], kPL);
}

long long pt_tiles(const vup_mm& mm) {
  return (long long)pt_div(mm.grid.n[1], kPX) * pt_div(mm.grid.n[0], kPY);
}

}  // namespace

// 8 bytes per ten cells: the entries of model matrices with runs of three
// cells or more; 64 more are read past the last
void tile_entry_sizes(const vup_grid& g, size_t* ents, size_t* chunks, size_t* blocks) {
  const long long nb = (long long)pt_div(g.n[1], kPX) * pt_div(g.n[0], kPL);
  *ents = (size_t)(((long long)g.n[0] * g.n[1] / 10 + 64) * sizeof(uint2));
  *chunks = (size_t)nb * kPCh * sizeof(PtChunk);
  *blocks = (size_t)nb * sizeof(PtBlock);
}

bool propagate_tiled_applies(const vup_mm& mm, const vup_dists& d, int prec) {
  if (mm.grid.ndim != 2 || d.ncomp != 1 || prec != VUP_FP32) return false;
  if (mm.sweep != VUP_SWEEP_RUNS || !runs_allowed(mm) || mm.reserved == kTilesNot) return false;
  return d.K >= kPtMinK && d.K < (1ll << 24) && d.K * mm.B < (1ll << 30) && mm.N < (1ll << 28) &&
         pt_blocks(mm) <= kPMaxBlocks &&
         pt_tiles(mm) * pt_div((int)d.K, kPPart) * kPPart <= kPMaxList;
}

size_t propagate_tiled_ws_bytes(const vup_mm& mm, long long K) {
  return pt_layout(pt_tiles(mm), K).bytes;
}

hipError_t launch_propagate_tiled(const vup_mm& mm, const vup_dists& d, void* ws, float* P,
                                  double* Z, hipStream_t s) {
  PtArgs a{};
  for (int i = 0; i < 2; ++i) {
    a.n[i] = mm.grid.n[i];
    a.lo[i] = mm.grid.lo[i];
    a.hi[i] = mm.grid.hi[i];
  }
  const char* mws = static_cast<const char*>(mm.ws);
  WsLayout W;
  ws_layout(mm.grid, mm.B, &W);
  a.entries = reinterpret_cast<const uint2*>(mws + W.off_tents);
  a.chunks = reinterpret_cast<const PtChunk*>(mws + W.off_tchunks);
  a.blocks = reinterpret_cast<const PtBlock*>(mws + W.off_tblocks);
  a.counters = reinterpret_cast<const unsigned long long*>(mws + mm.off_counters);
  a.K = d.K;
  a.ns = d.n_sigma;
  a.mu = d.mu;
  a.sigma = d.sigma;
  a.B = mm.B;
  a.ntx = pt_div(a.n[1], kPX);
  a.nty = pt_div(a.n[0], kPY);
  a.nly = pt_div(a.n[0], kPL);
  const long long ntiles = pt_tiles(mm);
  a.parts = (int)((d.K + kPPart - 1) / kPPart);
  const PtLayout L = pt_layout(ntiles, d.K);
  char* base = static_cast<char*>(ws);
  a.rec = reinterpret_cast<PtRec*>(base + L.rec);
  a.bbox = reinterpret_cast<unsigned long long*>(base + L.bbox);
  a.lists = reinterpret_cast<uint16_t*>(base + L.lists);
  a.counts = reinterpret_cast<int*>(base + L.counts);
  a.batches = reinterpret_cast<uint32_t*>(base + L.batches);
  a.state = reinterpret_cast<int*>(base + L.state);
  a.none = reinterpret_cast<uint32_t*>(base + L.none);
  a.klist = reinterpret_cast<int*>(base + L.klist);
  a.P = P;
  a.Z = Z;
  const long long pb = (d.K + 255) / 256;
  hipLaunchKernelGGL(k_pt_prep, dim3((unsigned)(pb > 2048 ? pb : 2048)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_pt_scan, dim3((unsigned)(ntiles * a.parts)), dim3(kPScan), 0, s, a);
  // as many workgroups as fit on the GPU (four per CU)
  hipLaunchKernelGGL(k_pt_main, dim3(1024), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_pt_final, dim3((unsigned)((d.K + 3) / 4)), dim3(256), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_propagate_list(mm, d, a.klist, a.klist + d.K, P, Z, s);
}

}  // namespace vup
