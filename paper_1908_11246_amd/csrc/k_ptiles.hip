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
// nothing); the bin's mass is sum_i gx_i times row i's step of G. tile_entries
// (k_ptiles.hpp, part of vup_bin) builds the entries of every chunk, once per
// model matrix: the next bin is the lowest, the highest, or that of the row
// furthest behind, whichever rule gives the chunk the fewest entries (rising,
// falling, other model values along the row). On the sin/cos model at 1024^2
// cells and 256 bins that is 1.15 row steps per run. k_pt_scan lists the pdfs
// that meet each tile, so a batch is full except the last of a list and any
// order of the pdfs will do.
//
// Numbers. Column factors are formed by the FP64 recurrence g' = g r,
// r' = r q (q = exp(-(h/sigma)^2)), in units of the tile's largest factor,
// rounded to integers of 2^-25 of that or finer and summed exactly in 32 bits.
// An LDS word read into the low half of a register pair whose high half holds
// the exponent of 2^52 is the double 2^52 + G, without a conversion, and the
// difference of two of them is a row's step, exact. The row factors stay FP64
// and carry the fixed-point scale that makes the pdf's whole mass 2^51 at most.
// An entry's mass is rounded to that (adding 2^52 puts it into the low 52 bits
// of the double) and added to its slot with a 64-bit integer LDS atomic; a
// tile's slots are added, as integers, to the pdf's 64-bit sums with global
// atomics: exact, so the result does not depend on any order. k_pt_final
// divides each pdf's sums by their total. So a bin's digits do not depend on
// the other bins' mass: against FP64 at 1024^2 cells, deviations of 8.5 to 85
// cells, the bins' relative errors are (median, 99th percentile; per-pdf form
// in brackets) 2e-8, 5e-8 (6e-8, 1e-6) above a thousandth of the mass, 3e-8,
// 2e-6 (5e-5, 2e-3) around 1e-6, 7e-7, 1e-5 (6e-3, 9e-2) around 1e-10; columns'
// L1 error 2.1e-8 (6.4e-8). Sums in 32 bits of the whole mass lost bins below
// 1e-10 altogether.
//
// Measured, 65 536 pdfs on 1024^2 cells, 256 bins, deviations of 8.5 to 85
// cells: 1.23 ms per-pdf form, 0.71 ms here (k_pt_main 0.64; k_pt_prep, which
// clears the sums, k_pt_scan and k_pt_final 0.022, 0.017 and 0.035). k_pt_main
// is bound by the LDS pipe, with VALU issue close behind (per entry and wave
// four 4-byte reads of 5 clocks and an atomic of 8, measured alone, 15 VALU
// instructions, eight of them FP64). With 32-bit sums (running sums over the
// four rows, 13 VALU instructions, an atomic of 5.5 clocks) 0.58 ms. Workgroups of four waves and 66
// bins, three to a CU: 0.77 ms, 0.57 instead of 0.42 where tiles need two
// passes; 42 bins, four to a CU, 0.84; two pairs of entries and a copy of the
// last instead of the ring 0.72; an entry's mass rounded once, after a chain of
// multiply-adds from 0, 0.02 ms more, slots read one entry at a time 0.01.
// Integer sums with conversions and FP32 FMAs took 24 VALU instructions per
// entry; one wave per workgroup with its own tables left two waves per SIMD
// (2.2 ms); entries through scalar loads were slower (the wait for a scalar
// load is a wait for the LDS too), and so was looking for the tile's pdfs
// inside the sweep.
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
// fixed-point mass of a pdf (at most), and the bits of a sum: the words added
// to it are doubles 2^52 + v, whose other bits a sum of v below 2^52 leaves alone
constexpr double kPMass = 2251799813685248.0;
constexpr unsigned long long kPSum = (1ull << 52) - 1ull;
// recurrences step by at most so many deviations, from so far out (t^2 / 2)
constexpr double kPMaxStep = 1.0, kPMaxOff = 450.0;
// -log of a pdf's largest density, in units of its peak
constexpr double kPMaxExp = 700.0;

struct PtRec {
  uint16_t lo[2], hi[2];  // window
  int k;                  // pdf
  uint32_t pad;
  double t0[2];           // (x of the window's first cell - mu) / sigma
  double dt[2];           // h / sigma
  double e[2];            // t^2 / 2 of the window's cell nearest the mean
  double scale;           // fixed-point units per unit of gx gy e^(e[0] + e[1]); 0: not in the tiles
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
  unsigned long long* acc;    // [K][B + 1] fixed-point mass of each bin and of the cells without
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
// per pdf: window, fixed-point scale; clears the sums
// ---------------------------------------------------------------------------
// e - t^2 / 2, exactly 0 where e is that t^2 / 2
__device__ __forceinline__ double pt_arg(double e, double t) {
#pragma clang fp contract(off)
  return e - 0.5 * (t * t);
}

// one axis of a pdf's record
__device__ __forceinline__ void pt_axis(PtRec& r, int d, double lo, double hi, int n, int jlo,
                                        int jhi, double mu, double sigma) {
  const double h = (hi - lo) / n, rs = 1.0 / sigma;
  double c = floor((mu - lo) / h);
  c = c >= (double)jlo ? c : (double)jlo;
  c = c <= (double)jhi ? c : (double)jhi;
  r.lo[d] = (uint16_t)jlo;
  r.hi[d] = (uint16_t)jhi;
  r.t0[d] = (cell_centre(lo, hi, n, jlo) - mu) * rs;
  r.dt[d] = h * rs;
  r.e[d] = -pt_arg(0.0, fma(c - jlo, r.dt[d], r.t0[d]));
}

// Upper bound of the sum of a window's factors in units of its largest one, for
// W of its cells: on either side of the mean they fall from at most 1, so they
// add up to at most 1 and the integral from there on (Mills' ratio: at most
// sqrt(pi / 2) deviations).
__device__ __forceinline__ double mass_bound(int W, double dt) {
  return fmin((double)W, 2.0 + 2.5066282746310007 / dt);
}

__global__ __launch_bounds__(256) void k_pt_prep(PtArgs a) {
  const long long t0 = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t0 == 0) a.klist[a.K] = a.state[0] = a.state[1] = 0;
  const long long words = a.K * (a.B + 1), step = (long long)gridDim.x * 256;
  ulonglong2* acc2 = reinterpret_cast<ulonglong2*>(a.acc);
  for (long long i = t0; i < words / 2; i += step) acc2[i] = make_ulonglong2(0ull, 0ull);
  if (t0 == 0 && (words & 1)) a.acc[words - 1] = 0ull;
  const long long k = t0;
  PtRec r = {};
  unsigned long long bb = kPNoTile;
  if (k < a.K) {
    const double mu0 = a.mu[2 * k], mu1 = a.mu[2 * k + 1];
    const double s0 = a.sigma[2 * k], s1 = a.sigma[2 * k + 1];
    int lo0, hi0, lo1, hi1;
    const bool ok0 = axis_window(a.lo[0], a.hi[0], a.n[0], mu0, s0, a.ns, lo0, hi0);
    const bool ok1 = axis_window(a.lo[1], a.hi[1], a.n[1], mu1, s1, a.ns, lo1, hi1);
    r.k = (int)k;
    // in the tiles: all but invalid pdfs, empty windows and densities at the end
    // of FP64's range (or past it), which take the per-pdf kernel
    const bool in = ok0 && ok1 && lo0 <= hi0 && lo1 <= hi1;
    if (in) {
      pt_axis(r, 0, a.lo[0], a.hi[0], a.n[0], lo0, hi0, mu0, s0);
      pt_axis(r, 1, a.lo[1], a.hi[1], a.n[1], lo1, hi1, mu1, s1);
    }
    if (in && r.e[0] + r.e[1] <= kPMaxExp) {
      r.scale = kPMass / (mass_bound(hi0 - lo0 + 1, r.dt[0]) * mass_bound(hi1 - lo1 + 1, r.dt[1]));
      bb = (unsigned long long)(lo1 / kPX) | ((unsigned long long)(hi1 / kPX) << 16) |
           ((unsigned long long)(lo0 / kPY) << 32) | ((unsigned long long)(hi0 / kPY) << 48);
    }
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
  // otherwise the per-pdf kernel takes all pdfs
  const bool use = tiles_pay(a.counters[kCntTiles], a.counters[kCntRuns], a.counters[kCntPasses],
                             a.ntx * a.nty);
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
// per batch (64 pdfs of a tile's lists, one per lane): eight waves; wave w
// forms the prefix sums of columns 8 w .. 8 w + 7 and sweeps rows 16 w ..
// 16 w + 15. Eight waves share the sums of 120 bins: two workgroups to a CU,
// four waves per SIMD, and tiles of 120 bins in one pass.
// ---------------------------------------------------------------------------
// bit j of a lane's mask as 0 or -1
__device__ __forceinline__ uint32_t bit_mask(uint32_t m, int j) {
  return (uint32_t)__builtin_amdgcn_sbfe((int)m, j, 1);
}

constexpr int kPWaves = 8;
constexpr int kPWCols = kPX / kPWaves;            // columns of a wave
constexpr int kPWRows = kPY / kPWaves;            // rows of a wave
constexpr int kPWCh = kPWRows / kPR;              // chunks of a wave
static_assert(kPWCh * kPWaves == 2 * kPCh && kPL % kPWRows == 0, "a wave's rows lie in one block");

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(64 * kPWaves, 4) void k_pt_main(PtArgs a) {
  __shared__ uint32_t sG[(kPX + 1) * 64];        // [column][lane] prefix sums
  // [slot][lane xor slot] sums; slot kPSlots: cells without a bin, then a
  // slot for bins outside the pass
  __shared__ unsigned long long sH[(kPSlots + 2) * 64];
  __shared__ uint32_t sOff[64];                  // the batch's rows of sums (element offsets)
  __shared__ uint32_t wtot[kPWaves][64];
  __shared__ int snext;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane4 = 4u * (uint32_t)lane, lane8 = 8u * (uint32_t)lane;
  // byte n of a word over the lane's byte offset: v_perm_b32 selectors, kept
  // in vector registers (an instruction reads one scalar register)
  uint32_t sel0 = 0x0c0c0400u, sel1 = 0x0c0c0500u, sel2 = 0x0c0c0600u, sel3 = 0x0c0c0700u;
  asm("" : "+v"(sel0), "+v"(sel1), "+v"(sel2), "+v"(sel3));
  uint32_t two52 = 0x43300000u;  // high word of 2^52 (kept from the optimiser)
  asm("" : "+v"(two52));
  if (w == 0) sG[lane] = 0u;
  for (int i = threadIdx.x; i < (kPSlots + 2) * 64; i += 64 * kPWaves) sH[i] = 0ull;
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
  const int ly = 2 * ty + w / (kPWaves / 2);
  const long long blk = (long long)ly * a.ntx + tx;
  const bool have = ly < a.nly;
  const PtChunk* cs = a.chunks + blk * kPCh + kPWCh * (w & (kPWaves / 2 - 1));
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
  const int passes = tile_passes(tmn, tmx);

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
    // A factor is formed as exp(e - t^2 / 2), the row's with e of the window's
    // cell nearest the mean, the column's with that of the tile's: both are at
    // most 1, and what the column's exceed the window's by, exp(e[1] - ec),
    // goes to the row factors, with the fixed-point scale.
    const int ca = max((int)r.lo[1], tx * kPX), cb = min((int)r.hi[1], tx * kPX + kPX - 1);
    const double ta = fma((double)(ca - r.lo[1]), dt1, r.t0[1]);
    const double tb = fma((double)(cb - r.lo[1]), dt1, r.t0[1]);
    const double ec = ta >= 0.0 ? -pt_arg(0.0, ta) : tb <= 0.0 ? -pt_arg(0.0, tb) : r.e[1];
    const double er = r.e[1] - ec;
    // The columns' unit 2^-cexp: the finest power of two (so that the row
    // factors can undo it exactly) with their sum's bound below 2^32. (The bound
    // in FP32 is at least an ulp below a power of two or at it, so the 64 halves
    // of a unit that rounding may add stay within 32 bits.)
    const float cmass = fminf((float)(cb - ca + 1), 2.0001f + 2.5067f * __builtin_amdgcn_rcpf((float)dt1));
    const int cexp = 32 - __builtin_amdgcn_frexp_expf(cmass);
    const double S0 = ldexp(r.scale, -cexp), unit = ldexp(1.0, cexp);
    const double ty0 = fma((double)(r0 - r.lo[0]), dt0, r.t0[0]);
    const double tx0 = fma((double)(c0 - r.lo[1]), dt1, r.t0[1]);
    // The recurrences start at the wave's first row and column, which may lie
    // outside the window, n dt deviations further out (7 columns, 15 rows). A
    // factor e^-36 below the largest is below the units used; one that counts
    // has a start above e^-620 while n dt <= 16 and e <= kPMaxOff, so it is
    // never lost to underflow. Pdfs narrower than a cell, and means far outside
    // the grid, have each of their factors formed by itself (with the t of
    // k_pt_prep, so that the largest is exactly 1 however narrow the pdf).
    const bool direct = __any(valid && (fmax(dt0, dt1) > kPMaxStep || fmax(r.e[0], r.e[1]) > kPMaxOff));
    static_assert((kPWCols - 1) * kPMaxStep <= 16 && (kPWRows - 1) * kPMaxStep <= 16, "range");
    uint32_t G[kPWCols], sum = 0u;
    if (!direct) {
      double g = unit * pt_exp(pt_arg(ec, tx0));
      double q = pt_exp(fmin(-(tx0 + 0.5 * dt1) * dt1, 700.0));
      const double qq = pt_exp(-dt1 * dt1);
#pragma unroll
      for (int c = 0; c < kPWCols; ++c) {
        // + 2^52: the low word is g rounded to an integer
        const uint32_t u = (uint32_t)__double_as_longlong(g + 4503599627370496.0);
        sum += u & bit_mask(cmask, c);
        G[c] = sum;
        g *= q;
        q *= qq;
      }
    } else {  // (uniform over the workgroup)
      __syncthreads();  // the last batch's readers of sG are done
#pragma unroll 1
      for (int c = 0; c < kPWCols; ++c) {
        const double g = unit * pt_exp(fmin(pt_arg(ec, fma((double)(c0 + c - r.lo[1]), dt1, r.t0[1])), 0.0));
        sG[(kPWCols * w + c + 1) * 64 + lane] = (uint32_t)__double_as_longlong(g + 4503599627370496.0);
      }
#pragma unroll
      for (int c = 0; c < kPWCols; ++c) {
        sum += sG[(kPWCols * w + c + 1) * 64 + lane] & bit_mask(cmask, c);
        G[c] = sum;
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
    if (w == 0) sOff[lane] = (uint32_t)(valid ? k : 0) * (uint32_t)(a.B + 1);
    __syncthreads();
    for (int ps = 0; ps < passes; ++ps) {
      const int base = tmn + ps * kPSlots;
      if (have) {
        // the wave's chunks of the pass: those with bins of it (cells without a
        // bin go to the first)
        uint32_t todo = (1u << kPWCh) - 1u;
        if (passes > 1) {
          const PtChunk c = cs[lane & (kPWCh - 1)];
          todo &= (uint32_t)__ballot((c.mn < base + kPSlots && c.mx >= base) || (ps == 0 && c.mn < 0));
        }
        double g = S0 * pt_exp(pt_arg(r.e[0], ty0) + er);
        double q = pt_exp(fmin(-(ty0 + 0.5 * dt0) * dt0, 700.0));
        const double qq = pt_exp(-dt0 * dt0);
        uint32_t rm = rmask;
        // prefix sums as doubles 2^52 + G (only the low words change): a ring of
        // four entries, this one, the next, and two on their way; the last one's
        // place is free once this one's steps are formed
        u32x2 Q[4][kPR];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < kPR; ++j) {
            Q[u][j][0] = 0u;
            Q[u][j][1] = two52;
          }
        int cn = __builtin_amdgcn_readfirstlane(cs[0].n);
        const uint2* ev = a.entries + __builtin_amdgcn_readfirstlane(cs[0].first);
        uint2 ent = ev[lane];  // (there are 64 entries more than the model matrix has)
#pragma unroll 1
        for (int ch = 0; ch < kPWCh; ++ch) {
          double gx[kPR];
#pragma unroll
          for (int i = 0; i < kPR; ++i) {
            gx[i] = g;
            g *= q;
            q *= qq;
          }
          if (direct) {
#pragma unroll
            for (int i = 0; i < kPR; ++i)
              gx[i] = S0 * pt_exp(fmin(pt_arg(r.e[0], fma((double)(r0 + kPR * ch + i - r.lo[0]), dt0, r.t0[0])), 0.0) + er);
          }
#pragma unroll
          for (int i = 0; i < kPR; ++i) {
            const long long b = __double_as_longlong(gx[i]);
            const uint32_t on = bit_mask(rm, i);
            gx[i] = __hiloint2double((int)((uint32_t)(b >> 32) & on), (int)((uint32_t)b & on));
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
          if (!any || !(todo >> ch & 1u)) continue;  // no pdf of the batch has these rows
          // every row stands at column 0
#pragma unroll
          for (int j = 0; j < kPR; ++j) Q[3][j][0] = 0u;
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
            // the slots of an even entry and the next one (row_shl:1; a pair lies in a
            // row of 16 lanes)
            const uint32_t slots =
                slot | (uint32_t)__builtin_amdgcn_mov_dpp((int)slot, 0x101, 0xF, 0xF, true) << 16;
            auto load = [&](int i, u32x2 (&o)[kPR]) {
              const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)e.x, i);
              const char* p = reinterpret_cast<const char*>(sG);
              o[0][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel0));
              o[1][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel1));
              o[2][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel2));
              o[3][0] = *reinterpret_cast<const uint32_t*>(p + __builtin_amdgcn_perm(c, lane4, sel3));
            };
            // 2^52 and the bin's mass: the rows' steps of G (exact differences)
            // times their factors, each rounded to the fixed point
            auto add = [&](uint32_t at, const u32x2 (&o)[kPR], const u32x2 (&before)[kPR]) {
              double sum = 4503599627370496.0;
#pragma unroll
              for (int j = 0; j < kPR; ++j)
                sum = __builtin_fma(gx[j],
                                    __builtin_bit_cast(double, o[j]) -
                                        __builtin_bit_cast(double, before[j]),
                                    sum);
              unsigned long long* h = reinterpret_cast<unsigned long long*>(
                  reinterpret_cast<char*>(sH) + (at ^ lane8));
              __hip_atomic_fetch_add(h, (unsigned long long)__double_as_longlong(sum),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            // (m is even; a whole segment ends on the ring's last place, where the
            // next one looks for it)
            load(0, Q[0]);
            load(1, Q[1]);
            for (int i = 0;; i += 4) {
              const bool more = i + 2 < m, more2 = i + 4 < m;
              uint32_t both = (uint32_t)__builtin_amdgcn_readlane((int)slots, i);
              add(both & 0xFFFFu, Q[0], Q[3]);
              if (more) {
                load(i + 2, Q[2]);
                load(i + 3, Q[3]);
              }
              __builtin_amdgcn_sched_barrier(0);
              add(both >> 16, Q[1], Q[0]);
              if (!more) break;
              both = (uint32_t)__builtin_amdgcn_readlane((int)slots, i + 2);
              add(both & 0xFFFFu, Q[2], Q[1]);
              if (more2) {
                load(i + 4, Q[0]);
                load(i + 5, Q[1]);
              }
              __builtin_amdgcn_sched_barrier(0);
              add(both >> 16, Q[3], Q[2]);
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
        if (b >= span) return;
        const int s = b0 + b < kPSlots ? b0 + b : b0 + b - kPSlots;
        const int at = s * 64 + (p ^ (s & 63));
        const unsigned long long v = sH[at] & kPSum;
        const uint32_t o = sOff[p] + (uint32_t)(base + b);
        sH[at] = 0ull;
        if (v) __hip_atomic_fetch_add(&a.acc[o], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      if (span > 32) {
        for (int b = 0; b < span; b += 64) {
#pragma unroll 4
          for (int i = 0; i < 64 / kPWaves; ++i) give(b + lane, kPWaves * i + w);
        }
      } else {
#pragma unroll 4
        for (int i = 0; i < 32 / kPWaves; ++i)
          give(lane & 31, 2 * kPWaves * i + 2 * w + (lane >> 5));
      }
      if (ps + 1 < passes) __syncthreads();
    }
    if (tnone && w == 0) {
      const int at = kPSlots * 64 + (lane ^ (kPSlots & 63));
      const unsigned long long v = sH[at] & kPSum;
      sH[at] = 0ull;
      if (valid && v)
        __hip_atomic_fetch_add(&a.acc[sOff[lane] + (uint32_t)a.B], v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  }
}

// ---------------------------------------------------------------------------
// per pdf: the row of P, its sums divided by their total; a wave per row
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pt_final(PtArgs a) {
  const int lane = threadIdx.x & 63;
  const long long k = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= a.K) return;
  const double scale = a.rec[k].scale;
  if (!(scale > 0.0)) return;  // the per-pdf kernel's row
  const unsigned long long* u = a.acc + k * (a.B + 1);
  float* p = a.P + k * a.B;
  // (sums below 2^52: a double holds them)
  double sum = 0.0, tot;
  if (a.B < 320) {
    double v[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      v[i] = lane + 64 * i <= a.B ? (double)u[lane + 64 * i] : 0.0;
      sum += v[i];
    }
    tot = wave_sum(sum);
    const double f = 1.0 / tot;
#pragma unroll
    for (int i = 0; i < 5; ++i)
      if (lane + 64 * i < a.B) p[lane + 64 * i] = (float)(v[i] * f);
  } else {
    for (int b = lane; b <= a.B; b += 64) sum += (double)u[b];
    tot = wave_sum(sum);
    const double f = 1.0 / tot;
    for (int b = lane; b < a.B; b += 64) p[b] = (float)((double)u[b] * f);
  }
  if (a.Z && lane == 0) a.Z[k] = tot / scale * pt_exp(-(a.rec[k].e[0] + a.rec[k].e[1]));
}

constexpr size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct PtLayout {
  size_t rec, bbox, lists, counts, batches, state, klist, acc;  // acc: to the end
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
  L.klist = L.state + 256;
  L.acc = L.klist + al256((size_t)(K + 1) * 4);
  return L;
}

// workspace of one pass over kg pdfs
size_t pt_pass_bytes(long long ntiles, int B, long long kg) {
  return pt_layout(ntiles, kg).acc + (size_t)kg * (size_t)(B + 1) * 8;
}

// pdfs of a pass when it is up to the library: all, or even shares that keep
// the sums within about 256 MB (and the batches full)
long long pt_share(long long K, int B) {
  long long most = (1ll << 25) / (B + 1);
  if (most < 2 * kPtMinK) most = 2 * kPtMinK;
  const long long passes = (K + most - 1) / most;
  return (K + passes - 1) / passes;
}

int pt_div(int n, int m) { return (n + m - 1) / m; }

// blocks of lists of a grid
long long pt_blocks(const vup_mm& mm) {
  return (long long)pt_div(mm.grid.n[1], kPX) * pt_div(mm.grid.n[0], kPL);
}

}  // namespace

long long tile_count(const vup_grid& g) {
  return (long long)pt_div(g.n[1], kPX) * pt_div(g.n[0], kPY);
}

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
         tile_count(mm.grid) * pt_div((int)d.K, kPPart) * kPPart <= kPMaxList;
}

size_t propagate_tiled_ws_bytes(const vup_mm& mm, long long K) {
  return pt_layout(tile_count(mm.grid), K).acc + al256((size_t)K * 4);
}

size_t propagate_tiled_full_bytes(const vup_mm& mm, long long K) {
  const size_t least = propagate_tiled_ws_bytes(mm, K);
  const size_t full = pt_pass_bytes(tile_count(mm.grid), mm.B, pt_share(K, mm.B));
  return full > least ? full : least;
}

long long propagate_tiled_pass(const vup_mm& mm, long long K, size_t ws_bytes) {
  const long long ntiles = tile_count(mm.grid);
  long long kg = pt_share(K, mm.B);
  for (long long passes = (K + kg - 1) / kg; kg >= kPtMinK; ++passes, kg = (K + passes - 1) / passes)
    if (pt_pass_bytes(ntiles, mm.B, kg) <= ws_bytes) return kg;
  return 0;
}

// one pass
static hipError_t launch_pass(const vup_mm& mm, const vup_dists& d, void* ws, float* P, double* Z,
                              hipStream_t s) {
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
  const long long ntiles = tile_count(mm.grid);
  a.parts = (int)((d.K + kPPart - 1) / kPPart);
  const PtLayout L = pt_layout(ntiles, d.K);
  char* base = static_cast<char*>(ws);
  a.rec = reinterpret_cast<PtRec*>(base + L.rec);
  a.bbox = reinterpret_cast<unsigned long long*>(base + L.bbox);
  a.lists = reinterpret_cast<uint16_t*>(base + L.lists);
  a.counts = reinterpret_cast<int*>(base + L.counts);
  a.batches = reinterpret_cast<uint32_t*>(base + L.batches);
  a.state = reinterpret_cast<int*>(base + L.state);
  a.acc = reinterpret_cast<unsigned long long*>(base + L.acc);
  a.klist = reinterpret_cast<int*>(base + L.klist);
  a.P = P;
  a.Z = Z;
  const long long pb = (d.K + 255) / 256;
  hipLaunchKernelGGL(k_pt_prep, dim3((unsigned)(pb > 2048 ? pb : 2048)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_pt_scan, dim3((unsigned)(ntiles * a.parts)), dim3(kPScan), 0, s, a);
  // as many workgroups as fit on the GPU (two per CU)
  hipLaunchKernelGGL(k_pt_main, dim3(512), dim3(64 * kPWaves), 0, s, a);
  hipLaunchKernelGGL(k_pt_final, dim3((unsigned)((d.K + 3) / 4)), dim3(256), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_propagate_list(mm, d, a.klist, a.klist + d.K, P, Z, s);
}

hipError_t launch_propagate_tiled(const vup_mm& mm, const vup_dists& d, long long kg, void* ws,
                                  float* P, double* Z, hipStream_t s) {
  for (long long k = 0; k < d.K; k += kg) {
    vup_dists part = d;
    part.K = d.K - k < kg ? d.K - k : kg;
    part.mu = d.mu + 2 * k;
    part.sigma = d.sigma + 2 * k;
    const hipError_t e = launch_pass(mm, part, ws, P + k * mm.B, Z ? Z + k : nullptr, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace vup
