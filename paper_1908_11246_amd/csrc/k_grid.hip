// Model-matrix construction (done once per grid and model, Appendix A: the
// N model evaluations and the sort are amortised over all propagated pdfs):
//   k_eval_grid     f_i = M(x_i) at cell centres, FP64
//   k_minmax / k_edges  B uniform bins over [min f, max f]
//   k_bin           indicator of eq. (4) as a bin index; padded bin map
//                   (4*bin, LDS byte offsets for the sweep kernels), padded
//                   FP32 copy of f in anchored form (every eighth column
//                   holds f, the columns after it their offset from it),
//                   per-chunk bin counts
//   k_count         per bin the exclusive scan of its chunk counts; runs of
//                   equal bin per row
//   k_offsets       CSR row starts (scan over the bins), run row pointers
//   k_fill          stable scatter of cell indices into compressed-by-bin
//                   order (the sparse one-hot model matrix of eq. (5)); run
//                   records and the cells' run indices; on 2-D grids the
//                   tiled propagation's entries (k_ptiles.hpp)
// Each of these launches covers both the compressed-by-bin form and the run
// form, which only depend on the bin map: at 1024^2 cells a launch's start and
// end cost about as much as its work. (1024^2 cells, 256 bins: vup_bin's
// kernels took 66 to 94 us in 13 launches with one launch per part, 41 us in
// these 4, with the entries, which took 20 us by themselves; evaluation, edges,
// vup_bin and the choice of the form together 158 and 122 us of wall time.)
// plus the per-distribution window listing.
#include <hip/hip_runtime.h>

#include "k_ptiles.hpp"
#include "vup_device.hpp"
#include "vup_internal.hpp"

namespace vup {

// ---------------------------------------------------------------------------
// model evaluation
// ---------------------------------------------------------------------------
struct EvalArgs {
  int ndim;
  int n[4];
  double lo[4], hi[4];
  vup_model m;
  long long N;
};

__global__ __launch_bounds__(256) void k_eval_grid(EvalArgs a, double* __restrict__ f) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.N) return;
  double x[4];
  long long t = i;
  for (int d = a.ndim - 1; d >= 0; --d) {
    const int j = (int)(t % a.n[d]);
    t /= a.n[d];
    x[d] = cell_centre(a.lo[d], a.hi[d], a.n[d], j);
  }
  f[i] = model_at(a.m.kind, a.ndim, a.m.theta, x);
}

hipError_t launch_eval_grid(const vup_grid& g, const vup_model& m, double* f, hipStream_t s) {
  EvalArgs a{};
  a.ndim = g.ndim;
  a.N = 1;
  for (int d = 0; d < g.ndim; ++d) {
    a.n[d] = g.n[d];
    a.lo[d] = g.lo[d];
    a.hi[d] = g.hi[d];
    a.N *= g.n[d];
  }
  a.m = m;
  const long long blocks = (a.N + 255) / 256;
  hipLaunchKernelGGL(k_eval_grid, dim3((unsigned)blocks), dim3(256), 0, s, a, f);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// uniform edges: min/max via order-preserving integer images of the doubles
// (exact, order independent), then e_b = lo + b*((hi - lo)/B), e_B = hi.
// The two extreme slots of `edges` hold the running min/max images.
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long ord_of(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double of_ord(unsigned long long o) {
  const unsigned long long u = (o >> 63) ? (o & 0x7FFFFFFFFFFFFFFFull) : ~o;
  return __longlong_as_double((long long)u);
}

// Min and max of the non-NaN model values as order-preserving integer images.
// A thread reads eight values at once (independent loads in flight), the
// workgroup reduces in LDS and leaves its pair in edges[2 block], [2 block + 1]
// (there are at most (B + 1) / 2 workgroups), or, with few edges, merges it
// into edges[0] and edges[B] with atomics.
__global__ void k_minmax_init(unsigned long long* e, int B) {
  if (threadIdx.x == 0) {
    e[0] = ~0ull;  // running min image
    e[B] = 0ull;   // running max image
  }
}

__device__ __forceinline__ void reduce_minmax(unsigned long long& mn, unsigned long long& mx,
                                              unsigned long long* smn, unsigned long long* smx) {
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  if ((threadIdx.x & 63) == 0) {
    smn[threadIdx.x >> 6] = mn;
    smx[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      mn = smn[w] < mn ? smn[w] : mn;
      mx = smx[w] > mx ? smx[w] : mx;
    }
  }
}

template <bool PART>
__global__ __launch_bounds__(256) void k_minmax(const double* __restrict__ f, long long N,
                                                unsigned long long* e, int B) {
  __shared__ unsigned long long smn[4], smx[4];
  unsigned long long mn = ~0ull, mx = 0ull;
  const long long stride = (long long)gridDim.x * 256;
  for (long long i0 = (long long)blockIdx.x * 256 + threadIdx.x; i0 < N; i0 += 8 * stride) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long i = i0 + u * stride;
      v[u] = i < N ? f[i] : __builtin_nan("");
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (v[u] != v[u]) continue;
      const unsigned long long o = ord_of(v[u]);
      mn = o < mn ? o : mn;
      mx = o > mx ? o : mx;
    }
  }
  reduce_minmax(mn, mx, smn, smx);
  if (threadIdx.x == 0) {
    if constexpr (PART) {
      e[2 * blockIdx.x] = mn;
      e[2 * blockIdx.x + 1] = mx;
    } else {
      atomicMin(e, mn);
      atomicMax(e + B, mx);
    }
  }
}

// parts > 0: the pairs k_minmax<true> left; 0: edges[0] and edges[B]
__global__ __launch_bounds__(256) void k_edges(double* e, int B, int parts) {
#pragma clang fp contract(off)
  __shared__ unsigned long long smn[4], smx[4];
  __shared__ double lohi[2];
  const unsigned long long* u = reinterpret_cast<const unsigned long long*>(e);
  unsigned long long mn = ~0ull, mx = 0ull;
  if (parts > 0) {
    for (int p = threadIdx.x; p < parts; p += 256) {
      mn = u[2 * p] < mn ? u[2 * p] : mn;
      mx = u[2 * p + 1] > mx ? u[2 * p + 1] : mx;
    }
    reduce_minmax(mn, mx, smn, smx);
  } else if (threadIdx.x == 0) {
    mn = u[0];
    mx = u[B];
  }
  if (threadIdx.x == 0) {
    lohi[0] = of_ord(mn);
    lohi[1] = of_ord(mx);
  }
  __syncthreads();
  const double lo = lohi[0], hi = lohi[1];
  const double w = (hi - lo) / B;
  for (int b = threadIdx.x; b <= B; b += blockDim.x) e[b] = (b == B) ? hi : lo + b * w;
}

hipError_t launch_uniform_edges(const double* f, int64_t N, int B, double* edges, hipStream_t s) {
  unsigned long long* e = reinterpret_cast<unsigned long long*>(edges);
  long long blocks = (N + 2047) / 2048;  // eight values per thread
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  // the edges themselves hold the workgroups' pairs when there is room for
  // enough of them: two launches and no atomics (at 2^20 cells and 256 bins 7.5
  // + 2.8 us; 1.4 + 9.4 + 2.4 us with atomics and one value in flight per
  // thread). A workgroup takes about 0.47 ns a value: with 128 of them, 2^21
  // values take 12 us (19 with atomics), 2^22 18.5 (20), 2^24 69 (34)
  long long parts = (B + 1) / 2 < blocks ? (B + 1) / 2 : blocks;
  if (parts >= 320 || N <= 20480 * parts) {
    hipLaunchKernelGGL(k_minmax<true>, dim3((unsigned)parts), dim3(256), 0, s, f, (long long)N, e,
                       B);
  } else {
    parts = 0;
    hipLaunchKernelGGL(k_minmax_init, dim3(1), dim3(64), 0, s, e, B);
    hipLaunchKernelGGL(k_minmax<false>, dim3((unsigned)blocks), dim3(256), 0, s, f, (long long)N,
                       e, B);
  }
  hipLaunchKernelGGL(k_edges, dim3(1), dim3(256), 0, s, edges, B, (int)parts);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// binning
// ---------------------------------------------------------------------------
struct BinArgs {
  const double* __restrict__ f;
  const double* __restrict__ edges_in;
  double* edges_ws;
  int32_t* bin;       // may be null
  uint16_t* binmap;   // [rows*pitch]
  float* f32;         // [rows*pitch]
  int* chunk_counts;  // [(B+1) * nblk], bin-major
  unsigned long long* counters;
  int B;
  int nL;             // cells on the fastest axis
  int pitch;
  long long rows;
  long long nblk;
  int chunk;          // padded positions per chunk
  PtBlock* tblocks;   // the tiles' blocks (2-D grids)
  int ntblocks;
};

// bin index of y: largest b < B with e[b] <= y, when e[0] <= y <= e[B]
// (inv: B over the span of the edges; a finite positive number)
__device__ __forceinline__ int bin_search(const double* e, int B, double inv, double y) {
  if (!(y >= e[0] && y <= e[B])) return -1;
  // where uniform edges would have it, when that is right
  int lo = 0, hi = B - 1;  // answer in [lo, hi]
  const int g = min((int)((y - e[0]) * inv), B - 1);
  if (e[g] <= y) {
    if (y < e[g + 1]) return g;
    lo = g;
  } else {
    hi = g - 1;
  }
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (e[mid] <= y) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__global__ __launch_bounds__(256) void k_bin(BinArgs a) {
  extern __shared__ double sh[];  // edges[B+1], then int counts[B+1]
  double* e = sh;
  int* cnt = reinterpret_cast<int*>(sh + a.B + 1);
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  for (int b = threadIdx.x; b <= a.B; b += 256) {
    const double v = a.edges_in[b];
    e[b] = v;
    if (!isfinite(v)) atomicOr(&bad, 1);
    if (b > 0 && !(a.edges_in[b - 1] < v)) atomicOr(&bad, 1);
    cnt[b] = 0;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int b = threadIdx.x; b <= a.B; b += 256) a.edges_ws[b] = e[b];
    // the counters start here (cells without a bin and runs follow)
    if (threadIdx.x < 8) a.counters[threadIdx.x] = threadIdx.x == kCntBadEdges && bad ? 1ull : 0ull;
  }
  for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < a.ntblocks; t += a.nblk * 256)
    a.tblocks[t].both = 0ull;
  const double span = e[a.B] - e[0];
  const double inv = span > 0.0 && span < 1e300 && span > 1e-280 ? a.B / span : 0.0;
  const long long base = (long long)blockIdx.x * a.chunk;
  const long long total = a.rows * a.pitch;
  for (int q = threadIdx.x; q < a.chunk; q += 256) {
    const long long p = base + q;
    if (p >= total) break;
    const long long row = p / a.pitch;
    const int col = (int)(p - row * a.pitch);
    uint16_t code = (uint16_t)(4 * a.B);
    float fv = 0.0f;
    if (col < a.nL) {
      const long long cell = row * a.nL + col;
      const double y = a.f[cell];
      const int b = bad ? -1 : bin_search(e, a.B, inv, y);
      if (a.bin) a.bin[cell] = b;
      if (b >= 0) {
        code = (uint16_t)(4 * b);
        atomicAdd(&cnt[b], 1);
      } else {
        atomicAdd(&cnt[a.B], 1);
      }
      // anchored FP32 form: columns 8m hold f, the seven after each their
      // difference from it (taken in FP64, rounded once); after a non-finite
      // anchor they hold their own values, which the difference would lose
      const int c0 = col & ~7;
      const double f0 = a.f[row * a.nL + c0];
      fv = col == c0 ? (float)y : (float)(isfinite(f0) ? y - f0 : y);
    }
    a.binmap[p] = code;
    a.f32[p] = fv;
  }
  __syncthreads();
  for (int b = threadIdx.x; b <= a.B; b += 256) a.chunk_counts[(long long)b * a.nblk + blockIdx.x] = cnt[b];
}

// ---------------------------------------------------------------------------
// exclusive prefix sum of n ints in place (values and sums below 2^31), by
// tiles of kScanTile: tile totals, one workgroup scanning the totals, then
// each tile scanned from its offset. `tsum` holds ceil(n / kScanTile) int64.
// ---------------------------------------------------------------------------
constexpr int kScanPer = 4;                  // elements per thread (one 16-byte load)
constexpr int kScanTile = 256 * kScanPer;    // elements per workgroup

// this thread's four consecutive elements of the tile (zeros past n); the
// array is 16-byte aligned and tiles are whole multiples of four elements
__device__ __forceinline__ int4 scan_load4(const int* __restrict__ v, long long n, long long p) {
  if (p + 3 < n) return *reinterpret_cast<const int4*>(v + p);
  return make_int4(p < n ? v[p] : 0, p + 1 < n ? v[p + 1] : 0, p + 2 < n ? v[p + 2] : 0,
                   p + 3 < n ? v[p + 3] : 0);
}

__global__ __launch_bounds__(256) void k_tile_sums(const int* __restrict__ v, long long n,
                                                   long long* __restrict__ tsum) {
  __shared__ long long red[4];
  const long long p = (long long)blockIdx.x * kScanTile + kScanPer * threadIdx.x;
  const int4 x = scan_load4(v, n, p);
  long long sum = (long long)x.x + x.y + x.z + x.w;
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) tsum[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// inclusive scan of one value per thread across a 1024-thread (or smaller)
// workgroup; `wsum` is LDS for one value per wave
__device__ __forceinline__ long long block_incl_scan(long long x, long long* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const long long t = __shfl_up(x, o, 64);
    if (lane >= o) x += t;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  long long off = 0;
  for (int w = 0; w < wave; ++w) off += wsum[w];
  __syncthreads();
  return x + off;
}

__global__ __launch_bounds__(1024) void k_scan_tile_sums(long long* tsum, long long ntiles,
                                                         int* total) {
  __shared__ long long wsum[16];
  __shared__ long long last;
  long long carry = 0;
  for (long long b0 = 0; b0 < ntiles; b0 += 1024) {
    const long long i = b0 + threadIdx.x;
    const long long x = i < ntiles ? tsum[i] : 0;
    const long long incl = block_incl_scan(x, wsum);
    if (i < ntiles) tsum[i] = carry + incl - x;
    if (threadIdx.x == 1023) last = incl;
    __syncthreads();
    carry += last;
    __syncthreads();
  }
  if (threadIdx.x == 0 && total) *total = (int)carry;
}

__global__ __launch_bounds__(256) void k_tile_scan(int* __restrict__ v, long long n,
                                                   const long long* __restrict__ tsum) {
  __shared__ long long wsum[4];
  const long long p = (long long)blockIdx.x * kScanTile + kScanPer * threadIdx.x;
  const int4 x = scan_load4(v, n, p);
  const long long s = (long long)x.x + x.y + x.z + x.w;
  const long long e0 = block_incl_scan(s, wsum) - s + tsum[blockIdx.x];
  const int4 y = make_int4((int)e0, (int)(e0 + x.x), (int)(e0 + x.x + x.y),
                           (int)(e0 + x.x + x.y + x.z));
  if (p + 3 < n) {
    *reinterpret_cast<int4*>(v + p) = y;
  } else {
    if (p < n) v[p] = y.x;
    if (p + 1 < n) v[p + 1] = y.y;
    if (p + 2 < n) v[p + 2] = y.z;
  }
}

long long scan_tiles(long long n) { return (n + kScanTile - 1) / kScanTile; }

hipError_t launch_scan_excl(int* v, long long n, long long* tsum, int* total, hipStream_t s) {
  const long long nt = scan_tiles(n);
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)nt), dim3(256), 0, s, v, n, tsum);
  hipLaunchKernelGGL(k_scan_tile_sums, dim3(1), dim3(1024), 0, s, tsum, nt, total);
  hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)nt), dim3(256), 0, s, v, n, tsum);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// windows of every (k, c)
// ---------------------------------------------------------------------------
struct WinArgs {
  int ndim;
  int n[4];
  double lo[4], hi[4];
  DistsDev d;
};

__global__ __launch_bounds__(256) void k_windows(WinArgs a, int32_t* __restrict__ win) {
  const long long kc = (long long)blockIdx.x * 256 + threadIdx.x;
  if (kc >= a.d.K * a.d.C) return;
  const int D = a.ndim;
  int lo[4], hi[4];
  bool bad = false;
  for (int d = 0; d < D; ++d) {
    if (!axis_window(a.lo[d], a.hi[d], a.n[d], a.d.mu[kc * D + d], a.d.sigma[kc * D + d], a.d.ns,
                     lo[d], hi[d]))
      bad = true;
  }
  for (int d = 0; d < D; ++d) {
    win[(kc * D + d) * 2 + 0] = bad ? 0 : lo[d];
    win[(kc * D + d) * 2 + 1] = bad ? -1 : hi[d];
  }
}

hipError_t launch_windows(const vup_grid& g, const vup_dists& d, int32_t* win, hipStream_t s) {
  const long long n = d.K * d.ncomp;
  if (n == 0) return hipSuccess;
  WinArgs a{};
  a.ndim = g.ndim;
  for (int i = 0; i < g.ndim; ++i) {
    a.n[i] = g.n[i];
    a.lo[i] = g.lo[i];
    a.hi[i] = g.hi[i];
  }
  a.d = make_dists_dev(d);
  hipLaunchKernelGGL(k_windows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, win);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------
// 32-cell blocks of a row segment: a wave counts and fills a segment's runs
constexpr int kSegBlocks = 64;

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

bool ws_layout(const vup_grid& g, int B, WsLayout* out) {
  WsLayout L{};
  const int nL = g.n[g.ndim - 1];
  L.pitch = (nL + 31) / 32 * 32;
  L.rows = 1;
  for (int d = 0; d + 1 < g.ndim; ++d) L.rows *= g.n[d];
  const long long N = L.rows * nL;
  const long long padded = L.rows * L.pitch;
  // chunks of the bin sort: small for parallelism, larger when the (bin,
  // chunk) count table would grow past 2^24 entries
  L.chunk = 1024;
  while ((long long)(B + 1) * ((padded + L.chunk - 1) / L.chunk) > (1ll << 24) && L.chunk < 65536)
    L.chunk *= 2;
  L.nblk = (padded + L.chunk - 1) / L.chunk;
  const long long rowblocks = L.rows * (L.pitch / 32);
  L.nseg = (L.pitch / 32 + kSegBlocks - 1) / kSegBlocks;
  size_t o = 0;
  L.off_edges = o;
  o = align256(o + (size_t)(B + 1) * 8);
  L.off_binmap = o;
  o = align256(o + (size_t)padded * 2);
  L.off_f32 = o;
  o = align256(o + (size_t)padded * 4);
  L.off_counts = o;
  o = align256(o + (size_t)(B + 1) * 8);
  L.off_offsets = o;
  o = align256(o + (size_t)(B + 1) * 8);
  L.off_perm = o;
  o = align256(o + (size_t)N * 4);
  L.off_scratch = o;
  const size_t sort_scratch = (size_t)(B + 1) * (size_t)L.nblk * 4;
  const size_t run_scratch = (size_t)rowblocks * 4;
  const size_t scratch = sort_scratch > run_scratch ? sort_scratch : run_scratch;
  o = align256(o + scratch);
  L.off_tsum = o;  // tile sums of the prefix scans
  o = align256(o + (size_t)(scan_tiles((long long)(scratch / 4)) + 1) * 8);
  L.off_segs = o;  // rows of several segments: the segments' first runs
  if (L.nseg > 1) o = align256(o + (size_t)(L.rows * L.nseg + 1) * 4);
  L.off_counters = o;
  o = align256(o + 8 * 8);
  L.off_runs = o;
  // up to one record per cell plus a terminator per row, and 128 records of
  // padding: the run sweep reads up to 79 records past a row segment's end
  o = align256(o + (size_t)(N + L.rows + 128) * 4);
  L.off_rowptr = o;
  o = align256(o + (size_t)(L.rows + 1) * 4);
  L.off_runidx = o;
  o = align256(o + (size_t)padded * 2);
  if (g.ndim == 2) {
    size_t ents, chunks, blocks;
    tile_entry_sizes(g, &ents, &chunks, &blocks);
    L.off_tents = o;
    o = align256(o + ents);
    L.off_tchunks = o;
    o = align256(o + chunks);
    L.off_tblocks = o;
    o = align256(o + blocks);
  }
  L.bytes = o;
  *out = L;
  return true;
}

// ---------------------------------------------------------------------------
// the compressed-by-bin form and the runs of equal bin along the fastest axis
// (a run-length form of the model matrix's rows), from the bin map
// ---------------------------------------------------------------------------
struct FormArgs {
  const uint16_t* __restrict__ binmap;
  // compressed by bin
  int* cc;             // [(B+1) * nblk] chunk counts, bin-major; scanned per bin
  long long* counts;   // [B+1]
  long long* offsets;  // [B+1]
  int32_t* perm;
  int B;
  long long nblk;
  int chunk;
  // runs
  uint32_t* runs;
  int* rowptr;         // [rows + 1] first run of each row
  // [rows * nseg + 1]: runs of each row segment of 64 blocks, with the terminator
  // in the row's last, then their scan; rowptr itself for rows of one segment
  int* segs;
  int nseg;
  uint16_t* runidx;
  unsigned long long* counters;
  long long rows;
  int nL, pitch, nb;   // nb 32-cell blocks per row
  int group;           // lanes per segment: a power of two, at least nb up to 64
  int rowblocks;       // workgroups of the run part
  int swaves;          // chunks per workgroup of the scatter
  int scan_segs;       // k_offsets scans the segments too
  // entries of the tiled propagation (2-D grids)
  int entblocks;       // workgroups of that part
  PtEntArgs ent;
};

// the 32 bin codes of block q of a row (the row pitch is a multiple of 32
// cells, so a block is 64 aligned bytes: four 16-byte loads) and the code of
// the cell before it (0xFFFFFFFF for the row's first block, so cell 0 starts
// a run)
struct Block32 {
  uint32_t w[16];  // two codes per word, the lower column in the low half
  uint32_t prev;
};

__device__ __forceinline__ Block32 load_block32(const uint16_t* row, int q) {
  Block32 b;
  const uint4* p = reinterpret_cast<const uint4*>(row + q * 32);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint4 v = p[i];
    b.w[4 * i] = v.x;
    b.w[4 * i + 1] = v.y;
    b.w[4 * i + 2] = v.z;
    b.w[4 * i + 3] = v.w;
  }
  b.prev = q == 0 ? 0xFFFFFFFFu : (uint32_t)row[q * 32 - 1];
  return b;
}

__device__ __forceinline__ uint32_t code_at(const Block32& b, int j) {
  return (j & 1) ? (b.w[j >> 1] >> 16) : (b.w[j >> 1] & 0xFFFFu);
}

// bit j set when cell q*32 + j (a cell of the row) starts a run
__device__ __forceinline__ uint32_t run_starts(const Block32& b, int q, int nL) {
  uint32_t m = 0;
  uint32_t before = b.prev;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const uint32_t c = code_at(b, j);
    if (c != before && q * 32 + j < nL) m |= 1u << j;
    before = c;
  }
  return m;
}

// Workgroups 0 .. B: bin b's chunk counts, scanned (exclusive) in place, and
// its total. The others: `group` lanes per row segment count its runs.
__global__ __launch_bounds__(256) void k_count(FormArgs a) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if ((int)blockIdx.x <= a.B) {
    __shared__ int wsum[2][4];
    int* v = a.cc + (long long)blockIdx.x * a.nblk;
    int carry = 0;  // uniform
    int odd = 0;
    for (long long p0 = 0; p0 < a.nblk; p0 += 1024, odd ^= 1) {
      // a thread takes four consecutive chunks (their first need not be
      // 16-byte aligned)
      const long long p = p0 + 4 * (int)threadIdx.x;
      int x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = p + u < a.nblk ? v[p + u] : 0;
      int incl = (x[0] + x[1]) + (x[2] + x[3]);
      const int own = incl;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      if (lane == 63) wsum[odd][w] = incl;
      __syncthreads();
      int run = carry + incl - own;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < w) run += wsum[odd][q];
        carry += wsum[odd][q];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (p + u < a.nblk) v[p + u] = run;
        run += x[u];
      }
    }
    if (threadIdx.x == 0) a.counts[blockIdx.x] = carry;
    return;
  }
  const long long t = (long long)(blockIdx.x - a.B - 1) * 256 + threadIdx.x;
  const long long sg = t / a.group;
  if (sg >= a.rows * a.nseg) return;  // whole groups
  const long long r = sg / a.nseg;
  const int part = (int)(sg - r * a.nseg);
  const int q = part * kSegBlocks + (int)(t % a.group);
  int cnt = 0;
  if (q < a.nb) cnt = __popc(run_starts(load_block32(a.binmap + r * a.pitch, q), q, a.nL));
  for (int o = a.group >> 1; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
  if (t % a.group == 0) a.segs[sg] = cnt + (part == a.nseg - 1 ? 1 : 0);
}

// exclusive scan of n values by one workgroup of 1024 threads; returns the sum
template <typename T>
__device__ __forceinline__ long long scan_block(const T* in, T* out, long long n, long long* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long carry = 0;
  for (long long p0 = 0; p0 < n; p0 += 4096) {
    const long long p = p0 + 4 * (int)threadIdx.x;
    long long x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = p + u < n ? (long long)in[p + u] : 0;
    const long long own = (x[0] + x[1]) + (x[2] + x[3]);
    long long incl = own;
    for (int o = 1; o < 64; o <<= 1) {
      const long long t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    __syncthreads();
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    long long run = carry + incl - own;
    for (int q = 0; q < 16; ++q) {
      if (q < w) run += wsum[q];
      carry += wsum[q];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p + u < n) out[p + u] = (T)run;
      run += x[u];
    }
  }
  return carry;
}

// workgroup 0: CSR row starts from the bins' counts; workgroup 1: the row
// segments' first runs. The run and outside counts go to the counters.
__global__ __launch_bounds__(1024) void k_offsets(FormArgs a) {
  __shared__ long long wsum[16];
  if (blockIdx.x == 0) {
    scan_block(a.counts, a.offsets, (long long)a.B + 1, wsum);
    if (threadIdx.x == 0) a.counters[kCntOutside] = (unsigned long long)a.counts[a.B];
  } else {
    long long total;
    const long long n = a.rows * a.nseg;
    if (a.scan_segs) {
      total = scan_block(a.segs, a.segs, n, wsum);
      if (threadIdx.x == 0) a.segs[n] = (int)total;
    } else {
      total = a.segs[n];  // scanned by launch_scan_excl
    }
    if (threadIdx.x == 0) a.counters[kCntRuns] = (unsigned long long)(total - a.rows);
  }
}

// one wave per chunk: cells in increasing order, stable within each bin
__device__ __forceinline__ void scatter_chunk(const FormArgs& a, long long c, int* pos) {
  const int lane = threadIdx.x & 63;
  for (int b = lane; b <= a.B; b += 64)
    pos[b] = (int)a.offsets[b] + a.cc[(long long)b * a.nblk + c];
  const long long base = c * a.chunk;
  const long long total = a.rows * a.pitch;
  long long row = (base + lane) / a.pitch;
  int col = (int)(base + lane - row * a.pitch);
  constexpr int kAhead = 16;  // codes of 16 steps in flight
  for (int q0 = 0; q0 < a.chunk; q0 += 64 * kAhead) {
    int code[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const long long p = base + q0 + 64 * u + lane;
      code[u] = q0 + 64 * u < a.chunk && p < total ? (int)a.binmap[p] : 4 * a.B;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int cell = (int)(row * a.nL + col);
      const int b = code[u] == 4 * a.B || col >= a.nL ? -2 : code[u] >> 2;
      col += 64;
      while (col >= a.pitch) {
        col -= a.pitch;
        ++row;
      }
      // lanes holding the same bin as this lane (found one distinct bin at a
      // time with ballots), then one LDS read of the bin's position per lane;
      // the highest lane of each bin advances it. The wave has its positions
      // to itself: its LDS reads and writes take effect in program order, so
      // no barrier.
      unsigned long long todo = __ballot(b >= 0), same = 0ull;
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int bl = __builtin_amdgcn_readlane(b, leader);
        const unsigned long long m = __ballot(b == bl);
        if (b == bl) same = m;
        todo &= ~m;
      }
      if (b >= 0) {
        const int start = pos[b];
        a.perm[start + __popcll(same & ((1ull << lane) - 1ull))] = (int32_t)cell;
        if ((same >> lane) == 1ull) pos[b] = start + __popcll(same);
      }
    }
  }
}

// run records and run indices of the 32 cells of block q of row r; pos: the
// block's first record
__device__ __forceinline__ void fill_runs(const FormArgs& a, long long r, int q, const Block32& blk,
                                          uint32_t starts, int rowstart, int pos) {
  int cur = pos - 1 - rowstart;  // run holding the cell before this block
  uint32_t idx[16];              // run indices of the 32 cells, two per word
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const int c = q * 32 + j;
    if ((starts >> j) & 1u) {
      a.runs[pos] = (uint32_t)c | (code_at(blk, j) << 16);
      cur = pos - rowstart;
      ++pos;
    } else if (c == a.nL) {
      // terminator: first column past the row, no bin
      a.runs[pos] = (uint32_t)a.nL | ((uint32_t)(4 * a.B) << 16);
      cur = pos - rowstart;
      ++pos;
    }
    if (j & 1) idx[j >> 1] |= (uint32_t)(uint16_t)cur << 16;
    else idx[j >> 1] = (uint32_t)(uint16_t)cur;
  }
  uint4* out = reinterpret_cast<uint4*>(a.runidx + r * a.pitch + q * 32);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    out[i] = make_uint4(idx[4 * i], idx[4 * i + 1], idx[4 * i + 2], idx[4 * i + 3]);
  if (q == a.nb - 1 && a.nL == a.nb * 32) {
    // row length is a multiple of 32: terminator after the last block
    a.runs[pos] = (uint32_t)a.nL | ((uint32_t)(4 * a.B) << 16);
  }
}

// the first workgroups build the tiled propagation's entries, the next fill
// the runs (`group` lanes per row segment), the others scatter (a wave per chunk)
__global__ __launch_bounds__(256) void k_fill(FormArgs a) {
  // [waves][B+1] running positions of the chunks, or TileEntriesLds
  extern __shared__ __align__(16) int pos[];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if ((int)blockIdx.x < a.entblocks) {
    tile_entries(a.ent, (int)blockIdx.x, *reinterpret_cast<TileEntriesLds*>(pos));
    return;
  }
  const int block = (int)blockIdx.x - a.entblocks;
  if (block >= a.rowblocks) {
    const long long c = (long long)(block - a.rowblocks) * a.swaves + w;
    if (w < a.swaves && c < a.nblk) scatter_chunk(a, c, pos + w * (a.B + 1));
    return;
  }
  const long long t = (long long)block * 256 + threadIdx.x;
  const long long sg = t / a.group;
  const bool in = sg < a.rows * a.nseg;
  const long long r = in ? sg / a.nseg : 0;
  const int part = (int)(sg - r * a.nseg);
  const int g = lane & (a.group - 1), q = part * kSegBlocks + g;
  const int rowstart = in ? a.segs[r * a.nseg] : 0;
  if (in && a.nseg > 1 && g == 0) {
    if (part == 0) a.rowptr[r] = rowstart;
    if (sg == a.rows * a.nseg - 1) a.rowptr[a.rows] = a.segs[sg + 1];
  }
  Block32 blk = {};
  uint32_t starts = 0;
  if (in && q < a.nb) {
    blk = load_block32(a.binmap + r * a.pitch, q);
    starts = run_starts(blk, q, a.nL);
  }
  const int cnt = __popc(starts);
  int incl = cnt;
  for (int o = 1; o < a.group; o <<= 1) {
    const int x = __shfl_up(incl, o, a.group);
    if (g >= o) incl += x;
  }
  if (in && q < a.nb) fill_runs(a, r, q, blk, starts, rowstart, a.segs[sg] + incl - cnt);
}

hipError_t launch_bin(const vup_mm& mm, const double* f, const double* edges, int32_t* bin,
                      hipStream_t s) {
  char* ws = static_cast<char*>(mm.ws);
  WsLayout L;
  ws_layout(mm.grid, mm.B, &L);
  BinArgs a{};
  a.f = f;
  a.edges_in = edges;
  a.edges_ws = reinterpret_cast<double*>(ws + mm.off_edges);
  a.bin = bin;
  a.binmap = reinterpret_cast<uint16_t*>(ws + mm.off_binmap);
  a.f32 = reinterpret_cast<float*>(ws + mm.off_f32);
  a.chunk_counts = reinterpret_cast<int*>(ws + mm.off_scratch);
  a.counters = reinterpret_cast<unsigned long long*>(ws + mm.off_counters);
  a.B = mm.B;
  a.nL = mm.grid.n[mm.grid.ndim - 1];
  a.pitch = mm.pitch;
  a.rows = mm.rows;
  a.nblk = L.nblk;
  a.chunk = L.chunk;
  const int nbx = (mm.grid.n[1] + kPX - 1) / kPX, nby = (mm.grid.n[0] + kPL - 1) / kPL;
  if (mm.grid.ndim == 2) {
    a.tblocks = reinterpret_cast<PtBlock*>(ws + L.off_tblocks);
    a.ntblocks = nbx * nby;
  }
  const size_t lds = (size_t)(mm.B + 1) * 8 + (size_t)(mm.B + 1) * 4;
  hipLaunchKernelGGL(k_bin, dim3((unsigned)L.nblk), dim3(256), lds, s, a);
  FormArgs m{};
  m.binmap = a.binmap;
  m.cc = a.chunk_counts;
  m.counts = reinterpret_cast<long long*>(ws + mm.off_counts);
  m.offsets = reinterpret_cast<long long*>(ws + mm.off_offsets);
  m.perm = reinterpret_cast<int32_t*>(ws + mm.off_perm);
  m.B = mm.B;
  m.nblk = L.nblk;
  m.chunk = L.chunk;
  m.runs = reinterpret_cast<uint32_t*>(ws + mm.off_runs);
  m.rowptr = reinterpret_cast<int*>(ws + mm.off_rowptr);
  m.runidx = reinterpret_cast<uint16_t*>(ws + mm.off_runidx);
  m.counters = a.counters;
  m.rows = mm.rows;
  m.nL = a.nL;
  m.pitch = a.pitch;
  m.nb = a.pitch / 32;
  m.group = 1;
  while (m.group < m.nb && m.group < 64) m.group *= 2;
  // one workgroup scans up to 16384 segments in four steps (12.4 us, 3.1
  // us at 1024 rows of one); more take three launches over many workgroups (13.8 us
  // at 110592 rows), where one workgroup would take 27 steps
  const long long nsegs = mm.rows * L.nseg;
  m.nseg = L.nseg;
  m.segs = L.nseg > 1 ? reinterpret_cast<int*>(ws + L.off_segs) : m.rowptr;
  m.scan_segs = nsegs <= 16384;
  const long long rowthreads = nsegs * m.group;
  hipLaunchKernelGGL(k_count, dim3((unsigned)(mm.B + 1 + (rowthreads + 255) / 256)), dim3(256), 0,
                     s, m);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (!m.scan_segs) {
    err = launch_scan_excl(m.segs, nsegs, reinterpret_cast<long long*>(ws + L.off_tsum),
                           m.segs + nsegs, s);
    if (err != hipSuccess) return err;
  }
  hipLaunchKernelGGL(k_offsets, dim3(2), dim3(1024), 0, s, m);
  m.rowblocks = (int)((rowthreads + 255) / 256);
  // four chunks per workgroup while their positions fit in 64 KB of LDS
  m.swaves = (size_t)(mm.B + 1) * 16 <= 65536 ? 4 : 2;
  size_t fill_lds = (size_t)(mm.B + 1) * 4 * m.swaves;
  if (mm.grid.ndim == 2) {
    m.ent.n[0] = mm.grid.n[0];
    m.ent.n[1] = mm.grid.n[1];
    m.ent.pitch = mm.pitch;
    m.ent.B = mm.B;
    m.ent.ntx = nbx;
    m.ent.binmap = a.binmap;
    m.ent.entries = reinterpret_cast<uint2*>(ws + L.off_tents);
    m.ent.chunks = reinterpret_cast<PtChunk*>(ws + L.off_tchunks);
    m.ent.blocks = a.tblocks;
    m.ent.cap = mm.N / 10;
    m.ent.counter = a.counters + kCntTiles;
    m.ent.extra = a.counters + kCntPasses;
    m.entblocks = nbx * nby;
    if (fill_lds < sizeof(TileEntriesLds)) fill_lds = sizeof(TileEntriesLds);
  }
  const long long blocks = m.entblocks + m.rowblocks + (L.nblk + m.swaves - 1) / m.swaves;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), fill_lds, s, m);
  return hipGetLastError();
}

__global__ void k_set_mode(unsigned long long* counters, int mode) {
  if (threadIdx.x == 0) counters[kCntMode] = (unsigned long long)mode;
}

hipError_t launch_set_mode(const vup_mm& mm, int mode, hipStream_t s) {
  unsigned long long* c =
      reinterpret_cast<unsigned long long*>(static_cast<char*>(mm.ws) + mm.off_counters);
  hipLaunchKernelGGL(k_set_mode, dim3(1), dim3(64), 0, s, c, mode);
  return hipGetLastError();
}

}  // namespace vup
