// Bayes inversion over the model matrix (Sec. 3, the Bayes theorem paragraph
// and its footnote): the columns of the "inverted model matrix",
//   post[t][i] = [bin(i) = b] p_k(x_i) / P[k][b],  k = sel[t],
// i.e. the posterior over input cells given that the output fell in bin b,
// relative to the forward propagation that produced P (and its per-component
// normalisation Z). p_k is the same truncated, normalised Gaussian mixture the
// propagation sums: FP32 per-axis factors (gauss_factor_r, each axis scaled by
// its power of two 2^m) and their product; the mixture weight, 2^-sum m,
// 1/Z_{k,c} and 1/P_b are combined in FP64 per bin and applied in FP32.
//   k_posterior       workgroups over grid rows: per-bin factors
//                     pi_c / (Z_c P_b) in LDS, the rows' factor products and
//                     the columns' factors staged, one multiply-add per cell
//                     and component
//   k_posterior_mean_tab  E[x_d | y in b, k] = sum over the bin's cells of
//                     post x_d, over the part of the model matrix's
//                     compressed-by-bin cell list inside the window's index
//                     range (fixed summation order)
//   k_posterior_mean  the same where factor tables do not fit or pay, one
//                     wave per (t, b), reading post
//
// 64 of 256 locations, 1000^2 cells, 1000 bins: k_posterior writes 256 MB in
// 40 us (82 us with a row's factors computed by every thread and one row in
// flight), the means 49 us (133 us reading post; 93 us from tables with a wave
// per bin, where the searches and wave sums of 64 000 bins of 300 cells cost
// more than the cells). Copies reach 5.1 TB/s, so k_posterior is bound by its
// stores; the means by their LDS gathers and the walk's instructions.
#include <hip/hip_runtime.h>

#include "vup_device.hpp"
#include "vup_inverse.hpp"

namespace vup {

struct PostArgs {
  int ndim;
  int n[4];
  double lo[4], hi[4];
  int pitch;                // padded length of the fastest axis in the bin map
  const uint16_t* binmap;   // 4 * bin, 4 * B for no bin
  const long long* offsets; // CSR row starts [B + 1]
  const int* perm;          // cells sorted by bin
  long long N, rows;
  int B;
  // distributions
  long long K;
  int C;
  double ns;
  const double* mu;
  const double* sigma;
  const double* weight;
  const long long* sel;
  long long n_sel;
  const float* P;
  const double* Z;
  float* post;
  double* mean;
  int gtab;                 // the fastest-axis factor table fits in LDS
  int vec;                  // rows of post take float4 stores (n_L % 4 == 0, aligned)
  double rn[4];             // 1 / n_d, for the index arithmetic of the means
};

// One workgroup per (rows of the grid, selected distribution t). Per
// workgroup: the distribution's windows and reciprocal deviations, and the
// factor f[c][b] = pi_c / (Z_c P[k][b]) of every bin (0 where P is 0), so a
// cell costs its fastest-axis factor and one multiply-add per component.
// Per row: the product of the other axes' factors (uniform over the row).
// COLS: a thread keeps the fastest-axis factors of its columns and goes down
// the workgroup's rows (with float4 stores only); otherwise the factors are
// formed once per workgroup, side by side, and kept in LDS.
constexpr int kPostRows = 64;  // rows whose factors are kept at once
template <bool COLS>
__global__ __launch_bounds__(256) void k_posterior(PostArgs a) {
  extern __shared__ float sfb[];  // [C][B + 1], then (!COLS, when it fits) fastest-axis factors [C][n_L]
  __shared__ int swin[VUP_MAX_COMP][VUP_MAX_DIM][2];
  __shared__ double smu[VUP_MAX_COMP][VUP_MAX_DIM], srs[VUP_MAX_COMP][VUP_MAX_DIM];
  __shared__ int sm[VUP_MAX_COMP][VUP_MAX_DIM];  // the factors' scale exponents
  __shared__ double sfac[VUP_MAX_COMP];            // pi_c 2^-sum_d m_d / Z_{k,c}
  __shared__ int sbad;
  const int t = blockIdx.y;
  const long long k = a.sel[t];
  const bool kok = k >= 0 && k < a.K;
  const int D = a.ndim, C = a.C, B = a.B;
  if (threadIdx.x == 0) sbad = kok ? 0 : 1;
  __syncthreads();
  if (threadIdx.x < C * D && kok) {
    const int c = threadIdx.x / D, d = threadIdx.x % D;
    const long long pidx = (k * C + c) * D + d;
    const double mu = a.mu[pidx], sg = a.sigma[pidx];
    int lo, hi;
    const bool ok = axis_window(a.lo[d], a.hi[d], a.n[d], mu, sg, a.ns, lo, hi);
    swin[c][d][0] = lo;
    swin[c][d][1] = hi;
    smu[c][d] = mu;
    srs[c][d] = 1.0 / sg;
    sm[c][d] = (ok && hi >= lo) ? axis_scale_exp(a.lo[d], a.hi[d], a.n[d], lo, hi, mu, 1.0 / sg)
                                : 0;
    if (!ok) atomicOr(&sbad, 1);
  }
  __syncthreads();
  if (threadIdx.x < C && kok) {
    // the scaled factors' product is 2^(sum_d m_d) times the density, as in
    // the propagation that reported Z
    const int c = threadIdx.x;
    int ms = 0;
    for (int d = 0; d < D; ++d) ms += sm[c][d];
    const double z = a.Z[k * C + c];
    const double w = C > 1 ? a.weight[k * C + c] : 1.0;
    sfac[c] = ldexp(w / z, -ms);
    if (!isfinite(z)) atomicOr(&sbad, 1);
  }
  __syncthreads();
  if (kok) {
    for (int e = threadIdx.x; e < C * B; e += blockDim.x) {
      const int c = e / B, b = e - c * B;
      const float ev = a.P[k * B + b];
      if (!isfinite(ev)) atomicOr(&sbad, 1);
      sfb[c * (B + 1) + b] = ev > 0.0f ? (float)(sfac[c] / (double)ev) : 0.0f;
    }
  }
  if (threadIdx.x < C) sfb[threadIdx.x * (B + 1) + B] = 0.0f;  // cells without a bin
  const int nL = a.n[D - 1];
  // the fastest-axis factor of every column inside each component's window,
  // shared by all rows of this distribution
  float* gtab = sfb + C * (B + 1);
  if (!COLS && a.gtab && kok) {
    // only the window's columns: the cells read no others
    for (int c = 0; c < C; ++c) {
      const int wlo = swin[c][D - 1][0], whi = swin[c][D - 1][1];
      for (int col = wlo + (int)threadIdx.x; col <= whi; col += blockDim.x)
        gtab[c * nL + col] = gauss_factor_r(cell_centre(a.lo[D - 1], a.hi[D - 1], nL, col),
                                            smu[c][D - 1], srs[c][D - 1],
                                            scale_log(sm[c][D - 1]));
    }
  }
  __syncthreads();
  const bool bad = sbad != 0;
  float* post = a.post + (long long)t * a.N;
  // a row's factor product per component (0 outside the component's window)
  // and the columns any window covers; outside them, and in rows no window
  // covers, post is 0 (NaN for an invalid distribution)
  struct RowInfo {
    float rf[VUP_MAX_COMP];
    int clo[VUP_MAX_COMP], chi[VUP_MAX_COMP];
    int ulo, uhi;
  };
  auto row_info = [&](int r, RowInfo& ri) {
    int j[4] = {0, 0, 0, 0};
    int q = r;
    for (int d = D - 2; d >= 0; --d) {
      j[d] = q % a.n[d];
      q /= a.n[d];
    }
    ri.ulo = 0x7fffffff;
    ri.uhi = -1;
#pragma unroll
    for (int c = 0; c < VUP_MAX_COMP; ++c) {
      ri.rf[c] = 0.0f;
      ri.clo[c] = 0;
      ri.chi[c] = -1;
      if (c < C) {
        bool in = true;
        float f = 1.0f;
        for (int d = 0; d + 1 < D; ++d) {
          in = in && j[d] >= swin[c][d][0] && j[d] <= swin[c][d][1];
          if (in) f *= gauss_factor_r(cell_centre(a.lo[d], a.hi[d], a.n[d], j[d]), smu[c][d],
                                      srs[c][d], scale_log(sm[c][d]));
        }
        if (in && swin[c][D - 1][1] >= swin[c][D - 1][0]) {
          ri.rf[c] = f;
          ri.clo[c] = swin[c][D - 1][0];
          ri.chi[c] = swin[c][D - 1][1];
          ri.ulo = min(ri.ulo, ri.clo[c]);
          ri.uhi = max(ri.uhi, ri.chi[c]);
        }
      }
    }
  };
  auto cell = [&](const RowInfo& ri, int col, uint32_t code) {
    float v = 0.0f;
    if (code < 4u * (uint32_t)B) {
      const int b = (int)(code >> 2);
#pragma unroll
      for (int c = 0; c < VUP_MAX_COMP; ++c) {
        if (c < C && col >= ri.clo[c] && col <= ri.chi[c]) {
          const float g = a.gtab ? gtab[c * nL + col]
                                 : gauss_factor_r(cell_centre(a.lo[D - 1], a.hi[D - 1], nL, col),
                                                  smu[c][D - 1], srs[c][D - 1],
                                                  scale_log(sm[c][D - 1]));
          v = fmaf(ri.rf[c] * g, sfb[c * (B + 1) + b], v);
        }
      }
    }
    return v;
  };
  if constexpr (COLS) {
    // A thread owns four columns: their fastest-axis factors stay in registers
    // (-1 outside the component's window) while it goes down the workgroup's
    // rows, four rows at once (four 8-byte loads of bin codes, four 16-byte
    // stores). A row's factor products are computed once per 64 rows, one row
    // per thread.
    __shared__ float srow[kPostRows][VUP_MAX_COMP];
    const float fill = bad ? __builtin_nanf("") : 0.0f;
    const int n4 = nL >> 2;
    int tx = 256;
    while (tx > 4 && tx / 2 >= n4) tx >>= 1;  // threads along a row
    const int ty = 256 / tx;
    const int x = threadIdx.x & (tx - 1), y = threadIdx.x / tx;
    const int stride = gridDim.x;
    for (int rbase = blockIdx.x; rbase < a.rows; rbase += kPostRows * stride) {
      const int nr = min(kPostRows, (int)((a.rows - rbase + stride - 1) / stride));
      __syncthreads();
      if ((int)threadIdx.x < nr) {
        RowInfo ri;
        row_info(rbase + (int)threadIdx.x * stride, ri);
#pragma unroll
        for (int c = 0; c < VUP_MAX_COMP; ++c)
          srow[threadIdx.x][c] = ri.chi[c] >= ri.clo[c] ? ri.rf[c] : -1.0f;
      }
      __syncthreads();
      for (int c4 = x; c4 < n4; c4 += tx) {
        const int col0 = 4 * c4;
        float g[VUP_MAX_COMP][4];
        bool any = false;
#pragma unroll
        for (int c = 0; c < VUP_MAX_COMP; ++c) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            g[c][e] = -1.0f;
            if (c < C && !bad && col0 + e >= swin[c][D - 1][0] && col0 + e <= swin[c][D - 1][1]) {
              g[c][e] = gauss_factor_r(cell_centre(a.lo[D - 1], a.hi[D - 1], nL, col0 + e),
                                       smu[c][D - 1], srs[c][D - 1], scale_log(sm[c][D - 1]));
              any = true;
            }
          }
        }
        constexpr int U = 4;
        for (int q0 = y; q0 < nr; q0 += U * ty) {
          uint2 cw[U];
          float rf[U][VUP_MAX_COMP];
          bool on[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = min(q0 + u * ty, nr - 1);
            on[u] = false;
#pragma unroll
            for (int c = 0; c < VUP_MAX_COMP; ++c) {
              rf[u][c] = srow[q][c];
              on[u] = on[u] || rf[u][c] >= 0.0f;
            }
            on[u] = on[u] && any;
            cw[u] = make_uint2(0u, 0u);
            if (on[u])
              cw[u] = *reinterpret_cast<const uint2*>(
                  a.binmap + (long long)(rbase + q * stride) * a.pitch + col0);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int q = q0 + u * ty;
            float o[4] = {fill, fill, fill, fill};
            if (on[u]) {
              const uint32_t code[4] = {cw[u].x & 0xFFFFu, cw[u].x >> 16, cw[u].y & 0xFFFFu,
                                        cw[u].y >> 16};
#pragma unroll
              for (int c = 0; c < VUP_MAX_COMP; ++c) {
                if (c < C && rf[u][c] >= 0.0f) {
#pragma unroll
                  for (int e = 0; e < 4; ++e) {
                    const float fb = *reinterpret_cast<const float*>(
                        reinterpret_cast<const char*>(sfb + c * (B + 1)) + code[e]);
                    const float v = fmaf(rf[u][c] * g[c][e], fb, o[e]);
                    if (g[c][e] >= 0.0f) o[e] = v;
                  }
                }
              }
            }
            if (q < nr)
              *reinterpret_cast<float4*>(post + (long long)(rbase + q * stride) * nL + col0) =
                  make_float4(o[0], o[1], o[2], o[3]);
          }
        }
      }
    }
  } else if (a.vec) {
    // four columns per thread: one 8-byte load of bin codes, one 16-byte store
    const float fill = bad ? __builtin_nanf("") : 0.0f;
    for (int r = blockIdx.x; r < a.rows; r += gridDim.x) {
      RowInfo ri;
      row_info(r, ri);
      const uint16_t* brow = a.binmap + (long long)r * a.pitch;
      float4* prow4 = reinterpret_cast<float4*>(post + (long long)r * nL);
      for (int c4 = threadIdx.x; c4 < (nL >> 2); c4 += blockDim.x) {
        const int col0 = 4 * c4;
        float4 o = make_float4(fill, fill, fill, fill);
        if (!bad && col0 + 3 >= ri.ulo && col0 <= ri.uhi) {
          const uint2 cw = *reinterpret_cast<const uint2*>(brow + col0);
          o.x = cell(ri, col0, cw.x & 0xFFFFu);
          o.y = cell(ri, col0 + 1, cw.x >> 16);
          o.z = cell(ri, col0 + 2, cw.y & 0xFFFFu);
          o.w = cell(ri, col0 + 3, cw.y >> 16);
        }
        prow4[c4] = o;
      }
    }
  } else {
    for (int r = blockIdx.x; r < a.rows; r += gridDim.x) {
      RowInfo ri;
      row_info(r, ri);
      const uint16_t* brow = a.binmap + (long long)r * a.pitch;
      float* prow = post + (long long)r * nL;
      for (int col = threadIdx.x; col < nL; col += blockDim.x) {
        float v = 0.0f;
        if (col >= ri.ulo && col <= ri.uhi) v = cell(ri, col, brow[col]);
        prow[col] = bad ? __builtin_nanf("") : v;
      }
    }
  }
}

// first positions s in [s0, s1) of the ascending cell list with list[s] >= x0
// and with list[s] >= x1 (s1 if none), by the whole wave, both searches in the
// same rounds (their loads in flight together): each round probes 64
// positions spread over a search's remaining range and keeps the part between
// the last probe below its target and the first at or above it, so a range of
// n shrinks to n / 65 per round
struct WaveSearch {
  long long lo, hi;  // the answer lies in [lo, hi]
};

__device__ __forceinline__ long long probe_at(const WaveSearch& w, int i) {
  return w.lo + ((w.hi - w.lo) * (i + 1)) / 65;  // in (lo, hi) while hi - lo > 64
}

__device__ __forceinline__ void narrow(WaveSearch& w, bool ge) {
  const unsigned long long m = __ballot(ge);
  const int f = m ? __builtin_ctzll(m) : 64;  // first probe at or above the target
  const long long pf = probe_at(w, f), pb = probe_at(w, f - 1);
  if (f < 64) w.hi = pf;
  if (f > 0) w.lo = pb + 1;
}

__device__ __forceinline__ long long finish_search(const int* list, const WaveSearch& w,
                                                   long long x, int lane) {
  const long long p = w.lo + lane;
  const bool ge = p < w.hi && (long long)list[p] >= x;
  const unsigned long long m = __ballot(ge);
  return m ? w.lo + __builtin_ctzll(m) : w.hi;
}

__device__ __forceinline__ void wave_lower_bounds(const int* list, long long s0, long long s1,
                                                  long long x0, long long x1, int lane,
                                                  long long& r0, long long& r1) {
  WaveSearch a{s0, s1}, b{s0, s1};
  for (;;) {
    const bool on_a = a.hi - a.lo > 64, on_b = b.hi - b.lo > 64;  // uniform
    if (!on_a && !on_b) break;
    const int va = on_a ? list[probe_at(a, lane)] : 0;
    const int vb = on_b ? list[probe_at(b, lane)] : 0;
    if (on_a) narrow(a, (long long)va >= x0);
    if (on_b) narrow(b, (long long)vb >= x1);
  }
  r0 = finish_search(list, a, x0, lane);
  r1 = finish_search(list, b, x1, lane);
}

// The means without reading post: a workgroup per (t, a stretch of bins) keeps
// the factor tables of all axes in LDS and forms a cell's posterior again from
// its factors, with k_posterior's operations in k_posterior's order
// (bit-identical), so the cells' 4-byte gathers from post, each a 128-byte
// line from memory for a bin one cell wide, fall away. The parts of the bins'
// lists inside the window's index range are found first, a thread per bin and
// end; then LPB lanes walk a bin (lane l the cells l, l + LPB, ... of its
// part) and their sums are taken in a fixed order.
// sum over the lane's row of 16 lanes, given to all of them
__device__ __forceinline__ double row_last(double v) {
  const long long b = __double_as_longlong(row_scan(v));
  const int src = (threadIdx.x & 63) | 15;
  const int lo = __shfl((int)(b & 0xFFFFFFFF), src, 64), hi = __shfl((int)(b >> 32), src, 64);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

struct MeanDiv {
  uint32_t mul[4];  // j / n_d = mulhi(j, mul) >> shift for j < 2^31 (n_d > 1)
  int shift[4];
};

template <int D, int C, int LPB>
__global__ __launch_bounds__(256) void k_posterior_mean_tab(PostArgs a, MeanDiv dv, int per) {
  // [C][n_0 + ... + n_(D-1)] factors, -1 outside the component's window;
  // [2][per] ends of the bins' parts
  extern __shared__ float tab[];
  __shared__ int swin[C][D][2];
  __shared__ double smu[C][D], srs[C][D];
  __shared__ int sm[C][D];
  __shared__ double sfac[C];
  __shared__ int sbad;
  const long long t = blockIdx.y;
  const long long k = a.sel[t];
  const bool kok = k >= 0 && k < a.K;
  if (threadIdx.x == 0) sbad = kok ? 0 : 1;
  __syncthreads();
  if (threadIdx.x < C * D && kok) {
    const int c = threadIdx.x / D, d = threadIdx.x % D;
    const long long pidx = (k * C + c) * D + d;
    const double mu = a.mu[pidx], sg = a.sigma[pidx];
    int lo, hi;
    const bool ok = axis_window(a.lo[d], a.hi[d], a.n[d], mu, sg, a.ns, lo, hi);
    swin[c][d][0] = lo;
    swin[c][d][1] = hi;
    smu[c][d] = mu;
    srs[c][d] = 1.0 / sg;
    sm[c][d] = (ok && hi >= lo) ? axis_scale_exp(a.lo[d], a.hi[d], a.n[d], lo, hi, mu, 1.0 / sg)
                                : 0;
    if (!ok) atomicOr(&sbad, 1);
  }
  if (kok)
    for (int e = threadIdx.x; e < a.B; e += 256)
      if (!isfinite(a.P[k * a.B + e])) atomicOr(&sbad, 1);
  __syncthreads();
  if (threadIdx.x < C && kok) {
    const int c = threadIdx.x;
    int ms = 0;
    for (int d = 0; d < D; ++d) ms += sm[c][d];
    const double z = a.Z[k * C + c];
    const double w = C > 1 ? a.weight[k * C + c] : 1.0;
    sfac[c] = ldexp(w / z, -ms);
    if (!isfinite(z)) atomicOr(&sbad, 1);
  }
  __syncthreads();
  const bool bad = sbad != 0;
  int blo[D], bhi[D], base[D + 1];
  base[0] = 0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    blo[d] = 0x7fffffff;
    bhi[d] = -1;
    base[d + 1] = base[d] + a.n[d];
  }
  bool any = false;  // some component's window is not empty
  if (!bad) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      bool cin = true;
#pragma unroll
      for (int d = 0; d < D; ++d) cin = cin && swin[c][d][1] >= swin[c][d][0];
      any = any || cin;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int lo = swin[c][d][0], hi = swin[c][d][1];
        if (cin) {
          blo[d] = min(blo[d], lo);
          bhi[d] = max(bhi[d], hi);
        }
        const double mu = smu[c][d], rs = srs[c][d], off = scale_log(sm[c][d]);
        for (int i = threadIdx.x; i < a.n[d]; i += 256)
          tab[c * base[D] + base[d] + i] =
              cin && i >= lo && i <= hi
                  ? gauss_factor_r(cell_centre(a.lo[d], a.hi[d], a.n[d], i), mu, rs, off)
                  : -1.0f;
      }
    }
  }
  // ends of the bins' parts: first positions with a cell >= first and > last,
  // by three probes a step
  int* ends = reinterpret_cast<int*>(tab + C * base[D]);
  const int b0 = blockIdx.x * per, nb = min(per, a.B - b0);
  if (!bad && any) {
    long long first = 0, last = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      first = first * a.n[d] + blo[d];
      last = last * a.n[d] + bhi[d];
    }
    for (int e = threadIdx.x; e < 2 * nb; e += 256) {
      const int b = b0 + (e >> 1);
      const int x = (int)((e & 1) ? last + 1 : first);  // at most the number of cells
      int lo = (int)a.offsets[b], hi = (int)a.offsets[b + 1];
      while (lo < hi) {
        const int q = (hi - lo) >> 2;
        const int p0 = lo + q, p1 = lo + ((hi - lo) >> 1), p2 = hi - 1 - q;
        const int v0 = a.perm[p0], v1 = a.perm[p1], v2 = a.perm[max(p2, p1)];
        if (v0 >= x) hi = p0;
        else if (v1 >= x) { lo = p0 + 1; hi = p1; }
        else if (v2 >= x) { lo = p1 + 1; hi = max(p2, p1); }
        else lo = max(p2, p1) + 1;
      }
      ends[e] = lo;
    }
  }
  __syncthreads();
  constexpr int G = 64 / LPB;  // bins of a wave
  const int lane = threadIdx.x & 63, l = lane & (LPB - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the bins are dealt out by the wave's number, a uniform value, and the
  // wave is kept together at the end of each)
  for (int g0 = w * G; g0 < nb; g0 += 4 * G) {
    const int g = g0 + lane / LPB;
    const int b = b0 + g;
    const bool live = g < nb;
    const float ev = live && kok ? a.P[k * a.B + b] : 0.0f;
    // a bin without mass has post 0 on all its cells (k_posterior's factor is
    // 0 there): its sums are exact zeros
    const bool on = live && !bad && any && ev > 0.0f;
    float fb[C];
    int s = 0, e = 0;
    if (on) {
#pragma unroll
      for (int c = 0; c < C; ++c) fb[c] = (float)(sfac[c] / (double)ev);
      s = ends[2 * g];
      e = ends[2 * g + 1];
    }
    double S0 = 0.0, S[D];
#pragma unroll
    for (int d = 0; d < D; ++d) S[d] = 0.0;
    constexpr int U = 4;  // cells per lane and step, their loads in flight together
    for (s += l; s < e; s += LPB * U) {
      int ci[U];
#pragma unroll
      for (int u = 0; u < U; ++u) ci[u] = s + LPB * u < e ? a.perm[s + LPB * u] : -1;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int j[D];
        uint32_t rest = ci[u] < 0 ? 0u : (uint32_t)ci[u];
#pragma unroll
        for (int d = D - 1; d >= 1; --d) {
          const uint32_t quo = a.n[d] == 1 ? rest : __umulhi(rest, dv.mul[d]) >> dv.shift[d];
          j[d] = (int)(rest - quo * (uint32_t)a.n[d]);
          rest = quo;
        }
        j[0] = (int)rest;
        float v = 0.0f;
        bool in = false;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          // the slower axes' product, then the fastest axis' factor
          float f = 1.0f, fac = 1.0f;
          bool cin = ci[u] >= 0;
#pragma unroll
          for (int d = 0; d < D; ++d) {
            fac = tab[c * base[D] + base[d] + j[d]];
            cin = cin && fac >= 0.0f;
            if (d + 1 < D) f *= fac;
          }
          const float x = fmaf(f * fac, fb[c], v);
          if (cin) v = x;
          in = in || cin;
        }
        const double qd = in ? (double)v : 0.0;
        S0 += qd;
#pragma unroll
        for (int d = 0; d < D; ++d) S[d] += qd * (double)j[d];
      }
    }
    double mine = 0.0;  // lane d of a bin: component d
    S0 = LPB == 64 ? wave_sum(S0) : row_last(S0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const double Sd = LPB == 64 ? wave_sum(S[d]) : row_last(S[d]);
      const double h = (a.hi[d] - a.lo[d]) / a.n[d];
      const double md = a.lo[d] * S0 + h * (Sd + 0.5 * S0);
      if (l == d) mine = md;
    }
    if (live && l < D) {
      // NaN where the posterior row is NaN (0 for a bin without cells)
      if (!on) mine = bad && a.offsets[b + 1] > a.offsets[b] ? __builtin_nan("") : 0.0;
      a.mean[(t * a.B + b) * D + l] = mine;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <int D>
static void launch_mean_tab(const PostArgs& a, const MeanDiv& dv, int per, bool narrow, dim3 grid,
                            size_t lds, hipStream_t s) {
  void (*kern)(PostArgs, MeanDiv, int) =
      a.C == 1 ? (narrow ? k_posterior_mean_tab<D, 1, 16> : k_posterior_mean_tab<D, 1, 64>)
               : (narrow ? k_posterior_mean_tab<D, 2, 16> : k_posterior_mean_tab<D, 2, 64>);
  hipLaunchKernelGGL(kern, grid, dim3(256), lds, s, a, dv, per);
}

// one wave per (t, b): lanes take the bin's cells lane, lane + 64, ... of the
// compressed-by-bin list; the wave sum fixes the order. Only the part of the
// list inside the row-major index range of the distribution's window (the
// bounding box of its components' windows) can hold nonzero posteriors: the
// wave finds it by search and walks it with the same lane assignment as a
// walk of the whole list, skipping the loads of cells outside the box (their
// terms are exact zeros), so the sums do not depend on the skipping. With
// cell centres x_d = lo_d + (j_d + 1/2) h_d, the sums are kept as S0 = sum q
// and S_d = sum q j_d (FP64) and combined at the end; the row-major index is
// split with a double reciprocal and one correction step.
__global__ __launch_bounds__(256) void k_posterior_mean(PostArgs a) {
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
  const long long t = blockIdx.y;
  if (b >= a.B) return;  // whole waves leave together
  const long long s0 = a.offsets[b], s1 = a.offsets[b + 1];
  const float* post = a.post + t * a.N;
  const int D = a.ndim, C = a.C;
  double* out = a.mean + (t * a.B + b) * a.ndim;
  // the posterior row is NaN (the same conditions as k_posterior): mean NaN,
  // 0 for a bin without cells
  const long long k = a.sel[t];
  bool bad = !(k >= 0 && k < a.K);
  int blo[4] = {0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff}, bhi[4] = {-1, -1, -1, -1};
  bool any = false;  // some component's window is not empty
  if (!bad) {
    for (int c = 0; c < C; ++c) {
      bool cin = true;
      int wl[4], wh[4];
      for (int d = 0; d < D; ++d) {
        const long long pidx = (k * C + c) * D + d;
        if (!axis_window(a.lo[d], a.hi[d], a.n[d], a.mu[pidx], a.sigma[pidx], a.ns, wl[d], wh[d]))
          bad = true;
        cin = cin && wh[d] >= wl[d];
      }
      if (!isfinite(a.Z[k * C + c])) bad = true;
      if (cin) {
        any = true;
        for (int d = 0; d < D; ++d) {
          blo[d] = min(blo[d], wl[d]);
          bhi[d] = max(bhi[d], wh[d]);
        }
      }
    }
    for (int e = lane; e < a.B; e += 64)
      if (!isfinite(a.P[k * a.B + e])) bad = true;
    bad = __ballot(bad) != 0;
  }
  // a bin without mass has post 0 on all its cells (k_posterior's factor is 0
  // there): its sums are exact zeros, so the mean is 0 without a walk
  if (bad || !any || !(a.P[k * a.B + b] > 0.0f)) {
    if (lane < D) out[lane] = (bad && s1 > s0) ? __builtin_nan("") : 0.0;
    return;
  }
  // row-major index range of the window box, and its part of the list
  long long first = 0, last = 0;
  for (int d = 0; d < D; ++d) {
    first = first * a.n[d] + blo[d];
    last = last * a.n[d] + bhi[d];
  }
  long long sa, sb;
  wave_lower_bounds(a.perm, s0, s1, first, last + 1, lane, sa, sb);
  double S0 = 0.0, S[4] = {0.0, 0.0, 0.0, 0.0};
  // four cells per lane per pass, their loads in flight together; lane l
  // takes the cells s0 + l + 64 m in increasing m whatever the pass size, so
  // the sums are those of a walk of the whole list
  constexpr int U = 4;
  // start at the pass of the whole-list walk that reaches sa
  const long long sstart = s0 + ((sa - s0) / (64 * U)) * (64 * U);
  for (long long s = sstart + lane; s < sb; s += 64 * U) {
    int ci[U], jd[U][4];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long su = s + 64 * u;
      ci[u] = (su >= sa && su < sb) ? a.perm[su] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      in[u] = ci[u] >= 0;
      int rest = ci[u] < 0 ? 0 : ci[u];
#pragma unroll
      for (int d = 3; d >= 1; --d) {
        jd[u][d] = 0;
        if (d < D) {
          const int n = a.n[d];
          int quo = (int)((double)rest * a.rn[d]);
          int rem = rest - quo * n;
          if (rem < 0) {
            --quo;
            rem += n;
          } else if (rem >= n) {
            ++quo;
            rem -= n;
          }
          jd[u][d] = rem;
          in[u] = in[u] && rem >= blo[d] && rem <= bhi[d];
          rest = quo;
        }
      }
      jd[u][0] = rest;
      in[u] = in[u] && rest >= blo[0] && rest <= bhi[0];
    }
    float q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = in[u] ? post[ci[u]] : 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!in[u]) continue;
      const double qd = (double)q[u];
      S0 += qd;
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (d < D) S[d] += qd * (double)jd[u][d];
    }
  }
  S0 = wave_sum(S0);
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    if (d < D) {
      const double Sd = wave_sum(S[d]);
      const double h = (a.hi[d] - a.lo[d]) / a.n[d];
      if (lane == 0) out[d] = a.lo[d] * S0 + h * (Sd + 0.5 * S0);
    }
  }
}

hipError_t launch_posterior(const vup_mm& mm, const vup_dists& d, int64_t n_sel,
                            const int64_t* sel, const float* P, const double* Z, float* post,
                            double* mean, hipStream_t s) {
  if (n_sel == 0) return hipSuccess;
  PostArgs a{};
  a.ndim = mm.grid.ndim;
  for (int x = 0; x < 4; ++x) {
    a.n[x] = x < a.ndim ? mm.grid.n[x] : 1;
    a.lo[x] = mm.grid.lo[x];
    a.hi[x] = mm.grid.hi[x];
  }
  a.pitch = mm.pitch;
  const char* ws = static_cast<const char*>(mm.ws);
  a.binmap = reinterpret_cast<const uint16_t*>(ws + mm.off_binmap);
  a.offsets = reinterpret_cast<const long long*>(ws + mm.off_offsets);
  a.perm = reinterpret_cast<const int*>(ws + mm.off_perm);
  a.N = mm.N;
  a.rows = mm.rows;
  a.B = mm.B;
  a.K = d.K;
  a.C = d.ncomp;
  a.ns = d.n_sigma;
  a.mu = d.mu;
  a.sigma = d.sigma;
  a.weight = d.weight;
  a.sel = reinterpret_cast<const long long*>(sel);
  a.n_sel = n_sel;
  a.P = P;
  a.Z = Z;
  a.post = post;
  a.mean = mean;
  for (int x = 0; x < 4; ++x) a.rn[x] = 1.0 / a.n[x];
  const int nL = a.n[a.ndim - 1];
  a.vec = (nL % 4 == 0) && ((reinterpret_cast<uintptr_t>(post) & 15u) == 0);
  a.gtab = (size_t)d.ncomp * (mm.B + 1 + nL) * sizeof(float) <= 65536 ? 1 : 0;
  // about 32 rows per workgroup, so the per-bin factors and the factor table
  // are set up rarely, but at least 2048 workgroups in all while rows last
  // (4096 where they have few rows each)
  auto groups = [&](long long least) {
    long long gx = (mm.rows + 31) / 32;
    const long long want = (least + n_sel - 1) / n_sel;
    if (gx < want) gx = want < mm.rows ? want : mm.rows;
    return gx < 1 ? 1 : (gx > 4096 ? 4096 : gx);
  };
  long long gx = groups(2048);
  // Factors in registers pay from two rows per workgroup on (1000^2 cells: 4
  // locations, two rows, 18.5 -> 16.0 us, 64 locations, 31 rows, 77 -> 40; 20^4
  // cells, 8 locations 101 -> 16). A thread forms its four columns' factors one
  // after the other, which a single row does not pay back: 1000^2 cells, one
  // location 7.8 us side by side, 9.1 so; 10 x 4096, 64 locations 9.2 and 13.8.
  const bool cols = a.vec && mm.rows >= 2 * gx;
  if (!cols) gx = groups(4096);
  const size_t lds = (size_t)d.ncomp * (mm.B + 1 + (a.gtab && !cols ? nL : 0)) * sizeof(float);
  const dim3 grid((unsigned)gx, (unsigned)n_sel);
  if (cols) hipLaunchKernelGGL(k_posterior<true>, grid, dim3(256), lds, s, a);
  else hipLaunchKernelGGL(k_posterior<false>, grid, dim3(256), lds, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !mean) return e;
  size_t tab = 0;
  for (int x = 0; x < a.ndim; ++x) tab += (size_t)a.n[x];
  tab *= d.ncomp * sizeof(float);
  // Tables up to 32 KB leave four workgroups to a CU. A quarter of a wave per
  // bin fills the chip from 16 384 bins on, 16 bins to a workgroup, one for each
  // of its groups of lanes, so that they share its tables (64 locations, 1000^2
  // cells, 1000 bins, the kernel: 48 us, 56 with 32 bins, 69 with 64, 93 with a
  // wave per bin, 131 reading post), more bins once there are 4096 workgroups.
  // Fewer bins take a wave each, four to a workgroup while there are fewer than
  // 1024 (48^4 cells, 256 bins of one location, the call: 468 us reading post
  // with a wave per bin, 582 from tables with 16 bins to a workgroup, 172 so).
  // Long tables for few and small bins are not worth forming (8000 cells on one
  // axis, 64 bins, the call: one location 14.4 us reading post, 17 from tables;
  // four locations 21.7 and 20.0).
  const long long bins = n_sel * mm.B;
  const bool narrow = bins >= 16384;
  long long per = narrow ? (bins + 4095) / 4096 : bins / 1024;
  if (per < (narrow ? 16 : 4)) per = narrow ? 16 : 4;
  if (per > 256) per = 256;
  const long long entries = (long long)(tab / sizeof(float));
  if (tab <= 32768 && (48 * bins >= entries || mm.N >= entries * mm.B)) {
    MeanDiv dv{};
    for (int x = 0; x < a.ndim; ++x) {
      int l = 0;
      while ((1ll << l) < a.n[x]) ++l;
      // ceil(2^(31 + l) / n) < 2^32, exact for dividends below 2^31
      if (l > 0) {
        dv.mul[x] = (uint32_t)(((1ull << (31 + l)) + a.n[x] - 1) / a.n[x]);
        dv.shift[x] = l - 1;
      }
    }
    const dim3 mgrid((unsigned)((mm.B + per - 1) / per), (unsigned)n_sel);
    const size_t mlds = tab + 2 * (size_t)per * sizeof(int);
    if (a.ndim == 1) launch_mean_tab<1>(a, dv, (int)per, narrow, mgrid, mlds, s);
    else if (a.ndim == 2) launch_mean_tab<2>(a, dv, (int)per, narrow, mgrid, mlds, s);
    else if (a.ndim == 3) launch_mean_tab<3>(a, dv, (int)per, narrow, mgrid, mlds, s);
    else launch_mean_tab<4>(a, dv, (int)per, narrow, mgrid, mlds, s);
  } else {
    hipLaunchKernelGGL(k_posterior_mean, dim3((unsigned)((mm.B + 3) / 4), (unsigned)n_sel),
                       dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace vup
