// The entries of the tiled propagation: their layout, and the construction of
// a block's entries (vup_bin's last launch, next to the run records).
#ifndef VUP_K_PTILES_HPP
#define VUP_K_PTILES_HPP

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/vup.h"

namespace vup {
namespace {

constexpr int kPX = 64;            // tile columns
constexpr int kPL = 64;            // rows of a block of entries
constexpr int kPR = 4;             // rows of a chunk
constexpr int kPCh = kPL / kPR;    // chunks of a block
constexpr int kPEnt = 128;         // entries a chunk may have
constexpr int kPSlots = 120;       // bins a pass over a tile covers: two workgroups' LDS fit on a CU
constexpr int kPNoBin = 0xFFFF;    // entry of cells without a bin

// one chunk's entries
struct PtChunk {
  uint32_t first;  // index of the first entry
  uint32_t n;      // entries (an even number)
  int mn, mx;      // lowest and highest bin (mn > mx: none); mn -1: cells without one
};
static_assert(sizeof(PtChunk) == 16, "chunk layout");

// a block's bins
struct PtBlock {
  int16_t mn, mx;
  int none;                 // it has cells without a bin
  unsigned long long both;  // in the first of a tile's two blocks: the bins of those built
};
static_assert(sizeof(PtBlock) == 16, "block layout");

// the entries of a model matrix (in vup_bin's workspace)
struct PtEntArgs {
  int n[2];
  int pitch, B, ntx;
  const uint16_t* __restrict__ binmap;
  uint2* entries;               // four columns (a byte each); bin | byte offset of its slot << 16
  PtChunk* chunks;              // [blocks][kPCh]
  PtBlock* blocks;              // [blocks]
  long long cap;                // entries there is room for
  unsigned long long* counter;  // entries; kPUnfit and more: they do not fit
  unsigned long long* extra;    // passes over the tiles past the first over each
};
constexpr unsigned long long kPUnfit = 1ull << 40;

// byte offset of a slot's lane 0 in the sums of k_pt_main (8 bytes each): slot
// s, lane l is number 64 s + (l xor s mod 64), so that both the lanes of a slot
// and the slots of a lane fall evenly on the banks
__device__ __forceinline__ uint32_t slot_code(int s) {
  return (uint32_t)s * 512u + ((uint32_t)s & 63u) * 8u;
}
static_assert((kPSlots + 2) * 512 <= 65536, "16 bits of an entry");

// passes over a tile of bins mn .. mx
__device__ __forceinline__ int tile_passes(int mn, int mx) {
  return mx >= mn ? (mx - mn) / kPSlots + 1 : 1;
}

template <int CTRL>
__device__ __forceinline__ int quad(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ int quad_min(int v) {
  v = min(v, quad<0xB1>(v));
  return min(v, quad<0x4E>(v));
}
__device__ __forceinline__ int quad_max(int v) {
  v = max(v, quad<0xB1>(v));
  return max(v, quad<0x4E>(v));
}
__device__ __forceinline__ int quad_or(int v) {
  v |= quad<0xB1>(v);
  return v | quad<0x4E>(v);
}

// ---------------------------------------------------------------------------
// entries of one block of 64 x 64 cells (256 threads): a wave per rule; in
// each, lane r walks row r, four lanes a chunk. A chunk keeps the shortest of
// its three lists, of equally short ones that of the first rule: lists are
// compared by their own lengths (before they are made even), the same that a
// wave gives up against, so that every list that could win is whole and the
// choice does not depend on which wave comes first. Bound by the latency of one row's walk (about 50 steps at
// 1024^2 cells and 256 bins); the workgroups of a grid of 1024^2 all run at
// once, next to those of the scatter and the run records.
// ---------------------------------------------------------------------------
constexpr int kPRules = 3;

struct TileEntriesLds {
  uint16_t code[kPL][kPX + 2];
  unsigned long long starts[kPL];
  uint32_t cols[kPRules][kPCh][kPEnt];
  uint16_t bins[kPRules][kPCh][kPEnt];
  int count[kPRules][kPCh];
  int best[kPCh];      // length of the shortest whole list so far
  int chosen[kPCh][2];  // rule, entries
  int range[kPCh][3];   // mn, mx, none
  long long base;
};

__device__ __forceinline__ void tile_entries(const PtEntArgs& a, int block, TileEntriesLds& sh) {
  static_assert(kPL == 64 && kPX == 64 && kPR == 4, "a lane per row, a quad per chunk");
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tx = block % a.ntx, ty = block / a.ntx;
  const int c0 = tx * kPX, r0 = ty * kPL;
  const int ncol = min(kPX, a.n[1] - c0), nrow = min(kPL, a.n[0] - r0);
  const int none = 4 * a.B;
  if (threadIdx.x < kPCh) sh.best[threadIdx.x] = kPEnt + 1;
  // (an old value will do)
  if (threadIdx.x == 0) sh.base = (long long)*a.counter;
  // bit c of a row's mask: a run starts at column c > 0
  {
    int v[kPL / 4];
#pragma unroll
    for (int i = 0; i < kPL / 4; ++i) {
      const int r = w * (kPL / 4) + i;
      v[i] = none;
      if (r < nrow && lane < ncol) v[i] = a.binmap[(long long)(r0 + r) * a.pitch + c0 + lane];
    }
#pragma unroll
    for (int i = 0; i < kPL / 4; ++i) {
      const int r = w * (kPL / 4) + i;
      sh.code[r][lane] = (uint16_t)v[i];
      const int before = __shfl_up(v[i], 1, 64);
      const unsigned long long m = __ballot(lane > 0 && lane < ncol && v[i] != before);
      if (lane == 0) sh.starts[r] = m;
    }
  }
  __syncthreads();
  if (sh.base >= (long long)kPUnfit) return;  // no use of any (uniform)
  const unsigned long long mask = sh.starts[lane];
  const int end = lane < nrow ? ncol : 0;
  const int ch = lane >> 2, li = lane & 3;
  int c = 0, n = 0;
  int v = sh.code[lane][0];
  while (w < kPRules) {
    // the bin code the chunk takes next, from its rows' columns; -1: done
    const bool done = c >= end;
    int b;
    if (w == 0) {
      b = quad_min(done ? 0x7fffffff : v);
      if (b == 0x7fffffff) b = -1;
    } else if (w == 1) {
      b = quad_max(done ? -1 : v);
    } else {
      b = quad_min(done ? 0x7fffffff : (c << 16) | v);
      b = b == 0x7fffffff ? -1 : (b & 0xFFFF);
    }
    // a list that has come to the length of a whole one is longer: given up
    const bool go = b >= 0 && n < *(volatile int*)&sh.best[ch];
    if (!__any(go)) break;
    if (go) {  // uniform in the quad
      if (!done && v == b) {
        const unsigned long long m = c < 63 ? mask >> (c + 1) : 0ull;  // next run start
        c = m ? c + __ffsll((long long)m) : end;
        v = sh.code[lane][min(c, kPX - 1)];
      }
      const uint32_t at = (uint32_t)quad_or(c << (8 * li));
      if (li == 0 && n < kPEnt) {
        sh.cols[w][ch][n] = at;
        sh.bins[w][ch][n] = (uint16_t)(b == none ? kPNoBin : b >> 2);
      }
      ++n;
      // done when every row stands at its end
      if (quad_min(c >= end ? 1 : 0) && li == 0) atomicMin(&sh.best[ch], n);
    }
  }
  const bool whole = quad_min(c >= end ? 1 : 0) != 0;
  if (li == 0 && w < kPRules) {
    if ((n & 1) && n < kPEnt) {  // an even number: the last one adds nothing
      sh.cols[w][ch][n] = n > 0 ? sh.cols[w][ch][n - 1] : 0u;
      sh.bins[w][ch][n] = (uint16_t)kPNoBin;
    }
    sh.count[w][ch] = whole && n <= kPEnt ? n : kPEnt + 2;
  }
  __syncthreads();
  // the shortest list of each chunk, and room for them
  if (threadIdx.x < kPCh) {
    int rule = 0;
    for (int t = 1; t < kPRules; ++t)
      if (sh.count[t][threadIdx.x] < sh.count[rule][threadIdx.x]) rule = t;
    const int n_rule = sh.count[rule][threadIdx.x];
    sh.chosen[threadIdx.x][0] = rule;
    sh.chosen[threadIdx.x][1] = n_rule + (n_rule & 1);
  }
  __syncthreads();
  int before[kPCh + 1];  // uniform
  before[0] = 0;
  bool fits = true;
#pragma unroll
  for (int q = 0; q < kPCh; ++q) {
    const int m = sh.chosen[q][1];
    fits = fits && m <= kPEnt;
    before[q + 1] = before[q] + min(m, kPEnt);
  }
  if (threadIdx.x == 0) {
    sh.base = (long long)atomicAdd(a.counter, (unsigned long long)before[kPCh]);
    // (a counter past kPUnfit leaves the entries unused, whatever they hold)
    if (!fits || sh.base + before[kPCh] > a.cap) atomicAdd(a.counter, kPUnfit);
  }
  __syncthreads();
  const long long b0 = sh.base;
  const bool room = b0 + before[kPCh] <= a.cap;
  // a wave per chunk
#pragma unroll
  for (int u = 0; u < kPCh / 4; ++u) {
    const int q = 4 * u + w, rule = sh.chosen[q][0], m = min(sh.chosen[q][1], kPEnt);
    int first = 0;
#pragma unroll
    for (int v = 0; v < kPCh; ++v) first = v == q ? before[v] : first;
    int mn = 0x7fff, mx = -1, hasnone = 0;
    for (int i = lane; i < m; i += 64) {
      const int b = sh.bins[rule][q][i];
      const int slot = b == kPNoBin ? kPSlots : b % kPSlots;
      if (room) a.entries[b0 + first + i] = make_uint2(sh.cols[rule][q][i], (uint32_t)b | slot_code(slot) << 16);
      if (b == kPNoBin) {
        if (i < sh.count[rule][q]) hasnone = 1;  // (not the entry that makes the list even)
      } else {
        mn = min(mn, b);
        mx = max(mx, b);
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      mn = min(mn, __shfl_xor(mn, o, 64));
      mx = max(mx, __shfl_xor(mx, o, 64));
    }
    hasnone = __any(hasnone) ? 1 : 0;
    if (lane == 0) {
      a.chunks[(long long)block * kPCh + q] =
          PtChunk{room ? (uint32_t)(b0 + first) : 0u, room ? (uint32_t)m : 0u, hasnone ? -1 : mn, mx};
      sh.range[q][0] = mn;
      sh.range[q][1] = mx;
      sh.range[q][2] = hasnone;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int mn = 0x7fff, mx = -1, none = 0;
    for (int q = 0; q < kPCh; ++q) {
      mn = min(mn, sh.range[q][0]);
      mx = max(mx, sh.range[q][1]);
      none |= sh.range[q][2];
    }
    PtBlock* t = a.blocks + block;
    t->mn = (int16_t)mn;
    t->mx = (int16_t)mx;
    t->none = none;
    // the tile's passes, by whichever of its two blocks comes second: the bins
    // go round with the count, a half of the word each, so no fence is needed
    // (with fences vup_bin took 371 us at 4096^2 cells, 230 so)
    bool count = true;
    if ((ty ^ 1) * kPL < a.n[0]) {
      static_assert(VUP_MAX_BINS < (1 << 14), "14 bits a bin");
      const uint32_t mine = 1u << 30 | (uint32_t)(mx + 1) << 14 | (uint32_t)min(mn, 0x3fff);
      const unsigned long long was =
          atomicAdd(&a.blocks[tx + (ty & ~1) * a.ntx].both, (unsigned long long)mine << (32 * (ty & 1)));
      const uint32_t other = (uint32_t)(was >> (32 * (~ty & 1)));
      count = other != 0u;
      mn = min(mn, (int)(other & 0x3fffu));
      mx = max(mx, (int)(other >> 14 & 0xffffu) - 1);
    }
    const int extra = tile_passes(mn, mx) - 1;
    if (count && extra > 0) atomicAdd(a.extra, (unsigned long long)extra);
  }
}

}  // namespace
}  // namespace vup

#endif
