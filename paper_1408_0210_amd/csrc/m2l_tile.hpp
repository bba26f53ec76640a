// m2l_tile.hpp -- what the M2L kernels share: a tile's columns and terms, the loads that go
// straight to LDS, and the sum of split tiles.
#pragma once
#include <climits>
#include <type_traits>

#include <vector>

#include "devutil.hpp"
#include "plan.hpp"

namespace eifmm {
namespace {

// Global memory straight into LDS, 16 bytes per lane (lane l's to lds + 16 l; lds is
// wave-uniform; an instruction's offset moves both addresses).  The loads are
// outstanding on the vector-memory counter: the caller waits for it before the
// barrier that hands the data over.
// fragment OFF / 1024 of consecutive ones in both memories; src is wave-uniform, lane l
// reads src + OFF + 16 l
template <int OFF>
__device__ inline void fragment_to_lds(uint64_t src, uint32_t lds, uint32_t lane16) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
               :
               : "s"(lds), "v"(lane16), "s"(src), "i"(OFF)
               : "memory", "m0");
}
// one fragment, each lane from its own address src + OFF (the offset is taken off the
// LDS address again)
template <int OFF>
__device__ inline void column_to_lds(const int8_t *src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off offset:%2"
               :
               : "s"(lds - OFF), "v"(src), "i"(OFF)
               : "memory", "m0");
}
__device__ inline uint64_t uniform64(uint64_t p) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// f(integral_constant<int, I>) for I in [I0, I1)
template <int I0, int I1, typename F>
__device__ inline void for_each_from(F &f) {
  if constexpr (I0 < I1) {
    f(std::integral_constant<int, I0>{});
    for_each_from<I0 + 1, I1>(f);
  }
}

__device__ int g_no_slot = -1;  // the slot of a missing source

// a tile's target column
struct TileCol {
  const int *slot_map;  // slot map of the level
  const void *B;        // source columns
  const ColScale *bs;   // their scales (FP64)
  uint32_t tkey;        // target key
  int r, valid;
};

// column jc of job J; bb: the target box's coordinates as its own bounds
__device__ inline TileCol tile_column(const GemmJob &J, int jc, int (&bb)[6]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    bb[a] = INT_MAX;
    bb[3 + a] = INT_MIN;
  }
  TileCol c{};
  c.valid = jc < J.ntgt * J.nrhs;
  c.slot_map = J.src_slot;
  c.B = J.Bsrc;
  c.bs = J.bscale;
  if (c.valid) {
    const int tt = jc / J.nrhs;
    c.r = jc - tt * J.nrhs;
    if (J.colref) {
      const ColRef cr = J.colref[tt];
      const ColSrc &cs = J.colsrc[cr.rec];
      c.tkey = ldg(cs.keys + cr.slot);
      c.slot_map = cs.slot;
      c.B = cs.B;
      c.bs = cs.bscale;
    } else {
      c.tkey = ldg(J.tgt_keys + ldg(J.tgt + tt));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) bb[a] = bb[3 + a] = (int)morton_axis(c.tkey, a);
  }
  return c;
}

// result column of job J's column jo
__device__ inline double *tile_output(const GemmJob &J, int jo) {
  const int tt = jo / J.nrhs, ro = jo - tt * J.nrhs;
  int tso;
  double *Cout = J.C;
  if (J.colref) {
    const ColRef cr = J.colref[tt];
    tso = cr.slot;
    Cout = J.colsrc[cr.rec].C;
  } else {
    tso = ldg(J.tgt + tt);
  }
  return Cout + ((int64_t)tso * J.nrhs + ro) * J.dpm;
}

// One wave: the terms in [term0, term1) that reach inside the domain from some box of
// [lo, hi], in order into sdel (LDS), packed (dx+3) | (dy+3) << 3 | (dz+3) << 6 | id << 9;
// returns their number.  Offset delta reaches inside when hi + delta >= 0 and
// lo + delta < side on every axis.
__device__ inline int list_terms(const GemmJob &J, int term0, int term1, const int (&lo)[3],
                                 const int (&hi)[3], const int8_t *__restrict__ dvec, int *sdel) {
  const int lane = threadIdx.x & 63;
  const int side = 1 << J.level;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int nk = 0;
  for (int b = term0; b < term1; b += 64) {
    const int i = b + lane;
    bool keep = false;
    int pk = 0;
    if (i < term1) {
      const int id = ldg(J.terms + i);
      const int d0 = dvec[3 * id], d1 = dvec[3 * id + 1], d2 = dvec[3 * id + 2];
      pk = (d0 + 3) | ((d1 + 3) << 3) | ((d2 + 3) << 6) | (id << 9);
      keep = hi[0] + d0 >= 0 && lo[0] + d0 < side && hi[1] + d1 >= 0 && lo[1] + d1 < side &&
             hi[2] + d2 >= 0 && lo[2] + d2 < side;
    }
    const uint64_t m = __ballot(keep);
    if (keep) sdel[nk + (int)__popcll(m & below)] = pk;
    nk += (int)__popcll(m);
  }
  return nk;
}

// The terms in [term0, term1) of an 8-wave tile whose source box lies inside the domain
// for some of its columns (list_terms).  bb: the box of this lane's column (16 columns
// per wave, equal in lanes 16 apart).  Two workgroup barriers.
__device__ inline int tile_terms(const GemmJob &J, int term0, int term1, int (&bb)[6],
                                 const int8_t *__restrict__ dvec, int *sdel) {
  __shared__ int sbox[8][6];
  __shared__ int snk;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      bb[a] = min(bb[a], __shfl_xor(bb[a], o));
      bb[3 + a] = max(bb[3 + a], __shfl_xor(bb[3 + a], o));
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int a = 0; a < 6; ++a) sbox[w][a] = bb[a];
  }
  lds_barrier();
  if (w == 0) {
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = INT_MAX;
      hi[a] = INT_MIN;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        lo[a] = min(lo[a], sbox[q][a]);
        hi[a] = max(hi[a], sbox[q][3 + a]);
      }
    }
    const int nk = list_terms(J, term0, term1, lo, hi, dvec, sdel);
    if (lane == 0) snk = nk;
  }
  lds_barrier();
  return __builtin_amdgcn_readfirstlane(snk);
}

// where the slot of the source of term q is read (-1: no box)
__device__ inline const int *source_slot(const GemmJob &J, const TileCol &c, int q, int nt,
                                         const int *sdel) {
  if (q >= nt || !c.valid || !c.slot_map) return &g_no_slot;
  const int pk = sdel[q];
  const int side = 1 << J.level;
  const int m0 = (int)morton_axis(c.tkey, 0) + (pk & 7) - 3;
  const int m1 = (int)morton_axis(c.tkey, 1) + ((pk >> 3) & 7) - 3;
  const int m2 = (int)morton_axis(c.tkey, 2) + ((pk >> 6) & 7) - 3;
  const bool in = m0 >= 0 && m1 >= 0 && m2 >= 0 && m0 < side && m1 < side && m2 < side;
  return in ? c.slot_map + morton_encode((uint32_t)m0, (uint32_t)m1, (uint32_t)m2) : &g_no_slot;
}

__device__ inline int job_of_tile(const GemmJob *__restrict__ jobs, int njobs, int tile) {
  return find_last_le(njobs, tile, [&](int m) { return (int64_t)jobs[m].tiles_start; });
}

// adds the pieces of the split tiles in part order (kSumSplit blocks per tile) and
// sets the counter back for the next launch
constexpr int kSumSplit = 4;
__global__ __launch_bounds__(256) void k_m2l_sum(const GemmJob *__restrict__ jobs, int njobs,
                                                  int ntiles, int full, int parts, int height,
                                                  int cols,
                                                  const double *__restrict__ ws,
                                                  int *__restrict__ ctr) {
  if (blockIdx.x == 0 && threadIdx.x == 0) stg(ctr, 0);
  const int tile = full + (int)(blockIdx.x / kSumSplit);
  if (tile >= ntiles) return;
  const GemmJob J = jobs[job_of_tile(jobs, njobs, tile)];
  const int rows = 16 * height, size = rows * cols;
  const int tile_local = tile - J.tiles_start;
  const int row0 = (tile_local % J.nrowtiles) * rows, col0 = (tile_local / J.nrowtiles) * cols;
  const int nrows = min(rows, J.dpm - row0), ncols = J.ntgt * J.nrhs;
  const double *p = ws + (size_t)(tile - full) * parts * size;
  for (int e = (int)(blockIdx.x % kSumSplit) * 256 + (int)threadIdx.x; e < size;
       e += 256 * kSumSplit) {
    const int jt = e / rows, rt = e - jt * rows, jo = col0 + jt;
    if (rt >= nrows || jo >= ncols) continue;
    double v = 0.0;
    int i = 0;
    for (; i + 8 <= parts; i += 8) {
      double u[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = ldg(p + (size_t)(i + q) * size + e);
#pragma unroll
      for (int q = 0; q < 8; ++q) v += u[q];
    }
    for (; i < parts; ++i) v += ldg(p + (size_t)i * size + e);
    stg(tile_output(J, jo) + row0 + rt, v);
  }
}

// How a launch of `tiles` tiles (tile doubles each) on `cus` workgroups is split: whole
// tiles, then `rest` tiles in `parts` pieces each, about 4 items per workgroup and at
// least 4 terms an item, as many as the workspace holds
struct TileSplit {
  int grid, full, rest, parts;
};
inline TileSplit split_tiles(int tiles, int cus, size_t tile, size_t ws_len) {
  TileSplit T{cus, (tiles / cus) * cus, 0, 0};
  T.rest = tiles - T.full;
  if (T.rest > 0) {
    const size_t pieces = (ws_len - kCounterDoubles) / tile;
    T.parts = 4 * cus / T.rest;
    T.parts = T.parts < 4 ? 4 : T.parts > 47 ? 47 : T.parts;
    if ((size_t)T.parts * T.rest > pieces) T.parts = (int)(pieces / T.rest);
    if (T.parts < 2) {  // the pieces do not fit: every tile whole
      T.full = tiles;
      T.rest = 0;
    }
  }
  if (T.full == 0 && T.rest * T.parts < cus) T.grid = T.rest * T.parts;
  return T;
}

}  // namespace
}  // namespace eifmm
