// m2l32.hip -- the mixed-precision M2L (Algorithm 3 step 4): FP32 products on the FP32
// matrix cores, each offset's product added to an FP64 sum over the offsets.
//
// A workgroup of 8 waves computes all 16 RB rows of a row tile (up to 9 blocks, so one
// row tile for most compressed operators: a source column is read once per offset
// instead of once per 3- or 4-block tile) of 128 columns; each wave holds every row of
// its 16 columns.  The operators pass through LDS in chunks of 16 S values of k, loaded
// straight to LDS one chunk ahead in two buffers, the source columns go to registers a
// chunk ahead, the slots of the sources a term ahead; the loads are issued between the
// products.  The order of the products of an offset, k by k in the table's order, is the
// one the accumulation of a single chain has, whatever the chunks.
//
// Bound by the FP32 matrix cores (32 cycles a product; a bare probe reaches 155 TFLOP/s),
// then by the wait at a chunk's barrier.  2^20 points, 64 right-hand sides, rank 144 (9 row
// blocks, one tile, chunks of 3): 189.9 ms as 3-block tiles of 4 waves with the operators
// passed through registers to LDS, 141.7 ms now (114 TFLOP/s).  10^6 points, one right-hand
// side, rank 128, the near field beside it: the pass 3.93 -> 3.63 ms.
#include <algorithm>
#include <vector>

#include "m2l_tile.hpp"

namespace eifmm {

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int kCols = 128;    // columns of a tile: 8 waves x 16
constexpr int kFrag = 1024;   // bytes of a 16 x 16 operand fragment (64 lanes x 4 k)
__device__ float g_zero_col[1024];  // read in place of a missing source column

template <int RB, int S>
__device__ inline void m2l32_tile(const GemmJob &J, int tile_local, int term0, int term1,
                                  double *__restrict__ part, const int8_t *__restrict__ dvec,
                                  char (*As)[RB * S * kFrag], TileCol *cst, int *sdel) {
  typedef double D4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rowtile = tile_local % J.nrowtiles, coltile = tile_local / J.nrowtiles;
  const int rb0 = rowtile * RB, col0 = coltile * kCols;
  const int nrb = J.dpm >> 4, nsub = J.dpk >> 4, nkc = (nsub + S - 1) / S;
  const int nv = min(RB, nrb - rb0);  // row blocks of this tile
  const int ncols = J.ntgt * J.nrhs;
  TileCol *my = cst + 16 * w + (lane & 15);
  int bb[6];
  *my = tile_column(J, col0 + 16 * w + (lane & 15), bb);
  const int nt = tile_terms(J, term0, term1, bb, dvec, sdel);

  D4 sum[RB];
  f4v acc[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) sum[i] = D4{0, 0, 0, 0};
  if (nt > 0) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&As[0][0];
    const uint32_t lane16 = 16u * (uint32_t)lane;
    // operator blocks: [row block][16-k sub-chunk][64 lanes][4 k]
    const char *Abase = (const char *)J.A + (int64_t)rb0 * nsub * kFrag;
    int slotn = ldg(source_slot(J, *my, 0, nt, sdel));
    const float *srcp = nullptr;
    const char *At = nullptr;
    bool haven = false, haveq = false;  // the wave has a source: term aimed at, term loaded
    int fq = 0, fk = 0;                 // next chunk to load: term, chunk
    // the addresses of the next chunk, if it starts a term (a step ahead of its loads)
    auto aim = [&]() {
      if (fq >= nt || fk != 0) return;
      const TileCol c = *my;
      const int sl = slotn;
      srcp = (sl < 0 ? g_zero_col : (const float *)c.B + ((int64_t)sl * J.nrhs + c.r) * J.dpk) +
             4 * (lane >> 4);
      haven = __ballot(sl >= 0) != 0;
      At = Abase + (int64_t)(__builtin_amdgcn_readfirstlane(sdel[fq]) >> 9) * J.a_stride;
      slotn = ldg(source_slot(J, c, fq + 1, nt, sdel));
    };
    // the loads of the next chunk: a row block's S fragments per wave and turn
    constexpr int NP = (RB + 7) / 8;
    bool live = false;
    int fs = 0;  // sub-chunks of the chunk being loaded
    const float *sp = nullptr;
    uint64_t ap[NP];
    uint32_t lp[NP];
    auto fetch_begin = [&](int buf) {
      live = fq < nt;
      if (!live) return;
      if (fk == 0) haveq = haven;
      fs = min(S, nsub - fk * S);
      sp = srcp + fk * (16 * S);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int blk = w + 8 * i;
        ap[i] = uniform64((uint64_t)(At + (int64_t)(blk * nsub + fk * S) * kFrag));
        lp[i] = __builtin_amdgcn_readfirstlane(lds0 +
                                               (uint32_t)(buf * (RB * S * kFrag) + blk * (S * kFrag)));
      }
      if (++fk == nkc) {
        fk = 0;
        ++fq;
      }
    };
    constexpr int NL = NP * S;
    auto fetch_one = [&](auto N) {
      constexpr int n = decltype(N)::value, i = n / S, j = n % S;
      if constexpr (n < NL)
        if (live && w + 8 * i < nv && j < fs) fragment_to_lds<j * kFrag>(ap[i], lp[i], lane16);
    };
    auto columns = [&](f4v(&Bn)[S]) {
      if (!live) return;
#pragma unroll
      for (int j = 0; j < S; ++j)
        if (j < fs) Bn[j] = ldg((const f4v *)(sp + 16 * j));
    };
    auto fetch_all = [&](auto N0) { for_each_from<decltype(N0)::value, NL>(fetch_one); };
    bool have = false;
    int kc = 0, ns = 0, nsn = 0;  // chunk of the current term, its sub-chunks, the next one's
    // the products of one chunk (first: the sums start at zero), its row blocks side by
    // side, the operator fragments read AHEAD ahead
    auto products = [&](auto first, int buf, const f4v(&b)[S]) {
      constexpr int AHEAD = RB < 3 ? RB : 3;
      const char *Ap = &As[buf][16 * lane];
      auto sub = [&](auto Jc) {
        constexpr int j = decltype(Jc)::value;
        if (j >= ns) return;
        f4v a[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) a[i] = *(const f4v *)(Ap + (i * S + j) * kFrag);
        __builtin_amdgcn_sched_barrier(0);
        auto block = [&](auto Ic) {
          constexpr int i = decltype(Ic)::value;
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const f4v c = decltype(first)::value && j == 0 && ks == 0 ? f4v{0, 0, 0, 0} : acc[i];
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i % AHEAD][ks], b[j][ks], c, 0, 0, 0);
          }
          if (i + AHEAD < RB) a[i % AHEAD] = *(const f4v *)(Ap + ((i + AHEAD) * S + j) * kFrag);
          fetch_one(std::integral_constant<int, (i % 2 == 0) ? j * ((RB + 1) / 2) + i / 2 : NL>{});
          __builtin_amdgcn_sched_barrier(0);
        };
        for_each_from<0, RB>(block);
      };
      for_each_from<0, S>(sub);
      // (loads that found no place between the products of a short last chunk)
      if (ns < S) {
        auto late = [&](auto N) {
          constexpr int n = decltype(N)::value;
          if (n >= ns * ((RB + 1) / 2)) fetch_one(N);
        };
        for_each_from<0, NL>(late);
      }
    };
    static_assert(NL <= S * ((RB + 1) / 2), "a load per two row blocks");
    auto step = [&](int buf, const f4v(&Bc)[S], f4v(&Bn)[S]) {
      // what this wave issued in the last step has arrived, after the barrier the
      // others' too (and nobody reads the buffer that the next loads overwrite)
      __builtin_amdgcn_s_waitcnt(0x0f70);
      lds_barrier();
      ns = nsn;
      const bool fst = kc == 0;
      if (fst) have = haveq;
      fetch_begin(buf ^ 1);
      nsn = fs;
      columns(Bn);
      if (!have)
        fetch_all(std::integral_constant<int, 0>{});
      else if (fst)
        products(std::true_type{}, buf, Bc);
      else
        products(std::false_type{}, buf, Bc);
      aim();
      if (++kc == nkc) {
        kc = 0;
        if (have) {  // a term is complete
#pragma unroll
          for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[i][q] += (double)acc[i][q];
        }
      }
    };
    f4v B0[S], B1[S];
    aim();
    fetch_begin(0);
    nsn = fs;
    columns(B0);
    fetch_all(std::integral_constant<int, 0>{});
    aim();
    const int steps = nt * nkc;
    for (int it = 0; it < steps; it += 2) {
      step(0, B0, B1);
      if (it + 1 < steps) step(1, B1, B0);
    }
  }
  // result row 16 block + 4 (lane / 16) + q of column lane % 16
  const int jt = 16 * w + (lane & 15), jo = col0 + jt;
  if (jo >= ncols) return;
  double *out = part ? part + (size_t)jt * (16 * RB) : tile_output(J, jo) + 16 * rb0;
#pragma unroll
  for (int i = 0; i < RB; ++i)
    if (i < nv) {
      double *o = out + 16 * i + 4 * (lane >> 4);
      d2v v;
      v.x = sum[i][0];
      v.y = sum[i][1];
      stg((d2v *)o, v);
      v.x = sum[i][2];
      v.y = sum[i][3];
      stg((d2v *)(o + 2), v);
    }
}

// tiles whole or in parts as in m2l.hip
template <int RB, int S>
__global__ __launch_bounds__(512, 2) void k_m2l32(const GemmJob *__restrict__ jobs, int njobs, int G,
                                                  int full, int items, int parts,
                                                  double *__restrict__ ws,
                                                  const int8_t *__restrict__ dvec,
                                                  int *__restrict__ ctr) {
  constexpr int TILE = RB * 16 * kCols;
  __shared__ __align__(16) char As[2][RB * S * kFrag];
  __shared__ TileCol cst[kCols];
  __shared__ int sdel[189];
  __shared__ int item_sh;
  const int g = blockIdx.x;
  const int gx = (G % 8 == 0) ? (g % 8) * (G / 8) + g / 8 : g;
  for (int tile = gx; tile < full; tile += G) {
    const GemmJob J = jobs[job_of_tile(jobs, njobs, tile)];
    m2l32_tile<RB, S>(J, tile - J.tiles_start, 0, J.nterms, nullptr, dvec, As, cst, sdel);
  }
  if (items <= 0) return;
  for (;;) {
    if (threadIdx.x == 0) item_sh = atomicAdd(ctr, 1);
    __syncthreads();
    const int item = item_sh;
    __syncthreads();
    if ((unsigned)item >= (unsigned)items) return;
    const int tile = full + item / parts, q = item % parts;
    const GemmJob J = jobs[job_of_tile(jobs, njobs, tile)];
    m2l32_tile<RB, S>(J, tile - J.tiles_start, q * J.nterms / parts, (q + 1) * J.nterms / parts,
                      ws + (size_t)item * TILE, dvec, As, cst, sdel);
  }
}

template <int RB, int S>
void launch(const GemmJob *jobs, int n, int tiles, int cus, double *ws, size_t ws_len,
            const int8_t *dvec, hipStream_t s) {
  const TileSplit T = split_tiles(tiles, cus, (size_t)RB * 16 * kCols, ws_len);
  int *ctr = (int *)(ws + ws_len - kCounterDoubles);
  hipLaunchKernelGGL((k_m2l32<RB, S>), dim3(T.grid), dim3(512), 0, s, jobs, n, T.grid, T.full,
                     T.rest * T.parts, T.parts, ws, dvec, ctr);
  if (T.rest > 0)
    hipLaunchKernelGGL(k_m2l_sum, dim3(T.rest * kSumSplit), dim3(256), 0, s, jobs, n, tiles, T.full,
                       T.parts, RB, kCols, ws, ctr);
}

template <int RB>
void launch_s(const GemmJob *jobs, int n, int tiles, int sub, int cus, double *ws, size_t ws_len,
              const int8_t *dvec, hipStream_t s) {
  if (sub == 3)
    launch<RB, 3>(jobs, n, tiles, cus, ws, ws_len, dvec, s);
  else
    launch<RB, 4>(jobs, n, tiles, cus, ws, ws_len, dvec, s);
}

}  // namespace

// Row blocks of a tile for nrb blocks: the fewest idle blocks, the taller on a tie.
int pick_m2l32(int nrb) {
  int best = 9, waste = 1 << 30;
  for (int h : {9, 8, 6, 5, 4, 3, 2}) {
    const int w = (nrb + h - 1) / h * h - nrb;
    if (w < waste) {
      waste = w;
      best = h;
    }
  }
  return best;
}

// dk: columns of the (finest level's) operators, which decides whether a chunk has 3 or
// 4 sub-chunks of 16 (the one that leaves less of the last chunk empty)
void launch_m2l32(const GemmJob *jobs, int n, int tiles, int height, int dk, int cus, double *ws,
                  size_t ws_len, const int8_t *dvec, hipStream_t s) {
  if (n == 0 || tiles == 0) return;
  const int nsub = dk / 16;
  const int sub = (nsub + 2) / 3 * 3 < (nsub + 3) / 4 * 4 ? 3 : 4;
  switch (height) {
    case 9: launch_s<9>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    case 8: launch_s<8>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    case 6: launch_s<6>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    case 5: launch_s<5>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    case 4: launch_s<4>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    case 3: launch_s<3>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
    default: launch_s<2>(jobs, n, tiles, sub, cus, ws, ws_len, dvec, s); break;
  }
}

}  // namespace eifmm
