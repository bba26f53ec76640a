// m2l_small.hip -- the FP64 M2L of levels whose operators are at most 32 x 32, on the
// FP64 matrix cores.
//
// Operators this small (316 of them, 10 KB at d = 20) stay in every XCD's L2 and a term is
// a handful of products, so that the digit kernel spends its time on barriers, on 64-k
// chunks of which 20 are used and on adding the digits' sums.  Here a workgroup computes
// 32 columns and all rows; its 4 waves take every fourth term and never meet until the
// end, where their sums are added in wave order.  Operators and columns go from memory to
// registers a term ahead, the slots of the sources two terms ahead; k is walked in 4s up to
// d, not up to its padding.  The products of a column accumulate in FP64 over a wave's
// terms.
// Bound by the FP64 matrix cores (64 cycles a product) and the cache lookups of the columns
// beside them.  2^20 uniform points, d = 24 and 20 on levels 4 and 5: 594 us as digits
// (562 us as 3-block FP64 tiles of 4 waves); this way 287, tiles dealt to the XCDs by place
// 270, a column's loads side by side 213 us, 102 us of them products.  Larger operators
// stay with the digits: there the FP64 matrix rate, 75 TFLOP/s, is the lower bound.
// A batch packs the columns of its problems into the same tiles: 16 problems of 2e4 to 1.1e5
// points, depth 4, e^-r^2: the whole pass 2.01 ms as digits, 1.44 this way.
#include "m2l_tile.hpp"

namespace eifmm {

namespace {

constexpr int kCols = 32;       // columns of a tile
__device__ double g_zero_col[32];  // read in place of a missing source column

// k-steps of 4 that a kernel exists for, at least s
__host__ __device__ constexpr int round_steps(int s) { return s <= 2 ? 2 : s == 7 ? 8 : s == 3 ? 4 : s; }

// k of lane group g (lane / 16) in step s of KS: steps come in pairs whose two k are
// neighbours in memory (one 16-byte load), an odd last step by itself
__host__ __device__ constexpr int step_k(int ks, int s, int g) {
  return s < ks / 2 * 2 ? 8 * (s / 2) + 2 * g + (s & 1) : 8 * (ks / 2) + g;
}

// A term in LDS: its offset as dilated integers modulo 2^10 (the axes' bits interleaved as
// in a key) and its operator
struct Term {
  uint32_t delta;
  int id;
};
// key + delta, axis by axis modulo 2^10: ones in the other axes' bits carry across them.
// A box outside the domain has a bit set at or above 3 level.
__device__ inline uint32_t moved(uint32_t key, uint32_t delta) {
  uint32_t r = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const uint32_t m = 0x09249249u << a;
    r |= ((key | ~m) + (delta & m)) & m;
  }
  return r;
}

// A column's loads are spread over 4 neighbouring lanes (column lane / 4, part lane % 4:
// 64 bytes of one column side by side; with the product's own layout, 16 lanes side by side
// read 16 columns and the cache is looked up once per lane); the lanes' values then change
// places to column lane % 16, group lane / 16.
__device__ inline double to_operand(double v, int from) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_ds_bpermute(from, (int)u);
  const int hi = __builtin_amdgcn_ds_bpermute(from, (int)(u >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// PACKED: the columns belong to several problems (ColRef), each with a slot map and sources
// of its own
template <int NB, int KS, bool PACKED>
__device__ inline void small_tile(const GemmJob &J, int tile_local, const int8_t *__restrict__ dvec,
                                  double *red, Term *terms, int *sdel, int *snk) {
  constexpr int NP = KS / 2, ODD = KS & 1;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col0 = tile_local * kCols;
  uint32_t key[2];
  int rr[2];
  bool valid[2];
  const int *map[2];
  const double *src[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    int bb[6];
    const TileCol tc = tile_column(J, col0 + 16 * c + (lane >> 2), bb);
    key[c] = tc.tkey;
    rr[c] = tc.r;
    valid[c] = tc.valid;
    map[c] = PACKED ? tc.slot_map : J.src_slot;
    src[c] = (const double *)(PACKED ? tc.B : J.Bsrc);
  }
  // the terms that reach inside the domain for some column
  if (w == 0) {
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int m0 = (int)morton_axis(key[0], a), m1 = (int)morton_axis(key[1], a);
      lo[a] = min(valid[0] ? m0 : INT_MAX, valid[1] ? m1 : INT_MAX);
      hi[a] = max(valid[0] ? m0 : INT_MIN, valid[1] ? m1 : INT_MIN);
#pragma unroll
      for (int o = 4; o < 64; o <<= 1) {
        lo[a] = min(lo[a], __shfl_xor(lo[a], o));
        hi[a] = max(hi[a], __shfl_xor(hi[a], o));
      }
    }
    const int nk = list_terms(J, 0, J.nterms, lo, hi, dvec, sdel);
    for (int q = lane; q < nk; q += 64) {
      const int pk = sdel[q];
      terms[q].delta = morton_encode((uint32_t)((pk & 7) - 3) & 1023u,
                                     (uint32_t)(((pk >> 3) & 7) - 3) & 1023u,
                                     (uint32_t)(((pk >> 6) & 7) - 3) & 1023u);
      terms[q].id = pk >> 9;
    }
    if (lane == 0) *snk = nk;
  }
  __syncthreads();
  const int nt = __builtin_amdgcn_readfirstlane(*snk);

  d4v acc[NB][2];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[i][c] = d4v{0, 0, 0, 0};
  struct Set {  // operands of a term: pairs of k-steps, the odd one
    d2v a[NB][NP], b[2][NP];
    double a1[NB], b1[2];
  };
  int slot[2];
  const int bits = 3 * J.level;
  auto lookup = [&](int q) {
    const uint32_t d = __builtin_amdgcn_readfirstlane((int)terms[min(q, nt - 1)].delta);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const uint32_t m = moved(key[c], d);
      slot[c] = ldg(valid[c] && (m >> bits) == 0 && q < nt ? map[c] + m : &g_no_slot);
    }
  };
  const int g = lane & 3, from = 4 * (4 * (lane & 15) + (lane >> 4));
  auto load = [&](Set &S, int q) {
    const int o = __builtin_amdgcn_readfirstlane(terms[min(q, nt - 1)].id);
    const double *A = (const double *)J.A + (int64_t)o * (NB * KS * 64);
    const double *B[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      B[c] = slot[c] < 0 ? g_zero_col
                         : src[c] + ((int64_t)slot[c] * J.nrhs + rr[c]) * J.dpk;
    lookup(q + 4);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int p = 0; p < NP; ++p) S.b[c][p] = ldg((const d2v *)(B[c] + 8 * p + 2 * g));
      if (ODD) S.b1[c] = ldg(B[c] + 8 * NP + g);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const double *Ai = A + i * (KS * 64);
#pragma unroll
      for (int p = 0; p < NP; ++p) S.a[i][p] = ldg((const d2v *)(Ai + 128 * p + 2 * lane));
      if (ODD) S.a1[i] = ldg(Ai + 128 * NP + lane);
    }
  };
  auto products = [&](const Set &S) {
    d2v b[2][NP];
    double b1[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        b[c][p] = d2v{to_operand(S.b[c][p].x, from), to_operand(S.b[c][p].y, from)};
      if (ODD) b1[c] = to_operand(S.b1[c], from);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(S.a[i][p][e], b[c][p][e], acc[i][c],
                                                             0, 0, 0);
    if (ODD)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(S.a1[i], b1[c], acc[i][c], 0, 0, 0);
  };
  if (w < nt) {
    Set S0, S1;
    lookup(w);
    load(S0, w);
    for (int q = w; q < nt; q += 8) {
      load(S1, q + 4);  // (past the last term: missing sources)
      products(S0);
      if (q + 4 >= nt) break;
      load(S0, q + 8);
      products(S1);
    }
  }
  // the waves' sums, added in wave order: wave w those of (row block, column block) w
  double *mine = red + w * (NB * 512) + 4 * lane;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      *(d2v *)(mine + (2 * i + c) * 256) = d2v{acc[i][c][0], acc[i][c][1]};
      *(d2v *)(mine + (2 * i + c) * 256 + 2) = d2v{acc[i][c][2], acc[i][c][3]};
    }
  __syncthreads();
  if (w >= 2 * NB) return;
  const int i = w >> 1, jo = col0 + 16 * (w & 1) + (lane & 15);
  if (jo >= J.ntgt * J.nrhs) return;
  double v[4] = {0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const double *p = red + u * (NB * 512) + w * 256 + 4 * lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] += p[q];
  }
  // rows (lane / 16) + 4 q of the block
  double *out = tile_output(J, jo) + 16 * i + (lane >> 4);
#pragma unroll
  for (int q = 0; q < 4; ++q) stg(out + 4 * q, v[q]);
}

struct SmallShared {
  __align__(16) double red[4 * 2 * 512];
  Term terms[189];
  int sdel[189];
  int snk;
};

template <bool PACKED>
__device__ inline void small_tile_of(const GemmJob &J, int tl, const int8_t *__restrict__ dvec,
                                     SmallShared &S) {
  auto run = [&](auto nb, auto ks) {
    small_tile<decltype(nb)::value, decltype(ks)::value, PACKED>(J, tl, dvec, S.red, S.terms, S.sdel,
                                                                 &S.snk);
  };
  auto steps = [&](auto nb) {
    switch (J.ksteps) {
      case 8: run(nb, std::integral_constant<int, 8>{}); break;
      case 6: run(nb, std::integral_constant<int, 6>{}); break;
      case 5: run(nb, std::integral_constant<int, 5>{}); break;
      case 4: run(nb, std::integral_constant<int, 4>{}); break;
      default: run(nb, std::integral_constant<int, 2>{}); break;
    }
  };
  if (J.dpm > 16)
    steps(std::integral_constant<int, 2>{});
  else
    steps(std::integral_constant<int, 1>{});
}

// One workgroup per tile.  XCD x (workgroup mod 8) takes the x-th eighth of every job's
// tiles: the same part of the domain from all child classes, whose source columns then
// stay in its L2 (contiguous tiles over all jobs would give an XCD one class and with it
// every source of the level).
__global__ __launch_bounds__(256, 3) void k_m2l_small(const GemmJob *__restrict__ jobs, int njobs,
                                                      const int8_t *__restrict__ dvec) {
  __shared__ SmallShared S;
  const int x = blockIdx.x % 8, i = blockIdx.x / 8, lane = threadIdx.x & 63;
  const int n = lane < njobs ? ldg(&jobs[lane].ncoltiles) : 0;
  const int first = x * n / 8, count = (x + 1) * n / 8 - first;
  int end = count;  // this XCD's tiles in the jobs up to this lane's
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(end, o);
    if (lane >= o) end += v;
  }
  const unsigned long long after = __ballot(end > i);
  if (after == 0) return;
  const int j = __builtin_ctzll(after);
  const GemmJob J = jobs[j];
  const int tl = __builtin_amdgcn_readfirstlane(__shfl(first + i - (end - count), j));
  small_tile_of<false>(J, tl, dvec, S);
}

// A batch: any number of jobs, an eighth of all tiles per XCD
__global__ __launch_bounds__(256, 3) void k_m2l_small_packed(const GemmJob *__restrict__ jobs,
                                                             int njobs, int tiles,
                                                             const int8_t *__restrict__ dvec) {
  __shared__ SmallShared S;
  const int x = blockIdx.x % 8, tile = x * ((tiles + 7) / 8) + blockIdx.x / 8;
  if (tile >= tiles) return;
  const GemmJob J = jobs[job_of_tile(jobs, njobs, tile)];
  small_tile_of<true>(J, tile - J.tiles_start, dvec, S);
}

}  // namespace

int m2l_small_steps(int d) { return round_steps((d + 3) / 4); }

// frag: the operators in the gathered GEMM's order ([offset][row block][cols / 4][64]);
// returns [offset][row block] of ks k-steps as the kernel reads them
std::vector<double> m2l_small_operators(const std::vector<double> &frag, int rows, int cols, int ks) {
  const int nrb = rows / 16, nks = cols / 4;
  std::vector<double> out((size_t)kNumOffsets * nrb * ks * 64);
  for (int ob = 0; ob < kNumOffsets * nrb; ++ob)
    for (int s = 0; s < ks; ++s)
      for (int l = 0; l < 64; ++l) {
        const int k = step_k(ks, s, l >> 4);
        const double v =
            frag[((size_t)ob * nks + 4 * (k >> 4) + (k & 3)) * 64 + 16 * ((k >> 2) & 3) + (l & 15)];
        const size_t base = (size_t)ob * ks * 64;
        out[s < ks / 2 * 2 ? base + (s / 2) * 128 + 2 * l + (s & 1) : base + ks / 2 * 128 + l] = v;
      }
  return out;
}

// grid: 8 times the sum of the jobs' tiles over 8, rounded up
void launch_m2l_small(const GemmJob *jobs, int n, int grid, const int8_t *dvec, hipStream_t s) {
  static_assert(8 * (EIFMM_MAX_DEPTH - 1) <= 64, "a lane per job");
  if (n == 0 || grid == 0) return;
  hipLaunchKernelGGL(k_m2l_small, dim3(grid), dim3(256), 0, s, jobs, n, dvec);
}

void launch_m2l_small_packed(const GemmJob *jobs, int n, int tiles, const int8_t *dvec,
                             hipStream_t s) {
  if (n == 0 || tiles == 0) return;
  hipLaunchKernelGGL(k_m2l_small_packed, dim3((tiles + 7) / 8 * 8), dim3(256), 0, s, jobs, n, tiles,
                     dvec);
}

}  // namespace eifmm
