// pass.hip -- the EIFMM evaluation pass (Algorithm 3 plus the near field).
//
// Expansions of level k live in slot-major arrays [slot][rhs][dp_k] (slot =
// rank of a non-empty box in key order; dp_k = d_k padded to 16 with zeros).
// Steps and kernels:
//   near field, eq. (13)        k_p2p64 / k_p2p32   one wave per 32 targets of a leaf
//   1  P2M                      k_p2m               one workgroup per leaf or segment of it
//   2  M2M (Sec. 4.1 operators) k_gemm<MODE_M2M>    MFMA, 8 children per parent
//   3  What = Delta W           k_trsm              blocked triangular solves (MFMA)
//   4  M2L (Sec. 4.2 matrices)  189 offsets per class; FP64: k_m2l8 (m2l.hip, int8 MFMA),
//                               mixed: k_m2l32 (m2l32.hip, FP32 MFMA)
//   5  L2L                      k_gemm<MODE_L2L>    MFMA, adds g
//   6  lhat = Delta^T l         k_trsm
//   7  L2P and f = f_far + f_near, input order  k_l2p  one wave per 32 targets
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cstring>
#include <type_traits>
#include <vector>

#include "devutil.hpp"
#include "m2l_tile.hpp"
#include "plan.hpp"

namespace eifmm {

// ------------------------------------------------------------------ kernels k
// 1/sqrt(r2) for r2 > 0: the hardware reciprocal square root y, refined with
// t = 1 - r2 y^2 by the series (1 - t)^(-1/2) = 1 + t/2 + 3 t^2 / 8 + ...,
// i.e. y (1 + t (1/2 + 3 t / 8)).  r2 = 0 gives NaN; the callers that can meet
// it (the near field of a singular kernel) replace the value.
__device__ inline double rsq_refined(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double t = fma(-r2 * y, y, 1.0);
  return fma(y * t, fma(t, 0.375, 0.5), y);
}

// exp(x) for x <= 0 (up to rounding): x = n ln 2 + r with |r| <= ln 2 / 2, and
// exp(r) = 1 + r + r^2 Q(r), Q the polynomial of degree 9 through the Chebyshev nodes of
// the interval (1.6e-17 relative, an eighth of a rounding); 2^n by the exponent
// instruction, which also rounds into the denormals.  Below -750 the result is 0 as
// exp(x) is.  The library routine's checks for large arguments (a compare and two
// selects each way) are not needed: e^-r/r pairs 4.77 -> 4.13 ms on 3e5 clustered points.
__device__ inline double exp_nonpos(double x) {
  x = fmax(x, -750.0);
  const double n = rint(x * 0x1.71547652b82fep+0);
  double r = fma(n, -0x1.62e42fe800000p-1, x);  // exact: 32 + 11 bits of product
  r = fma(n, -0x1.e8e7bcd5e4f1ep-31, r);
  double q = 0x1.af38a9b0ec855p-26;
  q = fma(q, r, 0x1.289185613a3d6p-22);
  q = fma(q, r, 0x1.71de0dae63bb3p-19);
  q = fma(q, r, 0x1.a019b90d2ae7ap-16);
  q = fma(q, r, 0x1.a01a01a7c41d5p-13);
  q = fma(q, r, 0x1.6c16c1788bd90p-10);
  q = fma(q, r, 0x1.11111111109b3p-7);
  q = fma(q, r, 0x1.5555555553d63p-5);
  q = fma(q, r, 0x1.5555555555556p-3);
  q = fma(q, r, 0x1.0000000000001p-1);
  return ldexp(fma(r, fma(r, q, 1.0), 1.0), (int)n);
}

template <int KIND>
struct KF {
  static constexpr bool singular = (KIND == EIFMM_K_LAPLACE || KIND == EIFMM_K_YUKAWA ||
                                     KIND == EIFMM_K_COSR || KIND == EIFMM_K_ADVDIFF);
  // the library's exponential where it shows (what_rounded)
  static constexpr bool exponential =
      (KIND == EIFMM_K_YUKAWA || KIND == EIFMM_K_GAUSS || KIND == EIFMM_K_ADVDIFF);
  __device__ static inline double eval_lib(double r2, double zx, double p) {
    const double ri = KIND == EIFMM_K_GAUSS ? 0.0 : rsq_refined(r2);
    if constexpr (KIND == EIFMM_K_YUKAWA)
      return exp(-p * (r2 * ri)) * ri;
    else if constexpr (KIND == EIFMM_K_GAUSS)
      return exp(-r2 * p);
    else
      return exp(p * (zx - r2 * ri)) * ri;
  }
  // k at z with r2 = |z|^2 and zx its first component (read by the kernel that
  // is not radial); p: Yukawa a, Gauss 1/h2, cos(w r)/r w, multiquadric c,
  // advection-diffusion a
  __device__ static inline double eval(double r2, double zx, double p) {
    if constexpr (KIND == EIFMM_K_LAPLACE) {
      return rsq_refined(r2);
    } else if constexpr (KIND == EIFMM_K_YUKAWA) {
      double ri = rsq_refined(r2);
      return exp_nonpos(-p * (r2 * ri)) * ri;
    } else if constexpr (KIND == EIFMM_K_GAUSS) {
      return exp_nonpos(-r2 * p);
    } else if constexpr (KIND == EIFMM_K_COSR) {
      double ri = rsq_refined(r2);
      return cos(p * (r2 * ri)) * ri;
    } else if constexpr (KIND == EIFMM_K_MQ) {
      return sqrt(r2 + p);
    } else if constexpr (KIND == EIFMM_K_ADVDIFF) {
      double ri = rsq_refined(r2);
      return exp_nonpos(p * (zx - r2 * ri)) * ri;
    } else {
      return r2;
    }
  }
  __device__ static inline float evalf(float r2, float zx, float p) {
    if constexpr (KIND == EIFMM_K_LAPLACE) {
      return rsqrtf(r2);
    } else if constexpr (KIND == EIFMM_K_YUKAWA) {
      float ri = rsqrtf(r2);
      return expf(-p * (r2 * ri)) * ri;
    } else if constexpr (KIND == EIFMM_K_GAUSS) {
      return expf(-r2 * p);
    } else if constexpr (KIND == EIFMM_K_COSR) {
      float ri = rsqrtf(r2);
      return cosf(p * (r2 * ri)) * ri;
    } else if constexpr (KIND == EIFMM_K_MQ) {
      return sqrtf(r2 + p);
    } else if constexpr (KIND == EIFMM_K_ADVDIFF) {
      float ri = rsqrtf(r2);
      return expf(p * (zx - r2 * ri)) * ri;
    } else {
      return r2;
    }
  }
};

// (1 / h2 of a denormal h2 stays finite: 0 times infinity at r = 0 would be no number)
inline double dev_param(int kind, double p) {
  return kind == EIFMM_K_GAUSS ? std::min(1.0 / p, DBL_MAX) : p;
}

// ------------------------------------------------------------------ leaf level
// The kernels of the leaf level (sigma gather, near field, P2M, L2P) read one
// problem's arrays from a LeafDesc.  A plan launches them with its descriptor by
// value (BATCH = false); a batch of problems launches each kernel once over the
// chunks / leaves / points of all its problems with an array of descriptors in
// device memory (BATCH = true): each workgroup finds its problem by a binary
// search over the first chunk (leaf, point) of every problem.
//
// Near field and L2P work on chunks of up to 32 consecutive targets of a leaf
// (chunk_ptr: exclusive prefix sum of ceil(count / 32) over the active leaves;
// chunk_leaf: the leaf of each),
// one chunk per 64-lane workgroup whose two halves share the chunk's work, so
// a crowded leaf of a clustered cloud spreads over many workgroups and a sparse
// one (~30 points) does not idle half a wave.

// the descriptor of work item b (a chunk or a leaf of the launch) and b's index
// within its problem
template <bool BATCH, int WHICH>  // WHICH: 0 chunk, 1 P2M segment
__device__ inline void pick_desc_at(const LeafDesc &one, const LeafDesc *__restrict__ many,
                                    int nmany, int b, LeafDesc &D, int &local, int &prob) {
  if constexpr (BATCH) {
    prob = find_last_le(nmany, b, [&](int m) {
      return WHICH == 0 ? many[m].chunk_base : many[m].seg_base;
    });
    D = many[prob];
    local = b - (int)(WHICH == 0 ? D.chunk_base : D.seg_base);
  } else {
    prob = 0;
    D = one;
    local = b;
  }
}

template <bool BATCH, int WHICH>
__device__ inline void pick_desc(const LeafDesc &one, const LeafDesc *__restrict__ many,
                                 int nmany, LeafDesc &D, int &local, int &prob) {
  pick_desc_at<BATCH, WHICH>(one, many, nmany, (int)blockIdx.x, D, local, prob);
}

// ------------------------------------------------------------------ sigma
// sig[s][r] = sigma[perm[s] + r ld] (sorted order; 0 at targets)
template <bool BATCH>
__global__ void k_gather_sigma(LeafDesc one, IoDesc ione, const LeafDesc *__restrict__ many,
                               const IoDesc *__restrict__ io, int nmany, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  LeafDesc D;
  IoDesc O;
  int64_t el = e;
  if constexpr (BATCH) {
    const int pr = find_last_le(nmany, e, [&](int m) { return many[m].pt_base; });
    D = many[pr];
    O = io[pr];
    el = e - D.pt_base;
  } else {
    D = one;
    O = ione;
  }
  const int64_t s = el / D.nrhs;
  const int r = (int)(el - s * D.nrhs);
  const int64_t src = D.perm[s];  // a target (src >= nsrc) carries no potential
  D.sig[el] = src < D.nsrc ? O.sigma[src + (int64_t)r * O.ld] : 0.0;
}

// ------------------------------------------------------------------ near field
// One 64-lane workgroup per chunk of up to 32 targets.  The sources of the
// chunk's neighbour leaves are numbered consecutively (a prefix sum over the
// near list, in LDS) and staged 64 at a time, so every batch is full whatever
// the leaf sizes; lane l and lane l + 32 hold the same target and take the
// first and the second half of each batch, and their sums are added at the end.
// The next batch is loaded into registers while the current one is used.
struct NearSrc {
  int nq;        // neighbour leaves
  int total;     // sources over all of them
  // source numbers of the chunk's own leaf, the one neighbour with pairs at r = 0
  // (a target and itself, or coincident points)
  int own_lo, own_hi;
};

// pre[e] = first source number of neighbour e, start[e] = its first point.  Lane q < 27
// looks up the box at offset (q % 3, q / 3 % 3, q / 9) - 1 of leaf j in the leaf ranges;
// the boxes that hold sources are numbered in key order (the order of their points), by
// counting the smaller keys.  No near list is read or built (a list's two passes over
// the boxes took 43-63 us of every tree, and reading it three dependent loads).
__device__ inline NearSrc near_sources(const LeafDesc &D, int j, int *pre, int *start) {
  const int lane = threadIdx.x;
  const uint32_t own = D.act[j];
  const int side = 1 << D.depth;
  const int m0 = (int)morton_axis(own, 0) + lane % 3 - 1,
            m1 = (int)morton_axis(own, 1) + lane / 3 % 3 - 1,
            m2 = (int)morton_axis(own, 2) + lane / 9 - 1;
  uint32_t key = 0xffffffffu;
  int cnt = 0, first = 0;
  if (lane < 27 && m0 >= 0 && m1 >= 0 && m2 >= 0 && m0 < side && m1 < side && m2 < side) {
    const uint32_t k = morton_encode((uint32_t)m0, (uint32_t)m1, (uint32_t)m2);
    first = D.ls[k];
    cnt = D.se[k] - first;
    if (cnt > 0) key = k;
  }
  const bool have = cnt > 0;
  const unsigned long long hb = __ballot(have);
  int rank = 0;
#pragma unroll
  for (int q = 0; q < 27; ++q)
    rank += (uint32_t)__builtin_amdgcn_readlane((int)key, q) < key ? 1 : 0;
  if (have) {
    start[rank] = first;
    pre[rank + 1] = cnt;
  }
  if (lane == 0) pre[0] = 0;
  __syncthreads();
  const int nq = (int)__popcll(hb);
  // inclusive scan of the counts over the (at most 27) neighbours
  int v = lane < nq ? pre[lane + 1] : 0;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const int u = __shfl_up(v, o);
    if ((lane & 31) >= o) v += u;
  }
  __syncthreads();
  if (lane < nq) pre[lane + 1] = v;
  __syncthreads();
  // the own leaf is offset 13 (it may hold targets only)
  const bool self = (hb >> 13) & 1ull;
  const int eo = __builtin_amdgcn_readlane(rank, 13);
  return NearSrc{nq, pre[nq], self ? pre[eo] : 0, self ? pre[eo + 1] : 0};
}

// point index of source number v (0 <= v < total); e is the neighbour of the
// lane's previous (smaller) source number, so the search resumes there
__device__ inline int near_point(int v, int nq, const int *pre, const int *start, int &e) {
  while (e + 1 < nq && pre[e + 1] <= v) ++e;
  return start[e] + (v - pre[e]);
}

// The lanes of chunk c of leaf j: with k targets (a chunk holds up to 32) and P
// the smallest power of two >= k, lane l holds target l mod P and takes sources
// [P (l / P), P (l / P + 1)) of every 64-source batch, so that a chunk of few
// targets (the last of a leaf) spreads each target's sources over 64 / P lanes
// instead of leaving lanes idle.  A full chunk has P = 32: lanes l and l + 32
// share a target and take the two halves of each batch.
struct ChunkLanes {
  int i;     // the lane's target point
  bool tv;   // the target exists
  int P;     // targets' lane period
  int u0;    // first source of the lane's range in a batch
};
// (spread: false keeps P = 32: the FP64 near field with several right-hand
// sides, whose RB sums per pair already fill the lanes' registers)
__device__ inline ChunkLanes chunk_lanes(const LeafDesc &D, int j, int c, int lane, bool spread) {
  const uint32_t key = D.act[j];
  const int i0 = D.tb[key] + 32 * (c - D.chunk_ptr[j]);
  const int k = min(32, D.ls[key + 1] - i0);
  const int P = !spread ? 32 : k <= 1 ? 1 : 1 << (32 - __clz(k - 1));
  const int ti = lane & (P - 1);
  return ChunkLanes{i0 + ti, ti < k, P, lane - ti};
}

// (cos(wr)/r asks for three waves per SIMD: its kernel value would otherwise
// take registers for two only)
template <int KIND, int RB, bool BATCH>
__global__ __launch_bounds__(64, KIND == EIFMM_K_COSR ? 3 : 1) void k_p2p64(
    LeafDesc one, const LeafDesc *__restrict__ many, int nmany) {
  __shared__ double sx[64], sy[64], sz[64], ss[64 * RB];
  __shared__ int pre[28], start[27];
  LeafDesc D;
  int c, prob;
  pick_desc<BATCH, 0>(one, many, nmany, D, c, prob);
  if (c >= D.chunk_ptr[D.nleaf]) return;  // past the last chunk (the grid is a bound)
  const int lane = threadIdx.x;
  const int64_t n = D.n;
  const int nrhs = D.nrhs;
  const double *__restrict__ xyz = D.xyz;
  const double *__restrict__ sig = D.sig;
  const int j = D.chunk_leaf[c];
  const ChunkLanes CL = chunk_lanes(D, j, c, lane, RB == 1);
  const int i = CL.i;
  const bool tv = CL.tv;
  const double xi = tv ? xyz[i] : 0.0, yi = tv ? xyz[n + i] : 0.0, zi = tv ? xyz[2 * n + i] : 0.0;
  const NearSrc S = near_sources(D, j, pre, start);
  for (int r0 = 0; r0 < nrhs; r0 += RB) {
    double acc[RB];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) acc[rr] = 0.0;
    double px = 0, py = 0, pz = 0, ps[RB];
    // a block past the end is padded with the last source at zero potential, so
    // every block has 64 sources and the pair loop a fixed trip count
    int ecur = 0;  // neighbour of this lane's last source number
    auto load = [&](int base) {
      const int v = base + lane;
      if (S.total > 0) {
        const int sidx = near_point(v < S.total ? v : S.total - 1, S.nq, pre, start, ecur);
        px = xyz[sidx];
        py = xyz[n + sidx];
        pz = xyz[2 * n + sidx];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr)
          ps[rr] = (v < S.total && r0 + rr < nrhs) ? sig[(int64_t)sidx * nrhs + r0 + rr] : 0.0;
      }
    };
    load(0);
    for (int base = 0; base < S.total; base += 64) {
      __syncthreads();
      sx[lane] = px;
      sy[lane] = py;
      sz[lane] = pz;
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) ss[lane * RB + rr] = ps[rr];
      __syncthreads();
      if (base + 64 < S.total) load(base + 64);
      // r = 0 (a pair the sum leaves out) needs the mask only in the batches that
      // hold sources of the own leaf: points of two different leaves are apart (a
      // leaf boundary lies between them), so r2 > 0 there, unless both lie within
      // about 1e-154 of a boundary at the origin, which the library does not
      // support.  The padding past the end repeats the last source, so it needs
      // the mask only when that source is the own leaf's, whose batch has it.
      // (several RHS share each pair's mask: they keep the one loop)
      const bool own =
          KF<KIND>::singular && (RB > 1 || (base < S.own_hi && base + 64 > S.own_lo));
      // (a full chunk's loop has a fixed trip count of 32)
      // (several RHS hold RB sums per pair already; a partial chunk's loop runs
      // at most 16 times)
      auto pairs = [&](auto masked, auto full) {
        constexpr bool F = decltype(full)::value;
        constexpr int kUnroll = RB > 1 ? 2 : (F ? 8 : 1);
        const int cnt = F ? 32 : CL.P;
#pragma unroll kUnroll
        for (int q = 0; q < cnt; ++q) {
          const int u = CL.u0 + q;
          const double dx = xi - sx[u], dy = yi - sy[u], dz = zi - sz[u];
          const double r2 = dx * dx + dy * dy + dz * dz;
          double kv = KF<KIND>::eval(r2, dx, D.p);
          if constexpr (decltype(masked)::value) kv = (r2 == 0.0) ? 0.0 : kv;
#pragma unroll
          for (int rr = 0; rr < RB; ++rr) acc[rr] += ss[u * RB + rr] * kv;
        }
      };
      if (RB > 1 || CL.P == 32) {
        if (own)
          pairs(std::true_type{}, std::true_type{});
        else
          pairs(std::false_type{}, std::true_type{});
      } else {
        if (own)
          pairs(std::true_type{}, std::false_type{});
        else
          pairs(std::false_type{}, std::false_type{});
      }
    }
    // the target's 64 / P partial sums (lanes l, l + P, ...)
    for (int o = CL.P; o < 64; o <<= 1) {
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) acc[rr] += __shfl_xor(acc[rr], o);
    }
    if (tv && lane < CL.P) {
#pragma unroll
      for (int rr = 0; rr < RB; ++rr)
        if (r0 + rr < nrhs) D.fnear[(int64_t)i * nrhs + r0 + rr] = acc[rr];
    }
  }
}

// Mixed-precision near field: the coordinate differences are taken in FP64 and
// rounded once to FP32 (so a close pair keeps its relative accuracy however
// crowded the leaf), kernel values and products in FP32, two-sum-compensated
// FP32 sums per half, the two halves and their compensations added in FP64.
template <int KIND, int RB, bool BATCH>
__global__ __launch_bounds__(64) void k_p2p32(LeafDesc one, const LeafDesc *__restrict__ many,
                                              int nmany) {
  __shared__ double sx[64], sy[64], sz[64];
  __shared__ float ss[64 * RB];
  __shared__ int pre[28], start[27];
  LeafDesc D;
  int c, prob;
  pick_desc<BATCH, 0>(one, many, nmany, D, c, prob);
  if (c >= D.chunk_ptr[D.nleaf]) return;  // past the last chunk (the grid is a bound)
  const int lane = threadIdx.x;
  const int64_t n = D.n;
  const int nrhs = D.nrhs;
  const float p = (float)D.p;
  const double *__restrict__ xyz = D.xyz;
  const double *__restrict__ sig = D.sig;
  const int j = D.chunk_leaf[c];
  // (several RHS too: 64 RHS on 2^20 points, 264 -> 261 ms)
  const ChunkLanes CL = chunk_lanes(D, j, c, lane, true);
  const int i = CL.i;
  const bool tv = CL.tv;
  const double xi = tv ? xyz[i] : 0.0, yi = tv ? xyz[n + i] : 0.0, zi = tv ? xyz[2 * n + i] : 0.0;
  const NearSrc S = near_sources(D, j, pre, start);
  for (int r0 = 0; r0 < nrhs; r0 += RB) {
    float sum[RB], cmp[RB];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) sum[rr] = cmp[rr] = 0.f;
    double px = 0, py = 0, pz = 0;
    float ps[RB];
    // padding past the end as in k_p2p64 (zero potential adds exactly zero to
    // the compensated sums)
    int ecur = 0;  // neighbour of this lane's last source number
    auto load = [&](int base) {
      const int v = base + lane;
      if (S.total > 0) {
        const int sidx = near_point(v < S.total ? v : S.total - 1, S.nq, pre, start, ecur);
        px = xyz[sidx];
        py = xyz[n + sidx];
        pz = xyz[2 * n + sidx];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr)
          ps[rr] = (v < S.total && r0 + rr < nrhs) ? (float)sig[(int64_t)sidx * nrhs + r0 + rr]
                                                   : 0.f;
      }
    };
    load(0);
    for (int base = 0; base < S.total; base += 64) {
      __syncthreads();
      sx[lane] = px;
      sy[lane] = py;
      sz[lane] = pz;
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) ss[lane * RB + rr] = ps[rr];
      __syncthreads();
      if (base + 64 < S.total) load(base + 64);
      // the r = 0 mask only in batches with the own leaf's sources, as in
      // k_p2p64 (here r2 is FP32: two points of different leaves give r2 = 0
      // only when under about 1e-22 apart, next to a boundary at the origin)
      // (several RHS share each pair's mask: they keep the one loop)
      const bool own =
          KF<KIND>::singular && (RB > 1 || (base < S.own_hi && base + 64 > S.own_lo));
      auto pairs = [&](auto masked, auto full) {
        constexpr bool F = decltype(full)::value;
        constexpr int kUnroll = RB > 1 ? 2 : (F ? 4 : 2);
        const int cnt = F ? 32 : CL.P;
#pragma unroll kUnroll
        for (int q = 0; q < cnt; ++q) {
          const int u = CL.u0 + q;
          const float dx = (float)(xi - sx[u]), dy = (float)(yi - sy[u]),
                      dz = (float)(zi - sz[u]);
          const float r2 = dx * dx + dy * dy + dz * dz;
          float kv = KF<KIND>::evalf(r2, dx, p);
          if constexpr (decltype(masked)::value) kv = (r2 == 0.f) ? 0.f : kv;
#pragma unroll
          for (int rr = 0; rr < RB; ++rr) {
            // the rounding error of sum + w, exactly, by the branch-free two-sum
            // (Knuth): no magnitude comparison as in Neumaier's form
            const float w = ss[u * RB + rr] * kv;
            const float tsum = sum[rr] + w;
            const float bv = tsum - sum[rr];
            cmp[rr] += (sum[rr] - (tsum - bv)) + (w - bv);
            sum[rr] = tsum;
          }
        }
      };
      if (CL.P == 32) {
        if (own)
          pairs(std::true_type{}, std::true_type{});
        else
          pairs(std::false_type{}, std::true_type{});
      } else {
        if (own)
          pairs(std::true_type{}, std::false_type{});
        else
          pairs(std::false_type{}, std::false_type{});
      }
    }
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      // the target's 64 / P partial sums (lanes l, l + P, ...), in FP64
      double mine = (double)sum[rr] + (double)cmp[rr];
      for (int o = CL.P; o < 64; o <<= 1) mine += __shfl_xor(mine, o);
      if (tv && lane < CL.P && r0 + rr < nrhs) D.fnear[(int64_t)i * nrhs + r0 + rr] = mine;
    }
  }
}

// ------------------------------------------------------------------ P2M
// W^I_m = sum_{y_j in I} sigma_j K(x_m^{I_0}, y_j - c_I)  (Algorithm 3, step 1)
// One NT-thread workgroup per leaf, or with one right-hand side per segment of up to
// kSegSources sources of a leaf: a crowded leaf's sources spread over many workgroups
// (32 problems with four clusters each and d = 433 spent 4.5 ms on the workgroups of a
// few leaves of 1e4 sources).  A leaf's first segment writes W, the others their sums
// to w_ext (extra i of the leaves before it and of its own), which k_p2m_ext adds.
// (Where the solved What is rounded to FP32, what_rounded, a leaf is one segment.)
// Rows are taken in groups of 4 NT, thread t
// owning rows m0 + t + NT u, u < 4, of group m0.  NT = 0: the launch's block size
// (one right-hand side on leaves of many points: a whole number of waves
// covering d_p, up to 1024, so that every wave takes one row per lane and none
// waits at the batch barriers for a wave with two); otherwise 256 threads
// (several right-hand sides: their registers rule out 1024-thread blocks), or
// one wave when d_p <= 64.
template <int KIND, int RB, bool BATCH, int NT, bool LIB>
__global__ __launch_bounds__(NT ? NT : 1024) void k_p2m(LeafDesc one,
                                                        const LeafDesc *__restrict__ many,
                                                        int nmany) {
  __shared__ double px[64], py[64], pz[64], ps[64 * RB];
  LeafDesc D;
  int j, prob;
  pick_desc<BATCH, 1>(one, many, nmany, D, j, prob);
  int seg = 0;
  double *Wj = nullptr;
  if constexpr (RB == 1) {  // j: segment -> leaf
    const int sj = j;
    j = D.seg_leaf[sj];
    const int s0 = D.seg_ptr[j];
    seg = sj - s0;
    Wj = seg == 0 ? D.W + (int64_t)j * D.dp : D.w_ext + (int64_t)(s0 - j + seg - 1) * D.dp;
  }
  const int t = threadIdx.x;
  const int nt = NT ? NT : (int)blockDim.x;
  const int64_t n = D.n;
  const int nrhs = D.nrhs, d = D.d, dp = D.dp;
  const double *__restrict__ xyz = D.xyz;
  const double *__restrict__ sig = D.sig;
  const uint32_t key = D.act[j];
  const int a = D.ls[key] + D.seg_len * seg;
  const int b = RB == 1 ? min(D.se[key], a + D.seg_len) : D.se[key];
  const double cx = D.lo0 + ((double)morton_axis(key, 0) + 0.5) * D.h;
  const double cy = D.lo1 + ((double)morton_axis(key, 1) + 0.5) * D.h;
  const double cz = D.lo2 + ((double)morton_axis(key, 2) + 0.5) * D.h;
  for (int m0 = 0; m0 < dp; m0 += 4 * nt) {
    const int nu = min(4, (dp - m0 + nt - 1) / nt);
    double xm[4], ym[4], zm[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = m0 + t + nt * u;
      const bool ok = u < nu && m < d;
      xm[u] = ok ? D.X[3 * m] : 0.0;
      ym[u] = ok ? D.X[3 * m + 1] : 0.0;
      zm[u] = ok ? D.X[3 * m + 2] : 0.0;
    }
    for (int r0 = 0; r0 < nrhs; r0 += RB) {
      double acc[4][RB];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) acc[u][rr] = 0.0;
      for (int s0 = a; s0 < b; s0 += 64) {
        const int cnt = min(64, b - s0);
        __syncthreads();
        if (t < cnt) {
          const int s = s0 + t;
          px[t] = xyz[s] - cx;
          py[t] = xyz[n + s] - cy;
          pz[t] = xyz[2 * n + s] - cz;
#pragma unroll
          for (int rr = 0; rr < RB; ++rr)
            ps[t * RB + rr] = (r0 + rr < nrhs) ? sig[(int64_t)s * nrhs + r0 + rr] : 0.0;
        }
        __syncthreads();
        for (int q = 0; q < cnt; ++q) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            // skipped by a whole wave whose rows all lie past d (rows d..dp-1
            // are stored as zeros)
            if (u < nu && m0 + nt * u + (t & ~63) < d) {
              const double dx = xm[u] - px[q], dy = ym[u] - py[q], dz = zm[u] - pz[q];
              const double r2 = dx * dx + dy * dy + dz * dz;
              double kv;
              if constexpr (LIB)
                kv = KF<KIND>::eval_lib(r2, dx, D.p);
              else
                kv = KF<KIND>::eval(r2, dx, D.p);
#pragma unroll
              for (int rr = 0; rr < RB; ++rr) acc[u][rr] += ps[q * RB + rr] * kv;
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int m = m0 + t + nt * u;
        if (u < nu && m < dp) {
#pragma unroll
          for (int rr = 0; rr < RB; ++rr)
            if (RB == 1)
              Wj[m] = m < d ? acc[u][rr] : 0.0;
            else if (r0 + rr < nrhs)
              D.W[((int64_t)j * nrhs + r0 + rr) * dp + m] = m < d ? acc[u][rr] : 0.0;
        }
      }
    }
  }
}

// adds the sums of a leaf's later segments to its first one's, in order (one workgroup
// per segment; those that are not a leaf's first of several exit)
template <bool BATCH>
__global__ __launch_bounds__(256) void k_p2m_ext(LeafDesc one, const LeafDesc *__restrict__ many,
                                                 int nmany) {
  LeafDesc D;
  int s, prob;
  pick_desc<BATCH, 1>(one, many, nmany, D, s, prob);
  const int j = D.seg_leaf[s], s0 = D.seg_ptr[j], n = D.seg_ptr[j + 1] - s0;
  if (s != s0 || n < 2) return;
  const double *e = D.w_ext + (int64_t)(s0 - j) * D.dp;
  for (int m = threadIdx.x; m < D.d; m += 256) {
    double v = D.W[(int64_t)j * D.dp + m];
    for (int i = 0; i < n - 1; ++i) v += e[(int64_t)i * D.dp + m];
    D.W[(int64_t)j * D.dp + m] = v;
  }
}

// ------------------------------------------------------------------ L2P + combine
// f(x_i) = sum_{l'} K(x_i - c_I, y_{l'}^{I_0}) lhat_{l'}^I + f_near(x_i), written to
// the input position of x_i (Algorithm 3, step 7).  One 64-lane workgroup per
// chunk of up to 32 targets: lane l and lane l + 32 hold the same target and sum
// the first and the second half of the d terms (a chunk of fewer targets
// spreads each over more lanes: chunk_lanes).
template <int KIND, int RB, bool BATCH>
__global__ __launch_bounds__(64) void k_l2p(LeafDesc one, IoDesc ione,
                                            const LeafDesc *__restrict__ many,
                                            const IoDesc *__restrict__ io, int nmany) {
  extern __shared__ double sm[];
  LeafDesc D;
  int c, prob;
  pick_desc<BATCH, 0>(one, many, nmany, D, c, prob);
  if (c >= D.chunk_ptr[D.nleaf]) return;  // past the last chunk (the grid is a bound)
  IoDesc O;
  if constexpr (BATCH)
    O = io[prob];
  else
    O = ione;
  // lhat and its points: the second EIM's size and y^{I_0} with two EIMs per level
  const int dp = D.dpL, d = D.dL, nrhs = D.nrhs;
  const int64_t n = D.n;
  double *sX = sm, *sl = sm + 3 * dp;
  const int lane = threadIdx.x;
  const int j = D.chunk_leaf[c];
  const uint32_t key = D.act[j];
  // the chunk's lanes as in the near field: 64 / P lanes per target, each
  // summing one of 64 / P equal ranges of the d terms (P = 32: two halves)
  const ChunkLanes CL = chunk_lanes(D, j, c, lane, true);
  const int i = CL.i;
  const double cx = D.lo0 + ((double)morton_axis(key, 0) + 0.5) * D.h;
  const double cy = D.lo1 + ((double)morton_axis(key, 1) + 0.5) * D.h;
  const double cz = D.lo2 + ((double)morton_axis(key, 2) + 0.5) * D.h;
  for (int e = lane; e < 3 * d; e += 64) sX[e] = D.XL[e];
  const bool tv = CL.tv;
  const double xc = tv ? D.xyz[i] - cx : 0.0, yc = tv ? D.xyz[n + i] - cy : 0.0,
               zc = tv ? D.xyz[2 * n + i] - cz : 0.0;
  const int ng = 64 / CL.P, grp = lane / CL.P;
  const int dh = (d + ng - 1) / ng, l0 = grp * dh, l1 = min(d, l0 + dh);
  for (int r0 = 0; r0 < nrhs; r0 += RB) {
    __syncthreads();
    for (int e = lane; e < RB * d; e += 64) {
      const int rr = e / d, l = e - rr * d;
      sl[rr * dp + l] = (r0 + rr < nrhs) ? D.lhat[((int64_t)j * nrhs + r0 + rr) * dp + l] : 0.0;
    }
    __syncthreads();
    double acc[RB];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) acc[rr] = 0.0;
#pragma unroll 4
    for (int l = l0; l < l1; ++l) {
      const double dx = xc - sX[3 * l], dy = yc - sX[3 * l + 1], dz = zc - sX[3 * l + 2];
      const double kv = KF<KIND>::eval(dx * dx + dy * dy + dz * dz, dx, D.p);
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) acc[rr] += kv * sl[rr * dp + l];
    }
    for (int o = CL.P; o < 64; o <<= 1) {
#pragma unroll
      for (int rr = 0; rr < RB; ++rr) acc[rr] += __shfl_xor(acc[rr], o);
    }
    if (tv && lane < CL.P) {
      const int64_t o = D.perm[i] - D.toff;
#pragma unroll
      for (int rr = 0; rr < RB; ++rr)
        if (r0 + rr < nrhs)
          O.f[o + (int64_t)(r0 + rr) * O.ldf] = acc[rr] + D.fnear[(int64_t)i * nrhs + r0 + rr];
    }
  }
}

// depth < 2: no far field, f = f_near in input order
// (targets only: input indices from toff on)
__global__ void k_combine_near(int64_t n, int nrhs, const double *__restrict__ fnear,
                               const int *__restrict__ perm, int64_t toff, double *__restrict__ f,
                               int64_t ldf) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * nrhs) return;
  int64_t s = e / nrhs;
  int r = (int)(e - s * nrhs);
  const int64_t o = (int64_t)perm[s] - toff;
  if (o >= 0) f[o + (int64_t)r * ldf] = fnear[e];
}

// ------------------------------------------------------------------ triangular solves
// One wave per 16 columns (box, rhs).  Forward substitution with the lower
// factor, then backward substitution with the upper factor, in 16-row tiles:
//   r_bi = v_bi - sum_{bj < bi} T[bi][bj] z_bj        (MFMA, -T tiles in the table)
//   z_bi = T[bi][bi]^{-1} r_bi                       (MFMA with the inverted tile)
// The solved tiles of the 16 columns stay in LDS.  In the FP64 16x16x4 MFMA the
// result register q of lane l holds row (l / 16) + 4 q of column l % 16, which
// is exactly the B operand that lane supplies at k-step q, so tiles feed the
// next product without data movement.
//   Delta   v: Gamma z = v, then B^T w = z
//   Delta^T v: B z = v,     then Gamma^T w = z
struct SolveArgs {
  SolveDesc lv[kMaxLevels];
  int nlev;
};

__device__ inline void trsm_body(const SolveDesc &D, double *zs) {
  typedef double v4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x;
  const int c = ((int)blockIdx.x - D.blk_start) * 16 + (lane & 15);
  const bool cv = c < D.ncols;
  const int dp = D.dp, nb = dp >> 4, rs = lane >> 4;
  const double *x = D.in + (int64_t)(cv ? c : 0) * dp;
  double *y = D.out + (int64_t)(cv ? c : 0) * dp;
  // acc += sum over tiles j in [j0, j1) of row Ar's tile j times z_j, in two
  // accumulation chains (even and odd tiles).  The operator fragments of a pair
  // of tiles are loaded a pair ahead; past the end the loads read the row's last
  // tile, so the loads in flight do not depend on the data.
  auto row_sum = [&](const double *Ar, int j0, int j1, v4 &acc) {
    v4 acc2 = {0, 0, 0, 0};
    const int npair = (j1 - j0) >> 1;
    double fa[2][4], fb[2][4];
    auto load = [&](double(&f)[2][4], int j) {
      const int ja = min(j, nb - 1), jb = min(j + 1, nb - 1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        f[0][ks] = Ar[ja * 256 + ks * 64];
        f[1][ks] = Ar[jb * 256 + ks * 64];
      }
    };
    auto mul = [&](const double(&f)[2][4], int j) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[0][ks], zs[(j * 4 + ks) * 64 + lane], acc, 0,
                                                   0, 0);
        acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(f[1][ks], zs[((j + 1) * 4 + ks) * 64 + lane],
                                                    acc2, 0, 0, 0);
      }
    };
    int p = 0, j = j0;
    load(fa, j);
    for (; p + 2 <= npair; p += 2, j += 4) {
      load(fb, j + 2);
      mul(fa, j);
      load(fa, j + 4);
      mul(fb, j + 2);
    }
    if (p < npair) {
      mul(fa, j);
      j += 2;
    }
    if (j < j1) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Ar[j * 256 + ks * 64],
                                                   zs[(j * 4 + ks) * 64 + lane], acc, 0, 0, 0);
    }
    acc += acc2;
  };
  if (!D.Tf) {
    // no forward factor (folded into the producers of the input): z = v
    for (int bi = 0; bi < nb; ++bi)
#pragma unroll
      for (int q = 0; q < 4; ++q) zs[(bi * 4 + q) * 64 + lane] = cv ? x[16 * bi + rs + 4 * q] : 0.0;
  }
  v4 xn;
#pragma unroll
  for (int q = 0; q < 4; ++q) xn[q] = (cv && D.Tf) ? x[rs + 4 * q] : 0.0;
  for (int bi = 0; D.Tf && bi < nb; ++bi) {
    v4 acc = xn;
    // the next row's right-hand side, loaded during this row's products
    const int bn = min(bi + 1, nb - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) xn[q] = cv ? x[16 * bn + rs + 4 * q] : 0.0;
    const double *Ar = D.Tf + (int64_t)bi * nb * 256 + lane;
    double dg[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) dg[ks] = Ar[bi * 256 + ks * 64];
    row_sum(Ar, 0, bi, acc);
    v4 z = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) z = __builtin_amdgcn_mfma_f64_16x16x4f64(dg[ks], acc[ks], z, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) zs[(bi * 4 + q) * 64 + lane] = z[q];
    if (!D.Tb && cv) {
#pragma unroll
      for (int q = 0; q < 4; ++q) y[16 * bi + rs + 4 * q] = z[q];
    }
  }
  if (!D.Tb) return;  // forward solve only
  for (int bi = nb - 1; bi >= 0; --bi) {
    v4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = zs[(bi * 4 + q) * 64 + lane];
    const double *Ar = D.Tb + (int64_t)bi * nb * 256 + lane;
    double dg[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) dg[ks] = Ar[bi * 256 + ks * 64];
    row_sum(Ar, bi + 1, nb, acc);
    v4 w = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) w = __builtin_amdgcn_mfma_f64_16x16x4f64(dg[ks], acc[ks], w, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) zs[(bi * 4 + q) * 64 + lane] = w[q];
    if (cv) {
#pragma unroll
      for (int q = 0; q < 4; ++q) y[16 * bi + rs + 4 * q] = w[q];
      if (D.out32) {
        float *y32 = D.out32 + (int64_t)c * dp;
#pragma unroll
        for (int q = 0; q < 4; ++q) y32[16 * bi + rs + 4 * q] = (float)w[q];
      }
    }
  }
}

// The same solve by four waves per 16 columns, for FP64 results.  Each wave owns every
// fourth row tile: once tile bi is solved (by every wave for itself, from the right-hand
// side in LDS), each takes its product off its own rows, so the chain from one tile to
// the next is four products, an LDS hand-off and four more instead of a whole row of
// products, and the loads of the next tile's operators (which need no solved value) are
// in flight meanwhile.  On 287 rows a solve of 576 columns takes 46 us against 85 by one
// wave, half a solve of 4,096 columns 26 against 62; on 37,440 columns, where the
// matrix cores are busy either way, the repeated diagonal products cost more than the
// waits (157 against 126 us), so the one-wave form serves more than kSolveFew groups.
// The products of a row are added in another order, which changes FP64 results in the
// last bits; the FP32 copy of a solve (mixed precision, uncompressed levels) would
// change in its own last bit, so the mixed pass solves for What by the one-wave form.
// Neither order is nearer to the exact solve: this only keeps the results that the mixed
// pass had (on every mixed plan: the compressed ones' FP32 copy is taken after the
// projection, where the order hardly shows, but they keep it too).
constexpr int kSolveOwn = 5;  // tiles of a wave with their operators loaded ahead
constexpr int kSolveFew = 1024;  // 16-column groups up to which the four-wave form serves
__device__ inline void trsm4_body(const SolveDesc &D, double *zs) {
  typedef double v4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = ((int)blockIdx.x - D.blk_start) * 16 + (lane & 15);
  const bool cv = c < D.ncols;
  const int dp = D.dp, nb = dp >> 4, rs = lane >> 4;
  const double *x = D.in + (int64_t)(cv ? c : 0) * dp;
  double *y = D.out + (int64_t)(cv ? c : 0) * dp;
  for (int bi = w; bi < nb; bi += 4)
#pragma unroll
    for (int q = 0; q < 4; ++q) zs[(bi * 4 + q) * 64 + lane] = cv ? x[16 * bi + rs + 4 * q] : 0.0;
  // one triangle: step s solves tile bi(s); FWD from the first tile down, else from the
  // last one up; store: the solved tiles are the result
  auto sweep = [&](auto fwd, const double *T, bool store) {
    constexpr bool FWD = decltype(fwd)::value;
    auto tile_of = [&](int s) { return FWD ? s : nb - 1 - s; };
    // the wave's rows after step s: own0(s), own0(s) + DIR 4, ..., count(s) of them
    constexpr int DIR = FWD ? 4 : -4;
    auto own0 = [&](int s) {
      return FWD ? s + 1 + ((w - (s + 1)) & 3) : nb - 2 - s - ((nb - 2 - s - w) & 3);
    };
    auto count = [&](int s) {
      const int b = own0(s);
      return FWD ? (b < nb ? (nb - 1 - b) / 4 + 1 : 0) : (b >= 0 ? b / 4 + 1 : 0);
    };
    // diagonal and own operators of a step, loaded two steps ahead
    struct Ops {
      double dg[4], a[kSolveOwn][4];
    };
    Ops o0, o1;
    auto load = [&](int s, Ops &o) {
      if (s >= nb) return;
      const int bi = tile_of(s), n = count(s);
      const double *Tl = T + lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) o.dg[k] = Tl[((int64_t)bi * nb + bi) * 256 + k * 64];
      const double *Tr = Tl + ((int64_t)own0(s) * nb + bi) * 256;
#pragma unroll
      for (int i = 0; i < kSolveOwn; ++i)
        if (i < n)
#pragma unroll
          for (int k = 0; k < 4; ++k) o.a[i][k] = Tr[(int64_t)i * DIR * nb * 256 + k * 64];
    };
    load(0, o0);
    load(1, o1);
    v4 zp = {0, 0, 0, 0};
    // the products of the wave's first N rows with the solved tile z, all rows at once
    auto rows = [&](auto N, int b0, const Ops &o, const v4 &z) {
      constexpr int n = decltype(N)::value;
      double *zr = zs + b0 * 256 + lane;
      v4 r[n];
#pragma unroll
      for (int i = 0; i < n; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) r[i][q] = zr[i * DIR * 256 + q * 64];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < n; ++i)
          r[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[i][k], z[k], r[i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < n; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) zr[i * DIR * 256 + q * 64] = r[i][q];
    };
    auto step = [&](int s, Ops &o) {
      const int bi = tile_of(s), n = count(s), b0 = own0(s);
      lds_barrier();  // the rows' right-hand sides are up to date
      if (s > 0 && w == ((s - 1) & 3)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) zs[(tile_of(s - 1) * 4 + q) * 64 + lane] = zp[q];
      }
      v4 z = {0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        z = __builtin_amdgcn_mfma_f64_16x16x4f64(o.dg[k], zs[(bi * 4 + k) * 64 + lane], z, 0, 0, 0);
      static_assert(kSolveOwn == 5, "cases below");
      switch (n) {
        case 0: break;
        case 1: rows(std::integral_constant<int, 1>{}, b0, o, z); break;
        case 2: rows(std::integral_constant<int, 2>{}, b0, o, z); break;
        case 3: rows(std::integral_constant<int, 3>{}, b0, o, z); break;
        case 4: rows(std::integral_constant<int, 4>{}, b0, o, z); break;
        default: rows(std::integral_constant<int, 5>{}, b0, o, z); break;
      }
      load(s + 2, o);
      // rows further on
      for (int i = kSolveOwn; i < n; ++i) {
        const int bj = b0 + DIR * i;
        v4 rr;
#pragma unroll
        for (int q = 0; q < 4; ++q) rr[q] = zs[(bj * 4 + q) * 64 + lane];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          rr = __builtin_amdgcn_mfma_f64_16x16x4f64(T[((int64_t)bj * nb + bi) * 256 + k * 64 + lane],
                                                    z[k], rr, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) zs[(bj * 4 + q) * 64 + lane] = rr[q];
      }
      zp = z;
      if (store && cv && w == (s & 3)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) y[16 * bi + rs + 4 * q] = z[q];
      }
    };
    for (int s = 0; s < nb; s += 2) {
      step(s, o0);
      if (s + 1 < nb) step(s + 1, o1);
    }
    if (w == ((nb - 1) & 3)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) zs[(tile_of(nb - 1) * 4 + q) * 64 + lane] = zp[q];
    }
  };
  if (D.Tf) sweep(std::true_type{}, D.Tf, D.Tb == nullptr);
  if (D.Tb) sweep(std::false_type{}, D.Tb, true);
}

// LDS bytes of a solve launch: the solved tiles of the 16 columns
inline size_t trsm_shm(int dp) { return sizeof(double) * 4 * 64 * (size_t)(dp / 16); }

// one plan: up to one descriptor per level, passed by value
__global__ __launch_bounds__(64) void k_trsm(SolveArgs A) {
  extern __shared__ double zs[];  // [nb][4][64]
  int li = 0;
  for (int q = 1; q < A.nlev; ++q)
    if ((int)blockIdx.x >= A.lv[q].blk_start) li = q;
  trsm_body(A.lv[li], zs);
}

__global__ __launch_bounds__(256) void k_trsm4(SolveArgs A) {
  extern __shared__ double zs[];  // [nb][4][64]
  int li = 0;
  for (int q = 1; q < A.nlev; ++q)
    if ((int)blockIdx.x >= A.lv[q].blk_start) li = q;
  trsm4_body(A.lv[li], zs);
}

__global__ __launch_bounds__(256) void k_trsm4_list(const SolveDesc *__restrict__ L, int n) {
  extern __shared__ double zs[];
  const int li = find_last_le(n, blockIdx.x, [&](int m) { return (int64_t)L[m].blk_start; });
  const SolveDesc D = L[li];
  trsm4_body(D, zs);
}

// a batch: every (problem, level) of the launch, descriptors in device memory
__global__ __launch_bounds__(64) void k_trsm_list(const SolveDesc *__restrict__ L, int n) {
  extern __shared__ double zs[];
  const int li = find_last_le(n, blockIdx.x, [&](int m) { return (int64_t)L[m].blk_start; });
  const SolveDesc D = L[li];
  trsm_body(D, zs);
}

// ------------------------------------------------------------------ gathered GEMM
// C[:, col] (+)= sum_t A_t B_t[:, col] for the columns (box, RHS) of a target
// group, where B_t[:, col] is the expansion of the source box that term t pairs
// with the column's target box: M2M child t; L2L the parent; PROJ the box itself
// (compression projections).  (The M2L has kernels of its own.)  A workgroup
// computes a (16 RBT)-row tile, 128 columns wide for 3 and 4 row blocks and 64 for
// 5 and 6, with 16x16x4 MFMAs; each of the 4 waves owns a quarter of the columns
// and all RBT row blocks.  The operator chunks of 16 k values pass through LDS in
// MFMA fragment order, loaded two chunks ahead of their products.
constexpr int MODE_M2M = 0, MODE_M2L = 1, MODE_L2L = 2, MODE_PROJ = 3;
// 16-column blocks per wave: 2 (128-column tiles) for 3- and 4-block tiles, 1
// (64 columns) for taller ones, whose accumulators and three sets of prefetched
// operands would not fit the registers of two waves per SIMD otherwise
__host__ __device__ constexpr int gemm_cpw(int rbt) { return rbt >= 5 ? 1 : 2; }
static_assert(gemm_cpw(6) == 1 && gemm_cpw(4) == 2 && gemm_cpw(3) == 2, "tile widths");
__host__ __device__ constexpr int gemm_cols(int rbt) { return 64 * gemm_cpw(rbt); }
// zeros, read in place of a missing source column or of operator rows past the
// operator, so that every chunk issues the same loads (static device memory is
// zero-initialized; 1024 covers the longest column, d_k <= 1024)
__device__ double g_gemm_zero[1024];
// the slots read for a missing source: no box (one per column of a lane, so that
// the dummy loads stay distinct loads)
__device__ int g_slot_none[2] = {-1, -1};

// Operand layouts: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and rows
// (l / 16) + 4 q of column l % 16 of the result in register q.
__device__ inline d4v mfma_f64(double a, double b, d4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Where the slot of the source box that term `term` pairs with target (tkey, ts)
// is read: M2M child `term`, L2L the parent (entries of the source level's slot
// map, which holds -1 for an empty box); PROJ needs no read (the box itself).  For
// a missing column the address is g_slot_none[jj] (-1, no box), so that every lane reads,
// the number of loads in flight does not depend on the data, and the value read
// needs no select (a select right after the load would wait for it).
template <int MODE>
__device__ inline const int *gemm_source_addr(int term, bool cvalid, uint32_t tkey,
                                              const int *__restrict__ src_slot, int jj) {
  const uint32_t skey = MODE == MODE_M2M ? tkey * 8u + (uint32_t)term : tkey >> 3;
  return (cvalid && src_slot) ? src_slot + skey : &g_slot_none[jj];
}

__device__ inline const double *gemm_source_ptr(const GemmJob &J, int s, int r,
                                                const double *Bsrc) {
  return s < 0 ? nullptr : Bsrc + ((int64_t)s * J.nrhs + r) * J.dpk;
}

template <int MODE>
__device__ inline const double *gemm_operand(const GemmJob &J, int term) {
  const int64_t idx = MODE == MODE_M2M ? term : MODE == MODE_L2L ? J.cls : 0;
  return (const double *)J.A + idx * J.a_stride;
}

// Schedule (data-parallel + Stream-K): the units of a launch are (tile, term)
// pairs numbered job by job, tile by tile, term by term.  With G persistent
// workgroups, the first F = floor(T / G) G tiles run whole, G at a time, all
// workgroups walking the terms in the same order (so the operators they read are
// shared in L2); within a round the tiles of one XCD are contiguous in space.
// The R units of the remaining tiles are split evenly over G_t = min(G, R)
// workgroups: workgroup g < G_t takes [S + B_g, S + B_{g+1}) with
// B_g = floor(g R / G_t) and S the first remaining unit.  A tile split between
// workgroups is stored in pieces (slot 2g for the first remaining tile of g,
// 2g + 1 for its last) that k_gemm_fixup adds in workgroup order, so results do
// not depend on timing.
__device__ inline int64_t sk_bound(int64_t g, int64_t units, int G) { return g * units / G; }

__device__ inline int find_job_units(const GemmJob *__restrict__ jobs, int njobs, int64_t u) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].units_start <= u)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__device__ inline int find_job_tiles(const GemmJob *__restrict__ jobs, int njobs, int tile) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].tiles_start <= tile)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Source metadata of one target column of a gathered-GEMM tile.
struct ColState {
  const int *slot_map;  // slot map of the source level
  const void *B;        // source expansions
  uint32_t tkey;        // target key
  int tsl, r;           // target slot, right-hand side
  int valid;
};

// terms [term0, term1) of one tile; writes the result (part == nullptr) or a piece.
// A (the operators) is shared by the 4 waves and staged through LDS; each wave
// multiplies its own 32 columns, so B (the gathered source expansions) goes
// straight from memory to registers: within each 16-k chunk lane l supplies
// k = 4 (l / 16) + ks at k-step ks, four consecutive elements of its column, and
// the operator tables use the same k order (setup.cpp).
template <int MODE, int RBT>
__device__ inline void gemm_tile(const GemmJob &J, int tile_local, int term0, int term1,
                                 double *__restrict__ part, double (*As)[RBT * 4 * 64],
                                 ColState *cst) {
  constexpr int CPW = gemm_cpw(RBT), COLS = 64 * CPW;
  constexpr int NA = RBT * 128;         // A chunk, in pairs
  constexpr int QA = (NA + 255) / 256;  // pairs per thread
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rowtile = tile_local % J.nrowtiles, coltile = tile_local / J.nrowtiles;
  const int rb0 = rowtile * RBT, col0 = coltile * COLS;
  const int nrb = J.dpm >> 4, nks = J.dpk >> 2, nkc = J.dpk >> 4;
  const int ncols = J.ntgt * J.nrhs;
  const int koff = 4 * (lane >> 4);

  // the CPW columns of this lane (one per 16-column block of the wave); their
  // source metadata waits in LDS (this thread's own slots) until each term
  // starts, which keeps it out of the registers the accumulators need
  ColState *my = cst + CPW * t;
#pragma unroll
  for (int jj = 0; jj < CPW; ++jj) {
    const int jc = col0 + 16 * (CPW * w + jj) + (lane & 15);
    ColState c{};
    c.valid = jc < ncols;
    c.slot_map = J.src_slot;
    c.B = J.Bsrc;
    if (c.valid) {
      const int tt = jc / J.nrhs;
      c.r = jc - tt * J.nrhs;
      c.tsl = J.tgt ? ldg(J.tgt + tt) : tt;
      if (MODE != MODE_PROJ) c.tkey = ldg(J.tgt_keys + c.tsl);
    }
    my[jj] = c;
  }
  d4v acc[RBT][CPW];
  bool rowok[RBT];
#pragma unroll
  for (int i = 0; i < RBT; ++i) {
    rowok[i] = rb0 + i < nrb;
#pragma unroll
    for (int jj = 0; jj < CPW; ++jj) acc[i][jj] = d4v{0, 0, 0, 0};
  }
  // Chunks are loaded two ahead of their products: during the products of
  // chunk it, the loads of chunk it + 2 are in flight and chunk it + 1 goes from
  // registers into the LDS buffer that chunk it - 1 used.  The barriers order
  // LDS accesses only, so loads stay in flight across them.  Three register sets
  // (R, B) rotate by name over a loop unrolled by 3 (a copy from a register a
  // load is filling would wait for that load), and every chunk issues the same
  // loads, so that the waits for them are exact.
  d2v R0[QA], R1[QA], R2[QA];               // A of a chunk, on its way to LDS
  d2v B0[CPW][2], B1[CPW][2], B2[CPW][2];   // B of a chunk: [column][pair]
  const double *srcp[CPW];
  const double *Ap = nullptr;
  // source slots of the next term (-1: none): read by the fetch of a term's
  // last chunk (the other fetches read g_slot_none), used at the next term's
  // first chunk
  int nslot[CPW];
#pragma unroll
  for (int jj = 0; jj < CPW; ++jj) {
    srcp[jj] = nullptr;
    nslot[jj] = -1;
  }
  auto lookup = [&](int term, bool real) {
#pragma unroll
    for (int jj = 0; jj < CPW; ++jj) {
      const ColState c = my[jj];
      if constexpr (MODE == MODE_PROJ) {
        nslot[jj] = c.valid ? c.tsl : -1;
      } else {
        const int *addr = &g_slot_none[jj];
        if (real) addr = gemm_source_addr<MODE>(term, c.valid, c.tkey, c.slot_map, jj);
        nslot[jj] = ldg(addr);
      }
    }
  };
  // loads chunk (fterm, fkc), the next one in order, into raD and bD; with live
  // false (past the last chunk) the same loads read zeros
  int fterm = term0, fkc = 0;
  const double *zero = g_gemm_zero;
  auto fetch = [&](d2v(&raD)[QA], d2v(&bD)[CPW][2], bool live) {
    const int term = fterm, kc = fkc;
    if (live) {
      if (++fkc == nkc) {
        fkc = 0;
        ++fterm;
      }
      if (kc == 0) {
#pragma unroll
        for (int jj = 0; jj < CPW; ++jj) {
          const ColState c = my[jj];
          srcp[jj] = gemm_source_ptr(J, nslot[jj], c.r, (const double *)c.B);
        }
        Ap = gemm_operand<MODE>(J, term);
      }
    }
    // the slots of the next term, at the term's last chunk
    lookup(term + 1, live && kc == nkc - 1 && term + 1 < term1);
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int e = t + 256 * q;  // pair index in the chunk
      const int rb = rb0 + (e >> 7);
      if (e < NA) {
        const double *src = (live && rb < nrb) ? Ap + ((int64_t)rb * nks + kc * 4) * 64 : zero;
        raD[q] = ldg((const d2v *)(src + 2 * (e & 127)));
      }
    }
#pragma unroll
    for (int jj = 0; jj < CPW; ++jj) {
      const double *col = (live && srcp[jj]) ? srcp[jj] + kc * 16 : zero;
      const d2v *s2 = (const d2v *)(col + koff);
      bD[jj][0] = ldg(s2);
      bD[jj][1] = ldg(s2 + 1);
    }
  };
  auto stash = [&](int buf, const d2v(&raS)[QA]) {
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int e = t + 256 * q;
      if (e < NA) *(d2v *)(&As[buf][2 * e]) = raS[q];
    }
  };
  const int it0 = term0 * nkc, it1 = term1 * nkc;
  // the products of chunk it (its A in LDS buffer (it - it0) & 1, its B in Bc),
  // with the loads of chunk it + 2 into (Rf, Bf) and chunk it + 1 (Rn) stashed
  // The products of a chunk's last k-step are deferred to the start of the next
  // step, after the barrier, so that their MFMAs run while the wave issues the
  // next chunk's loads; their operands wait in registers.
  double a3[RBT], b3[CPW];
  bool dpend = false;  // deferred products pending (wave-uniform)
  auto deferred = [&]() {
    if (dpend) {
#pragma unroll
      for (int i = 0; i < RBT; ++i)
        if (RBT != 6 || rowok[i]) {
#pragma unroll
          for (int jj = 0; jj < CPW; ++jj) acc[i][jj] = mfma_f64(a3[i], b3[jj], acc[i][jj]);
        }
    }
    dpend = false;
  };
  // k-steps 0..2 of one chunk, and the operands of k-step 3
  auto products = [&](int cur, const d2v(&Bc)[CPW][2]) {
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      double a[RBT], b[CPW];
#pragma unroll
      for (int i = 0; i < RBT; ++i) a[i] = As[cur][(i * 4 + ks) * 64 + lane];
#pragma unroll
      for (int jj = 0; jj < CPW; ++jj) b[jj] = (ks & 1) ? Bc[jj][ks >> 1].y : Bc[jj][ks >> 1].x;
      // every row block is multiplied (except with 6 blocks): the A chunk holds
      // zeros beyond the operator's rows (their results are not stored), and a
      // branch per block would split the products into pieces that each wait for
      // their LDS reads.  With 6 blocks the unbranched form runs out of registers.
#pragma unroll
      for (int i = 0; i < RBT; ++i)
        if (RBT != 6 || rowok[i]) {
#pragma unroll
          for (int jj = 0; jj < CPW; ++jj) acc[i][jj] = mfma_f64(a[i], b[jj], acc[i][jj]);
        }
    }
#pragma unroll
    for (int i = 0; i < RBT; ++i) a3[i] = As[cur][(i * 4 + 3) * 64 + lane];
#pragma unroll
    for (int jj = 0; jj < CPW; ++jj) b3[jj] = Bc[jj][1].y;
  };
  auto step = [&](int it, const d2v(&Bc)[CPW][2], const d2v(&Rn)[QA], d2v(&Rf)[QA],
                  d2v(&Bf)[CPW][2]) {
    const int cur = (it - it0) & 1;
    deferred();  // the previous chunk's last k-step
    fetch(Rf, Bf, it + 2 < it1);
    stash(cur ^ 1, Rn);
    products(cur, Bc);
    dpend = true;
    lds_barrier();
  };

  if (it0 < it1) {
    lookup(term0, true);
    fetch(R0, B0, true);
    stash(0, R0);
    fetch(R1, B1, it0 + 1 < it1);
    lds_barrier();
    int it = it0;
    for (; it + 3 <= it1; it += 3) {
      step(it, B0, R1, R2, B2);
      step(it + 1, B1, R2, R0, B0);
      step(it + 2, B2, R0, R1, B1);
    }
    if (it < it1) step(it, B0, R1, R2, B2);
    if (it + 1 < it1) step(it + 1, B1, R2, R0, B0);
    deferred();
  }

#pragma unroll
  for (int jj = 0; jj < CPW; ++jj) {
    const int jt = 16 * (CPW * w + jj) + (lane & 15);
    const int jo = col0 + jt;
    if (jo >= ncols) continue;
    const int tt = jo / J.nrhs, ro = jo - tt * J.nrhs;
    const int tso = J.tgt ? ldg(J.tgt + tt) : tt;
    const int64_t cbase = ((int64_t)tso * J.nrhs + ro) * J.dpm;
#pragma unroll
    for (int i = 0; i < RBT; ++i) {
      if (!rowok[i]) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int rt = 16 * i + (lane >> 4) + 4 * q;
        double v = acc[i][jj][q];
        if (part) {
          stg(part + (size_t)rt * COLS + jt, v);
        } else {
          const int64_t o = cbase + 16 * rb0 + rt;
          if constexpr (MODE == MODE_L2L) v += ldg(J.Cadd + o);
          stg(J.C + o, v);
          if (J.C32) stg(J.C32 + o, (float)v);
        }
      }
    }
  }
}

template <int MODE, int RBT>
__global__ __launch_bounds__(256, 2) void k_gemm(const GemmJob *__restrict__ jobs, int njobs,
                                                 int ntiles, int64_t units, int G, int GT,
                                                 double *__restrict__ ws) {
  constexpr int TILE = RBT * 16 * 64 * gemm_cpw(RBT);
  __shared__ double As[2][RBT * 4 * 64];
  __shared__ ColState cst[2 * 256];
  const int g = blockIdx.x;
  // whole tiles, G at a time; the tiles of one XCD (g mod 8) are contiguous
  const int full = (ntiles / G) * G;
  const int per = G / 8;
  const int gx = (G % 8 == 0) ? (g % 8) * per + g / 8 : g;
  for (int t0 = 0; t0 < full; t0 += G) {
    const int tile = t0 + gx;
    const GemmJob J = jobs[find_job_tiles(jobs, njobs, tile)];
    gemm_tile<MODE, RBT>(J, tile - J.tiles_start, 0, J.nterms, nullptr, As, cst);
  }
  if (full == ntiles) return;
  // the remaining units, split evenly
  const GemmJob Jr = jobs[find_job_tiles(jobs, njobs, full)];
  const int64_t S = Jr.units_start + (int64_t)(full - Jr.tiles_start) * Jr.nterms;
  const int64_t R = units - S;
  // workgroups sharing the tail (at most GT, so that the 2 GT pieces fit the
  // workspace): each owns >= 1 unit
  const int Gt = (int)min((int64_t)GT, R);
  if (g >= Gt) return;
  const int64_t ua = S + sk_bound(g, R, Gt), ub = S + sk_bound(g + 1, R, Gt);
  for (int64_t u = ua; u < ub;) {
    const GemmJob J = jobs[find_job_units(jobs, njobs, u)];
    const int64_t local = u - J.units_start;
    const int tile_local = (int)(local / J.nterms);
    const int term0 = (int)(local - (int64_t)tile_local * J.nterms);
    const int64_t ts = J.units_start + (int64_t)tile_local * J.nterms;
    const int term1 = (int)(min(ts + J.nterms, ub) - ts);
    u = ts + term1;
    const bool whole = term0 == 0 && term1 == J.nterms;
    double *part = whole ? nullptr : ws + (size_t)(2 * g + (ua >= ts ? 0 : 1)) * TILE;
    gemm_tile<MODE, RBT>(J, tile_local, term0, term1, part, As, cst);
  }
}

// Adds the pieces of the tiles split between workgroups; kFixupSplit blocks per
// tile, each adding a slice of its elements.  The workgroups meeting a tile are
// consecutive, glo..ghi: glo's piece is in slot 2 glo + 1 unless glo starts at
// the tile (then 2 glo), the others start inside it (slot 2 g).  The pieces are
// added in workgroup order, 8 loads in flight at a time.
constexpr int kFixupSplit = 4;
template <int RBT>
__global__ __launch_bounds__(256) void k_gemm_fixup(const GemmJob *__restrict__ jobs, int njobs,
                                                    int ntiles, int64_t units, int G, int GT,
                                                    const double *__restrict__ ws) {
  constexpr int COLS = 64 * gemm_cpw(RBT), TILE = RBT * 16 * COLS;
  constexpr int SLICE = TILE / kFixupSplit;
  static_assert(SLICE % 256 == 0 && 256 % COLS == 0, "fixup slices");
  const int full = (ntiles / G) * G;
  const int tile = full + (int)(blockIdx.x / kFixupSplit);
  const int slice = (int)(blockIdx.x % kFixupSplit);
  if (tile >= ntiles) return;
  const GemmJob J = jobs[find_job_tiles(jobs, njobs, tile)];
  const int tile_local = tile - J.tiles_start;
  const GemmJob Jr = jobs[find_job_tiles(jobs, njobs, full)];
  const int64_t S = Jr.units_start + (int64_t)(full - Jr.tiles_start) * Jr.nterms;
  const int64_t R = units - S;
  const int Gt = (int)min((int64_t)GT, R);
  // unit range of the tile relative to S; workgroup g starts at unit
  // sk_bound(g) = floor(g R / Gt), so the last one starting at or before ts is
  // floor(((ts + 1) Gt - 1) / R) and the last one starting before te is
  // floor((te Gt - 1) / R)
  const int64_t ts = J.units_start + (int64_t)tile_local * J.nterms - S, te = ts + J.nterms;
  const int64_t glo = min(((ts + 1) * Gt - 1) / R, (int64_t)Gt - 1);
  const int64_t ghi = min((te * Gt - 1) / R, (int64_t)Gt - 1);
  if (ghi == glo) return;  // written directly
  const int np = (int)(ghi - glo + 1);
  const int first = (int)(2 * glo + (sk_bound(glo, R, Gt) == ts ? 0 : 1));
  // slot of piece i: glo's piece, then the first slot of each later workgroup
  auto slot_of = [&](int i) { return i == 0 ? first : (int)(2 * (glo + i)); };
  const int rowtile = tile_local % J.nrowtiles, coltile = tile_local / J.nrowtiles;
  const int rb0 = rowtile * RBT, col0 = coltile * COLS;
  const int nrows = min(RBT * 16, J.dpm - 16 * rb0);
  const int ncols = J.ntgt * J.nrhs;
  // this thread's column (the same for all its elements, 256 being a multiple of COLS)
  const int jt = (int)threadIdx.x % COLS;
  const int jo = col0 + jt;
  if (jo >= ncols) return;
  const int tt = jo / J.nrhs, ro = jo - tt * J.nrhs;
  const int tso = J.tgt ? ldg(J.tgt + tt) : tt;
  const int64_t obase = ((int64_t)tso * J.nrhs + ro) * J.dpm + 16 * rb0;
  for (int e = slice * SLICE + (int)threadIdx.x; e < (slice + 1) * SLICE; e += 256) {
    const int rt = e / COLS;
    if (rt >= nrows) break;
    double v = 0.0;
    int i = 0;
    for (; i + 8 <= np; i += 8) {
      double p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = ldg(ws + (size_t)slot_of(i + u) * TILE + e);
#pragma unroll
      for (int u = 0; u < 8; ++u) v += p[u];
    }
    for (; i < np; ++i) v += ldg(ws + (size_t)slot_of(i) * TILE + e);
    const int64_t o = obase + rt;
    if (J.mode == MODE_L2L) v += ldg(J.Cadd + o);
    stg(J.C + o, v);
    if (J.C32) stg(J.C32 + o, (float)v);
  }
}

// The same products for launches too small to fill the chip with the tiles above (a tile
// walks 18 chunks of k with 24 products each at d = 287, and the upper levels have a few
// dozen of them): a wave takes 48 rows of 16 columns and one term, operators and columns
// straight to registers two chunks ahead, no barrier.  M2M: the 8 children of a parent by
// the 8 waves of a workgroup, summed in their order; else 4 waves of neighbouring items.  A
// term's products are in the order of the tiles, so L2L and PROJ give the same bits.
// Bound by the latency of its loads and, on the lower levels, the FP64 matrix cores.  10^5
// uniform points, depth 4, rank 128: L2L 33 -> 27 us and projections 25 -> 19 us a level,
// M2M (beside the near field) 54 with its fixup -> 51, the pass 850 -> 798 us; 2^20 points,
// depth 5: 4230 -> 4090 us.
constexpr int kFewRows = 3;  // row blocks of a wave
__host__ __device__ constexpr int few_waves(int mode) { return mode == MODE_M2M ? 8 : 4; }

template <int MODE>
__global__ __launch_bounds__(64 * few_waves(MODE), 2) void k_gemm_few(
    const GemmJob *__restrict__ jobs, int njobs) {
  constexpr int R = kFewRows;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = MODE == MODE_M2M ? (int)blockIdx.x : (int)blockIdx.x * 4 + w;
  // the job of the item: a lane per job, items column block by column block
  int nrg = 1, count = 0;
  if (lane < njobs) {
    const GemmJob &Q = jobs[lane];
    nrg = (ldg(&Q.dpm) / 16 + R - 1) / R;
    count = nrg * ((ldg(&Q.ntgt) * ldg(&Q.nrhs) + 15) / 16);
  }
  int end = count;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(end, o);
    if (lane >= o) end += v;
  }
  const unsigned long long after = __ballot(end > item);
  if (after == 0) return;  // (M2M: the whole workgroup)
  const int j = __builtin_ctzll(after);
  const int local = __builtin_amdgcn_readfirstlane(__shfl(item - (end - count), j));
  nrg = __builtin_amdgcn_readfirstlane(__shfl(nrg, j));
  const GemmJob J = jobs[j];
  const int rb0 = local % nrg * R, col0 = local / nrg * 16;
  const int nrb = J.dpm >> 4, nks = J.dpk >> 2, nkc = J.dpk >> 4;
  const int term = MODE == MODE_M2M ? w : 0;
  // this lane's column
  const int jc = col0 + (lane & 15);
  const bool valid = jc < J.ntgt * J.nrhs;
  int tsl = 0, r = 0, slot = -1;
  if (valid) {
    const int tt = jc / J.nrhs;
    r = jc - tt * J.nrhs;
    tsl = J.tgt ? ldg(J.tgt + tt) : tt;
    if constexpr (MODE == MODE_PROJ)
      slot = tsl;
    else
      slot = ldg(gemm_source_addr<MODE>(term, true, ldg(J.tgt_keys + tsl), J.src_slot, 0));
  }
  const double *col = gemm_source_ptr(J, slot, r, (const double *)J.Bsrc);
  const bool some = col != nullptr;
  col = (some ? col : g_gemm_zero) + 4 * (lane >> 4);
  const double *A[R];
#pragma unroll
  for (int i = 0; i < R; ++i)
    A[i] = gemm_operand<MODE>(J, term) + (int64_t)min(rb0 + i, nrb - 1) * nks * 64 + lane;
  d4v acc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) acc[i] = d4v{0, 0, 0, 0};
  struct Set {
    double a[R][4];
    d2v b[2];
  } S0, S1, S2;
  auto load = [&](Set &S, int kc) {
    kc = min(kc, nkc - 1);
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) S.a[i][ks] = ldg(A[i] + (4 * kc + ks) * 64);
    S.b[0] = ldg((const d2v *)(col + 16 * kc));
    S.b[1] = ldg((const d2v *)(col + 16 * kc + 2));
  };
  auto products = [&](const Set &S) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < R; ++i) acc[i] = mfma_f64(S.a[i][ks], S.b[ks >> 1][ks & 1], acc[i]);
  };
  if (__ballot(some) != 0) {
    load(S0, 0);
    load(S1, 1);
    for (int kc = 0; kc < nkc; kc += 3) {
      load(S2, kc + 2);
      products(S0);
      if (kc + 1 >= nkc) break;
      load(S0, kc + 3);
      products(S1);
      if (kc + 2 >= nkc) break;
      load(S1, kc + 4);
      products(S2);
    }
  }
  int i0 = 0, i1 = R;  // row blocks that this wave stores
  if constexpr (MODE == MODE_M2M) {
    __shared__ double part[8][R * 256];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[w][(4 * i + q) * 64 + lane] = acc[i][q];
    __syncthreads();
    if (w >= R) return;
    i0 = w;
    i1 = w + 1;
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) v += part[u][(4 * w + q) * 64 + lane];
        acc[i][q] = v;
      }
  }
  if (!valid) return;
  const int64_t cbase = ((int64_t)tsl * J.nrhs + r) * J.dpm + (lane >> 4);
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (i < i0 || i >= i1 || rb0 + i >= nrb) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t o = cbase + 16 * (rb0 + i) + 4 * q;
      double v = acc[i][q];
      if constexpr (MODE == MODE_L2L) v += ldg(J.Cadd + o);
      stg(J.C + o, v);
      if (J.C32) stg(J.C32 + o, (float)v);
    }
  }
}

// L2L and the projections of many columns: a workgroup of 4 waves computes 16 RB rows (5 to
// 9 blocks) of 64 columns, each wave every row of its 16.  The operator passes through LDS
// in 16-k chunks, loaded straight to it one chunk ahead in two buffers, the source columns
// a chunk ahead in registers; with 4 RB products of 64 cycles a chunk, two workgroups per CU
// cover the loads.  The products of a result are in the order of the tiles above: same bits.
// Bound by the FP64 matrix cores, at 64 right-hand sides half by memory too (the columns in,
// the added l and the result out).  2^20 points, d = 287, rank 144: L2L 9.8 -> 8.3 ms and the
// projections 10.4 -> 9.3 at 64 right-hand sides; at one, L2L of the leaf level 180 -> 164 us,
// projections 171 -> 153.
template <int MODE, int RB>
__global__ __launch_bounds__(256, 2) void k_gemm_tall(const GemmJob *__restrict__ jobs, int njobs) {
  static_assert(MODE != MODE_M2M, "one term");
  __shared__ __align__(16) double As[2][RB * 256];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the tile: a lane per job counts its tiles, those of one XCD (workgroup mod 8) contiguous
  int nrg = 1, count = 0;
  if (lane < njobs) {
    const GemmJob &Q = jobs[lane];
    nrg = (ldg(&Q.dpm) / 16 + RB - 1) / RB;
    count = nrg * ((ldg(&Q.ntgt) * ldg(&Q.nrhs) + 63) / 64);
  }
  int end = count;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(end, o);
    if (lane >= o) end += v;
  }
  const int total = __builtin_amdgcn_readfirstlane(__shfl(end, 63));
  const int x = blockIdx.x % 8, xi = blockIdx.x / 8;
  if (xi >= total / 8 + (x < total % 8 ? 1 : 0)) return;
  const int tile = x * (total / 8) + min(x, total % 8) + xi;
  const int j = __builtin_ctzll(__ballot(end > tile));
  const int local = __builtin_amdgcn_readfirstlane(__shfl(tile - (end - count), j));
  nrg = __builtin_amdgcn_readfirstlane(__shfl(nrg, j));
  const GemmJob J = jobs[j];
  const int rb0 = local % nrg * RB, col0 = local / nrg * 64;
  const int nrb = J.dpm >> 4, nkc = J.dpk >> 4, nv = min(RB, nrb - rb0);
  // this lane's column
  const int jc = col0 + 16 * w + (lane & 15);
  const bool valid = jc < J.ntgt * J.nrhs;
  int tsl = 0, r = 0, slot = -1;
  if (valid) {
    const int tt = jc / J.nrhs;
    r = jc - tt * J.nrhs;
    tsl = J.tgt ? ldg(J.tgt + tt) : tt;
    if constexpr (MODE == MODE_PROJ)
      slot = tsl;
    else
      slot = ldg(gemm_source_addr<MODE>(0, true, ldg(J.tgt_keys + tsl), J.src_slot, 0));
  }
  const double *col = gemm_source_ptr(J, slot, r, (const double *)J.Bsrc);
  col = (col ? col : g_gemm_zero) + 4 * (lane >> 4);
  const char *Abase = (const char *)(gemm_operand<MODE>(J, 0) + (int64_t)rb0 * nkc * 256);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) double *)&As[0][0];
  const uint32_t lane16 = 16u * (uint32_t)lane;
  auto load_a = [&](int buf, int kc) {  // a row block's 2 KB per wave and turn
#pragma unroll
    for (int i = 0; i < (RB + 3) / 4; ++i) {
      const int blk = w + 4 * i;
      if (blk >= nv) continue;
      const uint64_t src = uniform64((uint64_t)(Abase + ((int64_t)blk * nkc + kc) * 2048));
      const uint32_t dst =
          __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(buf * (RB * 2048) + blk * 2048));
      fragment_to_lds<0>(src, dst, lane16);
      fragment_to_lds<1024>(src, dst, lane16);
    }
  };
  d4v acc[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) acc[i] = d4v{0, 0, 0, 0};
  auto step = [&](int kc, const d2v(&B)[2], d2v(&Bn)[2]) {
    // what this wave issued in the last step has arrived, after the barrier the others'
    // too, and nobody reads the buffer that the next loads overwrite
    __builtin_amdgcn_s_waitcnt(0x0f70);
    lds_barrier();
    if (kc + 1 < nkc) {
      load_a((kc + 1) & 1, kc + 1);
      Bn[0] = ldg((const d2v *)(col + 16 * (kc + 1)));
      Bn[1] = ldg((const d2v *)(col + 16 * (kc + 1) + 2));
    }
    const double *Ap = &As[kc & 1][lane];
    double a[2][RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) a[0][i] = Ap[i * 256];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks < 3) {
#pragma unroll
        for (int i = 0; i < RB; ++i) a[(ks + 1) & 1][i] = Ap[i * 256 + (ks + 1) * 64];
      }
#pragma unroll
      for (int i = 0; i < RB; ++i) acc[i] = mfma_f64(a[ks & 1][i], B[ks >> 1][ks & 1], acc[i]);
    }
  };
  d2v B0[2], B1[2];
  load_a(0, 0);
  B0[0] = B1[0] = ldg((const d2v *)col);
  B0[1] = B1[1] = ldg((const d2v *)(col + 2));
  for (int kc = 0; kc < nkc; kc += 2) {
    step(kc, B0, B1);
    if (kc + 1 < nkc) step(kc + 1, B1, B0);
  }
  if (!valid) return;
  const int64_t cbase = ((int64_t)tsl * J.nrhs + r) * J.dpm + 16 * rb0 + (lane >> 4);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    if (i >= nv) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t o = cbase + 16 * i + 4 * q;
      double v = acc[i][q];
      if constexpr (MODE == MODE_L2L) v += ldg(J.Cadd + o);
      stg(J.C + o, v);
      if (J.C32) stg(J.C32 + o, (float)v);
    }
  }
}

// ------------------------------------------------------------------ factored M2L
// Second compression stage (Sec. 4.2): per offset o the r x r matrix C^delta is
// the product Ut_o Vt_o of an r x s_o and an s_o x r factor, so a column's
// contribution is Ut_o (Vt_o w), w the What' column of its source.  A work item is
// (64-column tile, range of terms); each of the 4 waves owns 16 columns and all
// rp rows of g'.  Per term a wave forms t = Vt_o w (s_o x 16) on FP64 MFMA, with
// w loaded straight from memory in the gathered GEMM's k order, then
// g' += Ut_o t, feeding t from its result registers as the B operand: result
// register q of lane l holds row (l / 16) + 4 q, the k order of the Ut fragments.
// Factor fragments are read from memory; the tiles of a class walk the same terms
// in the same order, so they stay in L1 / L2.
constexpr int kM2l2Sb = kMaxRank2 / 16;  // most 16-row blocks of t

template <int RB>
__global__ __launch_bounds__(256, 2) void k_m2l2(const M2l2Job *__restrict__ jobs, int njobs,
                                                 int nitems, const int8_t *__restrict__ dvec,
                                                 double *__restrict__ ws) {
  typedef double v4 __attribute__((ext_vector_type(4)));
  constexpr int rp = 16 * RB;
  const int item = blockIdx.x;
  if (item >= nitems) return;
  const int ji = find_last_le(njobs, item, [&](int m) { return (int64_t)jobs[m].item_start; });
  const M2l2Job J = jobs[ji];
  const int local = item - J.item_start;
  const int tile = local / kM2l2Parts, part = local - tile * kM2l2Parts;
  const int term0 = 189 * part / kM2l2Parts, term1 = 189 * (part + 1) / kM2l2Parts;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = tile * 64 + 16 * w + (lane & 15);
  const bool cv = col < J.ntgt * J.nrhs;
  const int tt = cv ? col / J.nrhs : 0;
  const int rr = cv ? col - tt * J.nrhs : 0;
  const int tsl = cv ? J.tgt[tt] : 0;
  const uint32_t tkey = cv ? J.keys[tsl] : 0u;
  const int side = 1 << J.level;
  const int c0 = (int)morton_axis(tkey, 0), c1 = (int)morton_axis(tkey, 1),
            c2 = (int)morton_axis(tkey, 2);
  const int g4 = 4 * (lane >> 4);
  v4 acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb] = v4{0, 0, 0, 0};
  for (int term = term0; term < term1; ++term) {
    const int o = J.terms[term];
    const int sp = J.sp[o];
    if (sp == 0) continue;
    const int nsb = sp >> 4;
    int sl = -1;
    if (cv) {
      const int m0 = c0 + dvec[3 * o], m1 = c1 + dvec[3 * o + 1], m2 = c2 + dvec[3 * o + 2];
      if (m0 >= 0 && m1 >= 0 && m2 >= 0 && m0 < side && m1 < side && m2 < side)
        sl = J.slot[morton_encode((uint32_t)m0, (uint32_t)m1, (uint32_t)m2)];
    }
    const double *src = sl >= 0 ? J.B + ((int64_t)sl * J.nrhs + rr) * rp : nullptr;
    const double *V = J.vf + J.voff[o] + lane;
    const double *U = J.uf + J.uoff[o] + lane;
    v4 t[kM2l2Sb];
#pragma unroll
    for (int sb = 0; sb < kM2l2Sb; ++sb) t[sb] = v4{0, 0, 0, 0};
    // t = Vt_o w
#pragma unroll
    for (int kc = 0; kc < RB; ++kc) {
      double b[4] = {0, 0, 0, 0};
      if (src) {
        const double2 *s2 = (const double2 *)(src + kc * 16 + g4);
        const double2 x = s2[0], y = s2[1];
        b[0] = x.x;
        b[1] = x.y;
        b[2] = y.x;
        b[3] = y.y;
      }
#pragma unroll
      for (int sb = 0; sb < kM2l2Sb; ++sb)
        if (sb < nsb) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            t[sb] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                V[((int64_t)sb * (rp / 4) + kc * 4 + q) * 64], b[q], t[sb], 0, 0, 0);
        }
    }
    // g' += Ut_o t
#pragma unroll
    for (int sb = 0; sb < kM2l2Sb; ++sb)
      if (sb < nsb) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            acc[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                U[((int64_t)rb * (sp / 4) + sb * 4 + q) * 64], t[sb][q], acc[rb], 0, 0, 0);
      }
  }
  // partial block of the item, column-major: ws[item][column][row]
  double *out = ws + (size_t)item * rp * 64 + (size_t)(16 * w + (lane & 15)) * rp;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[16 * rb + (lane >> 4) + 4 * q] = acc[rb][q];
}

// g' of each tile: the kM2l2Parts partial blocks added in part order
__global__ __launch_bounds__(256) void k_m2l2_sum(const M2l2Job *__restrict__ jobs, int njobs,
                                                  int ntiles, const double *__restrict__ ws) {
  const int tg = blockIdx.x;
  if (tg >= ntiles) return;
  const int ji = find_last_le(njobs, tg, [&](int m) { return (int64_t)jobs[m].tile_start; });
  const M2l2Job J = jobs[ji];
  const int tile = tg - J.tile_start, rp = J.rp;
  const int ncols = J.ntgt * J.nrhs;
  const size_t blk = (size_t)rp * 64;
  const double *base = ws + (size_t)(J.item_start + tile * kM2l2Parts) * blk;
  for (int e = threadIdx.x; e < rp * 64; e += 256) {
    const int jc = e / rp, row = e - jc * rp;
    const int col = tile * 64 + jc;
    if (col >= ncols) continue;
    double v = 0.0;
#pragma unroll
    for (int p = 0; p < kM2l2Parts; ++p) v += base[p * blk + e];
    const int tt = col / J.nrhs, r = col - tt * J.nrhs;
    J.C[((int64_t)J.tgt[tt] * J.nrhs + r) * rp + row] = v;
  }
}

template <int RB>
void launch_m2l2_rb(const M2l2Job *jobs, const M2l2Launch &L, const int8_t *dvec, double *ws,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_m2l2<RB>, dim3(L.nitems), dim3(256), 0, s, jobs + L.first_job, L.njobs,
                     L.nitems, dvec, ws + L.ws_off);
  hipLaunchKernelGGL(k_m2l2_sum, dim3(L.ntiles), dim3(256), 0, s, jobs + L.first_job, L.njobs,
                     L.ntiles, ws + L.ws_off);
}

void launch_m2l2(const M2l2Job *jobs, const M2l2Launch &L, const int8_t *dvec, double *ws,
                 hipStream_t s) {
  if (L.nitems == 0) return;
  switch (L.rb) {
    case 4: launch_m2l2_rb<4>(jobs, L, dvec, ws, s); break;
    case 5: launch_m2l2_rb<5>(jobs, L, dvec, ws, s); break;
    case 6: launch_m2l2_rb<6>(jobs, L, dvec, ws, s); break;
    case 7: launch_m2l2_rb<7>(jobs, L, dvec, ws, s); break;
    case 8: launch_m2l2_rb<8>(jobs, L, dvec, ws, s); break;
    case 9: launch_m2l2_rb<9>(jobs, L, dvec, ws, s); break;
    case 10: launch_m2l2_rb<10>(jobs, L, dvec, ws, s); break;
    case 11: launch_m2l2_rb<11>(jobs, L, dvec, ws, s); break;
    case 12: launch_m2l2_rb<12>(jobs, L, dvec, ws, s); break;
    case 13: launch_m2l2_rb<13>(jobs, L, dvec, ws, s); break;
    case 14: launch_m2l2_rb<14>(jobs, L, dvec, ws, s); break;
    case 15: launch_m2l2_rb<15>(jobs, L, dvec, ws, s); break;
    default: launch_m2l2_rb<16>(jobs, L, dvec, ws, s); break;
  }
}

// ------------------------------------------------------------------ host side
namespace {

// Per-phase HIP events; elapsed times are collected by timing_drain.
struct Timer {
  Plan &P;
  hipStream_t s;
  EventPair ep;
  bool on;
  Timer(Plan &P_, hipStream_t s_, int ph)
      : P(P_), s(s_), on(P_.timing == 1 || (P_.timing == 2 && ph == EIFMM_PH_M2L)) {
    if (!on) return;
    if (P.ev_pending.size() > 4096) timing_drain(P);
    if (P.ev_free.empty()) {
      EventPair e;
      hipEventCreate(&e.a);
      hipEventCreate(&e.b);
      P.ev_free.push_back(e);
    }
    ep = P.ev_free.back();
    P.ev_free.pop_back();
    ep.phase = ph;
    hipEventRecord(ep.a, s);
  }
  ~Timer() {
    if (!on) return;
    hipEventRecord(ep.b, s);
    P.ev_pending.push_back(ep);
  }
};

int tiles_of(const GemmJob &J) { return J.ncoltiles * J.nrowtiles; }

// cols: columns of a tile (0: the gathered GEMM's for the height rbt)
void finish_job(GemmJob &J, int &tiles, int rbt, int cols = 0) {
  const int ncols = J.ntgt * J.nrhs;
  if (cols == 0) cols = gemm_cols(rbt);
  J.ncoltiles = (ncols + cols - 1) / cols;
  J.nrowtiles = (J.dpm / 16 + rbt - 1) / rbt;
  J.tiles_start = tiles;
  tiles += tiles_of(J);
}

// unit offsets (tile x term) of the jobs of one launch group
int64_t finish_units(std::vector<GemmJob> &h, int first) {
  int64_t u = 0;
  for (size_t j = first; j < h.size(); ++j) {
    h[j].units_start = u;
    u += (int64_t)tiles_of(h[j]) * h[j].nterms;
  }
  return u;
}

}  // namespace

// Job tables of a (points, nrhs) pair, uploaded once and reused.
int build_jobs(Plan &P, int nrhs, hipStream_t s) {
  const int depth = P.depth;
  const bool mixed = P.cfg.precision == EIFMM_PREC_MIXED;
  std::vector<GemmJob> h;
  auto &jt = P.jobs;
  jt = JobTables{};
  // M2M, one job per parent level k = depth-1 .. 2
  for (int k = depth - 1; k >= 2; --k) {
    int tiles = 0;
    GemmJob J{};
    J.A = P.ld[k].m2m;
    J.Bsrc = P.ld[k + 1].W;
    J.C = P.ld[k].W;
    J.tgt = nullptr;
    J.tgt_keys = P.ld[k].act;
    J.src_slot = P.ld[k + 1].slot;
    J.a_stride = (int64_t)P.lh[k].dp * P.lh[k + 1].dp;
    J.ntgt = (int)P.nact[k];
    J.nterms = 8;
    J.dpm = P.lh[k].dp;
    J.dpk = P.lh[k + 1].dp;
    J.level = k;
    J.mode = MODE_M2M;
    J.nrhs = nrhs;
    jt.m2m_rbt[k] = pick_rbt(J.dpm / 16);
    finish_job(J, tiles, jt.m2m_rbt[k]);
    jt.m2m_first[k] = (int)h.size();
    jt.m2m_n[k] = 1;
    jt.m2m_tiles[k] = tiles;
    h.push_back(J);
    jt.m2m_units[k] = finish_units(h, jt.m2m_first[k]);
  }
  // compression projections What' = U^T B^{-T} z with z = Gamma^{-1} W from the
  // forward solve, one job per compressed level (What' = (U^T B^{-T} Gamma^{-1}) W
  // from W itself where the operator folds the solve in)
  {
    int tiles = 0;
    jt.pre_first = (int)h.size();
    jt.pre_rbt = pick_rbt(P.lh[depth].rp / 16 > 0 ? P.lh[depth].rp / 16 : 1);
    double pf = 0;
    for (int k = depth; k >= 2; --k) {
      if (P.lh[k].r == 0 || P.nact[k] == 0) continue;
      GemmJob J{};
      J.A = P.ld[k].pfrag;
      J.Bsrc = P.lh[k].fold_what ? P.ld[k].W : P.ld[k].Wh;
      J.C = P.ld[k].Whp;
      J.C32 = mixed ? P.ld[k].Whp32 : nullptr;
      J.ntgt = (int)P.nact[k];
      J.nterms = 1;
      J.dpm = P.lh[k].rp;
      J.dpk = P.lh[k].dp;
      J.level = k;
      J.mode = MODE_PROJ;
      J.nrhs = nrhs;
      finish_job(J, tiles, jt.pre_rbt);
      h.push_back(J);
      pf += 2.0 * (P.lh[k].d + P.lh[k].dB) * (double)P.lh[k].r * (double)P.nact[k] * nrhs;
    }
    jt.pre_n = (int)h.size() - jt.pre_first;
    jt.pre_tiles = tiles;
    jt.pre_units = finish_units(h, jt.pre_first);
    P.proj_flops = pf;
  }
  // M2L, every level in one launch, finest level first
  {
    int tiles = 0;
    jt.m2l_first = (int)h.size();
    int kf = depth;  // the tile height serves the finest level of this launch
    while (kf > 2 && (P.ld[kf].ksmall || P.ld[kf].nd == kDigitsSteep)) --kf;
    int ks = depth;  // (the same of the steep levels)
    while (ks > 2 && P.ld[ks].nd != kDigitsSteep) --ks;
    auto row_blocks = [&](int k) { return (P.lh[k].r ? P.lh[k].rp : P.lh[k].dpB) / 16; };
    jt.m2l_rbt = mixed ? pick_m2l32(row_blocks(kf)) : pick_m2l8(row_blocks(kf), kDigits);
    jt.steep_rbt = pick_m2l8(row_blocks(ks), kDigitsSteep);
    // levels of small operators and steep levels: launches of their own
    std::vector<GemmJob> small_jobs, steep_jobs;
    int small_tiles = 0, steep_tiles = 0;
    for (int k = depth; k >= 2; --k) {
      if (uses_m2l2(P, k)) continue;  // the factored M2L below
      if (m2l_by_offset(P, k, nrhs)) continue;
      const bool small = P.ld[k].ksmall != nullptr;
      const bool cz = P.lh[k].r > 0;
      // rows: g (the second EIM's size); columns: What
      // (FP64: whole 64-element chunks)
      const int dm = cz ? P.lh[k].rp : P.lh[k].dpB;
      const int dc = cz ? P.lh[k].rp : P.lh[k].dp;
      const int dk = mixed || small ? dc : digit_kp(dc);
      for (int c = 0; c < 8; ++c) {
        const int64_t nt = P.cls_off[k][c + 1] - P.cls_off[k][c];
        if (nt == 0) continue;
        GemmJob J{};
        if (mixed) {
          J.A = P.ld[k].kfrag32;
          J.Bsrc = cz ? P.ld[k].Whp32 : P.ld[k].Wh32;
          J.a_stride = (int64_t)dm * dk * sizeof(float);
        } else if (small) {
          J.A = P.ld[k].ksmall;
          J.Bsrc = cz ? P.ld[k].Whp : P.ld[k].Wh;
          J.ksteps = m2l_small_steps(cz ? P.lh[k].r : P.lh[k].d);
        } else {
          J.A = P.ld[k].k8;
          J.Bsrc = P.ld[k].w8;
          J.bscale = P.ld[k].wscale;
          J.kexp = P.ld[k].kexp;
          J.a_stride = (int64_t)dm * dk * P.ld[k].nd;
        }
        J.C = cz ? P.ld[k].gp : P.ld[k].g;
        J.tgt = (P.ld[k].ord ? P.ld[k].ord : P.ld[k].cls) + P.cls_off[k][c];
        J.tgt_keys = P.ld[k].act;
        J.src_slot = P.ld[k].slot;
        J.terms = P.dlist + 189 * c;
        J.ntgt = (int)nt;
        J.nterms = 189;
        J.dpm = dm;
        J.dpk = dk;
        J.level = k;
        J.cls = c;
        J.mode = MODE_M2L;
        J.nrhs = nrhs;
        if (small) {
          finish_job(J, small_tiles, kSmallM2l / 16, kSmallM2lCols);
          small_jobs.push_back(J);
          continue;
        }
        if (P.ld[k].nd == kDigitsSteep) {
          finish_job(J, steep_tiles, jt.steep_rbt, m2l8_cols(jt.steep_rbt));
          steep_jobs.push_back(J);
          continue;
        }
        finish_job(J, tiles, jt.m2l_rbt, mixed ? kM2l32Cols : m2l8_cols(jt.m2l_rbt));
        h.push_back(J);
      }
    }
    jt.m2l_n = (int)h.size() - jt.m2l_first;
    jt.m2l_tiles = tiles;
    // executed work: every column walks all terms of its class, over whole row
    // tiles of the padded operators
    double fx = 0;
    for (int j = jt.m2l_first; j < jt.m2l_first + jt.m2l_n; ++j)
      fx += 2.0 * (double)h[j].nrowtiles * 16 * jt.m2l_rbt * h[j].dpk * (double)h[j].ntgt *
            h[j].nrhs * h[j].nterms;
    jt.steep_first = (int)h.size();
    jt.steep_n = (int)steep_jobs.size();
    jt.steep_tiles = steep_tiles;
    for (const GemmJob &J : steep_jobs) {
      fx += 2.0 * (double)J.nrowtiles * 16 * jt.steep_rbt * J.dpk * (double)J.ntgt * J.nrhs * J.nterms;
      h.push_back(J);
    }
    jt.small_first = (int)h.size();
    jt.small_n = (int)small_jobs.size();
    jt.small_grid = 0;
    for (const GemmJob &J : small_jobs) {
      jt.small_grid += (J.ncoltiles + 7) / 8 * 8;
      fx += 2.0 * (double)J.dpm * 4 * J.ksteps * (double)J.ntgt * J.nrhs * J.nterms;
      h.push_back(J);
    }
    if (depth >= 2 && m2l_by_offset(P, 2, nrhs) && P.nact[2] > 0) {
      // whole 16-column blocks of the (4 - |dx|) (4 - |dy|) (4 - |dz|) targets of an offset
      const LevelHost &H = P.lh[2];
      double cols = 0;
      for (int x = -3; x <= 3; ++x)
        for (int y = -3; y <= 3; ++y)
          for (int z = -3; z <= 3; ++z)
            if (std::max({std::abs(x), std::abs(y), std::abs(z)}) > 1)
              cols += ((4 - std::abs(x)) * (4 - std::abs(y)) * (4 - std::abs(z)) + 15) / 16 * 16;
      fx += 2.0 * cols * (H.r ? H.rp : H.dpB) * (H.r ? H.rp : H.dp);
    }
    P.m2l_flops_exec = fx;
    // factored M2L levels: one job per child class, grouped by rp; algorithmic
    // flops 2 (r s_o + s_o r) per interaction pair, with the mean s_o over the
    // 316 offsets standing in for the offsets the pairs actually use
    auto &mj = P.m2l2_host;
    auto &ml = P.m2l2_launch;
    mj.clear();
    ml.clear();
    int item = 0, tilec = 0;
    for (int rb = kM2l2RbMin; rb <= kM2l2RbMax; ++rb) {
      M2l2Launch L{(int)mj.size(), 0, item, 0, tilec, 0, rb};
      for (int k = depth; k >= 2; --k) {
        if (!uses_m2l2(P, k) || P.lh[k].rp != 16 * rb) continue;
        for (int c = 0; c < 8; ++c) {
          const int64_t nt = P.cls_off[k][c + 1] - P.cls_off[k][c];
          if (nt == 0) continue;
          M2l2Job J{};
          J.tgt = P.ld[k].cls + P.cls_off[k][c];
          J.keys = P.ld[k].act;
          J.slot = P.ld[k].slot;
          J.B = P.ld[k].Whp;
          J.C = P.ld[k].gp;
          J.terms = P.dlist + 189 * c;
          J.vf = P.ld[k].vf2;
          J.uf = P.ld[k].uf2;
          J.voff = P.ld[k].voff2;
          J.uoff = P.ld[k].uoff2;
          J.sp = P.ld[k].sp2;
          J.ntgt = (int)nt;
          J.nrhs = nrhs;
          J.level = k;
          J.rp = P.lh[k].rp;
          J.ntiles = (int)((nt * nrhs + 63) / 64);
          J.tile_start = tilec - L.first_tile;
          J.item_start = item - L.first_item;
          tilec += J.ntiles;
          item += J.ntiles * kM2l2Parts;
          mj.push_back(J);
        }
      }
      L.njobs = (int)mj.size() - L.first_job;
      L.nitems = item - L.first_item;
      L.ntiles = tilec - L.first_tile;
      if (L.njobs) ml.push_back(L);
    }
    P.m2l_flops = m2l_flops_of(P, nrhs);
  }
  // g = U g' on compressed levels
  {
    int tiles = 0;
    jt.post_first = (int)h.size();
    jt.post_rbt = pick_rbt(P.lh[depth].dpB / 16);
    for (int k = depth; k >= 2; --k) {
      if (P.lh[k].r == 0 || P.nact[k] == 0) continue;
      GemmJob J{};
      J.A = P.ld[k].ufrag;
      J.Bsrc = P.ld[k].gp;
      J.C = P.ld[k].g;
      J.ntgt = (int)P.nact[k];
      J.nterms = 1;
      J.dpm = P.lh[k].dpB;
      J.dpk = P.lh[k].rp;
      J.level = k;
      J.mode = MODE_PROJ;
      J.nrhs = nrhs;
      finish_job(J, tiles, jt.post_rbt);
      h.push_back(J);
    }
    jt.post_n = (int)h.size() - jt.post_first;
    jt.post_tiles = tiles;
    jt.post_units = finish_units(h, jt.post_first);
  }
  // L2L, per child level k = 3 .. depth, one job per child class
  for (int k = 3; k <= depth; ++k) {
    int tiles = 0;
    jt.l2l_first[k] = (int)h.size();
    for (int c = 0; c < 8; ++c) {
      const int64_t nt = P.cls_off[k][c + 1] - P.cls_off[k][c];
      if (nt == 0) continue;
      GemmJob J{};
      J.A = P.ld[k - 1].l2l;
      J.Bsrc = P.ld[k - 1].l;
      J.C = P.ld[k].l;
      J.Cadd = P.ld[k].g;
      J.tgt = P.ld[k].cls + P.cls_off[k][c];
      J.tgt_keys = P.ld[k].act;
      J.src_slot = P.ld[k - 1].slot;
      J.a_stride = (int64_t)P.lh[k].dpB * P.lh[k - 1].dpB;
      J.ntgt = (int)nt;
      J.nterms = 1;
      J.dpm = P.lh[k].dpB;
      J.dpk = P.lh[k - 1].dpB;
      J.level = k;
      J.cls = c;
      J.mode = MODE_L2L;
      J.nrhs = nrhs;
      jt.l2l_rbt[k] = pick_rbt(J.dpm / 16);
      finish_job(J, tiles, jt.l2l_rbt[k]);
      h.push_back(J);
    }
    jt.l2l_n[k] = (int)h.size() - jt.l2l_first[k];
    jt.l2l_tiles[k] = tiles;
    jt.l2l_units[k] = finish_units(h, jt.l2l_first[k]);
  }
  P.jobs_host = h;
  if (!h.empty()) {
    // the table goes to the device from pinned memory, asynchronously on the
    // stream of the evaluation; buffers grow only when the job count does
    if (h.size() > P.job_cap) {
      if (P.job_evt) hipEventSynchronize(P.job_evt);
      if (P.job_dev) hipFree(P.job_dev);
      if (P.job_pin) hipHostFree(P.job_pin);
      P.job_dev = nullptr;
      P.job_pin = nullptr;
      P.job_cap = 0;
      const size_t cap = h.size() + h.size() / 2 + 16;
      if (hipMalloc(&P.job_dev, sizeof(GemmJob) * cap) != hipSuccess ||
          hipHostMalloc((void **)&P.job_pin, sizeof(GemmJob) * cap) != hipSuccess) {
        hipGetLastError();
        return EIFMM_ENOMEM;
      }
      P.job_cap = cap;
      if (!P.job_evt && hipEventCreateWithFlags(&P.job_evt, hipEventDisableTiming) != hipSuccess)
        return EIFMM_EHIP;
    }
    if (hipEventSynchronize(P.job_evt) != hipSuccess) return EIFMM_EHIP;
    std::memcpy(P.job_pin, h.data(), sizeof(GemmJob) * h.size());
    if (hipMemcpyAsync(P.job_dev, P.job_pin, sizeof(GemmJob) * h.size(), hipMemcpyHostToDevice,
                       s) != hipSuccess ||
        hipEventRecord(P.job_evt, s) != hipSuccess)
      return EIFMM_EHIP;
  }
  if (!P.m2l2_host.empty()) {
    // factored M2L jobs: the same pinned, asynchronous upload; the workspace
    // holds one rp x 64 block per work item, launch after launch
    const size_t nj = P.m2l2_host.size();
    size_t need = 0;
    for (auto &L : P.m2l2_launch) {
      L.ws_off = need;
      need += (size_t)L.nitems * 16 * L.rb * 64;
    }
    if (P.job_evt) hipEventSynchronize(P.job_evt);
    if (nj > P.m2l2_cap) {
      if (P.m2l2_dev) hipFree(P.m2l2_dev);
      if (P.m2l2_pin) hipHostFree(P.m2l2_pin);
      P.m2l2_dev = nullptr;
      P.m2l2_pin = nullptr;
      P.m2l2_cap = 0;
      const size_t cap = nj + nj / 2 + 8;
      if (hipMalloc(&P.m2l2_dev, sizeof(M2l2Job) * cap) != hipSuccess ||
          hipHostMalloc((void **)&P.m2l2_pin, sizeof(M2l2Job) * cap) != hipSuccess) {
        hipGetLastError();
        return EIFMM_ENOMEM;
      }
      P.m2l2_cap = cap;
    }
    if (need > P.m2l2_ws_cap) {
      if (P.m2l2_ws) hipFree(P.m2l2_ws);
      P.m2l2_ws = nullptr;
      P.m2l2_ws_cap = 0;
      if (hipMalloc(&P.m2l2_ws, sizeof(double) * need) != hipSuccess) {
        hipGetLastError();
        return EIFMM_ENOMEM;
      }
      P.m2l2_ws_cap = need;
    }
    if (!P.job_evt && hipEventCreateWithFlags(&P.job_evt, hipEventDisableTiming) != hipSuccess)
      return EIFMM_EHIP;
    std::memcpy(P.m2l2_pin, P.m2l2_host.data(), sizeof(M2l2Job) * nj);
    if (hipMemcpyAsync(P.m2l2_dev, P.m2l2_pin, sizeof(M2l2Job) * nj, hipMemcpyHostToDevice, s) !=
            hipSuccess ||
        hipEventRecord(P.job_evt, s) != hipSuccess)
      return EIFMM_EHIP;
  }
  jt.nrhs = nrhs;
  return EIFMM_OK;
}

namespace {

// ws holds ws_len doubles: the pieces of the Stream-K tail, TILE doubles each, 2
// per tail workgroup, so the tail is split over at most ws_len / (2 TILE)
// workgroups (G itself for the plan's own workspace, fewer for a smaller one)
template <int MODE, int RBT>
void launch_gemm_rbt(const GemmJob *jobs, int n, int tiles, int64_t units, int gmax,
                     double *ws, size_t ws_len, hipStream_t s) {
  const size_t TILE = (size_t)RBT * 16 * gemm_cols(RBT);
  const size_t len = ws_len - kCounterDoubles;  // pieces
  const int G = (int)std::min<int64_t>(units, gmax);
  const int GT = (int)std::min<size_t>((size_t)G, len / (2 * TILE));
  const int rest = tiles - (tiles / G) * G;
  hipLaunchKernelGGL((k_gemm<MODE, RBT>), dim3(G), dim3(256), 0, s, jobs, n, tiles, units, G, GT,
                     ws);
  if (G > 1 && rest > 0)
    hipLaunchKernelGGL((k_gemm_fixup<RBT>), dim3(rest * kFixupSplit), dim3(256), 0, s, jobs, n,
                       tiles, units, G, GT, ws);
}

template <int MODE, int RB>
void launch_tall(const GemmJob *jobs, int n, int grid, hipStream_t s) {
  hipLaunchKernelGGL((k_gemm_tall<MODE, RB>), dim3(grid), dim3(256), 0, s, jobs, n);
}
// row blocks of a tall tile: the fewest idle ones, the taller on a tie
int pick_tall(int nrb) {
  int best = 9;
  for (int h = 8; h >= 5; --h)
    if ((nrb + h - 1) / h * h < (nrb + best - 1) / best * best) best = h;
  return best;
}

// few: the launch may take the form for few columns (k_gemm_few).  It does when the tiles
// leave compute units idle: fewer (tile, term) pairs than workgroups.
// nrb: row blocks of the finest level's operators; more than 4 take the tall tiles (L2L and
// the projections; below that a tile of 3 or 4 blocks and 128 columns is as good).
template <int MODE>
void launch_gemm_tab(const GemmJob *jobs, int n, int tiles, int64_t units, int rbt, int gmax,
                     double *ws, size_t ws_len, bool few, int nrb, hipStream_t s) {
  if (n == 0 || tiles == 0 || units == 0) return;
  if (few && n <= 64 && units < gmax) {
    // at most this many items (a job's last tiles may hold fewer; the rest return)
    const int items = tiles * ((rbt + kFewRows - 1) / kFewRows) * (gemm_cols(rbt) / 16);
    const int waves = few_waves(MODE), grid = MODE == MODE_M2M ? items : (items + 3) / 4;
    hipLaunchKernelGGL(k_gemm_few<MODE>, dim3(grid), dim3(64 * waves), 0, s, jobs, n);
    return;
  }
  if constexpr (MODE != MODE_M2M) {
    if (n <= 64 && nrb > 4) {
      // at most this many 64-column tiles (the row tiles are no fewer at rbt <= 6 blocks
      // than at 6 and more; at 5 at most twice as few): the rest return
      const int cols = tiles * (gemm_cols(rbt) / 64);
      switch (pick_tall(nrb)) {
        case 9: launch_tall<MODE, 9>(jobs, n, cols, s); break;
        case 8: launch_tall<MODE, 8>(jobs, n, cols, s); break;
        case 7: launch_tall<MODE, 7>(jobs, n, cols, s); break;
        case 6: launch_tall<MODE, 6>(jobs, n, cols, s); break;
        default: launch_tall<MODE, 5>(jobs, n, 2 * cols, s); break;
      }
      return;
    }
  }
  switch (rbt) {
    case 4: launch_gemm_rbt<MODE, 4>(jobs, n, tiles, units, gmax, ws, ws_len, s); break;
    case 3: launch_gemm_rbt<MODE, 3>(jobs, n, tiles, units, gmax, ws, ws_len, s); break;
    case 5: launch_gemm_rbt<MODE, 5>(jobs, n, tiles, units, gmax, ws, ws_len, s); break;
    default: launch_gemm_rbt<MODE, 6>(jobs, n, tiles, units, gmax, ws, ws_len, s); break;
  }
}

// a plan's launch: its Stream-K workspace, or the one its caller lends for this
// pass (P.run_ws, P.run_ws_len)
template <int MODE>
void launch_gemm(Plan &P, int first, int n, int tiles, int64_t units, hipStream_t s,
                 int rbt, int nrb) {
  double *ws = P.run_ws ? P.run_ws : P.sk_ws;
  const size_t len = P.run_ws ? P.run_ws_len : stream_k_ws_len(P.sk_groups);
  // (mixed precision rounds the solved expansions to FP32, which would show an M2M sum in
  // another order, no better or worse: its results stay what they were)
  const bool few = MODE != MODE_M2M || P.cfg.precision == EIFMM_PREC_FP64;
  launch_gemm_tab<MODE>(P.job_dev + first, n, tiles, units, rbt, P.sk_groups, ws, len, few, nrb, s);
}

void launch_gemm_fused(const FusedGemm &F, int mode, bool fp32, int gmax, double *ws,
                       const int8_t *dvec, hipStream_t s) {
  const size_t len = stream_k_ws_len(gmax);
  switch (mode) {
    case MODE_M2M:
      launch_gemm_tab<MODE_M2M>(F.dev, F.n, F.tiles, F.units, F.rbt, gmax, ws, len, false, 0, s);
      break;
    case MODE_L2L:
      launch_gemm_tab<MODE_L2L>(F.dev, F.n, F.tiles, F.units, F.rbt, gmax, ws, len, true, 0, s);
      break;
    case MODE_PROJ:
      launch_gemm_tab<MODE_PROJ>(F.dev, F.n, F.tiles, F.units, F.rbt, gmax, ws, len, true, 0, s);
      break;
    default:
      if (fp32)
        launch_m2l32(F.dev, F.n, F.tiles, F.rbt, F.dk, gmax / 2, ws, len, dvec, s);
      else
        launch_m2l8(F.dev, F.n, F.tiles, F.rbt, F.nd, gmax / 2, ws, len, dvec, s);
  }
}

// ---- leaf-level launches (one plan: BATCH = false; a batch group: BATCH = true)
// workgroups of a chunk launch: one per 32-target chunk
unsigned chunk_grid(int64_t nchunk) { return (unsigned)nchunk; }

template <int KIND, bool BATCH>
void launch_p2p(bool mixed, int nrhs, int64_t nchunk, const LeafDesc &one, const LeafDesc *many,
                int nmany, hipStream_t s) {
  const unsigned grid = chunk_grid(nchunk);
  if (grid == 0) return;
  if (mixed) {
    if (nrhs == 1)
      hipLaunchKernelGGL((k_p2p32<KIND, 1, BATCH>), dim3(grid), dim3(64), 0, s, one, many, nmany);
    else
      hipLaunchKernelGGL((k_p2p32<KIND, 8, BATCH>), dim3(grid), dim3(64), 0, s, one, many, nmany);
  } else {
    if (nrhs == 1)
      hipLaunchKernelGGL((k_p2p64<KIND, 1, BATCH>), dim3(grid), dim3(64), 0, s, one, many, nmany);
    else
      hipLaunchKernelGGL((k_p2p64<KIND, 8, BATCH>), dim3(grid), dim3(64), 0, s, one, many, nmany);
  }
}

// crowded: the leaves hold more than 64 points on average, so that a workgroup
// spends its time in the batch loop (1e6 clustered points at depth 5: P2M 2.95
// -> 2.66 ms); on leaves of a few dozen points the 256-thread form is faster
// (1e6 uniform points at depth 5: 0.21 against 0.25 ms)
template <int KIND, bool BATCH, bool LIB>
void launch_p2m_exp(int nrhs, unsigned grid, int dpmax, const LeafDesc &one, const LeafDesc *many,
                int nmany, hipStream_t s, bool crowded) {
  if (grid == 0) return;
  if (dpmax <= 64) {  // one row per thread: a 64-lane workgroup wastes no lanes on small d
    if (nrhs == 1)
      hipLaunchKernelGGL((k_p2m<KIND, 1, BATCH, 64, LIB>), dim3(grid), dim3(64), 0, s, one, many,
                         nmany);
    else
      hipLaunchKernelGGL((k_p2m<KIND, 8, BATCH, 64, LIB>), dim3(grid), dim3(64), 0, s, one, many,
                         nmany);
  } else {
    if (nrhs == 1 && crowded) {
      const int nt = std::min(1024, (dpmax + 63) / 64 * 64);
      hipLaunchKernelGGL((k_p2m<KIND, 1, BATCH, 0, LIB>), dim3(grid), dim3(nt), 0, s, one, many,
                         nmany);
    } else if (nrhs == 1) {
      hipLaunchKernelGGL((k_p2m<KIND, 1, BATCH, 256, LIB>), dim3(grid), dim3(256), 0, s, one, many,
                         nmany);
    } else {
      hipLaunchKernelGGL((k_p2m<KIND, 8, BATCH, 256, LIB>), dim3(grid), dim3(256), 0, s, one, many,
                         nmany);
    }
  }
}
// lib_exp: P2M by the library's exponential (what_rounded)
template <int KIND, bool BATCH>
void launch_p2m(int nrhs, unsigned grid, int dpmax, const LeafDesc &one, const LeafDesc *many,
                int nmany, hipStream_t s, bool lib_exp, bool crowded = false) {
  if constexpr (KF<KIND>::exponential) {
    if (lib_exp) {
      launch_p2m_exp<KIND, BATCH, true>(nrhs, grid, dpmax, one, many, nmany, s, crowded);
      return;
    }
  }
  launch_p2m_exp<KIND, BATCH, false>(nrhs, grid, dpmax, one, many, nmany, s, crowded);
}

size_t l2p_shm(int nrhs, int dpmax) {
  const int rb = nrhs == 1 ? 1 : 8;
  return sizeof(double) * (3 * (size_t)dpmax + (size_t)rb * dpmax);
}

template <int KIND, bool BATCH>
void launch_l2p(int nrhs, int64_t nchunk, int dpmax, const LeafDesc &one, const IoDesc &ione,
                const LeafDesc *many, const IoDesc *io, int nmany, hipStream_t s) {
  const unsigned grid = chunk_grid(nchunk);
  if (grid == 0) return;
  const size_t shm = l2p_shm(nrhs, dpmax);
  if (nrhs == 1)
    hipLaunchKernelGGL((k_l2p<KIND, 1, BATCH>), dim3(grid), dim3(64), shm, s, one, ione, many, io,
                       nmany);
  else
    hipLaunchKernelGGL((k_l2p<KIND, 8, BATCH>), dim3(grid), dim3(64), shm, s, one, ione, many, io,
                       nmany);
}

LeafDesc leaf_desc(const Plan &P, int nrhs) {
  const int depth = P.depth;
  LeafDesc D{};
  D.act = P.ld[depth].act;
  D.ls = P.leaf_start;
  // targets = sources: every point of a leaf is both; otherwise each leaf holds
  // its sources, then its targets
  D.se = P.nt ? P.tgt_begin : P.leaf_start + 1;
  D.tb = P.nt ? P.tgt_begin : P.leaf_start;
  D.chunk_ptr = P.chunk_ptr;
  D.chunk_leaf = P.chunk_leaf;
  D.seg_ptr = P.seg_ptr;
  D.seg_leaf = P.seg_leaf;
  D.w_ext = P.w_ext;
  D.seg_len = seg_len(P);
  D.perm = P.idx;
  D.xyz = P.xyz;
  D.X = P.ld[depth].X;
  D.XL = P.ld[depth].XL;
  D.lhat = P.lhat;
  D.sig = P.sig;
  D.fnear = P.fnear;
  D.W = P.ld[depth].W;
  D.n = P.n;
  D.nsrc = P.nt ? P.ns : P.n;
  D.toff = P.nt ? P.ns : 0;
  D.nleaf = (int)P.nact[depth];
  D.nrhs = nrhs;
  D.depth = depth;
  D.d = depth >= 2 ? P.lh[depth].d : 0;
  D.dp = depth >= 2 ? P.lh[depth].dp : 0;
  D.dL = depth >= 2 ? P.lh[depth].dB : 0;
  D.dpL = depth >= 2 ? P.lh[depth].dpB : 0;
  D.lo0 = P.cfg.lo[0];
  D.lo1 = P.cfg.lo[1];
  D.lo2 = P.cfg.lo[2];
  D.h = std::ldexp(P.cfg.L, -depth);
  D.p = dev_param(P.cfg.kernel, P.cfg.kernel_param);
  return D;
}

// level k's M2L sources (What' on a compressed level, What otherwise) as digits
DigitDesc digit_desc(const Plan &P, int k, int nrhs, int blk_start) {
  const bool cz = P.lh[k].r > 0;
  DigitDesc D{};
  D.in = cz ? P.ld[k].Whp : P.ld[k].Wh;
  D.out = P.ld[k].w8;
  D.scale = P.ld[k].wscale;
  D.ncols = (int)(P.nact[k] * nrhs);
  D.ld = cz ? P.lh[k].rp : P.lh[k].dp;
  D.kp = digit_kp(D.ld);
  D.nd = P.ld[k].nd;
  D.blk_start = blk_start;
  return D;
}

template <int KIND>
void run_kind(Plan &P, int nrhs, const IoDesc &io, hipStream_t s) {
  const int depth = P.depth;
  const bool mixed = P.cfg.precision == EIFMM_PREC_MIXED;
  const int64_t n = P.n;
  const int nleafa = (int)P.nact[depth];
  const int64_t nchunk = P.nchunk;
  const LeafDesc LD = leaf_desc(P, nrhs);
  LevelDev &LL = P.ld[depth];
  // near field: with a far field to compute it runs on the plan's second stream
  // and L2P waits for it. In FP64 it starts after P2M, so that it overlaps M2M,
  // the solves and the projections (small MFMA launches that leave the vector
  // units idle); the FP64 M2L's workgroups hold up to 256 registers per lane at two
  // waves per SIMD and 148 KB of LDS, which leaves no registers for near-field waves
  // beside them. In mixed precision
  // it starts just before M2L: the FP32 M2L and FP32 near-field waves fit on a
  // SIMD together, and the near field then fills the M2L's ramp-down as well.
  // With many right-hand sides the near field is long enough to take CUs from
  // the M2L's persistent workgroups when it is dispatched first (the order of
  // the two streams' first dispatches is not fixed), so it starts after P2M.
  const bool fork = depth >= 2 && nleafa > 0 && P.side;
  const bool fork_late = fork && mixed && nrhs == 1;
  P.near_mode = fork_late ? 2 : fork ? 1 : 0;
  auto near_field = [&](hipStream_t sn) {
    if (sn != s) {
      hipEventRecord(P.ev_fork, s);
      hipStreamWaitEvent(sn, P.ev_fork, 0);
    }
    {
      Timer tm(P, sn, EIFMM_PH_P2P);
      launch_p2p<KIND, false>(mixed, nrhs, nchunk, LD, nullptr, 0, sn);
    }
    if (sn != s) hipEventRecord(P.ev_join, sn);
  };
  if (nleafa > 0 && !fork) near_field(s);
  if (depth < 2) {
    const int64_t m = n * nrhs;
    if (m > 0)
      hipLaunchKernelGGL(k_combine_near, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, n,
                         nrhs, P.fnear, P.idx, LD.toff, io.f, io.ldf);
    return;
  }
  const LevelHost &HL = P.lh[depth];
  // step 1: P2M
  if (nleafa > 0) {
    Timer tm(P, s, EIFMM_PH_P2M);
    launch_p2m<KIND, false>(nrhs, (unsigned)(nrhs == 1 ? P.nseg : nleafa), HL.dp, LD, nullptr, 0, s,
                            what_rounded(P), n > 64 * (int64_t)nleafa);
    if (nrhs == 1 && P.nseg > nleafa)
      hipLaunchKernelGGL((k_p2m_ext<false>), dim3((unsigned)P.nseg), dim3(256), 0, s, LD, nullptr,
                         0);
  }
  if (fork && !fork_late) near_field(P.side);
  // step 2: M2M
  {
    Timer tm(P, s, EIFMM_PH_M2M);
    for (int k = depth - 1; k >= 2; --k)
      launch_gemm<MODE_M2M>(P, P.jobs.m2m_first[k], P.jobs.m2m_n[k], P.jobs.m2m_tiles[k],
                                    P.jobs.m2m_units[k], s, P.jobs.m2m_rbt[k], 0);
  }
  // step 3: What = Delta W = B^{-T} Gamma^{-1} W on uncompressed levels; on
  // compressed ones z = Gamma^{-1} W (the projection applies U^T B^{-T}), or
  // nothing where the projection's operator holds Gamma^{-1} too (fold_what)
  {
    Timer tm(P, s, EIFMM_PH_WHAT);
    SolveArgs A{};
    int blk = 0, q = 0;
    size_t shm = 0;
    for (int k = 2; k <= depth; ++k) {
      const int nc = (int)(P.nact[k] * nrhs);
      if (nc == 0 || !what_level(P, k)) continue;
      SolveDesc &D = A.lv[q++];
      D.in = P.ld[k].W;
      D.out = P.ld[k].Wh;
      D.out32 = (mixed && P.lh[k].r == 0) ? P.ld[k].Wh32 : nullptr;
      D.Tf = P.ld[k].tri[0];
      D.Tb = solves_what(P, k) ? P.ld[k].tri[1] : nullptr;
      D.ncols = nc;
      D.dp = P.lh[k].dp;
      D.blk_start = blk;
      blk += (nc + 15) / 16;
      shm = std::max(shm, trsm_shm(P.lh[k].dp));
    }
    A.nlev = q;
    if (blk > 0 && (mixed || blk > kSolveFew))
      hipLaunchKernelGGL(k_trsm, dim3(blk), dim3(64), shm, s, A);
    else if (blk > 0)
      hipLaunchKernelGGL(k_trsm4, dim3(blk), dim3(256), shm, s, A);
  }
  // step 4: M2L (with the compression projections around it when enabled)
  if (P.jobs.pre_n) {
    Timer tm(P, s, EIFMM_PH_PROJ);
    launch_gemm<MODE_PROJ>(P, P.jobs.pre_first, P.jobs.pre_n, P.jobs.pre_tiles,
                                   P.jobs.pre_units, s, P.jobs.pre_rbt, HL.rp / 16);
  }
  if (fork_late) hipEventRecord(P.ev_fork, s);
  {
    Timer tm(P, s, EIFMM_PH_M2L);
    double *ws = P.run_ws ? P.run_ws : P.sk_ws;
    const size_t ws_len = P.run_ws ? P.run_ws_len : stream_k_ws_len(P.sk_groups);
    const bool few = m2l_by_offset(P, 2, nrhs) && P.nact[2] > 0;
    if (mixed)
      launch_m2l32(P.job_dev + P.jobs.m2l_first, P.jobs.m2l_n, P.jobs.m2l_tiles, P.jobs.m2l_rbt,
                   HL.r > 0 ? HL.rp : HL.dp, P.sk_groups / 2, ws, ws_len, P.dvec, s);
    else if (P.jobs.m2l_n || P.jobs.steep_n || few) {
      DigitDesc dd[kMaxLevels];
      int nd = 0, blk = 0;
      for (int k = depth; k >= 2; --k) {
        if (P.nact[k] == 0 || uses_m2l2(P, k) || P.ld[k].ksmall) continue;
        dd[nd] = digit_desc(P, k, nrhs, blk);
        blk += digit_blocks(dd[nd++].ncols);
      }
      launch_digits(dd, nd, blk, s);
      launch_m2l8(P.job_dev + P.jobs.m2l_first, P.jobs.m2l_n, P.jobs.m2l_tiles, P.jobs.m2l_rbt,
                  kDigits, P.sk_groups / 2, ws, ws_len, P.dvec, s);
      launch_m2l8(P.job_dev + P.jobs.steep_first, P.jobs.steep_n, P.jobs.steep_tiles,
                  P.jobs.steep_rbt, kDigitsSteep, P.sk_groups / 2, ws, ws_len, P.dvec, s);
    }
    launch_m2l_small(P.job_dev + P.jobs.small_first, P.jobs.small_n, P.jobs.small_grid, P.dvec, s);
    if (few) {
      const LevelHost &H = P.lh[2];
      const LevelDev &L2 = P.ld[2];
      const bool cz = H.r > 0;
      const void *B = !mixed ? (const void *)L2.w8
                             : cz ? (const void *)L2.Whp32 : (const void *)L2.Wh32;
      launch_m2l_few(L2, mixed, B, cz ? H.rp : H.dpB, cz ? H.rp : H.dp, cz ? L2.gp : L2.g,
                     P.few_ws, P.dlist, P.dvec, s);
    }
    for (const M2l2Launch &L : P.m2l2_launch) launch_m2l2(P.m2l2_dev, L, P.dvec, P.m2l2_ws, s);
  }
  // launched after the M2L so that the M2L's workgroups are dispatched first
  if (fork_late) {
    hipStreamWaitEvent(P.side, P.ev_fork, 0);
    {
      Timer tm(P, P.side, EIFMM_PH_P2P);
      launch_p2p<KIND, false>(mixed, nrhs, nchunk, LD, nullptr, 0, P.side);
    }
    hipEventRecord(P.ev_join, P.side);
  }
  if (P.jobs.post_n) {
    Timer tm(P, s, EIFMM_PH_PROJ);
    launch_gemm<MODE_PROJ>(P, P.jobs.post_first, P.jobs.post_n, P.jobs.post_tiles,
                                   P.jobs.post_units, s, P.jobs.post_rbt, HL.dpB / 16);
  }
  // step 5: l^2 = g^2, then L2L downwards
  {
    Timer tm(P, s, EIFMM_PH_L2L);
    for (int k = 3; k <= depth; ++k)
      launch_gemm<MODE_L2L>(P, P.jobs.l2l_first[k], P.jobs.l2l_n[k], P.jobs.l2l_tiles[k],
                                    P.jobs.l2l_units[k], s, P.jobs.l2l_rbt[k], P.lh[k].dpB / 16);
  }
  // step 6: lhat = Delta^{J_0,I_0} l on the leaf level (Delta^T l with one EIM)
  {
    Timer tm(P, s, EIFMM_PH_LHAT);
    SolveArgs A{};
    const int nc = nleafa * nrhs;
    A.lv[0].in = LL.l;
    A.lv[0].out = P.lhat;
    A.lv[0].out32 = nullptr;
    A.lv[0].Tf = P.fold_leaf ? nullptr : LL.tri[2];  // B^{-1} folded into l (the Gamma^T solve only)
    A.lv[0].Tb = LL.tri[3];
    A.lv[0].ncols = nc;
    A.lv[0].dp = HL.dpB;
    A.lv[0].blk_start = 0;
    A.nlev = 1;
    if (nc > 16 * kSolveFew)
      hipLaunchKernelGGL(k_trsm, dim3((nc + 15) / 16), dim3(64), trsm_shm(HL.dpB), s, A);
    else if (nc > 0)
      hipLaunchKernelGGL(k_trsm4, dim3((nc + 15) / 16), dim3(256), trsm_shm(HL.dpB), s, A);
  }
  // step 7: L2P and the final sum (after the near field)
  if (fork) hipStreamWaitEvent(s, P.ev_join, 0);
  if (nleafa > 0) {
    Timer tm(P, s, EIFMM_PH_L2P);
    launch_l2p<KIND, false>(nrhs, nchunk, HL.dpB, LD, io, nullptr, nullptr, 0, s);
  }
}

}  // namespace

void timing_drain(Plan &P) {
  for (auto &e : P.ev_pending) {
    hipEventSynchronize(e.b);
    float ms = 0;
    hipEventElapsedTime(&ms, e.a, e.b);
    P.phase_ms[e.phase] += ms;
    P.phase_calls[e.phase] += 1;
    P.ev_free.push_back(e);
  }
  P.ev_pending.clear();
}

int pass_run(Plan &P, const double *sigma, int nrhs, int64_t ld, double *f, int64_t ldf,
             hipStream_t s) {
  if (P.jobs.nrhs != nrhs) {
    int st = build_jobs(P, nrhs, s);
    if (st != EIFMM_OK) return st;
  }
  const int64_t m = P.n * nrhs;
  const IoDesc io{sigma, ld, f, ldf};
  if (m > 0)
    hipLaunchKernelGGL((k_gather_sigma<false>), dim3((unsigned)((m + 255) / 256)), dim3(256), 0,
                       s, leaf_desc(P, nrhs), io, nullptr, nullptr, 0, m);
  switch (P.cfg.kernel) {
    case EIFMM_K_LAPLACE:
      run_kind<EIFMM_K_LAPLACE>(P, nrhs, io, s);
      break;
    case EIFMM_K_YUKAWA:
      run_kind<EIFMM_K_YUKAWA>(P, nrhs, io, s);
      break;
    case EIFMM_K_GAUSS:
      run_kind<EIFMM_K_GAUSS>(P, nrhs, io, s);
      break;
    case EIFMM_K_COSR:
      run_kind<EIFMM_K_COSR>(P, nrhs, io, s);
      break;
    case EIFMM_K_MQ:
      run_kind<EIFMM_K_MQ>(P, nrhs, io, s);
      break;
    case EIFMM_K_ADVDIFF:
      run_kind<EIFMM_K_ADVDIFF>(P, nrhs, io, s);
      break;
    default:
      run_kind<EIFMM_K_SQDIST>(P, nrhs, io, s);
      break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    P.last_hip_error = (int)e;
    return EIFMM_EHIP;
  }
  P.last_rhs = nrhs;
  return EIFMM_OK;
}

// 2 (rows x columns) per interaction pair on dense and stage-1 levels (the
// compressed sizes where compressed); 2 (r s + s r) with the factored M2L, s the
// mean second-stage rank over the 316 offsets standing in for the offsets the
// pairs actually use
double m2l_flops_of(const Plan &P, int nrhs) {
  double f = 0;
  for (int k = 2; k <= P.depth; ++k) {
    const LevelHost &L = P.lh[k];
    const double pairs = (double)P.il_pairs[k] * nrhs;
    if (uses_m2l2(P, k)) {
      double smean = 0;
      for (int o = 0; o < kNumOffsets; ++o) smean += L.s2[o];
      smean /= kNumOffsets;
      f += 4.0 * L.r * smean * pairs;
    } else {
      const bool cz = L.r > 0;
      const double rm = cz ? L.r : L.dB, rk = cz ? L.r : L.d;
      f += 2.0 * rm * rk * pairs;
    }
  }
  return f;
}

int materialize_expansion(Plan &P, int which, int k) {
  const int nrhs = P.jobs.nrhs;
  if (nrhs < 1 || k < 2 || k > P.depth || P.nact[k] == 0) return EIFMM_OK;
  hipStream_t s = nullptr;
  if (which == 1 && !solves_what(P, k)) {
    // What = Delta W, as the pass computes it on uncompressed levels
    SolveArgs A{};
    SolveDesc &D = A.lv[0];
    D.in = P.ld[k].W;
    D.out = P.ld[k].Wh;
    D.out32 = nullptr;
    D.Tf = P.ld[k].tri[0];
    D.Tb = P.ld[k].tri[1];
    D.ncols = (int)(P.nact[k] * nrhs);
    D.dp = P.lh[k].dp;
    D.blk_start = 0;
    A.nlev = 1;
    hipLaunchKernelGGL(k_trsm, dim3((D.ncols + 15) / 16), dim3(64), trsm_shm(D.dp), s, A);
  } else {
    return EIFMM_OK;
  }
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) {
    P.last_hip_error = (int)e;
    return EIFMM_EHIP;
  }
  return EIFMM_OK;
}

// M2M and L2L operators of parent level k (Sec. 4.1) by the blocked MFMA solves of
// the pass, one launch for both: the M2M rows K(X^k - s_i, Y^{k+1}) times
// M^{-1} of the child, i.e. M^{-T} applied to each row (B forward, Gamma^T
// backward); the L2L rows times the parent's Delta^T (one EIM: M^{-1} applied to
// each row, Gamma forward, B^T backward) or M_B^{-1} (two EIMs: M_B^{-T} applied,
// B_B forward, Gamma_B^T backward).  Rows are padded to the solve's dp with
// zeros, which the identity-padded tables keep at zero.
int solve_operators_gpu(Plan &P, int k) {
  LevelHost &lp = P.lh[k], &lc = P.lh[k + 1];
  const int n0 = 8 * lp.d, n1 = 8 * lc.dB;
  const int dp0 = lc.dp, dp1 = lp.dpB;
  const size_t sz0 = (size_t)n0 * dp0, sz1 = (size_t)n1 * dp1;
  if (lp.m2m_rows.size() != sz0 || lp.l2l_rows.size() != sz1) return EIFMM_EINVAL;
  double *rows = nullptr, *tabs[4] = {nullptr, nullptr, nullptr, nullptr};
  hipError_t e = hipMalloc(&rows, sizeof(double) * (sz0 + sz1 > 0 ? sz0 + sz1 : 1));
  if (e == hipSuccess && sz0) e = hipMemcpy(rows, lp.m2m_rows.data(), sizeof(double) * sz0, hipMemcpyHostToDevice);
  if (e == hipSuccess && sz1)
    e = hipMemcpy(rows + sz0, lp.l2l_rows.data(), sizeof(double) * sz1, hipMemcpyHostToDevice);
  const double *T[4];
  if (P.two_eim) {
    for (int q = 0; q < 4 && e == hipSuccess; ++q) {
      e = hipMalloc(&tabs[q], sizeof(double) * std::max<size_t>(lp.op_tri[q].size(), 1));
      if (e == hipSuccess && !lp.op_tri[q].empty())
        e = hipMemcpy(tabs[q], lp.op_tri[q].data(), sizeof(double) * lp.op_tri[q].size(),
                      hipMemcpyHostToDevice);
      T[q] = tabs[q];
    }
  } else {
    T[0] = P.ld[k + 1].tri[2];  // the child's Delta^T tables: B, Gamma^T
    T[1] = P.ld[k + 1].tri[3];
    T[2] = P.ld[k].tri[0];      // the parent's Delta tables: Gamma, B^T
    T[3] = P.ld[k].tri[1];
  }
  if (e == hipSuccess) {
    SolveArgs A{};
    A.lv[0] = SolveDesc{rows, rows, nullptr, T[0], T[1], n0, dp0, 0, 0};
    A.lv[1] = SolveDesc{rows + sz0, rows + sz0, nullptr, T[2], T[3], n1, dp1, (n0 + 15) / 16, 0};
    A.nlev = 2;
    const int blk = (n0 + 15) / 16 + (n1 + 15) / 16;
    // in place: a wave reads all tiles of its columns (forward pass) before it
    // writes any (backward pass)
    if (blk > 0) {
      hipLaunchKernelGGL(k_trsm, dim3(blk), dim3(64), trsm_shm(std::max(dp0, dp1)), nullptr, A);
      e = hipGetLastError();
    }
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess && sz0)
    e = hipMemcpy(lp.m2m_rows.data(), rows, sizeof(double) * sz0, hipMemcpyDeviceToHost);
  if (e == hipSuccess && sz1)
    e = hipMemcpy(lp.l2l_rows.data(), rows + sz0, sizeof(double) * sz1, hipMemcpyDeviceToHost);
  hipFree(rows);
  for (double *t : tabs) hipFree(t);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? EIFMM_ENOMEM : EIFMM_EHIP;
  }
  return EIFMM_OK;
}

// ------------------------------------------------------------------ batches
// A batch runs the pass of many independent problems (one plan each) as a fixed,
// short sequence of launches, each covering every problem: the leaf-level
// kernels once per kernel kind with an array of LeafDesc, the triangular solves
// once per step with a list of SolveDesc, and each gathered-GEMM step once with
// the concatenated jobs of all plans (re-tiled for the fused launch).  The
// sequence contains no host synchronisation and no allocation, so it can be
// captured once into a HIP graph and replayed.

namespace {

template <typename T>
int bupload(T **p, const std::vector<T> &v, std::vector<void *> &track) {
  *p = nullptr;
  if (v.empty()) return EIFMM_OK;
  if (hipMalloc((void **)p, sizeof(T) * v.size()) != hipSuccess) {
    hipGetLastError();
    return EIFMM_ENOMEM;
  }
  track.push_back((void *)*p);
  if (hipMemcpy(*p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice) != hipSuccess)
    return EIFMM_EHIP;
  return EIFMM_OK;
}

// concatenate the job ranges [first, first + n) of every plan into one launch
int fuse_jobs(FusedGemm &F, const std::vector<Plan *> &plans,
              const std::vector<std::pair<int, int>> &ranges, int rbt,
              std::vector<void *> &track) {
  std::vector<GemmJob> h;
  int dmax = 16;
  for (size_t q = 0; q < plans.size(); ++q)
    for (int j = ranges[q].first; j < ranges[q].first + ranges[q].second; ++j) {
      const GemmJob &J = plans[q]->jobs_host[j];
      if (J.ntgt == 0) continue;
      h.push_back(J);
      dmax = std::max(dmax, J.dpm);
    }
  F = FusedGemm{};
  F.rbt = rbt > 0 ? rbt : pick_rbt(dmax / 16);
  int tiles = 0;
  for (auto &J : h) finish_job(J, tiles, F.rbt);
  F.units = finish_units(h, 0);
  F.tiles = tiles;
  F.n = (int)h.size();
  return bupload(&F.dev, h, track);
}

// Packed M2L: one job per (operator set, level, child class) whose columns are
// the targets of that class in every problem using the set, so the coarse
// levels of small problems (a few boxes per class each) fill whole tiles.  kind: the
// levels to take (of a mixed batch all).
enum M2lKind { kM2lMixed, kM2lDigits, kM2lSteep, kM2lSmall };
M2lKind m2l_kind(const Plan &P, int k) {
  if (P.cfg.precision == EIFMM_PREC_MIXED) return kM2lMixed;
  return P.ld[k].ksmall ? kM2lSmall : P.ld[k].nd == kDigitsSteep ? kM2lSteep : kM2lDigits;
}
int pack_m2l(FusedGemm &F, const std::vector<Plan *> &plans, int rbt, M2lKind kind,
             std::vector<void *> &track) {
  const bool mixed = kind == kM2lMixed, small = kind == kM2lSmall;
  const int nd = kind == kM2lSteep ? kDigitsSteep : kind == kM2lDigits ? kDigits : 0;
  struct Key {
    const void *A;
    int k, c;
  };
  std::vector<Key> keys;
  std::vector<GemmJob> jobs;
  std::vector<std::vector<ColRef>> refs;
  std::vector<ColSrc> srcs;
  std::vector<int> cls;
  int dmax = 16, kmax = 0;
  for (Plan *Pp : plans) {
    const Plan &P = *Pp;
    for (int k = P.depth; k >= 2; --k) {
      const int64_t na = P.nact[k];
      if (na == 0 || m2l_kind(P, k) != kind) continue;
      cls.resize(na);
      if (hipMemcpy(cls.data(), P.ld[k].cls, sizeof(int) * na, hipMemcpyDeviceToHost) !=
          hipSuccess)
        return EIFMM_EHIP;
      const bool cz = P.lh[k].r > 0;
      const int dm = cz ? P.lh[k].rp : P.lh[k].dp, dk = nd == 0 ? dm : digit_kp(dm);
      dmax = k > kmax ? dm : k == kmax ? std::max(dmax, dm) : dmax;  // of the finest level
      kmax = std::max(kmax, k);
      const void *A = mixed   ? (const void *)P.ld[k].kfrag32
                      : small ? (const void *)P.ld[k].ksmall
                              : (const void *)P.ld[k].k8;
      ColSrc cs{};
      cs.keys = P.ld[k].act;
      cs.slot = P.ld[k].slot;
      if (mixed) {
        cs.B = cz ? P.ld[k].Whp32 : P.ld[k].Wh32;
      } else if (small) {
        cs.B = cz ? P.ld[k].Whp : P.ld[k].Wh;
      } else {
        cs.B = P.ld[k].w8;
        cs.bscale = P.ld[k].wscale;
      }
      cs.C = cz ? P.ld[k].gp : P.ld[k].g;
      const int rec = (int)srcs.size();
      srcs.push_back(cs);
      for (int c = 0; c < 8; ++c) {
        const int64_t c0 = P.cls_off[k][c], c1 = P.cls_off[k][c + 1];
        if (c1 == c0) continue;
        size_t j = 0;
        while (j < keys.size() && !(keys[j].A == A && keys[j].k == k && keys[j].c == c)) ++j;
        if (j == keys.size()) {
          keys.push_back(Key{A, k, c});
          GemmJob J{};
          J.A = A;
          J.terms = P.dlist + 189 * c;
          J.a_stride = (int64_t)dm * dk * (mixed ? sizeof(float) : nd);
          J.kexp = P.ld[k].kexp;
          J.ksteps = m2l_small_steps(cz ? P.lh[k].r : P.lh[k].d);
          J.nterms = 189;
          J.dpm = dm;
          J.dpk = dk;
          J.level = k;
          J.cls = c;
          J.mode = MODE_M2L;
          J.nrhs = 1;
          jobs.push_back(J);
          refs.emplace_back();
        }
        for (int64_t i = c0; i < c1; ++i) refs[j].push_back(ColRef{rec, cls[i]});
      }
    }
  }
  F = FusedGemm{};
  F.rbt = rbt > 0 ? rbt
          : mixed ? pick_m2l32(dmax / 16)
          : small ? kSmallM2l / 16
                  : pick_m2l8(dmax / 16, nd);
  F.nd = nd;
  if (jobs.empty()) return EIFMM_OK;
  // finest level first (as in a plan's own launch), then operator set and class
  std::vector<int> order(jobs.size());
  for (size_t j = 0; j < jobs.size(); ++j) order[j] = (int)j;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return jobs[a].level > jobs[b].level; });
  std::vector<ColRef> all;
  std::vector<GemmJob> h;
  std::vector<size_t> off;
  for (int j : order) {
    off.push_back(all.size());
    all.insert(all.end(), refs[j].begin(), refs[j].end());
    GemmJob J = jobs[j];
    J.ntgt = (int)refs[j].size();
    h.push_back(J);
  }
  ColSrc *srcs_dev = nullptr;
  ColRef *refs_dev = nullptr;
  int st = bupload(&srcs_dev, srcs, track);
  if (!st) st = bupload(&refs_dev, all, track);
  if (st) return st;
  int tiles = 0;
  for (size_t j = 0; j < h.size(); ++j) {
    h[j].colsrc = srcs_dev;
    h[j].colref = refs_dev + off[j];
    finish_job(h[j], tiles, F.rbt,
               mixed ? kM2l32Cols : small ? kSmallM2lCols : m2l8_cols(F.rbt));
  }
  F.units = finish_units(h, 0);
  F.tiles = tiles;
  F.n = (int)h.size();
  F.dk = h[0].dpk;
  return bupload(&F.dev, h, track);
}

template <int KIND>
void run_group(const BatchExec &B, const BatchGroup &g, int phase, hipStream_t s) {
  const LeafDesc *many = B.leaf_dev + g.first;
  const LeafDesc none{};
  const IoDesc inone{};
  if (phase == 0)
    launch_p2p<KIND, true>(B.mixed, 1, g.nchunk, none, many, g.count, s);
  else if (phase == 1) {
    for (int rounded = 1; rounded >= 0; --rounded) {
      const LeafDesc *d = rounded ? many : many + g.rounded;
      const int n = rounded ? g.rounded : g.count - g.rounded;
      const unsigned nseg = (unsigned)g.nseg[rounded];
      launch_p2m<KIND, true>(1, nseg, g.dpmax, none, d, n, s, rounded);
      if (g.nseg[rounded] > g.nleaf[rounded])
        hipLaunchKernelGGL((k_p2m_ext<true>), dim3(nseg), dim3(256), 0, s, none, d, n);
    }
  } else {
    launch_l2p<KIND, true>(1, g.nchunk, g.dpmax, none, inone, many, B.io_dev + g.first, g.count,
                           s);
  }
}

void run_groups(const BatchExec &B, int phase, hipStream_t s, const hipEvent_t *mark,
                int &m) {
  for (const BatchGroup &g : B.groups) {
    switch (g.kind) {
      case EIFMM_K_LAPLACE: run_group<EIFMM_K_LAPLACE>(B, g, phase, s); break;
      case EIFMM_K_YUKAWA: run_group<EIFMM_K_YUKAWA>(B, g, phase, s); break;
      case EIFMM_K_GAUSS: run_group<EIFMM_K_GAUSS>(B, g, phase, s); break;
      case EIFMM_K_COSR: run_group<EIFMM_K_COSR>(B, g, phase, s); break;
      case EIFMM_K_MQ: run_group<EIFMM_K_MQ>(B, g, phase, s); break;
      default: run_group<EIFMM_K_SQDIST>(B, g, phase, s); break;
    }
    if (mark) hipEventRecord(mark[m++], s);
  }
}

}  // namespace

void batch_release(BatchExec &B) {
  if (!B.track.empty()) hipDeviceSynchronize();  // launches may still read the tables
  for (void *p : B.track) hipFree(p);
  B = BatchExec{};
}

int batch_prepare(BatchExec &B, const std::vector<Plan *> &plans_in, int m2l_rbt, int sk_groups,
                  double *sk_ws) {
  batch_release(B);
  const int np = (int)plans_in.size();
  if (np == 0) return EIFMM_EINVAL;
  B.nprob = np;
  B.mixed = plans_in[0]->cfg.precision == EIFMM_PREC_MIXED;
  for (Plan *P : plans_in) {
    if (!P->points_set || P->depth < 2) return EIFMM_ESTATE;
    if ((P->cfg.precision == EIFMM_PREC_MIXED) != B.mixed) return EIFMM_EINVAL;
    if (P->jobs.nrhs != 1) {
      int st = build_jobs(*P, 1, nullptr);
      if (st) return st;
    }
    B.maxdepth = std::max(B.maxdepth, P->depth);
  }
  // descriptor order: problems grouped by kernel kind, in a group those whose What is
  // rounded first, then batch order
  std::vector<Plan *> plans;
  for (int kind = EIFMM_K_LAPLACE; kind <= EIFMM_K_MQ; ++kind) {
    BatchGroup g;
    g.kind = kind;
    g.first = (int)plans.size();
    for (int rounded = 1; rounded >= 0; --rounded) {
      for (int q = 0; q < np; ++q)
        if (plans_in[q]->cfg.kernel == kind && what_rounded(*plans_in[q]) == (rounded == 1)) {
          B.order.push_back(q);
          plans.push_back(plans_in[q]);
        }
      g.count = (int)plans.size() - g.first;
      if (rounded) g.rounded = g.count;
    }
    if (g.count) B.groups.push_back(g);
  }
  std::vector<LeafDesc> leaf(np);
  int64_t pts = 0;
  for (BatchGroup &g : B.groups) {
    int64_t ch = 0;
    for (int q = g.first; q < g.first + g.count; ++q) {
      const Plan &P = *plans[q];
      const int rounded = q < g.first + g.rounded ? 1 : 0;
      LeafDesc D = leaf_desc(P, 1);
      D.chunk_base = ch;
      D.seg_base = g.nseg[rounded];
      D.pt_base = pts;
      ch += P.nchunk;
      g.nleaf[rounded] += P.nact[P.depth];
      g.nseg[rounded] += P.nseg;
      pts += P.n;
      g.dpmax = std::max(g.dpmax, std::max(P.lh[P.depth].dp, P.lh[P.depth].dpB));
      leaf[q] = D;
    }
    g.nchunk = ch;
  }
  B.total_pts = pts;
  int st = bupload(&B.leaf_dev, leaf, B.track);
  if (st) return st;
  {
    std::vector<IoDesc> io(np, IoDesc{nullptr, 0, nullptr, 0});
    if ((st = bupload(&B.io_dev, io, B.track))) return st;
  }
  // triangular solves: What (z on compressed levels) on every level, lhat on the leaf level
  {
    std::vector<SolveDesc> w, l;
    int bw = 0, bl = 0;
    for (Plan *Pp : plans) {
      const Plan &P = *Pp;
      for (int k = 2; k <= P.depth; ++k) {
        const int nc = (int)P.nact[k];
        if (nc == 0) continue;
        SolveDesc D{};
        D.in = P.ld[k].W;
        D.out = P.ld[k].Wh;
        D.out32 = (B.mixed && P.lh[k].r == 0) ? P.ld[k].Wh32 : nullptr;
        D.Tf = P.ld[k].tri[0];
        D.Tb = solves_what(P, k) ? P.ld[k].tri[1] : nullptr;
        D.ncols = nc;
        D.dp = P.lh[k].dp;
        D.blk_start = bw;
        bw += (nc + 15) / 16;
        B.what_shm = std::max(B.what_shm, trsm_shm(D.dp));
        w.push_back(D);
      }
      const int k = P.depth, nc = (int)P.nact[k];
      if (nc == 0) continue;
      SolveDesc D{};
      D.in = P.ld[k].l;
      D.out = P.lhat;
      D.out32 = nullptr;
      D.Tf = P.ld[k].tri[2];
      D.Tb = P.ld[k].tri[3];
      D.ncols = nc;
      D.dp = P.lh[k].dpB;
      D.blk_start = bl;
      bl += (nc + 15) / 16;
      B.lhat_shm = std::max(B.lhat_shm, trsm_shm(D.dp));
      l.push_back(D);
    }
    if (!B.mixed) {
      std::vector<DigitDesc> dd;
      int blk = 0;
      for (Plan *Pp : plans)
        for (int k = Pp->depth; k >= 2; --k) {
          if (Pp->nact[k] == 0 || Pp->ld[k].ksmall) continue;
          dd.push_back(digit_desc(*Pp, k, 1, blk));
          blk += digit_blocks(dd.back().ncols);
        }
      B.digit_n = (int)dd.size();
      B.digit_blk = blk;
      if ((st = bupload(&B.digit_dev, dd, B.track))) return st;
    }
    B.what_n = (int)w.size();
    B.what_blk = bw;
    B.lhat_n = (int)l.size();
    B.lhat_blk = bl;
    if ((st = bupload(&B.what_dev, w, B.track))) return st;
    if ((st = bupload(&B.lhat_dev, l, B.track))) return st;
  }
  // gathered GEMMs
  const int nq = (int)plans.size();
  std::vector<std::pair<int, int>> r(nq);
  for (int k = B.maxdepth - 1; k >= 2; --k) {
    for (int q = 0; q < nq; ++q)
      r[q] = {plans[q]->jobs.m2m_first[k], k < plans[q]->depth ? plans[q]->jobs.m2m_n[k] : 0};
    if ((st = fuse_jobs(B.m2m[k], plans, r, 0, B.track))) return st;
  }
  for (int q = 0; q < nq; ++q) r[q] = {plans[q]->jobs.pre_first, plans[q]->jobs.pre_n};
  if ((st = fuse_jobs(B.pre, plans, r, 0, B.track))) return st;
  if ((st = pack_m2l(B.m2l, plans, m2l_rbt, B.mixed ? kM2lMixed : kM2lDigits, B.track))) return st;
  if (!B.mixed && (st = pack_m2l(B.m2l_steep, plans, 0, kM2lSteep, B.track))) return st;
  if (!B.mixed && (st = pack_m2l(B.m2l_small, plans, 0, kM2lSmall, B.track))) return st;
  for (int q = 0; q < nq; ++q) r[q] = {plans[q]->jobs.post_first, plans[q]->jobs.post_n};
  if ((st = fuse_jobs(B.post, plans, r, 0, B.track))) return st;
  for (int k = 3; k <= B.maxdepth; ++k) {
    for (int q = 0; q < nq; ++q)
      r[q] = {plans[q]->jobs.l2l_first[k], k <= plans[q]->depth ? plans[q]->jobs.l2l_n[k] : 0};
    if ((st = fuse_jobs(B.l2l[k], plans, r, 0, B.track))) return st;
  }
  B.m2l_flops = 0;
  for (Plan *P : plans) B.m2l_flops += P->m2l_flops;
  B.sk_groups = sk_groups;
  B.sk_ws = sk_ws;
  B.dvec = plans[0]->dvec;
  hipError_t e = hipDeviceSynchronize();
  return e == hipSuccess ? EIFMM_OK : EIFMM_EHIP;
}

void batch_run_m2l(const BatchExec &B, hipStream_t s) {
  launch_gemm_fused(B.m2l, MODE_M2L, B.mixed, B.sk_groups, B.sk_ws, B.dvec, s);
  launch_gemm_fused(B.m2l_steep, MODE_M2L, false, B.sk_groups, B.sk_ws, B.dvec, s);
  launch_m2l_small_packed(B.m2l_small.dev, B.m2l_small.n, B.m2l_small.tiles, B.dvec, s);
}

int batch_marks(const BatchExec &B) { return 9 + 3 * (int)B.groups.size(); }

void batch_run(const BatchExec &B, hipStream_t s, const hipEvent_t *mark) {
  int m = 0;
  auto tick = [&]() {
    if (mark) hipEventRecord(mark[m++], s);
  };
  tick();
  if (B.total_pts > 0)
    hipLaunchKernelGGL((k_gather_sigma<true>), dim3((unsigned)((B.total_pts + 255) / 256)),
                       dim3(256), 0, s, LeafDesc{}, IoDesc{}, B.leaf_dev, B.io_dev, B.nprob,
                       B.total_pts);
  tick();
  run_groups(B, 0, s, mark, m);  // near field, one mark per kernel kind
  run_groups(B, 1, s, mark, m);  // P2M
  for (int k = B.maxdepth - 1; k >= 2; --k)
    launch_gemm_fused(B.m2m[k], MODE_M2M, false, B.sk_groups, B.sk_ws, B.dvec, s);
  tick();
  if (B.what_blk > 0 && (B.mixed || B.what_blk > kSolveFew))
    hipLaunchKernelGGL(k_trsm_list, dim3(B.what_blk), dim3(64), B.what_shm, s, B.what_dev,
                       B.what_n);
  else if (B.what_blk > 0)
    hipLaunchKernelGGL(k_trsm4_list, dim3(B.what_blk), dim3(256), B.what_shm, s, B.what_dev,
                       B.what_n);
  tick();
  launch_gemm_fused(B.pre, MODE_PROJ, false, B.sk_groups, B.sk_ws, B.dvec, s);
  tick();
  if (!B.mixed) launch_digits_list(B.digit_dev, B.digit_n, B.digit_blk, s);
  batch_run_m2l(B, s);
  tick();
  launch_gemm_fused(B.post, MODE_PROJ, false, B.sk_groups, B.sk_ws, B.dvec, s);
  tick();
  for (int k = 3; k <= B.maxdepth; ++k)
    launch_gemm_fused(B.l2l[k], MODE_L2L, false, B.sk_groups, B.sk_ws, B.dvec, s);
  tick();
  if (B.lhat_blk > kSolveFew)
    hipLaunchKernelGGL(k_trsm_list, dim3(B.lhat_blk), dim3(64), B.lhat_shm, s, B.lhat_dev,
                       B.lhat_n);
  else if (B.lhat_blk > 0)
    hipLaunchKernelGGL(k_trsm4_list, dim3(B.lhat_blk), dim3(256), B.lhat_shm, s, B.lhat_dev,
                       B.lhat_n);
  tick();
  run_groups(B, 2, s, mark, m);  // L2P and the final sum
}

}  // namespace eifmm
