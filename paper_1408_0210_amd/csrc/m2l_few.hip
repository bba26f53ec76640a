// m2l_few.hip -- the M2L of level 2 for one right-hand side, offset by offset.
//
// A class has 8 of the level's 64 boxes, half a block of 16 columns, and the 8 classes
// read 1512 operators where 316 exist.  So the products are formed offset by offset over
// all classes (k_few_products: up to 32 columns, the targets whose source box exists;
// each wave takes a 16-row block of one offset and reads its operator fragments, which no
// other wave needs, straight from memory) and added up target by target in the order of
// the class's terms (k_few_sum).  A term's product is formed in the order of the tiled
// kernels, so it is the same number.
// Bound by reading the operators once (316 d^2: 105 MB in FP32, 204 MB as digits at
// d = 287: 21 and 41 us at the 5 TB/s of a copy).
// d = 287, FP64: 50 us products + 6 us sums where the tiles took half of a 391 us launch
// (depth 3, 2000 points; the pass 705 -> 591 us); d = 287, mixed, depth 2: 25 + 12 us
// instead of 200 (the pass of 777 points 452 -> 272 us).
#include "m2l_tile.hpp"

namespace eifmm {

namespace {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int kFrag = 1024;   // bytes of an operand fragment: 64 lanes x 16
constexpr int kFewCols = 32;  // most targets of an offset (delta = 2 along one axis)

struct FewArgs {
  const void *A;            // operators: FP32 fragments, or digits
  const int *slot;          // slot map of level 2
  const void *B;            // source columns: FP32, or digits
  const ColScale *bscale;   // digits: scale of each source column,
  const int *kexp;          // exponent of each row of each offset
  void *prod;               // [316][32][dm]: FP32 or FP64
  unsigned long long *mask; // [316] targets of each offset
  double *C;                // result [slot][dm]
  const int16_t *terms;     // 8 x 189 offset ids per child class
  int dm, dk;               // rows, columns (FP32: padded to 16, digits: to 64)
};

// ND: digits per operand, 0 for FP32
template <int ND>
__global__ __launch_bounds__(256) void k_few_products(FewArgs F, const int8_t *__restrict__ dvec) {
  __shared__ int tgt[64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nrb = F.dm >> 4, o = blockIdx.x, rb = blockIdx.y * 4 + w;
  // the offset's targets: boxes (by key) whose source box exists, in key order
  const int ts = F.slot[lane];
  const int m0 = (int)morton_axis(lane, 0) + dvec[3 * o],
            m1 = (int)morton_axis(lane, 1) + dvec[3 * o + 1],
            m2 = (int)morton_axis(lane, 2) + dvec[3 * o + 2];
  int ss = -1;
  if (ts >= 0 && m0 >= 0 && m1 >= 0 && m2 >= 0 && m0 < 4 && m1 < 4 && m2 < 4)
    ss = F.slot[morton_encode((uint32_t)m0, (uint32_t)m1, (uint32_t)m2)];
  const unsigned long long mask = __ballot(ss >= 0);
  const int n = (int)__popcll(mask);
  if (w == 0) {
    if (ss >= 0) tgt[(int)__popcll(mask & ((1ull << lane) - 1))] = ss;
    if (blockIdx.y == 0 && lane == 0) F.mask[o] = mask;
  }
  __syncthreads();
  if (rb >= nrb || n == 0) return;
  const int c0 = lane & 15, c1 = 16 + c0;
  // (a column past the last reads the last's source; its result is not stored)
  const int s0 = tgt[min(c0, n - 1)], s1 = tgt[min(c1, n - 1)];
  const bool two = n > 16;
  if constexpr (ND > 0) {
    const int nkc = F.dk >> 6;
    const int64_t cb = (int64_t)F.dk * ND;
    const int8_t *b0 = (const int8_t *)F.B + s0 * cb + 16 * (lane >> 4);
    const int8_t *b1 = (const int8_t *)F.B + s1 * cb + 16 * (lane >> 4);
    const int8_t *A = (const int8_t *)F.A + ((int64_t)o * nrb + rb) * nkc * (ND * kFrag) + 16 * lane;
    i4v acc[2][ND];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int s = 0; s < ND; ++s) acc[j][s] = i4v{0, 0, 0, 0};
    for (int kc = 0; kc < nkc; ++kc) {
      i4v a[ND], b[ND];
#pragma unroll
      for (int s = 0; s < ND; ++s) {
        a[s] = ldg((const i4v *)(A + kc * (ND * kFrag) + s * kFrag));
        b[s] = ldg((const i4v *)(b0 + kc * (64 * ND) + 64 * s));
      }
#pragma unroll
      for (int da = 0; da < ND; ++da)
#pragma unroll
        for (int db = 0; db + da < ND; ++db)
          acc[0][da + db] =
              __builtin_amdgcn_mfma_i32_16x16x64_i8(a[da], b[db], acc[0][da + db], 0, 0, 0);
      if (two) {
#pragma unroll
        for (int s = 0; s < ND; ++s) b[s] = ldg((const i4v *)(b1 + kc * (64 * ND) + 64 * s));
#pragma unroll
        for (int da = 0; da < ND; ++da)
#pragma unroll
          for (int db = 0; db + da < ND; ++db)
            acc[1][da + db] =
                __builtin_amdgcn_mfma_i32_16x16x64_i8(a[da], b[db], acc[1][da + db], 0, 0, 0);
      }
    }
    const int row = 16 * rb + 4 * (lane >> 4);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = j ? c1 : c0, sl = j ? s1 : s0;
      if (c >= n) continue;
      const ColScale sc = F.bscale[sl];
      double *P = (double *)F.prod + ((int64_t)o * kFewCols + c) * F.dm + row;
      const int *ex = F.kexp + (int64_t)o * F.dm + row;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double v = (double)acc[j][ND - 1][q];
#pragma unroll
        for (int s = ND - 2; s >= 0; --s) v = fma(v, 1.0 / 256.0, (double)acc[j][s][q]);
        P[q] = ldexp(v, ldg(ex + q) + sc.e) * sc.sign;
      }
    }
  } else {
    const int nkc = F.dk >> 4;
    const float *b0 = (const float *)F.B + (int64_t)s0 * F.dk + 4 * (lane >> 4);
    const float *b1 = (const float *)F.B + (int64_t)s1 * F.dk + 4 * (lane >> 4);
    const float *A = (const float *)F.A + ((int64_t)o * nrb + rb) * nkc * 256 + 4 * lane;
    f4v a0 = {0, 0, 0, 0}, a1 = {0, 0, 0, 0};
#pragma unroll 4
    for (int kc = 0; kc < nkc; ++kc) {
      const f4v x = ldg((const f4v *)(b0 + 16 * kc));
      f4v y = {0, 0, 0, 0};
      if (two) y = ldg((const f4v *)(b1 + 16 * kc));
      const f4v a = ldg((const f4v *)(A + 256 * kc));
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks], x[ks], a0, 0, 0, 0);
        if (two) a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks], y[ks], a1, 0, 0, 0);
      }
    }
    const int row = 16 * rb + 4 * (lane >> 4);
    float *P = (float *)F.prod + (int64_t)o * kFewCols * F.dm + row;
    if (c0 < n) stg((f4v *)(P + (int64_t)c0 * F.dm), a0);
    if (c1 < n) stg((f4v *)(P + (int64_t)c1 * F.dm), a1);
  }
}

// one workgroup per box and 64 rows: a lane per row and quarter of the terms, the
// quarters added in order
template <typename T>
__global__ __launch_bounds__(256) void k_few_sum(FewArgs F, const int8_t *__restrict__ dvec) {
  __shared__ int at[192];  // product column of each term, -1: no source
  __shared__ double part[4][64];
  const int key = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int ts = F.slot[key];
  if (ts < 0) return;
  const int16_t *terms = F.terms + 189 * (key & 7);
  if (t < 192) {
    int c = -1;
    if (t < 189) {
      const int o = terms[t];
      const unsigned long long m = F.mask[o];
      if ((m >> key) & 1ull)
        c = o * kFewCols + (int)__popcll(m & ((1ull << key) - 1));
    }
    at[t] = c;
  }
  __syncthreads();
  const int row = blockIdx.y * 64 + lane;
  const bool ok = row < F.dm;
  const T *P = (const T *)F.prod + (ok ? row : 0);
  double v = 0.0;
  for (int q = 48 * w; q < 48 * w + 48; q += 8) {
    T p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = at[q + u];
      p[u] = c >= 0 ? ldg(P + (int64_t)c * F.dm) : T(0);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) v += (double)p[u];
  }
  part[w][lane] = v;
  __syncthreads();
  if (w == 0 && ok) {
    v = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
    F.C[(int64_t)ts * F.dm + row] = v;
  }
}

}  // namespace

size_t m2l_few_bytes(int dm, bool mixed) {
  return (size_t)kNumOffsets * kFewCols * dm * (mixed ? sizeof(float) : sizeof(double)) +
         sizeof(unsigned long long) * kNumOffsets;
}

void launch_m2l_few(const LevelDev &D, bool mixed, const void *B, int dm, int dk, double *C, void *ws,
                    const int16_t *terms, const int8_t *dvec, hipStream_t s) {
  FewArgs F{};
  F.A = mixed ? (const void *)D.kfrag32 : (const void *)D.k8;
  F.slot = D.slot;
  F.B = B;
  F.bscale = D.wscale;
  F.kexp = D.kexp;
  F.mask = (unsigned long long *)ws;
  F.prod = F.mask + kNumOffsets;
  F.C = C;
  F.terms = terms;
  F.dm = dm;
  F.dk = mixed ? dk : digit_kp(dk);
  const dim3 gp(kNumOffsets, (dm / 16 + 3) / 4), gs(64, (dm + 63) / 64);
  if (mixed) {
    hipLaunchKernelGGL(k_few_products<0>, gp, dim3(256), 0, s, F, dvec);
    hipLaunchKernelGGL(k_few_sum<float>, gs, dim3(256), 0, s, F, dvec);
  } else {
    if (D.nd == kDigitsSteep)
      hipLaunchKernelGGL(k_few_products<kDigitsSteep>, gp, dim3(256), 0, s, F, dvec);
    else
      hipLaunchKernelGGL(k_few_products<kDigits>, gp, dim3(256), 0, s, F, dvec);
    hipLaunchKernelGGL(k_few_sum<double>, gs, dim3(256), 0, s, F, dvec);
  }
}

}  // namespace eifmm
