// m2l.hip -- the FP64 M2L (Algorithm 3 step 4) on the int8 matrix cores.
//
// C[:, col] = sum over the 189 offsets o of the column's child class of A_o b(o, col),
// A_o the K^delta or C^delta of the level and b the source expansion at that offset.
// The FP64 MFMA runs at 1/56 of the int8 one on gfx950 (75 TFLOP/s against 4.0 POP/s
// measured), so every operand is split into 7 signed 8-bit digits (56 bits; 8 on steep
// levels, below) and the product is summed from the digit products, which are exact in
// 32-bit integers:
//   a = 2^ea sum_i da_i 256^-(i+1),  b = 2^eb sum_j db_j 256^-(j+1),  -128 <= d <= 127,
//   sum_k a_k b_k = 2^(ea + eb - 16) sum_s 256^-s S_s,  S_s = sum_{i+j=s} sum_k da_ik db_jk.
// One exponent per operator row of each offset and one per source column.  Digit
// pairs with i + j > 6 lie below 2^-56 of the largest product and are left out: 28
// products instead of 49.  The seven sums S_s of an offset are joined and scaled in
// FP64 and added to an FP64 sum over the offsets.
// An entry keeps 56 bits below the largest of its row or column, so an offset's product
// is off by about d^1/2 2^-56 max_k |a_k| max_k |b_k|, where a chain of FP64 FMAs is off by
// some 2^-53 of its partial sums.  (Were a row's exponent one for all offsets, a far
// offset of a decaying kernel would keep what its entries have above 2^-56 of the nearest
// ones': g in the corner opposite to the sources, level 2, would be off by 1e-5 of itself for
// e^-30r/r and wholly for e^-60r/r, as against 6e-15 and 6e-13.)  Where the kernel falls so
// far across one pair of boxes that this is more than the chain's error (kSteep), operands
// have 8 digits (64 bits) and take 36 products, s to 7.  Error of single offsets' products
// over that of the chain, offsets (2,0,0) to (3,3,3), level 2, tau 1e-5, against extended
// precision, uncompressed: 1/r 0.2-0.3, cos(20 r)/r 0.3-0.5, e^-r^2 0.4-0.6, e^-8r/r
// 0.5-0.8, e^-12r/r 0.8-1.5, e^(-r^2/0.1) 0.7-1.9, e^-30r/r 0.9-4.7, e^-60r/r 0.4-18 with
// 7 digits, and 0.01-0.2 with 8 for all of these; compressed: 1/r 0.6-1.0, cos(20 r)/r
// 1.3-1.9, e^(-r^2/0.01) 4.4-8.4, and 0.04-0.1 with 8.  Whole interaction lists (189
// offsets, boxes of 30 random points, tau 1e-6, against an 80-bit evaluation): 1/r at rank
// 128 0.75e-15 relative against 5.3e-15 for the chain, e^-r/r 0.6e-15 / 5.5e-15, cos(20 r)/r
// 0.6e-15 / 6.9e-15, 1/r uncompressed (d = 287) 0.5e-15 / 8.0e-15, e^-r^2 0.5e-15 / 3.5e-15,
// e^(-r^2/0.01) 0.4e-15 with 8 digits (1.8e-15 with 7) / 8.0e-15.
// (The method is the splitting of Ozaki, Ogita, Oishi and Rump, "Error-free transformations
// of matrix multiplication by using fast routines of matrix multiplication and its
// applications", 2012, with slices of fixed width.)
//
// Time of the launch against tiles of FP64 MFMAs: 2.50 ms against 3.96 on 1e6 uniform
// points (1/r, rank 128, levels 2..5), 2.05 against 2.88 on 2e5 points uncompressed
// (d = 287, levels 2..4), 0.38 against 0.67 on 2000 points (d = 287, levels 2 and 3).
// The matrix cores are busy half of the time (1.73e8 products of 16 cycles); copies that
// load nothing take 1.51 ms and copies that load one operator and no sources (always in
// L2) 2.07, so what bounds it is the way through LDS (84 KB in and 280 KB out per chunk
// and CU, 2850 cycles at 128 bytes, beside 3584 of products) and the fabric's latency.
#include <algorithm>
#include <cmath>
#include <vector>

#include "m2l_tile.hpp"

namespace eifmm {

namespace {

typedef int i4v __attribute__((ext_vector_type(4)));
constexpr int kFrag = 1024;  // bytes of one 16 x 64 operand fragment (64 lanes x 16)

// zeros, read in place of a missing source column (digits of 1024 elements) and,
// as a ColScale, of its scale
__device__ i4v g_digit_zero[kDigitsSteep * 1024 / 16];

// the exponent e of the smallest power of two with m 2^-e <= 0.498, so that the top
// digit of every |x| <= m stays within [-127, 127]; m > 0 and finite
__device__ inline int digit_exponent(double m) {
  int e;
  const double f = frexp(m, &e);  // f in [0.5, 1)
  return e + 1 + (f > 0.996 ? 1 : 0);
}

// the digits of x 2^-e, most significant first
template <int ND>
__device__ inline void digits_of(double x, int e, int8_t (&d)[ND]) {
  long long q = __double2ll_rn(ldexp(x, 8 * ND - e));
#pragma unroll
  for (int s = ND - 1; s >= 0; --s) {
    d[s] = (int8_t)(q & 255);
    q = (q - d[s]) >> 8;
  }
}

// The operators' digit fragments, [offset][row block][64-k chunk][digit][lane][16 k],
// lane l holding row l % 16 and k = 16 (l / 16) .. + 15 of the chunk, and the exponent of
// each row of each offset, [offset][row]: value = 2^exponent * (source scale) *
// sum_s 256^-s S_s.  frag is the table in FP64 fragment order (setup.cpp: lane l of a
// fragment holds row l % 16).  One workgroup per (offset, row block).  A row holding an
// infinity or a NaN gets the digit 1 everywhere and an exponent that makes its results
// infinite.
template <int ND>
__global__ __launch_bounds__(256) void k_op_digits(const double *__restrict__ frag, int nrb, int nks,
                                                   int nkc, int8_t *__restrict__ out,
                                                   int *__restrict__ kexp) {
  __shared__ double mx[4][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *F = frag + (size_t)blockIdx.x * nks * 64;
  double m = 0.0;
  bool bad = false;
  for (int ks = w; ks < nks; ks += 4) {
    const double x = fabs(F[(size_t)ks * 64 + lane]);
    bad = bad || !(x < INFINITY);
    m = fmax(m, x);
  }
  if (bad) m = INFINITY;
  m = fmax(m, __shfl_xor(m, 16));
  m = fmax(m, __shfl_xor(m, 32));
  if (lane < 16) mx[w][lane] = m;
  __syncthreads();
  const int row = lane & 15;
  m = fmax(fmax(mx[0][row], mx[1][row]), fmax(mx[2][row], mx[3][row]));
  bad = !(m < INFINITY);
  const int e = !bad && m > 0.0 ? digit_exponent(m) : 0;
  if (threadIdx.x < 16) kexp[(size_t)blockIdx.x * 16 + row] = bad ? 1 << 20 : e - 16;
  for (int kc = w; kc < nkc; kc += 4) {
    const int c16 = kc * 4 + (lane >> 4);  // 16-column chunk of the table
    union {
      int8_t b[16];
      i4v v;
    } dig[ND];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      double x = 0.0;
      if (4 * c16 < nks) x = F[(size_t)(4 * c16 + (k & 3)) * 64 + 16 * (k >> 2) + row];
      int8_t d[ND] = {1};
      if (!bad) digits_of<ND>(x, e, d);
#pragma unroll
      for (int s = 0; s < ND; ++s) dig[s].b[k] = d[s];
    }
    int8_t *o = out + ((size_t)blockIdx.x * nkc + kc) * (ND * kFrag) + 16 * lane;
#pragma unroll
    for (int s = 0; s < ND; ++s) *(i4v *)(o + s * kFrag) = dig[s].v;
  }
}

// Source columns into digits: 16 lanes per column, 4 consecutive k per lane and
// 64-k chunk; out: [column][chunk][digit][64 k] bytes, scale: ColScale.  The digits
// are those of the column with its first entry that is not zero made positive, and the
// scale carries the sign: the digits of x and -x differ otherwise (a digit of -128 has
// no counterpart), and a pass of -sigma would not be exactly the negative one.
// Bound by memory (8 bytes read and 7 or 8 written per element).
template <int ND>
__device__ inline void digit_column(const DigitDesc &D, int col) {
  const int li = threadIdx.x & 15;
  const double *in = D.in + (int64_t)col * D.ld;
  const int nkc = D.kp >> 6;
  double m = 0.0;
  bool bad = false;
  int first = INT_MAX;  // 2 k + (entry k < 0) of the first entry that is not zero
  for (int kc = 0; kc < nkc; ++kc) {
    const int k = 64 * kc + 4 * li;
    if (k < D.ld) {
      const d2v a = ldg((const d2v *)(in + k)), b = ldg((const d2v *)(in + k + 2));
      const double v[4] = {a.x, a.y, b.x, b.y};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bad = bad || !(fabs(v[q]) < INFINITY);
        m = fmax(m, fabs(v[q]));
        if (v[q] != 0.0) first = min(first, 2 * (k + q) + (v[q] < 0.0 ? 1 : 0));
      }
    }
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    m = fmax(m, __shfl_xor(m, o));
    bad = __shfl_xor((int)bad, o) || bad;
    first = min(first, __shfl_xor(first, o));
  }
  const bool use = !bad && m > 0.0, neg = use && (first & 1);
  const int e = use ? digit_exponent(m) : 0;
  for (int kc = 0; kc < nkc; ++kc) {
    const int k = 64 * kc + 4 * li;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (use && k < D.ld) {
      const d2v a = ldg((const d2v *)(in + k)), b = ldg((const d2v *)(in + k + 2));
      v[0] = a.x;
      v[1] = a.y;
      v[2] = b.x;
      v[3] = b.y;
    }
    uint32_t pk[ND] = {};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int8_t d[ND];
      digits_of<ND>(neg ? -v[q] : v[q], e, d);
#pragma unroll
      for (int s = 0; s < ND; ++s) pk[s] |= (uint32_t)(uint8_t)d[s] << (8 * q);
    }
    int8_t *o = D.out + (int64_t)col * D.kp * ND + (size_t)kc * 64 * ND + 4 * li;
#pragma unroll
    for (int s = 0; s < ND; ++s) stg((uint32_t *)(o + 64 * s), pk[s]);
  }
  if (li == 0) {
    D.scale[col].sign = bad ? NAN : !use ? 0.0f : neg ? -1.0f : 1.0f;
    D.scale[col].e = e;
  }
}

__device__ inline void digit_column_of(const DigitDesc &D, int col) {
  if (D.nd == kDigitsSteep)
    digit_column<kDigitsSteep>(D, col);
  else
    digit_column<kDigits>(D, col);
}

struct DigitArgs {
  DigitDesc lv[kMaxLevels];
  int nlev;
};

// one plan: a descriptor per level, by value
__global__ __launch_bounds__(256) void k_digits(DigitArgs A) {
  int li = 0;
  for (int q = 1; q < A.nlev; ++q)
    if ((int)blockIdx.x >= A.lv[q].blk_start) li = q;
  const DigitDesc &D = A.lv[li];
  const int col = ((int)blockIdx.x - D.blk_start) * kDigitCols + (int)(threadIdx.x >> 4);
  if (col < D.ncols) digit_column_of(D, col);
}

// a batch: every (problem, level), descriptors in device memory
__global__ __launch_bounds__(256) void k_digits_list(const DigitDesc *__restrict__ L, int n) {
  const int li =
      find_last_le(n, blockIdx.x, [&](int m) { return (int64_t)L[m].blk_start; });
  const DigitDesc D = L[li];
  const int col = ((int)blockIdx.x - D.blk_start) * kDigitCols + (int)(threadIdx.x >> 4);
  if (col < D.ncols) digit_column_of(D, col);
}

// Terms [term0, term1) of one tile of 16 RB RG rows and 128 / RG columns: the result,
// or a piece (part).  8 waves, RG groups of rows by 8 / RG groups of 16 columns; a wave
// holds RB row blocks of its 16 columns; operands of ND digits.  The operator fragments
// of a 64-k chunk go to LDS one chunk ahead, in two buffers; the source digits (16 columns
// and 64 k are one fragment per digit) one chunk ahead too, in one buffer that every wave
// copies to registers at the start of the chunk.  Both are direct loads, which need no
// registers: the digit sums and the FP64 sums take 144 of a lane's 256 (RB = 4, 7 digits).
// The rows' exponents of a term go to LDS with its first chunk, in three buffers: a wave may
// still join the sums of the term before the last one written.  The slots of the sources
// are read one term ahead.  A step waits for all of them at its start, a whole chunk of
// products (RB x 28 or 36 MFMAs per wave) after they were issued.
template <int ND, int RB, int RG>
__device__ inline void m2l8_tile(const GemmJob &J, int tile_local, int term0, int term1,
                                 double *__restrict__ part, const int8_t *__restrict__ dvec,
                                 int8_t (*As)[RB * RG * ND * kFrag], int8_t *Bs,
                                 int (*Es)[16 * RB * RG], TileCol *cst, int *sdel) {
  constexpr int CG = 8 / RG, H = RB * RG, COLS = 16 * CG;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rg = w / CG, cg = w % CG;
  const int rowtile = tile_local % J.nrowtiles, coltile = tile_local / J.nrowtiles;
  const int rb0 = rowtile * H, col0 = coltile * COLS;
  const int nrb = J.dpm >> 4, nkc = J.dpk >> 6;
  const int nv = min(H, nrb - rb0);             // row blocks of this tile
  const int nw = max(0, min(RB, nv - rg * RB));  // row blocks of this wave
  const int ncols = J.ntgt * J.nrhs;
  const int64_t colbytes = (int64_t)J.dpk * ND;

  TileCol *my = cst + 16 * cg + (lane & 15);  // (the waves of a column group write the same)
  int bb[6];
  *my = tile_column(J, col0 + 16 * cg + (lane & 15), bb);
  const int nt = tile_terms(J, term0, term1, bb, dvec, sdel);
  double sum[RB][4];
  i4v acc[RB][ND];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[i][q] = 0.0;
  }
  if (nt > 0) {
    const uint32_t lds0 =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)&As[0][0];
    const uint32_t lane16 = 16u * (uint32_t)lane;
    const int8_t *Abase = (const int8_t *)J.A + (int64_t)rb0 * nkc * ND * kFrag;
    const uint32_t ldsb =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)Bs + cg * (ND * kFrag);
    int slotn = ldg(source_slot(J, *my, 0, nt, sdel));  // slot of the next term to load
    const int8_t *srcp = nullptr, *At = nullptr;
    // scale of the source and whether the wave has any: of the term aimed at (n), of
    // the last one loaded (q)
    ColScale scn{}, scq{};
    bool haven = false, haveq = false;
    int en = 0;          // a row's exponent of the term aimed at (the first 16 H threads)
    int ew = 0, er = 2;  // buffer of exponents: the next one to write, the current term's
    int fq = 0, fk = 0;  // next chunk to load: term, chunk
    // the addresses of the next chunk to load, if it starts a term; runs a step ahead of
    // that load, behind the products, since its chain of reads is long
    auto aim = [&]() {
      if (fq >= nt || fk != 0) return;
      const TileCol c = *my;
      const int sl = slotn;
      const int64_t col = (int64_t)sl * J.nrhs + c.r;
      srcp = (sl < 0 ? (const int8_t *)g_digit_zero : (const int8_t *)c.B + col * colbytes) + 16 * (lane >> 4);
      const ColScale *bs = sl < 0 ? (const ColScale *)g_digit_zero : c.bs + col;
      scn = ColScale{ldg(&bs->sign), ldg(&bs->e)};
      haven = __ballot(sl >= 0) != 0;
      const int o = __builtin_amdgcn_readfirstlane(sdel[fq]) >> 9;
      At = Abase + (int64_t)o * J.a_stride;
      if (64 * w < 16 * H) en = ldg(J.kexp + (int64_t)o * J.dpm + min(16 * rb0 + t, J.dpm - 1));
      slotn = ldg(source_slot(J, c, fq + 1, nt, sdel));
    };
    // The loads of the next chunk, operators to LDS buffer `buf` and sources to Bs, are
    // issued one at a time between the products: a burst of them would hold up the
    // wave.  A column group's digits are shared out to its RG waves; a row block's
    // operator fragments make two pieces (4 and the rest), dealt to the waves.
    constexpr int NB = RG == 2 ? 4 : ND, NP = (2 * H + 7) / 8, NL = NB + 4 * NP;
    static_assert(NL <= ND * RB, "a load per fragment of the products");
    bool live = false;
    const int8_t *sp = nullptr;
    uint64_t ap[NP];
    uint32_t lp[NP];
    const int half = w & 1;
    auto fetch_begin = [&](int buf) {
      live = fq < nt;
      if (!live) return;
      if (fk == 0) {
        scq = scn;
        haveq = haven;
        if (t < 16 * H) Es[ew][t] = en;
        ew = ew == 2 ? 0 : ew + 1;
      }
      sp = srcp + fk * (64 * ND) + (RG == 2 ? rg * 256 : 0);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int blk = (w >> 1) + 4 * i;
        ap[i] = uniform64((uint64_t)(At + (int64_t)(blk * nkc + fk) * (ND * kFrag) + half * 4 * kFrag));
        lp[i] = __builtin_amdgcn_readfirstlane(
            lds0 + (uint32_t)(buf * (H * ND * kFrag) + (blk * ND + half * 4) * kFrag));
      }
      if (++fk == nkc) {
        fk = 0;
        ++fq;
      }
    };
    const uint32_t ldsw = __builtin_amdgcn_readfirstlane(ldsb + (RG == 2 ? rg * 4 * kFrag : 0));
    auto fetch_one = [&](auto N) {
      constexpr int n = decltype(N)::value;
      if (!live) return;
      if constexpr (n < NB) {
        if (RG == 1 || n < ND - 4 || rg == 0) column_to_lds<64 * n>(sp, ldsw + n * kFrag);
      } else if constexpr (n < NL) {
        constexpr int i = (n - NB) / 4, j = (n - NB) % 4;
        if ((w >> 1) + 4 * i < nv && (j < ND - 4 || half == 0))
          fragment_to_lds<j * kFrag>(ap[i], lp[i], lane16);
      }
    };
    auto fetch_all = [&](auto N0) { for_each_from<decltype(N0)::value, NL>(fetch_one); };
    // The 28 (36) digit products of each of the wave's row blocks [i0, i1) in one chunk, the
    // operator fragments read three ahead of their products (blocks past the tile's
    // rows multiply what the buffer holds; their sums are not stored).  first: the
    // term's first chunk, whose sums start at zero.
    auto products = [&](auto first, int buf, const i4v(&b)[ND]) {
      constexpr int NF = RB * ND, AHEAD = 3;
      const int8_t *Ap = &As[buf][rg * RB * ND * kFrag + 16 * lane];
      i4v a[AHEAD];
#pragma unroll
      for (int f = 0; f < AHEAD; ++f) a[f] = *(const i4v *)(Ap + f * kFrag);
      __builtin_amdgcn_sched_barrier(0);
      auto group = [&](auto Fc) {
        constexpr int f = decltype(Fc)::value, i = f / ND, da = f % ND;
#pragma unroll
        for (int db = 0; db + da < ND; ++db) {
          const i4v c = decltype(first)::value && da == 0 ? i4v{0, 0, 0, 0} : acc[i][da + db];
          acc[i][da + db] =
              __builtin_amdgcn_mfma_i32_16x16x64_i8(a[f % AHEAD], b[db], c, 0, 0, 0);
        }
        if (f + AHEAD < NF) a[f % AHEAD] = *(const i4v *)(Ap + (f + AHEAD) * kFrag);
        constexpr int SP = 2 * NL + 4 <= NF ? 2 : 1;  // (the last loads early enough)
        if constexpr (f % SP == 0) fetch_one(std::integral_constant<int, f / SP>{});
        __builtin_amdgcn_sched_barrier(0);
      };
      for_each_from<0, NF>(group);
    };
    // a term's digit sums, joined in FP64 and scaled (by the sum of the exponents, so that
    // nothing but the product itself has to lie in range), added to the tile's sums
    auto fold = [&](ColScale scf) {
      const double sign = scf.sign;
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const i4v ex = *(const i4v *)&Es[er][16 * (rg * RB + i) + 4 * (lane >> 4)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double v = (double)acc[i][ND - 1][q];
#pragma unroll
          for (int s = ND - 2; s >= 0; --s) v = fma(v, 1.0 / 256.0, (double)acc[i][s][q]);
          sum[i][q] = fma(ldexp(v, ex[q] + scf.e), sign, sum[i][q]);
        }
      }
    };
    // The two waves of a SIMD (w and w + 4) take turns on its matrix core: the first
    // has priority and joins a term's sums at the end of the term's last chunk, while
    // the second multiplies; the second joins them at the start of the next chunk,
    // while the first multiplies, and issues its loads after its first row block.
    const bool lead = w < 4;
    if (lead)
      __builtin_amdgcn_s_setprio(1);
    else
      __builtin_amdgcn_s_setprio(0);
    ColScale sc{};
    bool have = false, pend = false;  // pend: the last term's sums are not joined yet
    int kc = 0;                       // chunk of the current term
    auto step = [&](int buf) {
      // everything this wave issued in the last step has arrived, and after the
      // barrier what the others issued; the second barrier ends the reads of Bs,
      // which the next loads overwrite
      __builtin_amdgcn_s_waitcnt(0x0f70);
      lds_barrier();
      i4v Bc[ND];
#pragma unroll
      for (int s = 0; s < ND; ++s)
        Bc[s] = *(const i4v *)&Bs[(cg * ND + s) * kFrag + 16 * lane];
      lds_barrier();
      if (pend) {
        fold(sc);
        pend = false;
      }
      const bool fst = kc == 0;
      if (fst) {
        sc = scq;
        er = er == 2 ? 0 : er + 1;
        have = haveq && nw > 0;
      }
      fetch_begin(buf ^ 1);
      if (!have)
        fetch_all(std::integral_constant<int, 0>{});
      else if (fst)
        products(std::true_type{}, buf, Bc);
      else
        products(std::false_type{}, buf, Bc);
      aim();
      if (++kc == nkc) {
        kc = 0;
        if (have && lead)
          fold(sc);
        else
          pend = have;
      }
    };
    aim();
    fetch_begin(0);
    fetch_all(std::integral_constant<int, 0>{});
    aim();
    const int steps = nt * nkc;
    for (int it = 0; it < steps; ++it) step(it & 1);
    if (pend) fold(sc);
    __builtin_amdgcn_s_setprio(0);
  }

  // result row 16 block + 4 (lane / 16) + q of column lane % 16
  const int jt = 16 * cg + (lane & 15), jo = col0 + jt;
  if (jo >= ncols) return;
  double *out;
  if (part) {
    out = part + (size_t)jt * (16 * H);
  } else {
    out = tile_output(J, jo) + 16 * rb0;
  }
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    if (i < nw) {
      const int rt = 16 * (rg * RB + i) + 4 * (lane >> 4);
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        d2v v;
        v.x = sum[i][q];
        v.y = sum[i][q + 1];
        stg((d2v *)(out + rt + q), v);
      }
    }
  }
}

// Tiles [0, full) run whole, G workgroups at a time in the order of the terms (so that
// the operators they read are shared in L2; the tiles of one XCD (g mod 8) are
// contiguous); the others are cut into `parts` term ranges each, taken in order from
// a counter and summed by k_m2l_sum, so that workgroups whose tiles dropped terms
// take more of them.  A workgroup that reads a value outside [0, items) stops.
template <int ND, int RB, int RG>
__global__ __launch_bounds__(512, 2) void k_m2l8(const GemmJob *__restrict__ jobs, int njobs,
                                                 int G, int full, int items, int parts,
                                                 double *__restrict__ ws,
                                                 const int8_t *__restrict__ dvec,
                                                 int *__restrict__ ctr) {
  constexpr int H = RB * RG, TILE = H * 16 * (128 / RG);
  __shared__ __align__(16) int8_t As[2][H * ND * kFrag];
  __shared__ __align__(16) int8_t Bs[(8 / RG) * ND * kFrag];
  __shared__ __align__(16) int Es[3][16 * H];
  __shared__ TileCol cst[128 / RG];
  __shared__ int sdel[189];
  __shared__ int item_sh;
  const int g = blockIdx.x;
  const int gx = (G % 8 == 0) ? (g % 8) * (G / 8) + g / 8 : g;
  for (int tile = gx; tile < full; tile += G) {
    const GemmJob J = jobs[job_of_tile(jobs, njobs, tile)];
    m2l8_tile<ND, RB, RG>(J, tile - J.tiles_start, 0, J.nterms, nullptr, dvec, As, Bs, Es, cst, sdel);
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
    m2l8_tile<ND, RB, RG>(J, tile - J.tiles_start, q * J.nterms / parts, (q + 1) * J.nterms / parts,
                          ws + (size_t)item * TILE, dvec, As, Bs, Es, cst, sdel);
  }
}

template <int ND, int RB, int RG>
void launch(const GemmJob *jobs, int n, int tiles, int cus, double *ws, size_t ws_len,
            const int8_t *dvec, hipStream_t s) {
  constexpr int H = RB * RG;
  // one workgroup per CU (its operator buffers take most of the LDS)
  const TileSplit T = split_tiles(tiles, cus, (size_t)H * 16 * (128 / RG), ws_len);
  int *ctr = (int *)(ws + ws_len - kCounterDoubles);
  hipLaunchKernelGGL((k_m2l8<ND, RB, RG>), dim3(T.grid), dim3(512), 0, s, jobs, n, T.grid, T.full,
                     T.rest * T.parts, T.parts, ws, dvec, ctr);
  if (T.rest > 0)
    hipLaunchKernelGGL(k_m2l_sum, dim3(T.rest * kSumSplit), dim3(256), 0, s, jobs, n, tiles, T.full,
                       T.parts, H, m2l8_cols(H), ws, ctr);
}

}  // namespace

// The tile height that leaves the fewest idle row blocks, the taller one on a tie (with 8
// digits the lower one).  8 and 6 blocks are 64 columns wide, the lower ones 128.  Eight
// digits leave LDS for at most 6; there 4 take 2.97 ms where 3 take 3.70 and 6 (20 % idle)
// 3.71 (32 problems, half of them e^(-r^2 / 0.01), 20 row blocks).  (Operators of 2 row
// blocks and as many columns go to m2l_small.hip.)
int pick_m2l8(int nrb, int nd) {
  auto waste = [&](int h) { return (nrb + h - 1) / h * h - nrb; };
  if (nd == kDigitsSteep) return waste(6) < waste(4) ? 6 : 4;
  int best = 8;
  for (int h : {6, 4, 3})
    if (waste(h) < waste(best)) best = h;
  return best;
}

void launch_m2l8(const GemmJob *jobs, int n, int tiles, int height, int nd, int cus, double *ws,
                 size_t ws_len, const int8_t *dvec, hipStream_t s) {
  if (n == 0 || tiles == 0) return;
  if (nd == kDigitsSteep) {
    constexpr int N = kDigitsSteep;
    if (height == 6)
      launch<N, 3, 2>(jobs, n, tiles, cus, ws, ws_len, dvec, s);
    else
      launch<N, 4, 1>(jobs, n, tiles, cus, ws, ws_len, dvec, s);
    return;
  }
  constexpr int N = kDigits;
  switch (height) {
    case 8: launch<N, 4, 2>(jobs, n, tiles, cus, ws, ws_len, dvec, s); break;
    case 6: launch<N, 3, 2>(jobs, n, tiles, cus, ws, ws_len, dvec, s); break;
    case 4: launch<N, 4, 1>(jobs, n, tiles, cus, ws, ws_len, dvec, s); break;
    default: launch<N, 3, 1>(jobs, n, tiles, cus, ws, ws_len, dvec, s); break;
  }
}

int digit_blocks(int ncols) { return (ncols + kDigitCols - 1) / kDigitCols; }

void launch_digits(const DigitDesc *lv, int nlev, int blocks, hipStream_t s) {
  if (nlev == 0 || blocks == 0) return;
  DigitArgs A{};
  for (int q = 0; q < nlev; ++q) A.lv[q] = lv[q];
  A.nlev = nlev;
  hipLaunchKernelGGL(k_digits, dim3(blocks), dim3(256), 0, s, A);
}

void launch_digits_list(const DigitDesc *dev, int n, int blocks, hipStream_t s) {
  if (n == 0 || blocks == 0) return;
  hipLaunchKernelGGL(k_digits_list, dim3(blocks), dim3(256), 0, s, dev, n);
}

// The digit fragments of one level's M2L operators (rows x cols, both multiples of 16) and
// the exponents of their rows, from their FP64 fragments on the host.
int upload_digit_operators(const std::vector<double> &frag, int rows, int cols, int nd,
                           int8_t *dig, int *kexp) {
  const int nrb = rows / 16, nks = cols / 4, nkc = digit_kp(cols) / 64;
  double *tab = nullptr;
  hipError_t e = hipMalloc(&tab, sizeof(double) * std::max<size_t>(frag.size(), 1));
  if (e == hipSuccess)
    e = hipMemcpy(tab, frag.data(), sizeof(double) * frag.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(nd == kDigitsSteep ? k_op_digits<kDigitsSteep> : k_op_digits<kDigits>,
                       dim3(kNumOffsets * nrb), dim3(256), 0, nullptr, tab, nrb, nks, nkc, dig,
                       kexp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  hipFree(tab);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? EIFMM_ENOMEM : EIFMM_EHIP;
  }
  return EIFMM_OK;
}

}  // namespace eifmm
