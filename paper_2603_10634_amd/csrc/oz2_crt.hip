// Chinese-remainder reconstruction and inverse scaling (eqs.
// CRT_finalreduction, inversescaling), fused with alpha/beta.
//
// Per output entry (i, j): the residues u_l = C'_l (symmetric range) from the
// int16 planes; S = sum_l w_l u_l in limbs held as exact FP64 integers; C' = S
// mods P, the representative in [-floor(P/2), P - 1 - floor(P/2)], which is
// the product itself by condition (3).  Then Chat = C' 2^-(log2 mu_i + log2
// nu_j) rounded once to nearest-even, including gradual underflow.  C =
// RN(alpha Chat) (+ RN(beta C_in)).
//
// Nearly every entry is decided by crt_rn (balanced 40-bit limbs, sums of
// doubles with their exact errors); the others (ties where P >= 2^96, tiny C'
// against P, subnormal results) by 32-bit limbs and integer rounding (crt_exact).
//
// A thread computes two consecutive rows of a column, so that the planes are
// read 4 bytes per lane, a wave 64 rows x 2 columns (outputs with few rows
// leave few threads idle).
//
// Bound by HBM: 2 N + 8 bytes per output.  8192^2 outputs, N = 12: 0.41 ms (5.2
// TB/s); 16384^2: 1.57 ms (0.455 and 1.80 through the caches).  With 32-bit limbs,
// a borrow chain and integer rounding for every entry it was bound by vector
// issue, 218 instructions per output against about 120: 0.58 and 2.20 ms.
#include <string.h>

#include "oz2_crt_math.h"
#include "oz2_internal.h"

namespace oz2 {

namespace {

// Sum over the copies of the planes (k parts of the products) of entry `e` of
// modulus l, reduced to |u| <= p / 2 + 1 (|sum| < 2^13: the float quotient is
// within one).
__device__ __forceinline__ int residue_at(const int16_t *__restrict__ pl, int64_t e, int l,
                                          int64_t pstride, int64_t cstride, int parts,
                                          CTables *tab) {
  int sum = pl[e + l * pstride];
  if (parts > 1) {
    for (int c = 1; c < parts; ++c) sum += pl[e + l * pstride + c * cstride];
    const int p = tab->p[l];
    sum -= p * (int)rintf((float)sum * tab->inv_p[l]);
  }
  return sum;
}

// RN(C' 2^-t) of entry e through 32-bit limbs, whatever the value.
template <int LL>
__device__ __noinline__ double crt_exact(const int16_t *__restrict__ pl, int64_t e, int N,
                                         int64_t pstride, int parts,
                                         const Tables *__restrict__ tab, int t) {
  double acc[LL];
#pragma unroll
  for (int q = 0; q < LL; ++q) acc[q] = 0.0;
  for (int l = 0; l < N; ++l) {
    const double ud = (double)residue_at(pl, e, l, pstride, N * pstride, parts,
                                         (CTables *)(uintptr_t)tab);
#pragma unroll
    for (int q = 0; q < LL; ++q) acc[q] = fma(tab->wd[l][q], ud, acc[q]);
  }
  uint32_t mag[LL];
  const bool negative = crt_reduce<LL>(acc, tab, mag);
  const double v = scaled_rn<LL>(mag, t);
  return negative ? -v : v;
}

typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));

// Rows i, i + 1 (i even) of column j.  LL 32-bit limbs of P, L wide ones; NF >
// 0: the number of moduli is the compile-time NF (no per-modulus branches); NF
// = 0: N at run time.
template <int LL, int L, int NF>
__device__ __forceinline__ void crt_pair(const Problem &P, const Tables *__restrict__ tabp,
                                         int64_t i, int64_t j) {
  CTables *tab = (CTables *)(uintptr_t)tabp;
  const int N = NF > 0 ? NF : P.g.N;
  const int64_t mp = P.g.mp, pstride = mp * P.g.np, lineB = P.w.lineB;
  const int parts = P.parts;
  const int16_t *pl = P.w.planes + j * mp + i;
  // every modulus is requested before the first is used
  uint32_t uu[kMaxN];
  const int16_t *ql = pl;
#pragma unroll
  for (int l = 0; l < (NF > 0 ? NF : kMaxN); ++l)
    if (l < N) {
      uu[l] = __builtin_nontemporal_load((const uint32_t *)ql);
      ql += pstride;
    }
  const uint2 fl = *(const uint2 *)(P.w.flags + i);
  const int2 si = *(const int2 *)(P.w.shift + i);
  const uint32_t fj = P.w.flags[lineB + j];
  const int sj = P.w.shift[lineB + j];
  if (parts > 1) {
#pragma unroll
    for (int l = 0; l < (NF > 0 ? NF : kMaxN); ++l)
      if (l < N) {
        int s0 = (int16_t)(uu[l] & 0xFFFFu), s1 = (int)uu[l] >> 16;
        const int16_t *cp = pl + l * pstride;
        for (int c = 1; c < parts; ++c) {
          cp += N * pstride;
          const uint32_t x = *(const uint32_t *)cp;
          s0 += (int16_t)(x & 0xFFFFu);
          s1 += (int)x >> 16;
        }
        const int p = tab->p[l];
        s0 -= p * (int)rintf((float)s0 * tab->inv_p[l]);
        s1 -= p * (int)rintf((float)s1 * tab->inv_p[l]);
        uu[l] = ((uint32_t)s0 & 0xFFFFu) | ((uint32_t)s1 << 16);
      }
  }
  double cP[L];
#pragma unroll
  for (int q = 0; q < L; ++q) cP[q] = tab->cP[q];
  const double inv_P = tab->inv_P_d, crt_fast = tab->crt_fast;
  double acc[2][L];
#pragma unroll
  for (int q = 0; q < L; ++q) acc[0][q] = acc[1][q] = 0.0;
#pragma unroll
  for (int l = 0; l < (NF > 0 ? NF : kMaxN); ++l)
    if (l < N) {
      const double u0 = (double)(int16_t)(uu[l] & 0xFFFFu), u1 = (double)((int)uu[l] >> 16);
#pragma unroll
      for (int q = 0; q < L; ++q) {
        const double w = tab->cw[l][q];
        acc[0][q] = fma(w, u0, acc[0][q]);
        acc[1][q] = fma(w, u1, acc[1][q]);
      }
    }
  double out[2];
  const int t[2] = {si.x + sj, si.y + sj};
  constexpr bool exact = LL <= 3;  // (P < 2^96 in LL 40-bit limbs)
  bool ok = crt_rn<L, exact>(acc[0], cP, inv_P, crt_fast, t[0], out[0]);
  ok = crt_rn<L, exact>(acc[1], cP, inv_P, crt_fast, t[1], out[1]) && ok;
  if (!ok)
#pragma unroll 1
    for (int z = 0; z < 2; ++z) {
      const double v = crt_exact<LL>(pl, z, N, pstride, parts, tabp, z ? t[1] : t[0]);
      out[0] = z ? out[0] : v;
      out[1] = z ? v : out[1];
    }
  const double nan = __longlong_as_double(0x7FF8000000000000ll);
  if ((fl.x | fj) & kNonFinite) out[0] = nan;
  if ((fl.y | fj) & kNonFinite) out[1] = nan;
  const double alpha = P.alpha, beta = P.beta;
  double *C = P.C + i + j * P.ldc;
  d2 r = {__dmul_rn(alpha, out[0]), __dmul_rn(alpha, out[1])};
  if (i + 1 < P.g.m) {
    if (beta != 0.0) {
      const d2 c = *(const d2 *)C;
      r[0] = __dadd_rn(r[0], __dmul_rn(beta, c[0]));
      r[1] = __dadd_rn(r[1], __dmul_rn(beta, c[1]));
    }
    if (P.stream_c) {
      // (the empty statements keep the two stores from being merged into one
      // ordinary one)
      asm volatile("");
      __builtin_nontemporal_store(r, (d2 *)C);
      asm volatile("");
    } else {
      *(d2 *)C = r;
    }
  } else {
    if (beta != 0.0) r[0] = __dadd_rn(r[0], __dmul_rn(beta, C[0]));
    C[0] = r[0];
  }
}

template <int LL, int L, int NF, bool GROUPED>
__global__ __launch_bounds__(256) void k_crt(Problem P1, Group G) {
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims c = decode_block(family_dims(kFamCrt, P), local);
  const int64_t i = c.x * 64 + 2 * (threadIdx.x & 31);
  const int64_t j = c.y * 8 + (threadIdx.x >> 5);
  if (j >= P.g.n || i >= P.g.m) return;
  crt_pair<LL, L, NF>(P, tables_of<GROUPED>(P1, G), i, j);
}

__global__ void k_scal(int64_t m, double beta, double *__restrict__ C, int64_t ldc) {
  const int64_t nbx = (m + 255) / 256;
  const int64_t i = (int64_t)(blockIdx.x % nbx) * 256 + threadIdx.x;
  const int64_t j = blockIdx.x / nbx;
  if (i >= m) return;
  double *c = C + i + j * ldc;
  *c = beta == 0.0 ? 0.0 : __dmul_rn(beta, *c);
}

}  // namespace

hipError_t launch_crt_family(const Problem *P, const Group *G, int shape_limbs, int N,
                             hipStream_t st) {
  const int limbs = shape_limbs & 0xFF, wide = shape_limbs >> 8;
  const bool grouped = G != nullptr;
  Problem p1;
  Group g1;
  memset(&p1, 0, sizeof(p1));
  memset(&g1, 0, sizeof(g1));
  if (grouped)
    g1 = *G;
  else
    p1 = *P;
  const int64_t blocks = grouped ? G->total : family_blocks(kFamCrt, *P);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), blk(256);
#define OZ2_CRT_LAUNCH(LL, L, NF)                                             \
  if (grouped)                                                                \
    hipLaunchKernelGGL((k_crt<LL, L, NF, true>), grid, blk, 0, st, p1, g1);   \
  else                                                                        \
    hipLaunchKernelGGL((k_crt<LL, L, NF, false>), grid, blk, 0, st, p1, g1);
  // the moduli counts of full accuracy get kernels without per-modulus
  // branches (three wide limbs: P < 2^121, Tables::wlimbs)
  const int shape = wide == 3 && limbs == 4 && N >= 12 && N <= 15   ? 300 + N
                    : wide == 4 && limbs == 5 && N >= 14 && N <= 17 ? 400 + N
                                                                    : 0;
  switch (shape) {
    case 312: OZ2_CRT_LAUNCH(4, 3, 12) return hipGetLastError();
    case 313: OZ2_CRT_LAUNCH(4, 3, 13) return hipGetLastError();
    case 314: OZ2_CRT_LAUNCH(4, 3, 14) return hipGetLastError();
    case 315: OZ2_CRT_LAUNCH(4, 3, 15) return hipGetLastError();
    case 414: OZ2_CRT_LAUNCH(5, 4, 14) return hipGetLastError();
    case 415: OZ2_CRT_LAUNCH(5, 4, 15) return hipGetLastError();
    case 416: OZ2_CRT_LAUNCH(5, 4, 16) return hipGetLastError();
    case 417: OZ2_CRT_LAUNCH(5, 4, 17) return hipGetLastError();
    default: break;
  }
  if (limbs == 4 && wide == 3) {
    OZ2_CRT_LAUNCH(4, 3, 0)
    return hipGetLastError();
  }
#define OZ2_CRT_CASE(LL)                  \
  case LL:                                \
    OZ2_CRT_LAUNCH(LL, wide_limbs(LL), 0) \
    break;
  switch (limbs) {
    OZ2_CRT_CASE(1)
    OZ2_CRT_CASE(2)
    OZ2_CRT_CASE(3)
    OZ2_CRT_CASE(4)
    OZ2_CRT_CASE(5)
    OZ2_CRT_CASE(6)
    OZ2_CRT_CASE(7)
    OZ2_CRT_CASE(8)
    OZ2_CRT_CASE(9)
    OZ2_CRT_CASE(10)
    default:
      return hipErrorInvalidValue;
  }
#undef OZ2_CRT_CASE
#undef OZ2_CRT_LAUNCH
  return hipGetLastError();
}

hipError_t launch_scal(int64_t m, int64_t n, double beta, double *C, int64_t ldc, hipStream_t st) {
  if (m == 0 || n == 0) return hipSuccess;
  const int64_t blocks = (m + 255) / 256 * n;
  if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scal, dim3((unsigned)blocks), dim3(256), 0, st, m, beta, C, ldc);
  return hipGetLastError();
}

}  // namespace oz2
