// Scale exponents (Section III-E).
//
// Fast mode takes r_i from the Cauchy-Schwarz inequality instead: the squared
// norm of row i of Abar, summed exactly by the quantization pass; every line
// is then finalized from that exact value.  The accurate mode follows.
//
// For each row i of op(A) let r_i be the maximum over j of the bound product
// (Abar Bbar)_ij, and likewise c_j for the columns of op(B).  The scale
// exponent is e_i = max{e : 2^(2e+1) r_i <= P - 1}, giving log2 mu_i =
// log2 mu'_i + e_i; this makes 2 mu_i nu_j sum |a||b| < P (condition (3)),
// because each bound entry is at most sqrt(r_i c_j).
//
// The bound product runs on FP8 MFMA, so the computed maxima r'_i carry an
// error; the paper bounds it by (k - 1) 2^-24 (FP32 summation rounded to
// nearest), which gfx950's FP8 MFMA does not meet.  Each line is therefore
// decided from a window that holds the exact maximum under a stated worst
// case of the MFMA's accumulation (oz2_window.h).  When the whole window gives
// the same exponent, it is the exponent of the exact r_i.  Lines whose window
// straddles a threshold are recomputed exactly: Abar and Bbar are multiples
// of 2^-9 up to 256, so 2^18 (Abar Bbar)_ij is an integer below 2^52 for
// k <= 2^18 and is summed exactly in FP64.  The result is a
// deterministic function of the inputs, independent of the MFMA's summation
// order.  (Integer digit products stay exact: every product is an integer of
// magnitude <= 256, far inside the 2^-13 window, and every partial sum is at
// most 2^24.)
#include <string.h>

#include "oz2_device.h"
#include "oz2_internal.h"
#include "oz2_window.h"

namespace oz2 {

namespace {

template <bool GROUPED>
__global__ __launch_bounds__(256) void k_scale_decide(Problem P1, Group G) {
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const int64_t L = local * 256 + threadIdx.x;
  const int64_t lines = P.g.mp + P.g.np;
  if (L >= lines) return;
  const Work &w = P.w;
  const float r = __uint_as_float(w.rmax[L]);
  int ev = 0;
  if (r > 0.0f && !(w.flags[L] & kZeroLine)) {
    int e_small, e_large;
    window_exponents((double)r, P.g.kp, P.bparts, tables_of<GROUPED>(P1, G)->D, &e_small,
                     &e_large);
    ev = e_small;
    if (e_small != e_large) {
      // rows of op(A) from the front of the list, columns of op(B) from the back
      if (L < P.g.mp)
        w.amb[2 + atomicAdd(&w.amb[0], 1u)] = (uint32_t)L;
      else
        w.amb[1 + lines - atomicAdd(&w.amb[1], 1u)] = (uint32_t)L;
      w.flags[L] |= kFixup;
    }
  }
  w.e[L] = ev;
  w.shift[L] = 7 - w.E[L] + ev;  // (an undecided line's is replaced with its residues)
}

// Exact maxima of the bound product over the flagged lines, on FP64 matrix
// instructions: products of entries of Abar and Bbar are multiples of 2^-18 up
// to 2^16, so every partial sum over k <= 2^18 is an integer below 2^52 times
// 2^-18 and exact in any order.  An item is 16 flagged lines of a side (rows of
// op(A), columns of op(B): the two ends of the list) against 16 partner lines,
// one wave; the 64 k of a k-block are summed in 16 steps of 4, step s taking
// byte s of each lane's 16 (lane group lane / 16 holds k 16 (lane / 16) ..
// + 15 of its line, on both sides).  The partners are the instruction's rows,
// so a lane's four sums all belong to flagged line lane % 16, whatever its
// rows; their maximum over the lanes goes to rfix (2^18 x the exact maximum) by
// an atomic maximum.  Each of the problem's nblk one-wave workgroups walks
// items blk, blk + nblk, ...
//
// Loads run four k-blocks ahead: a wave has no other way to hide them, and
// the matrix instructions and the conversions (24 per 16 bytes) take turns.
// 16384 x 16384 x 1024 (59 lines flagged), with k_scale_decide: 362 -> 150 us
// against pairs of lines in LDS, a table lookup per partner byte and FP64
// multiply-adds; 48 products of 192 x 224 x 160 .. 1344: 77 -> 53 us.
typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kFixG = 16;  // flagged lines and partners per item

// Sixteen E4M3 codes as doubles.
__device__ __forceinline__ void decode16(const uint4 &w, double (&x)[16]) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)u[q], false);
    const v2f hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)u[q], true);
    x[4 * q] = (double)lo[0];
    x[4 * q + 1] = (double)lo[1];
    x[4 * q + 2] = (double)hi[0];
    x[4 * q + 3] = (double)hi[1];
  }
}

__device__ __forceinline__ void scale_fixup(const uint8_t *__restrict__ Abar,
                                            const uint8_t *__restrict__ Bbar, int64_t mp,
                                            int64_t np, int64_t kp,
                                            const uint32_t *__restrict__ amb,
                                            uint64_t *__restrict__ rfix, int64_t blk,
                                            int64_t nblk) {
  const int lane = threadIdx.x, row = lane & 15, grp = lane >> 4;
  const int64_t lines = mp + np;
  const int64_t countA = amb[0], countB = amb[1];
  const int64_t groupsA = (countA + kFixG - 1) / kFixG, groupsB = (countB + kFixG - 1) / kFixG;
  // partners: the columns of op(B) for rows of op(A), and the other way
  const int64_t chunksA = np / kFixG, chunksB = mp / kFixG;
  const int64_t itemsA = groupsA * chunksA, items = itemsA + groupsB * chunksB;
  for (int64_t it = blk; it < items; it += nblk) {
    const bool rows = it < itemsA;  // flagged rows of op(A) against the columns of op(B)
    const int64_t r = rows ? it : it - itemsA;
    const int64_t groups = rows ? groupsA : groupsB;
    const int64_t c = r / groups, g = r - c * groups;
    const int64_t count = rows ? countA : countB;
    const uint8_t *own_op = rows ? Abar : Bbar, *part_op = rows ? Bbar : Abar;
    const int64_t nown = rows ? mp : np, npart = rows ? np : mp;
    const int64_t e = g * kFixG + row;  // this lane's flagged line, if any
    const bool have = e < count;
    const int64_t L = have ? (int64_t)amb[rows ? 2 + e : 1 + lines - e] : 0;
    const uint8_t *own = own_op + (have ? L - (rows ? 0 : mp) : 0) * 64 + 16 * grp;
    const uint8_t *part = part_op + (c * kFixG + row) * 64 + 16 * grp;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
    // four k-blocks (kp is a multiple of 256), the next four loaded meanwhile
    uint4 wo[4], wp[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      wo[q] = *(const uint4 *)(own + q * nown * 64);
      wp[q] = *(const uint4 *)(part + q * npart * 64);
    }
    for (int64_t kb = 256; kb <= kp; kb += 256) {
      own += nown * 256;
      part += npart * 256;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double xo[16], xp[16];
        decode16(wo[q], xo);
        decode16(wp[q], xp);
        if (kb < kp) {
          wo[q] = *(const uint4 *)(own + q * nown * 64);
          wp[q] = *(const uint4 *)(part + q * npart * 64);
        }
#pragma unroll
        for (int s = 0; s < 16; ++s)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xp[s], xo[s], acc, 0, 0, 0);
      }
    }
    double m = fmax(fmax(acc[0], acc[1]), fmax(acc[2], acc[3]));
    m = fmax(m, __shfl_xor(m, 16, 64));
    m = fmax(m, __shfl_xor(m, 32, 64));
    const uint64_t m18 = (uint64_t)(m * 0x1p18);
    if (lane < kFixG && have && m18)
      atomicMax((unsigned long long *)&rfix[L], (unsigned long long)m18);
  }
}

template <bool GROUPED>
__global__ __launch_bounds__(64) void k_scale_fixup(Problem P1, Group G) {
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims d = family_dims(kFamFixup, P);
  scale_fixup(P.w.Abar, P.w.Bbar, P.g.mp, P.g.np, P.g.kp, P.w.amb, P.w.rfix, local, d.x);
}

}  // namespace

hipError_t launch_scale_family(int fam, const Problem *P, const Group *G, hipStream_t st) {
  const bool grouped = G != nullptr;
  Problem p1;
  Group g1;
  memset(&p1, 0, sizeof(p1));
  memset(&g1, 0, sizeof(g1));
  if (grouped)
    g1 = *G;
  else
    p1 = *P;
  const int64_t blocks = grouped ? G->total : family_blocks(fam, *P);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), blk(fam == kFamFixup ? 64 : 256);
#define OZ2_S(KER)                                             \
  if (grouped)                                                 \
    hipLaunchKernelGGL((KER<true>), grid, blk, 0, st, p1, g1); \
  else                                                         \
    hipLaunchKernelGGL((KER<false>), grid, blk, 0, st, p1, g1);
  switch (fam) {
    case kFamDecide: OZ2_S(k_scale_decide) break;
    case kFamFixup: OZ2_S(k_scale_fixup) break;
    default: return hipErrorInvalidValue;
  }
#undef OZ2_S
  return hipGetLastError();
}

}  // namespace oz2
