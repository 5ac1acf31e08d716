// Quantization passes over the FP64 inputs (HBM-bound):
//  - line maxima of op(A) rows / op(B) columns (for mu', nu', eq. def:mu'nu'),
//  - the round-up FP8 bound operands Abar, Bbar (Section III-E), or in fast
//    mode the squared norms of their lines (Cauchy-Schwarz bound); both steps in
//    one pass for lines of up to 8192 k,
//  - the residues of A', B' for every modulus, split into FP8 digits
//    (eqs. def:A', def:B', CRTmatmul; digit splits of Sections III-B..III-D).
// Outputs are k-blocked (kblocked in oz2_internal.h) or, the slices of
// k_residue6, in its fragment order; zero padded.
#include <string.h>

#include "oz2_device.h"
#include "oz2_internal.h"
#include "oz2_window.h"

namespace oz2 {

namespace {

constexpr uint64_t kAbsMask = 0x7FFFFFFFFFFFFFFFull;
constexpr uint64_t kInfBits = 0x7FF0000000000000ull;
// class mask of the finite nonzero doubles (negative and positive normal and
// subnormal numbers)
constexpr int kFiniteNonzero = 0x198;

__device__ __forceinline__ void fill_zero(uint32_t *p, int64_t count, int64_t blk,
                                          int64_t nblk) {
  for (int64_t i = blk * 256 + threadIdx.x; i < count; i += nblk * 256) p[i] = 0u;
}

constexpr int kLmaxU = 8;  // independent loads per trip of the line-maximum loops

// Maxima of |x| over finite entries, per line; non-finite entries flag the line.
// Lines with contiguous k: one wave per line and k-chunk.
__device__ __forceinline__ void line_max_kcontig(const Operand &op, const LmaxShape &sh,
                                                 int64_t bx, int64_t by, uint64_t *amax,
                                                 uint32_t *flags) {
  const int lane = threadIdx.x & 63;
  const int64_t r = bx * 4 + (threadIdx.x >> 6);
  if (r >= op.lines) return;
  const int64_t h0 = by * sh.hchunk;
  const int64_t h1 = min(op.k, h0 + sh.hchunk);
  const double *row = op.ptr + r * op.sr;
  uint64_t m = 0;
  int bad = 0;
  int64_t h = h0 + lane;
  // kLmaxU loads in flight per trip, then a remainder of single loads
  for (; h + 64 * (kLmaxU - 1) < h1; h += 64 * kLmaxU) {
    uint64_t b[kLmaxU];
#pragma unroll
    for (int u = 0; u < kLmaxU; ++u)
      b[u] = (uint64_t)__double_as_longlong(row[h + 64 * u]) & kAbsMask;
#pragma unroll
    for (int u = 0; u < kLmaxU; ++u) {
      if (b[u] >= kInfBits)
        bad = 1;
      else
        m = b[u] > m ? b[u] : m;
    }
  }
  for (; h < h1; h += 64) {
    uint64_t b = (uint64_t)__double_as_longlong(row[h]) & kAbsMask;
    if (b >= kInfBits)
      bad = 1;
    else
      m = b > m ? b : m;
  }
  for (int off = 32; off > 0; off >>= 1) {
    uint64_t o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  bad = __any(bad);
  if (lane == 0) {
    if (m) atomicMax((unsigned long long *)&amax[r], (unsigned long long)m);
    if (bad) atomicOr(&flags[r], kNonFinite);
  }
}

// Lines contiguous in memory: one thread per line, k split over blocks.
__device__ __forceinline__ void line_max_lcontig(const Operand &op, const LmaxShape &sh,
                                                 int64_t bx, int64_t by, uint64_t *amax,
                                                 uint32_t *flags) {
  const int64_t r = bx * 256 + threadIdx.x;
  if (r >= op.lines) return;
  const int64_t h0 = by * sh.hchunk;
  const int64_t h1 = min(op.k, h0 + sh.hchunk);
  uint64_t m = 0;
  int bad = 0;
  int64_t h = h0;
  for (; h + kLmaxU <= h1; h += kLmaxU) {
    uint64_t b[kLmaxU];
#pragma unroll
    for (int u = 0; u < kLmaxU; ++u)
      b[u] = (uint64_t)__double_as_longlong(op.ptr[r + (h + u) * op.sh]) & kAbsMask;
#pragma unroll
    for (int u = 0; u < kLmaxU; ++u) {
      if (b[u] >= kInfBits)
        bad = 1;
      else
        m = b[u] > m ? b[u] : m;
    }
  }
  for (; h < h1; ++h) {
    uint64_t b = (uint64_t)__double_as_longlong(op.ptr[r + h * op.sh]) & kAbsMask;
    if (b >= kInfBits)
      bad = 1;
    else
      m = b > m ? b : m;
  }
  if (m) atomicMax((unsigned long long *)&amax[r], (unsigned long long)m);
  if (bad) atomicOr(&flags[r], kNonFinite);
}

template <bool GROUPED>
__global__ __launch_bounds__(256) void k_fill(Problem P1, Group G) {
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims d = family_dims(kFamFill, P);
  fill_zero(P.w.zero, P.w.zero_words, local, d.x);
}

// Both operands of a problem in one launch: the blocks of op(A)'s lines (0 ..
// mp - 1 of the per-line vectors), then those of op(B)'s (from mp).  A pass over
// a small operand costs its launch (256^3: 4-5 us each), whichever the size.
__device__ __forceinline__ Operand operand(const Problem &P, bool b) {
  Operand o;
  o.ptr = b ? P.B.ptr : P.A.ptr;
  o.lines = b ? P.B.lines : P.A.lines;
  o.k = b ? P.B.k : P.A.k;
  o.sr = b ? P.B.sr : P.A.sr;
  o.sh = b ? P.B.sh : P.A.sh;
  return o;
}

template <bool GROUPED>
__global__ __launch_bounds__(256) void k_line_max(Problem P1, Group G) {
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const LmaxShape sa = lmax_shape(P.A);
  const bool side = local >= sa.gx * sa.splits;
  if (side) local -= sa.gx * sa.splits;
  const Operand op = operand(P, side);
  const int64_t base = side ? P.g.mp : 0;
  const LmaxShape sh = lmax_shape(op);
  const int64_t by = (uint32_t)local / (uint32_t)sh.gx, bx = local - by * sh.gx;
  if (op.sh == 1)
    line_max_kcontig(op, sh, bx, by, P.w.amax + base, P.w.flags + base);
  else
    line_max_lcontig(op, sh, bx, by, P.w.amax + base, P.w.flags + base);
}

// Quantization tiles: 16 lines x 128 k per workgroup of 256 threads; thread t
// owns line t / 16 and the 8 consecutive k (t % 16) * 8 .. + 7, so a line's
// bytes of a tile leave as one 128-byte segment per output slice.  Small
// tiles and 8 inputs per thread keep the register and LDS footprint low, so
// many waves stream through each CU.  The FP64
// tile is staged in LDS to read along whichever dimension is contiguous;
// element h of a row sits at h + h / 16 (one pad double per 16) so that the
// threads of one read (same q, consecutive t) fall into different banks.
constexpr int kRowLd = kQK + kQK / 16 + 1;   // 137 doubles per staged row

__device__ __forceinline__ int tile_at(int rr, int hh) { return rr * kRowLd + hh + (hh >> 4); }

template <bool LCONTIG, int QL>
__device__ __forceinline__ void load_tile(const double *__restrict__ x, int64_t lines, int64_t k,
                                          int64_t sr, int64_t sh, int64_t r0, int64_t h0,
                                          double *tile) {
#pragma unroll
  for (int q = 0; q < QL * kQK / 256; ++q) {
    const int idx = threadIdx.x + 256 * q;
    const int rr = LCONTIG ? (idx % QL) : (idx >> 7);
    const int hh = LCONTIG ? (idx / QL) : (idx & 127);
    const int64_t r = r0 + rr, h = h0 + hh;
    double v = 0.0;
    if (r < lines && h < k) v = x[r * sr + h * sh];
    tile[tile_at(rr, hh)] = v;
  }
}

template <int QL = kQL>
__device__ __forceinline__ void stage_tile(const Operand &op, int64_t r0, int64_t h0,
                                           double *tile) {
  if (op.sr == 1)
    load_tile<true, QL>(op.ptr, op.lines, op.k, op.sr, op.sh, r0, h0, tile);
  else
    load_tile<false, QL>(op.ptr, op.lines, op.k, op.sr, op.sh, r0, h0, tile);
}

// FP8 round-up bound operand of one tile (lines r0.., k h0..).
__device__ __forceinline__ void bound_operand_tile(const Operand &op, int64_t lines_pad,
                                                   int64_t r0, int64_t h0, const uint64_t *amax,
                                                   int32_t *E, uint32_t *flags, uint8_t *bar,
                                                   double *tile) {
  stage_tile(op, r0, h0, tile);
  __syncthreads();
  const int rl = threadIdx.x >> 4, b = threadIdx.x & 15;
  const int64_t r = r0 + rl;
  const uint64_t am = r < op.lines ? amax[r] : 0ull;
  const int Er = am ? ufp_exponent(am) : 0;
  if (h0 == 0 && b == 0) {
    E[r] = Er;
    if (am == 0) flags[r] |= kZeroLine;
  }
  const int sh7 = 7 - Er;  // mu' = 2^(7 - E)
  uint32_t packed[2];
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    uint32_t word = 0;
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const double v = tile[tile_at(rl, b * 8 + w * 4 + z)];
      const uint32_t code =
          __builtin_amdgcn_class(v, kFiniteNonzero) ? e4m3_round_up(v, sh7) : 0u;
      word |= code << (8 * z);
    }
    packed[w] = word;
  }
  *(uint2 *)(bar + kblocked(r, h0 + b * 8, lines_pad)) = make_uint2(packed[0], packed[1]);
}

template <bool GROUPED>
__global__ __launch_bounds__(256) void k_bound_operand(Problem P1, Group G) {
  __shared__ double tile[kQL * kRowLd];
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims c = decode_block(family_dims(kFamBar, P), local);
  const int64_t r0 = c.x * kQL, by = c.y;
  const bool side = r0 >= P.g.mp;
  const int64_t base = side ? P.g.mp : 0;
  bound_operand_tile(operand(P, side), side ? P.g.np : P.g.mp, r0 - base, by * kQK,
                     P.w.amax + base, P.w.E + base, P.w.flags + base,
                     side ? P.w.Bbar : P.w.Abar, tile);
}

// Fast mode: 2^18 x the squared Euclidean norm of every line of the round-up
// bound operand over one tile, added to norm[r] (Section III-E, the
// Cauchy-Schwarz bound; with r_i, c_j these norms, the bound product obeys
// (Abar Bbar)_ij <= sqrt(r_i c_j)).  Abar is not stored.  Each 2^9 Abar is an
// integer of at most 2^17, so the sums are exact 64-bit integers (at most
// 2^52 for k <= 2^18) and do not depend on the order of the additions.
// Every line is flagged to take its exponent from this exact value.
__device__ __forceinline__ void bound_norm_tile(const Operand &op, int64_t r0, int64_t h0,
                                                const uint64_t *amax, int32_t *E,
                                                uint32_t *flags, uint64_t *norm,
                                                double *tile) {
  stage_tile(op, r0, h0, tile);
  __syncthreads();
  const int rl = threadIdx.x >> 4, b = threadIdx.x & 15;
  const int64_t r = r0 + rl;
  const uint64_t am = r < op.lines ? amax[r] : 0ull;
  const int Er = am ? ufp_exponent(am) : 0;
  if (h0 == 0 && b == 0) {
    E[r] = Er;
    flags[r] |= am ? kFixup : (kFixup | kZeroLine);
  }
  const int sh7 = 7 - Er;  // mu' = 2^(7 - E)
  uint64_t sum = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const double v = tile[tile_at(rl, b * 8 + q)];
    const uint32_t q9 =
        __builtin_amdgcn_class(v, kFiniteNonzero) ? e4m3_q9(e4m3_round_up(v, sh7)) : 0u;
    sum += (uint64_t)q9 * q9;
  }
  // the 16 threads of a line are 16 consecutive lanes
  sum += __shfl_xor(sum, 1, 64);
  sum += __shfl_xor(sum, 2, 64);
  sum += __shfl_xor(sum, 4, 64);
  sum += __shfl_xor(sum, 8, 64);
  if (b == 0 && sum) atomicAdd((unsigned long long *)&norm[r], (unsigned long long)sum);
}

template <bool GROUPED>
__global__ __launch_bounds__(256) void k_bound_norm(Problem P1, Group G) {
  __shared__ double tile[kQL * kRowLd];
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims c = decode_block(family_dims(kFamNorm, P), local);
  const int64_t r0 = c.x * kQL, by = c.y;
  const bool side = r0 >= P.g.mp;
  const int64_t base = side ? P.g.mp : 0;
  bound_norm_tile(operand(P, side), r0 - base, by * kQK, P.w.amax + base, P.w.E + base,
                  P.w.flags + base, P.w.rfix + base, tile);
}

// ---- maxima and bound operands in one pass ----
//
// A workgroup of two groups of 256 threads holds 16 whole lines, a group every
// second tile of 128 k, so that the inputs are read once and nothing has to be
// cleared beforehand.  What the bound operand needs of a value until its line's
// maximum is known are 16 bits: exponent and three mantissa bits, with one bit
// for whether anything follows (rounding up asks no more).  The 8 values of a
// thread and tile are 4 registers, T tiles per group.  A subnormal value keeps
// fewer mantissa bits than that: scaled, it is below 2^-9 and rounds up to it
// whatever its bits while the line's maximum is at least 2^kDeep; workgroups
// with a smaller maximum read their lines again.
//
// Bound by memory, and by the latency of its T loads in turn where there are few
// lines.  Both operands, against clearing, maxima and bound operand in three
// launches: 8192^3 480 -> 333 us (3.6 TB/s), 4096^3 136 -> 88, 16384 x 16384 x
// 1024 130 -> 72, 3000 x 2000 x 256 17.7 -> 9.4, 256^3 14.4 -> 7.2.  Four groups
// (one workgroup per CU) reach 370 us at 8192^3.  512 products of 64 .. 4096 with
// every line running the trips of the longest k: 4.5 ms, its own: 2.3.
constexpr int kLinesG = 2;  // groups of 256 threads
constexpr int kDeep = -1006;

// Exponent, three mantissa bits and the bit for the rest (of a non-finite value
// 0x7FF0 or more).
__device__ __forceinline__ uint32_t line_code(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t hi = (uint32_t)(b >> 32);
  return (hi >> 16 & 0x7FFFu) | (((hi << 16) | (uint32_t)b) != 0 ? 1u : 0u);
}

// e4m3_round_up of a value given by its code, 8 sh = 8 (sh7 - 1023) + 56: above
// 2^-6 the code rounded up to three mantissa bits and rebased, below that
// ceil((1 + m / 16) 2^fl 2^9) with s = -(fl + 5) bits dropped from 16 + m.
__device__ __forceinline__ uint32_t round_up_code(uint32_t c, int rebase) {
  const int normal = (int)((c + 1) >> 1) + rebase;
  const int fl = (int)(c >> 4) + ((rebase - 56) >> 3);
  int s = -5 - fl;
  s = s < 0 ? 0 : s > 8 ? 8 : s;
  const int small = (int)((16u + (c & 15u) + (1u << s) - 1u) >> s);
  const int code = normal < 8 ? small : normal;
  return c ? (uint32_t)code : 0u;
}

template <bool GROUPED, bool NORM, int T>
__global__ __launch_bounds__(256 * kLinesG, T <= 16 ? 4 : 2) void k_lines(Problem P1, Group G) {
  __shared__ double tiles[kLinesG][kQL * kRowLd];
  __shared__ uint64_t red[kLinesG][kQL];
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const bool side = local * kQL >= P.g.mp;
  const int64_t base = side ? P.g.mp : 0, r0 = local * kQL - base;
  const Operand op = operand(P, side);
  const int64_t kp = P.g.kp, lines_pad = side ? P.g.np : P.g.mp;
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;
  const int rl = t >> 4, b = t & 15;
  double *tile = tiles[grp];
  auto first_k = [&](int u) { return (int64_t)kQK * (grp + kLinesG * u); };
  // a thread's 8 values of a tile: of one line at every 16th k, or of every
  // second line at one k; invalid ones read element 0 of the operand instead
  const bool lcontig = op.sr == 1;
  const int dr = lcontig ? 0 : 2, dh = lcontig ? 16 : 0;
  const int64_t rt = r0 + (lcontig ? t & 15 : t >> 7);
  const int ht = lcontig ? t >> 4 : t & 127;
  const int64_t dq = lcontig ? 16 * op.sh : 2 * op.sr;
  const int64_t at = rt * op.sr + ht * op.sh;
  const int lines_left = (int)(op.lines - rt), k = (int)op.k;
  auto valid = [&](int u, int q) {
    return dr * q < lines_left && (int)first_k(u) + ht + dh * q < k;
  };
  double x[8];
  auto load = [&](int u) {
    const int64_t tile0 = at + first_k(u) * op.sh;
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = op.ptr[valid(u, q) ? tile0 + q * dq : 0];
    __builtin_amdgcn_sched_barrier(0);  // (nothing that waits for them in between)
  };
  auto stage = [&](int u) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int idx = t + 256 * q;
      tile[lcontig ? tile_at(idx & 15, idx >> 4) : tile_at(idx >> 7, idx & 127)] =
          valid(u, q) ? x[q] : 0.0;
    }
  };

  uint32_t code[T][4] = {}, top = 0;
  bool bad = false;
  load(0);
#pragma unroll
  for (int u = 0; u < T; ++u) {
    if (kQK * kLinesG * u < kp) {  // (of a batch, T serves its longest k)
      stage(u);
      if (u + 1 < T) load(u + 1);
      __syncthreads();
  #pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t c[2];
  #pragma unroll
        for (int z = 0; z < 2; ++z) {
          c[z] = line_code(tile[tile_at(rl, b * 8 + w * 2 + z)]);
          const bool finite = c[z] < 0x7FF0u;
          bad |= !finite;
          c[z] = finite ? c[z] : 0u;
          top = c[z] > top ? c[z] : top;
        }
        code[u][w] = c[0] | (c[1] << 16);
        // packed here and now: kept as its doubles a tile is 16 registers
        asm volatile("" : "+v"(code[u][w]));
      }
      if (u + 1 < T) __syncthreads();
    }
  }
  // the line's maximum: over its 16 lanes, then over the groups
  top |= bad ? 0x8000u : 0u;
  auto larger = [](uint32_t a, uint32_t o) {
    const uint32_t x = a & 0x7FFFu, y = o & 0x7FFFu;
    return (x > y ? x : y) | ((a | o) & 0x8000u);
  };
  for (int off = 1; off < 16; off <<= 1) top = larger(top, __shfl_xor(top, off, 64));
  if (b == 0) red[grp][rl] = top;
  __syncthreads();
  top = 0;
#pragma unroll
  for (int q = 0; q < kLinesG; ++q) top = larger(top, (uint32_t)red[q][rl]);
  bad = (top & 0x8000u) != 0;
  top &= 0x7FFFu;
  int E = top ? (int)(top >> 4) - 1023 : 0;
  const bool again = __syncthreads_or(top != 0 && E < kDeep);
  auto read = [&](int u) {
    load(u);
    __syncthreads();
    stage(u);
    __syncthreads();
  };
  auto value = [&](int q) {
    const double v = tile[tile_at(rl, b * 8 + q)];
    return __builtin_amdgcn_class(v, kFiniteNonzero) ? v : 0.0;
  };
  if (again) {  // the exponent of a subnormal maximum
    double m = 0.0;
#pragma unroll 1
    for (int u = 0; u < T; ++u) {
      read(u);
      for (int q = 0; q < 8; ++q) m = fmax(m, fabs(value(q)));
    }
    for (int off = 1; off < 16; off <<= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if (b == 0) red[grp][rl] = (uint64_t)__double_as_longlong(m);
    __syncthreads();
    uint64_t am = 0;  // (of non-negative doubles the bits are in order)
    for (int q = 0; q < kLinesG; ++q) am = red[q][rl] > am ? red[q][rl] : am;
    E = am ? ufp_exponent(am) : 0;
  }
  const int64_t L = base + r0 + rl;
  if (grp == 0 && b == 0) {
    P.w.E[L] = E;
    P.w.flags[L] = (bad ? kNonFinite : 0u) | (top ? 0u : kZeroLine) | (NORM ? kFixup : 0u);
    P.w.rmax[L] = 0u;
    if (!NORM) P.w.rfix[L] = 0ull;
    if (local == 0 && t == 0) P.w.amb[0] = P.w.amb[1] = 0u;
  }
  uint8_t *bar = (side ? P.w.Bbar : P.w.Abar) + kblocked(r0 + rl, b * 8, lines_pad);
  uint64_t sum = 0;
  // a tile's bound operand (mu' = 2^(7 - E)) from the codes of its values
  auto put = [&](int64_t h0, auto &&e4m3) {
    if (h0 >= kp) return;
    uint32_t packed[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t e = e4m3(q);
      if (NORM) {
        const uint32_t q9 = e4m3_q9(e);
        sum += (uint64_t)q9 * q9;
      }
      packed[q >> 2] |= e << (8 * (q & 3));
    }
    if (!NORM) *(uint2 *)(bar + h0 * lines_pad) = make_uint2(packed[0], packed[1]);
  };
  if (!again) {
    const int rebase = 8 * (7 - E - 1023) + 56;
#pragma unroll
    for (int u = 0; u < T; ++u) {
      put(first_k(u), [&](int q) {
        return round_up_code(code[u][q >> 1] >> (16 * (q & 1)) & 0xFFFFu, rebase);
      });
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll 1
    for (int u = 0; u < T; ++u) {
      read(u);
      put(first_k(u), [&](int q) {
        const double v = value(q);
        return v != 0.0 ? e4m3_round_up(v, 7 - E) : 0u;
      });
    }
  }
  if (NORM) {
    // 2^18 x the squared norm (see bound_norm_tile)
    for (int off = 1; off < 16; off <<= 1) sum += __shfl_xor(sum, off, 64);
    __syncthreads();
    if (b == 0) red[grp][rl] = sum;
    __syncthreads();
    if (grp == 0 && b == 0) {
      sum = 0;
#pragma unroll
      for (int q = 0; q < kLinesG; ++q) sum += red[q][rl];
      P.w.rfix[L] = sum;
    }
  }
}

// Residues of a' (eq. def:A') for every modulus, split into digits, for one
// tile (lines r0.., k h0..).
//
// Each finite nonzero input is |a| = F 2^(E - 53) with E its frexp exponent
// and F < 2^53 an integer (also for subnormal a); with s = log2 mu_r the
// integer is a' = sign (F 2^t) for t = E - 53 + s > 0, else sign floor(F 2^t)
// (eq. def:A': truncation toward zero).  Per input the signed integer
// x = sign F 2^min(t, 10) (t > 0) or a' (t <= 0) is held exactly in a double
// (|x| < 2^63): x = trunc(a 2^(s - max(t - 10, 0))), where the scaling is
// exact whenever the result is at least 2^-1022 and otherwise is below one in
// magnitude, so that the truncation gives zero either way.  Zero, infinite and
// NaN inputs give x = +0 (their lines are flagged, or their digits are zero).
// One FP64 step serves two consecutive moduli p, p' of one kind (R = p p' <
// 2^21), or one modulus alone (R = p): q = rint(x R^-1) is within
// 2^63 / R 2^-52 = 2^11 / R of x / R (both roundings), so
// |f| = |x - q R| < R / 2 + 2^11 < 2^20 + 2^11, and f is exact in one fused
// multiply-add.  Per modulus, one FP32 step f - p rint(f p^-1) then removes
// the nearest multiple of p: the computed quotient is within
// |f / p| 2^-23 < 1 / (8p) (1 + 2^-9) of f / p (f is exact in FP32), while
// for odd p an integer f / p is at least 1 / (2p) from a tie,
// so the result is exactly in [-(p - 1)/2, (p - 1)/2]; for even p it is
// in [-p/2, p/2] and a tie's +p/2 is moved to -p/2, giving the symmetric
// range [-floor(p/2), ceil(p/2) - 1] in both cases.  Inputs with t > 10 (only
// for large N: t <= e - 45 for the scale exponent e) are multiplied by
// 2^(t - 10) mod p (tables) and reduced by the same FP32 step (products below
// p^2 / 2 < 2^20, exact; quotient error below p 2^-24 < 1 / (2p) for
// p < 2896).  Digits (Sections
// III-B, III-C) are formed in FP32, exact for these small integers, and
// packed to E4M3 two at a time by the hardware conversion (exact: every digit
// has |d| <= 16).  An INT8 modulus (Section II) stores the residue itself,
// in [-128, 127], as one INT8 byte.  The moduli are visited kind by kind
// (squares, then Karatsuba, then INT8), so no loop body branches on the kind.
constexpr int kDirectT = 10;  // powers 2^t applied in FP64 directly

constexpr int kRE = kQK * kQL / 256;  // inputs per thread of a quantization tile (8)

struct ResidueIn {
  double x[kRE];  // sign F 2^min(t, 10) (t > 0) or signed a' (t <= 0), exact, never -0
  int t[kRE];     // t > 10: the power of two t - 10 still to apply, else 0
};

// HUGE: some lane of the wave has t > 10 (a wave-uniform choice of the
// whole modulus loop, so that the common loop carries nothing of the table
// lookup of 2^(t - 10) mod p).
// The FP64 step: f = x - R rint(x R^-1), exact, |f| < 2^20 + 2^11.
__device__ __forceinline__ void fp64_step(const ResidueIn &in, double R, double invR,
                                          float (&f)[kRE]) {
#pragma unroll
  for (int q = 0; q < kRE; ++q) f[q] = (float)fma(-rint(in.x[q] * invR), R, in.x[q]);
}

template <int KIND, bool EVEN, bool HUGE>
__device__ __forceinline__ void modulus_pass(const float (&f)[kRE], const ResidueIn &in,
                                             CTables *tab, int l, uint8_t *dst,
                                             int64_t slice_stride) {
  const int p = tab->p[l];
  const float pf = (float)p;
  const float hif = (float)(p - 1 - (p >> 1));
  const float invpf = tab->inv_p[l];
  float fu[kRE];
#pragma unroll
  for (int q = 0; q < kRE; ++q) fu[q] = fmaf(-rintf(f[q] * invpf), pf, f[q]);
  if (HUGE) {
#pragma unroll
    for (int q = 0; q < kRE; ++q) {
      if (in.t[q] > 0) {
        const float prod = fu[q] * (float)tab->pw[l][in.t[q]];
        fu[q] = fmaf(-rintf(prod * invpf), pf, prod);
      }
    }
  }
  if (EVEN) {
    // a tie leaves +p/2, which belongs to -p/2
#pragma unroll
    for (int q = 0; q < kRE; ++q) fu[q] = fu[q] > hif ? fu[q] - pf : fu[q];
  }
  constexpr int G = kRE / 4;
  int w1[G], w2[G], w3[G];
  if (KIND == 2) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      uint32_t word = 0;
#pragma unroll
      for (int z = 0; z < 4; ++z) word |= ((uint32_t)(int)fu[4 * g + z] & 0xFFu) << (8 * z);
      w1[g] = (int)word;
    }
    *(uint2 *)dst = make_uint2(w1[0], w1[1]);
    return;
  }
  const float sf = (float)tab->s[l], invs = tab->inv_s[l];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float x1[4], x2[4], x3[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const float f = fu[4 * g + z];
      if (KIND == 0) {
        // p = s^2: x1 = round(u / s) (ties away from zero), x2 = u - s x1;
        // for odd s, u / s is never a tie and rint rounds to the nearest
        const float tq = f * invs;
        if (EVEN)
          x1[z] = truncf(tq + copysignf(0.5f, tq)) + 0.0f;  // + 0 turns -0 into +0
        else
          x1[z] = rintf(tq) + 0.0f;
        x2[z] = fmaf(-sf, x1[z], f);
      } else {
        // s = 16: x1 = sign(u) ceil(|u| / 16), x2 = u - 16 x1, x3 = x1 + x2
        x1[z] = copysignf(ceilf(fabsf(f) * 0.0625f), f);
        x2[z] = fmaf(-16.0f, x1[z], f);
        x3[z] = x1[z] + x2[z];
      }
    }
    // the first conversion's old word is a register no longer needed (the
    // residues themselves): its upper half is replaced by the second one
    w1[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x1[0], x1[1], __float_as_int(fu[4 * g]), false);
    w1[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x1[2], x1[3], w1[g], true);
    w2[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x2[0], x2[1], __float_as_int(fu[4 * g + 1]), false);
    w2[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x2[2], x2[3], w2[g], true);
    if (KIND == 1) {
      w3[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x3[0], x3[1], __float_as_int(fu[4 * g + 2]), false);
      w3[g] = __builtin_amdgcn_cvt_pk_fp8_f32(x3[2], x3[3], w3[g], true);
    }
  }
  *(uint2 *)dst = make_uint2(w1[0], w1[1]);
  *(uint2 *)(dst + slice_stride) = make_uint2(w2[0], w2[1]);
  if (KIND == 1) *(uint2 *)(dst + 2 * slice_stride) = make_uint2(w3[0], w3[1]);
}

template <int KIND, bool HUGE>
__device__ __forceinline__ void one_modulus(const float (&f)[kRE], const ResidueIn &in,
                                            CTables *tab, int l, uint8_t *base,
                                            int64_t slice_stride) {
  uint8_t *dst = base + (int64_t)tab->slice0[l] * slice_stride;
  // p is uniform: the parity test is a branch, not a select
  if (tab->p[l] & 1)
    modulus_pass<KIND, false, HUGE>(f, in, tab, l, dst, slice_stride);
  else
    modulus_pass<KIND, true, HUGE>(f, in, tab, l, dst, slice_stride);
}

// The moduli l0 .. l1 - 1 of one kind, two per FP64 step (one per step on
// the rare path with t > 10, which holds more registers).
template <int KIND, bool HUGE>
__device__ __forceinline__ void kind_moduli(const ResidueIn &in, CTables *tab,
                                            int l0, int l1, uint8_t *base, int64_t slice_stride) {
  int l = l0;
  for (; !HUGE && l + 1 < l1; l += 2) {
    float f[kRE];
    fp64_step(in, (double)(tab->p[l] * tab->p[l + 1]), tab->inv_pair[l], f);
    one_modulus<KIND, HUGE>(f, in, tab, l, base, slice_stride);
    one_modulus<KIND, HUGE>(f, in, tab, l + 1, base, slice_stride);
  }
  for (; l < l1; ++l) {
    float f[kRE];
    fp64_step(in, (double)tab->p[l], tab->inv_pd[l], f);
    one_modulus<KIND, HUGE>(f, in, tab, l, base, slice_stride);
  }
}

// The moduli [l0, l1) of the workgroup's group, split by kind.
struct ModuliRange {
  int l0, a, b, l1;  // squares [l0, a), Karatsuba [a, b), INT8 [b, l1)
};

__device__ __forceinline__ ModuliRange moduli_range(const Geometry &g, int64_t z, int64_t groups) {
  ModuliRange r;
  // (a division, of 64 bits above all, is felt in a block of a few microseconds)
  const uint32_t N = (uint32_t)g.N, n = (uint32_t)groups, q = (uint32_t)z;
  r.l0 = n == 1 ? 0 : (int)(q * N / n);
  r.l1 = n == 1 ? g.N : (int)((q + 1) * N / n);
  r.a = max(r.l0, min(r.l1, g.nsq));
  r.b = max(r.l0, min(r.l1, g.nsq + g.nka));
  return r;
}

// Those moduli of one thread's inputs, kind by kind.
template <bool HUGE>
__device__ __forceinline__ void residue_moduli(const ResidueIn &in, CTables *tab,
                                               const ModuliRange &r, uint8_t *base,
                                               int64_t slice_stride) {
  kind_moduli<0, HUGE>(in, tab, r.l0, r.a, base, slice_stride);
  kind_moduli<1, HUGE>(in, tab, r.a, r.b, base, slice_stride);
  kind_moduli<2, HUGE>(in, tab, r.b, r.l1, base, slice_stride);
}

// log2 of the scale of line r (in the per-line vectors of its side, from
// `base`): the stored shift, or for a line with an exact bound (2^18 x the
// line's maximum or norm, < 2^53, in rfix) the one this bound gives, stored by
// the thread with `store` for the CRT and for inspection.  Taking it here
// spares a launch over the lines between the bound and the residues.
__device__ __forceinline__ int final_shift(const Work &w, int64_t base, int64_t r, double D,
                                           bool store, int *e) {
  const int64_t L = base + r;
  if (!(w.flags[L] & kFixup)) {
    *e = w.e[L];
    return w.shift[L];
  }
  const uint64_t r18 = w.rfix[L];
  const int ev = r18 ? exponent_rule(ldexp((double)r18, -18), D) : 0;
  const int s = 7 - w.E[L] + ev;
  if (store) {
    w.e[L] = ev;
    w.shift[L] = s;
  }
  *e = ev;
  return s;
}

__device__ __forceinline__ void residues_tile(const Operand &op, int64_t kp, int64_t lines_pad,
                                              int64_t r0, int64_t h0, const Work &w,
                                              int64_t base_line,
                                              CTables *tab,
                                              const ModuliRange &range,
                                              uint8_t *__restrict__ slices, double *tile) {
  // thread t: line t / 16, the kRE = 8 consecutive k (t % 16) * 8 .. + 7
  const int rl = threadIdx.x >> 4, b = threadIdx.x & 15;
  const int64_t r = r0 + rl;
  // asked for before the tile: after it, one after the other, they are two more
  // latencies of a block that is mostly latency
  const uint32_t flags = w.flags[base_line + r];
  int s = w.shift[base_line + r];  // log2(mu_r)
  stage_tile(op, r0, h0, tile);
  __syncthreads();
  if (flags & kFixup) {
    int e;
    s = final_shift(w, base_line, r, tab->D, h0 == 0 && b == 0, &e);
  }

  ResidueIn in;
  bool huge = false;
#pragma unroll
  for (int q = 0; q < kRE; ++q) {
    const double a = tile[tile_at(rl, b * kRE + q)];
    const bool nz = __builtin_amdgcn_class(a, kFiniteNonzero);
    int t = nz ? __builtin_amdgcn_frexp_exp(a) - 53 + s : 0;
    t = t < kPowT ? t : kPowT - 1;
    const int tt = t > kDirectT ? t - kDirectT : 0;
    // + 0 turns the -0 of a negative input with |a'| < 1 into +0
    const double x = trunc(ldexp(a, s - tt)) + 0.0;
    in.x[q] = nz ? x : 0.0;
    in.t[q] = tt;
    huge |= tt > 0;
  }

  const int64_t slice_stride = lines_pad * kp;
  uint8_t *base = slices + kblocked(r, h0 + b * kRE, lines_pad);
  if (__any(huge))
    residue_moduli<true>(in, tab, range, base, slice_stride);
  else
    residue_moduli<false>(in, tab, range, base, slice_stride);
}

// (single problems only: a batch's slices are in fragment order)  The tables are read
// through the constant address space: the stores of final_shift would otherwise make
// every modulus' constants vector loads, waited for together with the stores before
// them.  op(A)'s tiles first, then op(B)'s, each line by line at one k: in turn they
// are two regions of memory at a time.  512 x 512 x 120000, N = 12: 906 us; with
// vector loads of the tables 1308, with both sides in turn 941; INT8, N = 14: 600, 900
// and 655.
__global__ __launch_bounds__(256) void k_residues(Problem P) {
  __shared__ double tile[kQL * kRowLd];
  const Dims d = family_dims(kFamRes, P);
  const uint32_t y = (uint32_t)d.y, per = (uint32_t)d.x * y;
  const uint32_t z = d.z == 1 ? 0u : blockIdx.x / per;
  const uint32_t xa = (uint32_t)(P.res_sides & 1 ? P.g.mp / kQL : 0);
  uint32_t q = blockIdx.x - z * per;
  const bool side = q >= xa * y;
  if (side) q -= xa * y;
  const uint32_t x = side ? (uint32_t)d.x - xa : xa, by = q / x;
  residues_tile(operand(P, side), P.g.kp, side ? P.g.np : P.g.mp, (int64_t)(q - by * x) * kQL,
                (int64_t)by * kQK, P.w, side ? P.w.lineB : 0, (CTables *)(uintptr_t)P.tab,
                moduli_range(P.g, z, d.z), side ? P.w.Bsl : P.w.Asl, tile);
}

// ---- slices in fragment order ----
//
// The slices of k_residue6 (oz2_gemm6.hip).  E2M3 digits: the code of d / 8 is
// the sign and |d| as a 5-bit integer, for |d| <= 16.  INT8 residues: bytes.
//
// A thread owns one line and 32 consecutive k, i.e. one lane's 24 bytes of
// every slice, a wave 64 lines, a workgroup 64 lines x 128 k (a whole group of
// a stage, 6 KB contiguous per slice).  Lines contiguous in memory are read
// straight into registers, 512 bytes per load; lines with contiguous k in runs
// of 16 k that are turned through LDS.
//
// Bound by vector issue.  Against the E4M3 pass (198 vector instructions per
// input at N = 12) the set-up is two FP64 operations: a' = trunc(a 2^s) may be
// large, NaN or infinite (the line's outputs are then NaN whatever its digits),
// because each FP64 step takes 51 bits off it (mod_step) and a line's scale
// exponent says how many steps its entries need; the digits are split in
// packed FP16 (integers up to 547, exact), two per instruction, and converted
// 32 at a time.  8192^3, N = 12, both operands: 0.83 ms, 0.99 ms before, and
// 4.1 GB moved instead of 5.1.
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h32 __attribute__((ext_vector_type(32)));
typedef uint32_t u6 __attribute__((ext_vector_type(6)));

constexpr int kR6L = 64, kR6K = 128;  // lines x k per workgroup
constexpr int kR6E = 32;              // inputs per thread
constexpr int kR6Ld = 18;             // doubles per staged row of 16 (16-byte rows, skewed)

__device__ __forceinline__ void store6(const h32 &d, uint8_t *slice, uint32_t off16,
                                       uint32_t off8) {
  // scale 8: the code of d / 8
  const u6 w = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(d, 8.0f);
  *(uint4 *)(slice + off16) = make_uint4(w[0], w[1], w[2], w[3]);
  *(uint2 *)(slice + off8) = make_uint2(w[4], w[5]);
}

// rint(x m) of both halves for |x m| < 512: the one rounding of x m + 1.5 2^10,
// where FP16 has unit spacing.
__device__ __forceinline__ h2 rint_h2(h2 x, h2 m) {
  const h2 magic = {(_Float16)1536.0f, (_Float16)1536.0f};
  return __builtin_elementwise_fma(x, m, magic) - magic;
}

// The digits of one modulus from f (|f| < 2^20 + 2^11, congruent to the
// inputs): the nearest multiple of p removed in FP32 (exact, |u| <= (p + 1) / 2
// at most at an even p's half), then, in FP16,
//   square p = s^2: x1 = rint(u / s), x2 = u - s x1 (|u / s - x1| stays within
//     1 / 2 although 1 / s is rounded: an odd s has no ties, and any choice
//     does at a tie of s = 32);
//   Karatsuba, s = 16: x1 = u / 16 away from zero, as rint of (|u| + 7.5) / 16,
//     x2 = u - 16 x1, x3 = x1 + x2.
// All have magnitude at most 16 for every modulus of both lists.
template <int KIND>
__device__ __forceinline__ void digits6(const float (&f)[kR6E], CTables *tab, int l,
                                        uint8_t *base, int64_t slice_stride, uint32_t off16,
                                        uint32_t off8) {
  const float pf = (float)tab->p[l], invpf = tab->inv_p[l];
  const h2 s2 = {(_Float16)tab->s[l], (_Float16)tab->s[l]};
  const h2 is2 = {(_Float16)tab->inv_s[l], (_Float16)tab->inv_s[l]};
  uint8_t *dst = base + (int64_t)tab->slice0[l] * slice_stride;
  h32 d1, d2, d3;
#pragma unroll
  for (int q = 0; q < kR6E; q += 2) {
    const float a = fmaf(-rintf(f[q] * invpf), pf, f[q]);
    const float b = fmaf(-rintf(f[q + 1] * invpf), pf, f[q + 1]);
    const h2 u = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(a, b));
    h2 x1, x2;
    if (KIND == 0) {
      x1 = rint_h2(u, is2);
      x2 = __builtin_elementwise_fma(-s2, x1, u);
    } else {
      const uint32_t bias = (__builtin_bit_cast(uint32_t, u) & 0x80008000u) | 0x47804780u;  // 7.5
      const h2 t = u + __builtin_bit_cast(h2, bias);
      const h2 r16 = {(_Float16)0.0625f, (_Float16)0.0625f};
      x1 = rint_h2(t, r16);
      const h2 m16 = {(_Float16)-16.0f, (_Float16)-16.0f};
      x2 = __builtin_elementwise_fma(m16, x1, u);
      const h2 x3 = x1 + x2;
      d3[q] = x3[0];
      d3[q + 1] = x3[1];
    }
    d1[q] = x1[0];
    d1[q + 1] = x1[1];
    d2[q] = x2[0];
    d2[q + 1] = x2[1];
  }
  store6(d1, dst, off16, off8);
  store6(d2, dst + slice_stride, off16, off8);
  if (KIND == 1) store6(d3, dst + 2 * slice_stride, off16, off8);
}

// The residue of one INT8 modulus as the low bytes of its integers (an even p's
// half may be +p / 2: for p = 256 the byte of -128), 32 bytes of the line in two
// lanes' pieces of a 64-k stage.
__device__ __forceinline__ void digits8(const float (&f)[kR6E], CTables *tab, int l, uint8_t *base,
                                        int64_t slice_stride, uint32_t off) {
  const float pf = (float)tab->p[l], invpf = tab->inv_p[l];
  uint32_t w[kR6E / 4];
#pragma unroll
  for (int g = 0; g < kR6E / 4; ++g) {
    uint32_t b[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const float u = fmaf(-rintf(f[4 * g + z] * invpf), pf, f[4 * g + z]);
      b[z] = __float_as_uint(u + 0x1.8p23f);  // the integer in the low bits
    }
    const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0C0C0400u);
    const uint32_t hi = __builtin_amdgcn_perm(b[3], b[2], 0x04000C0Cu);
    w[g] = lo | hi;
  }
  uint8_t *dst = base + (int64_t)tab->slice0[l] * slice_stride + off;
  *(uint4 *)dst = make_uint4(w[0], w[1], w[2], w[3]);
  *(uint4 *)(dst + 256) = make_uint4(w[4], w[5], w[6], w[7]);
}

// x - R rint(x / R) for an integer x: with q the computed quotient (within
// 2^-52 of x / R, relatively) it is a multiple of ulp(q) or 1 below
// 2^-51 |x| + R / 2, i.e. of fewer than 53 bits (R < 2^21), so the fused
// multiply-add is exact; each step takes 51 bits off a large x.
__device__ __forceinline__ double mod_step(double x, double R, double invR) {
  return fma(-rint(x * invR), R, x);
}

template <int KIND, int STEPS>
__device__ __forceinline__ void kind6(const double (&x)[kR6E], CTables *tab, int l0, int l1,
                                      uint8_t *base, int64_t slice_stride, uint32_t off16,
                                      uint32_t off8) {
  for (int l = l0; l < l1; l += 2) {
    const bool two = l + 1 < l1;
    const double R = two ? (double)(tab->p[l] * tab->p[l + 1]) : (double)tab->p[l];
    const double invR = two ? tab->inv_pair[l] : tab->inv_pd[l];
    float f[kR6E];
#pragma unroll
    for (int q = 0; q < kR6E; ++q) {
      double y = mod_step(x[q], R, invR);
#pragma unroll
      for (int s = 1; s < STEPS; ++s) y = mod_step(y, R, invR);
      f[q] = (float)y;
    }
    if constexpr (KIND == 2) {
      digits8(f, tab, l, base, slice_stride, off16);
      if (two) digits8(f, tab, l + 1, base, slice_stride, off16);
    } else {
      digits6<KIND>(f, tab, l, base, slice_stride, off16, off8);
      if (two) digits6<KIND>(f, tab, l + 1, base, slice_stride, off16, off8);
    }
  }
}

template <int STEPS>
__device__ __forceinline__ void moduli6(const double (&x)[kR6E], CTables *tab,
                                        const ModuliRange &m, uint8_t *base, int64_t slice_stride, uint32_t off16,
                                        uint32_t off8) {
  kind6<0, STEPS>(x, tab, m.l0, m.a, base, slice_stride, off16, off8);
  kind6<1, STEPS>(x, tab, m.a, m.b, base, slice_stride, off16, off8);
  kind6<2, STEPS>(x, tab, m.b, m.l1, base, slice_stride, off16, off8);
}

template <bool GROUPED>
__global__ __launch_bounds__(256, 2) void k_residues6(Problem P1, Group G) {
  __shared__ __attribute__((aligned(16))) double tile[4][kR6L * kR6Ld];
  int64_t local;
  const Problem &P = *locate<GROUPED>(P1, G, blockIdx.x, local);
  const Dims d = family_dims(kFamRes6, P), c = decode_block(d, local);
  int64_t bx = c.x;
  const int64_t by = c.y;
  const int64_t first = P.res_sides & 1 ? P.g.mp / kR6L : 0;
  const bool side = bx >= first;
  if (side) bx -= first;
  const Operand op = operand(P, side);
  const int64_t R = side ? P.g.np : P.g.mp, kp = P.g.kp;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = bx * kR6L, h0 = by * kR6K + 32 * wave;
  const int64_t r = r0 + lane;
  double x[kR6E];
  if (op.sr == 1) {
    // lines contiguous: lane = line
    const bool in = r < op.lines;
    const double *src = op.ptr + r + h0 * op.sh;
#pragma unroll
    for (int q = 0; q < kR6E; ++q) x[q] = in && h0 + q < op.k ? src[q * op.sh] : 0.0;
  } else {
    // k contiguous: runs of 16 k of each line, turned through LDS
    double v[kR6E];
#pragma unroll
    for (int q = 0; q < kR6E; ++q) {
      const int64_t rr = r0 + 4 * (q & 15) + (lane >> 4), h = h0 + 16 * (q >> 4) + (lane & 15);
      v[q] = rr < op.lines && h < op.k ? op.ptr[rr * op.sr + h * op.sh] : 0.0;
    }
    double *mine = tile[wave];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half) __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q)
        mine[(4 * q + (lane >> 4)) * kR6Ld + (lane & 15)] = v[16 * half + q];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 16; ++q) x[16 * half + q] = mine[lane * kR6Ld + q];
    }
  }
  // a' = trunc(a 2^s); its magnitude is below 2^(e + 8)
  const int64_t base_line = side ? P.w.lineB : 0;
  CTables *tab = (CTables *)(uintptr_t)tables_of<GROUPED>(P1, G);
  int e;
  const int s = final_shift(P.w, base_line, r, tab->D, h0 == 0 && c.z == 0, &e);
#pragma unroll
  for (int q = 0; q < kR6E; ++q) x[q] = trunc(ldexp(x[q], s));
  // INT8: stages of 64 k, 4096 bytes per 64 lines, 16-byte pieces of 16 k; E2M3:
  // stages of 128 k, 6144 bytes per 64 lines
  const bool int8 = P.g.list == OZ2_MODULI_INT8;
  const int64_t slice_stride = int8 ? R * kp : R * kp / 4 * 3;
  const uint32_t kg = int8 ? 2 * (wave & 1) : wave, fragment = (lane & 3) * (int8 ? 1024u : 1536u);
  const uint32_t off16 = fragment + 16 * ((lane >> 2) + 16 * kg);
  const uint32_t off8 = fragment + 1024 + 8 * ((lane >> 2) + 16 * kg);
  uint8_t *base = (side ? P.w.Bsl : P.w.Asl) +
                  (int8 ? (h0 >> 6) * (R * 64) + bx * 4096 : by * (R * 96) + bx * 6144);
  const ModuliRange m = moduli_range(P.g, c.z, d.z);
  // |x| < 2^(e + 8): a step leaves |f| < R / 2 + 2^12 from below 2^63, two from
  // below 2^113; the scale exponent stays below 160, so four always do
  if (!__any(e > 55))
    moduli6<1>(x, tab, m, base, slice_stride, off16, off8);
  else if (!__any(e > 105))
    moduli6<2>(x, tab, m, base, slice_stride, off16, off8);
  else
    moduli6<4>(x, tab, m, base, slice_stride, off16, off8);
}

}  // namespace

hipError_t launch_quant_family(int fam, const Problem *P, const Group *G, hipStream_t st) {
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
  const dim3 grid((unsigned)blocks), blk(256);
#define OZ2_Q(KER)                                                          \
  if (grouped)                                                              \
    hipLaunchKernelGGL((KER<true>), grid, blk, 0, st, p1, g1);              \
  else                                                                      \
    hipLaunchKernelGGL((KER<false>), grid, blk, 0, st, p1, g1);
  if (fam == kFamLines) {
    const bool norm = grouped ? G->norm : p1.mode == OZ2_MODE_FAST;
    const int64_t k = grouped ? G->max_k : p1.g.k;
#define OZ2_L(T)                                                              \
  if (k <= kQK * kLinesG * T) {                                               \
    if (grouped && norm)                                                      \
      hipLaunchKernelGGL((k_lines<true, true, T>), grid, wide, 0, st, p1, g1);  \
    else if (grouped)                                                         \
      hipLaunchKernelGGL((k_lines<true, false, T>), grid, wide, 0, st, p1, g1); \
    else if (norm)                                                            \
      hipLaunchKernelGGL((k_lines<false, true, T>), grid, wide, 0, st, p1, g1); \
    else                                                                      \
      hipLaunchKernelGGL((k_lines<false, false, T>), grid, wide, 0, st, p1, g1); \
    return hipGetLastError();                                                 \
  }
    const dim3 wide(256 * kLinesG);
    OZ2_L(1) OZ2_L(2) OZ2_L(4) OZ2_L(8) OZ2_L(16) OZ2_L(32)
#undef OZ2_L
    return hipErrorInvalidValue;
  }
  switch (fam) {
    case kFamFill: OZ2_Q(k_fill) break;
    case kFamLmax: OZ2_Q(k_line_max) break;
    case kFamBar: OZ2_Q(k_bound_operand) break;
    case kFamNorm: OZ2_Q(k_bound_norm) break;
    case kFamRes:
      if (grouped) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_residues, grid, blk, 0, st, p1);
      break;
    case kFamRes6: OZ2_Q(k_residues6) break;
    default: return hipErrorInvalidValue;
  }
#undef OZ2_Q
  return hipGetLastError();
}

}  // namespace oz2
