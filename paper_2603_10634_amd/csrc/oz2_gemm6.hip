// Residue products of calls of more than four output tiles and of batches: on
// E2M3 digits (v_mfma_f32_16x16x128_f8f6f4, FP32 accumulation), or on INT8
// residues (v_mfma_i32_16x16x64_i8, INT32 accumulation).
//
// Every digit of Sections III-B and III-C is an integer of magnitude at most
// 16, and E2M3 (6 bits, steps of 1/8 up to 2, OCP MX) holds d / 8 exactly for
// each of them, so the products are those of the E4M3 digits: integers over
// 64, exact in FP32 below 2^24 / 64.  The format halves the MFMA's cycles (16
// per 16 x 16 x 128 step against 32) and takes a quarter off the bytes of
// every slice.
//
// What bounds it: power.  A register-only loop on digits of this range
// sustains 7.2 PFLOP/s with the 16 x 16 x 128 form and 6.2 with 32 x 32 x 64
// (E4M3: 4.2), the chip lowering its clock to 1.5-1.6 GHz; hence the 16-wide
// form, whose accumulators cost half as much register traffic per operation.
// At 8192^3, N = 12 the 36 products run at 4.6 PFLOP/s (8.55 ms; 12.7 ms on
// E4M3), with the MFMA busy 65 % of the cycles at 1.62 GHz.  Other orders of
// the same work (a barrier per 64 or per 256 k, the barrier in the middle of
// a stage, wave priorities, 32 x 32 x 64 steps at 71 % busy and 1.40 GHz)
// came out within 2 % of one another or slower.  Left out in turn: the loads into
// LDS account for a fifth of the time, of it 6 % (10 % at k = 1024) for lines that
// are not in L2; the planes' stores for 5 % at k = 4096 and 11 % at k = 1024.
//
// Layout (digit6): a slice of R lines is cut into stages of 128 k, a stage
// into groups of 64 lines, a group into the fragments of its lines r = q (mod
// 4), q = 0 .. 3; fragment q holds, for lane l = r / 4 + 16 (h / 32), the 32
// digits of line r and k h .. h + 31 as 24 bytes: the first 16 bytes of the 64
// lanes in lane order, then their last 8.  One stage of 256 lines is 24 KB of
// contiguous memory, LDS is filled by copies of it, and every fragment read
// (one ds_read_b128 and one ds_read_b64 per lane) covers consecutive bytes
// across the lanes, free of bank conflicts.  Interleaving the lines by four
// gives each lane four consecutive rows i of its column j in the accumulators,
// so the int16 planes are stored 8 bytes per lane.
//
// INT8 residues (Section II, one product per modulus) keep the same order with
// stages of 64 k, fragments of 1 KB and lane l = r / 4 + 16 (h / 16) holding 16
// k.  A register-only loop sustains 4.17 POP/s with 16 x 16 x 64 steps and 3.47
// with 32 x 32 x 32.  4096^3, N = 14: residues 248 -> 151 us and products 933 ->
// 789 us (2.4 POP/s) against k-blocked slices and a workgroup per tile on 32 x
// 32 x 32 steps.
//
// Workgroup: 256 (j) x 256 (i) outputs, 8 waves of 128 x 64 (128 accumulator
// registers each, two waves per SIMD), one per CU, walking the (part,
// modulus, tile) items in rounds of the grid.  The stages of an
// item's three passes and of the next item form one sequence through an LDS
// ring of three 48 KB slots, so the loads never stop: the next pass's first
// stages land during the fold between the passes, the next item's during the
// epilogue.
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "oz2_internal.h"

namespace oz2 {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NW = 8;                       // waves: 2 (j) x 4 (i)
constexpr int TJ = 8, TI = 4;               // MFMA tiles of 16 x 16 per wave: 128 x 64
constexpr int64_t kCUs = 256;               // one workgroup per CU

// The two formats of the slices: fragments of FRAG bytes, 16 lines x BK k (an
// MFMA step, and a stage), S ring slots, PASSES products per modulus.
template <bool I8_>
struct Format {
  static constexpr bool I8 = I8_;
  static constexpr int FRAG = I8 ? 1024 : 1536;
  static constexpr int BK = I8 ? kStage8 : kStage6;
  static constexpr int S = I8 ? 4 : 3;
  static constexpr int PASSES = I8 ? 1 : 3;
  static constexpr int SIDE = kGemmTJ / 16 * FRAG;  // one side of a stage: 256 lines
  static constexpr int STAGE = 2 * SIDE;            // B side, then A side
  static constexpr int RING = S * STAGE;            // 144 KB (E2M3), 128 KB (INT8)
  static constexpr int LPW = STAGE / 1024 / NW;     // 1 KB loads per wave and stage
  typedef typename std::conditional<I8, v4i, v8i>::type Frag;
  typedef typename std::conditional<I8, v4i, v4f>::type Acc;
  static_assert(kGemmTJ == 32 * TJ && kGemmTIW == 64 * TI && LPW == (I8 ? 4 : 6) &&
                kPad % (2 * BK) == 0, "tile shape");
};
typedef Format<false> E2M3;
typedef Format<true> Int8;

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkm0() {
  __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x0 << 8) | (0x3 << 14));
}

__device__ __forceinline__ int uni32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ v4f mma(v8i a, v8i b, v4f c) {
  // cbsz = blgp = 2 selects E2M3 for both operands
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);
}
__device__ __forceinline__ v4i mma(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// A fragment: of E2M3, lane l's 32 digits (192 bits) as its first 16 bytes in
// one run of 64 lanes and its last 8 in another; of INT8, its 16 bytes.
__device__ __forceinline__ void frag(v8i &f, const uint8_t *p, int lane) {
  const v4i lo = *(const v4i *)(p + 16 * lane);
  const v2i hi = *(const v2i *)(p + 1024 + 8 * lane);
  f = __builtin_shufflevector(lo, __builtin_shufflevector(hi, hi, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5,
                              -1, -1);
}
__device__ __forceinline__ void frag(v4i &f, const uint8_t *p, int lane) {
  f = *(const v4i *)(p + 16 * lane);
}

__device__ __forceinline__ void dma16(const uint8_t *base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base),
               "{m0}"(lds_off)
               : "memory");
}

__device__ __forceinline__ uint32_t lds_offset(const uint8_t *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint8_t *)p;
}

// One tile of one modulus over a k range: what the loads need.
struct Item {
  const uint8_t *A, *B;   // slice 0 of the modulus at (k0, i0) / (k0, j0)
  int64_t sA, sB;         // bytes between slices of a side
  int64_t stA, stB;       // bytes of a stage of all lines of a side
  int nk;                 // stages per pass
  int ab;                 // slices of the passes: 2 bits each, a1 b1 a2 b2 a3 b3
};

// The stage to load next: its item, pass and place, and the item after it.
struct Producer {
  Item it, next;
  const uint8_t *pB, *pA;
  int left, pass;
};

__device__ __forceinline__ void start_pass(Producer &p) {
  const int sl = p.it.ab >> (4 * p.pass);
  p.pA = p.it.A + (int64_t)(sl & 3) * p.it.sA;
  p.pB = p.it.B + (int64_t)((sl >> 2) & 3) * p.it.sB;
  p.left = p.it.nk;
}

// On to the next stage: of the pass, of the item's next pass or of the next item.
template <int PASSES>
__device__ __forceinline__ void advance(Producer &p) {
  p.pA += p.it.stA;
  p.pB += p.it.stB;
  if (__builtin_expect(--p.left == 0, 0)) {
    if (++p.pass == PASSES) {
      p.pass = 0;
      p.it = p.next;
    }
    start_pass(p);
  }
}

template <int LPW>
struct Lanes {
  uint32_t vo[LPW / 2];  // byte offset of this lane in each of its wave's loads of a side
  uint32_t ls;           // place of the wave's first load in a slot
};

// Load u of the producer's stage (the first half of the B side, the second of
// the A side) into the slot at LDS byte address `slot`.
template <class F, int U>
__device__ __forceinline__ void load(const Producer &p, const Lanes<F::LPW> &ln, uint32_t slot) {
  constexpr int H = F::LPW / 2;
  dma16(U < H ? p.pB : p.pA, ln.vo[U % H], slot + ln.ls + 1024u * NW * U);
  __builtin_amdgcn_sched_barrier(0);
}

struct Ring {
  uint32_t base;     // LDS byte address of the ring
  uint32_t cur;      // slot offset of the stage being summed
  uint32_t fill;     // slot offset of the stage being loaded
};

template <class F>
__device__ __forceinline__ uint32_t next_slot(uint32_t s) {
  return s + F::STAGE == F::RING ? 0u : s + F::STAGE;
}

// One stage j of a wave's 128 x 64 outputs: rows tj of four MFMAs, the B fragment of row tj + 3 read and the loads of stage j + S - 1 (into the
// slot stage j - 1 left) issued between them; before the last two rows the barrier
// B_j, at which the wave's own loads of stage j + 1 have landed and its reads
// of stage j are done; under those rows the A fragments and first three B
// fragments of stage j + 1 are read.  ZERO: the accumulators start at zero.
// WAIT: wait for the loads (else they are known to be there).
template <bool ZERO, bool WAIT, class F>
__device__ __forceinline__ void stage(Producer &p, const Lanes<F::LPW> &ln, Ring &r,
                                      const uint8_t *lds, const typename F::Frag (&fa)[TI],
                                      typename F::Frag (&fan)[TI],
                                      typename F::Frag (&fb0)[3],
                                      typename F::Acc (&acc)[TJ][TI], int lane, int wj,
                                      int wi) {
  constexpr int FRAG = F::FRAG;
  const uint8_t *cur = lds + r.cur + wj * TJ * FRAG;
  const uint32_t fill = r.base + r.fill;
  const typename F::Acc zero = {0, 0, 0, 0};
  typename F::Frag fb[TJ];
#pragma unroll
  for (int t = 0; t < 3; ++t) fb[t] = fb0[t];
#pragma unroll
  for (int tj = 0; tj < TJ - 2; ++tj)
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
      acc[tj][ti] = mma(fb[tj], fa[ti], ZERO ? zero : acc[tj][ti]);
      __builtin_amdgcn_sched_barrier(0);
      if (ti == 0 && tj + 3 < TJ) {
        frag(fb[tj + 3], cur + (tj + 3) * FRAG, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int q = tj * TI + ti;
      if constexpr (F::LPW == 6) {
        if (q == 1) load<F, 0>(p, ln, fill);
        if (q == 3) load<F, 3>(p, ln, fill);
        if (q == 5) load<F, 1>(p, ln, fill);
        if (q == 7) load<F, 4>(p, ln, fill);
        if (q == 9) load<F, 2>(p, ln, fill);
        if (q == 11) load<F, 5>(p, ln, fill);
      } else {
        if (q == 1) load<F, 0>(p, ln, fill);
        if (q == 4) load<F, 2>(p, ln, fill);
        if (q == 7) load<F, 1>(p, ln, fill);
        if (q == 10) load<F, 3>(p, ln, fill);
      }
    }
  advance<F::PASSES>(p);
  r.fill = next_slot<F>(r.fill);
  wait_lgkm0();
  if (WAIT) wait_vm<(F::S - 2) * F::LPW>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  // stage j + 1 is readable by all waves and slot j is free
  r.cur = next_slot<F>(r.cur);
  const uint8_t *nb = lds + r.cur + wj * TJ * FRAG, *na = lds + r.cur + F::SIDE + wi * TI * FRAG;
#pragma unroll
  for (int tj = TJ - 2; tj < TJ; ++tj)
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
      acc[tj][ti] = mma(fb[tj], fa[ti], ZERO ? zero : acc[tj][ti]);
      __builtin_amdgcn_sched_barrier(0);
      const int q = (tj - (TJ - 2)) * TI + ti;  // next: a0 b0 a1 a2 a3 b1 b2
      if (q == 0) frag(fan[0], na, lane);
      if (q == 1) frag(fb0[0], nb, lane);
      if (q >= 2 && q <= 4) frag(fan[q - 1], na + (q - 1) * FRAG, lane);
      if (q == 5 || q == 6) frag(fb0[q - 4], nb + (q - 4) * FRAG, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
}

// An item's stages of a wave whose outputs are all padding: its share of the loads
// and one barrier per stage, as in stage(), then the next item's first fragments.
// (Its matrix instructions were power and time of the others: 48 products of 64 ..
// 2048, 47 % of their work padding, 443 -> 409 us.)
template <class F>
__device__ __forceinline__ void pad_item(Producer &p, const Lanes<F::LPW> &ln, Ring &r,
                                         const uint8_t *lds, typename F::Frag (&fa)[TI],
                                         typename F::Frag (&fb)[3], int stages, int lane, int wj,
                                         int wi) {
#pragma unroll 1
  for (int j = 0; j < stages; ++j) {
    const uint32_t slot = r.base + r.fill;
    load<F, 0>(p, ln, slot);
    load<F, 1>(p, ln, slot);
    load<F, 2>(p, ln, slot);
    load<F, 3>(p, ln, slot);
    if constexpr (F::LPW > 4) {
      load<F, 4>(p, ln, slot);
      load<F, 5>(p, ln, slot);
    }
    advance<F::PASSES>(p);
    r.fill = next_slot<F>(r.fill);
    wait_lgkm0();
    wait_vm<(F::S - 2) * F::LPW>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    r.cur = next_slot<F>(r.cur);
  }
  wait_vm<0>();  // the next item's first stages, as before the result's stores
#pragma unroll
  for (int t = 0; t < TI; ++t)
    frag(fa[t], lds + r.cur + F::SIDE + (wi * TI + t) * F::FRAG, lane);
#pragma unroll
  for (int t = 0; t < 3; ++t) frag(fb[t], lds + r.cur + (wj * TJ + t) * F::FRAG, lane);
  __builtin_amdgcn_sched_barrier(0);
}

// acc = acc mods q up to a multiple of q: for an exact x (in units of 1/64: q64
// = q / 64, inv64 = 64 / q) with |64 x| < 2^24, x - rint(x / q) q is exact in one
// fused multiply-add and at most q / 2 + 2 in magnitude; times a multiplier it
// is below 258 256 < 2^17, and the next chunk's sums (at most 2^23 more) stay
// exact.  (Only a square's first pass of one chunk goes on unreduced: 2^24.)
__device__ __forceinline__ void reduce(v4f (&acc)[TJ][TI], float q64, float inv64) {
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = acc[tj][ti][v];
        acc[tj][ti][v] = fmaf(-rintf(x * inv64), q64, x);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
}
__device__ __forceinline__ void scale(v4f (&acc)[TJ][TI], float m) {
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[tj][ti][v] *= m;
      __builtin_amdgcn_sched_barrier(0);
    }
}

// Where an item's tile is: a modulus, output tile and k range of a problem.
struct Place {
  CProblem *P;
  int l, part, tx, ty;  // tile numbers in units of the shape
  int k0, nk;           // first k, stages per pass
};

template <class F>
__device__ __forceinline__ Item make_item(const Place &c, CTables *tab) {
  const int64_t mp = c.P->g.mp, np = c.P->g.np, kp = c.P->g.kp;
  const int sl0 = tab->slice0[c.l];
  Item I;
  I.stA = mp / 16 * F::FRAG;
  I.stB = np / 16 * F::FRAG;
  I.sA = kp / F::BK * I.stA;
  I.sB = kp / F::BK * I.stB;
  I.A = c.P->w.Asl + sl0 * I.sA + c.k0 / F::BK * I.stA + c.tx * (int64_t)F::SIDE;
  I.B = c.P->w.Bsl + sl0 * I.sB + c.k0 / F::BK * I.stB + c.ty * (int64_t)F::SIDE;
  I.nk = c.nk;
  I.ab = 0;
  if constexpr (!F::I8) {
    const int second = tab->kfold[c.l][3], third = 3 - second;
    I.ab = tab->kind[c.l] == 0 ? ((1 << 2) | (1 << 4) | (1 << 8) | (1 << 10))
                               : ((second << 4) | (second << 6) | (third << 8) | (third << 10));
  }
  return I;
}

// Item `it` of a single problem: tiles within moduli within k parts, the tiles
// in bands of kBand rows j, column by column, so that 32 consecutive items
// (what the CUs of one XCD sum at a time, see item_of) share 8 strips of A and
// 4 of B in that XCD's L2 wherever the tile grid allows: 12 strips instead of
// the 48 of a 4 x 4 grid dealt out tile by tile (1024 x 1024 x 65536).
constexpr uint32_t kBand = 4;

template <class F>
__device__ __forceinline__ Place place_single(CProblem *P, int it) {
  const uint32_t tx_n = (uint32_t)(P->g.mp / kGemmTIW), ty_n = (uint32_t)(P->g.np / kGemmTJ);
  const uint32_t N = (uint32_t)P->g.N, parts = (uint32_t)P->parts;
  const uint32_t nb = (uint32_t)(P->g.kp / kPad);
  const uint32_t u = (uint32_t)it, tiles = tx_n * ty_n, b = u / tiles, z = b / N;
  const uint32_t t = u - b * tiles, band = t / (kBand * tx_n), r = t - band * (kBand * tx_n);
  const uint32_t left = ty_n - kBand * band, h = left < kBand ? left : kBand, x = r / h;
  const uint32_t k0 = z * nb / parts, k1 = (z + 1) * nb / parts;  // part_range, in 32 bits
  Place c;
  c.P = P;
  c.l = uni32((int)(b - z * N));
  c.part = uni32((int)z);
  c.tx = uni32((int)x);
  c.ty = uni32((int)(kBand * band + (r - x * h)));
  c.k0 = uni32((int)k0 * kPad);
  c.nk = uni32((int)(k1 - k0) * (kPad / F::BK));
  return c;
}

template <class F>
__device__ __forceinline__ Place place_list(const WorkList &W, int it) {
  OZ2_CONST ProductItem *I = (OZ2_CONST ProductItem *)(uintptr_t)W.items + it;
  Place c;
  c.P = (CProblem *)(uintptr_t)W.probs + I->prob;
  c.l = I->l;
  c.part = I->part;
  c.tx = I->tx;
  c.ty = I->ty;
  c.k0 = I->k0;
  c.nk = (I->k1 - I->k0) / F::BK;
  return c;
}

// The residue products of one problem (LIST false) or of a batch's work list:
// per (modulus, tile, k part) the three passes of the modulus (square: A1 B2 +
// A2 B1, fold s (. mod s), + A2 B2; Karatsuba: X, fold a, + Y, fold b, + Z,
// times c, see the tables) into one accumulator, then the symmetric residue
// into the modulus's int16 plane.  A pass of a list item longer than kChunkK is
// summed in chunks of that length, each but the last reduced modulo p, and the
// last by the pass's fold.  Items
// go to the workgroups in rounds, a list's every second one backwards: sorted
// longest first it comes out within 3 % of the average (48 problems log-uniform
// in [64, 2048]), with no counter to fetch from.
template <bool LIST, class F>
__global__ __launch_bounds__(64 * NW, 1) void k_residue6(Problem, WorkList W, int count) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[F::RING];
  // the problem by value is the first kernel argument
  CProblem *P1 = (CProblem *)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wj = wave >> 2, wi = wave & 3;
  const int grid = (int)gridDim.x;
  // This workgroup's item of round q (count: none).  Workgroups are dealt out
  // over the eight XCDs in turn, so XCD b mod 8 takes the (b mod 8)-th run of
  // ceil(n / 8) consecutive items of the round's n; a list's odd rounds run
  // backwards.
  auto item_of = [&](int q) {
    const int left = count - q * grid, n = left < grid ? left : grid;
    const int per = (n + 7) / 8, y = (int)blockIdx.x / 8, at = (int)(blockIdx.x % 8) * per + y;
    if (n <= 0 || y >= per || at >= n) return count;
    return q * grid + (LIST && (q & 1) ? n - 1 - at : at);
  };
  int round = 0, item = item_of(0);
  if (item >= count) return;
  const int first = item;
  auto place = [&](int it) {
    const int i = it < count ? it : first;  // past the end: loads that nothing reads
    return LIST ? place_list<F>(W, i) : place_single<F>(P1, i);
  };
  auto loads_of = [&](int it) {
    const Place c = place(it);
    return make_item<F>(c, (CTables *)(uintptr_t)c.P->tab);
  };
  Lanes<F::LPW> ln;
  ln.ls = 1024u * wave;
#pragma unroll
  for (int u = 0; u < F::LPW / 2; ++u) ln.vo[u] = 1024u * (wave + NW * u) + 16u * lane;

  Ring r;
  r.base = lds_offset(lds);
  r.cur = 0;
  r.fill = 0;
  Producer p;
  p.it = loads_of(item);
  p.next = p.it;
  p.pass = 0;
  start_pass(p);
  // stages 0 .. S - 2
#pragma unroll 1
  for (int t = 0; t < F::S - 1; ++t) {
    const uint32_t slot = r.base + r.fill;
    load<F, 0>(p, ln, slot);
    load<F, 1>(p, ln, slot);
    load<F, 2>(p, ln, slot);
    if constexpr (F::LPW > 3) load<F, 3>(p, ln, slot);
    if constexpr (F::LPW > 4) {
      load<F, 4>(p, ln, slot);
      load<F, 5>(p, ln, slot);
    }
    advance<F::PASSES>(p);
    r.fill = next_slot<F>(r.fill);
  }
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  typename F::Frag fa0[TI], fa1[TI], fb[3];
#pragma unroll
  for (int t = 0; t < TI; ++t) {
    frag(fa0[t], lds + F::SIDE + (wi * TI + t) * F::FRAG, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    frag(fb[t], lds + (wj * TJ + t) * F::FRAG, lane);
    __builtin_amdgcn_sched_barrier(0);
  }

  for (; item < count; item = item_of(++round)) {
    const Place c = place(item);
    CTables *tab = (CTables *)(uintptr_t)c.P->tab;
    const int l = c.l;
    // the loads run at most S - 1 stages ahead, less than an item (six)
    p.next = loads_of(item_of(round + 1));
    // a scalar load still pending would turn every LDS wait of the loops into
    // a full drain (both count on LGKM, out of order): wait for them here
    asm volatile("" ::"s"(p.next.ab), "s"(p.next.A), "s"(p.next.B), "s"(p.next.nk));
    if (c.ty * kGemmTJ + wj * 128 >= c.P->g.n || c.tx * kGemmTIW + wi * 64 >= c.P->g.m) {
      pad_item<F>(p, ln, r, lds, fa0, fb, F::PASSES * c.nk, lane, wj, wi);
      continue;
    }
    constexpr int kMaxStages = kChunkK / F::BK;
    typename F::Acc acc[TJ][TI];
    // the loop over the stages [j, n) of one chunk
    auto loop = [&](int j, int n) {
#pragma unroll 1
      for (; j < n; j += 2) {
        stage<false, true, F>(p, ln, r, lds, fa0, fa1, fb, acc, lane, wj, wi);
        stage<false, true, F>(p, ln, r, lds, fa1, fa0, fb, acc, lane, wj, wi);
      }
    };
    // stages 0 .. S - 2 had landed before the previous item's stores
    stage<true, false, F>(p, ln, r, lds, fa0, fa1, fb, acc, lane, wj, wi);
    stage<false, F::S == 3, F>(p, ln, r, lds, fa1, fa0, fb, acc, lane, wj, wi);
    const float pf = (float)tab->p[l], inv = tab->inv_p[l];
    const int64_t mp = c.P->g.mp, np = c.P->g.np;
    int16_t *out = c.P->w.planes + ((int64_t)c.part * c.P->g.N + l) * mp * np +
                   ((int64_t)c.ty * kGemmTJ + wj * 128 + (lane >> 4) * 16) * mp +
                   (int64_t)c.tx * kGemmTIW + wi * 64 + 4 * (lane & 15);
    // Four consecutive rows i of a column.  Planes are read once, by another
    // kernel: past the caches they leave the slices' strips there (16384 x 16384 x
    // 1024: 5.58 -> 5.33 ms, 2048^3 in fast mode 209 -> 194 us).
    auto store = [&](int tj, int v, const int (&res)[TI]) {
      int16_t *dst = out + ((tj >> 2) * 64 + 4 * v + (tj & 3)) * mp;
      // the next item's first stages (their loads count with the stores)
      if (tj == 0 && v == 0) wait_vm<0>();
      // the low halves of two values in one instruction
      const v2i w = {(int)__builtin_amdgcn_perm(res[1], res[0], 0x05040100u),
                     (int)__builtin_amdgcn_perm(res[3], res[2], 0x05040100u)};
      __builtin_nontemporal_store(w, (v2i *)dst);
    };
    if constexpr (F::I8) {
      // one product; the symmetric residue of an INT32 sum in FP64, where the
      // quotient is exact to 2^-28: one step, nudged like the last one below
      const double pd = (double)tab->p[l], invd = tab->inv_pd[l], nudge = 0.25 * invd;
      int left = c.nk, j0 = 2;
      if (LIST)
        for (; left > kMaxStages; left -= kMaxStages, j0 = 0) {
          loop(j0, kMaxStages);
#pragma unroll
          for (int tj = 0; tj < TJ; ++tj) {
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const double x = (double)acc[tj][ti][v];
                acc[tj][ti][v] = (int)fma(-rint(x * invd), pd, x);
              }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      loop(j0, left);
#pragma unroll
      for (int tj = 0; tj < TJ; ++tj) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          int res[TI];
#pragma unroll
          for (int ti = 0; ti < TI; ++ti) {
            const double x = (double)acc[tj][ti][v];
            res[ti] = (int)fma(-rint(fma(x, invd, nudge)), pd, x);
          }
          store(tj, v, res);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      // one pass (from stage j0 of it) and the fold that ends it: acc mods q
      // unless q = 0 after the last chunk, acc mods p after the others, then m acc
      auto pass = [&](int j0, float q, float iq, float m, float pf, float inv) {
        int left = c.nk;
        for (;;) {
          const int n = LIST && left > kMaxStages ? kMaxStages : left;
          loop(j0, n);
          left -= n;
          const bool last = !LIST || left == 0;
          const float qq = last ? q : pf;
          if (qq != 0.0f) reduce(acc, qq * 0.015625f, (last ? iq : inv) * 64.0f);
          if (last) break;
          j0 = 0;
        }
        if (m != 1.0f) scale(acc, m);
      };
      // The vector work between an item's MFMAs (4 instructions per output for a
      // fold, 5 for the result) is felt at short k, so what short sums don't need
      // is left out (products of 3000 x 2000 x 256 64.5 -> 58.7 us, 16384 x 16384 x
      // 1024 5.71 -> 5.58 ms):
      //  - squares, one chunk: the first two passes sum to at most 2^24 (a longer
      //    item's first pass ends at up to 2^23 + p / 2 + 2 and is reduced);
      //  - Karatsuba, k <= 3840: |a X + Y| <= 17 256 k < 2^24 without reducing X;
      //  - no reduction before the multiplier c and the result's own when the
      //    quotient's error stays below 1 / (4 p) (see the result below), about
      //    |c acc| <= 2^21: squares to k = 8192, Karatsuba at k = 256.
      const bool square = tab->kind[l] == 0;
      const int k = c.nk * F::BK;
      const bool plain = k <= (square ? kChunkK : 3840);
      pass(2, plain ? 0.0f : pf, inv, square ? 1.0f : (float)tab->kfold[l][0], pf, inv);
      const float q2 = square ? (float)tab->s[l] : pf, iq2 = square ? tab->inv_s[l] : inv;
      pass(0, q2, iq2, square ? q2 : (float)tab->kfold[l][1], pf, inv);
      pass(0, k <= (square ? 8192 : 256) ? 0.0f : pf, inv, 1.0f, pf, inv);
      // symmetric residue of c acc, four consecutive rows i per lane, its quotient
      // nudged by 1 / (4 p), so that an exact half (even p) goes to -p / 2 and no
      // other value (at least 1 / (2 p) from a half) moves
      const float mc = 64.0f * (square ? 1.0f : (float)tab->kfold[l][2]), bias = 0.25f * inv;
#pragma unroll
      for (int tj = 0; tj < TJ; ++tj) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          int res[TI];
#pragma unroll
          for (int ti = 0; ti < TI; ++ti) {
            const float y = acc[tj][ti][v] * mc;
            res[ti] = (int)fmaf(-rintf(fmaf(y, inv, bias)), pf, y);
          }
          store(tj, v, res);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  wait_vm<0>();
}

}  // namespace

// Workgroups for `count` items: a multiple of eight (see item_of), at most
// `cus` rounded down to one.
static int64_t grid_for(int64_t count, int64_t cus) {
  return std::min((count + 7) / 8 * 8, std::max<int64_t>(cus / 8, 1) * 8);
}

hipError_t launch_gemm6(const Problem &P, hipStream_t st) {
  const int64_t count = family_blocks(kFamGemm6, P);
  if (count <= 0) return hipSuccess;
  if (count > 0x7FFFFFFFll - 2 * kCUs) return hipErrorInvalidValue;
  const dim3 gr((unsigned)grid_for(count, kCUs)), blk(64 * NW);
  if (P.g.list == OZ2_MODULI_INT8)
    hipLaunchKernelGGL((k_residue6<false, Int8>), gr, blk, 0, st, P, WorkList{}, (int)count);
  else
    hipLaunchKernelGGL((k_residue6<false, E2M3>), gr, blk, 0, st, P, WorkList{}, (int)count);
  return hipGetLastError();
}

hipError_t launch_gemm6_list(bool int8, const WorkList &W, int64_t cus, hipStream_t st) {
  if (cus <= 0 || W.count > 0x7FFFFFFFll - 2 * cus) return hipErrorInvalidValue;
  Problem none;
  memset(&none, 0, sizeof(none));
  const dim3 gr((unsigned)grid_for(W.count, cus)), blk(64 * NW);
  if (int8)
    hipLaunchKernelGGL((k_residue6<true, Int8>), gr, blk, 0, st, none, W, (int)W.count);
  else
    hipLaunchKernelGGL((k_residue6<true, E2M3>), gr, blk, 0, st, none, W, (int)W.count);
  return hipGetLastError();
}

}  // namespace oz2
