// Products of few output tiles: the residue products on k-blocked slices and
// the bound product of calls whose tiles of 256 x 256 leave most CUs idle.
// There the one workgroup of a tile runs its loads, passes, epilogue and stores
// one after another; here a wave takes 32 x 32 outputs of a modulus (W = 1) or
// 64 x 64 (W = 2), four waves a tile of twice that.
//
// Bound by latency (a load from memory, the k steps, the epilogue), then by the
// L2 caches (10 TB/s), so nothing is staged: the k-blocked layout puts 32 lines
// x 64 k in 2 KB of contiguous memory, one MFMA operand read straight into
// registers, all digits' slices at once and up to three steps ahead.  The three
// digit products run side by side in accumulators of their own and are folded
// once.  Tiles and k beyond the operands (padding) are not computed.
// Consecutive items, which share slices, go to one XCD.
// 256^3, N = 12: products 24 -> 9.8 us, bound product 11.4 -> 6.6; 512 x 512 x
// 2048: 62 -> 52 and 27 -> 13; 1111 x 777 x 1999: bound product 27 -> 13.
#include <string.h>

#include "oz2_internal.h"

namespace oz2 {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v16f mma(v8i a, v8i b, v16f c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}
__device__ __forceinline__ v16i mma(v8i a, v8i b, v16i c) {
  const v4i a0 = __builtin_shufflevector(a, a, 0, 1, 2, 3);
  const v4i a1 = __builtin_shufflevector(a, a, 4, 5, 6, 7);
  const v4i b0 = __builtin_shufflevector(b, b, 0, 1, 2, 3);
  const v4i b1 = __builtin_shufflevector(b, b, 4, 5, 6, 7);
  c = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, c, 0, 0, 0);
}

__device__ __forceinline__ v8i frag(const uint8_t *p) {
  const v4i lo = *(const v4i *)p, hi = *(const v4i *)(p + 16);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// An integer congruent to x modulo p of magnitude at most p / 2 + 2.
__device__ __forceinline__ float reduce(float x, float p, float inv) {
  return fmaf(-rintf(x * inv), p, x);
}

// The symmetric residue of an integer |x| < 2^30 (INT8 sums reach 2^29) as an int16:
// one FP64 step
// whose quotient is nudged by 1 / (4 p), so that an exact half (even p) goes to
// -p / 2 and no other value (at least 1 / (2 p) from a half) moves.
__device__ __forceinline__ int16_t residue(double x, double p, double inv) {
  return (int16_t)(int)fma(-rint(fma(x, inv, 0.25 * inv)), p, x);
}

// The item of a workgroup: an eighth of the items, in order, per XCD.
__device__ __forceinline__ uint32_t item_of(uint32_t items) {
  return (blockIdx.x & 7) * ((items + 7) / 8) + (blockIdx.x >> 3);
}

struct Tile {
  int64_t i, j;  // the wave's first row and column
  uint32_t z;    // part * N + modulus
  bool any;      // whether the wave has outputs
};

template <int W>
__device__ __forceinline__ Tile tile_of(const Geometry &g, uint32_t it) {
  constexpr int T = 64 * W;
  const uint32_t x = ((uint32_t)g.m + T - 1) / T, y = ((uint32_t)g.n + T - 1) / T;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Tile t;
  t.z = it / (x * y);
  const uint32_t r = it - t.z * (x * y), ty = r / x;
  t.i = (int64_t)(r - ty * x) * T + 32 * W * (wave & 1);
  t.j = (int64_t)ty * T + 32 * W * (wave >> 1);
  t.any = t.i < g.m && t.j < g.n;
  return t;
}

// nk steps of 64 k of a wave's 32 W x 32 W outputs with the NS slices of each
// side, loaded D steps ahead; product(fb, fa, c) of one MFMA tile.
template <int W, int NS, int D, class ACC, int NA, class F>
__device__ __forceinline__ void steps(const uint8_t *a, const uint8_t *b, int64_t sa, int64_t sb,
                                      int64_t ka, int64_t kb, int nk, ACC (&acc)[W][W][NA],
                                      F &&product) {
  v8i fa[D][W][NS], fb[D][W][NS];
  auto load = [&](int d) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int w = 0; w < W; ++w) {
        fa[d][w][s] = frag(a + s * sa + w * 2048);
        fb[d][w][s] = frag(b + s * sb + w * 2048);
      }
    a += ka;
    b += kb;
  };
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < nk) load(d);
#pragma unroll 1
  for (int q = 0; q < nk; q += D)
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (q + d < nk) {
#pragma unroll
        for (int tj = 0; tj < W; ++tj)
#pragma unroll
          for (int ti = 0; ti < W; ++ti) product(fb[d][tj], fa[d][ti], acc[tj][ti]);
        if (q + d + D < nk) load(d);
      }
}

template <bool INT8, int W>
__global__ __launch_bounds__(256, W == 1 ? 2 : 1) void k_residue_small(Problem P, uint32_t items) {
  const uint32_t it = item_of(items);
  if (it >= items) return;
  const Geometry &g = P.g;
  const Tile t = tile_of<W>(g, it);
  if (!t.any) return;
  const uint32_t part = t.z / (uint32_t)g.N;
  const int l = (int)(t.z - part * (uint32_t)g.N);
  int64_t k0, k1;
  part_range(g.kp, P.parts, (int)part, &k0, &k1);
  const int64_t kend = (g.k + 63) / 64 * 64;
  const int nk = (int)(((k1 < kend ? k1 : kend) - k0) / 64);
  CTables *tab = (CTables *)(uintptr_t)P.tab;
  const int lane = threadIdx.x & 63;
  const int64_t sa = g.mp * g.kp, sb = g.np * g.kp, ka = g.mp * 64, kb = g.np * 64;
  const int64_t sl0 = tab->slice0[l];
  const uint8_t *a = P.w.Asl + sl0 * sa + k0 * g.mp + (t.i + (lane & 31)) * 64 + (lane >> 5) * 32;
  const uint8_t *b = P.w.Bsl + sl0 * sb + k0 * g.np + (t.j + (lane & 31)) * 64 + (lane >> 5) * 32;
  // accumulator value v of a lane: row t.i + 32 ti + lane % 32, column
  // t.j + 32 tj + 8 (v / 4) + 4 (lane / 32) + v % 4
  int16_t *out = P.w.planes + ((int64_t)part * g.N + l) * g.mp * g.np +
                 (t.j + 4 * (lane >> 5)) * g.mp + t.i + (lane & 31);
  const double pd = (double)tab->p[l], invd = tab->inv_pd[l];
  auto store = [&](auto &acc, auto &&value) {
#pragma unroll
    for (int tj = 0; tj < W; ++tj)
#pragma unroll
      for (int ti = 0; ti < W; ++ti) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          out[(tj * 32 + (v >> 2) * 8 + (v & 3)) * g.mp + ti * 32] =
              residue((double)value(acc[tj][ti], v), pd, invd);
        if (W > 1) __builtin_amdgcn_sched_barrier(0);
      }
  };
  const float p = (float)tab->p[l], inv = tab->inv_p[l];
  if constexpr (INT8) {
    v16i acc[W][W][1] = {};
    steps<W, 1, 4 / W>(a, b, sa, sb, ka, kb, nk, acc, [](auto &fb, auto &fa, auto &c) {
      c[0] = mma(fb[0], fa[0], c[0]);
    });
    store(acc, [](auto &c, int v) { return c[0][v]; });
  } else if (l < g.nsq) {
    // A1 B2 + A2 B1 (sums up to 2^24), A2 B2; p = s^2
    v16f acc[W][W][2] = {};
    steps<W, 2, W == 1 ? 3 : 2>(a, b, sa, sb, ka, kb, nk, acc, [](auto &fb, auto &fa, auto &c) {
      c[0] = mma(fb[1], fa[0], c[0]);
      c[1] = mma(fb[1], fa[1], c[1]);
      c[0] = mma(fb[0], fa[1], c[0]);
    });
    const float s = (float)tab->s[l], inv_s = tab->inv_s[l];
    store(acc, [=](auto &c, int v) { return fmaf(reduce(c[0][v], s, inv_s), s, c[1][v]); });
  } else {
    // c (b (a X + Y) + Z), X = A1 B1, Y and Z the other two by the table
    v16f acc[W][W][3] = {};
    steps<W, 3, W == 1 ? 2 : 1>(a, b, sa, sb, ka, kb, nk, acc, [](auto &fb, auto &fa, auto &c) {
#pragma unroll
      for (int d = 0; d < 3; ++d) c[d] = mma(fb[d], fa[d], c[d]);
    });
    const float ma = (float)tab->kfold[l][0], mb = (float)tab->kfold[l][1];
    const float mc = (float)tab->kfold[l][2];
    const bool second1 = tab->kfold[l][3] == 1;
    store(acc, [=](auto &c, int v) {
      const float y = second1 ? c[1][v] : c[2][v], z = second1 ? c[2][v] : c[1][v];
      const float u = fmaf(reduce(c[0][v], p, inv), ma, y);
      return reduce(fmaf(reduce(u, p, inv), mb, z), p, inv) * mc;
    });
  }
}

// The bound product's line maxima: 32 x 32 outputs per wave over all of k.
__device__ __forceinline__ float keep_half(float lo, float hi, int lane, int off) {
  const bool up = (lane & off) != 0;
  return fmaxf(up ? hi : lo, __shfl_xor(up ? lo : hi, off, 64));
}

__global__ __launch_bounds__(256) void k_bound_small(Problem P, uint32_t items) {
  const uint32_t it = item_of(items);
  if (it >= items) return;
  const Geometry &g = P.g;
  const Tile t = tile_of<1>(g, it);
  if (!t.any) return;
  const int lane = threadIdx.x & 63;
  const uint8_t *a = P.w.Abar + (t.i + (lane & 31)) * 64 + (lane >> 5) * 32;
  const uint8_t *b = P.w.Bbar + (t.j + (lane & 31)) * 64 + (lane >> 5) * 32;
  v16f acc[1][1][1] = {};
  steps<1, 1, 4>(a, b, 0, 0, g.mp * 64, g.np * 64, (int)((g.k + 63) / 64), acc,
                 [](auto &fb, auto &fa, auto &c) { c[0] = mma(fb[0], fa[0], c[0]); });
  float c[16], m = 0.0f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    c[v] = acc[0][0][0][v];
    m = fmaxf(m, c[v]);
  }
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  if (lane < 32) atomicMax(&P.w.rmax[t.i + lane], __float_as_uint(m));
  // the 16 columns' maxima, dealt out over the lanes while they are reduced:
  // after the exchange at distance 16 >> s a lane keeps half of its values
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < (8 >> s); ++q) c[q] = keep_half(c[q], c[q + (8 >> s)], lane, 16 >> s);
  const float cm = fmaxf(c[0], __shfl_xor(c[0], 1, 64));
  const int v = 8 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1) + ((lane >> 1) & 1);
  if (!(lane & 1))
    atomicMax(&P.w.rmax[g.mp + t.j + (v >> 2) * 8 + 4 * (lane >> 5) + (v & 3)], __float_as_uint(cm));
}

int64_t tiles(const Problem &P, int w) {
  const int64_t t = 64 * w;
  return (P.g.m + t - 1) / t * ((P.g.n + t - 1) / t);
}

}  // namespace

// Up to two 64 x 64 tiles per CU the smaller tile wins at any k (512 x 256,
// k = 2048, 384 items: 50.3 us, W = 2 51.3, a 256 x 256 tile 62.4; 400 x 400, 588
// items, 70.4, 51.7 and 64.4); W = 2 while a CU has one (512 x 512, 192 items at
// k = 2048 51.9 against 62.8, 384 at k = 4096 98.7 against 66.0).  The bound
// product at 512 items of 64 x 64 and fewer (234 items, k = 1999: 13.1 against
// 27.0; 1024 items, k = 1024: 20.4 against 18.9); a split one has its own tiles.
int small_width(int fam, const Problem &P) {
  if (fam == kFamBgemm) return P.bparts == 1 && tiles(P, 1) <= 512 ? 1 : 0;
  if (fam != kFamGemm8 && fam != kFamGemmI8) return 0;
  const int64_t z = (int64_t)P.g.N * P.parts;
  return tiles(P, 1) * z <= 512 ? 1 : tiles(P, 2) * z <= 256 ? 2 : 0;
}

hipError_t launch_small(int fam, const Problem &P, int w, hipStream_t st) {
  const int64_t items = tiles(P, w) * (fam == kFamBgemm ? 1 : (int64_t)P.g.N * P.parts);
  if (items <= 0) return hipSuccess;
  if (items > 0x7FFFFF00ll) return hipErrorInvalidValue;
  const dim3 gr((unsigned)((items + 7) / 8 * 8)), blk(256);
  const uint32_t n = (uint32_t)items;
  if (fam == kFamBgemm)
    hipLaunchKernelGGL(k_bound_small, gr, blk, 0, st, P, n);
  else if (fam == kFamGemmI8 && w == 1)
    hipLaunchKernelGGL((k_residue_small<true, 1>), gr, blk, 0, st, P, n);
  else if (fam == kFamGemmI8)
    hipLaunchKernelGGL((k_residue_small<true, 2>), gr, blk, 0, st, P, n);
  else if (w == 1)
    hipLaunchKernelGGL((k_residue_small<false, 1>), gr, blk, 0, st, P, n);
  else
    hipLaunchKernelGGL((k_residue_small<false, 2>), gr, blk, 0, st, P, n);
  return hipGetLastError();
}

}  // namespace oz2
