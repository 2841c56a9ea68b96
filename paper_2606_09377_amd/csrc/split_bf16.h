// float32 products on the bf16 matrix cores: a float32 operand is the exact sum of three bf16
// values (8 significand bits each, 24 in all),
//   x = h + m + l,  h = bf16(x), m = bf16(x - h), l = x - h - m  (both differences are exact),
// and a product takes six of its nine partial products,
//   x y = h h' + (h l' + l h' + m m' + h m' + m h').
// The three left out, m l' + l m' + l l', are at most 2^-24 of the product together (|m| <= 2^-8,
// |l| <= 2^-17 of the power of two below |x|; x = y = 0x3f807fc0 leaves out 2^-24.01).  A lone
// product is so off by up to 1.65 2^-24 of itself, where a float32 multiply rounds by 2^-24 (rms
// 2.59e-8 against 2.53e-8); sums gain what the accumulators below give.
//
// Range:
// - Weights are split times 2^24 (SPLIT_SCALE), results multiplied back: every part is then a
//   multiple of 2^-125 (float32's values are multiples of 2^-149), so the sum is exact for all of
//   them, subnormal ones included.
// - Coefficients are split as they are (scaling them too cost 3% of a large product, in the
//   vector instructions of the split).  The sum is exact from 2^-110 on; below, what of a
//   coefficient is less than 2^-133, the least bf16 value, is rounded: by up to 2^-134.
// - Operands that round to infinity in bf16 (weights from 2^104, coefficients from 2^128 - 2^119),
//   infinite or NaN ones and sums from 2^104 on leave results that are not finite.  Those are
//   taken again in float32 from the float32 operands (split_finish), with the value, infinity
//   or NaN that float32 gives.
//
// h h' and the five small ones are summed in two
// accumulators, added once at the end.  In one accumulator the small partial products are
// cut off at the large sum's precision, towards minus infinity: sums over K = 1024 normal
// products came out 7.6e-8 of the result too low on average (3.3e-6 at K = 65536), and since a
// bound adds many such sums that bias stayed where rounding errors cancel: bounds were up to 20
// times as far from 64 bits.  With two accumulators the mean error is 3e-10 (K = 65536: 1.6e-8)
// and a sum is a third as far off as by the chain of v_mfma_f32_32x32x2f32 it replaces (K =
// 1024: 1.9e-7 of the result against 5.7e-7; K = 65536: 1.6e-6 against 4.6e-6).
//
// Why: the float32 matrix rate of gfx950 is 157 TFLOP/s; six bf16 products run at a sixth of
// 2.5 PFLOP/s nominal, 338 to 352 TFLOP/s of float32 products measured with random operands in
// registers, 406 to 414 with zeros (the card's power limit sets the rate, not the issue).
//
// Instruction: v_mfma_f32_16x16x32_bf16, in this order of partial products for every K step of
// 32 everywhere, so that a result does not depend on which tile size computed it.  The 32x32x16
// form runs as fast, but a lone wave's chain over K = 1024 takes 5.4 us for its 32 x 32 block
// against 1.6 us for a 16 x 16 one, and the small launches are such chains.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vcr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32v4 __attribute__((ext_vector_type(4)));

constexpr float SPLIT_SCALE = 0x1p24f, SPLIT_UNSCALE = 0x1p-24f;   // of a weight before its split, of a result

// two values at once: the packed pairs of bf16 (element 0 in the low half)
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t &h, uint32_t &m, uint32_t &l) {
  typedef float f32v2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto pack = [](float a, float b) {   // v_cvt_pk_bf16_f32, round to nearest even
    const f32v2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  };
  auto lo = [](uint32_t u) { return __builtin_bit_cast(float, u << 16); };
  auto hi = [](uint32_t u) { return __builtin_bit_cast(float, u & 0xffff0000u); };
  h = pack(x0, x1);
  x0 -= lo(h);
  x1 -= hi(h);
  m = pack(x0, x1);
  x0 -= lo(m);
  x1 -= hi(m);
  l = pack(x0, x1);
}

// the three bf16 operands of eight consecutive float32 values
struct Split8 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ Split8 split8(f32v4 x, f32v4 y) {
  typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));
  u32v4 h, m, l;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t a, b, c;
    split_pair(q < 2 ? x[2 * q] : y[2 * q - 4], q < 2 ? x[2 * q + 1] : y[2 * q - 3], a, b, c);
    h[q] = a;
    m[q] = b;
    l[q] = c;
  }
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// |w| of a split operand (mask 0x80008000; w itself with mask 0): the sign of w is h's, and the
// three parts change sign together
__device__ __forceinline__ Split8 split_abs(Split8 w, uint32_t mask) {
  typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));
  const u32v4 h = __builtin_bit_cast(u32v4, w.h);
  const u32v4 s = h & mask;
  return {__builtin_bit_cast(bf16x8, h ^ s), __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32v4, w.m) ^ s),
          __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32v4, w.l) ^ s)};
}

// acc += W A^T over 32 k: 16 weight rows (the accumulator's rows) and 16 coefficient rows (its
// columns).  Lane (r = lane % 16, g = lane / 16) holds k = 8 g .. 8 g + 7 of row r of both
// operands, and of the result column r, rows 4 g .. 4 g + 3: a lane ends with four consecutive
// output columns of one coefficient row.
__device__ __forceinline__ f32v4 mfma_bf16(bf16x8 w, bf16x8 a, f32v4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, acc, 0, 0, 0);
}
// One column block of a wave's MB row blocks: hi takes h h', lo the small partial products
template <int MB, int NB>
__device__ __forceinline__ void split_mma(const Split8 (&a)[MB], const Split8 &w, f32v4 (&hi)[MB][NB],
                                          f32v4 (&lo)[MB][NB], int j) {
#pragma unroll
  for (int i = 0; i < MB; ++i) lo[i][j] = mfma_bf16(w.l, a[i].h, lo[i][j]);
#pragma unroll
  for (int i = 0; i < MB; ++i) hi[i][j] = mfma_bf16(w.h, a[i].h, hi[i][j]);
#pragma unroll
  for (int i = 0; i < MB; ++i) lo[i][j] = mfma_bf16(w.h, a[i].l, lo[i][j]);
#pragma unroll
  for (int i = 0; i < MB; ++i) lo[i][j] = mfma_bf16(w.m, a[i].m, lo[i][j]);
#pragma unroll
  for (int i = 0; i < MB; ++i) lo[i][j] = mfma_bf16(w.m, a[i].h, lo[i][j]);
#pragma unroll
  for (int i = 0; i < MB; ++i) lo[i][j] = mfma_bf16(w.h, a[i].m, lo[i][j]);
}
__device__ __forceinline__ void split_mma1(const Split8 &a, const Split8 &w, f32v4 &hi, f32v4 &lo) {
  lo = mfma_bf16(w.l, a.h, lo);
  hi = mfma_bf16(w.h, a.h, hi);
  lo = mfma_bf16(w.h, a.l, lo);
  lo = mfma_bf16(w.m, a.m, lo);
  lo = mfma_bf16(w.m, a.h, lo);
  lo = mfma_bf16(w.h, a.m, lo);
}

// Layout of a split weight operand of N rows and K columns (N a multiple of 16, K of 32), in
// the order the instruction reads it: [N / 16][K / 32][h, m, l][64 lanes][8 k].  One (block,
// K step, part) is 1 KB, loaded by one wave-wide 16-byte load and read from LDS at 16 bytes a
// lane without bank conflicts.
constexpr int SPLIT_BLOCK = 3 * 64 * 8;   // bf16 values of one 16 x 32 block

// Column block j of a wave's weights from LDS: ws is the lane's part of the first block, its three
// split parts, or (WF) its first row of float32 weights, laid out as the coefficients below and
// split here, into the same bits.
template <bool WF>
__device__ __forceinline__ Split8 split_weights(const void *ws, int j, int ch0, int ch1) {
  if constexpr (WF) {
    const float *w = static_cast<const float *>(ws) + j * 512;
    return split8(*reinterpret_cast<const f32v4 *>(w + ch0) * SPLIT_SCALE,
                  *reinterpret_cast<const f32v4 *>(w + ch1) * SPLIT_SCALE);
  } else {
    const bf16x8 *w = static_cast<const bf16x8 *>(ws) + j * 192;
    return Split8{w[0], w[64], w[128]};
  }
}

// One K step of a wave from LDS: MB row blocks of coefficients (as: the lane's first row, 32
// floats a row, 16 rows a block, the lane's two 16-byte chunks at ch0 and ch1) times NB column
// blocks of weights (ws, see split_weights), the first nj of which hold real
// columns (wave-uniform).  The first column block multiplies each row block as soon as it is
// split; every block's weights are read from LDS while the block before is multiplied.
template <int MB, int NB, bool ABS, bool WF = false>
__device__ __forceinline__ void split_step(const float *as, int ch0, int ch1, const void *ws, int nj,
                                           uint32_t abs_mask, f32v4 (&hi)[MB][NB], f32v4 (&lo)[MB][NB]) {
  auto load_w = [&](int j) {
    const Split8 w = split_weights<WF>(ws, j, ch0, ch1);
    return ABS ? split_abs(w, abs_mask) : w;
  };
  f32v4 x[MB], y[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    x[i] = *reinterpret_cast<const f32v4 *>(as + i * 512 + ch0);
    y[i] = *reinterpret_cast<const f32v4 *>(as + i * 512 + ch1);
  }
  Split8 a[MB], w[2];
  w[0] = load_w(0);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (j < nj) {
      if (j + 1 < NB) w[(j + 1) & 1] = load_w(j + 1);
      if (j == 0) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          a[i] = split8(x[i], y[i]);
          split_mma1(a[i], w[0], hi[i][0], lo[i][0]);
        }
      } else {
        split_mma<MB, NB>(a, w[j & 1], hi, lo, j);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A K step's operands of a wave in registers, read whole from LDS (the layout of split_step)
template <int MB, int NB>
struct SplitRaw {
  f32v4 x[MB], y[MB];
  Split8 w[NB];
};
template <int MB, int NB, bool ABS, bool WF>
__device__ __forceinline__ void split_read(SplitRaw<MB, NB> &r, const float *as, int ch0, int ch1, const void *ws,
                                           uint32_t abs_mask) {
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    r.x[i] = *reinterpret_cast<const f32v4 *>(as + i * 512 + ch0);
    r.y[i] = *reinterpret_cast<const f32v4 *>(as + i * 512 + ch1);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const Split8 w = split_weights<WF>(ws, j, ch0, ch1);
    r.w[j] = ABS ? split_abs(w, abs_mask) : w;
  }
}
// its products, every accumulator's in split_mma's order
template <int MB, int NB>
__device__ __forceinline__ void split_mma_all(const SplitRaw<MB, NB> &r, f32v4 (&hi)[MB][NB], f32v4 (&lo)[MB][NB]) {
  Split8 a[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) a[i] = split8(r.x[i], r.y[i]);
  auto each = [&](auto &&f) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) f(a[i], r.w[j], hi[i][j], lo[i][j]);
  };
  each([](const Split8 &p, const Split8 &w, f32v4 &, f32v4 &l) { l = mfma_bf16(w.l, p.h, l); });
  each([](const Split8 &p, const Split8 &w, f32v4 &h, f32v4 &) { h = mfma_bf16(w.h, p.h, h); });
  each([](const Split8 &p, const Split8 &w, f32v4 &, f32v4 &l) { l = mfma_bf16(w.h, p.l, l); });
  each([](const Split8 &p, const Split8 &w, f32v4 &, f32v4 &l) { l = mfma_bf16(w.m, p.m, l); });
  each([](const Split8 &p, const Split8 &w, f32v4 &, f32v4 &l) { l = mfma_bf16(w.m, p.h, l); });
  each([](const Split8 &p, const Split8 &w, f32v4 &, f32v4 &l) { l = mfma_bf16(w.h, p.m, l); });
}

// ---- results out of the split range --------------------------------------------------------
// 16 x 16 results in float32, the lane's four as mfma_bf16 leaves them: n contraction values
// from the lane's two rows, a of coefficients and w of weights (|w| with mask 0x7fffffff), which
// are 16-byte aligned and readable up to the next multiple of 16 values; a lane's null a is a row
// of zeros.
__device__ __forceinline__ f32v4 mma_float32(const float *a, const float *w, int n, int g4, uint32_t mask, f32v4 acc) {
  for (int k = 4 * g4; k - 4 * g4 < n; k += 16) {   // as many rounds in every lane
    const f32v4 y = *reinterpret_cast<const f32v4 *>(w + k);
    f32v4 x = {0.f, 0.f, 0.f, 0.f};
    if (a) x = *reinterpret_cast<const f32v4 *>(a + k);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float yq = y[q];   // (a bit cast of the vector's element itself takes element 0)
      const float u = k + q < n ? x[q] : 0.f;
      const float v = k + q < n ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, yq) & mask) : 0.f;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v, u, acc, 0, 0, 0);
    }
  }
  return acc;
}

// A wave's results, hi + lo of every element, times a factor (returned, wave-uniform, left to the
// caller's next multiply-add).  Elements that are not finite are replaced by their float32 values.
// One multiply-add of two elements finds them (its sum is not finite then, nor where products
// of elements overflow); the blocks that do hold one, in a row that counts (row_ok(i)), are taken
// again one after the other, by again(i, j).  Columns from N on are padding, whose weights are zero,
// and give zero.  The replacement is by element, so a result does not depend on its tile.
template <int MB, int NB, class RowOk, class Again>
__device__ __forceinline__ float split_finish(f32v4 (&v)[MB][NB], const f32v4 (&lo)[MB][NB], int col0, int N, int g4,
                                              RowOk &&row_ok, Again &&again) {
  auto finite = [](float x) { return fabsf(x) < __builtin_huge_valf(); };
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      v[i][j] += lo[i][j];
      s = fmaf(v[i][j][2], v[i][j][3], fmaf(v[i][j][0], v[i][j][1], s));
    }
    bad |= !finite(s) && row_ok(i);
  }
  if (__builtin_expect(!__any(bad), 1)) return SPLIT_UNSCALE;
  uint32_t need = 0;   // a bit per block, wave-uniform
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32v4 q = v[i][j] *= SPLIT_UNSCALE;
      const bool b = !(finite(q[0]) && finite(q[1]) && finite(q[2]) && finite(q[3])) && row_ok(i);
      need |= (uint32_t)(__any(b) != 0) << (i * NB + j);
    }
#pragma unroll 1
  while (need) {
    const int b = __builtin_amdgcn_readfirstlane(__builtin_ctz(need));
    need &= need - 1;
    const f32v4 x = again(b / NB, b % NB);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (b == i * NB + j) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (!finite(v[i][j][q])) v[i][j][q] = col0 + 16 * j + 4 * g4 + q < N ? x[q] : 0.f;
        }
  }
  return 1.f;
}

}  // namespace vcr
