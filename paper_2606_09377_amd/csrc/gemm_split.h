// The dense backward, forward and IBP steps on split operands (split_bf16.h).  Part of gemm.hip.
//
// A workgroup owns a BM x BN tile of the output, WM x WN waves of (BM / WM) x (BN / WN), in
// 16 x 16 blocks.  Per K step of 32 the coefficient rows (float32, 128 bytes a row) and the
// weights' three parts go from global memory straight into double-buffered LDS; a wave splits
// its coefficient rows into bf16 parts in registers (5.5 vector instructions a value, under
// the matrix instructions of the other wave of its SIMD) and multiplies.
//
// WF: a layer without split weights in memory (GemmArgs.Bs null: the device had no room for them, or
// the caller wants none) has its float32 weights staged like the coefficients and split by every
// wave that multiplies them: the same bits, without the memory, at the cost of those
// instructions (784-1024x6 MLP, 64 inputs: 21.8 against 18.6 ms with split weights and 30.4 on the
// float32 instructions; one input, a chain on small tiles: 0.97 against 0.64 and 0.89).
//
// The coefficients stay float32 in memory (splitting them where they are produced would save
// those instructions but cost half as much memory again, in traffic and in workspace).
#pragma once

#include "split_bf16.h"

namespace vcr {

// The tile shapes, by launch size; every shape gives the same bits.
//   SplitL  128 x 128, 4 waves of 64 x 64, two stages of 40 KB: two workgroups per compute unit
//   SplitM  64 x 64, 4 waves of 16 x 64
//   SplitS  32 x 64, 4 waves of 16 x 32, three stages: a long contraction on one or two
//           workgroups per compute unit waits on nothing but its own chain (1024 x 1024 outputs over
//           K = 65536: 1465 us with two stages and LDS reads in line, 1277 us)
template <int BM_, int BN_, int WM_, int WN_, int NS_, int MINB_, bool PIPE_ = false>
struct SplitTile {
  static constexpr bool PIPE = PIPE_;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_, MINB = MINB_;
  static constexpr int NW = WM * WN, T = 64 * NW;
  static constexpr int MB = BM / WM / 16, NB = BN / WN / 16;   // 16 x 16 blocks of a wave
  static constexpr int A_FLOATS = BM * 32, B_FLOATS = BN / 16 * SPLIT_BLOCK / 2;   // a stage
  static_assert(BN * 32 <= B_FLOATS, "float32 weights fit the stage of their split parts");
  static constexpr int LDS_FLOATS = NS * (A_FLOATS + B_FLOATS);
};
typedef SplitTile<128, 128, 2, 2, 2, 2> SplitL;
typedef SplitTile<64, 64, 4, 1, 2, 2> SplitM;
typedef SplitTile<32, 64, 2, 2, 3, 2, true> SplitS;

// Parameters of four consecutive columns for one coefficient row, with the row's split neuron
// (if any) replaced.  flags: the tile's split table (four entries of the row's domain), or null
// for the walk over the domain's entries.
__device__ __forceinline__ void split_params4(const GemmArgs &p, const TileSplits &ts, int row, int n,
                                              float4 (&prm)[4], int (&ent)[4], float (&sterm)[4]) {
  if (ts.flags) {
    int d = row / p.splits.rows_per_domain;
    d = d < p.splits.D ? d : p.splits.D - 1;
    const int f = *reinterpret_cast<const int *>(ts.flags + (d - ts.d0) * ts.cols + (n - ts.n0));
    if (f == -1) return;   // none of the four columns
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) prm[v] = split_lookup(p.splits, ts, row, p.relu_index, n + v, prm[v], &ent[v], &sterm[v]);
}

// Epilogue of one wave: MB x NB blocks from tile-relative row wrow and column col0.  A lane
// holds, of coefficient row m0 + wrow + 16 i + lane % 16, the four columns
// col0 + 16 j + 4 (lane / 16) + v.
//
// Row sums (the constant terms): per block the lane's four terms in column order, then the four
// blocks of a 64-column slab in order, then the four lanes of a row; a wave narrower than a
// slab hands its block sums to the slab's reduction through LDS (xp), in that same order.
template <class TS, bool FWD, bool AL, bool AFF>
__device__ __forceinline__ void split_epilogue(const GemmArgs &p, f32v4 (&acc)[TS::MB][TS::NB], int m0, int wm, int wn,
                                               int n0, int lane, float *lds) {
  constexpr int MB = TS::MB, NB = TS::NB;
  constexpr bool WIDE = NB % 4 == 0;   // the wave holds whole slabs
  const int r16 = lane & 15, g4 = lane >> 4;
  const int wrow = wm * (TS::BM / TS::WM), col0 = n0 + wn * (TS::BN / TS::WN);
  TileSplits ts{nullptr, 0, n0, TS::BN};
  if (!AFF && p.mode != EPI_CONCRETIZE)
    ts = tile_splits_build(p.splits, p.relu_index, m0, TS::BM, n0, TS::BN, reinterpret_cast<signed char *>(lds));
  const bool has_splits = p.splits.D > 0;
  const int64_t ld = p.mode == EPI_CONCRETIZE ? p.ld_pre : p.ldo;
  const int u_first = min((m0 + wrow) / p.rows_per_unit, p.n_units - 1);
  const int u_last = min((m0 + wrow + 16 * MB - 1) / p.rows_per_unit, p.n_units - 1);
  const bool one_unit = u_first == u_last;   // wave-uniform
  // restrict-qualified copies: loads of later rows may go ahead of earlier stores
  const float4 *__restrict__ Pp = p.P;
  const float *__restrict__ alpha = p.alpha;
  float *__restrict__ pre = p.pre;
  float *__restrict__ out = p.out;
  float *__restrict__ grad = p.grad;
  float *__restrict__ gbeta = p.splits.grad_beta;
  const float *__restrict__ sbeta = p.splits.beta;

  float slab[MB][WIDE ? NB / 4 : NB];   // WIDE: slab sums; else block sums
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int s = 0; s < (WIDE ? NB / 4 : NB); ++s) slab[i][s] = 0.f;

  int urow[MB];   // unit of each of the lane's rows (when they differ)
#pragma unroll
  for (int i = 0; i < MB; ++i)
    urow[i] = one_unit ? u_first : min((m0 + wrow + 16 * i + r16) / p.rows_per_unit, p.n_units - 1);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = col0 + 16 * j + 4 * g4;
    float4 prm_u[4];
    float4 c_u = make_float4(0.f, 0.f, 0.f, 0.f), r_u = c_u;
    if constexpr (AFF) {
      if (p.bias) c_u = *reinterpret_cast<const float4 *>(p.bias + n);
    } else if (p.mode != EPI_CONCRETIZE) {
#pragma unroll
      for (int v = 0; v < 4; ++v) prm_u[v] = Pp[(int64_t)u_first * p.ldp + n + v];
    } else {
      c_u = *reinterpret_cast<const float4 *>(p.c0 + (int64_t)u_first * p.ldc + n);
      r_u = *reinterpret_cast<const float4 *>(p.r0 + (int64_t)u_first * p.ldc + n);
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = m0 + wrow + 16 * i + r16;
      const int64_t off = (int64_t)row * ld + n;
      const f32v4 a = acc[i][j];
      if constexpr (AFF) {
        *reinterpret_cast<float4 *>(out + off) = make_float4(a[0] + c_u.x, a[1] + c_u.y, a[2] + c_u.z, a[3] + c_u.w);
      } else if (FWD || p.mode == EPI_RELAX) {
        float4 prm[4] = {prm_u[0], prm_u[1], prm_u[2], prm_u[3]};
        if (!one_unit) {
#pragma unroll
          for (int v = 0; v < 4; ++v) prm[v] = Pp[(int64_t)urow[i] * p.ldp + n + v];
        }
        int ent[4] = {-1, -1, -1, -1};
        float sterm[4] = {0.f, 0.f, 0.f, 0.f};
        if (has_splits) split_params4(p, ts, row, n, prm, ent, sterm);
        float o[4];
        if constexpr (FWD) {
          // the relaxed network evaluated forward: D = W_k E + b_k, then the line of ReLU k
          // that the backward pass chose for this row (by the sign of its coefficient)
          const f32v4 al = *reinterpret_cast<const f32v4 *>(alpha + off);
          const f32v4 an = *reinterpret_cast<const f32v4 *>(pre + off);
          float gr[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const bool unst = prm[v].z > 0.f;
            const float lam = unst ? al[v] : prm[v].x;
            const float D = a[v] + prm[v].w;
            if (ent[v] >= 0 && gbeta) gbeta[(int64_t)row * p.splits.S + ent[v]] = sterm[v] * D;
            o[v] = an[v] > 0.f ? lam * D : fmaf(prm[v].y, D, an[v] < 0.f ? prm[v].z : 0.f);
            gr[v] = (unst && an[v] > 0.f) ? an[v] * D : 0.f;
          }
          *reinterpret_cast<float4 *>(grad + off) = make_float4(gr[0], gr[1], gr[2], gr[3]);
        } else {
          f32v4 al = {0.f, 0.f, 0.f, 0.f};
          if constexpr (AL) {
            if (alpha) al = *reinterpret_cast<const f32v4 *>(alpha + off);
          }
          float x = 0.f;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            float lam = prm[v].x;
            if constexpr (AL) {
              if (alpha) lam = prm[v].z > 0.f ? al[v] : lam;
            }
            float ap = a[v] > 0.f ? a[v] * lam : a[v] * prm[v].y;
            if constexpr (AL) {
              if (ent[v] >= 0 && sbeta) ap = fmaf(sbeta[(int64_t)row * p.splits.S + ent[v]], sterm[v], ap);
            }
            o[v] = ap;
            x += fmaf(ap, prm[v].w, fminf(a[v], 0.f) * prm[v].z);
          }
          slab[i][WIDE ? j / 4 : j] += x;
          if constexpr (AL) {
            if (pre) *reinterpret_cast<f32v4 *>(pre + off) = a;
          }
        }
        *reinterpret_cast<float4 *>(out + off) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
        float4 c = c_u, r = r_u;
        if (!one_unit) {
          c = *reinterpret_cast<const float4 *>(p.c0 + (int64_t)urow[i] * p.ldc + n);
          r = *reinterpret_cast<const float4 *>(p.r0 + (int64_t)urow[i] * p.ldc + n);
        }
        if constexpr (AL) {
          if (pre) *reinterpret_cast<f32v4 *>(pre + off) = a;
        }
        float x = fmaf(a[0], c.x, -(fabsf(a[0]) * r.x));
        x += fmaf(a[1], c.y, -(fabsf(a[1]) * r.y));
        x += fmaf(a[2], c.z, -(fabsf(a[2]) * r.z));
        x += fmaf(a[3], c.w, -(fabsf(a[3]) * r.w));
        slab[i][WIDE ? j / 4 : j] += x;
      }
    }
  }
  if constexpr (FWD || AFF) return;
  // slabs that hold the sums of an earlier step of this pass are added to
  auto add_part = [&](int s, int row, float x) {
    float *d = p.part + (int64_t)s * p.M_pad + row;
    *d = p.mode == EPI_RELAX && s < p.part_slabs ? *d + x : x;
  };
  if constexpr (WIDE) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int s = 0; s < NB / 4; ++s) {
        float x = slab[i][s];
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        if (g4 == 0) add_part(col0 / PART_COLS + s, m0 + wrow + 16 * i + r16, x);
      }
  } else {
    static_assert(WIDE || TS::BN % PART_COLS == 0, "a workgroup holds whole slabs");
    float *xp = lds + SPLIT_ND * TS::BN / 4;   // after the split table: [BN / 16 blocks][BM rows][4]
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) xp[((wn * NB + j) * TS::BM + wrow + 16 * i + r16) * 4 + g4] = slab[i][j];
    __syncthreads();
    for (int t = threadIdx.x; t < TS::BN / PART_COLS * TS::BM * 4; t += TS::T) {
      const int s = t / (TS::BM * 4), q = t - s * (TS::BM * 4);   // q = row, lane of the row
      const float *b = xp + s * 4 * (TS::BM * 4) + q;
      float x = b[0] + b[TS::BM * 4];
      x += b[2 * TS::BM * 4];
      x += b[3 * TS::BM * 4];
      x += __shfl_xor(x, 1);
      x += __shfl_xor(x, 2);
      if ((q & 3) == 0) add_part(n0 / PART_COLS + s, m0 + (q >> 2), x);
    }
  }
}

template <class TS, bool FWD, bool AL, bool AFF, bool WF>
__global__ __launch_bounds__(TS::T, TS::MINB) void k_gemm_split(const GemmArgs p) {
  constexpr int MB = TS::MB, NB = TS::NB, NS = TS::NS, NW = TS::NW;
  __shared__ __attribute__((aligned(16))) float lds[TS::LDS_FLOATS];
  float *As = lds, *Bs = lds + NS * TS::A_FLOATS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % TS::WM, wn = wave / TS::WM;
  const int n_mt = (p.M + TS::BM - 1) / TS::BM, n_nt = p.N_pad / TS::BN;
  int mt, nt;
  map_tile(blockIdx.x, n_mt * n_nt, n_mt, n_nt, mt, nt);
  const int m0 = mt * TS::BM, n0 = nt * TS::BN;
  // K steps and 16-column blocks that hold real values; the rest is zero padding
  const int KT = n0 < p.N ? (p.K_real + 31) / 32 : 0;
  const int nj = min(max((p.N - (n0 + wn * (TS::BN / TS::WN)) + 15) / 16, 0), NB);   // wave-uniform

  // One load of a wave fills 1 KB of LDS in lane order: 8 coefficient rows (lane = row, 16-byte
  // chunk; the chunk that lands in a slot is swizzled by lds_swz, the swizzle applied on the
  // fetch side), or as many rows of float32 weights, or one part of a 16-column block of weights.
  // (By the counters each 16-byte read of coefficients still spends 4 cycles on bank conflicts, a
  // read of split weights none.)
  constexpr int AI = TS::BM / 8, BI = WF ? TS::BN / 8 : 3 * (TS::BN / 16);
  constexpr int AQ = AI / NW, BQ = BI / NW;
  static_assert(AI % NW == 0 && BI % NW == 0, "loads spread evenly over the waves");
  const int kblocks = p.K / 32;
  uint32_t a_off[AQ];   // bytes from the tile's first row, under 2^32 (use_split)
#pragma unroll
  for (int q = 0; q < AQ; ++q) {
    const int row = (q * NW + wave) * 8 + (lane >> 3);
    a_off[q] = (uint32_t)row * (uint32_t)(p.lda * 4) + ((lane & 7) ^ lds_swz<32>(row)) * 16;
  }
  const float *a_tile = p.A + (int64_t)m0 * p.lda;
  const float *w_tile = p.Bt + (int64_t)n0 * p.ldb;
  const uint16_t *b_tile = WF ? nullptr : p.Bs + (int64_t)(n0 / 16) * kblocks * SPLIT_BLOCK;
  auto issue = [&](int kt, int buf) {
#pragma unroll
    for (int q = 0; q < AQ; ++q) dma16(a_tile + kt * 32, a_off[q], As + buf * TS::A_FLOATS + (q * NW + wave) * 256);
#pragma unroll
    for (int q = 0; q < BQ; ++q) {
      const int i = q * NW + wave;
      if constexpr (WF) {
        const int row = i * 8 + (lane >> 3);
        dma16(w_tile + kt * 32, (uint32_t)row * (uint32_t)(p.ldb * 4) + ((lane & 7) ^ lds_swz<32>(row)) * 16,
              Bs + buf * TS::B_FLOATS + i * 256);
      } else {
        const int nb = i / 3, part = i - 3 * nb;
        dma16(b_tile + ((int64_t)nb * kblocks + kt) * SPLIT_BLOCK + part * 512, (uint32_t)lane * 16,
              Bs + buf * TS::B_FLOATS + i * 256);
      }
    }
  };
  [[maybe_unused]] constexpr int LPT = AQ + BQ;   // loads of a wave per K step

  f32v4 hi[MB][NB], lo[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) hi[i][j] = lo[i][j] = f32v4{0.f, 0.f, 0.f, 0.f};

  const int r16 = lane & 15, g4 = lane >> 4, sw = lds_swz<32>(r16);
  const uint32_t abs_mask = AFF && p.abs_b ? 0x80008000u : 0u;
  const int ch0 = ((2 * g4) ^ sw) * 4, ch1 = ((2 * g4 + 1) ^ sw) * 4;
  // the lane's part of the wave's first column block in a stage
  const float *b_lane = Bs + (WF ? (wn * NB * 16 + r16) * 32 : (wn * NB * 192 + lane) * 4);
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < KT) issue(s, s);
  if constexpr (TS::PIPE) {
    // A few waves alone on a compute unit: step kt + 1's operands are read from LDS while step kt
    // is split and multiplied.  A step's operands are all in registers by the barrier, so the
    // barrier that publishes step kt + 1 also frees step kt's stage for step kt + NS.  (Two
    // register sets, the loop unrolled by two, so that no set is copied.)
    const float *as = As + (wm * (TS::BM / TS::WM) + r16) * 32;
    auto read = [&](int buf, SplitRaw<MB, NB> &r) {
      split_read<MB, NB, AFF, WF>(r, as + buf * TS::A_FLOATS, ch0, ch1, b_lane + buf * TS::B_FLOATS, abs_mask);
    };
    static_assert(NS == 3, "one step in flight behind the one waited for");
    int cur = 0;   // step kt's stage
    auto step = [&](int kt, const SplitRaw<MB, NB> &now, SplitRaw<MB, NB> &next) {
      const int nxt = cur + 1 == NS ? 0 : cur + 1;
      if (kt + 1 < KT) {
        if (kt + 2 < KT) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
        barrier_only();
        if (kt + NS < KT) issue(kt + NS, cur);
        read(nxt, next);
      }
      split_mma_all<MB, NB>(now, hi, lo);
      cur = nxt;
    };
    SplitRaw<MB, NB> r0, r1;
    if (KT > 0) {
      if (NS - 1 < KT) issue(NS - 1, NS - 1);
      if (KT >= NS) wait_vmcnt<2 * LPT>();   // the first step has landed, the other stages' are in flight
      else if (KT == 2) wait_vmcnt<LPT>();
      else wait_vmcnt<0>();
      barrier_only();
      read(0, r0);
    }
    for (int kt = 0; kt < KT; kt += 2) {
      step(kt, r0, r1);
      if (kt + 1 < KT) step(kt + 1, r1, r0);
    }
  } else {
    static_assert(NS == 2, "no step in flight behind the one waited for");
    int cur = 0;
    for (int kt = 0; kt < KT; ++kt) {
      wait_vmcnt<0>();   // this wave's part of step kt has landed
      barrier_only();    // every wave's has, and step kt - 1's stage is free
      if (kt + 1 < KT) issue(kt + 1, cur ^ 1);
      const float *as = As + cur * TS::A_FLOATS + (wm * (TS::BM / TS::WM) + r16) * 32;
      split_step<MB, NB, AFF, WF>(as, ch0, ch1, b_lane + cur * TS::B_FLOATS, nj, abs_mask, hi, lo);
      cur ^= 1;
    }
  }
  {
    const int row0 = wm * (TS::BM / TS::WM) + r16, col0 = n0 + wn * (TS::BN / TS::WN);
    const float unscale = split_finish<MB, NB>(
        hi, lo, col0, p.N, g4, [&](int i) { return m0 + row0 + 16 * i < p.M; },
        [&](int i, int j) {
          return mma_float32(a_tile + (int64_t)(row0 + 16 * i) * p.lda, w_tile + (int64_t)(col0 - n0 + 16 * j + r16) * p.ldb,
                             p.K_real, g4, AFF && p.abs_b ? 0x7fffffffu : 0xffffffffu, f32v4{0.f, 0.f, 0.f, 0.f});
        });
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) hi[i][j] *= unscale;
  }
  __syncthreads();   // every wave is done with the operand buffers, which the epilogue reuses
  split_epilogue<TS, FWD, AL, AFF>(p, hi, m0, wm, wn, n0, lane, lds);
}

// Split copy of the weights src [N][K] (float32, pitch ld): a thread per 8 consecutive k
__global__ void k_split_weights(const float *src, int64_t ld, int64_t N, int64_t K, uint16_t *dst) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = K / 8;
  if (t >= N * per) return;
  const int64_t row = t / per;
  const int64_t k = (t - row * per) * 8;
  const f32v4 x = *reinterpret_cast<const f32v4 *>(src + row * ld + k);
  const f32v4 y = *reinterpret_cast<const f32v4 *>(src + row * ld + k + 4);
  const Split8 s = split8(x * SPLIT_SCALE, y * SPLIT_SCALE);
  const int lane = (int)((k & 31) >> 3) * 16 + (int)(row & 15);
  bf16x8 *o = reinterpret_cast<bf16x8 *>(dst + ((row >> 4) * (K >> 5) + (k >> 5)) * SPLIT_BLOCK) + lane;
  o[0] = s.h;
  o[64] = s.m;
  o[128] = s.l;
}

hipError_t launch_split_weights(const float *src, int64_t ld, int64_t N, int64_t K, uint16_t *dst, hipStream_t s) {
  if (N <= 0 || K <= 0 || N % 16 || K % 32 || ld % 4 || ld < K) return hipErrorInvalidValue;
  const int64_t tot = N * (K / 8);
  if ((tot + 255) / 256 > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_weights, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, src, ld, N, K, dst);
  return hipGetLastError();
}

template <class TS, bool WF>
static hipError_t launch_split_tile(const GemmArgs &a, hipStream_t s) {
  const int64_t grid = (int64_t)((a.M + TS::BM - 1) / TS::BM) * (a.N_pad / TS::BN);
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 g((unsigned)grid), t(TS::T);
  if (a.mode == EPI_AFFINE)
    hipLaunchKernelGGL((k_gemm_split<TS, false, false, true, WF>), g, t, 0, s, a);
  else if (a.mode == EPI_FORWARD)
    hipLaunchKernelGGL((k_gemm_split<TS, true, true, false, WF>), g, t, 0, s, a);
  else if (a.alpha || a.pre)
    hipLaunchKernelGGL((k_gemm_split<TS, false, true, false, WF>), g, t, 0, s, a);
  else
    hipLaunchKernelGGL((k_gemm_split<TS, false, false, false, WF>), g, t, 0, s, a);
  return hipGetLastError();
}

template <class TS>
static hipError_t launch_split_tile(const GemmArgs &a, hipStream_t s) {
  return a.Bs ? launch_split_tile<TS, false>(a, s) : launch_split_tile<TS, true>(a, s);
}

// The split kernels address a tile of coefficient or weight rows by 32-bit byte offsets; longer
// rows are multiplied in float32, like those of a caller who asks for it.
static bool use_split(const GemmArgs &a) { return !a.float32 && std::max(a.lda, a.ldb) <= (int64_t)1 << 23; }

// 0: SplitL, 3: SplitM, 2: SplitS.  In its own loop (K = 1024, N = 1024) SplitL reaches 228
// TFLOP/s and SplitM 187; SplitL holds 512 workgroups on the chip at once, so it runs where its
// rounds of 512 are full enough to keep that lead.  SplitS runs up to 256 tiles of 64 x 64, two
// of its own per compute unit; beyond, its third one costs more than SplitM's larger tile (us, SplitS
// against SplitM, at 256 and at 320 tiles: K = 512 12.7 / 12.5 and 16.0 / 14.4, K = 1024 20.6 / 21.5
// and 26.9 / 23.8, K = 8192 133 / 141 and 179 / 154, K = 32768 552 / 714 and 683 / 717; at 384 SplitM
// leads by 5 to 27%).
static int split_kind(const GemmArgs &a) {
  const int64_t big = (int64_t)((a.M + 127) / 128) * (a.N_pad / 128);
  const int64_t rounds = (big + 511) / 512;
  if (big >= 512 && big * 100 >= rounds * 512 * 82) return 0;
  const int64_t mid = (int64_t)((a.M + 63) / 64) * (a.N_pad / 64);
  return mid > 256 ? 3 : 2;
}

}  // namespace vcr
