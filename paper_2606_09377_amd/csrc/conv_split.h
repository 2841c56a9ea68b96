// The transposed convolution and the gradient pass's forward convolution on split operands
// (split_bf16.h), run unless the network was loaded with float32 products.  Part of conv.hip.
//
// The same implicit GEMMs as k_convt and k_fwd_conv (rows, position classes, taps, epilogues),
// with K steps of 32 channels of one tap: a step gathers 128 contiguous bytes of each of the
// tile's source positions (one cache line, where the 16-channel steps of the float32 kernels
// read two halves) and the weights' three parts, straight into double-buffered LDS.  Waves of
// 32 x 64: three share a 96 x 64 tile (54 KB: three workgroups per compute unit), eight a 128 x
// 128 one.  The 64-column tile is that small for the sake of those workgroups: on the 3 x 32 x
// 32 ResNet a 128-row one (two workgroups) spends 19 us in its K loop, at 233 TFLOP/s, and as
// much before and after it, which only other workgroups' K loops can hide.  The 128-column tile
// has twice the K loop: 96 rows (two workgroups) took 255 us a dispatch there, 128 rows 207.
#pragma once

#include "split_bf16.h"

namespace vcr {

template <int WN>
struct ConvSplit {
  static constexpr int BM = WN == 1 ? 96 : 128;              // GEMM rows per workgroup
  static constexpr int WM = BM / 32, NW = WM * WN, T = 64 * NW, BN = 64 * WN;
  static constexpr int MINB = WN == 1 ? 3 : 2;               // waves per SIMD the registers are sized for
  static constexpr int MB = 2, NB = 4;                       // a wave: 32 rows x 64 columns
  static constexpr int A_FLOATS = BM * 32, B_FLOATS = BN / 16 * SPLIT_BLOCK / 2;
  static constexpr int AQ = BM / 8 / NW, BQ = 3 * (BN / 16) / NW;   // loads of a wave per K step
  static_assert(BM / 8 % NW == 0 && 3 * (BN / 16) % NW == 0, "loads spread evenly over the waves");
};

// Four consecutive channels of one destination position: the split neurons of the row's domain
// among them (their relaxation replaces prm; ent, sterm as in split_override)
__device__ __forceinline__ void split_override4(const SplitTable &st, int row, int relu, int n, float4 (&prm)[4],
                                                int (&ent)[4], float (&sterm)[4]) {
  int d = row / st.rows_per_domain;
  d = d < st.D ? d : st.D - 1;
  const int e0 = st.off[d * (st.R + 1) + relu];
  const int e1 = st.off[d * (st.R + 1) + relu + 1];
  for (int e = e0; e < e1; ++e) {
    const int v = st.ent_n[d * st.S + e] - n;
    if (v < 0 || v > 3) continue;
    const float4 q = st.ent_p[d * st.S + e];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k == v) {
        prm[k] = make_float4(q.x, q.y, q.z, prm[k].w);
        ent[k] = e;
        sterm[k] = q.w;
      }
  }
}

// What the epilogue needs of a tile row, computed once per workgroup while the first K step is
// in flight: output and residual offsets (residual -1: none), parameter offset (-1 outside the
// image), partial-sum index (-1 past the last row) and coefficient row.
// Sized for the tile: at 128 rows it takes the third workgroup of 96-row tiles off a compute
// unit (3 x 32 x 32 ResNet, two inputs: 55.6 against 47.4 ms).
template <int ROWS>
struct ConvRows {
  int64_t ob[ROWS], rb[ROWS];
  int pb[ROWS], mo[ROWS], r[ROWS];
  uint32_t yx[ROWS];   // iy, ix, anchor y, anchor x, a byte each
};

template <int ROWS>
__device__ __forceinline__ void conv_row_info(const ConvTArgs &p, const ConvClass &cl, ConvRows<ROWS> &rows, int m0, int tr) {
  const bool valid = m0 + tr < cl.M;
  const int r = rows.r[tr];
  const uint32_t yx = rows.yx[tr];
  const int u = cl.u0 + (int)(yx & 255) * cl.ustep;
  const int w = cl.w0 + (int)((yx >> 8) & 255) * cl.wstep;
  const int4 an = p.rows[r];   // (unit, anchor y, anchor x, -)
  const int gy = p.dense ? u : an.y * p.scale - p.h_in + u;
  const int gx = p.dense ? w : an.z * p.scale - p.h_in + w;
  const bool inside = valid && gy >= 0 && gx >= 0 && gy < p.H_in && gx < p.H_in;
  const int du = u - p.res_off, dw = w - p.res_off;
  rows.mo[tr] = valid ? r * (p.S_in * p.S_in) + u * p.S_in + w : -1;
  rows.ob[tr] = (int64_t)r * p.row_stride_in + ((int64_t)u * p.S_in + w) * p.C_in;
  rows.pb[tr] = inside ? ((an.x * p.H_in + gy) * p.H_in + gx) * p.C_in : -1;
  rows.rb[tr] = inside && p.res && du >= 0 && dw >= 0 && du < p.res_S && dw < p.res_S
                    ? (int64_t)r * p.res_row_stride + ((int64_t)du * p.res_S + dw) * p.C_in
                    : -1;
}

// Epilogue of the transposed convolution (see convt_epilogue): a lane holds, of GEMM rows
// 16 i + lane % 16 of its wave, channels 16 j + 4 (lane / 16) .. + 3.  The relaxation parameters
// or residuals are loaded four blocks ahead: with one block ahead the eight blocks of a wave
// were eight waits on the L2.  finish() completes acc, up to the
// factor it returns, under the first of those loads.
template <int WN, bool RELU, bool AL, bool SPL, class Finish>
__device__ __forceinline__ void convt_split_epilogue(const ConvTArgs &p, const f32v4 (&acc)[2][4],
                                                     const ConvRows<ConvSplit<WN>::BM> &rows,
                                                     int n0, int nt, int wm, int wn, int nj, Finish &&finish) {
  typedef ConvSplit<WN> CS;
  constexpr int MB = CS::MB, NB = CS::NB;
  const int lane = threadIdx.x & 63, r16 = lane & 15, g4 = lane >> 4;
  const float4 *__restrict__ Pp = p.P_pos;
  const float *__restrict__ resp = p.res;
  float *__restrict__ outp = p.out;
  const float *__restrict__ alp = p.alpha;
  float *__restrict__ prep = p.pre;
  const int nw = n0 + wn * 64 + 4 * g4;   // the lane's first channel
  const int lr0 = wm * 32 + r16;
  float4 prm[NB][4];
  f32v4 rv[NB];
  // positions outside the image read parameter 0 (it meets a zero coefficient)
  auto fetch = [&](int i, int j) {
    const int lr = lr0 + i * 16, n = nw + j * 16;
    if constexpr (RELU) {
      const uint32_t off = rows.pb[lr] >= 0 ? (uint32_t)(rows.pb[lr] + n) : 0u;
#pragma unroll
      for (int v = 0; v < 4; ++v) prm[j][v] = Pp[off + v];
    }
    rv[j] = f32v4{0.f, 0.f, 0.f, 0.f};
    if (resp) rv[j] = *reinterpret_cast<const f32v4 *>(rows.rb[lr] >= 0 ? resp + rows.rb[lr] + n : g_zero4);
  };
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j < nj) fetch(0, j);
  const float unscale = finish();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int lr = lr0 + i * 16;
    const int pb = rows.pb[lr], mo = rows.mo[lr], rr = rows.r[lr];
    const int64_t ob = rows.ob[lr];
    float x = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j >= nj) continue;   // columns past C_in
      const int n = nw + j * 16;
      f32v4 a;
#pragma unroll
      for (int v = 0; v < 4; ++v) a[v] = fmaf(acc[i][j][v], unscale, rv[j][v]);
      float4 pr[4] = {prm[j][0], prm[j][1], prm[j][2], prm[j][3]};
      if (i + 1 < MB) fetch(i + 1, j);
      f32v4 o = {0.f, 0.f, 0.f, 0.f};
      if (pb >= 0) {   // inside the image: relax (or identity) and constant terms
        if constexpr (RELU) {
          int ent[4] = {-1, -1, -1, -1};
          float sterm[4] = {0.f, 0.f, 0.f, 0.f};
          if constexpr (SPL) {   // subdomains: a split neuron's clamped relaxation
            if (mo >= 0) split_override4(p.splits, rr, p.relu_index, pb + n, pr, ent, sterm);
          }
          f32v4 al = {0.f, 0.f, 0.f, 0.f};
          if constexpr (AL) {   // alpha-CROWN: the row's own slopes at unstable neurons; the
                                // coefficients before relaxation are recorded (the gradient pass
                                // uses them at unstable neurons only)
            if (mo >= 0 && fmaxf(fmaxf(pr[0].z, pr[1].z), fmaxf(pr[2].z, pr[3].z)) > 0.f) {
              al = *reinterpret_cast<const f32v4 *>(alp + ob + n);
              *reinterpret_cast<f32v4 *>(prep + ob + n) = a;
            }
          }
          float xb = 0.f;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float lam = AL && pr[v].z > 0.f ? al[v] : pr[v].x;
            float ap = a[v] > 0.f ? a[v] * lam : a[v] * pr[v].y;
            if constexpr (SPL) {   // beta-CROWN: the split's multiplier term
              if (ent[v] >= 0 && p.splits.beta)
                ap = fmaf(p.splits.beta[(int64_t)rr * p.splits.S + ent[v]], sterm[v], ap);
            }
            o[v] = ap;
            xb += fmaf(ap, pr[v].w, fminf(a[v], 0.f) * pr[v].z);
          }
          x += xb;
        } else {
          const float4 bn = *reinterpret_cast<const float4 *>(p.bias + n);
          o = a;
          x += fmaf(a[3], bn.w, fmaf(a[2], bn.z, fmaf(a[1], bn.y, a[0] * bn.x)));
        }
      }
      // (ordinary stores: a lane's 16 bytes and its three neighbours' make half a line, and the
      // cache joins the halves of blocks j and j + 1; non-temporal ones measured 3% slower)
      if (mo >= 0) *reinterpret_cast<f32v4 *>(outp + ob + n) = o;
    }
    x += __shfl_xor(x, 16);
    x += __shfl_xor(x, 32);
    if (g4 == 0 && mo >= 0) p.part[(int64_t)(nt * WN + wn) * p.M_pad + mo] = x;
  }
}

// The source window of a tile row: its position under a zero shift, and the positions that lie
// inside the window and, of a windowed source, inside the image
struct ConvSource {
  int iy, ix, ylo, yhi, xlo, xhi;
};
__device__ __forceinline__ ConvSource convt_source(const ConvTArgs &p, uint32_t yx) {
  ConvSource s{(int)(yx & 255), (int)((yx >> 8) & 255), 0, p.S_out, 0, p.S_out};
  if (p.src_scale > 0) {   // windowed source (Ha > 0)
    const int oy = (int)((yx >> 16) & 255) * p.src_scale - p.src_h, ox = (int)(yx >> 24) * p.src_scale - p.src_h;
    s.ylo = max(0, -oy);
    s.xlo = max(0, -ox);
    s.yhi = min(p.S_out, p.H_out - oy);
    s.xhi = min(p.S_out, p.H_out - ox);
  }
  return s;
}

template <int WN, bool RELU, bool AL, bool SPL>
__global__ __launch_bounds__(ConvSplit<WN>::T, ConvSplit<WN>::MINB) void k_convt_split(const ConvTArgs p) {
  typedef ConvSplit<WN> CS;
  constexpr int MB = CS::MB, NB = CS::NB;
  __shared__ __attribute__((aligned(16))) float lds[2 * (CS::A_FLOATS + CS::B_FLOATS)];
  __shared__ ClipTab tab;
  __shared__ ConvRows<CS::BM> rows;
  float *As = lds, *Bs = lds + 2 * CS::A_FLOATS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % CS::WM, wn = wave / CS::WM;

  // class of this workgroup (wave-uniform selects, no indexed argument access)
  const int bid = blockIdx.x;
  const int c = (bid >= p.cls[1].blk0) + (bid >= p.cls[2].blk0) + (bid >= p.cls[3].blk0);
  const ConvClass cl = c == 0 ? p.cls[0] : c == 1 ? p.cls[1] : c == 2 ? p.cls[2] : p.cls[3];
  const int n_nt = p.N_pad / CS::BN;
  const int lb = bid - cl.blk0;
  const int mt = lb / n_nt, nt = lb - mt * n_nt;
  const int m0 = mt * CS::BM, n0 = nt * CS::BN;
  const int sh = p.stride == 2 ? 1 : 0;
  const int nj = min(max((p.C_in - (n0 + wn * 64) + 15) / 16, 0), NB);   // column blocks with real channels
  if (cl.clip) {   // workgroup-uniform
    if (wave == 0) clip_tables(p, cl, tab, lane);
    __syncthreads();
  }

  // the tile's rows decoded once, a row per thread (the clipped decode is a chain of dependent
  // LDS reads)
  if (tid < CS::BM) {
    const uint32_t m = (uint32_t)(m0 + tid);
    uint32_t r = 0;
    int iy = 0, ix = 0, anc = 0;
    if (m < (uint32_t)cl.M) convt_row(p, cl, tab, m, &r, &iy, &ix, &anc);
    const int ay = p.src_scale > 0 ? anc / p.Ha : 0, ax = p.src_scale > 0 ? anc - ay * p.Ha : 0;
    rows.r[tid] = (int)r;
    rows.yx[tid] = (uint32_t)iy | (uint32_t)ix << 8 | (uint32_t)ay << 16 | (uint32_t)ax << 24;
  }
  __syncthreads();

  // Per load of this wave: 8 tile rows, a row's 8 chunks of 16 bytes over 8 lanes, the chunk a
  // lane fetches being the one lds_swz puts into its slot.  Of each row the address of its
  // position under a zero shift, and a bit per tap row and tap column of the class: whether the
  // tap's source position lies inside the source window and, of a windowed source, inside the
  // image.  Tap (ty, tx) then reads the address plus a wave-uniform offset, or a zero block.
  // (No division by the class's tap counts here or in the K loop: a division is some 30 vector
  // instructions, and nine of them a row cost more than the whole first K step.)
  auto shift_y = [&](int ty) { return (cl.u0 + p.delta - (cl.ky0 + cl.kys * ty)) >> sh; };   // exact
  auto shift_x = [&](int tx) { return (cl.w0 + p.delta - (cl.kx0 + cl.kxs * tx)) >> sh; };
  const float *a_row[CS::AQ];
  uint32_t ty_ok[CS::AQ], tx_ok[CS::AQ];
#pragma unroll
  for (int q = 0; q < CS::AQ; ++q) {
    const int row = (q * CS::NW + wave) * 8 + (lane >> 3);
    const ConvSource src = convt_source(p, rows.yx[row]);
    a_row[q] = p.A + (int64_t)rows.r[row] * p.row_stride_out + ((int64_t)src.iy * p.S_out + src.ix) * p.C_out +
               ((lane & 7) ^ lds_swz<32>(row)) * 4;
    ty_ok[q] = tx_ok[q] = 0;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int y = src.iy + shift_y(t), x = src.ix + shift_x(t);
      ty_ok[q] |= (uint32_t)(y >= src.ylo && y < src.yhi) << t;
      tx_ok[q] |= (uint32_t)(x >= src.xlo && x < src.xhi) << t;
    }
    if (m0 + row >= cl.M) ty_ok[q] = 0;
  }
  // K order: channel blocks outer, taps inner: the shifted re-reads of one source block follow
  // each other (they hit the caches instead of HBM)
  const int cpt = p.C_out / 32;
  int l_ty = 0, l_tx = 0, l_cb = 0;   // the next step to load
  auto gload = [&](int buf) {
    const int64_t off = ((int64_t)shift_y(l_ty) * p.S_out + shift_x(l_tx)) * p.C_out + l_cb * 32;
#pragma unroll
    for (int q = 0; q < CS::AQ; ++q) {
      const float *src = (ty_ok[q] >> l_ty) & (tx_ok[q] >> l_tx) & 1 ? a_row[q] + off : g_zero4;
      dma16(src, As + buf * CS::A_FLOATS + (q * CS::NW + wave) * 256);
    }
    const int kb = (3 * (cl.ky0 + cl.kys * l_ty) + cl.kx0 + cl.kxs * l_tx) * cpt + l_cb;
#pragma unroll
    for (int q = 0; q < CS::BQ; ++q) {
      const int i = q * CS::NW + wave, nb = i / 3, part = i - 3 * nb;
      dma16(p.Bs + ((int64_t)(n0 / 16 + nb) * (9 * cpt) + kb) * SPLIT_BLOCK + part * 512, (uint32_t)lane * 16,
            Bs + buf * CS::B_FLOATS + i * 256);
    }
    if (++l_tx == cl.ntx) {
      l_tx = 0;
      if (++l_ty == cl.nty) {
        l_ty = 0;
        ++l_cb;
      }
    }
  };

  f32v4 hi[MB][NB], lo[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) hi[i][j] = lo[i][j] = f32v4{0.f, 0.f, 0.f, 0.f};
  const int KT = cl.nty * cl.ntx * cpt;
  const int r16 = lane & 15, g4 = lane >> 4, sw = lds_swz<32>(r16);
  const int ch0 = ((2 * g4) ^ sw) * 4, ch1 = ((2 * g4 + 1) ^ sw) * 4;
  gload(0);
  if (tid < CS::BM) conv_row_info(p, cl, rows, m0, tid);   // read after the loop's barriers
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    wait_vmcnt<0>();   // this wave's part of step kt has landed
    barrier_only();    // every wave's has, and step kt - 1's stage is free
    if (kt + 1 < KT) gload(cur ^ 1);
    split_step<MB, NB, false>(As + cur * CS::A_FLOATS + (wm * 32 + r16) * 32, ch0, ch1,
                              reinterpret_cast<const bf16x8 *>(Bs + cur * CS::B_FLOATS) + wn * NB * 192 + lane, nj, 0u,
                              hi, lo);
  }
  auto finish = [&] {
    return split_finish<MB, NB>(
        hi, lo, n0 + wn * 64, p.C_in, g4, [](int) { return true; },   // rows past the last are zeros
        [&](int i, int j) {
          const int row = wm * 32 + 16 * i + r16;
          const ConvSource src = convt_source(p, rows.yx[row]);
          const float *a = p.A + (int64_t)rows.r[row] * p.row_stride_out;
          const float *w = p.Bt + (int64_t)(n0 + wn * 64 + 16 * j + r16) * p.ldb;
          f32v4 x = {0.f, 0.f, 0.f, 0.f};
          for (int ty = 0; ty < cl.nty; ++ty)
            for (int tx = 0; tx < cl.ntx; ++tx) {
              const int y = src.iy + shift_y(ty), xx = src.ix + shift_x(tx);
              const bool ok = rows.mo[row] >= 0 && y >= src.ylo && y < src.yhi && xx >= src.xlo && xx < src.xhi;
              x = mma_float32(ok ? a + ((int64_t)y * p.S_out + xx) * p.C_out : nullptr,
                              w + (3 * (cl.ky0 + cl.kys * ty) + cl.kx0 + cl.kxs * tx) * p.C_out, p.C_out, g4, ~0u, x);
            }
          return x;
        });
  };
  convt_split_epilogue<WN, RELU, AL, SPL>(p, hi, rows, n0, nt, wm, wn, nj, finish);
}

template <int WN>
static hipError_t launch_convt_split(const ConvTArgs &a, int64_t blk, hipStream_t s) {
  const bool al = a.alpha || a.pre, spl = a.splits.D > 0;
  const dim3 g((unsigned)blk), t(ConvSplit<WN>::T);
  if (blk <= 0) return hipSuccess;
  if (al && spl)
    hipLaunchKernelGGL((k_convt_split<WN, true, true, true>), g, t, 0, s, a);
  else if (spl)
    hipLaunchKernelGGL((k_convt_split<WN, true, false, true>), g, t, 0, s, a);
  else if (al)
    hipLaunchKernelGGL((k_convt_split<WN, true, true, false>), g, t, 0, s, a);
  else if (a.P_pos)
    hipLaunchKernelGGL((k_convt_split<WN, true, false, false>), g, t, 0, s, a);
  else
    hipLaunchKernelGGL((k_convt_split<WN, false, false, false>), g, t, 0, s, a);
  return hipGetLastError();
}

// Forward convolution of the gradient pass (k_fwd_conv) on the same tiles: the epilogue's row
// offsets are computed once per workgroup under the first K step.
template <int ROWS>
struct FwdRows {
  int64_t ob[ROWS], pb[ROWS], rb[ROWS];   // ob -1: past the last row
  int r[ROWS];
};

template <int WN>
__global__ __launch_bounds__(ConvSplit<WN>::T, ConvSplit<WN>::MINB) void k_fwd_conv_split(const FwdConvArgs p, FastDiv div_pos) {
  typedef ConvSplit<WN> CS;
  constexpr int MB = CS::MB, NB = CS::NB;
  __shared__ __attribute__((aligned(16))) float lds[2 * (CS::A_FLOATS + CS::B_FLOATS)];
  __shared__ FwdRows<CS::BM> rows;
  float *As = lds, *Bs = lds + 2 * CS::A_FLOATS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % CS::WM, wn = wave / CS::WM;
  const int n_nt = (p.Co + CS::BN - 1) / CS::BN;
  const int mt = blockIdx.x / n_nt, nt = blockIdx.x - mt * n_nt;
  const int64_t m0 = (int64_t)mt * CS::BM;
  const int n0 = nt * CS::BN;
  const int HW = p.Ho * p.Ho;
  const int64_t Mtot = (int64_t)p.rows * HW;
  const int nj = min(max((p.Co - (n0 + wn * 64) + 15) / 16, 0), NB);   // column blocks with real channels

  // per load of this wave: 8 output positions, 8 chunks of 16 bytes each; the source address
  // under tap (0, 0) and a bit per tap row and column that lies inside the image
  const float *a_row[CS::AQ];
  uint32_t ty_ok[CS::AQ], tx_ok[CS::AQ];
#pragma unroll
  for (int q = 0; q < CS::AQ; ++q) {
    const int row = (q * CS::NW + wave) * 8 + (lane >> 3);
    const bool valid = m0 + row < Mtot;
    const uint32_t m = valid ? (uint32_t)(m0 + row) : 0u;
    const uint32_t r = fdiv(m, div_pos);
    const int pos = (int)(m - r * (uint32_t)HW);
    const int yo = pos / p.Ho, xo = pos - yo * p.Ho;
    const int y0 = yo * p.stride - 1, x0 = xo * p.stride - 1;
    a_row[q] = p.in + (int64_t)r * p.in_rs + ((int64_t)y0 * p.Hi + x0) * p.Ci + ((lane & 7) ^ lds_swz<32>(row)) * 4;
    ty_ok[q] = tx_ok[q] = 0;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      ty_ok[q] |= (uint32_t)(valid && (unsigned)(y0 + t) < (unsigned)p.Hi) << t;
      tx_ok[q] |= (uint32_t)((unsigned)(x0 + t) < (unsigned)p.Hi) << t;
    }
  }
  const int cpt = p.Ci / 32;
  int l_ty = 0, l_tx = 0, l_cb = 0;   // the next step to load: channel blocks outer, taps inner
  auto gload = [&](int buf) {
    const int64_t off = ((int64_t)l_ty * p.Hi + l_tx) * p.Ci + l_cb * 32;
#pragma unroll
    for (int q = 0; q < CS::AQ; ++q) {
      const float *src = (ty_ok[q] >> l_ty) & (tx_ok[q] >> l_tx) & 1 ? a_row[q] + off : g_zero4;
      dma16(src, As + buf * CS::A_FLOATS + (q * CS::NW + wave) * 256);
    }
    const int kb = (3 * l_ty + l_tx) * cpt + l_cb;
#pragma unroll
    for (int q = 0; q < CS::BQ; ++q) {
      const int i = q * CS::NW + wave, nb = i / 3, part = i - 3 * nb;
      // column blocks past Co repeat the last one (never stored)
      dma16(p.Ws + ((int64_t)min(n0 / 16 + nb, p.Co / 16 - 1) * (9 * cpt) + kb) * SPLIT_BLOCK + part * 512,
            (uint32_t)lane * 16, Bs + buf * CS::B_FLOATS + i * 256);
    }
    if (++l_tx == 3) {
      l_tx = 0;
      if (++l_ty == 3) {
        l_ty = 0;
        ++l_cb;
      }
    }
  };

  f32v4 hi[MB][NB], lo[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) hi[i][j] = lo[i][j] = f32v4{0.f, 0.f, 0.f, 0.f};
  const int KT = 9 * cpt;
  const int r16 = lane & 15, g4 = lane >> 4, sw = lds_swz<32>(r16);
  const int ch0 = ((2 * g4) ^ sw) * 4, ch1 = ((2 * g4 + 1) ^ sw) * 4;
  gload(0);
  if (tid < CS::BM) {   // read after the loop's barriers
    rows.ob[tid] = -1;
    if (m0 + tid < Mtot) {
      const uint32_t m = (uint32_t)(m0 + tid), r = fdiv(m, div_pos);
      fwd_offsets(p, r, (int)(m - r * (uint32_t)HW), &rows.ob[tid], &rows.pb[tid], &rows.rb[tid]);
      rows.r[tid] = (int)r;
    }
  }
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    wait_vmcnt<0>();   // this wave's part of step kt has landed
    barrier_only();    // every wave's has, and step kt - 1's stage is free
    if (kt + 1 < KT) gload(cur ^ 1);
    split_step<MB, NB, false>(As + cur * CS::A_FLOATS + (wm * 32 + r16) * 32, ch0, ch1,
                              reinterpret_cast<const bf16x8 *>(Bs + cur * CS::B_FLOATS) + wn * NB * 192 + lane, nj, 0u,
                              hi, lo);
  }
  const float unscale = split_finish<MB, NB>(
      hi, lo, n0 + wn * 64, p.Co, g4, [](int) { return true; },   // rows past the last are zeros
      [&](int i, int j) {
        const int row = wm * 32 + 16 * i + r16;
        const bool valid = rows.ob[row] >= 0;
        const uint32_t m = valid ? (uint32_t)(m0 + row) : 0u, r = fdiv(m, div_pos);
        const int pos = (int)(m - r * (uint32_t)HW);
        const int y0 = pos / p.Ho * p.stride - 1, x0 = pos % p.Ho * p.stride - 1;
        const float *w = p.Wk + (int64_t)(n0 + wn * 64 + 16 * j + r16) * 9 * p.Ci;
        f32v4 x = {0.f, 0.f, 0.f, 0.f};
        for (int ty = 0; ty < 3; ++ty)
          for (int tx = 0; tx < 3; ++tx) {
            const bool ok = valid && (unsigned)(y0 + ty) < (unsigned)p.Hi && (unsigned)(x0 + tx) < (unsigned)p.Hi;
            x = mma_float32(ok ? p.in + (int64_t)r * p.in_rs + ((int64_t)(y0 + ty) * p.Hi + x0 + tx) * p.Ci : nullptr,
                            w + (3 * ty + tx) * p.Ci, p.Ci, g4, ~0u, x);
          }
        return x;
      });
  // epilogue: bias, then a residual, or the ReLU line with the slope gradient (fwd_apply), four
  // channels of a row at once
  const float4 *__restrict__ Pp = p.P;
  const float *__restrict__ resp = p.res;
  const float *__restrict__ alp = p.alpha;
  const float *__restrict__ prep = p.pre;
  float *__restrict__ outp = p.out;
  float *__restrict__ gradp = p.grad;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int lr = wm * 32 + 16 * i + r16;
    const int64_t ob = rows.ob[lr], pb = rows.pb[lr], rb = rows.rb[lr];
    const int r = rows.r[lr];
    if (ob < 0) continue;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j >= nj) continue;
      const int n = n0 + wn * 64 + 16 * j + 4 * g4;
      f32v4 D = *reinterpret_cast<const f32v4 *>(p.bias + n);
#pragma unroll
      for (int v = 0; v < 4; ++v) D[v] = fmaf(hi[i][j][v], unscale, D[v]);
      if (resp) D += *reinterpret_cast<const f32v4 *>(resp + rb + n);
      if (Pp) {
        float4 prm[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) prm[v] = Pp[pb + n + v];
        int ent[4] = {-1, -1, -1, -1};
        float sterm[4] = {0.f, 0.f, 0.f, 0.f};
        if (p.splits.D > 0) {   // subdomains (unit 0 only: pb + n is the neuron's index)
          split_override4(p.splits, r, p.relu_index, (int)(pb + n), prm, ent, sterm);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (ent[v] >= 0 && p.splits.grad_beta)
              p.splits.grad_beta[(int64_t)r * p.splits.S + ent[v]] = sterm[v] * D[v];
        }
        const f32v4 al = *reinterpret_cast<const f32v4 *>(alp + ob + n);
        const f32v4 an = *reinterpret_cast<const f32v4 *>(prep + ob + n);
        f32v4 o, gr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bool unst = prm[v].z > 0.f;
          const float lam = unst ? al[v] : prm[v].x;
          o[v] = an[v] > 0.f ? lam * D[v] : fmaf(prm[v].y, D[v], an[v] < 0.f ? prm[v].z : 0.f);
          gr[v] = (unst && an[v] > 0.f) ? an[v] * D[v] : 0.f;
        }
        *reinterpret_cast<f32v4 *>(outp + ob + n) = o;
        *reinterpret_cast<f32v4 *>(gradp + ob + n) = gr;
      } else {
        *reinterpret_cast<f32v4 *>(outp + ob + n) = D;
      }
    }
  }
}

static hipError_t launch_fwd_conv_split(const FwdConvArgs &a, FastDiv dp, hipStream_t s) {
  const int64_t M = (int64_t)a.rows * a.Ho * a.Ho;
  const int BM = a.Co % 128 == 0 ? ConvSplit<2>::BM : ConvSplit<1>::BM;
  const int64_t mt = (M + BM - 1) / BM;
  if (a.Co % 128 == 0)
    hipLaunchKernelGGL(k_fwd_conv_split<2>, dim3((unsigned)(mt * (a.Co / 128))), dim3(ConvSplit<2>::T), 0, s, a, dp);
  else
    hipLaunchKernelGGL(k_fwd_conv_split<1>, dim3((unsigned)(mt * ((a.Co + 63) / 64))), dim3(ConvSplit<1>::T), 0, s, a, dp);
  return hipGetLastError();
}

}  // namespace vcr
