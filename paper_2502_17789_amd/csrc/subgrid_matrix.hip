// FP32 (de)gridder on the matrix cores.
//
// With n1(l, m) = a(l) + a(m) + c(l, m), a(l) about n1(l, 0), the phasor of visibility k at
// subgrid pixel (x, y) factors into
//   alpha_k(x) = E(u_k l_x + w_k a(l_x)),   beta_k(y) = E(v_k m_y + w_k a(m_y)),
//   E(w_s c(x, y)) E(d_k c(x, y)),          w_k = w_s + d_k,   E(t) = exp(2 pi i t),
// with (u, v, w)_k relative to the subgrid's centre and layer and w_s the middle of the
// subgrid's w range.  The first two are per visibility and axis, the third per subgrid and
// pixel; the last is a short series: c = -b(x) b(y) to the accuracy the plan checks, so
// E(d_k c) = sum_j (-2 pi i d_k b(x) b(y))^j / j!, every term of which again separates.
// Gridding and degridding are then complex matrix products over visibilities and over x:
//   S(x, y) = E(w_s c) sum_k alpha_k(x) [V_k beta_k(y)]
//   V_k     = sum_y conj(beta_k(y)) sum_x conj(alpha_k(x)) [S'(x, y) E(-w_s c)],
// 16 real multiply-adds per visibility and pixel, with L + L phasors per visibility where
// the direct sum forms L^2.
//
// Precision: each FP32 factor is split into two FP16 numbers (x = hi + lo, both rounded to
// nearest: 2^-24 of the largest value, the data scaled to that by a power of two per
// subgrid and polarisation) and a product takes hi hi + hi lo + lo hi on
// v_mfma_f32_32x32x16_f16, which forms the products exactly and adds in FP32; the gridder adds eight visibilities' sum at
// once, the degridder sums the small products apart.  Every phase is formed and reduced to
// [-1/4, 1/4] turn in FP64; there is no recurrence.  The series' first term takes hi hi
// alone where its largest value, times the taper, is below 1.5e-5 (w_series_order), and
// otherwise split operands as well; a second term is smaller and takes hi hi.
//
// What bounds it: the matrix cores at 3 (hi, lo) + 1 (first-order w term) products, and
// beside them the VALU that forms the split operands: with 256 registers per lane two waves
// share a SIMD and overlap little.  128 stations x 60 times x 96 channels, L = 96 (46.8M
// visibilities): gridder 69.0 ms and degridder 73.3 (128.8 and 161.3 in the paired
// recurrence); the products alone need 26 ms at the clock they run at, the matrix cores are
// busy 37 and 35 % of the time.  64 stations x 30 x 48, L = 64: 2.33 and 2.62 ms
// (5.1 and 5.1); 48 x 12 x 3 of every 32nd channel, L = 96, degridder 0.265 (0.69).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "aidg_internal.h"
#include "device_common.h"
#include "matrix_common.h"
#include "subgrid_common.h"

namespace aidg {
namespace {

// exp(2 pi i (u x + w z)) for phases in turns, |u x + w z| < 2^18: the sum is formed onto
// 1.5 2^20, whose last place is 2^-32 turn, so that the low word of the FP64 result is the
// phase modulo a turn in fixed point (rounded twice, 2^-33 turn).  Reduced to [-1/4, 1/4] turn
// (sign changes make up for half a turn), one rounding to FP32 (2^-27 turn), then the
// transcendental unit's cosine and sine (absolute error at most 1.3e-7, rms 3.5e-8, measured
// over 2^24 points).  From [-1/2, 1/2] a product of two phasors was 10 % further off, and the
// visibilities of a few sources 4 % further than the general kernels'; the reduction is 2 % of
// the kernels' time.
__device__ __forceinline__ float2 turn_phasor(double u, double x, double w, double z) {
  const double th = fma(u, x, fma(w, z, 1572864.0));
  const unsigned p = (unsigned)__double_as_longlong(th);
  const unsigned flip = (p ^ (p << 1)) & 0x80000000u;
  const float t = (float)((int)(p << 1) >> 1) * 0x1p-32f;
  return {__uint_as_float(__float_as_uint(__builtin_amdgcn_cosf(t)) ^ flip),
          __uint_as_float(__float_as_uint(__builtin_amdgcn_sinf(t)) ^ flip)};
}

// Pixels whose Jones matrices are loaded ahead.
constexpr int kAhead = 2;
// Subgrid rows (y) of one workgroup pass: 8 per wave.
constexpr int kRows = 32;

// A block's visibilities: phase coefficients in turns per lattice step (u, v) and
// wavelengths (w), and d_k times KernelArgs' w_series, rounded to FP16 and what that leaves,
// as FP16 pairs.
template <int B>
struct VisBlock {
  double2 ku_w[B];
  double2 kv_w[B];
  unsigned dw[2][B];
};

// A visibility's uvw row and frequency, loaded ahead of the block that uses them.
struct VisPhase {
  double u, v, w, fc;
};
__device__ __forceinline__ VisPhase load_phase(const KernelArgs& a, const SubgridDev& s, int k, float inv_nc) {
  // (k + 1/2) / nc is at least 1 / (2 nc) from an integer, beyond FP32 rounding for k < 2048
  const int row = (int)(((float)k + 0.5f) * inv_nc), c = k - row * s.nc;
  const double* uvw = a.uvw + 3 * s.uvw0;
  return {gload<double>(uvw, 24 * row), gload<double>(uvw, 24 * row + 8), gload<double>(uvw, 24 * row + 16),
          gload<double>(a.fc + s.c0, 8 * c)};
}
template <int B>
__device__ __forceinline__ void store_phase(const KernelArgs& a, const SubgridDev& s, const VisPhase& p, bool valid, int k,
                                            VisBlock<B>* vb) {
  double ku = 0, kv = 0, kw = 0;
  unsigned dw = 0, dl = 0;
  if (valid) {
    ku = (p.u * p.fc - (s.U0 - a.N / 2) * a.du) * a.lstep;
    kv = (p.v * p.fc - (s.V0 - a.N / 2) * a.du) * a.lstep;
    kw = p.w * p.fc - s.w0;
    const float d = (float)((kw - (double)s.wmid) * a.w_series);
    dw = pair_of(d);
    dl = pair_of(d - (float)(_Float16)d);
  }
  vb->ku_w[k] = {ku, kw};
  vb->kv_w[k] = {kv, kw};
  vb->dw[0][k] = dw;
  vb->dw[1][k] = dl;
}

// beta_k(y) of the workgroup's 32 rows from y0 for the block's first n visibilities,
// FP32: [32][B + 2] (the pitch shifts each row by four banks: eight rows' 16-byte reads meet
// no bank twice).
template <int L, int B>
__device__ __forceinline__ void stage_beta(const VisBlock<B>* vb, const double* axis, int y0, int n, float2* beta) {
  static_assert(B == 32 && kThreads == 256 && kRows == 32, "four rows per thread");
  int tid = threadIdx.x;  // opaque: formed again for each block, not held across it
  asm volatile("" : "+v"(tid));
  const int k = tid & 31, y = tid >> 5;
  if (k >= n) return;
  const double2 kv = vb->kv_w[k];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = y + 8 * i;
    beta[r * (B + 2) + k] = turn_phasor(kv.x, (double)(y0 + r - L / 2), kv.y, axis[y0 + r]);
  }
}

// c + a b, fused.
__device__ __forceinline__ float2 cfma(float2 a, float2 b, float2 c) {
  return {fmaf(-a.y, b.y, fmaf(a.x, b.x, c.x)), fmaf(a.y, b.x, fmaf(a.x, b.y, c.y))};
}

// A subgrid pixel's two Jones matrices, taper and cross term.
struct PixelTerms {
  vec4 p0, p1, q0, q1;
  vec2 tc;
};
__device__ __forceinline__ PixelTerms load_pixel(const KernelArgs& a, const char* Ap, const char* Aq, unsigned pix) {
  return {gload<vec4>(Ap, 32 * pix), gload<vec4>(Ap, 32 * pix + 16), gload<vec4>(Aq, 32 * pix),
          gload<vec4>(Aq, 32 * pix + 16), gload<vec2>(a.taper_cross, 8 * pix)};
}
// d += A^H (f E(w_s c) S) B with A = (p0, p1), B = (q0, q1) and f a factor per polarisation;
// INV: scaled by 1 / ||A^H B||_F.
template <bool INV>
__device__ __forceinline__ void add_corrected(const PixelTerms& x, float wmid, const float4& f, const float2 (&s)[4],
                                              float (&d)[8]) {
  const float2 a0 = {x.p0.x, -x.p0.y}, a1 = {x.p0.z, -x.p0.w}, a2 = {x.p1.x, -x.p1.y}, a3 = {x.p1.z, -x.p1.w};  // conj
  const float2 b0 = {x.q0.x, x.q0.y}, b1 = {x.q0.z, x.q0.w}, b2 = {x.q1.x, x.q1.y}, b3 = {x.q1.z, x.q1.w};
  float w = x.tc.x;
  if constexpr (INV) {
    // ||B_p^H B_q||_F^2 with B_p^H = [[a0, a2], [a1, a3]] (a already conjugated)
    const float2 m0 = cmul<float>(a0, b0) + cmul<float>(a2, b2), m1 = cmul<float>(a0, b1) + cmul<float>(a2, b3);
    const float2 m2 = cmul<float>(a1, b0) + cmul<float>(a3, b2), m3 = cmul<float>(a1, b1) + cmul<float>(a3, b3);
    const float n2 = m0.x * m0.x + m0.y * m0.y + m1.x * m1.x + m1.y * m1.y + m2.x * m2.x + m2.y * m2.y + m3.x * m3.x +
                     m3.y * m3.y;
    const float v = w / sqrtf(n2 > 0.0f ? n2 : 1.0f);
    w = n2 > 0.0f ? v : 0.0f;
  }
  // taper and E(w_s c), |w_s c| <= 128 turns
  const float ph = wmid * x.tc.y;
  const float2 e = {w * __builtin_amdgcn_cosf(ph), w * __builtin_amdgcn_sinf(ph)};
  const float2 s0 = cmul<float>(e, s[0]) * f.x, s1 = cmul<float>(e, s[1]) * f.y;
  const float2 s2 = cmul<float>(e, s[2]) * f.z, s3 = cmul<float>(e, s[3]) * f.w;
  // A_p^H = [[conj a0, conj a2], [conj a1, conj a3]]
  const float2 t0 = cfma(a2, s2, cmul<float>(a0, s0)), t1 = cfma(a2, s3, cmul<float>(a0, s1));
  const float2 t2 = cfma(a3, s2, cmul<float>(a1, s0)), t3 = cfma(a3, s3, cmul<float>(a1, s1));
  const float2 c0 = cfma(t1, b2, cmul<float>(t0, b0)), c1 = cfma(t1, b3, cmul<float>(t0, b1));
  const float2 c2 = cfma(t3, b2, cmul<float>(t2, b0)), c3 = cfma(t3, b3, cmul<float>(t2, b1));
  // (added whole: a chain of products onto d would round at the size of the sum four times)
  d[0] += c0.x; d[1] += c0.y; d[2] += c1.x; d[3] += c1.y;
  d[4] += c2.x; d[5] += c2.y; d[6] += c3.x; d[7] += c3.y;
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(d[i]));  // here, not behind the later pixels
}

// ------------------------------------------------------------------ gridder

// Pixels of a lane whose group sums are held in LDS: at L = 96 the sums and accumulators of
// all twelve would leave 64 of 256 registers for everything else.
template <int L>
constexpr int kLdsPixels = L == 96 ? 5 : 0;

// Gridder LDS: alpha operands, beta, the visibilities [4][kBlk + 2], phases, axis tables.
template <int L>
struct GridLds {
  Frag alpha[kBlk / 8][L / 32][2][64];
  float2 beta[kRows * (kBlk + 2)];
  float2 vis[4 * (kBlk + 2)];
  VisBlock<kBlk> vb;
  double axis[L];
  unsigned b_rest[L];
  float4 unscale, shrink;  // of the polarisations
  int shrunk;
  float4 sum[kLdsPixels<L>][2][kThreads];
};

// Waves per SIMD that the registers are allocated for.  At L = 32 a lane has one column tile
// and three workgroups fit a compute unit: 72 stations x 16 times x 96 channels, folded, series
// terms of split operands: 1.51 ms against 1.70 with two; four spill, and so do three at L = 64.
template <int L>
constexpr int kGridWaves = L == 32 ? 3 : 2;

// One workgroup per (32 rows, group or part of one).  Each wave owns 8 rows x 4 polarisations (the 32
// rows of the matrix tiles) by L columns, real and imaginary parts in separate tiles, so
// that a lane ends with all four polarisations of its L/8 pixels: the Jones epilogue is
// lane-local and the group's sum stays in registers (a subgrid's image does not go through
// memory).  Rows are V_k beta_k(y), formed and split by the wave that uses them; columns are
// alpha_k(x), formed once per workgroup and read from LDS in the operand's lane order.
// The next block's visibilities and uvw are loaded (into registers) before the products of
// the current one, across subgrids as well.
template <int L, bool WIDE>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kGridWaves<L>, kGridWaves<L>))) void grid_matrix(const Group g) {
  constexpr int XT = L / 32, NP = 4, NPIX = XT * NP, P0 = kLdsPixels<L>;  // column tiles; pixels per lane
  extern __shared__ unsigned char smem_raw[];
  GridLds<L>& sh = *reinterpret_cast<GridLds<L>*>(smem_raw);
  int64_t local;
  int chunk;
  grid_work<L / kRows>(blockIdx.x, &local, &chunk);
  if (local >= (g.split ? g.total_part : g.total_grp)) return;  // padding of the last XCD round (whole workgroup)
  const GroupSlot gs = resolve_group(g, local, g.split != 0);
  const KernelArgs& a = gs.a;
  const bool inv = a.ainvh != nullptr;
  const char* At = static_cast<const char*>(inv ? a.ainvh : a.aterms);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, h = lane >> 5;
  const int y0 = chunk * kRows;
  for (int i = tid; i < L; i += kThreads) {
    sh.axis[i] = a.axis_n1[i];
    sh.b_rest[i] = a.axis_b[L + i];
  }
  // operand row of this lane: polarisation q of row yl of the wave's eight
  const int q = col & 3, yl = wave * 8 + (col >> 2);
  const unsigned pix0 = (y0 + wave * 8 + h) * L + col;  // pixel (t, p) is 2 p rows and 32 t columns on

  float sum[NPIX - P0][8];
#pragma unroll
  for (int p = P0; p < NPIX; ++p)
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[p - P0][i] = 0;
#pragma unroll
  for (int p = 0; p < P0; ++p) sh.sum[p][0][tid] = sh.sum[p][1][tid] = {0, 0, 0, 0};

  // Block loads: wave 0 one half (two polarisations) of a visibility per lane, wave 1 the uvw
  // and frequency of one.
  static_assert(2 * kBlk == 64, "one wave stages a block");
  VisPhase next;
  vec4 next_v;
  auto prefetch = [&](const SubgridDev& s, int k0) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int nv = s.nt * s.nc;
    const float inv_nc = 1.0f / (float)s.nc;
    if (tid < 2 * kBlk) {
      const int k = k0 + (tid >> 1);
      next_v = {0, 0, 0, 0};
      if (k < nv) {
        const int row = (int)(((float)k + 0.5f) * inv_nc), c = k - row * s.nc;
        const char* src = static_cast<const char*>(gs.in) + s.vis0 * 32 + vis_offset(row, c, a.nc_total);
        if (s.fold) {  // a folded sub-table is read as V^H
          const vec4 h0 = gload<vec4_of_2>(src, 0), h1 = gload<vec4_of_2>(src, 16);
          next_v = (tid & 1) ? vec4{h0.z, -h0.w, h1.z, -h1.w} : vec4{h0.x, -h0.y, h1.x, -h1.y};
        } else {
          next_v = gload<vec4_of_2>(src, 16 * (tid & 1));
        }
      }
    } else if (tid < 3 * kBlk) {
      const int k = k0 + tid - 2 * kBlk;
      if (k < nv) next = load_phase(a, s, k, inv_nc);
    }
  };

  acc16 re[XT], im[XT];
  // Row operands of step ks: W_k = V_k beta_k(y) for the lane's four visibilities, rows
  // (W_re, -W_im) for the real tile and (W_im, W_re) for the imaginary one, each hi and lo;
  // g: 2 pi d_k b(y) of the w series, whose first term takes rows times -i g and columns
  // times b(x).  (b is held over its peak and d_k with the peak's square: the factors of a
  // row stay below 4 and those of a column below 1, whatever the data are largest at.)
  struct Rows {
    Frag rh, rl, ih, il;
    unsigned g[4];
  };
  const unsigned by = a.axis_b[y0 + yl];
  unsigned bx[XT];
#pragma unroll
  for (int t = 0; t < XT; ++t) bx[t] = a.axis_b[t * 32 + col];
  auto rows = [&](int ks) -> Rows {
    Rows r;
    const int k = 8 * ks + 4 * h;
    // (16-byte aligned: even places of even rows)
    const float4* vp = reinterpret_cast<const float4*>(__builtin_assume_aligned(&sh.vis[q * (kBlk + 2) + k], 16));
    const float4* bp = reinterpret_cast<const float4*>(__builtin_assume_aligned(&sh.beta[yl * (kBlk + 2) + k], 16));
    const float4 v01 = vp[0], v23 = vp[1], b01 = bp[0], b23 = bp[1];
    const float2 vs[4] = {{v01.x, v01.y}, {v01.z, v01.w}, {v23.x, v23.y}, {v23.z, v23.w}};
    const float2 bs[4] = {{b01.x, b01.y}, {b01.z, b01.w}, {b23.x, b23.y}, {b23.z, b23.w}};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float2 v = vs[i], b = bs[i];
      split(fmaf(-v.y, b.y, v.x * b.x), fmaf(-v.y, b.x, -(v.x * b.y)), r.rh.w[i], r.rl.w[i]);
      r.ih.w[i] = rot90(r.rh.w[i]);
      r.il.w[i] = rot90(r.rl.w[i]);
      r.g[i] = pk_mul(sh.vb.dw[0][k + i], by);
    }
    return r;
  };
  // Products of step ks with the series' first term.  The small products come first and the
  // step's sum is added whole: a chain of products onto the accumulators would round at the
  // size of the subgrid's sum four times or more.
  auto products = [&](int ks) {
    Frag bh[XT], bl[XT];
#pragma unroll
    for (int t = 0; t < XT; ++t) {
      bh[t] = sh.alpha[ks][t][0][lane];
      bl[t] = sh.alpha[ks][t][1][lane];
    }
    const Rows r = rows(ks);
    Frag nr, ni;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      nr.w[i] = pk_mul(r.ih.w[i], r.g[i]);
      ni.w[i] = pk_mul_neg(r.rh.w[i], r.g[i]);
    }
#pragma unroll
    for (int t = 0; t < XT; ++t) {
      acc16 cr = mfma(r.rl, bh[t], acc16{0}), ci = mfma(r.il, bh[t], acc16{0});
      cr = mfma(r.rh, bl[t], cr);
      ci = mfma(r.ih, bl[t], ci);
      Frag c;
#pragma unroll
      for (int i = 0; i < 4; ++i) c.w[i] = pk_mul(bh[t].w[i], bx[t]);
      cr = mfma(nr, c, cr);
      ci = mfma(ni, c, ci);
      cr = mfma(r.rh, bh[t], cr);
      ci = mfma(r.ih, bh[t], ci);
      re[t] += cr;
      im[t] += ci;
    }
  };
  // The same with the first term in split operands and a second one, rows times
  // (-i 2 pi d_k b(y))^2 / 2 and columns times b(x)^2 (also where a subgrid does not need it: a
  // branch here, as all rows held at once, spilled a hundred registers at L = 96).  One column
  // tile at a time and, at L = 96, its real sum before the imaginary one, whose rows are formed
  // again.
  auto products_wide = [&](int ks) {
    Frag rh, rl, n, m, n2;  // rows, and rows times g and g g / 2
    {
      const Rows r = rows(ks);
      const unsigned y_rest = sh.b_rest[y0 + yl];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned dw = sh.vb.dw[0][8 * ks + 4 * h + i], dl = sh.vb.dw[1][8 * ks + 4 * h + i];
        rh.w[i] = r.rh.w[i];
        rl.w[i] = r.rl.w[i];
        n.w[i] = pk_mul(r.ih.w[i], r.g[i]);
        m.w[i] = mul_rest(r.ih.w[i], r.il.w[i], r.g[i], mul_rest(dw, dl, by, y_rest, r.g[i]), n.w[i]);
        n2.w[i] = rot90(pk_mul(n.w[i], pk_mul(r.g[i], pair_of(0.5f))));
      }
    }
#pragma unroll
    for (int t = 0; t < XT; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      const Frag bh = sh.alpha[ks][t][0][lane];
      Frag bl = sh.alpha[ks][t][1][lane], c, cl, c2;
      const unsigned x_rest = sh.b_rest[t * 32 + col];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        c.w[i] = pk_mul(bh.w[i], bx[t]);
        cl.w[i] = mul_rest(bh.w[i], bl.w[i], bx[t], x_rest, c.w[i]);
        c2.w[i] = pk_mul(c.w[i], bx[t]);
      }
      const Frag left[7] = {rl, rh, n, m, n2, n, rh}, right[7] = {bh, bl, cl, c, c2, c, bh};
      acc16 v = acc16{0}, u = acc16{0};
      if constexpr (XT < 3) {
#pragma unroll
        for (int k = 0; k < 7; ++k) {
          v = mfma(left[k], right[k], v);
          u = mfma(rot90(left[k]), right[k], u);
        }
        re[t] += v;
      } else {
#pragma unroll
        for (int k = 0; k < 7; ++k) v = mfma(left[k], right[k], v);
        re[t] += v;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 7; ++k) {
          Frag f = left[k];
#pragma unroll
          for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(f.w[i]));  // formed here, not held from the tile before
          u = mfma(rot90(f), right[k], u);
        }
      }
      im[t] += u;
    }
  };
  SubgridDev s = load_uniform(a.sg + gs.sb);
  int64_t si = gs.sb;
  int k0 = 0;
  prefetch(s, 0);
  while (true) {
    const int nv = s.nt * s.nc;
    const int n = min(kBlk, nv - k0), n8 = (n + 7) & ~7;
    // an opaque copy of the thread index: what derives from it is cheaper to form again for
    // each block than to hold in registers through the products
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    __syncthreads();  // the previous block's operands are no longer read
    if (tid < 2 * kBlk) {
      const int k = tid >> 1, p = 2 * (tid & 1);
      const vec4 v = next_v;
      // The scale of the lane's two polarisations' data: a power of two that fits the subgrid's
      // largest values so far (each polarisation has its own: cross hands may be orders of
      // magnitude below the parallel ones), and what brings sums under the previous one to it.
      const float2 before = reinterpret_cast<const float2*>(&sh.unscale)[tid & 1];
      float2 un, scale, shrink;
      fit_scale(parity_max(fmaxf(fabsf(v.x), fabsf(v.y))), scale.x, un.x);
      fit_scale(parity_max(fmaxf(fabsf(v.z), fabsf(v.w))), scale.y, un.y);
      if (k0) un = {fmaxf(un.x, before.x), fmaxf(un.y, before.y)};
      scale = {inverse_power(un.x), inverse_power(un.y)};
      shrink = {before.x * scale.x, before.y * scale.y};
      sh.vis[p * (kBlk + 2) + k] = {v.x * scale.x, v.y * scale.x};
      sh.vis[(p + 1) * (kBlk + 2) + k] = {v.z * scale.y, v.w * scale.y};
      const bool shrunk = __ballot(shrink.x < 1.0f || shrink.y < 1.0f) != 0;
      if (lane < 2) {
        reinterpret_cast<float2*>(&sh.unscale)[lane] = un;
        reinterpret_cast<float2*>(&sh.shrink)[lane] = shrink;
        sh.shrunk = shrunk;
      }
    } else if (tid < 3 * kBlk) {
      store_phase(a, s, next, k0 + tid - 2 * kBlk < nv, tid - 2 * kBlk, &sh.vb);
    }
    __syncthreads();
    if (k0 == 0) {
#pragma unroll
      for (int t = 0; t < XT; ++t) re[t] = im[t] = acc16{0};
    } else if (__builtin_amdgcn_readfirstlane(sh.shrunk)) {
      const float4 f = uniform(sh.shrink);
#pragma unroll
      for (int t = 0; t < XT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          re[t][i] *= (&f.x)[i & 3];
          im[t][i] *= (&f.x)[i & 3];
        }
    }
    // four visibilities per thread (kg), one column of each tile
    const int kg = tid >> 5, xc = tid & 31;
    if (4 * kg < n8) {
      double2 kuw[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) kuw[i] = sh.vb.ku_w[4 * kg + i];
#pragma unroll
      for (int t = 0; t < XT; ++t) {
        const int x = 32 * t + xc;
        const double dx = (double)(x - L / 2), ax = sh.axis[x];
        Frag fh, fl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 e = turn_phasor(kuw[i].x, dx, kuw[i].y, ax);
          split(e.x, e.y, fh.w[i], fl.w[i]);
        }
        Frag* f = &sh.alpha[kg >> 1][t][0][32 * (kg & 1) + xc];
        f[0] = fh;
        f[64] = fl;
      }
    }
    stage_beta<L>(&sh.vb, sh.axis, y0, n8, sh.beta);
    // the next block: of this subgrid, or the next one's first
    const SubgridDev cur = s;
    const bool last = k0 + kBlk >= nv, done = last && si + 1 == gs.se;
    k0 = last ? 0 : k0 + kBlk;
    if (last && !done) s = load_uniform(a.sg + ++si);
    if (!last) prefetch(s, k0);
    __syncthreads();

#pragma unroll 1
    for (int ks = 0; ks < n8 / 8; ++ks) {
      if constexpr (WIDE) products_wide(ks);
      else products(ks);
    }
    if (!last) continue;
    // Jones correction of this subgrid, A_p^H S A_q, tapered and added to the group's sum;
    // a pixel's terms are loaded while the one before is computed
    const char* Ap = At + (int64_t)cur.ap * L * L * 32;
    const char* Aq = At + (int64_t)cur.aq * L * L * 32;
    const float4 un = uniform(sh.unscale);
    auto epilogue = [&](auto inverse) {
      unsigned pe = pix0;
      asm volatile("" : "+v"(pe));  // the pixels' offsets are not worth holding across subgrids
      PixelTerms px[kAhead];
#pragma unroll
      for (int i = 0; i < kAhead; ++i) px[i] = load_pixel(a, Ap, Aq, pe + 2 * (i % NP) * L + 32 * (i / NP));
#pragma unroll
      for (int i = 0; i < NPIX; ++i) {
        const int t = i / NP, p = i % NP, n = i + kAhead;
        const float2 sv[4] = {{re[t][4 * p], im[t][4 * p]}, {re[t][4 * p + 1], im[t][4 * p + 1]},
                              {re[t][4 * p + 2], im[t][4 * p + 2]}, {re[t][4 * p + 3], im[t][4 * p + 3]}};
        if (i < P0) {
          const float4 o0 = sh.sum[i][0][tid], o1 = sh.sum[i][1][tid];
          float d[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
          add_corrected<decltype(inverse)::value>(px[i % kAhead], cur.wmid, un, sv, d);
          sh.sum[i][0][tid] = {d[0], d[1], d[2], d[3]};
          sh.sum[i][1][tid] = {d[4], d[5], d[6], d[7]};
        } else {
          add_corrected<decltype(inverse)::value>(px[i % kAhead], cur.wmid, un, sv, sum[i - P0]);
        }
        asm volatile("" : "+v"(pe));
        if (n < NPIX) px[i % kAhead] = load_pixel(a, Ap, Aq, pe + 2 * (n % NP) * L + 32 * (n / NP));
        if (i == 5 % NPIX && !done) prefetch(s, 0);  // behind pixels whose accumulators are free
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (inv) epilogue(std::true_type());
    else epilogue(std::false_type());
    if (done) break;
  }

  char* out = static_cast<char*>(g.scratch) + local * 4 * L * L * 8;
  // Stokes-I grid: I = (XX + YY) / 2 of the corrected image, plane 0 only
  const float fi = gs.adjoint ? 1.0f : 0.5f;
#pragma unroll
  for (int i = 0; i < NPIX; ++i) {
    const unsigned pix = pix0 + 2 * (i % NP) * L + 32 * (i / NP);
    float d[8];
    if (i < P0) {
      const float4 o0 = sh.sum[i][0][tid], o1 = sh.sum[i][1][tid];
      d[0] = o0.x; d[1] = o0.y; d[2] = o0.z; d[3] = o0.w;
      d[4] = o1.x; d[5] = o1.y; d[6] = o1.z; d[7] = o1.w;
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) d[k] = sum[i - P0][k];
    }
    if (a.npol == 1) {
      gstore(out, 8 * pix, vec2{(d[0] + d[6]) * fi, (d[1] + d[7]) * fi});
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) gstore(out, 8 * (k * L * L + pix), vec2{d[2 * k], d[2 * k + 1]});
    }
  }
}

// ------------------------------------------------------------------ degridder

// Visibilities per degridder block: one tile of the matrix product.
constexpr int kDegBlk = 32;
// Degridder LDS: alpha operands [x step][(re, im) hi, lo; (-im, re) hi, lo], beta, phases, the
// waves' partial visibilities, axis tables.  While a pass's image is laid out, the first part
// holds 32 columns of each wave's rows: [hi, lo][wave][row][kLayPitch].
constexpr int kLayPitch = 36;
template <int L>
struct DegridLds {
  union {
    Frag alpha[L / 8][4][64];
    unsigned lay[2][4][32][kLayPitch];
  };
  float2 beta[kRows * (kDegBlk + 2)];
  VisBlock<kDegBlk> vb;
  float2 part[4][kDegBlk * 4];
  double axis[L];
  alignas(16) unsigned b[2][L];  // (-b, b) pairs: FP16, and what that leaves
};

// One workgroup per subgrid, 32 rows of the subgrid at a time.  Each wave corrects its
// 8 rows of the group image (A_p S A_q^H, taper, E(-w_s c)), splits them and keeps them in
// registers as the operand [x][(row, polarisation)] for all visibilities of the pass;
// alpha_k(x) is formed by the workgroup, 32 visibilities at a time, as the other operand, in
// the two arrangements that give the real and the imaginary part.  A block's
// 32 visibilities x 8 rows x 4 polarisations are multiplied by conj(beta_k(y)) and summed over
// the rows across lanes; the waves' sums meet in LDS and are added to the output in wave
// order (deterministic, no atomics).
template <int L>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void degrid_matrix(const Group g) {
  constexpr int XT = L / 32, NP = 4, KS = L / 8, B = kDegBlk;
  extern __shared__ unsigned char smem_raw[];
  DegridLds<L>& sh = *reinterpret_cast<DegridLds<L>*>(smem_raw);
  const int64_t local = degrid_slot(blockIdx.x, g.total_sg);
  const Slot sl = resolve(g, local);
  const KernelArgs& a = sl.a;
  const SubgridDev& s = sl.s;
  char* vis = static_cast<char*>(sl.out) + s.vis0 * 32;
  const char* img = static_cast<const char*>(g.scratch) + sl.img_slot * 4 * L * L * 8;
  const char* Ap = static_cast<const char*>(a.aterms) + (int64_t)s.ap * L * L * 32;
  const char* Aq = static_cast<const char*>(a.aterms) + (int64_t)s.aq * L * L * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, h = lane >> 5;
  const int nv = s.nt * s.nc;
  const float inv_nc = 1.0f / (float)s.nc;
  for (int i = tid; i < L; i += kThreads) {
    sh.axis[i] = a.axis_n1[i];
    sh.b[0][i] = a.axis_b[i] ^ kNegLow;
    sh.b[1][i] = a.axis_b[L + i] ^ kNegLow;
  }
  // operand column of this lane: polarisation q of row yl of the wave's eight
  const int q = col & 3, yl = wave * 8 + (col >> 2);
  VisPhase next;
  if (tid < B && tid < nv) next = load_phase(a, s, tid, inv_nc);

  for (int y0 = 0; y0 < L; y0 += kRows) {
    // the wave's rows, corrected: lane (col, h) takes column x = 32 t + col of rows 2 p + h
    float c[XT][NP][8];
    float m[4] = {0, 0, 0, 0};  // largest of each polarisation
    unsigned pix0 = (y0 + wave * 8 + h) * L + col;
    struct Pixel {
      PixelTerms x;
      vec2 s[4];
    };
    auto load = [&](int i) -> Pixel {
      const unsigned pix = pix0 + 2 * (i % NP) * L + 32 * (i / NP);
      return {load_pixel(a, Ap, Aq, pix),
              {gload<vec2>(img, 8 * pix), gload<vec2>(img, 8 * (L * L + pix)), gload<vec2>(img, 8 * (2 * L * L + pix)),
               gload<vec2>(img, 8 * (3 * L * L + pix))}};
    };
    constexpr int kAhead = 3;  // with their image values
    Pixel px[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) px[i] = load(i);
#pragma unroll
    for (int i = 0; i < XT * NP; ++i) {
      const PixelTerms x = px[i % kAhead].x;
      vec2 sv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) sv[k] = px[i % kAhead].s[k];
      asm volatile("" : "+v"(pix0));  // loads stay this far ahead of their use
      if (i + kAhead < XT * NP) px[i % kAhead] = load(i + kAhead);
      const float2 a0 = {x.p0.x, x.p0.y}, a1 = {x.p0.z, x.p0.w}, a2 = {x.p1.x, x.p1.y}, a3 = {x.p1.z, x.p1.w};
      const float2 b0 = {x.q0.x, -x.q0.y}, b1 = {x.q0.z, -x.q0.w}, b2 = {x.q1.x, -x.q1.y}, b3 = {x.q1.z, -x.q1.w};
      const float ph = s.wmid * x.tc.y;
      const float2 e = {x.tc.x * __builtin_amdgcn_cosf(ph), -x.tc.x * __builtin_amdgcn_sinf(ph)};
      const float2 s0 = cmul<float>(e, float2{sv[0].x, sv[0].y}), s1 = cmul<float>(e, float2{sv[1].x, sv[1].y});
      const float2 s2 = cmul<float>(e, float2{sv[2].x, sv[2].y}), s3 = cmul<float>(e, float2{sv[3].x, sv[3].y});
      const float2 t0 = cfma(a1, s2, cmul<float>(a0, s0)), t1 = cfma(a1, s3, cmul<float>(a0, s1));
      const float2 t2 = cfma(a3, s2, cmul<float>(a2, s0)), t3 = cfma(a3, s3, cmul<float>(a2, s1));
      // A_q^H = [[conj b0, conj b2], [conj b1, conj b3]]
      const float2 r0 = cfma(t1, b1, cmul<float>(t0, b0)), r1 = cfma(t1, b3, cmul<float>(t0, b2));
      const float2 r2 = cfma(t3, b1, cmul<float>(t2, b0)), r3 = cfma(t3, b3, cmul<float>(t2, b2));
      float* d = c[i / NP][i % NP];
      d[0] = r0.x; d[1] = r0.y; d[2] = r1.x; d[3] = r1.y;
      d[4] = r2.x; d[5] = r2.y; d[6] = r3.x; d[7] = r3.y;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        asm volatile("" : "+v"(d[k]));
        m[k >> 1] = fmaxf(m[k >> 1], fabsf(d[k]));
      }
    }
    float scale[4], unscale = 0;  // a scale per polarisation, as in the gridder; the lane's q
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float un;
      fit_scale(wave_max(m[k]), scale[k], un);
      if (q == k) unscale = un;
    }
    __syncthreads();  // the previous pass's operands are no longer read
    // operand order: lane (col, h) holds row (yl, q), columns 8 ks + 4 h + 0 .. 3
    Frag sh_[KS], sl_[KS];
#pragma unroll
    for (int t = 0; t < XT; ++t) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          unsigned hi, lo;
          split(c[t][p][2 * k] * scale[k], c[t][p][2 * k + 1] * scale[k], hi, lo);
          sh.lay[0][wave][(2 * p + h) * 4 + k][col] = hi;
          sh.lay[1][wave][(2 * p + h) * 4 + k][col] = lo;
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sh_[4 * t + i] = *reinterpret_cast<const Frag*>(&sh.lay[0][wave][col][8 * i + 4 * h]);
        sl_[4 * t + i] = *reinterpret_cast<const Frag*>(&sh.lay[1][wave][col][8 * i + 4 * h]);
      }
    }

    for (int k0 = 0; k0 < nv; k0 += B) {
      const int n = min(B, nv - k0);
      int tid = threadIdx.x;  // opaque, as in the gridder
      asm volatile("" : "+v"(tid));
      __syncthreads();  // operands (or the laid-out image) and partial sums no longer read
      if (tid < B) {
        store_phase(a, s, next, tid < n, tid, &sh.vb);
        // the next block's phases (the next pass starts over)
        const int k = k0 + B < nv ? k0 + B + tid : tid;
        if (k < nv) next = load_phase(a, s, k, inv_nc);
      }
      __syncthreads();
      {
        // lane order of the operand: one visibility per thread, columns 4 xg .. 4 xg + 3
        const int k = tid & 31;
        const double2 kuw = sh.vb.ku_w[k];
#pragma unroll
        for (int t = 0; t < XT; ++t) {
          const int xg = (tid >> 5) + 8 * t;
          Frag rh, rl, jh, jl;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int x = 4 * xg + i;
            const float2 e = turn_phasor(kuw.x, (double)(x - L / 2), kuw.y, sh.axis[x]);
            split(e.x, e.y, rh.w[i], rl.w[i]);
            jh.w[i] = rot90(rh.w[i]);
            jl.w[i] = rot90(rl.w[i]);
          }
          Frag* f = &sh.alpha[xg >> 1][0][32 * (xg & 1) + k];
          f[0] = rh;
          f[64] = rl;
          f[128] = jh;
          f[192] = jl;
        }
      }
      stage_beta<L>(&sh.vb, sh.axis, y0, B, sh.beta);
      __syncthreads();

      // sum over x of conj(alpha) S': columns (S_re, S_im), rows (alpha_re, alpha_im) for the
      // real tile and (-alpha_im, alpha_re) for the imaginary one; ur, ui: the w series
      // without the factor 2 pi d_k b(y) of its terms, the first from columns i b(x) S'
      acc16 tr = acc16{0}, ti = acc16{0}, ur = acc16{0}, ui = acc16{0}, pr = acc16{0}, pi = acc16{0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const Frag rh = sh.alpha[ks][0][lane], rl = sh.alpha[ks][1][lane];
        const Frag jh = sh.alpha[ks][2][lane], jl = sh.alpha[ks][3][lane];
        pr = mfma(rh, sh_[ks], pr);
        pi = mfma(jh, sh_[ks], pi);
        tr = mfma(rh, sl_[ks], tr);
        ti = mfma(jh, sl_[ks], ti);
        tr = mfma(rl, sh_[ks], tr);
        ti = mfma(jl, sh_[ks], ti);
        if (s.order > 0) {
          const Frag bx = *reinterpret_cast<const Frag*>(&sh.b[0][8 * ks + 4 * h]);
          Frag u;
#pragma unroll
          for (int i = 0; i < 4; ++i) u.w[i] = swap_mul(sh_[ks].w[i], bx.w[i]);
          ur = mfma(rh, u, ur);
          ui = mfma(jh, u, ui);
          if (s.order & kWSplit) {
            const Frag b_rest = *reinterpret_cast<const Frag*>(&sh.b[1][8 * ks + 4 * h]);
            Frag rest;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const unsigned r = swap_fma_sub(sh_[ks].w[i], bx.w[i], u.w[i]);
              rest.w[i] = swap_fma(sl_[ks].w[i], bx.w[i], swap_fma(sh_[ks].w[i], b_rest.w[i], r));
            }
            ur = mfma(rh, rest, ur);
            ui = mfma(jh, rest, ui);
            ur = mfma(rl, u, ur);
            ui = mfma(jl, u, ui);
          }
          if ((s.order & kWTerms) > 1) {
            // wide fields: (2 pi d_k)^(j-1) / j! on the rows, (i b(x))^j b(y)^(j-1) S' on the columns
            const unsigned dw = sh.vb.dw[0][col], by = sh.b[0][y0 + yl] & 0xFFFF0000u;
            const unsigned by2 = by | by >> 16;
            Frag r2 = rh, j2 = jh;
            for (int j = 2; j <= (s.order & kWTerms); ++j) {
              const unsigned f = pk_mul(dw, pair_of(1.0f / (float)j));
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                r2.w[i] = pk_mul(r2.w[i], f);
                j2.w[i] = pk_mul(j2.w[i], f);
                u.w[i] = pk_mul(swap_mul(u.w[i], bx.w[i]), by2);
              }
              ur = mfma(r2, u, ur);
              ui = mfma(j2, u, ui);
            }
          }
        }
      }
      if (s.order > 0) {
        const float by = pair_high(sh.b[0][y0 + yl]) + pair_high(sh.b[1][y0 + yl]);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int k = 8 * (i >> 2) + 4 * h + (i & 3);
          const float f = by * (pair_high(sh.vb.dw[0][k]) + pair_high(sh.vb.dw[1][k]));
          tr[i] = fmaf(f, ur[i], tr[i]);
          ti[i] = fmaf(f, ui[i], ti[i]);
        }
      }
      tr += pr;
      ti += pi;
      // times conj(beta), the wave's eight rows summed: value 2 i + (0: re, 1: im) belongs to
      // visibility 8 (i >> 2) + 4 h + (i & 3) of the block
      float v[32];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float2 b = sh.beta[yl * (B + 2) + 8 * (i >> 2) + 4 * h + (i & 3)];
        v[2 * i] = b.x * tr[i] + b.y * ti[i];
        v[2 * i + 1] = b.x * ti[i] - b.y * tr[i];
      }
      // transpose-reduction over lane bits 4, 3 and 2 (the rows): each lane ends with four
      // values, 16 (bit 4) + 8 (bit 3) + 4 (bit 2) + 0 .. 3
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        swap16(v[i], v[i + 16]);
        v[i] = v[i] + v[i + 16];
      }
      const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float keep = b3 ? v[i + 8] : v[i], send = b3 ? v[i] : v[i + 8];
        v[i] = keep + dpp<kDppRowRor8>(send);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float keep = b2 ? v[i + 4] : v[i], send = b2 ? v[i] : v[i + 4];
        v[i] = keep + dpp<kDppQuadMirror>(dpp<kDppRowHalfMirror>(send));
      }
      const int i0 = 8 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1);
      const int kk = 8 * (i0 >> 2) + 4 * h + (i0 & 3);
      sh.part[wave][kk * 4 + q] = {v[0] * unscale, v[1] * unscale};
      sh.part[wave][(kk + 1) * 4 + q] = {v[2] * unscale, v[3] * unscale};
      __syncthreads();
      // the waves' sums in wave order; each output element has one thread, the same in
      // every pass
      if (tid < n * 8) {
        const float* p0 = reinterpret_cast<const float*>(sh.part[0]);
        float o = p0[tid];
#pragma unroll
        for (int w = 1; w < 4; ++w) o = o + p0[w * B * 8 + tid];
        const int k = k0 + (tid >> 3), row = (int)(((float)k + 0.5f) * inv_nc), ch = k - row * s.nc;
        int e = tid & 7;
        if (s.fold) {  // the conjugate transpose of the prediction at -uvw
          const int pol = e >> 1;
          if (e & 1) o = -o;
          e = (pol == 1 ? 4 : pol == 2 ? 2 : 2 * pol) + (e & 1);
        }
        char* dst = vis + vis_offset(row, ch, a.nc_total);
        if (y0) o += gload<float>(dst, 4 * e);
        gstore(dst, 4 * e, o);
      }
    }
  }
}

template <int L>
int launch_one(KernelClass k, const Group& g, hipStream_t st) {
  if (k == kGridDft) {
    const unsigned n = (unsigned)(g.split ? g.total_part : g.total_grp);
    const dim3 grid((n + kXcds - 1) / kXcds * kXcds * (L / kRows));
    if (g.matrix == kMatrixWide)
      hipLaunchKernelGGL((grid_matrix<L, true>), grid, dim3(kThreads), sizeof(GridLds<L>), st, g);
    else
      hipLaunchKernelGGL((grid_matrix<L, false>), grid, dim3(kThreads), sizeof(GridLds<L>), st, g);
  } else {
    hipLaunchKernelGGL((degrid_matrix<L>), dim3((unsigned)g.total_sg), dim3(kThreads), sizeof(DegridLds<L>), st, g);
  }
  return (int)hipGetLastError();
}

}  // namespace

int launch_matrix(KernelClass k, int L, const Group& g, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (g.total_sg <= 0) return 0;
  if (g.n < 1 || g.n > kMaxGroup || g.total_grp < 1 || g.total_grp > 65535 || g.total_grp > g.total_sg)
    return (int)hipErrorInvalidValue;
  switch (L) {
    case 32: return launch_one<32>(k, g, st);
    case 64: return launch_one<64>(k, g, st);
    case 96: return launch_one<96>(k, g, st);
  }
  return (int)hipErrorInvalidValue;
}

}  // namespace aidg
