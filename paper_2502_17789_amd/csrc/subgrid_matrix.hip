// FP32 (de)gridder on the matrix cores.
//
// With n1(l, m) = a(l) + a(m) + c(l, m), a(l) = n1(l, 0), the phasor of visibility k at
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
// subgrid) and a product takes hi hi + hi lo + lo hi on v_mfma_f32_32x32x16_f16, which
// forms the products exactly and adds in FP32.  Every phase is formed and reduced to
// [-1/2, 1/2] turn in FP64; there is no recurrence.  The series' terms j >= 1 are small (the
// plan takes this path only where their largest value, times the taper, is below 1e-3)
// and take hi hi alone.
//
// What bounds it: the matrix cores at 3 (hi, lo) + 1 (first-order w term) products, and
// beside them the VALU that forms the split operands.
#include <hip/hip_runtime.h>

#include "aidg_internal.h"
#include "device_common.h"
#include "subgrid_common.h"

namespace aidg {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float acc16 __attribute__((ext_vector_type(16)));

// Eight FP16 values of one lane's matrix operand, as four packed pairs.
struct alignas(16) Frag {
  unsigned w[4];
};

__device__ __forceinline__ acc16 mfma(const Frag& a, const Frag& b, const acc16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), c, 0,
                                                0, 0);
}
__device__ __forceinline__ unsigned pk_mul(unsigned a, unsigned b) {
  return __builtin_bit_cast(unsigned, __builtin_bit_cast(half2v, a) * __builtin_bit_cast(half2v, b));
}
__device__ __forceinline__ unsigned swap_halves(unsigned p) { return __builtin_amdgcn_alignbit(p, p, 16); }
constexpr unsigned kNegHigh = 0x80000000u, kNegBoth = 0x80008000u;

// (x, y) as FP16 pairs hi + lo.
__device__ __forceinline__ void split(float x, float y, unsigned& hi, unsigned& lo) {
  const half2v h = {(_Float16)x, (_Float16)y};
  const half2v l = {(_Float16)(x - (float)h.x), (_Float16)(y - (float)h.y)};
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, l);
}
__device__ __forceinline__ unsigned pair_of(float x) {
  const half2v h = {(_Float16)x, (_Float16)x};
  return __builtin_bit_cast(unsigned, h);
}

// exp(2 pi i theta) for a phase in turns: reduced in FP64, one rounding to FP32 (2^-26
// turn), the transcendental unit's cosine and sine (absolute error at most 1.3e-7, rms
// 3.5e-8 over [-1/2, 1/2] turn, measured over 2^24 points).
__device__ __forceinline__ float2 turn_phasor(double theta) {
  const float t = (float)(theta - rint(theta));
  return {__builtin_amdgcn_cosf(t), __builtin_amdgcn_sinf(t)};
}

// Power of two that brings a largest component m to [2^9, 2^10), and its reciprocal (so
// that the low halves stay normal FP16 numbers down to 2^-23 of m).  Infinities and NaNs
// stay what they are under either factor.
__device__ __forceinline__ void fit_scale(float m, float& scale, float& unscale) {
  int e = (int)((__float_as_uint(m) >> 23) & 255) - 127;
  e = max(-110, min(e, 127));
  scale = __uint_as_float((unsigned)(127 + 9 - e) << 23);
  unscale = __uint_as_float((unsigned)(127 - 9 + e) << 23);
}

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  return m;
}

// Visibilities per LDS block and the row pitch (complex values) of the tables a lane
// reads four consecutive visibilities of: 4 more than the block shifts each row by eight
// banks.
constexpr int kBlk = 64, kBlkPitch = kBlk + 4;
// Subgrid rows (y) of one workgroup pass: 8 per wave.
constexpr int kRows = 32;

// A block's visibilities: phase coefficients in turns per lattice step (u, v) and
// wavelengths (w), and 2 pi d_k 2^-12 as an FP16 pair.
struct VisBlock {
  double2 ku_w[kBlk];
  double2 kv_w[kBlk];
  unsigned dw[kBlk];
};

__device__ __forceinline__ void stage_vis_phases(const KernelArgs& a, const SubgridDev& s, int k0, int n, float inv_nc,
                                                 VisBlock* vb) {
  const int k = threadIdx.x;
  if (k >= kBlk) return;
  double ku = 0, kv = 0, kw = 0;
  unsigned dw = 0;
  if (k < n) {
    const int row = (int)(((float)(k0 + k) + 0.5f) * inv_nc), c = k0 + k - row * s.nc;
    const double* uvw = a.uvw + 3 * (s.uvw0 + row);
    const double fc = a.fc[s.c0 + c];
    ku = (uvw[0] * fc - (s.U0 - a.N / 2) * a.du) * a.lstep;
    kv = (uvw[1] * fc - (s.V0 - a.N / 2) * a.du) * a.lstep;
    kw = uvw[2] * fc - s.w0;
    dw = pair_of((float)((kw - (double)s.wmid) * (6.283185307179586 / 4096.0)));
  }
  vb->ku_w[k] = {ku, kw};
  vb->kv_w[k] = {kv, kw};
  vb->dw[k] = dw;
}

// beta_k(y) of the workgroup's 32 rows from y0, FP32: [32][kBlkPitch].
template <int L>
__device__ __forceinline__ void stage_beta(const VisBlock* vb, const double* axis, int y0, int n8, float2* beta) {
  const int k = threadIdx.x & (kBlk - 1);
  if (k >= n8) return;
  const double2 kv = vb->kv_w[k];
#pragma unroll 2
  for (int y = threadIdx.x / kBlk; y < kRows; y += kThreads / kBlk)
    beta[y * kBlkPitch + k] = turn_phasor(fma(kv.x, (double)(y0 + y - L / 2), kv.y * axis[y0 + y]));
}

// ------------------------------------------------------------------ gridder

// Gridder LDS: alpha operands, beta, the visibilities [4][kBlkPitch], phases, axis tables.
template <int L>
struct GridLds {
  Frag alpha[kBlk / 8][L / 32][2][64];
  float2 beta[kRows * kBlkPitch];
  float2 vis[4 * kBlkPitch];
  VisBlock vb;
  double axis[L];
  unsigned b[L];
  float red[4];
};

// One workgroup per (32 rows, group).  Each wave owns 8 rows x 4 polarisations (the 32
// rows of the matrix tiles) by L columns, real and imaginary parts in separate tiles, so
// that a lane ends with all four polarisations of its L/8 pixels: the Jones epilogue is
// lane-local and the group's sum stays in registers (a subgrid's image does not go through
// memory).  Rows are V_k beta_k(y), formed and split by the wave that uses them; columns are
// alpha_k(x), formed once per workgroup and read from LDS in the operand's lane order.
template <int L>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void grid_matrix(const Group g) {
  constexpr int XT = L / 32, NP = 4;  // column tiles; pixels per lane and tile
  extern __shared__ unsigned char smem_raw[];
  GridLds<L>& sh = *reinterpret_cast<GridLds<L>*>(smem_raw);
  int64_t local;
  int chunk;
  grid_work<L / kRows>(blockIdx.x, &local, &chunk);
  if (local >= g.total_grp) return;  // padding of the last XCD round (whole workgroup)
  const GroupSlot gs = resolve_group(g, local);
  const KernelArgs& a = gs.a;
  const float* __restrict__ vis = reinterpret_cast<const float*>(gs.in);
  const bool inv = a.ainvh != nullptr;
  const float2* At = reinterpret_cast<const float2*>(inv ? a.ainvh : a.aterms);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, h = lane >> 5;
  const int y0 = chunk * kRows;
  for (int i = tid; i < L; i += kThreads) {
    sh.axis[i] = a.axis_n1[i];
    sh.b[i] = a.axis_b[i];
  }
  // operand row of this lane: polarisation q of row yl of the wave's eight
  const int q = col & 3, yl = wave * 8 + (col >> 2);

  float sum[XT][NP][8];
#pragma unroll
  for (int t = 0; t < XT; ++t)
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int i = 0; i < 8; ++i) sum[t][p][i] = 0;

  for (int64_t si = gs.sb; si < gs.se; ++si) {
    const SubgridDev s = load_uniform(a.sg + si);
    const int nv = s.nt * s.nc;
    const float inv_nc = 1.0f / (float)s.nc;
    // half i & 1 (polarisations 2 (i & 1) and the next) of the subgrid's visibility i >> 1;
    // (k + 1/2) / nc is at least 1 / (2 nc) from an integer, beyond FP32 rounding for
    // k < 2048.  A folded sub-table is read as V^H.
    auto fetch = [&](int i) -> float4 {
      const int k = i >> 1, row = (int)(((float)k + 0.5f) * inv_nc), c = k - row * s.nc;
      const float4* src = reinterpret_cast<const float4*>(vis) + (s.vis0 + (int64_t)row * a.nc_total + c) * 2;
      if (s.fold) {
        const float4 h0 = src[0], h1 = src[1];
        return (i & 1) ? float4{h0.z, -h0.w, h1.z, -h1.w} : float4{h0.x, -h0.y, h1.x, -h1.y};
      }
      return src[i & 1];
    };
    float m = 0;
    float4 first = {0, 0, 0, 0};
    for (int i = tid; i < 2 * nv; i += kThreads) {
      const float4 v = fetch(i);
      if (i == tid) first = v;
      m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
    m = wave_max(m);
    if (lane == 0) sh.red[wave] = m;
    acc16 re[XT], im[XT];
#pragma unroll
    for (int t = 0; t < XT; ++t) re[t] = im[t] = acc16{0};
    float scale = 1, unscale = 1;

    for (int k0 = 0; k0 < nv; k0 += kBlk) {
      const int n = min(kBlk, nv - k0), n8 = (n + 7) & ~7;
      __syncthreads();  // the previous block is no longer read; the maxima are in
      if (k0 == 0) {
        fit_scale(fmaxf(fmaxf(sh.red[0], sh.red[1]), fmaxf(sh.red[2], sh.red[3])), scale, unscale);
      }
      stage_vis_phases(a, s, k0, n, inv_nc, &sh.vb);
      if (tid < 2 * kBlk) {
        const int k = tid >> 1, p = 2 * (tid & 1);
        float4 v = {0, 0, 0, 0};
        if (k < n) v = k0 == 0 ? first : fetch(2 * k0 + tid);
        sh.vis[p * kBlkPitch + k] = {v.x * scale, v.y * scale};
        sh.vis[(p + 1) * kBlkPitch + k] = {v.z * scale, v.w * scale};
      }
      __syncthreads();
      for (int id = tid; id < L * (n8 / 4); id += kThreads) {
        const int x = id % L, kg = id / L;
        const double dx = (double)(x - L / 2), ax = sh.axis[x];
        Frag fh, fl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double2 kuw = sh.vb.ku_w[4 * kg + i];
          const float2 e = turn_phasor(fma(kuw.x, dx, kuw.y * ax));
          split(e.x, e.y, fh.w[i], fl.w[i]);
        }
        sh.alpha[kg >> 1][x >> 5][0][32 * (kg & 1) + (x & 31)] = fh;
        sh.alpha[kg >> 1][x >> 5][1][32 * (kg & 1) + (x & 31)] = fl;
      }
      stage_beta<L>(&sh.vb, sh.axis, y0, n8, sh.beta);
      __syncthreads();

      for (int ks = 0; ks < n8 / 8; ++ks) {
        // W_k = V_k beta_k(y) for the lane's four visibilities: rows (W_re, -W_im) for the
        // real tile and (W_im, W_re) for the imaginary one
        const int k = 8 * ks + 4 * h;
        Frag rh, rl, ih, il;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float2 w = cmul<float>(sh.vis[q * kBlkPitch + k + i], sh.beta[yl * kBlkPitch + k + i]);
          unsigned hi, lo;
          split(w.x, w.y, hi, lo);
          rh.w[i] = hi ^ kNegHigh;
          rl.w[i] = lo ^ kNegHigh;
          ih.w[i] = swap_halves(hi);
          il.w[i] = swap_halves(lo);
        }
#pragma unroll
        for (int t = 0; t < XT; ++t) {
          const Frag bh = sh.alpha[ks][t][0][lane], bl = sh.alpha[ks][t][1][lane];
          re[t] = mfma(rh, bh, re[t]);
          im[t] = mfma(ih, bh, im[t]);
          re[t] = mfma(rh, bl, re[t]);
          im[t] = mfma(ih, bl, im[t]);
          re[t] = mfma(rl, bh, re[t]);
          im[t] = mfma(il, bh, im[t]);
        }
        if (s.order > 0) {
          // w series: rows times -i 2 pi d_k b(y) / j, columns times b(x), per order j (the
          // b tables hold 64 b and d 2^-12 of its value)
          const unsigned by = sh.b[y0 + yl];
          unsigned bx[XT], gk[4];
#pragma unroll
          for (int t = 0; t < XT; ++t) bx[t] = sh.b[t * 32 + col];
#pragma unroll
          for (int i = 0; i < 4; ++i) gk[i] = pk_mul(sh.vb.dw[k + i], by);
          for (int j = 1;; ++j) {
            Frag nr, ni;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              nr.w[i] = pk_mul(ih.w[i], gk[i]);
              ni.w[i] = pk_mul(rh.w[i] ^ kNegBoth, gk[i]);
            }
            rh = nr;
            ih = ni;
#pragma unroll
            for (int t = 0; t < XT; ++t) {
              Frag b = sh.alpha[ks][t][0][lane];
#pragma unroll
              for (int i = 0; i < 4; ++i) b.w[i] = pk_mul(b.w[i], bx[t]);
              re[t] = mfma(rh, b, re[t]);
              im[t] = mfma(ih, b, im[t]);
            }
            if (j == s.order) break;
            const unsigned f = pair_of((float)j / (float)(j + 1));
#pragma unroll
            for (int i = 0; i < 4; ++i) gk[i] = pk_mul(gk[i], f);
#pragma unroll
            for (int t = 0; t < XT; ++t) bx[t] = pk_mul(bx[t], sh.b[t * 32 + col]);
          }
        }
      }
    }
    // Jones correction of this subgrid, A_p^H S A_q, tapered and added to the group's sum
#pragma unroll
    for (int t = 0; t < XT; ++t) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int pix = (y0 + wave * 8 + 2 * p + h) * L + t * 32 + col;
        const float2* Ap = At + ((int64_t)s.ap * L * L + pix) * 4;
        const float2* Aq = At + ((int64_t)s.aq * L * L + pix) * 4;
        float2 a0 = Ap[0], a1 = Ap[1], a2 = Ap[2], a3 = Ap[3];
        a0.y = -a0.y; a1.y = -a1.y; a2.y = -a2.y; a3.y = -a3.y;  // conj
        float2 b0 = Aq[0], b1 = Aq[1], b2 = Aq[2], b3 = Aq[3];
        const float2 tc = a.taper_cross[pix];
        float w = tc.x * unscale;
        if (inv) {
          // ||B_p^H B_q||_F^2 with B_p^H = [[a0, a2], [a1, a3]] (a already conjugated)
          const float2 m0 = cmul<float>(a0, b0) + cmul<float>(a2, b2), m1 = cmul<float>(a0, b1) + cmul<float>(a2, b3);
          const float2 m2 = cmul<float>(a1, b0) + cmul<float>(a3, b2), m3 = cmul<float>(a1, b1) + cmul<float>(a3, b3);
          const float n2 = m0.x * m0.x + m0.y * m0.y + m1.x * m1.x + m1.y * m1.y + m2.x * m2.x + m2.y * m2.y +
                           m3.x * m3.x + m3.y * m3.y;
          w = n2 > 0.0f ? w / sqrtf(n2) : 0.0f;
        }
        // taper and E(w_s c), |w_s c| < 1/2 turn
        const float ph = s.wmid * tc.y;
        const float2 e = {w * __builtin_amdgcn_cosf(ph), w * __builtin_amdgcn_sinf(ph)};
        const float2 s0 = cmul<float>(e, float2{re[t][4 * p], im[t][4 * p]});
        const float2 s1 = cmul<float>(e, float2{re[t][4 * p + 1], im[t][4 * p + 1]});
        const float2 s2 = cmul<float>(e, float2{re[t][4 * p + 2], im[t][4 * p + 2]});
        const float2 s3 = cmul<float>(e, float2{re[t][4 * p + 3], im[t][4 * p + 3]});
        // A_p^H = [[conj a0, conj a2], [conj a1, conj a3]]
        const float2 t0 = cmul<float>(a0, s0) + cmul<float>(a2, s2);
        const float2 t1 = cmul<float>(a0, s1) + cmul<float>(a2, s3);
        const float2 t2 = cmul<float>(a1, s0) + cmul<float>(a3, s2);
        const float2 t3 = cmul<float>(a1, s1) + cmul<float>(a3, s3);
        const float2 c0 = cmul<float>(t0, b0) + cmul<float>(t1, b2), c1 = cmul<float>(t0, b1) + cmul<float>(t1, b3);
        const float2 c2 = cmul<float>(t2, b0) + cmul<float>(t3, b2), c3 = cmul<float>(t2, b1) + cmul<float>(t3, b3);
        float* d = sum[t][p];
        d[0] += c0.x; d[1] += c0.y; d[2] += c1.x; d[3] += c1.y;
        d[4] += c2.x; d[5] += c2.y; d[6] += c3.x; d[7] += c3.y;
      }
    }
  }

  float2* out = reinterpret_cast<float2*>(g.scratch) + local * 4 * L * L;
  // Stokes-I grid: I = (XX + YY) / 2 of the corrected image, plane 0 only
  const float fi = gs.adjoint ? 1.0f : 0.5f;
#pragma unroll
  for (int t = 0; t < XT; ++t) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int pix = (y0 + wave * 8 + 2 * p + h) * L + t * 32 + col;
      const float* d = sum[t][p];
      if (a.npol == 1) {
        out[pix] = {(d[0] + d[6]) * fi, (d[1] + d[7]) * fi};
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) out[k * L * L + pix] = {d[2 * k], d[2 * k + 1]};
      }
    }
  }
}

// ------------------------------------------------------------------ degridder

// Degridder LDS: alpha operands [tile of 32 visibilities][x step], beta, phases, the waves'
// partial visibilities, axis tables.  While a pass's image is laid out, the first part holds
// 32 columns of each wave's rows: [hi, lo][wave][row][kLayPitch].
constexpr int kLayPitch = 36;
template <int L>
struct DegridLds {
  union {
    Frag alpha[kBlk / 32][L / 8][2][64];
    unsigned lay[2][4][32][kLayPitch];
  };
  float2 beta[kRows * kBlkPitch];
  VisBlock vb;
  float2 part[4][kBlk * 4];
  double axis[L];
  unsigned b[L];
};

// One workgroup per subgrid, 32 rows of the subgrid at a time.  Each wave corrects its
// 8 rows of the group image (A_p S A_q^H, taper, E(-w_s c)), splits them and keeps them in
// registers as the operand [x][(row, polarisation)] for all visibilities of the pass;
// alpha_k(x) is formed by the workgroup, 64 visibilities at a time, as the other operand.
// A tile's 32 visibilities x 8 rows x 4 polarisations are multiplied by conj(beta_k(y)) and
// summed over the rows across lanes; the waves' sums meet in LDS and are added to the output
// in wave order (deterministic, no atomics).
template <int L>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void degrid_matrix(const Group g) {
  constexpr int XT = L / 32, NP = 4, KS = L / 8;
  extern __shared__ unsigned char smem_raw[];
  DegridLds<L>& sh = *reinterpret_cast<DegridLds<L>*>(smem_raw);
  const int64_t local = degrid_slot(blockIdx.x, g.total_sg);
  const Slot sl = resolve(g, local);
  const KernelArgs& a = sl.a;
  const SubgridDev& s = sl.s;
  float* __restrict__ vis = reinterpret_cast<float*>(sl.out);
  const float2* img = reinterpret_cast<const float2*>(g.scratch) + sl.img_slot * 4 * L * L;
  const float2* At = reinterpret_cast<const float2*>(a.aterms);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, h = lane >> 5;
  const int nv = s.nt * s.nc;
  const float inv_nc = 1.0f / (float)s.nc;
  for (int i = tid; i < L; i += kThreads) {
    sh.axis[i] = a.axis_n1[i];
    sh.b[i] = a.axis_b[i];
  }
  // operand column of this lane: polarisation q of row yl of the wave's eight
  const int q = col & 3, yl = wave * 8 + (col >> 2);

  for (int y0 = 0; y0 < L; y0 += kRows) {
    // the wave's rows, corrected: lane (col, h) takes column x = 32 t + col of rows 2 p + h
    float c[XT][NP][8];
    float m = 0;
#pragma unroll
    for (int t = 0; t < XT; ++t) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int pix = (y0 + wave * 8 + 2 * p + h) * L + t * 32 + col;
        const float2* Ap = At + ((int64_t)s.ap * L * L + pix) * 4;
        const float2* Aq = At + ((int64_t)s.aq * L * L + pix) * 4;
        const float2 a0 = Ap[0], a1 = Ap[1], a2 = Ap[2], a3 = Ap[3];
        float2 b0 = Aq[0], b1 = Aq[1], b2 = Aq[2], b3 = Aq[3];
        b0.y = -b0.y; b1.y = -b1.y; b2.y = -b2.y; b3.y = -b3.y;  // conj
        const float2 tc = a.taper_cross[pix];
        const float ph = s.wmid * tc.y;
        const float2 e = {tc.x * __builtin_amdgcn_cosf(ph), -tc.x * __builtin_amdgcn_sinf(ph)};
        const float2 s0 = cmul<float>(e, img[pix]), s1 = cmul<float>(e, img[L * L + pix]);
        const float2 s2 = cmul<float>(e, img[2 * L * L + pix]), s3 = cmul<float>(e, img[3 * L * L + pix]);
        const float2 t0 = cmul<float>(a0, s0) + cmul<float>(a1, s2);
        const float2 t1 = cmul<float>(a0, s1) + cmul<float>(a1, s3);
        const float2 t2 = cmul<float>(a2, s0) + cmul<float>(a3, s2);
        const float2 t3 = cmul<float>(a2, s1) + cmul<float>(a3, s3);
        // A_q^H = [[conj b0, conj b2], [conj b1, conj b3]]
        const float2 r0 = cmul<float>(t0, b0) + cmul<float>(t1, b1), r1 = cmul<float>(t0, b2) + cmul<float>(t1, b3);
        const float2 r2 = cmul<float>(t2, b0) + cmul<float>(t3, b1), r3 = cmul<float>(t2, b2) + cmul<float>(t3, b3);
        float* d = c[t][p];
        d[0] = r0.x; d[1] = r0.y; d[2] = r1.x; d[3] = r1.y;
        d[4] = r2.x; d[5] = r2.y; d[6] = r3.x; d[7] = r3.y;
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(d[i]));
      }
    }
    float scale, unscale;
    fit_scale(wave_max(m), scale, unscale);
    __syncthreads();  // the previous pass's operands are no longer read
    // operand order: lane (col, h) holds row (yl, q), columns 8 ks + 4 h + 0 .. 3
    Frag ih[KS], il[KS];
#pragma unroll
    for (int t = 0; t < XT; ++t) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          unsigned hi, lo;
          split(c[t][p][2 * k] * scale, c[t][p][2 * k + 1] * scale, hi, lo);
          sh.lay[0][wave][(2 * p + h) * 4 + k][col] = hi;
          sh.lay[1][wave][(2 * p + h) * 4 + k][col] = lo;
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ih[4 * t + i] = *reinterpret_cast<const Frag*>(&sh.lay[0][wave][col][8 * i + 4 * h]);
        il[4 * t + i] = *reinterpret_cast<const Frag*>(&sh.lay[1][wave][col][8 * i + 4 * h]);
      }
    }

    for (int k0 = 0; k0 < nv; k0 += kBlk) {
      const int n = min(kBlk, nv - k0);
      __syncthreads();  // operands (or the laid-out image) and partial sums no longer read
      stage_vis_phases(a, s, k0, n, inv_nc, &sh.vb);
      __syncthreads();
      const int tiles = (n + 31) / 32;
      for (int id = tid; id < (L / 4) * 32 * tiles; id += kThreads) {
        // lane order of the operand: visibility id & 31 of a tile, columns 4 xg .. 4 xg + 3
        const int k = id & 31, xg = (id >> 5) % (L / 4), tile = (id >> 5) / (L / 4);
        const double2 kuw = sh.vb.ku_w[32 * tile + k];
        Frag fh, fl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int x = 4 * xg + i;
          const float2 e = turn_phasor(fma(kuw.x, (double)(x - L / 2), kuw.y * sh.axis[x]));
          split(e.x, e.y, fh.w[i], fl.w[i]);
        }
        sh.alpha[tile][xg >> 1][0][32 * (xg & 1) + k] = fh;
        sh.alpha[tile][xg >> 1][1][32 * (xg & 1) + k] = fl;
      }
      stage_beta<L>(&sh.vb, sh.axis, y0, 32 * tiles, sh.beta);
      __syncthreads();

      for (int tile = 0; tile < tiles; ++tile) {
        // sum over x of conj(alpha) S': rows (alpha_re, alpha_im), columns (S_re, S_im) for
        // the real tile and (S_im, -S_re) for the imaginary one
        acc16 tr = acc16{0}, ti = acc16{0};
        const unsigned by = sh.b[y0 + yl], dw = sh.vb.dw[32 * tile + col];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const Frag ah = sh.alpha[tile][ks][0][lane], al = sh.alpha[tile][ks][1][lane];
          Frag jh, jl;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            jh.w[i] = swap_halves(ih[ks].w[i]) ^ kNegHigh;
            jl.w[i] = swap_halves(il[ks].w[i]) ^ kNegHigh;
          }
          tr = mfma(ah, ih[ks], tr);
          ti = mfma(ah, jh, ti);
          tr = mfma(ah, il[ks], tr);
          ti = mfma(ah, jl, ti);
          tr = mfma(al, ih[ks], tr);
          ti = mfma(al, jh, ti);
          if (s.order > 0) {
            // w series, conjugated: rows times 2 pi d_k / j, columns times i b(x) b(y)
            Frag ar = ah, cr = ih[ks], ci = jh;
            unsigned bb[4], f = dw;
            const Frag bx = {sh.b[8 * ks + 4 * h], sh.b[8 * ks + 4 * h + 1], sh.b[8 * ks + 4 * h + 2],
                             sh.b[8 * ks + 4 * h + 3]};
#pragma unroll
            for (int i = 0; i < 4; ++i) bb[i] = pk_mul(bx.w[i], by);
            for (int j = 1;; ++j) {
              Frag nr, ni;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                ar.w[i] = pk_mul(ar.w[i], f);
                nr.w[i] = pk_mul(ci.w[i] ^ kNegBoth, bb[i]);
                ni.w[i] = pk_mul(cr.w[i], bb[i]);
              }
              cr = nr;
              ci = ni;
              tr = mfma(ar, cr, tr);
              ti = mfma(ar, ci, ti);
              if (j == s.order) break;
              f = pk_mul(f, pair_of((float)j / (float)(j + 1)));
            }
          }
        }
        // times conj(beta), the wave's eight rows summed: value 2 i + (0: re, 1: im) belongs to
        // visibility 8 (i >> 2) + 4 h + (i & 3) of the tile
        float v[32];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float2 b = sh.beta[yl * kBlkPitch + 32 * tile + 8 * (i >> 2) + 4 * h + (i & 3)];
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
        const int kk = 32 * tile + 8 * (i0 >> 2) + 4 * h + (i0 & 3);
        sh.part[wave][kk * 4 + q] = {v[0] * unscale, v[1] * unscale};
        sh.part[wave][(kk + 1) * 4 + q] = {v[2] * unscale, v[3] * unscale};
      }
      __syncthreads();
      // the waves' sums in wave order; each output element has one thread, the same in
      // every pass
      for (int i = tid; i < n * 8; i += kThreads) {
        const float* p0 = reinterpret_cast<const float*>(sh.part[0]);
        float v = p0[i];
#pragma unroll
        for (int w = 1; w < 4; ++w) v = v + p0[w * kBlk * 8 + i];
        const int k = k0 + (i >> 3), row = (int)(((float)k + 0.5f) * inv_nc), ch = k - row * s.nc;
        store_vis(vis + (s.vis0 + (int64_t)row * a.nc_total + ch) * 8, i & 7, v, s.fold != 0, y0 != 0);
      }
    }
  }
}

template <int L>
int launch_one(KernelClass k, const Group& g, hipStream_t st) {
  if (k == kGridDft) {
    const unsigned n = (unsigned)g.total_grp;
    hipLaunchKernelGGL((grid_matrix<L>), dim3((n + kXcds - 1) / kXcds * kXcds * (L / kRows)), dim3(kThreads),
                       sizeof(GridLds<L>), st, g);
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
