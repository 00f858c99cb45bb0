// HIP kernels of the image-level step: w-stacking for imaging (Sec. 2.4, Eq. wstack;
// Sec. 2.5 imaging step 3) and its adjoint for prediction (Eq. wunstack, prediction
// step 2).  A centred N x N transform takes two or three passes over memory:
//   image_rows     whole rows through LDS.  The prediction first multiplies each image value
//                  by exp(-2 pi i w0 n1) / (L^2 T).  Up to kMaxImageStrip points the result
//                  is written transposed (kStrip rows at once), and a second such pass over
//                  the rows that were columns ends the transform.
//   image_columns  longer columns stay columns, in two steps, N = N1 N2, in tiles of 16
//                  columns: with y = y1 N2 + y2 and K = k1 + N1 k2, first the N1 rows y1 of
//                  one y2, times exp(DIR 2 pi i y2 k1 / N), in place; then the N2 rows of one
//                  k1, written as rows K.
// The last pass of the inversion multiplies by exp(+2 pi i w0 n1) / (L^2 T) and adds into the
// image (or stores, for the first layer; in the last layer's pass of the inverse A-term mode,
// the sum is divided by the normalisation map's bilinear interpolation).  All are mixed-radix
// Stockham passes through LDS; the first takes its points from memory and the last stores
// its own.  For even N, (-1)^k FFT[(-1)^x a](k) is the centred transform times (-1)^(N/2);
// the sign cancels between the two axes of a plane.
//
// Memory bounds the passes over long rows.  Per FP32 plane, inversion / prediction (W layers;
// the floor is the passes' own traffic at the 4.83 TB/s of a large copy): 8192^2 912 / 841 us
// (floor 778 / 667), 8000^2 875 / 800, 4096^2 238 / 208 (195 / 167), 2048^2 48 / 43 (35 / 28),
// 512^2 9 / 9; with four passes (row transforms of radix 5 and less, and transposes between
// them) they took 1259 / 1146, 1091 / 995, 314 / 290, 98 / 95 and 25 / 24.  FP64: 4096^2
// 418 / 361 for 785 / 751, 2048^2 104 / 102 for 209 / 206, 512^2 12 / 12 for 36 / 34.
//
// Why two ways: a strip's rows together fill half a compute unit's LDS, so beyond
// kMaxImageStrip points a strip would be narrower than 32 bytes of a column or be read several
// times (as parts of 2048 points, two passes: 4096^2 305 / 345, 8000^2 1094 / 1343), and up to
// there the third pass costs more than whole lines gain (2048^2 57 / 57 in three, 1000^2
// 25 / 24 for 16 / 16; FP64 2048^2 is even).  The written lines are shared by strips of one
// XCD's L2, which takes a contiguous range of them: dealt out over the XCDs, a transposing
// copy of 4096^2 took 64 us in place of 42.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "aidg_internal.h"
#include "device_common.h"
#include "subgrid_common.h"

namespace aidg {
namespace {

// Rows of a strip (32 bytes of a column) and threads along each; threads along a row beyond.
constexpr int kThreads1 = 512;
template <typename V2>
constexpr int kStrip = 32 / (int)sizeof(V2);
template <typename V2>
constexpr int kAlong = kThreads1 / kStrip<V2>;
// Columns of a tile and threads along each.
constexpr int kCols = 16;
template <typename V2>
constexpr int kColLanes = sizeof(V2) == 8 ? 8 : 16;
template <typename V2>
constexpr int kColThreads = kCols * kColLanes<V2>;
// The most points of a line per thread.
template <typename V2>
constexpr int kRowPoints = kMaxImageRowBytes / (int)sizeof(V2) / kThreads1;
template <typename V2>
constexpr int kStripPoints = kMaxImageStrip / kAlong<V2>;
template <typename V2>
constexpr int kColPoints = kMaxImagePart / kColLanes<V2>;
// Points that a thread takes together where the w-term's arithmetic is unrolled over them.
constexpr int kPointsW = 4;

// Place of a row's point m in LDS: a gap after every eighth point spreads the first pass's
// writes R points apart over the banks.  Rows of a strip start half the banks apart (16 mod
// 32 points): the transposed reads at the end take 16 points of four rows at once.
struct RowPlace {
  __device__ __forceinline__ int operator()(int m) const { return m + (m >> 3); }
};
__host__ __device__ inline int row_pitch(int N) { return (N - 1 + ((N - 1) >> 3) + 16) / 32 * 32 + 16; }
struct ColPlace {
  __device__ __forceinline__ int operator()(int m) const { return m * kCols; }
};

// A complex value at a byte offset from a uniform address in global memory.
template <typename V2>
__device__ __forceinline__ V2 load_at(const V2* base, unsigned off) {
  typedef decltype(V2{}.x) E __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(1))) char* Bytes;
  const E v = *(const __attribute__((address_space(1))) E*)((Bytes)base + off);
  return {v.x, v.y};
}
template <typename V2>
__device__ __forceinline__ void store_at(V2* base, unsigned off, V2 v) {
  typedef decltype(V2{}.x) E __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) char* Bytes;
  *(__attribute__((address_space(1))) E*)((Bytes)base + off) = E{v.x, v.y};
}

template <int DIR, typename V2>
__device__ __forceinline__ V2 directed(V2 w) {  // exp(-i t) -> exp(DIR i t)
  if (DIR > 0) w.y = -w.y;
  return w;
}

// y[i] *= exp(DIR 2 pi i k i / M), from the table of exp(-2 pi i a / N), N = step M.  FP32:
// the powers P b and a < P are read (six of fifteen at R = 16) and the others are one product
// of the two; FP64 powers are all read.
template <int R, int DIR, typename V2>
__device__ __forceinline__ void twiddle(V2 (&y)[R], int k, int step, const V2* __restrict__ tw) {
  using Rt = decltype(V2{}.x);
  constexpr int P = std::is_same_v<Rt, double> ? R : R <= 5 ? 2 : R <= 12 ? 3 : 4;
  const unsigned e = (unsigned)(k * step) * (unsigned)sizeof(V2);
  V2 a[P], w[(R + P - 1) / P];
#pragma unroll
  for (int i = 1; i < P; ++i) a[i] = directed<DIR>(load_at(tw, e * i));
#pragma unroll
  for (int b = 1; b * P < R; ++b) w[b] = directed<DIR>(load_at(tw, e * (P * b)));
#pragma unroll
  for (int i = 1; i < R; ++i)
    y[i] = cmul<Rt>(y[i], i < P ? a[i] : i % P == 0 ? w[i / P] : cmul<Rt>(w[i / P], a[i % P]));
}

// The Stockham passes of a line of M points in LDS, `lanes` threads (this one j0) taking
// butterflies j0, j0 + lanes, ... (Ls = product of the earlier radices): butterfly j < M / R
// reads points j + i M / R, multiplies them by exp(DIR 2 pi i k i / (Ls R)) with k = j mod Ls,
// and writes points (j / Ls) Ls R + k + i Ls.  The first pass takes its points from
// load(j, M / R, y), the last gives them to store(k, M / R, y); the others work in place:
// every read, a barrier, every write.
template <int R, int DIR, typename V2, typename Place, typename Load>
__device__ __forceinline__ void first_pass(V2* line, int M, int lanes, int j0, const Place& at, const Load& load) {
  const int m = M / R;
  for (int j = j0; j < m; j += lanes) {
    V2 y[R];
    load(j, m, y);
    butterfly<V2, R, DIR>(y);
#pragma unroll
    for (int i = 0; i < R; ++i) line[at(j * R + i)] = y[i];
  }
  __syncthreads();
}

// POINTS: the most points of a line per thread.
template <int R, int DIR, int POINTS, typename V2, typename Place>
__device__ __forceinline__ void middle_pass(V2* line, int M, int Ls, int step, int lanes, int j0, const Place& at,
                                            const V2* __restrict__ tw) {
  constexpr int T = (POINTS + R - 1) / R;
  const int m = M / R;
  const float inv_ls = 1.0f / (float)Ls;
  asm volatile("" : "+v"(j0));  // opaque: the addresses of every radix would be kept over the loop on passes
  V2 y[T][R];
  int out[T];
#pragma unroll
  for (int b = 0; b < T; ++b) {
    const int j = j0 + b * lanes;
    if (j < m) {
      // j / Ls from an FP32 quotient: (j + 1/2) / Ls is at least 1/(2 Ls) away from an
      // integer, far beyond the rounding for j < 8192 (checked exhaustively)
      const int g = (int)(((float)j + 0.5f) * inv_ls), k = j - g * Ls;
      out[b] = g * Ls * R + k;
#pragma unroll
      for (int i = 0; i < R; ++i) y[b][i] = line[at(j + i * m)];
      if (Ls > 1) twiddle<R, DIR, V2>(y[b], k, step, tw);
      butterfly<V2, R, DIR>(y[b]);
    }
  }
  __syncthreads();  // LDS reads before LDS writes
#pragma unroll
  for (int b = 0; b < T; ++b)
    if (j0 + b * lanes < m) {
#pragma unroll
      for (int i = 0; i < R; ++i) line[at(out[b] + i * Ls)] = y[b][i];
    }
  __syncthreads();
}

template <int R, int DIR, typename V2, typename Place, typename Store>
__device__ __forceinline__ void last_pass(const V2* line, int M, int step, int lanes, int j0, const Place& at,
                                          const V2* __restrict__ tw, const Store& store) {
  const int m = M / R;  // = Ls
  for (int j = j0; j < m; j += lanes) {
    V2 y[R];
#pragma unroll
    for (int i = 0; i < R; ++i) y[i] = line[at(j + i * m)];
    if (m > 1) twiddle<R, DIR, V2>(y, j, step, tw);
    butterfly<V2, R, DIR>(y);
    store(j, m, y);
  }
}

// f(radix as a constant).
template <typename R, typename F>
__device__ __forceinline__ void with_radix(int r, const F& f) {
  switch (r) {
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    case 5: return f(std::integral_constant<int, 5>());
    case 8: return f(std::integral_constant<int, 8>());
    case 10: return f(std::integral_constant<int, 10>());
  }
  if constexpr (std::is_same_v<R, float>) {  // (the registers of FP64 points end at ten)
    if (r == 16) f(std::integral_constant<int, 16>());
  }
}

// exp(sign 2 pi i w0 n1(X, Y)) / (L^2 T(X, Y)) at image pixel (X, Y), with
// l = (X - N/2) dl, m = (Y - N/2) dl and itaper[X] = 1 / t(X).  FP32 path: n1 = s - 1
// with s = sqrt(1 - l^2 - m^2) from an FP32 reciprocal square root and one FP64 residual
// correction (s to about 1e-14, so w0 n1 keeps ~1e-11 turns, far below the FP32
// phasor's own rounding).  FP64 path: the cancellation-free -r^2 / (1 + s) in FP64.
template <typename R>
__device__ __forceinline__ typename C2<R>::T wterm(int X, int Y, int N, double dl, double w0,
                                                   const double* __restrict__ itaper, double inv_l2,
                                                   double sign) {
  const R sc = (R)(inv_l2 * itaper[X] * itaper[Y]);
  if (w0 == 0.0) return {sc, (R)0};  // a layer at w = 0: the w-term is exactly 1
  const double l = (X - N / 2) * dl, m = (Y - N / 2) * dl;
  double n1;
  if constexpr (std::is_same_v<R, float>) {
    const double x = fma(-l, l, fma(-m, m, 1.0));
    const float r = __builtin_amdgcn_rsqf((float)x), s0 = (float)x * r;
    n1 = fma(fma(-(double)s0, (double)s0, x), (double)(0.5f * r), (double)s0 - 1.0);
  } else {
    const double r2 = l * l + m * m;
    n1 = -r2 / (1.0 + sqrt(1.0 - r2));
  }
  const auto ph = phasor(sign * w0 * n1, R());
  return {ph.x * sc, ph.y * sc};
}

// Bilinear interpolation of an L x L lattice map [y][x] at image pixel (X, Y), periodic
// over the field: pixel X sits at lattice coordinate g = (X - N/2) L / N + L/2, i.e.
// g N = (X - N/2) L + (L/2) N, an integer in [0, L N); its quotient by N is the lower
// lattice point (the upper one wraps to 0 past L - 1) and its remainder the weight.
template <typename R>
__device__ __forceinline__ R lattice_bilinear(const double* __restrict__ M, int L, int N, R inv_n, int X, int Y) {
  const int nx = (X - N / 2) * L + (L / 2) * N, ny = (Y - N / 2) * L + (L / 2) * N;
  const int x0 = nx / N, y0 = ny / N;
  const R fx = (R)(nx - x0 * N) * inv_n, fy = (R)(ny - y0 * N) * inv_n;
  const int x1 = x0 + 1 == L ? 0 : x0 + 1, y1 = y0 + 1 == L ? 0 : y0 + 1;
  const R r0 = (R)M[y0 * L + x0] * ((R)1 - fx) + (R)M[y0 * L + x1] * fx;
  const R r1 = (R)M[y1 * L + x0] * ((R)1 - fx) + (R)M[y1 * L + x1] * fx;
  return r0 * ((R)1 - fy) + r1 * fy;
}

template <typename V2>
struct ImageArgs {
  const V2* src;
  V2* dst;
  const V2* tw;          // exp(-2 pi i k / N)
  const double* itaper;
  const double* nmap;    // kInvertStack: normalisation map of the last layer, or null
  double dl, w0, inv_l2;
  int32_t N, L, assign;  // assign: store the first layer, do not add
  ImageRadices fr;
};

template <typename V2>
__device__ __forceinline__ V2 flip(V2 v, int odd) {  // v (-1)^odd
  return odd & 1 ? V2{-v.x, -v.y} : v;
}

// v, output (X, Y) of the layer's transform, times the w-term into the image at byte `off`,
// whose value so far is old.
template <typename R, typename V2>
__device__ __forceinline__ void stack(const ImageArgs<V2>& a, V2* img, unsigned off, V2 v, V2 old, int X, int Y) {
  v = cmul<R>(v, wterm<R>(X, Y, a.N, a.dl, a.w0, a.itaper, a.inv_l2, 1.0));
  if (!a.assign) v = V2{old.x + v.x, old.y + v.y};
  if (a.nmap) {  // divide the sum by the normalisation
    const R w = lattice_bilinear<R>(a.nmap, a.L, a.N, (R)1 / (R)a.N, X, Y);
    const R s = w > (R)0 ? (R)1 / w : (R)0;  // 0 where the map is 0
    v = V2{v.x * s, v.y * s};
  }
  store_at(img, off, v);
}

// Row transforms of the planes blockIdx.y.  STRIP: kStrip rows per workgroup, written
// transposed; otherwise one row, written in place of its own.  (PREDICT and STACK go over the
// row in LDS: the w-term's arithmetic unrolled over a butterfly's points would spill.)
template <typename R, int DIR, bool STRIP, bool PREDICT, bool STACK>
__global__ __launch_bounds__(kThreads1)
__attribute__((amdgpu_waves_per_eu(4, 4))) void image_rows(const ImageArgs<typename C2<R>::T> a) {
  using V2 = typename C2<R>::T;
  constexpr int along = STRIP ? kAlong<V2> : kThreads1, rows = STRIP ? kStrip<V2> : 1;
  extern __shared__ unsigned char smem_raw[];
  V2* buf = reinterpret_cast<V2*>(smem_raw);
  // each XCD's L2 a contiguous range of strips: neighbours share the lines they write
  const int N = a.N, per = (int)gridDim.x / kXcds;
  const int r0 = (((int)blockIdx.x % kXcds) * per + (int)blockIdx.x / kXcds) * rows;
  if (r0 >= N) return;  // padding of the last XCD (whole workgroup)
  const int c = threadIdx.x / along, j0 = threadIdx.x % along;
  const int row = min(r0 + c, N - 1);  // N is even, not always a multiple of the strip
  const RowPlace at;
  V2* line = buf + c * row_pitch(N);
  const V2* src = a.src + (size_t)blockIdx.y * N * N;  // (a plane is at most 2^29 bytes)
  V2* dst = a.dst + (size_t)blockIdx.y * N * N;
  const unsigned size = sizeof(V2), row0 = row * N * size;
  int p = 0, Ls = 1;
  if constexpr (PREDICT) {
    // points x and N - x together: their w-term is the same
    for (int jb = j0; jb <= N / 2; jb += kPointsW / 2 * along) {
      V2 v[kPointsW];
#pragma unroll
      for (int i = 0; i < kPointsW / 2; ++i) {
        const int x = min(jb + i * along, N / 2);
        v[2 * i] = load_at(src, row0 + (unsigned)x * size);
        v[2 * i + 1] = load_at(src, row0 + (unsigned)(x ? N - x : 0) * size);
      }
#pragma unroll
      for (int i = 0; i < kPointsW / 2; ++i) {
        const int x = jb + i * along;
        if (x > N / 2) break;
        const V2 w = flip(wterm<R>(x, row, N, a.dl, a.w0, a.itaper, a.inv_l2, -1.0), x);
        line[at(x)] = cmul<R>(v[2 * i], w);
        if (x) line[at(N - x)] = cmul<R>(v[2 * i + 1], w);
      }
    }
    __syncthreads();
  } else {
    auto load = [&](int j, int m, auto& y) {
      constexpr int P = sizeof(y) / sizeof(V2);
#pragma unroll
      for (int i = 0; i < P; ++i) y[i] = load_at(src, row0 + (unsigned)(j + i * m) * size);
#pragma unroll
      for (int i = 0; i < P; ++i) y[i] = flip(y[i], j + i * m);
    };
    with_radix<R>(a.fr.row.r[0], [&](auto r) { first_pass<decltype(r)::value, DIR>(line, N, along, j0, at, load); });
    Ls = a.fr.row.r[p++];
  }
  for (; p < a.fr.row.n - (STACK ? 0 : 1); ++p) {
    with_radix<R>(a.fr.row.r[p], [&](auto r) {
      constexpr int points = STRIP ? kStripPoints<V2> : kRowPoints<V2>;
      middle_pass<decltype(r)::value, DIR, points>(line, N, Ls, N / (Ls * decltype(r)::value), along, j0, at, a.tw);
    });
    Ls *= a.fr.row.r[p];
  }
  // across the rows of a strip, so that the 32 bytes of a column are written together
  const int c1 = STRIP ? threadIdx.x % rows : 0, j1 = STRIP ? threadIdx.x / rows : threadIdx.x;
  const unsigned out0 = STRIP ? (r0 + c1) * size : row0, pitch = STRIP ? N * size : size;
  if (STRIP && r0 + c1 >= N) return;
  line = buf + c1 * row_pitch(N);
  if constexpr (STACK) {
    for (int jb = j1; jb < N; jb += kPointsW * along) {
      V2 old[kPointsW];
      if (!a.assign) {
#pragma unroll
        for (int i = 0; i < kPointsW; ++i) old[i] = load_at((const V2*)dst, out0 + (unsigned)min(jb + i * along, N - 1) * pitch);
      }
#pragma unroll
      for (int i = 0; i < kPointsW; ++i) {
        const int K = jb + i * along;
        if (K >= N) break;
        stack<R, V2>(a, dst, out0 + (unsigned)K * pitch, flip(line[at(K)], K), old[i], r0 + c1, K);
      }
    }
  } else {
    auto store = [&](int k, int m, auto& y) {
      constexpr int P = sizeof(y) / sizeof(V2);
#pragma unroll
      for (int i = 0; i < P; ++i) store_at(dst, out0 + (unsigned)(k + i * m) * pitch, flip(y[i], k + i * m));
    };
    with_radix<R>(a.fr.row.r[p], [&](auto r) {
      last_pass<decltype(r)::value, DIR>((const V2*)line, N, 1, along, j1, at, a.tw, store);
    });
  }
}

// One step of the column transforms (STEP 0, 1), a workgroup the 16 columns from X0 of one
// y2 or k1 (q); STACK: the inversion's second step.
template <typename R, int DIR, int STEP, bool STACK>
__global__ __launch_bounds__(kColThreads<typename C2<R>::T>)
__attribute__((amdgpu_waves_per_eu(4, 4))) void image_columns(const ImageArgs<typename C2<R>::T> a) {
  using V2 = typename C2<R>::T;
  extern __shared__ unsigned char smem_raw[];
  const int N = a.N, N1 = a.fr.n1, N2 = N / N1, M = STEP == 0 ? N1 : N2, tiles = (N + kCols - 1) / kCols;
  const ImageFactors& f = STEP == 0 ? a.fr.col1 : a.fr.col2;
  // each XCD's L2 a contiguous range: neighbouring tiles share a line where N is no multiple of 16
  const int per = (int)gridDim.x / kXcds, unit = ((int)blockIdx.x % kXcds) * per + (int)blockIdx.x / kXcds;
  const int q = unit / tiles, X0 = (unit - q * tiles) * kCols;
  if (q >= N / M) return;  // padding of the last XCD (whole workgroup)
  const int c = threadIdx.x % kCols, j0 = threadIdx.x / kCols, X = min(X0 + c, N - 1);
  const bool live = X0 + c < N;
  constexpr int lanes = kColLanes<V2>;
  const ColPlace at;
  V2* line = reinterpret_cast<V2*>(smem_raw) + c;
  // row of point n, row of output k (a plane is at most 2^29 bytes)
  const int in_q = STEP == 0 ? 1 : N2, in_n = STEP == 0 ? N2 : 1, out_k = STEP == 0 ? N2 : N1;
  const V2* src = a.src + (size_t)blockIdx.y * N * N;
  V2* dst = a.dst + (size_t)blockIdx.y * N * N;
  const unsigned size = sizeof(V2), pitch = N * size, col = X * size;
  auto load = [&](int j, int m, auto& y) {
    constexpr int P = sizeof(y) / sizeof(V2);
#pragma unroll
    for (int i = 0; i < P; ++i) y[i] = load_at(src, (unsigned)(q * in_q + (j + i * m) * in_n) * pitch + col);
    if (STEP == 0) {
#pragma unroll
      for (int i = 0; i < P; ++i) y[i] = flip(y[i], q + (j + i * m) * N2);
    }
  };
  auto store = [&](int k, int m, auto& y) {
    constexpr int P = sizeof(y) / sizeof(V2);
    if (!live) return;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int K = q + (k + i * m) * out_k;
      V2 v = y[i];
      if (STEP == 0) v = cmul<R>(v, directed<DIR>(load_at(a.tw, (unsigned)(q * (k + i * m)) * size)));
      else v = flip(v, K);
      store_at(dst, (unsigned)K * pitch + col, v);
    }
  };
  int p = 0, Ls = 1;
  if (f.n > 1 || STACK) {
    with_radix<R>(f.r[0], [&](auto r) { first_pass<decltype(r)::value, DIR>(line, M, lanes, j0, at, load); });
    Ls = f.r[p++];
  }
  for (; p < f.n - (STACK ? 0 : 1); ++p) {
    with_radix<R>(f.r[p], [&](auto r) {
      middle_pass<decltype(r)::value, DIR, kColPoints<V2>>(line, M, Ls, N / (Ls * decltype(r)::value), lanes, j0, at,
                                                           a.tw);
    });
    Ls *= f.r[p];
  }
  if constexpr (!STACK) {
    if (f.n > 1) {
      with_radix<R>(f.r[p], [&](auto r) {
        last_pass<decltype(r)::value, DIR>(line, M, N / M, lanes, j0, at, a.tw, store);
      });
    } else {
      with_radix<R>(f.r[0], [&](auto r) {
        V2 y[decltype(r)::value];
        if (j0 > 0) return;
        load(0, 1, y);
        butterfly<V2, decltype(r)::value, DIR>(y);
        store(0, 1, y);
      });
    }
  } else {
    if (!live) return;
    for (int jb = j0; jb < M; jb += kPointsW * lanes) {
      V2 old[kPointsW];
      if (!a.assign) {
#pragma unroll
        for (int i = 0; i < kPointsW; ++i)
          old[i] = load_at((const V2*)dst, (unsigned)(q + min(jb + i * lanes, M - 1) * out_k) * pitch + col);
      }
#pragma unroll
      for (int i = 0; i < kPointsW; ++i) {
        const int j = jb + i * lanes, K = q + j * out_k;
        if (j >= M) break;
        stack<R, V2>(a, dst, (unsigned)K * pitch + col, flip(line[at(j)], K), old[i], X, K);
      }
    }
  }
}

template <typename R>
int launch_pass(ImagePass pass, const void* src, void* dst, int planes, int N, const ImageRadices& fr, const void* tw,
                const double* itaper, double dl, double w0, double inv_l2, int assign, const double* nmap, int L,
                hipStream_t st) {
  using V2 = typename C2<R>::T;
  const bool strip = image_strips(N);
  const int N1 = strip ? 0 : fr.n1, N2 = N1 > 0 ? N / N1 : 0;
  if (planes < 1 || fr.row.n < 2 || (!strip && (N1 * N2 != N || N1 > kMaxImagePart || N2 > kMaxImagePart)))
    return (int)hipErrorInvalidValue;
  const ImageArgs<V2> a = {reinterpret_cast<const V2*>(src), reinterpret_cast<V2*>(dst),
                           reinterpret_cast<const V2*>(tw), itaper, nmap, dl, w0, inv_l2, N, L, assign, fr};
  auto grid = [&](int units) { return dim3((units + kXcds - 1) / kXcds * kXcds, planes); };
  const int strips = (N + kStrip<V2> - 1) / kStrip<V2>, tiles = (N + kCols - 1) / kCols;
  const size_t lds_row = (size_t)row_pitch(N) * sizeof(V2), lds_col = (size_t)kCols * sizeof(V2);
  const dim3 rows(kThreads1), cols(kColThreads<V2>);
  const size_t lds_strip = kStrip<V2> * lds_row;
  switch (pass) {
    case kInvertRows:
      if (strip) hipLaunchKernelGGL((image_rows<R, 1, true, false, false>), grid(strips), rows, lds_strip, st, a);
      else hipLaunchKernelGGL((image_rows<R, 1, false, false, false>), grid(N), rows, lds_row, st, a);
      break;
    case kPredictRows:
      if (strip) hipLaunchKernelGGL((image_rows<R, -1, true, true, false>), grid(strips), rows, lds_strip, st, a);
      else hipLaunchKernelGGL((image_rows<R, -1, false, true, false>), grid(N), rows, lds_row, st, a);
      break;
    case kInvertColumns:
      hipLaunchKernelGGL((image_columns<R, 1, 0, false>), grid(tiles * N2), cols, N1 * lds_col, st, a);
      break;
    case kPredictColumns:
      hipLaunchKernelGGL((image_columns<R, -1, 0, false>), grid(tiles * N2), cols, N1 * lds_col, st, a);
      break;
    case kInvertStack:
      if (strip) hipLaunchKernelGGL((image_rows<R, 1, true, false, true>), grid(strips), rows, lds_strip, st, a);
      else hipLaunchKernelGGL((image_columns<R, 1, 1, true>), grid(tiles * N1), cols, N2 * lds_col, st, a);
      break;
    case kPredictGrid:
      if (strip) hipLaunchKernelGGL((image_rows<R, -1, true, false, false>), grid(strips), rows, lds_strip, st, a);
      else hipLaunchKernelGGL((image_columns<R, -1, 1, false>), grid(tiles * N1), cols, N2 * lds_col, st, a);
      break;
  }
  return (int)hipGetLastError();
}

}  // namespace

int launch_image_pass(int precision, ImagePass pass, const void* src, void* dst, int planes, int N,
                      const ImageRadices& fr, const void* tw, const double* itaper, double dl, double w0,
                      double inv_l2, int assign, const double* nmap, int L, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  return precision == AIDG_FP64
             ? launch_pass<double>(pass, src, dst, planes, N, fr, tw, itaper, dl, w0, inv_l2, assign, nmap, L, st)
             : launch_pass<float>(pass, src, dst, planes, N, fr, tw, itaper, dl, w0, inv_l2, assign, nmap, L, st);
}

}  // namespace aidg
