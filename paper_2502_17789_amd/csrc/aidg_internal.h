// Internal declarations shared by the host plan code and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/aidg.h"

namespace aidg {

constexpr double kSpeedOfLight = 299792458.0;
constexpr int kMaxSubgridVisDefault = 1024;
// The (de)gridder stages one subgrid's visibilities (8 values each) in LDS:
// 2048 of them take 64 KB in FP32 and 128 KB in FP64, within the 160 KB of a CU.
constexpr int kMaxSubgridVisLimit = 2048;
constexpr int kReseedDefault = 32;
constexpr int64_t kWorkspaceDefault = int64_t(2) << 30;
// Size of the static subgrid workspace of aidg_execute_static (AIDG_STATIC_WORKSPACE_BYTES).
constexpr int64_t kStaticWorkspaceBytes = int64_t(128) << 20;
// A group of same-centre subgrids holds at most this many times the mean
// visibilities per centre (and at least one subgrid).
constexpr int64_t kGroupVisFactor = 8;
// A part of a group costs the gridder at least this much (one subgrid excepted): three
// subgrids of up to 32 visibilities.
constexpr int64_t kMinPartCost = 156;

// Per-subgrid record the kernels read (device copy of the partition).
struct alignas(16) SubgridDev {
  int32_t t0, nt, c0, nc;      // sub-table
  int32_t U0, V0, wlayer, R;   // centre cell, layer, reseed interval (1: every channel)
  int32_t ap, aq, part, group; // A-term plane index (aint * n_st + station) of the left and
                               // right station (swapped for a folded sub-table); part of
                               // its group and (layer, centre) group, in the plan's order
  int64_t vis0;                // flat visibility index of (bl, t0, c0)
  int64_t uvw0;                // flat uvw row index of (bl, t0); folded sub-tables index the
                               // negated copy that follows the table
  double dfc;                  // channel spacing / c (s/m * Hz ... i.e. 1/m) for the recurrence
  double w0;                   // layer w, wavelengths
  int32_t fold;                // 1: visibilities enter and leave conjugate-transposed
  int32_t kind;                // degridder form: kDegridRecur, kDegridDirect or kDegridPerVis
  int32_t order;               // matrix kernels: terms of the w series (kWTerms, kWSplit)
  float wmid;                  // matrix kernels: middle of the w range, wavelengths from w0
};
// Degridder forms, chosen per subgrid by the plan (degrid_form).
constexpr int32_t kDegridRecur = 0;   // lanes own pixels; phasors step along each row's channels
constexpr int32_t kDegridDirect = 1;  // lanes own pixels; every visibility's phasor seeded directly
constexpr int32_t kDegridPerVis = 2;  // lanes own visibilities
static_assert(sizeof(SubgridDev) == 96, "SubgridDev layout");

// Geometry after validation, with derived quantities.
struct Geometry {
  int N, L, K, aterm_interval, precision, R, strict, max_sg_vis, lattice, fold, amode;
  int degrid_form;  // AIDG_DEGRID_AUTO, AIDG_DEGRID_COOPERATIVE or AIDG_DEGRID_PER_VIS
  int npol;  // grid planes: 4, or 1 for Stokes-I grids
  double dl, fov, du, beta, w_step;
  int64_t workspace;
};

// Tables of the matrix kernels.  The w-term n1(l, m) splits into a(l) + a(m) + c(l, m), a(l)
// n1(l, 0) but for what makes c smaller (axis_n1, cross), and c = -b(l) b(m) to the given
// taper-weighted residual; peak[j] is the largest taper-weighted |c|^j,
// axis_peak, cross_peak and b_peak the largest |a|, |c| and |b|.
constexpr int kMaxWOrder = 2;
constexpr int kWTerms = 3, kWSplit = 4;  // SubgridDev::order: number of terms; first term in split operands
struct WSeries {
  std::vector<double> axis_n1, b, cross;  // [L], [L], [L][L]
  double peak[kMaxWOrder + 2] = {0}, residual = 0, axis_peak = 0, cross_peak = 0, b_peak = 0;
};
void w_series(int L, double fov, const std::vector<double>& taper, WSeries* out);
// SubgridDev::order of a subgrid with |w - wmid| <= dw: the terms of the series in
// (w - wmid) c that it needs, or -1 where the matrix kernels do not apply.
int w_series_order(const WSeries& ws, double wmid, double dw);

// Host-side partition (library's own algorithm); table entries are aidg_subgrid.
struct PartitionResult {
  std::vector<aidg_subgrid> table;
  std::vector<int64_t> excluded;  // flat visibility indices
  double w_step = 0.0;            // 0: single layer
  int64_t jmin = 0, jmax = 0;
};

aidg_status validate_geometry(const aidg_geometry* g, Geometry* out, std::string* err);
double auto_w_step(const Geometry& g);
aidg_status partition(const Geometry& g, int n_st, int nbl, int nt, int nc, const int32_t* baselines,
                      const double* uvw, const double* freqs, PartitionResult* out, std::string* err);
// Host estimate of a partition's shape without building it: the w-layer range of the
// placeable visibilities, the unplaceable count, and an estimate of the number of
// subgrids (per row: the channel runs its uv extent needs, plus one per gap or layer
// change, plus the splits at max_sg_vis), and of the number of same-centre groups (the
// distinct (layer, lattice centre) pairs of the runs' midpoints, plus a quarter).
struct CentreEstimate {
  double n_subgrids = 0, n_vis = 0;
};
struct ShapeEstimate {
  int64_t jmin = 0, jmax = 0, n_excluded = 0, n_subgrids = 0, n_groups = 0;
  std::vector<CentreEstimate> centres;  // the distinct pairs
};
void estimate_shape(const Geometry& g, int nbl, int nt, int nc, const double* uvw, const double* freqs,
                    ShapeEstimate* out);
aidg_status adopt_table(const Geometry& g, int n_st, int nbl, int nt, int nc,
                        const int32_t* baselines, const aidg_subgrid* table, int64_t n_table,
                        PartitionResult* out, std::string* err);
std::vector<aidg_subgrid> split_large(const std::vector<aidg_subgrid>& t, int max_vis, int nt_total,
                                      int nc_total);
void kaiser_bessel_taper(int L, double beta, std::vector<double>* T);

// Launch parameters of one plan; the plan keeps a device copy that kernels read.
struct KernelArgs {
  const SubgridDev* sg;     // device subgrid table
  const double* uvw;        // device [nbl][nt][3] metres
  const double* fc;         // device [nc] f / c
  const void* aterms;       // device [n_int][n_st][L][L][4]
  const void* ainvh;        // device (A^-1)^H planes of the inverse A-term mode, else null
  const void* taper;        // device [L][L] taper times (-1)^(x+y)
  const void* twiddle;      // device [L] exp(-2 pi i k / L)
  // matrix kernels (FP32 plans): a (WSeries) along the lattice axis; the factor b of the
  // cross term over its largest value, rounded to FP16, then what that leaves, both as FP16
  // pairs; taper (as above) and cross term per pixel; 2 pi times the square of b's largest
  const double* axis_n1;    // device [L]
  const uint32_t* axis_b;   // device [2][L]
  const float2* taper_cross;  // device [L][L]
  double w_series;
  const int64_t* grp_begin; // device [n_groups + 1]: first subgrid of each (layer, centre) group
  const int64_t* part_begin;  // device [n_parts + 1]: the same of each part of a group
  int nt_total, nc_total, N;
  int npol;                 // grid planes: 4 (XX, XY, YX, YY) or 1 (Stokes I)
  double du;                // uv cell size, wavelengths
  double lstep;             // FOV / L, subgrid lattice spacing in direction cosines
};

// A grouped launch: consecutive ranges of subgrids from up to kMaxGroup plans
// share one kernel launch.  A plan's table is ordered so that subgrids with the
// same w-layer and centre are consecutive (a "group"); the gridder, FFT/adder and
// splitter/inverse FFT run one workgroup slot per group (slots gslot_begin..), the
// degridder one slot per subgrid (slots slot_begin..).  Group g of a range owns
// scratch slot gslot_begin + (g - g_first): its subgrid image sum, [4][L][L].  A launch
// with `split` grids by the parts of groups instead (slots pslot_begin.., scratch slot
// pslot_begin + (p - p_first)), and the adder sums the images of a group's parts.
constexpr int kMaxGroup = 16;
enum MatrixForm { kMatrixNone = 0, kMatrixPlain = 1, kMatrixWide = 2 };  // Wide: a subgrid of the plan has kWSplit
struct JobRef {
  const KernelArgs* args;   // device copy of the plan's parameters
  const void* in;           // visibilities (gridder) or grid (splitter)
  void* out;                // grid (adder) or visibilities (degridder)
  int64_t sg_begin, sg_end; // range of the plan's table
  int64_t g_first;          // group of subgrid sg_begin
  int64_t slot_begin;       // first per-subgrid slot of the range in this launch
  int64_t gslot_begin;      // first per-group slot of the range in this launch
  int32_t adjoint;          // 1: the exact adjoint of the other direction (Stokes-I plans
                            // grid XX + YY and split into diag(I, I) / 2)
  int32_t pad;
  int64_t p_first;          // part of subgrid sg_begin
  int64_t pslot_begin;      // first per-part slot of the range in this launch
};
struct Group {
  int32_t n;
  int32_t matrix;           // MatrixForm: whether the matrix kernels take the launch's DFTs
  int64_t total_sg;         // per-subgrid slots in the launch
  int64_t total_grp;        // per-group slots in the launch
  int64_t total_part;       // per-part slots in the launch
  int32_t split, pad;       // 1 (gridding): parts of groups
  void* scratch;            // [total_grp or total_part][4][L][L] subgrid images
  JobRef job[kMaxGroup];
};

// Kernel classes, in the order of aidg_kernel_times.
enum KernelClass {
  kGridDft = 0, kFftAdd = 1, kSplitIfft = 2, kDegridDft = 3, kZeroVis = 4,
  kImageFft = 5,      // image-level row and column passes (invert / predict)
  kImageWstack = 6    // invert's last column pass, with the w-stacking
};

// Degridder form of a sub-table of nt rows and nc channels (kernels.hip), `uniform`
// when its channels have a common spacing: the geometry's choice, or (automatic) the
// form of least modelled cost.  The recurrence needs a common spacing (else the
// direct form), and only sub-tables of at most the workgroup's lane count can take the
// per-visibility form (else the recurrence).
int32_t degrid_form(const Geometry& g, int nt, int nc, bool uniform);
// Modelled cost per pixel of a subgrid in its form, in visibilities of the recurrence.
double degrid_cost(int32_t kind, int nt, int nc);

// Launch one kernel class over a group (kernels.hip).  max_nv: the largest
// sub-table of the group (degridder LDS).  Returns a hipError_t as int.
int launch_group(KernelClass k, int L, int precision, const Group& g, void* stream, int max_nv);
// The DFT classes (kGridDft, kDegridDft) of an FP32 group on the matrix cores
// (subgrid_matrix.hip), for plans whose subgrids all qualify (w_series_order).
int launch_matrix(KernelClass k, int L, const Group& g, void* stream);
int launch_zero_vis(int precision, const int64_t* idx, int64_t n, void* vis, void* stream);

// Image level (image.hip).  A row of N complex values is transformed in LDS: N must
// factor into radices 4, 2, 3 and 5 and a row must fit in 64 KB.
constexpr int kMaxImageN = 8192;
constexpr int kMaxImageRowBytes = 65536;
constexpr int kMaxImageRadices = 9;
constexpr int kMaxImagePart = 128;    // points of a column step
constexpr int kMaxImageStrip = 2048;  // points of a row whose transform is written transposed
inline bool image_strips(int N) { return N <= kMaxImageStrip; }
struct ImageFactors {
  int32_t n;                     // number of Stockham passes
  int32_t r[kMaxImageRadices];   // radix of each pass
};
struct ImageRadices {
  int32_t n1;                    // column steps of n1 and N / n1 points
  ImageFactors row, col1, col2;
};
// Steps and passes of N; false when N is not supported.
bool image_radices(int N, int elem_bytes, ImageRadices* out);
void kaiser_bessel_axis(int n, double beta, std::vector<double>* t);
enum ImagePass { kInvertRows, kInvertColumns, kInvertStack, kPredictRows, kPredictColumns, kPredictGrid };
int launch_image_pass(int precision, ImagePass pass, const void* src, void* dst, int planes, int N,
                      const ImageRadices& fr, const void* tw, const double* itaper, double dl, double w0,
                      double inv_l2, int assign, const double* nmap, int L, void* stream);

// Device address of the static workspace (kStaticWorkspaceBytes) on `device`, which
// must be the current device; looked up on the first call per device, then cached.
// Null with a message in *err on failure (static_workspace.hip).
void* static_workspace(int device, std::string* err);

// Inverse A-term mode (aterm.hip): (A^-1)^H of n 2x2 matrices, and the weighted-average
// normalisation map [L2] from (A_p plane, A_q plane) pairs [n_pairs][2] with their
// visibility counts, summed in n_chunks chunks of chunk_len pairs through partial
// [n_chunks][L2].
int launch_aterm_inverse_h(int precision, const void* A, void* B, int64_t n, void* stream);
int launch_aterm_norm(int precision, const void* B, const int32_t* pairs, const double* count, int64_t n_pairs,
                      int n_chunks, int64_t chunk_len, int L2, double inv_total, double* partial, double* map,
                      void* stream);

}  // namespace aidg
