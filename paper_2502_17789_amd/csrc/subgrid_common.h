// Device helpers shared by the subgrid kernels (kernels.hip, subgrid_matrix.hip): work
// mapping onto the XCDs, wave-uniform loads, the slots of a grouped launch, cross-lane
// exchanges and the store of a degridded value.
#ifndef AIDG_SUBGRID_COMMON_H
#define AIDG_SUBGRID_COMMON_H

#include <hip/hip_runtime.h>

#include "aidg_internal.h"
#include "device_common.h"

namespace aidg {
namespace {

constexpr int kThreads = 256;
// Workgroups are dispatched to the 8 XCDs (each with its own L2) round-robin by
// linear workgroup index, so index b runs on XCD b % 8.
constexpr int kXcds = 8;

// Gridder work item of linear workgroup index b: (group slot, pixel chunk) such
// that all chunks of a slot share one XCD (its visibilities are fetched into one
// L2) while consecutive slots, longest first, spread over the XCDs.  The launch
// has ceil(slots / 8) * 8 * chunks workgroups; indices past the last slot exit.
template <int Chunks>
__device__ __forceinline__ void grid_work(int64_t b, int64_t* slot, int* chunk) {
  const int64_t k = b / kXcds;
  *chunk = (int)(k % Chunks);
  *slot = (k / Chunks) * kXcds + b % kXcds;
}

// Degridder subgrid slot of linear workgroup index b < n: within every full tile
// of 64, XCD x takes the 8 consecutive slots 8x..8x+7 (subgrids of one
// same-centre group then mostly share their image in one L2); a last partial
// tile maps one to one.
__device__ __forceinline__ int64_t degrid_slot(int64_t b, int64_t n) {
  return b < (n & ~int64_t(63)) ? ((b & ~int64_t(63)) | ((b & 7) << 3) | ((b >> 3) & 7)) : b;
}
// Values every lane of a wave holds identically, moved to scalar registers word
// by word so that loop bounds and addresses derived from them stay wave-uniform
// (scalar branches, scalar loads of visibilities and uvw).
template <typename T>
__device__ __forceinline__ T uniform(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "word-sized");
  int w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

// Read-only view of memory no kernel writes while the launch runs: wave-uniform
// loads through it become scalar loads (the scalar data cache broadcasts them).
template <typename T>
using const_view = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ const_view<T> as_const(const T* p) {
  return (const_view<T>)(uintptr_t)p;
}

// A record every lane reads from the same address: scalar loads word by word.
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "word-sized");
  const_view<int> q = as_const(reinterpret_cast<const int*>(p));
  int w[sizeof(T) / 4];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(q[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

// Group slot of a grouped launch (or slot of a part of a group): the plan's parameters and
// its subgrid range.
struct GroupSlot {
  KernelArgs a;
  int64_t sb, se;  // subgrids [sb, se) of the group or part within the job's range
  int job;
  const void* in;
  void* out;
  int adjoint;
};
__device__ __forceinline__ GroupSlot resolve_group(const Group& g, int64_t slot, bool parts = false) {
  int j = 0;
  for (int i = 1; i < g.n; ++i)
    if (slot >= (parts ? g.job[i].pslot_begin : g.job[i].gslot_begin)) j = i;
  GroupSlot r;
  r.job = j;
  r.a = load_uniform(g.job[j].args);
  const int64_t k = parts ? g.job[j].p_first + (slot - g.job[j].pslot_begin)
                          : g.job[j].g_first + (slot - g.job[j].gslot_begin);
  const_view<int64_t> begin = as_const(parts ? r.a.part_begin : r.a.grp_begin);
  r.sb = max(begin[k], g.job[j].sg_begin);
  r.se = min(begin[k + 1], g.job[j].sg_end);
  r.in = uniform(g.job[j].in);
  r.out = uniform(g.job[j].out);
  r.adjoint = uniform(g.job[j].adjoint);
  return r;
}

// Subgrid slot of a grouped launch (degridder): parameters, subgrid and the
// scratch slot holding its group's image.
struct Slot {
  KernelArgs a;
  SubgridDev s;
  int64_t img_slot;
  const void* in;
  void* out;
};
__device__ __forceinline__ Slot resolve(const Group& g, int64_t slot) {
  int j = 0;
  for (int i = 1; i < g.n; ++i)
    if (slot >= g.job[i].slot_begin) j = i;
  Slot r;
  r.a = load_uniform(g.job[j].args);
  r.s = load_uniform(r.a.sg + g.job[j].sg_begin + (slot - g.job[j].slot_begin));
  r.img_slot = g.job[j].gslot_begin + (r.s.group - g.job[j].g_first);
  r.in = uniform(g.job[j].in);
  r.out = uniform(g.job[j].out);
  return r;
}

__device__ __forceinline__ void swap32(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
constexpr int kDppRowMirror = 0x140;      // lane c of a row of 16 reads lane 15 - c
constexpr int kDppRowHalfMirror = 0x141;  // lane c of a half row of 8 reads lane 7 - c
constexpr int kDppRowRor8 = 0x128;        // lane c of a row of 16 reads lane (c + 8) mod 16
constexpr int kDppQuadMirror = 0x1B;      // quad_perm [3,2,1,0]

// Output element i (= 8 x channel offset + component) of a degridded row: a folded
// sub-table returns the conjugate transpose of its prediction at -uvw.
template <typename R>
__device__ __forceinline__ void store_vis(R* vrow, int i, R v, bool fold, bool add) {
  int d = i;
  if (fold) {
    const int comp = i & 7, pol = comp >> 1;
    d = i - comp + (pol == 1 ? 2 : pol == 2 ? 1 : pol) * 2 + (comp & 1);
    if (comp & 1) v = -v;
  }
  vrow[d] = add ? vrow[d] + v : v;
}

}  // namespace
}  // namespace aidg

#endif  // AIDG_SUBGRID_COMMON_H
