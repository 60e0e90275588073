// fg_device.h -- device-side building blocks shared by the kernel translation
// units: wavefront constants, vector loads and stores, cross-lane primitives,
// work items, and the small host helpers of the launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "fg_internal.h"

namespace fg {
namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;

// Work item of the calling wavefront, as a wave-uniform (scalar) value.
__device__ __forceinline__ int64_t wave_item() {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return (int64_t)blockIdx.x * kWavesPerBlock + w;
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Compile-time flag passed to generic lambdas (decltype(tag)::value).
template <bool B>
struct BoolTag {
  static constexpr bool value = B;
};

// Offset of source row `src` in a [rows, F] array.  Both factors are
// non-negative and below 2^32 (src < 2^31, F <= 65536), so one unsigned
// 32 x 32 -> 64-bit multiply replaces the signed 64-bit product, which costs
// two 32-bit multiplies, a 64-bit multiply-add and a sign extension (the
// gather kernels are partly bound by vector instruction issue).
__device__ __forceinline__ uint64_t row_off(int32_t src, int64_t F) {
  return (uint64_t)(uint32_t)src * (uint32_t)F;
}

// The same for a lane's element pointer xl (the array plus the lane's
// element offset) and the row size in bytes (F * 4 <= 2^18): one unsigned
// 32 x 32 + 64-bit multiply-add per gather, where p + row_off(src, F) + f
// takes a multiply, a shift and a 64-bit add.
__device__ __forceinline__ const float* row_at(const char* xl, int32_t src, uint32_t rb) {
  return reinterpret_cast<const float*>(xl + (uint64_t)(uint32_t)src * rb);
}

template <int VEC>
__device__ __forceinline__ void load_vec(const float* p, float (&r)[VEC]) {
  if constexpr (VEC == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    r[0] = t.x; r[1] = t.y; r[2] = t.z; r[3] = t.w;
  } else {
    r[0] = *p;
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&r)[VEC]) {
  if constexpr (VEC == 4) {
    *reinterpret_cast<float4*>(p) = make_float4(r[0], r[1], r[2], r[3]);
  } else {
    *p = r[0];
  }
}

// Non-temporal forms for results no later step of the kernel reads: they
// should not displace the gathered rows from the L2.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

template <int VEC>
__device__ __forceinline__ void store_vec_nt(float* p, const float (&r)[VEC]) {
  if constexpr (VEC == 4) {
    __builtin_nontemporal_store(f32x4{r[0], r[1], r[2], r[3]}, reinterpret_cast<f32x4*>(p));
  } else {
    __builtin_nontemporal_store(r[0], p);
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec_i_nt(int32_t* p, const int32_t (&r)[VEC]) {
  if constexpr (VEC == 4) {
    __builtin_nontemporal_store(i32x4{r[0], r[1], r[2], r[3]}, reinterpret_cast<i32x4*>(p));
  } else {
    __builtin_nontemporal_store(r[0], p);
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec_i(int32_t* p, const int32_t (&r)[VEC]) {
  if constexpr (VEC == 4) {
    *reinterpret_cast<int4*>(p) = make_int4(r[0], r[1], r[2], r[3]);
  } else {
    *p = r[0];
  }
}

// (value, edge id) order of the max reducer: larger value wins, equal values
// (IEEE ==, so -0 == +0) go to the smaller edge id.
__device__ __forceinline__ bool takes_over(float m, int32_t e, float best, int32_t best_e) {
  return m > best || (m == best && e < best_e);
}

// A NaN message competes as -inf: it never beats a number, and a row whose
// messages are all NaN or -inf reports -inf with its smallest edge id.  (The
// positional-id comparison "strictly greater replaces" behaves so by itself.)
__device__ __forceinline__ float max_key(float m) { return m != m ? -INFINITY : m; }

// ---- cross-lane primitives --------------------------------------------------

// DPP controls (GFX9 encoding, valid on gfx950).
constexpr int kDppQuadXor1 = 0xB1;      // quad_perm:[1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;      // quad_perm:[2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowBcast15 = 0x142;   // lane 15 of each row -> next row
constexpr int kDppRowBcast31 = 0x143;   // lane 31 -> rows 2 and 3
constexpr int kDppWaveShr1 = 0x138;     // lane l - 1 -> lane l

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}

// Sum over aligned groups of W lanes (W a power of two <= 64).  The total is
// valid in lane W-1 of every group; for W <= 16 in every lane of the group.
// Every lane of the wavefront must execute this.
template <int W>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (W >= 2) v += dpp_f<kDppQuadXor1>(v);
  if constexpr (W >= 4) v += dpp_f<kDppQuadXor2>(v);
  if constexpr (W >= 8) v += dpp_f<kDppRowHalfMirror>(v);
  if constexpr (W >= 16) v += dpp_f<kDppRowMirror>(v);
  if constexpr (W >= 32) v += dpp_f<kDppRowBcast15, 0xA>(v);
  if constexpr (W >= 64) v += dpp_f<kDppRowBcast31, 0x8>(v);
  return v;
}

// Value of lane (jb + gid) where jb is wave-uniform and gid < NG is the lane
// group of the caller.  One or two groups use scalar readlanes.
template <int NG>
__device__ __forceinline__ int bcast_lane(int v, int jb, int gid) {
  if constexpr (NG == 1) {
    return __builtin_amdgcn_readlane(v, jb);
  } else if constexpr (NG == 2) {
    const int a = __builtin_amdgcn_readlane(v, jb);
    const int b = __builtin_amdgcn_readlane(v, jb + 1);
    return gid ? b : a;
  } else {
    return __shfl(v, jb + gid);
  }
}

template <int NG>
__device__ __forceinline__ float bcast_lane_f(float v, int jb, int gid) {
  return __builtin_bit_cast(float, bcast_lane<NG>(__builtin_bit_cast(int, v), jb, gid));
}

// Wide batches of Q * 64 edges (gather kernels on long items): lane l holds
// edges Q*l .. Q*l + Q - 1 of the batch (Q = 4 when a step covers whole
// lanes, else 1), so the ids of 256 edges arrive in one 16-byte load per lane
// (and the SDDMM's results leave in one 16-byte store): the address unit that
// bounds the gather kernels spends one instruction on each instead of four,
// and an item of up to 256 edges waits for one id load instead of several.
template <int NG, int U>
constexpr int ids_per_lane() { return (NG * U) % 4 == 0 && (NG == 1 || U % 4 == 0) ? 4 : 1; }

// Average item length from which wide batches pay: two lane groups (rows of
// 65-128 floats) gain from the quarter of the id loads on long items only;
// four or more groups (narrower rows, where a step of U edges per group
// spans 64 or more edges) also gain from waiting for one id load per item.
template <int NG>
constexpr int64_t wide_item_edges() { return NG >= 4 ? kWideItemEdgesMany : kWideItemEdges; }


template <int Q, typename T>
__device__ __forceinline__ T pick(const T (&v)[Q], int c) {
  if constexpr (Q == 1) {
    return v[0];
  } else {
    return c == 0 ? v[0] : c == 1 ? v[1] : c == 2 ? v[2] : v[3];
  }
}

typedef int32_t int4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Four floats (ids) at p; RAG: p is only 4-byte aligned (gfx950 loads and
// stores it as one 16-byte access all the same).
template <bool RAG>
__device__ __forceinline__ void load4(const float* p, float (&r)[4]) {
  if constexpr (RAG) {
    const float4_a4 t = *reinterpret_cast<const float4_a4*>(p);
    r[0] = t.x; r[1] = t.y; r[2] = t.z; r[3] = t.w;
  } else {
    load_vec<4>(p, r);
  }
}

// Stores elements lo..3 (lo > 0 only with RAG: the tail of a ragged row,
// whose first lo elements belong to the neighbouring lane).
template <bool RAG>
__device__ __forceinline__ void store4_nt(float* p, const float (&r)[4], int lo) {
  if constexpr (RAG) {
    if (lo == 0) {
      __builtin_nontemporal_store(float4_a4{r[0], r[1], r[2], r[3]},
                                  reinterpret_cast<float4_a4*>(p));
    } else {
#pragma unroll
      for (int c = 1; c < 4; ++c)
        if (c >= lo) __builtin_nontemporal_store(r[c], p + c);
    }
  } else {
    store_vec_nt<4>(p, r);
  }
}

template <bool RAG>
__device__ __forceinline__ void store4_i_nt(int32_t* p, const int32_t (&r)[4], int lo) {
  if constexpr (RAG) {
    if (lo == 0) {
      __builtin_nontemporal_store(int4_a4{r[0], r[1], r[2], r[3]}, reinterpret_cast<int4_a4*>(p));
    } else {
#pragma unroll
      for (int c = 1; c < 4; ++c)
        if (c >= lo) __builtin_nontemporal_store(r[c], p + c);
    }
  } else {
    store_vec_i_nt<4>(p, r);
  }
}

// Edges base + Q*lane + q (q < Q) of a batch of `cnt` edges from a streamed
// int32 array of `len` elements (non-temporal); 0 past cnt.  A lane with
// edges in the batch takes its Q with one 16-byte load (4-byte aligned:
// gfx950 loads it unaligned) when they lie inside the array, else (only at
// its very end) one by one, so nothing past the array is read.
template <int Q>
__device__ __forceinline__ void load_ids(const int32_t* ptr, int64_t len, int64_t base, int lane,
                                         int cnt, int32_t (&out)[Q]) {
  const int k0 = lane * Q;
#pragma unroll
  for (int q = 0; q < Q; ++q) out[q] = 0;
  if (k0 >= cnt) return;
  if constexpr (Q == 1) {
    out[0] = __builtin_nontemporal_load(ptr + base + k0);
  } else if (base + k0 + Q <= len) {
    const int4_a4 v = __builtin_nontemporal_load(reinterpret_cast<const int4_a4*>(ptr + base + k0));
    out[0] = v.x;
    out[1] = k0 + 1 < cnt ? v.y : 0;
    out[2] = k0 + 2 < cnt ? v.z : 0;
    out[3] = k0 + 3 < cnt ? v.w : 0;
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (k0 + q < cnt) out[q] = __builtin_nontemporal_load(ptr + base + k0 + q);
  }
}

// Value of edge (jb + gid) of the batch (jb wave-uniform, gid < NG the
// caller's lane group) when each lane holds Q consecutive edges; jb % Q is
// c0, known after unrolling.  One group reads its id into a scalar
// register; two groups take theirs through one cross-lane permute (the
// vector unit, which partly bounds the gather kernels, then only forms the
// lane index).  Several groups with four ids per lane use the LDS table below.
template <int NG, int Q>
__device__ __forceinline__ int bcast_q(const int32_t (&v)[Q], int jb, int c0, int gid) {
  if constexpr (NG == 1) {
    return __builtin_amdgcn_readlane(pick<Q>(v, c0), jb / Q);
  } else {
    static_assert(Q == 1, "four ids per lane: one group, or the LDS table for two");
    if constexpr (NG == 2) return __shfl(v[0], jb + gid);
    else return bcast_lane<NG>(v[0], jb, gid);
  }
}

// Wide batches of NG >= 2 lane groups keep their 256 ids (or weights) in a
// per-wavefront LDS table, group by group: edge k of the batch at
// (k % NG) * wide_half<NG>() + k / NG, so that group g's edges of a step
// (j0 + NG u + g, u < U) are U consecutive entries, read with U / 4 16-byte
// LDS reads instead of one cross-lane permute (and a select) per edge.  The
// 4-entry pad after each group's 256 / NG entries puts the groups' reads of
// one step in different banks.
template <int NG>
constexpr int wide_half() { return 4 * kWave / NG + 4; }
template <int NG>
constexpr int wide_tab() { return NG * wide_half<NG>(); }

// Lane l holds edges 4l .. 4l + 3 of the batch.  Two groups: 4l and 4l + 2
// go to group 0's entries 2l and 2l + 1, 4l + 1 and 4l + 3 to group 1's.
// NG = 4m groups: edge 4l + q goes to group 4 (l % m) + q, entry l / m.
template <int NG, typename T>
__device__ __forceinline__ void wide_put(T* tab, int lane, const int32_t (&q)[4]) {
  static_assert(sizeof(T) == 4, "4-byte entries");
  static_assert(NG == 2 || NG % 4 == 0, "two lane groups or a multiple of four");
  int32_t* t = reinterpret_cast<int32_t*>(tab);
  constexpr int H = wide_half<NG>();
  if constexpr (NG == 2) {
    *reinterpret_cast<int2*>(t + 2 * lane) = make_int2(q[0], q[2]);
    *reinterpret_cast<int2*>(t + H + 2 * lane) = make_int2(q[1], q[3]);
  } else {
    constexpr int M = NG / 4;
    const int g0 = 4 * (lane % M), pos = lane / M;
#pragma unroll
    for (int c = 0; c < 4; ++c) t[(g0 + c) * H + pos] = q[c];
  }
}

// Place of entry k in that table.
template <int NG>
__device__ __forceinline__ int wide_at(int k) {
  return (k % NG) * wide_half<NG>() + k / NG;
}

// Group gid's U entries of the step that starts at batch edge j0 (a multiple
// of NG U, so the reads are 16-byte aligned).
template <int NG, int U, typename T>
__device__ __forceinline__ void wide_get(const T* tab, int gid, int j0, T (&out)[U]) {
  static_assert(U % 4 == 0, "whole 16-byte reads");
  const T* t = tab + gid * wide_half<NG>() + j0 / NG;
#pragma unroll
  for (int k = 0; k < U; k += 4) {
    typedef T T4 __attribute__((ext_vector_type(4)));
    const T4 v = *reinterpret_cast<const T4*>(t + k);
    out[k] = v.x;
    out[k + 1] = v.y;
    out[k + 2] = v.z;
    out[k + 3] = v.w;
  }
}

// Runs of equal ids in a batch of `cnt` edges, lane l holding edges 4l .. 4l +
// 3: whether each edge starts a run, the number of its run, and the number of
// runs.  (A repeated edge is next to its copies in a row with sorted sources;
// unsorted rows only have fewer runs to merge.)
__device__ __forceinline__ int batch_runs(const int32_t (&id)[4], int lane, int cnt,
                                          bool (&head)[4], int (&run)[4]) {
  const int before = __builtin_amdgcn_update_dpp(0, id[3], kDppWaveShr1, 0xF, 0xF, false);
  int n = 0, total = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = 4 * lane + q;
    head[q] = k < cnt && (k == 0 || id[q] != (q ? id[q - 1] : before));
    const uint64_t m = __ballot(head[q]);
    n = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n));
    total += __popcll(m);
  }
  // n: runs that start in earlier lanes
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    n += head[q] ? 1 : 0;
    run[q] = n - 1;
  }
  return total;
}

// Sums of v over the runs of a batch, in an order that the batch alone fixes
// (lane l holding edges 4l .. 4l + 3, runs as batch_runs numbers them):
// sum[q] is the run's sum where last[q], at the run's last edge.  Each lane adds
// its own elements of a run in edge order; the parts of a run that spans lanes
// then meet in steps of 1, 2, 4, ... lanes, as many as the longest run needs.
__device__ __forceinline__ void run_sums(const float (&v)[4], const bool (&head)[4], int lane,
                                         int cnt, float (&sum)[4], bool (&last)[4]) {
  sum[0] = v[0];
#pragma unroll
  for (int q = 1; q < 4; ++q) sum[q] = head[q] ? v[q] : sum[q - 1] + v[q];
  // lanes between this one and the lane where its last run starts (lanes past
  // the batch hold zeros and count as starting one)
  const bool starts = head[0] || head[1] || head[2] || head[3] || 4 * lane >= cnt;
  const uint64_t firsts = __ballot(head[0]), m = __ballot(starts);
  const int back = __clzll((long long)(m << (63 - lane)));
  float t = sum[3];
  const float below = dpp_f<kDppWaveShr1>(t);
  if (back >= 1) t = below + t;
  for (int d = 2; d < kWave; d <<= 1) {
    if (__ballot(back >= d) == 0) break;  // wave-uniform
    const float o = __shfl_up(t, d);
    if (back >= d) t = o + t;
  }
  const float before = dpp_f<kDppWaveShr1>(t);
  bool whole = false;  // the run started in this lane
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = 4 * lane + q;
    whole = whole || head[q];
    const bool next = q < 3 ? head[(q + 1) & 3] : lane < kWave - 1 && (firsts >> (lane + 1)) & 1;
    last[q] = k < cnt && (k == cnt - 1 || next);
    if (!whole) sum[q] = before + sum[q];
  }
}

// Key by which the copies of a weighted edge merge (q: the edge's place in its
// lane's four).  w1 x + w2 x is (w1 + w2) x for every x, infinities and NaN
// too, if the weights have one sign and their sum is finite: keys carry the
// sign, and weights of 0, of 2^120 or more (256 copies add up below 2^128),
// infinite or NaN get one that differs from both neighbours', so they stand
// alone.  (Ids stay below the two keys of those: 2^31 - 1 rows of the 32 floats
// or more that these kernels take do not fit the memory.)
__device__ __forceinline__ int32_t weighted_key(int32_t id, int32_t w_bits, int q) {
  const uint32_t mag = (uint32_t)w_bits & 0x7fffffffu;
  const uint32_t sign = (uint32_t)w_bits & 0x80000000u;
  if (mag - 1u < 0x7b800000u - 1u) return (int32_t)((uint32_t)id | sign);
  return (q & 1) ? -1 : 0x7fffffff;
}

// Largest head count whose per-batch edge values a wavefront stages in LDS.
constexpr int kTabHeads = 16;

// Orders one wavefront's LDS accesses around a cross-lane hand-off (the
// hardware executes a wavefront's LDS operations in order; the fences keep
// the compiler from moving accesses across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct Item {
  int64_t row, b, e;
  int32_t slot;
};

template <bool SEG>
__device__ __forceinline__ Item load_item(const Seg* segs, const int32_t* indptr, int64_t item) {
  Item it;
  if constexpr (SEG) {
    const Seg s = segs[item];
    it.row = s.row; it.b = s.begin; it.e = s.end; it.slot = s.slot;
  } else {
    it.row = item; it.b = indptr[item]; it.e = indptr[item + 1]; it.slot = -1;
  }
  return it;
}

// For launches that take a plan's cut rows whole: the first piece becomes the
// row, the others (false) have nothing to do.
__device__ __forceinline__ bool take_whole_row(Item& it, const int32_t* indptr) {
  if (it.slot < 0) return true;
  if (it.b != indptr[it.row]) return false;
  it.e = indptr[it.row + 1];
  it.slot = -1;
  return true;
}

inline int ilog2_ceil(int64_t q) {
  int l = 0;
  while ((int64_t(1) << l) < q) ++l;
  return l;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline dim3 grid_for(int64_t items, int64_t chunks) {
  return dim3((unsigned)((items + kWavesPerBlock - 1) / kWavesPerBlock), (unsigned)chunks, 1);
}

#define FG_LAUNCH(kernel, grid, stream, ...) \
  hipLaunchKernelGGL((kernel), (grid), dim3(kBlock), 0, (stream), __VA_ARGS__)

}  // namespace
}  // namespace fg
