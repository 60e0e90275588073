// fg_sddmm.h -- generalized SDDMM kernels with float4 lanes and their dispatch
// over lane layouts, instantiated by the kernel translation units.
#pragma once

#include "fg_device.h"

namespace fg {

struct SddmmParams {
  const int32_t* indptr;
  const int32_t* indices;
  const int32_t* eids;
  const float* xs;
  const float* xd;
  float* out;
  const Seg* segs;
  int64_t n_items;
  int64_t nnz;  // stored edges: elements of indices and eids
  int64_t F;
  int32_t H;
  int32_t dh;
  int32_t logG;  // lanes per feature row (runtime kernels)
  int32_t logS;  // lanes per head (scalar kernel)
  int32_t out_vec4;  // output rows of H values are 16-byte aligned float4s
  int32_t repeats;  // the graph repeats many edges (DUP kernels)
  int32_t heads_per_pass;  // heads per blockIdx.y (headed kernel)
};

// One translation unit each (they build in parallel): single-head SDDMM for
// 16-byte aligned rows and for any others of 4 to 1024 floats (ragged).  avg:
// the items' average edge count.
void sddmm_aligned(const SddmmParams& prm, bool seg, int64_t avg, hipStream_t st);
void sddmm_ragged(const SddmmParams& prm, bool seg, int64_t avg, hipStream_t st);
// The same for several heads of 4 to 256 features each.
void sddmm_headed_aligned(const SddmmParams& prm, bool seg, hipStream_t st);
void sddmm_headed_ragged(const SddmmParams& prm, bool seg, hipStream_t st);

namespace {


// Single head, float4 lanes, G lanes per feature row, NV float4 per lane.  The
// destination row stays in registers for the whole item; each edge gathers
// its source row, multiplies, and reduces across its G lanes with DPP.
// RAG: rows of any width F >= 4 and any 4-byte alignment.  The last lane of a
// row takes the row's last four floats; where F is no multiple of 4 the first
// lo of them are its neighbour's and count as 0 in both factors (an infinity
// there must not turn into a NaN).
// DUP (wide batches of several groups): a run of equal sources in a batch, the
// copies of a repeated edge, is gathered once; each of its edges reads the
// run's result (power-law graph, d = 128: 2115 -> 1863 us).
template <int G, int NV, int U, bool SEG, bool WIDE = false, bool RAG = false, bool DUP = false>
__global__ __launch_bounds__(kBlock) void sddmm_fast_kernel(SddmmParams p) {
  constexpr int NG = kWave / G;
  static_assert(NG * U <= kWave, "one batch of 64 edges must cover whole steps");
  constexpr int QB = WIDE ? ids_per_lane<NG, U>() : 1;
  // one or two groups, and wide batches, hand each edge's dot product over
  // through this per-wavefront table (the group's last lane writes it; each
  // lane reads its QB results after the batch) instead of readlanes and
  // selects, or a cross-lane permute per step
  constexpr bool RTAB = NG <= 2 || WIDE;
  __shared__ __align__(16) float res_all[RTAB ? kWavesPerBlock * kWave * QB : 1];
  float* res_tab = res_all + (RTAB ? (threadIdx.x >> 6) * kWave * QB : 0);
  // wide batches of several groups take their ids from the group-major table
  constexpr bool IDTAB = WIDE && NG >= 2;
  constexpr int WT = IDTAB ? wide_tab<NG>() : 1;
  __shared__ __align__(16) int32_t sid_all[IDTAB ? kWavesPerBlock * WT : 1];
  int32_t* sid = sid_all + (IDTAB ? (threadIdx.x >> 6) * WT : 0);
  const int64_t item = wave_item();
  if (item >= p.n_items) return;
  const Item it = load_item<SEG>(p.segs, p.indptr, item);
  if (it.row < 0) return;  // padding item of a partitioned schedule
  if (it.b >= it.e) return;
  const int lane = lane_id();
  const int gid = lane / G;
  const int li = lane % G;
  const int64_t F = p.F;

  int64_t f[NV];
  bool act[NV];
  int lo[NV];  // elements of the lane that its neighbour holds (ragged tail, else 0)
  float xd[NV][4];
  const char* xl[NV];  // this lane's elements of source row 0
  const uint32_t rb = (uint32_t)F * 4u;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    f[v] = (int64_t)(v * G + li) * 4;
    act[v] = f[v] < F;
    lo[v] = 0;
    if constexpr (RAG) {
      lo[v] = act[v] ? (int)max((int64_t)0, f[v] + 4 - F) : 0;
      f[v] -= lo[v];
    }
    xl[v] = reinterpret_cast<const char*>(p.xs) + f[v] * 4;
    if (act[v]) {
      load4<RAG>(p.xd + it.row * F + f[v], xd[v]);
      if constexpr (RAG) {
#pragma unroll
        for (int c = 0; c < 3; ++c) xd[v][c] = c < lo[v] ? 0.0f : xd[v][c];
      }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) xd[v][c] = 0.0f;
    }
  }

  const bool all_feat = (int64_t)G * 4 * NV <= F;
  constexpr int Q = WIDE ? ids_per_lane<NG, U>() : 1;
  static_assert((NG * U) % Q == 0, "every step starts on a lane's first edge");
  for (int64_t base = it.b; base < it.e; base += Q * kWave) {
    const int cnt = (int)min((int64_t)(Q * kWave), it.e - base);
    int rows = cnt;  // source rows to gather
    int32_t my_src[Q], my_eid[Q];
    int run[Q];
    load_ids<Q>(p.indices, p.nnz, base, lane, cnt, my_src);
    if constexpr (DUP) {
      bool head[4];
      rows = batch_runs(my_src, lane, cnt, head, run);
      wave_lds_sync();  // the previous batch's table reads are done
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (head[q]) sid[wide_at<NG>(run[q])] = my_src[q];
      wave_lds_sync();
    } else if constexpr (IDTAB) {
      wave_lds_sync();  // the previous batch's table reads are done
      wide_put<NG>(sid, lane, my_src);
      wave_lds_sync();
    }
    if (p.eids) {
      load_ids<Q>(p.eids, p.nnz, base, lane, cnt, my_eid);
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) my_eid[q] = (int)(base + lane * Q + q);
    }
    // lane j collects the dot products of edges base + Q*j + q, so the batch's
    // results leave in one store instead of one store per step with one lane
    // per group active, which would cost the address unit as much as a
    // gather: one or two groups, and wide batches, hand their sums over
    // through the LDS table, more groups with one cross-lane permute per step
    float res[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) res[q] = 0.0f;
    // one step of U edges per lane group; FULL: every edge of the step is in
    // the batch and every feature chunk in the row (no per-edge masking)
    auto step = [&](int j0, auto full_tag) {
      constexpr bool FULL = decltype(full_tag)::value;
      float val[U][NV][4];
      bool ok[U];
      int32_t tsrc[IDTAB ? U : 1];
      if constexpr (IDTAB) wide_get<NG, U>(sid, gid, j0, tsrc);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int jb = j0 + u * NG;
        ok[u] = FULL || jb + gid < rows;
        int src;
        if constexpr (IDTAB) src = tsrc[u];
        else src = bcast_q<NG, Q>(my_src, jb, (u * NG) % Q, gid);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if (FULL || (ok[u] && act[v])) {
            load4<RAG>(row_at(xl[v], src, rb), val[u][v]);
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) val[u][v][c] = 0.0f;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float part = 0.0f;
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float t = (RAG && c < lo[v]) ? 0.0f : val[u][v][c];
            part += t * xd[v][c];
          }
        part = group_sum<G>(part);
        const int jb = j0 + u * NG;
        // the last lane of group g holds the sum of edge jb + g
        if constexpr (RTAB) {
          if (li == G - 1 && (FULL || jb + gid < rows)) res_tab[jb + gid] = part;
        } else {
          const int rel = lane - jb;
          const bool mine = rel >= 0 && rel < NG && lane < cnt;
          const float got = __shfl(part, mine ? rel * G + (G - 1) : lane);
          if (mine) res[0] = got;  // Q == 1 without the table
        }
      }
    };
    // full steps (wave-uniform test) take the unmasked body
    int j0 = 0;
    if (all_feat)
      for (; j0 + NG * U <= rows; j0 += NG * U) step(j0, BoolTag<true>{});
    for (; j0 < rows; j0 += NG * U) step(j0, BoolTag<false>{});
    if constexpr (RTAB) {
      wave_lds_sync();  // the table holds the batch's results
      if constexpr (DUP) {
#pragma unroll
        for (int q = 0; q < 4; ++q) res[q] = res_tab[max(run[q], 0)];
      } else if constexpr (Q == 4) {
        const float4 t = *reinterpret_cast<const float4*>(res_tab + lane * Q);
        res[0] = t.x;
        res[1] = t.y;
        res[2] = t.z;
        res[3] = t.w;
      } else {
        res[0] = res_tab[lane];
      }
      wave_lds_sync();  // read before the next batch writes
    }
    bool stored = false;
    if constexpr (Q == 4) {
      if (!p.eids && lane * Q + Q <= cnt) {  // four positional results: one 16-byte store
        __builtin_nontemporal_store(float4_a4{res[0], res[1], res[2], res[3]},
                                    reinterpret_cast<float4_a4*>(p.out + base + lane * Q));
        stored = true;
      }
    }
    if (!stored) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (lane * Q + q < cnt) __builtin_nontemporal_store(res[q], p.out + my_eid[q]);
    }
  }
}

// Several heads of at least 4 features, float4 lanes, S (a power of two) lanes
// per head: the first (dh + 3) / 4 of them hold its features, the last of those
// the head's last four (RAG: where dh is no multiple of 4 the first lo of these
// are its neighbour's and count as 0; also for rows off 16-byte boundaries).
// Heads that are no power of two of lanes leave some idle, which costs less
// than one lane per value: 400K power-law edges, 8 heads of 8: 425 -> 69 us.
// blockIdx.y: chunk of up to kTabHeads heads; G = 2^logG lanes per chunk of a
// feature row.  Results of a batch are staged per edge in an LDS table (one
// row of hc values per edge) and leave in one pass of per-lane stores.
template <int S, bool SEG, bool RAG>
__global__ __launch_bounds__(kBlock) void sddmm_headed_kernel(SddmmParams p) {
  constexpr int U = 4;
  __shared__ __align__(16) float tab_all[kWavesPerBlock * kWave * kTabHeads];
  float* tab = tab_all + (threadIdx.x >> 6) * kWave * kTabHeads;
  const int64_t item = wave_item();
  if (item >= p.n_items) return;
  const Item it = load_item<SEG>(p.segs, p.indptr, item);
  if (it.row < 0) return;  // padding item of a partitioned schedule
  if (it.b >= it.e) return;
  const int lane = lane_id();
  const int h0 = (int)blockIdx.y * p.heads_per_pass;
  const int hc = min(p.heads_per_pass, p.H - h0);  // heads of this chunk
  const int lpe = (p.out_vec4 && (hc == 4 || hc == 8 || hc == 16)) ? hc >> 2 : 0;
  const int lpe_part = lpe ? lane % lpe : 0;
  const int lpe_sub = lpe ? lane / lpe : 0;
  const int G = 1 << p.logG;
  const int ngroups = kWave >> p.logG;
  const int gid = lane >> p.logG;
  const int li = lane & (G - 1);
  const int64_t F = p.F;
  const int hl = li / S, j4 = li % S * 4;
  const bool act = hl < hc && j4 < p.dh;
  const int lo = RAG && act ? max(0, j4 + 4 - p.dh) : 0;
  const int64_t f = act ? (int64_t)(h0 + hl) * p.dh + j4 - lo : 0;
  float xd[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (act) {
    load4<RAG>(p.xd + it.row * F + f, xd);
    if constexpr (RAG) {
#pragma unroll
      for (int c = 0; c < 3; ++c) xd[c] = c < lo ? 0.0f : xd[c];
    }
  }
  const char* xl = reinterpret_cast<const char*>(p.xs) + f * 4;  // lane's elements of row 0
  const uint32_t rb = (uint32_t)F * 4u;

  for (int64_t base = it.b; base < it.e; base += kWave) {
    const int cnt = (int)min((int64_t)kWave, it.e - base);
    int my_src = 0, my_eid = 0;
    if (lane < cnt) {
      my_src = __builtin_nontemporal_load(p.indices + base + lane);
      my_eid = p.eids ? __builtin_nontemporal_load(p.eids + base + lane) : (int)(base + lane);
    }
    for (int j0 = 0; j0 < cnt; j0 += ngroups * U) {
      float val[U][4];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * ngroups + gid;
        ok[u] = j < cnt;
        const int src = __shfl(my_src, j & (kWave - 1));
        if (ok[u] && act) {
          load4<RAG>(row_at(xl, src, rb), val[u]);
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) val[u][c] = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float part = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float t = (RAG && c < lo) ? 0.0f : val[u][c];
          part += t * xd[c];
        }
        part = group_sum<S>(part);
        if (ok[u] && hl < hc && (li % S) == S - 1) tab[(j0 + u * ngroups + gid) * hc + hl] = part;
      }
    }
    wave_lds_sync();
    if (lpe) {
      // lpe = hc / 4 lanes share an edge (one float4 each), so that a store
      // instruction writes 64 / lpe whole edge rows
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < lpe) {
          const int k = i * (kWave / lpe) + lpe_sub;
          const int ek = __shfl(my_eid, k);
          if (k < cnt) {
            float q[4];
            load_vec<4>(tab + k * hc + lpe_part * 4, q);
            store_vec<4>(p.out + (int64_t)ek * p.H + h0 + lpe_part * 4, q);
          }
        }
    } else if (lane < cnt) {
      const float* tr = tab + lane * hc;
      float* orow = p.out + (int64_t)my_eid * p.H + h0;
      for (int hh = 0; hh < hc; ++hh) orow[hh] = tr[hh];
    }
    wave_lds_sync();  // the table is rewritten by the next batch
  }
}

// avg: the items' average edge count (batches of four ids per lane where the
// lane layout allows it and the items are long enough, wide_item_edges)
template <int G, int NV, int U, bool RAG>
void sddmm_fast_go(const SddmmParams& prm, bool seg, int64_t avg, hipStream_t st) {
  const dim3 grid = grid_for(prm.n_items, 1);
  if constexpr (ids_per_lane<kWave / G, U>() > 1) {
    if (avg >= wide_item_edges<kWave / G>()) {
      if constexpr (!RAG && NV == 1 && G < kWave) {
        if (seg && prm.repeats) {
          FG_LAUNCH((sddmm_fast_kernel<G, NV, U, true, true, RAG, true>), grid, st, prm);
          return;
        }
      }
      if (seg) FG_LAUNCH((sddmm_fast_kernel<G, NV, U, true, true, RAG>), grid, st, prm);
      else FG_LAUNCH((sddmm_fast_kernel<G, NV, U, false, true, RAG>), grid, st, prm);
      return;
    }
  }
  if (seg) FG_LAUNCH((sddmm_fast_kernel<G, NV, U, true, false, RAG>), grid, st, prm);
  else FG_LAUNCH((sddmm_fast_kernel<G, NV, U, false, false, RAG>), grid, st, prm);
}

// Launches the kernel of the narrowest layout that covers rows of F <= 1024 floats.
template <bool RAG>
void sddmm_fast_dispatch(const SddmmParams& prm, bool seg, int64_t avg, hipStream_t st) {
  const int64_t Q = (prm.F + 3) / 4;
  if (Q <= 4) sddmm_fast_go<4, 1, 4, RAG>(prm, seg, avg, st);
  else if (Q <= 8) sddmm_fast_go<8, 1, 8, RAG>(prm, seg, avg, st);
  else if (Q <= 16) sddmm_fast_go<16, 1, 8, RAG>(prm, seg, avg, st);
  else if (Q <= 32) sddmm_fast_go<32, 1, 8, RAG>(prm, seg, avg, st);
  else if (Q <= 64) sddmm_fast_go<64, 1, 8, RAG>(prm, seg, avg, st);
  else if (Q <= 128) sddmm_fast_go<64, 2, 4, RAG>(prm, seg, avg, st);
  // (10M power-law edges of 520 floats: 1324 -> 1254 us; 32 x 3 for 257-384
  // floats gains 9% there but doubles the time of short items)
  else if (Q <= 192) sddmm_fast_go<64, 3, 2, RAG>(prm, seg, avg, st);
  else sddmm_fast_go<64, 4, 2, RAG>(prm, seg, avg, st);
}

template <int S, bool RAG>
void sddmm_headed_go(SddmmParams prm, bool seg, hipStream_t st) {
  prm.heads_per_pass = std::min<int32_t>(std::min(kWave / S, kTabHeads), prm.H);
  if (!prm.out_vec4) {  // equal passes (33 heads: 11 each, not 16, 16 and 1)
    const int32_t passes = (prm.H + prm.heads_per_pass - 1) / prm.heads_per_pass;
    prm.heads_per_pass = (prm.H + passes - 1) / passes;
  }
  prm.logG = ilog2_ceil((int64_t)prm.heads_per_pass * S);
  const dim3 grid =
      grid_for(prm.n_items, (prm.H + prm.heads_per_pass - 1) / prm.heads_per_pass);
  if (seg) FG_LAUNCH((sddmm_headed_kernel<S, true, RAG>), grid, st, prm);
  else FG_LAUNCH((sddmm_headed_kernel<S, false, RAG>), grid, st, prm);
}

// Heads of 4 to 256 features.
template <bool RAG>
void sddmm_headed_dispatch(const SddmmParams& prm, bool seg, hipStream_t st) {
  const int64_t n4 = (prm.dh + 3) / 4;
  if (n4 <= 1) sddmm_headed_go<1, RAG>(prm, seg, st);
  else if (n4 <= 2) sddmm_headed_go<2, RAG>(prm, seg, st);
  else if (n4 <= 4) sddmm_headed_go<4, RAG>(prm, seg, st);
  else if (n4 <= 8) sddmm_headed_go<8, RAG>(prm, seg, st);
  else if (n4 <= 16) sddmm_headed_go<16, RAG>(prm, seg, st);
  else if (n4 <= 32) sddmm_headed_go<32, RAG>(prm, seg, st);
  else sddmm_headed_go<64, RAG>(prm, seg, st);
}

}  // namespace
}  // namespace fg
