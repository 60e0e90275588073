// fg_spmm.h -- generalized SpMM kernels with float4 lanes and their dispatch
// over lane layouts, instantiated by the kernel translation units.
#pragma once

#include "fg_device.h"

namespace fg {

struct SpmmParams {
  const int32_t* indptr;
  const int32_t* indices;
  const int32_t* eids;
  const float* x;
  const float* ev;
  const float* xd;  // destination features of the u_add_v message (ADD kernels only)
  float* out;
  int32_t* arg;
  const Seg* segs;
  float* ws_f;
  int32_t* ws_i;
  int64_t n_items;
  int64_t nnz;      // length of indices (and of ev with one head and positional ids)
  int64_t F;
  int32_t H;
  int32_t dh;
  int32_t logG;     // runtime group width (generic kernel only)
  int32_t repeats;  // the graph repeats many edges (DUP kernels)
  int32_t ev_vec4;  // edge-value rows are 16-byte aligned float4s (H % 4 == 0)
};

// One translation unit each (they build in parallel): the float4 kernels of
// the sum and the max reducer, for 16-byte aligned rows and for any others of
// at least 4 floats (ragged).
// avg: the items' average edge count.
void spmm_sum(const SpmmParams& prm, bool mul, bool seg, int64_t avg, hipStream_t st);
void spmm_max(const SpmmParams& prm, bool mul, bool seg, int64_t avg, hipStream_t st);
void spmm_sum_ragged(const SpmmParams& prm, bool mul, bool seg, int64_t avg, hipStream_t st);
void spmm_max_ragged(const SpmmParams& prm, bool mul, bool seg, int64_t avg, hipStream_t st);

namespace {


// Epilogues of the u_add_v max (MLP aggregation).  Its edges are compared by
// their transformed source value P_src[u] (raw: before adding P_dst[v]); fp32
// rounding of a sum is monotone in each operand, so the edge with the largest
// raw value also has the largest rounded message relu(P_src[u] + P_dst[v]),
// and the row's output is relu(acc + xd[v]).  When that is not positive every
// message is 0 and the row's smallest edge id is reported.
//  kEpiFirst  (positional edge ids): acc / am are the max and smallest argmax
//             of the raw values; the smallest id of the row is its first
//             position.
//  kEpiMasked (any edge ids): edges whose rounded sum is not positive compete
//             as -inf, so am already is the smallest id of the row when
//             nothing is positive.
constexpr int kOneHead = 0, kHeadTable = 1, kManyHeads = 2;  // HM below
constexpr int kEpiNone = 0, kEpiFirst = 1, kEpiMasked = 2;

// Writes one lane's accumulated vector: to the plan workspace for a split
// row's segment, else to the output (max: empty -> 0 / -1; EPI: see above).
// RAG: rows of any width and alignment; lo: the lane's first element to store
// (its tail elements only, where the previous lane holds the others).
template <int VEC, bool MAX, bool SEG, int EPI = kEpiNone, bool RAG = false>
__device__ __forceinline__ void spmm_store(const SpmmParams& p, const Item& it, int64_t f,
                                           const float (&acc)[VEC], const int32_t (&am)[VEC],
                                           int lo = 0) {
  auto put = [&](float* q, const float (&r)[VEC]) {
    if constexpr (VEC == 4) store4_nt<RAG>(q, r, lo);
    else store_vec_nt<VEC>(q, r);
  };
  auto put_i = [&](int32_t* q, const int32_t (&r)[VEC]) {
    if constexpr (VEC == 4) store4_i_nt<RAG>(q, r, lo);
    else store_vec_i_nt<VEC>(q, r);
  };
  if (SEG && it.slot >= 0) {
    put(p.ws_f + (int64_t)it.slot * p.F + f, acc);
    if constexpr (MAX) put_i(p.ws_i + (int64_t)it.slot * p.F + f, am);
  } else if constexpr (MAX) {
    float o[VEC];
    int32_t a[VEC];
    float pdv[VEC];
    if constexpr (EPI != kEpiNone) {
      if constexpr (VEC == 4) load4<RAG>(p.xd + it.row * p.F + f, pdv);
      else load_vec<VEC>(p.xd + it.row * p.F + f, pdv);
    }
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
      const bool none = am[c] == INT_MAX;
      if constexpr (EPI != kEpiNone) {
        const float t = acc[c] + pdv[c];
        const bool pos = t > 0.0f;
        o[c] = (none || !pos) ? 0.0f : t;
        a[c] = none ? -1 : ((pos || EPI == kEpiMasked) ? am[c] : (int32_t)it.b);
      } else {
        o[c] = none ? 0.0f : acc[c];
        a[c] = none ? -1 : am[c];
      }
    }
    put(p.out + it.row * p.F + f, o);
    put_i(p.arg + it.row * p.F + f, a);
  } else {
    put(p.out + it.row * p.F + f, acc);
  }
}

// Fast path: float4 lanes, G (compile time) lanes per feature row, NV float4
// per lane per edge (feature chunk G*4*NV = blockIdx.y), U edges in flight per
// lane group, MUL: src_mul_edge, MAX: max/argmax, EIDS: the graph carries an
// edge-id array (else edge id = position), SEG: items from a plan.
//
// Max with positional edge ids: a lane group visits its edges in increasing
// position, hence increasing edge id, so "strictly greater replaces" keeps the
// smallest edge id among equal maxima; a group whose messages were all -inf
// never replaces and takes its first edge afterwards.  Groups, segments and
// slots are then merged with the full (value, edge id) order.
// ADD: the message is relu(x[u] + xd[v]) (MLP aggregation with the dense
// transform applied to the vertices beforehand); requires MAX and !MUL.  Edges
// compete by their raw x[u] (see the epilogues above spmm_store).  With
// positional edge ids the add and relu move to the store (kEpiFirst); with
// explicit edge ids each edge's sum is formed in the loop to mask the edges
// whose message is 0 (kEpiMasked).
// HM (how edge values are weighted in): kOneHead; kHeadTable (2 <= H <=
// kTabHeads); kManyHeads (more heads: a load per edge, element and step).  One
// kernel each: compiled together, the third's per-element weights cost the
// first its occupancy (weighted sum of 602 floats, 10M power-law edges: 2.3 ->
// 1.6 ms).
// kHeadTable: each batch of 64 edges
// stages its edge values in an LDS table, a few loads per lane, and every step
// reads its weights from there; loading them per step would add one more
// vector-memory instruction per gather, and the address unit is what bounds
// these kernels.
//
// RAG: rows of any width F >= 4 and any 4-byte alignment.  The last lane of a
// row takes the row's last four floats: where F is no multiple of 4 it repeats
// up to three of its neighbour's and stores only its own.  A gather costs what
// its 128-byte lines cost (a row of 41 floats at any offset touches 2.25), and
// scalar lanes, with four times the instructions, did not keep up with them:
// 10M uniform edges of 41 floats, weighted sum 550 -> 293 us, SDDMM 890 -> 293.
// Heads may straddle a lane, so each element then has its own weight.
//
// WIDE (two or more lane groups, positional ids, one head): 256-edge batches
// whose ids (and weights) arrive four per lane in one 16-byte load (a quarter
// of the id loads for the address unit) and go to the group-major LDS table.
// Without weights, one float4 a lane is held to 7 wavefronts per SIMD (72
// registers): the max kernel otherwise takes 85 (5 wavefronts), without a spill
// either way, and the DUP forms spill 1 to 3 registers.  The copy sums of 64-edge
// batches fit 64 registers (8 wavefronts), where the compiler left alone takes 70
// for a plan's items (400K edges in rows of 4, 64 floats: 30.7 -> 28.7 us).
//
// DUP (wide batches): graphs that repeat many edges.  Copies of an edge are
// neighbours in a row, so each batch is packed to one entry per run of equal
// sources before its gathers: their weights (1 for copies) are added in a fixed
// order (run_sums), and the max keeps a run's first edge.  On the power-law graph, where 32% of
// the edges repeat another, the address unit then serves as many fewer
// gathers: weighted sum 2224 -> 2002 us, max 2202 -> 1997.
template <int G, int NV, int U, bool MUL, bool MAX, bool EIDS, bool SEG, bool ADD, int HM,
          bool WIDE, bool RAG, bool DUP = false>
__global__ __launch_bounds__(kBlock, (MUL || NV > 1) ? 1 : WIDE ? 7 : MAX ? 1 : 8) void spmm_fast_kernel(SpmmParams p) {
  constexpr int NG = kWave / G;
  constexpr bool POS = MAX && !EIDS;
  constexpr bool TAB = MUL && HM == kHeadTable;
  static_assert(NG * U <= kWave, "one batch of 64 edges must cover whole steps");
  static_assert(!WIDE || (NG >= 2 && U % 4 == 0 && !EIDS && !TAB),
                "wide batches serve several lane groups with positional ids");
  constexpr int BATCH = WIDE ? 4 * kWave : kWave;
  constexpr int WT = WIDE ? wide_tab<NG>() : 1;
  __shared__ __align__(16) int32_t wid_all[WIDE ? kWavesPerBlock * WT : 1];
  // DUP copies weigh as much as their run is long
  constexpr bool WGT = MUL || (DUP && !MAX);
  __shared__ __align__(16) float wwt_all[WIDE && WGT ? kWavesPerBlock * WT : 1];
  static_assert(!DUP || (WIDE && !RAG && HM == kOneHead), "runs are packed in wide batches");
  __shared__ __align__(16) int32_t wk_all[DUP && MAX ? kWavesPerBlock * WT : 1];
  int32_t* wk = wk_all + (DUP && MAX ? (threadIdx.x >> 6) * WT : 0);  // first edge of each run
  int32_t* wid = wid_all + (WIDE ? (threadIdx.x >> 6) * WT : 0);
  float* wwt = wwt_all + (WIDE && WGT ? (threadIdx.x >> 6) * WT : 0);
  static_assert(!ADD || (MAX && !MUL), "u_add_v messages are max-reduced copies");
  static_assert(MUL || HM == kOneHead, "heads matter to edge values only");
  constexpr bool EPI = ADD && POS;
  constexpr bool ELEM = ADD && !POS;
  constexpr int EPK = EPI ? kEpiFirst : (ELEM ? kEpiMasked : kEpiNone);
  __shared__ __align__(16) float tab_all[TAB ? kWavesPerBlock * kWave * kTabHeads : 1];
  float* tab = tab_all + (TAB ? (threadIdx.x >> 6) * kWave * kTabHeads : 0);
  const int64_t item = wave_item();
  if (item >= p.n_items) return;
  const Item it = load_item<SEG>(p.segs, p.indptr, item);
  if (it.row < 0) return;  // padding item of a partitioned schedule
  const int lane = lane_id();
  const int gid = lane / G;
  const int li = lane % G;
  const int64_t F = p.F;
  const int64_t c0 = (int64_t)blockIdx.y * (G * 4 * NV);

  constexpr int WC = (RAG && HM != kOneHead) ? 4 : 1;  // heads may straddle a lane
  int64_t f[NV];
  bool act[NV];
  int lo[NV];  // first element this lane stores (ragged tail, else 0)
  int hv[NV][WC];
  const char* xl[NV];  // this lane's elements of source row 0
  const uint32_t rb = (uint32_t)F * 4u;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    f[v] = c0 + (int64_t)(v * G + li) * 4;
    act[v] = f[v] < F;
    lo[v] = 0;
    if constexpr (RAG) {
      lo[v] = act[v] ? (int)max((int64_t)0, f[v] + 4 - F) : 0;
      f[v] -= lo[v];
    }
#pragma unroll
    for (int c = 0; c < WC; ++c) hv[v][c] = (MUL && act[v]) ? (int)((f[v] + c) / p.dh) : 0;
    xl[v] = reinterpret_cast<const char*>(p.x) + f[v] * 4;
  }
  float acc[NV][4];
  int32_t am[NV][4];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[v][c] = MAX ? -INFINITY : 0.0f;
      am[v][c] = INT_MAX;
    }
  float pd[NV][4];  // this row's destination features (per-element messages)
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if (ELEM && act[v]) {
      load4<RAG>(p.xd + it.row * F + f[v], pd[v]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) pd[v][c] = 0.0f;
    }
  }

  // TAB with edge ids: the edge values of batch k+1 are fetched into
  // registers while batch k computes (ids two batches ahead)
  constexpr bool PIPE = TAB && EIDS;
  float qn[PIPE ? kTabHeads : 1];
  int eid_n1 = 0, eid_n2 = 0;  // edge ids of the next batch and the one after
  // The table's loads: with 4, 8 or 16 heads (16-byte aligned rows) lpe =
  // H / 4 lanes share an edge, one float4 each, so that an instruction reads
  // 64 / lpe whole edge rows (one 64-byte cache tag each for 8 heads) rather
  // than one float4 of 64 different edges; load i of a lane holds part
  // lane % lpe of edge i * 64 / lpe + lane / lpe.
  const int lpe = (TAB && p.ev_vec4 && (p.H == 4 || p.H == 8 || p.H == 16)) ? p.H >> 2 : 0;
  const int lpe_part = lpe ? lane % lpe : 0;
  const int lpe_sub = lpe ? lane / lpe : 0;
  auto fetch_ids = [&](int64_t b0, int& e) {
    e = 0;
    const int c = (int)min((int64_t)kWave, it.e - b0);
    if (b0 < it.e && lane < c) e = __builtin_nontemporal_load(p.eids + b0 + lane);
  };
  auto fetch_vals = [&](int64_t b0, int e) {
    const int c = (int)min((int64_t)kWave, it.e - b0);
    if (lpe) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < lpe) {
          const int k = i * (kWave / lpe) + lpe_sub;
          const int ek = __shfl(e, k);
          if (b0 < it.e && k < c) {
            float q4[4];
            load_vec<4>(p.ev + (int64_t)ek * p.H + lpe_part * 4, q4);
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) qn[4 * i + c4] = q4[c4];
          }
        }
      return;
    }
    if (b0 < it.e && lane < c) {
      const float* er = p.ev + (int64_t)e * p.H;
#pragma unroll
      for (int h = 0; h < kTabHeads; h += 4)
        if (h < p.H) {
          if (p.ev_vec4) {
            float q4[4];
            load_vec<4>(er + h, q4);
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) qn[h + c4] = q4[c4];
          } else {
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4)
              if (h + c4 < p.H) qn[h + c4] = er[h + c4];
          }
        }
    }
  };
  if constexpr (PIPE) {
    fetch_ids(it.b, eid_n1);
    fetch_vals(it.b, eid_n1);
    fetch_ids(it.b + kWave, eid_n2);
  }
  for (int64_t base = it.b; base < it.e; base += BATCH) {
    int cnt = (int)min((int64_t)BATCH, it.e - base);
    int my_src = 0, my_eid = 0;
    float my_w = 0.0f;
    if constexpr (WIDE) {
      int32_t qs[4], qw[4];
      load_ids<4>(p.indices, p.nnz, base, lane, cnt, qs);
      if constexpr (MUL)  // the weights' bits (0.0f past the batch)
        load_ids<4>(reinterpret_cast<const int32_t*>(p.ev), p.nnz, base, lane, cnt, qw);
      if constexpr (DUP) {
        bool head[4];
        int run[4];
        const int edges = cnt;
        if constexpr (MUL) {
          int32_t key[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) key[q] = weighted_key(qs[q], qw[q], q);
          cnt = batch_runs(key, lane, edges, head, run);
        } else {
          cnt = batch_runs(qs, lane, edges, head, run);
        }
        float w4[4], sum[4];
        bool last[4];
        if constexpr (WGT) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if constexpr (MUL) w4[q] = __builtin_bit_cast(float, qw[q]);
            else w4[q] = 4 * lane + q < edges ? 1.0f : 0.0f;
          }
          run_sums(w4, head, lane, edges, sum, last);
        }
        wave_lds_sync();  // the previous batch's table reads are done
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int at = wide_at<NG>(run[q]);
          if (head[q]) {
            wid[at] = qs[q];
            if constexpr (MAX) wk[at] = 4 * lane + q;
          }
          if constexpr (WGT) {
            if (last[q]) wwt[at] = sum[q];
          }
        }
      } else {
        wave_lds_sync();  // the previous batch's table reads are done
        wide_put<NG>(wid, lane, qs);
        if constexpr (MUL) wide_put<NG>(wwt, lane, qw);
      }
      wave_lds_sync();
    } else if (lane < cnt) {
      my_src = __builtin_nontemporal_load(p.indices + base + lane);
      if constexpr (PIPE) my_eid = eid_n1;
      else if constexpr (EIDS) my_eid = __builtin_nontemporal_load(p.eids + base + lane);
      else my_eid = (int)(base + lane);
      if constexpr (MUL) {
        if constexpr (HM == kOneHead) my_w = p.ev[my_eid];
      }
    }
    if constexpr (PIPE) {
      wave_lds_sync();
      if (lpe) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < lpe) {
            const int k = i * (kWave / lpe) + lpe_sub;
            if (k < cnt) {
              const float q4[4] = {qn[4 * i], qn[4 * i + 1], qn[4 * i + 2], qn[4 * i + 3]};
              store_vec<4>(tab + k * p.H + lpe_part * 4, q4);
            }
          }
      } else if (lane < cnt) {
        float* tr = tab + lane * p.H;
#pragma unroll
        for (int h = 0; h < kTabHeads; ++h)
          if (h < p.H) tr[h] = qn[h];
      }
      wave_lds_sync();
      eid_n1 = eid_n2;
      fetch_vals(base + kWave, eid_n1);       // next batch's values, in flight during this one
      fetch_ids(base + 2 * kWave, eid_n2);
    } else if constexpr (TAB) {
      wave_lds_sync();  // the previous batch's table reads are done
      if (lpe) {  // positional edge ids (explicit ones take the PIPE path)
        float q4[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = i * (kWave / lpe) + lpe_sub;
          if (i < lpe && k < cnt) {  // streamed once: keep the gathered rows in the L2s
            const f32x4 t4 = __builtin_nontemporal_load(
                reinterpret_cast<const f32x4*>(p.ev + (base + k) * p.H + lpe_part * 4));
            q4[i][0] = t4.x; q4[i][1] = t4.y; q4[i][2] = t4.z; q4[i][3] = t4.w;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = i * (kWave / lpe) + lpe_sub;
          if (i < lpe && k < cnt) store_vec<4>(tab + k * p.H + lpe_part * 4, q4[i]);
        }
      } else if (lane < cnt) {
        const float* er = p.ev + (int64_t)my_eid * p.H;
        float* tr = tab + lane * p.H;
        if (p.ev_vec4) {
          for (int h = 0; h < p.H; h += 4) {
            float q[4];
            load_vec<4>(er + h, q);
            store_vec<4>(tr + h, q);
          }
        } else {
          for (int h = 0; h < p.H; ++h) tr[h] = er[h];
        }
      }
      wave_lds_sync();
    }
    // one step of U edges per lane group; FULL: every edge of the step is in
    // the batch and every feature chunk in the row (no per-edge masking)
    auto step = [&](int j0, auto full_tag) {
      constexpr bool FULL = decltype(full_tag)::value;
      constexpr bool H1 = HM == kOneHead;  // weights broadcast from the batch
      float val[U][NV][4];
      float wv[U][NV][WC];
      int32_t eu[U];
      bool ok[U];
      // wide batches: this group's U ids (and weights) of the step
      int32_t tsrc[WIDE ? U : 1];
      float tw[WIDE && WGT ? U : 1];
      int32_t tk[DUP && MAX ? U : 1];
      if constexpr (DUP && MAX) wide_get<NG, U>(wk, gid, j0, tk);
      if constexpr (WIDE) {
        wide_get<NG, U>(wid, gid, j0, tsrc);
        if constexpr (WGT) wide_get<NG, U>(wwt, gid, j0, tw);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int jb = j0 + u * NG;
        ok[u] = FULL || jb + gid < cnt;
        int src;
        if constexpr (WIDE) src = tsrc[u];
        else src = __shfl(my_src, jb + gid);
        if constexpr (EIDS) eu[u] = bcast_lane<NG>(my_eid, jb, gid);
        else if constexpr (DUP && MAX) eu[u] = (int)base + tk[u];
        else eu[u] = (int)(base + jb + gid);
        // the weight via the LDS crossbar (one permute) rather than two
        // readlanes and a select on the vector unit
        float w1 = 1.0f;
        if constexpr (WGT && H1) {
          if constexpr (WIDE) w1 = tw[u];
          else w1 = __shfl(my_w, jb + gid);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if (FULL || (ok[u] && act[v])) {
            load4<RAG>(row_at(xl[v], src, rb), val[u][v]);
            if constexpr (ELEM) {
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const float t = val[u][v][c] + pd[v][c];
                val[u][v][c] = t > 0.0f ? val[u][v][c] : -INFINITY;
              }
            }
#pragma unroll
            for (int c = 0; c < WC; ++c) {
              if constexpr (TAB)
                wv[u][v][c] = tab[(jb + gid) * p.H + hv[v][c]];
              else
                wv[u][v][c] = (MUL && !H1) ? p.ev[(int64_t)eu[u] * p.H + hv[v][c]] : w1;
            }
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) val[u][v][c] = MAX ? -INFINITY : 0.0f;
#pragma unroll
            for (int c = 0; c < WC; ++c) wv[u][v][c] = 1.0f;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if constexpr (POS) {
              // invalid slots hold -inf with weight 1: never strictly greater
              const float m = MUL ? wv[u][v][c % WC] * val[u][v][c] : val[u][v][c];
              if (m > acc[v][c]) {
                acc[v][c] = m;
                am[v][c] = eu[u];
              }
            } else if constexpr (MAX) {
              const float m = max_key(MUL ? wv[u][v][c % WC] * val[u][v][c] : val[u][v][c]);
              if ((FULL || ok[u]) && takes_over(m, eu[u], acc[v][c], am[v][c])) {
                acc[v][c] = m;
                am[v][c] = eu[u];
              }
            } else if constexpr (WGT) {
              acc[v][c] += wv[u][v][c % WC] * val[u][v][c];
            } else {
              acc[v][c] += val[u][v][c];
            }
          }
    };
    // full steps (wave-uniform test) take the unmasked body
    const bool all_feat = c0 + (int64_t)G * 4 * NV <= F;
    int j0 = 0;
    if (all_feat)
      for (; j0 + NG * U <= cnt; j0 += NG * U) step(j0, BoolTag<true>{});
    for (; j0 < cnt; j0 += NG * U) step(j0, BoolTag<false>{});
  }
  if constexpr (POS) {
    const int64_t first = it.b + gid;  // this group's first edge
    if (first < it.e) {
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (am[v][c] == INT_MAX) am[v][c] = (int32_t)first;
    }
  }

  // merge the lane groups (each holds a strided subset of the edges)
#pragma unroll
  for (int s = G; s < kWave; s <<= 1) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (MAX) {
          const float ob = __shfl_xor(acc[v][c], s);
          const int32_t oa = __shfl_xor(am[v][c], s);
          if (takes_over(ob, oa, acc[v][c], am[v][c])) {
            acc[v][c] = ob;
            am[v][c] = oa;
          }
        } else {
          acc[v][c] += __shfl_xor(acc[v][c], s);
        }
      }
  }
  if (gid != 0) return;
#pragma unroll
  for (int v = 0; v < NV; ++v)
    if (act[v]) spmm_store<4, MAX, SEG, EPK, RAG>(p, it, f[v], acc[v], am[v], lo[v]);
}

// The same merge with float4 lanes (F % 4 == 0, 16-byte aligned out / arg):
// a wavefront covers 256 columns, so each slot costs one 1 KiB load per
// wavefront instead of four.  Same slot order and combination order.
// RAG: any width F >= 4 and alignment, the last lane on the last four columns.
template <bool MAX, int EPI = kEpiNone, bool RAG = false>
__global__ __launch_bounds__(kBlock) void spmm_fixup4_kernel(const Fix* fix, const float* ws_f,
                                                             const int32_t* ws_i, int64_t F,
                                                             float* out, int32_t* arg,
                                                             const float* xd,
                                                             const int32_t* indptr) {
  __shared__ float red_v[kWavesPerBlock][kWave][4];
  __shared__ int32_t red_a[kWavesPerBlock][kWave][4];
  const int w = threadIdx.x >> 6;
  const int lane = lane_id();
  int64_t col = ((int64_t)blockIdx.y * kWave + lane) * 4;
  const bool valid = col < F;
  int lo = 0;  // first element this lane stores (ragged tail, else 0)
  if constexpr (RAG) {
    lo = valid ? (int)max((int64_t)0, col + 4 - F) : 0;
    col -= lo;
  }
  const Fix fx = fix[blockIdx.x];
  constexpr int kStride = kWavesPerBlock;
  float acc[4];
  int32_t am[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    acc[c] = MAX ? -INFINITY : 0.0f;
    am[c] = INT_MAX;
  }
  if (valid) {
    for (int s0 = fx.slot_begin + w; s0 < fx.slot_end; s0 += 4 * kStride) {
      float v[4][4];
      int32_t a[4][4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int s = s0 + k * kStride;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[k][c] = MAX ? -INFINITY : 0.0f;
          a[k][c] = INT_MAX;
        }
        if (s < fx.slot_end) {
          load4<RAG>(ws_f + (int64_t)s * F + col, v[k]);
          if constexpr (MAX) {
            const int4_a4 t = *reinterpret_cast<const int4_a4*>(ws_i + (int64_t)s * F + col);
            a[k][0] = t.x; a[k][1] = t.y; a[k][2] = t.z; a[k][3] = t.w;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if constexpr (MAX) {
            if (takes_over(v[k][c], a[k][c], acc[c], am[c])) {
              acc[c] = v[k][c];
              am[c] = a[k][c];
            }
          } else {
            acc[c] += v[k][c];
          }
        }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    red_v[w][lane][c] = acc[c];
    red_a[w][lane][c] = am[c];
  }
  __syncthreads();
  if (w != 0 || !valid) return;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    acc[c] = red_v[0][lane][c];
    am[c] = red_a[0][lane][c];
  }
#pragma unroll
  for (int k = 1; k < kWavesPerBlock; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if constexpr (MAX) {
        if (takes_over(red_v[k][lane][c], red_a[k][lane][c], acc[c], am[c])) {
          acc[c] = red_v[k][lane][c];
          am[c] = red_a[k][lane][c];
        }
      } else {
        acc[c] += red_v[k][lane][c];
      }
    }
  const int64_t o = (int64_t)fx.row * F + col;
  if constexpr (EPI != kEpiNone || MAX) {
    float ov[4];
    int32_t oa[4];
    float xv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (EPI != kEpiNone) load4<RAG>(xd + o, xv);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const bool none = am[c] == INT_MAX;
      if constexpr (EPI != kEpiNone) {
        const float t = acc[c] + xv[c];
        const bool pos = t > 0.0f;
        ov[c] = (none || !pos) ? 0.0f : t;
        oa[c] = none ? -1 : ((pos || EPI == kEpiMasked) ? am[c] : indptr[fx.row]);
      } else {
        ov[c] = none ? 0.0f : acc[c];
        oa[c] = none ? -1 : am[c];
      }
    }
    if constexpr (RAG) {
      store4_nt<RAG>(out + o, ov, lo);
      store4_i_nt<RAG>(arg + o, oa, lo);
    } else {
      store_vec<4>(out + o, ov);
      store_vec_i<4>(arg + o, oa);
    }
  } else if constexpr (RAG) {
    store4_nt<RAG>(out + o, acc, lo);
  } else {
    store_vec<4>(out + o, acc);
  }
}

// Lane layout of the float4 kernels: G lanes per feature row, NV float4 per
// lane, U edges in flight per lane group; RAG: any width >= 4 and alignment.
// MANY: for edge values of more than kTabHeads heads (only then).
template <int G_, int NV_, int U_, bool RAG_, bool MANY_ = false>
struct SpmmLayout {
  static constexpr int G = G_, NV = NV_, U = U_;
  static constexpr bool RAG = RAG_, MANY = MANY_;
};

// avg: the items' average edge count (256-edge batches where the lane layout
// allows them and the items are long enough, wide_item_edges)
template <class L, bool MUL, bool MAX, bool EIDS, bool ADD, int HM>
void spmm_fast_seg2(const SpmmParams& prm, bool seg, int64_t avg, dim3 grid, hipStream_t st) {
  constexpr int G = L::G, NV = L::NV, U = L::U;
  constexpr bool RAG = L::RAG;
  if constexpr (kWave / G >= 2 && U % 4 == 0 && !EIDS && HM == kOneHead) {
    if (avg >= wide_item_edges<kWave / G>()) {
      // (the sums' run weights cost rows of 64 floats or less what they save: 20M
      // edges of 32 floats 149 -> 183 us; so does the max's table of first edges up
      // to 16 floats: communities of 300 edges a row, 8 floats, 109 -> 115 us,
      // 20M power-law edges of 16 134 -> 137)
      if constexpr (!RAG && NV == 1 && !(MUL && MAX) && (MAX ? G >= 8 : G == 32)) {
        if (seg && prm.repeats) {
          FG_LAUNCH((spmm_fast_kernel<G, NV, U, MUL, MAX, EIDS, true, ADD, HM, true, RAG, true>),
                    grid, st, prm);
          return;
        }
      }
      if (seg)
        FG_LAUNCH((spmm_fast_kernel<G, NV, U, MUL, MAX, EIDS, true, ADD, HM, true, RAG>), grid, st,
                  prm);
      else
        FG_LAUNCH((spmm_fast_kernel<G, NV, U, MUL, MAX, EIDS, false, ADD, HM, true, RAG>), grid,
                  st, prm);
      return;
    }
  }
  if (seg)
    FG_LAUNCH((spmm_fast_kernel<G, NV, U, MUL, MAX, EIDS, true, ADD, HM, false, RAG>), grid, st,
              prm);
  else
    FG_LAUNCH((spmm_fast_kernel<G, NV, U, MUL, MAX, EIDS, false, ADD, HM, false, RAG>), grid, st,
              prm);
}

template <class L, bool MUL, bool MAX, bool EIDS, bool ADD = false>
void spmm_fast_seg(const SpmmParams& prm, bool seg, int64_t avg, dim3 grid, hipStream_t st) {
  if constexpr (MUL) {
    if constexpr (L::MANY) {
      spmm_fast_seg2<L, MUL, MAX, EIDS, ADD, kManyHeads>(prm, seg, avg, grid, st);
      return;
    } else if (prm.H > 1) {
      spmm_fast_seg2<L, MUL, MAX, EIDS, ADD, kHeadTable>(prm, seg, avg, grid, st);
      return;
    }
  }
  if constexpr (!L::MANY) spmm_fast_seg2<L, MUL, MAX, EIDS, ADD, kOneHead>(prm, seg, avg, grid, st);
}

template <class L, bool MUL, bool MAX, bool ADD = false>
void spmm_fast_eids(const SpmmParams& prm, bool seg, int64_t avg, dim3 grid, hipStream_t st) {
  // copy + sum never looks at edge ids
  if constexpr (MUL || MAX) {
    if (prm.eids) {
      spmm_fast_seg<L, MUL, MAX, true, ADD>(prm, seg, avg, grid, st);
      return;
    }
  }
  spmm_fast_seg<L, MUL, MAX, false, ADD>(prm, seg, avg, grid, st);
}

// Launches the kernel of the narrowest layout that covers rows of F floats.
template <bool MAX, bool RAG>
void spmm_fast_dispatch(const SpmmParams& prm, bool mul, bool seg, int64_t avg, hipStream_t st) {
  const int64_t Q = (prm.F + 3) / 4;  // float4 per row
  auto go = [&](auto layout, int64_t chunks) {
    using L = decltype(layout);
    const dim3 grid = grid_for(prm.n_items, chunks);
    if constexpr (MAX && !L::MANY) {
      if (prm.xd) {
        spmm_fast_eids<L, false, true, true>(prm, seg, avg, grid, st);
        return;
      }
    }
    if (mul) spmm_fast_eids<L, true, MAX>(prm, seg, avg, grid, st);
    else if constexpr (!L::MANY) spmm_fast_eids<L, false, MAX>(prm, seg, avg, grid, st);
  };
  if constexpr (RAG) {
    if (mul && prm.H > kTabHeads) {  // at least 17 floats; wide rows in chunks of 256
      if (Q <= 8) go(SpmmLayout<8, 1, 4, RAG, true>{}, 1);
      else if (Q <= 16) go(SpmmLayout<16, 1, 4, RAG, true>{}, 1);
      else if (Q <= 32) go(SpmmLayout<32, 1, 4, RAG, true>{}, 1);
      else go(SpmmLayout<64, 1, 4, RAG, true>{}, (Q + 63) / 64);
      return;
    }
  }
  // the aligned rows' layouts, also with a weight load per float4 and step for
  // more heads than the table holds
  auto all = [&](auto many_tag) {
    constexpr bool MANY = decltype(many_tag)::value;
    if constexpr (!MANY) {  // (17 heads of 4 features take 17 float4s)
      if (Q <= 4) return go(SpmmLayout<4, 1, 4, RAG>{}, 1);
      if (Q <= 8) return go(SpmmLayout<8, 1, 8, RAG>{}, 1);
      if (Q <= 16) return go(SpmmLayout<16, 1, 8, RAG>{}, 1);
    }
    if (Q <= 32) go(SpmmLayout<32, 1, 8, RAG, MANY>{}, 1);
    else if (Q <= 64) go(SpmmLayout<64, 1, 8, RAG, MANY>{}, 1);
    // three float4 a lane where two or four would leave over a quarter of the
    // lanes idle (10M power-law edges, max: 300 floats 754 -> 725 us, 602 2253 ->
    // 1777; weighted sum 701 -> 653, 1585 -> 1478; uniform edges, bound by lines
    // rather than lanes, equal).  16 x 3 for 130-192 floats and 8 x 3 for 66-96
    // are slower on short rows and equal on long ones; the max of rows of a few
    // edges, which leave the second lane group idle, keeps 64 x 2 (4 edges a row, 300
    // floats 109 us, with 32 x 3 124).
    else if (MAX && Q > 64 && Q <= 96 && avg < 8) go(SpmmLayout<64, 2, 4, RAG, MANY>{}, 1);
    else if (Q <= 96) go(SpmmLayout<32, 3, 4, RAG, MANY>{}, 1);
    else if (Q <= 128) go(SpmmLayout<64, 2, 4, RAG, MANY>{}, 1);
    else if (Q <= 192) go(SpmmLayout<64, 3, 2, RAG, MANY>{}, 1);
    else go(SpmmLayout<64, 4, 2, RAG, MANY>{}, (Q + 255) / 256);
  };
  if constexpr (!RAG) {
    if (mul && prm.H > kTabHeads) {
      all(BoolTag<true>{});
      return;
    }
  }
  all(BoolTag<false>{});
}

}  // namespace
}  // namespace fg
