// Reverse-mode derivative of the calculation stage (TensorNEAT Section 3.3)
// with respect to connection weights and node biases, for gradient refinement
// of weights.
//
// Mapping: one wavefront per genome walks the genome's tiles of 64
// observations in order (lane = observation). Per tile, in LDS:
//   1. forward pass, keeping the value row v[p][.] of every position;
//   2. upstream gradient rows g[p][.]: dL/dy at the outputs (given, or the
//      fused mean-squared error 2 (y - t) * scale), 0 elsewhere;
//   3. reverse sweep over the topological order: delta_p = g_p * act'(z_p)
//      replaces g_p in place and is pushed to the sources through
//      g_src += delta_p * resp_p * d agg / d t_e * w_e;
//   4. lanes switch to edges: dW_e += resp_k * sum_b delta_k[b] * d agg/d t_e[b]
//      * v_src[b] and db_k += sum_b delta_k[b], as 64-term dot products over
//      the tile's rows, added to per-edge / per-position accumulators.
// The tile order and the in-tile summation order are fixed, so results are
// deterministic. act' comes from the stored value for identity, sigmoid, tanh
// and relu; sin, gaussian and abs re-evaluate z from the in-edges. Non-sum
// aggregations re-evaluate their terms in both phases.
#include <algorithm>
#include <type_traits>

#include "rf_file.hpp"

namespace tn {

namespace {

constexpr int kRow = kWave + 1;  // floats per LDS row (1 float of padding)

struct BwdArgs {
  int64_t obs_stride;
  int B;
  const float* dY;  // [P][B][O] upstream gradient, or null for the fused MSE
  int64_t dY_stride;
  const float* target;  // fused MSE targets (when dY is null)
  int64_t target_stride;
  float scale;  // MSE: loss = scale * sum (y - t)^2, dL/dy = 2 scale (y - t)
  float* loss;  // may be null
  float* dW;    // conn block
  float* db;    // node block
  // positions and in-edges of a genome of backward_rf_kernel, at most
  int rf_pos, rf_edges;
};

struct BwdLds {
  size_t rec_off, edge_off, edst_off, io_off, dw_off, db_off, v_off, g_off, bytes;
};

__host__ __device__ inline size_t al16(size_t x) { return (x + 15) & ~size_t(15); }

__host__ __device__ inline BwdLds bwd_lds(int N, int C, int nio) {
  BwdLds L;
  L.rec_off = 0;
  L.edge_off = al16(L.rec_off + sizeof(NodeRec) * (size_t)N);
  L.edst_off = al16(L.edge_off + sizeof(EdgeRec) * (size_t)C);
  L.io_off = al16(L.edst_off + sizeof(int32_t) * (size_t)C);
  L.dw_off = al16(L.io_off + sizeof(int32_t) * (size_t)nio);
  L.db_off = al16(L.dw_off + sizeof(float) * (size_t)C);
  L.v_off = al16(L.db_off + sizeof(float) * (size_t)N);
  L.g_off = al16(L.v_off + sizeof(float) * std::max((size_t)N * kRow, (size_t)(C + N)));
  L.bytes = al16(L.g_off + sizeof(float) * (size_t)N * kRow);
  return L;
}

// z of position p for this lane (re-evaluated from the in-edges).
__device__ float node_z(const NodeRec& rec, int f, const EdgeRec* edges, const float* v,
                        int lane) {
  const int er = __builtin_amdgcn_readfirstlane(rec.erange);
  const int e0 = er & 0xffff, e1 = (er >> 16) & 0xffff;
  const int agg = (f >> 8) & 0xff;
  float s = 0.0f;
  if (agg == TN_AGG_SUM) {
    for (int e = e0; e < e1; ++e) s = fmaf(edges[e].w, v[edges[e].src * kRow + lane], s);
  } else if (e1 > e0) {
    s = edges[e0].w * v[edges[e0].src * kRow + lane];
    for (int e = e0 + 1; e < e1; ++e) {
      const float t = edges[e].w * v[edges[e].src * kRow + lane];
      switch (agg) {
        case TN_AGG_PRODUCT: s = s * t; break;
        case TN_AGG_MAX: s = fmaxf(s, t); break;
        case TN_AGG_MIN: s = fminf(s, t); break;
        case TN_AGG_MEAN: s = s + t; break;
        default: s = fabsf(t) > fabsf(s) ? t : s; break;
      }
    }
    if (agg == TN_AGG_MEAN) s = s / (float)(e1 - e0);
  }
  return fmaf(rec.resp, s, rec.bias);
}

// d agg / d t_e for in-edge e of a node with a non-sum aggregation, this lane.
__device__ float agg_partial(int agg, int e, int e0, int e1, const EdgeRec* edges, const float* v,
                             int lane) {
  if (agg == TN_AGG_MEAN) return 1.0f / (float)(e1 - e0);
  if (agg == TN_AGG_PRODUCT) {
    float p = 1.0f;
    for (int x = e0; x < e1; ++x)
      if (x != e) p *= edges[x].w * v[edges[x].src * kRow + lane];
    return p;
  }
  // max / min / maxabs: the first extreme term in row order takes it
  int best = e0;
  float bv = edges[e0].w * v[edges[e0].src * kRow + lane];
  for (int x = e0 + 1; x < e1; ++x) {
    const float t = edges[x].w * v[edges[x].src * kRow + lane];
    const bool take = agg == TN_AGG_MAX ? t > bv : (agg == TN_AGG_MIN ? t < bv : fabsf(t) > fabsf(bv));
    if (take) {
      best = x;
      bv = t;
    }
  }
  return best == e ? 1.0f : 0.0f;
}

// Genomes the register-file adjoint (backward_rf_kernel, below) takes: at most
// kRfPos positions, kRfEdges in-edges and kRfSums rows of four sums, sum or
// mean aggregation; in some launches (see launch_backward) kRfPosLow and
// kRfEdgesLow.
constexpr int kRfPos = 64, kRfEdges = 192, kRfSums = 64;
constexpr int kRfPosLow = 48, kRfEdgesLow = 64;
constexpr int kRfWaves = 4;  // wavefronts per genome, at most
// Groups of steps, and LDS rows of a wavefront: its sums, and the folded ones of
// a group (20,240 bytes with the genome's tables: eight wavefronts fit a compute
// unit, as many as the registers allow).
constexpr int kRfGroups = 4, kRfRows = kRfSums + 4 * kRfSums / kWave;
// More observations than this take four tiles a step: 300 observations of 1500
// genomes 136 us with three steps of two tiles, 164 with two of four.
constexpr int kRfWide = 384;

// Whether genome g is backward_rf_kernel's; by one wavefront, lane = position.
__device__ __forceinline__ bool rf_bwd_eligible(int st, int n, const int32_t* rp,
                                                const int32_t* fnp, const BwdArgs& a) {
  if (st || n > a.rf_pos || rp[n] > a.rf_edges) return false;
  const int lane = lane_id();
  const int f = lane < n ? fnp[lane] : -1;
  const int ne = lane < n ? rp[lane + 1] - rp[lane] : 0;
  const int agg = (f >> 8) & 0xff;
  if (__ballot(ne > kWave || (f >= 0 && agg != TN_AGG_SUM && agg != TN_AGG_MEAN))) return false;
  return wave_sum_int(f >= 0 ? sum_rows(ne) : 0) <= kRfSums;
}

__global__ __launch_bounds__(kWave) void backward_kernel(
    PopView pop, const int32_t* __restrict__ status, const int32_t* __restrict__ n_valid,
    const int32_t* __restrict__ order, const int32_t* __restrict__ row_ptr,
    const int32_t* __restrict__ src, const int32_t* __restrict__ w_bits,
    const int32_t* __restrict__ edge_row, const int32_t* __restrict__ fn,
    const int32_t* __restrict__ bias_bits, const int32_t* __restrict__ resp_bits,
    const int32_t* __restrict__ io_pos, const float* __restrict__ obs, BwdArgs a, int lds_ok) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int g = blockIdx.x;
  const int lane = lane_id();
  const int I = pop.n_in, O = pop.n_out, nio = I + O;
  const int64_t nb = pop.node_base(g), cb = pop.conn_base(g), rb = pop.rowptr_base(g);
  const int64_t nrows = pop.node_rows(g), crows = pop.conn_rows(g);
  const int st = status[g];
  const BwdLds L = bwd_lds(pop.N_max, pop.C_max, nio);
  NodeRec* recs = reinterpret_cast<NodeRec*>(lds + L.rec_off);
  EdgeRec* edges = reinterpret_cast<EdgeRec*>(lds + L.edge_off);
  int32_t* edst = reinterpret_cast<int32_t*>(lds + L.edst_off);
  int32_t* io_l = reinterpret_cast<int32_t*>(lds + L.io_off);
  float* dwacc = reinterpret_cast<float*>(lds + L.dw_off);
  float* dbacc = reinterpret_cast<float*>(lds + L.db_off);
  float* v = reinterpret_cast<float*>(lds + L.v_off);
  float* gr = reinterpret_cast<float*>(lds + L.g_off);

  if (rf_bwd_eligible(st, n_valid[g], row_ptr + rb, fn + nb, a)) return;  // backward_rf_kernel's
  // flagged genomes, and (when N_max rows of values and gradients exceed the
  // device's LDS) every genome the register-file adjoint could not take
  if (st || !lds_ok) {
    const float nan = __builtin_nanf("");
    for (int64_t r = lane; r < crows; r += kWave) a.dW[cb + r] = nan;
    for (int64_t r = lane; r < nrows; r += kWave) a.db[nb + r] = nan;
    if (a.loss && lane == 0) a.loss[g] = nan;
    return;
  }
  const int n = n_valid[g];
  const int n_edges = row_ptr[rb + n];
  // stage the program; destination position of every edge
  for (int p = lane; p < n; p += kWave) {
    NodeRec r;
    const int e0 = row_ptr[rb + p], e1 = row_ptr[rb + p + 1];
    r.erange = e0 | (e1 << 16);
    r.fn = fn_with_row(fn[nb + p], p);  // one value row per position here
    r.bias = __int_as_float(bias_bits[nb + p]);
    r.resp = __int_as_float(resp_bits[nb + p]);
    recs[p] = r;
    for (int e = e0; e < e1; ++e) edst[e] = p;
    dbacc[p] = 0.0f;
  }
  for (int e = lane; e < n_edges; e += kWave) {
    EdgeRec q;
    q.src = src[cb + e];
    q.w = __int_as_float(w_bits[cb + e]);
    edges[e] = q;
    dwacc[e] = 0.0f;
  }
  for (int k = lane; k < nio; k += kWave) io_l[k] = io_pos[(int64_t)g * nio + k];
  wave_sync();

  float sse = 0.0f;
  const int n_tiles = (a.B + kWave - 1) / kWave;
  for (int t = 0; t < n_tiles; ++t) {
    const int b0 = t * kWave;
    const int nbat = min(kWave, a.B - b0);
    const bool live = lane < nbat;
    // 1. inputs and forward
    const float* xo = obs + (int64_t)g * a.obs_stride + (int64_t)b0 * I;
    for (int c = 0; c < I; ++c) v[io_l[c] * kRow + lane] = live ? xo[(int64_t)lane * I + c] : 0.0f;
    wave_sync();
    LdsProg lp{recs, edges};
    for (int p = 0; p < n; ++p) eval_node<1, kRow>(lp, p, v + lane);
    // 2. upstream gradient rows
    for (int p = 0; p < n; ++p) gr[p * kRow + lane] = 0.0f;
    wave_sync();
    for (int j = 0; j < O; ++j) {
      const int pj = io_l[I + j];
      float gy = 0.0f;
      if (live) {
        const int64_t o = (int64_t)lane * O + j;
        const float y = v[pj * kRow + lane];
        if (a.dY) {
          gy = a.dY[(int64_t)g * a.dY_stride + (int64_t)b0 * O + o];
        } else {
          const float d = y - a.target[(int64_t)g * a.target_stride + (int64_t)b0 * O + o];
          sse = fmaf(d, d, sse);
          gy = 2.0f * a.scale * d;
        }
      }
      gr[pj * kRow + lane] += gy;
    }
    wave_sync();
    // 3. reverse sweep: g_p -> delta_p, pushed to the sources
    for (int p = n - 1; p >= 0; --p) {
      const NodeRec rec = recs[p];
      const int f = __builtin_amdgcn_readfirstlane(rec.fn);
      if (f < 0) continue;
      const int act = f & 7, agg = (f >> 8) & 0xff;  // codes below 7: transformed genomes
      const float vp = v[p * kRow + lane];
      const float z = slope_needs_z(act) ? node_z(rec, f, edges, v, lane) : 0.0f;
      const float delta = live ? gr[p * kRow + lane] * act_slope(act, vp, z) : 0.0f;
      gr[p * kRow + lane] = delta;
      const int er = __builtin_amdgcn_readfirstlane(rec.erange);
      const int e0 = er & 0xffff, e1 = (er >> 16) & 0xffff;
      const float dr = delta * rec.resp;
      for (int e = e0; e < e1; ++e) {
        const EdgeRec q = edges[e];
        const float part = agg == TN_AGG_SUM ? 1.0f : agg_partial(agg, e, e0, e1, edges, v, lane);
        gr[q.src * kRow + lane] = fmaf(dr * part, q.w, gr[q.src * kRow + lane]);
      }
    }
    wave_sync();
    // 4. lanes over edges / positions: dot products over the tile
    for (int e = lane; e < n_edges; e += kWave) {
      const int k = edst[e];
      const NodeRec rk = recs[k];
      const int agg = (rk.fn >> 8) & 0xff;
      const int s = edges[e].src;
      float acc = 0.0f;
      if (agg == TN_AGG_SUM) {
        for (int b = 0; b < kWave; ++b) acc = fmaf(gr[k * kRow + b], v[s * kRow + b], acc);
      } else {
        const int e0 = rk.erange & 0xffff, e1 = (rk.erange >> 16) & 0xffff;
        for (int b = 0; b < kWave; ++b)
          acc = fmaf(gr[k * kRow + b] * agg_partial(agg, e, e0, e1, edges, v, b), v[s * kRow + b],
                     acc);
      }
      dwacc[e] = fmaf(rk.resp, acc, dwacc[e]);
    }
    for (int p = lane; p < n; p += kWave) {
      if (recs[p].fn < 0) continue;
      float acc = 0.0f;
      for (int b = 0; b < kWave; ++b) acc += gr[p * kRow + b];
      dbacc[p] += acc;
    }
    wave_sync();
  }
  // write out: every row of the genome's blocks exactly once, through
  // row -> edge / row -> position maps built in the (now free) value rows
  int32_t* row_edge = reinterpret_cast<int32_t*>(v);
  int32_t* row_pos = row_edge + pop.C_max;
  for (int64_t r = lane; r < crows; r += kWave) row_edge[r] = -1;
  for (int64_t r = lane; r < nrows; r += kWave) row_pos[r] = -1;
  wave_sync();
  for (int e = lane; e < n_edges; e += kWave) row_edge[edge_row[cb + e]] = e;
  for (int p = lane; p < n; p += kWave)
    if (recs[p].fn >= 0) row_pos[order[nb + p]] = p;
  wave_sync();
  for (int64_t r = lane; r < crows; r += kWave) {
    const int e = row_edge[r];
    a.dW[cb + r] = e >= 0 ? dwacc[e] : 0.0f;
  }
  for (int64_t r = lane; r < nrows; r += kWave) {
    const int p = row_pos[r];
    a.db[nb + r] = p >= 0 ? dbacc[p] : 0.0f;
  }
  if (a.loss) {
    const float total = wave_sum(sse);
    if (lane == 0) a.loss[g] = a.scale * total;
  }
}

// ------------------------------------------------ register-file adjoint
//
// The same derivative for the genomes that fit it (tn_backward runs both
// kernels; each takes the genomes the other leaves). One to four wavefronts per
// genome share its steps of K tiles of 64 observations (lane = observation):
// K = 4, 2 or 1, by the rows a genome needs. Values and upstream gradients live
// in registers: rows 2 i and 2 i + 1 of a tile are the value and the gradient
// of computed node i, then come the inputs' values (they need no gradient). The
// program sits in LDS and comes across the lanes (a node's words in lane i for
// computed node i, its in-edges one LDS read ahead). Per step:
//   forward: v_i = act(bias + resp * agg(w_e v_src)) at every computed
//     node (gradient row cleared in the same window);
//   outputs: gbar_out += dL/dy;
//   reverse: delta_i = gbar_i act'(z_i) (z re-evaluated for sin, gaussian,
//     abs); db_i += delta_i; dt = delta_i resp (/ n for mean); per in-edge
//     dW_e += dt v_src and, unless the source is an input, gbar_src += dt w_e
//     (one indexed read-modify-write).
// The sums of a node (its bias, then its in-edges) are taken four at a time:
// each is one value per lane (the step's tiles added first); swapping halves
// and quarters of the wavefront between registers adds lane l to lanes l + 32
// and l + 16, so that four sums of 64 lanes become one register of four times
// 16 lanes, added to one LDS row. That is a quarter of the LDS traffic and of
// the LDS itself of one slot per sum and lane, so the registers (two wavefronts
// per SIMD) and not the LDS limit occupancy, and genomes of up to 192 in-edges
// fit. At the end of a group of steps each sum's 16 lanes are added, then the
// groups in order: the same bits however the launch splits a genome. Bound by
// instruction issue. 4096 genomes (4 -> 2, 22 positions, 45 in-edges), 1024
// samples: 243 us; 569 us with a slot per sum and lane, two tiles a step. 1000
// genomes (17 -> 6, 39 positions, 126 in-edges), 256 observations: 51 us; 148 us in
// backward_kernel.

// What a step reads of its genome, and this lane's share of it (computed node
// i in lane i).
struct RfGenome {
  const int2* edge;  // LDS: the source's row, weight
  int nc;            // computed nodes
  int l_fn, l_bias, l_resp;
  int l_edge;        // byte offset of the first in-edge | in-edges << 16
  int l_sum;         // first row of sums
  int l_in, l_out;   // row of input / output `lane`
  int I, O;
};

// One step: K tiles of observations from b0 on; sums are added to acc, the
// wavefront's rows in LDS. Returns its part of the squared error.
template <int K>
__device__ __forceinline__ float rf_step(const RfGenome& q, int b0, const float* xg,
                                         const float* ug, const BwdArgs& a, float* acc) {
  using F = Files<K>;
  const int lane = lane_id();
  // 32-bit lane offsets from the step's own base: a register per address
  const float* xs = xg + (int64_t)b0 * q.I;
  const int left = a.B - b0;
  bool live[K];
#pragma unroll
  for (int k = 0; k < K; ++k) live[k] = k * kWave + lane < left;
  for (int c0 = 0; c0 < q.I; c0 += 2) {  // two inputs' loads in flight
    const int c1 = min(c0 + 1, q.I - 1);
    float x[2][K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t o = live[k] ? (uint32_t)((k * kWave + lane) * q.I) : 0u;
      x[0][k] = xs[o + (uint32_t)c0];
      x[1][k] = xs[o + (uint32_t)c1];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int k = 0; k < K; ++k) x[c][k] = live[k] ? x[c][k] : 0.0f;
      F::set_v(__builtin_amdgcn_readlane(q.l_in, c ? c1 : c0), x[c]);
    }
  }
  auto edges_of = [&](int i) {
    const int at = __builtin_amdgcn_readlane(q.l_edge, i) & 0xffff;
    return *reinterpret_cast<const int2*>(reinterpret_cast<const char*>(q.edge + lane) + at);
  };
  int2 ed = edges_of(0);
  auto row_of = [&](int e) { return __builtin_amdgcn_readlane(ed.x, e); };
  auto weight = [&](int e) { return __int_as_float(__builtin_amdgcn_readlane(ed.y, e)); };
  // pre-activations of computed node i
  auto pre = [&](int i, int f, int ne, float (&z)[K]) {
    float s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = 0.0f;
    if (ne > 0) {
      F::fma_v(s, weight(0), row_of(0));
      if (ne > 1) {
        F::fma_v(s, weight(1), row_of(1));
        for (int e = 2; e < ne; ++e) F::fma_v(s, weight(e), row_of(e));
      }
      if (((f >> 8) & 0xff) == TN_AGG_MEAN)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          s[k] = s[k] / (float)ne;
          asm volatile("" : "+v"(s[k]));
        }
    }
    const float rho = __int_as_float(__builtin_amdgcn_readlane(q.l_resp, i));
    const float bias = __int_as_float(__builtin_amdgcn_readlane(q.l_bias, i));
#pragma unroll
    for (int k = 0; k < K; ++k) z[k] = fmaf(rho, s[k], bias);
  };
  // forward
  for (int i = 0; i < q.nc; ++i) {
    const int2 en = edges_of(min(i + 1, q.nc - 1));
    const int f = __builtin_amdgcn_readlane(q.l_fn, i);
    float z[K], v[K];
    pre(i, f, __builtin_amdgcn_readlane(q.l_edge, i) >> 16, z);
    activate_all<K>(f & 7, z, v);  // codes below 7: transformed genomes
    F::set_vg(2 * i, v);
    ed = en;
  }
  // upstream gradient at the outputs
  const float* us = ug + (int64_t)b0 * q.O;
  float sse = 0.0f;
  for (int jo = 0; jo < q.O; ++jo) {
    const int pj = __builtin_amdgcn_readlane(q.l_out, jo);  // outputs are computed nodes
    float y[K], gy[K];
    F::get_v(pj, y);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t o = (uint32_t)((live[k] ? (k * kWave + lane) * q.O : 0) + jo);
      const float up = us[o];
      if (a.dY) {
        gy[k] = live[k] ? up : 0.0f;
      } else {
        const float d = live[k] ? y[k] - up : 0.0f;
        sse = fmaf(d, d, sse);
        gy[k] = 2.0f * a.scale * d;
      }
    }
    F::fma_g(pj, gy, 1.0f);
  }
  // reverse sweep
  ed = edges_of(q.nc - 1);
  for (int i = q.nc - 1; i >= 0; --i) {
    const int2 en = edges_of(max(i - 1, 0));
    const int f = __builtin_amdgcn_readlane(q.l_fn, i);
    const int ne = __builtin_amdgcn_readlane(q.l_edge, i) >> 16;
    const int act = f & 7;
    float* sum = acc + __builtin_amdgcn_readlane(q.l_sum, i) * kWave + lane;
    float old = *sum;
    float g[K], v[K], z[K], dt[K], db = 0.0f;
    F::get_gv(2 * i, g, v);
#pragma unroll
    for (int k = 0; k < K; ++k) z[k] = 0.0f;
    if (slope_needs_z(act)) pre(i, f, ne, z);
    float slope[K];
    act_slopes<K>(act, v, z, slope);
    const float rho = __int_as_float(__builtin_amdgcn_readlane(q.l_resp, i));
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float d = live[k] ? g[k] * slope[k] : 0.0f;
      db += d;
      dt[k] = d * rho;
    }
    if (((f >> 8) & 0xff) == TN_AGG_MEAN && ne > 0)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        dt[k] = dt[k] / (float)ne;
        asm volatile("" : "+v"(dt[k]));
      }
    auto term = [&](int e) {
      const int j = row_of(e);
      return j < 2 * q.nc ? F::dot_v_fma_g(j, dt, weight(e)) : F::dot_v(j, dt);  // else an input
    };
    float t1 = 0.0f, t2 = 0.0f, t3 = 0.0f;
    if (ne > 0) {
      t1 = term(0);
      if (ne > 1) {
        t2 = term(1);
        if (ne > 2) t3 = term(2);
      }
    }
    *sum = old + fold4(db, t1, t2, t3);
    for (int e = 3; e < ne; e += 4) {
      sum += kWave;
      old = *sum;
      float t0 = term(e);
      t1 = t2 = t3 = 0.0f;
      if (e + 1 < ne) {
        t1 = term(e + 1);
        if (e + 2 < ne) {
          t2 = term(e + 2);
          if (e + 3 < ne) t3 = term(e + 3);
        }
      }
      *sum = old + fold4(t0, t1, t2, t3);
    }
    ed = en;
  }
  return sse;
}

// kFold: a genome may have more groups of steps than wavefronts.
template <bool kFold>
__global__ __launch_bounds__(kWave * kRfWaves) __attribute__((amdgpu_num_vgpr(TN_RF_FILE / 2))) void
backward_rf_kernel(PopView pop, const int32_t* __restrict__ status,
                   const int32_t* __restrict__ n_valid, const int32_t* __restrict__ order,
                   const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ src,
                   const int32_t* __restrict__ w_bits, const int32_t* __restrict__ edge_row,
                   const int32_t* __restrict__ fn, const int32_t* __restrict__ bias_bits,
                   const int32_t* __restrict__ resp_bits, const int32_t* __restrict__ io_pos,
                   const float* __restrict__ obs, BwdArgs a) {
  rf_file_reserve();
  extern __shared__ __align__(16) float acc_all[];  // [waves][kRows][64]
  __shared__ int2 edge[kRfEdges + kWave];
  __shared__ int32_t sums_of[kRfSums];  // a row of sums' computed node | its row of the node << 8
  __shared__ int2 node[kRfPos];            // its position, l_edge
  __shared__ float part[kRfGroups];
  const int g = blockIdx.x, tid = threadIdx.x, T = blockDim.x;
  const int lane = lane_id(), wave = wave_id(), W = T / kWave;
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g)),
                rb = uniform64(pop.rowptr_base(g));
  const int nrows = (int)pop.node_rows(g), crows = (int)pop.conn_rows(g);
  const int n = n_valid[g];
  if (!rf_bwd_eligible(status[g], n, row_ptr + rb, fn + nb, a)) return;  // the LDS kernel's genome
  const int n_edges = row_ptr[rb + n];
  const int nio = pop.n_in + pop.n_out;
  constexpr int kRows = kFold ? kRfRows : kRfSums;
  float* acc = acc_all + wave * kRows * kWave;
  RfGenome q;
  q.edge = edge;
  q.I = pop.n_in;
  q.O = pop.n_out;
  // position p in lane p, then computed node i in lane i
  const int p_fn = lane < n ? fn[nb + lane] : -1;
  const int p_start = lane < n ? row_ptr[rb + lane] : 0, p_end = lane < n ? row_ptr[rb + lane + 1] : 0;
  const uint64_t nodes = __ballot(p_fn >= 0), inputs = __ballot(lane < n && p_fn < 0);
  q.nc = __popcll(nodes);
  auto row_at = [&](int p) {  // of position p
    const uint64_t below = ((uint64_t)1 << p) - 1;
    return (nodes >> p) & 1 ? 2 * __popcll(nodes & below)
                            : 2 * q.nc + __popcll(inputs & below);
  };
  for (int e = tid; e < n_edges; e += T)
    edge[e] = make_int2(row_at(src[cb + e]), w_bits[cb + e]);
  const int mine = p_fn >= 0 ? mbcnt(nodes) : -1;
  if (wave == 0 && mine >= 0)
    node[mine] = make_int2(lane, (p_start * (int)sizeof(int2)) | ((p_end - p_start) << 16));
  __syncthreads();
  const int2 nd = lane < q.nc ? node[lane] : make_int2(0, 0);
  const int rows = lane < q.nc ? sum_rows(nd.y >> 16) : 0;
  const int row_end = wave_inclusive_scan(rows), row0 = row_end - rows;
  const int n_sums = __builtin_amdgcn_readlane(row_end, kWave - 1);
  q.l_fn = __shfl(p_fn, nd.x, kWave);
  q.l_bias = lane < q.nc ? bias_bits[nb + nd.x] : 0;
  q.l_resp = lane < q.nc ? resp_bits[nb + nd.x] : 0;
  q.l_edge = nd.y;
  q.l_sum = row0;
  q.l_in = lane < q.I ? row_at(io_pos[(int64_t)g * nio + lane]) : 0;
  q.l_out = lane < q.O ? row_at(io_pos[(int64_t)g * nio + q.I + lane]) : 0;
  if (wave == 0)
    for (int c = 0; c < rows; ++c) sums_of[row0 + c] = lane | (c << 8);
  for (int r = 0; r < n_sums; ++r) acc[r * kWave + lane] = 0.0f;
  // rows without a sum stay 0; the others are stored after the last barrier
  for (int r = tid; r < crows; r += T) a.dW[cb + r] = 0.0f;
  for (int r = tid; r < nrows; r += T) a.db[nb + r] = 0.0f;
  const float* xg = obs + (int64_t)g * a.obs_stride;
  const float* ug = a.dY ? a.dY + (int64_t)g * a.dY_stride
                         : a.target + (int64_t)g * a.target_stride;
  // As many tiles a step as the genome's rows leave room for and the batch fills.
  // The steps belong to kRfGroups groups, whose sums are folded and then added
  // in order: which wavefront takes a group leaves the bits alone.
  float* kept = acc + kRfSums * kWave;  // kFold: folded sums of groups before the wavefront's last
  // sum i / 4, quarter i % 4: its 16 lanes, starting at a lane of its own so that
  // neighbours read different banks
  auto folded = [](const float* rows, int i) {
    const float* from = rows + (i >> 2) * kWave + (i & 3) * 16;
    float t = 0.0f;
#pragma unroll 8
    for (int b = 0; b < 16; ++b) t += from[(b + i) & 15];
    return t;
  };
  auto steps = [&](auto tiles) {
    constexpr int K = decltype(tiles)::value, kStep = K * kWave;
    if constexpr (!kFold) {  // wavefront v takes group v
      float sse = 0.0f;
      for (int b0 = wave * kStep; b0 < a.B; b0 += W * kStep)
        sse += rf_step<K>(q, b0, xg, ug, a, acc);
      if (a.loss) {
        const float total = wave_sum(sse);
        if (lane == 0) part[wave] = total;
      }
      return;
    }
    // one wavefront takes all groups in turn, else each its own and, back from
    // the last, another
    for (int v = wave; v < kRfGroups && v * kStep < a.B;) {
      float sse = 0.0f;
      for (int b0 = v * kStep; b0 < a.B; b0 += kRfGroups * kStep)
        sse += rf_step<K>(q, b0, xg, ug, a, acc);
      if (a.loss) {
        const float total = wave_sum(sse);
        if (lane == 0) part[v] = total;
      }
      const int next = W == 1 ? v + 1 : v < W ? 2 * W - 1 - v : kRfGroups;
      if (next >= kRfGroups || next * kStep >= a.B) break;
      wave_sync();
      for (int i = lane; i < 4 * n_sums; i += kWave)
        kept[i] = v > 0 && W == 1 ? kept[i] + folded(acc, i) : folded(acc, i);
      wave_sync();
      for (int r = 0; r < n_sums; ++r) acc[r * kWave + lane] = 0.0f;
      v = next;
    }
  };
  const int file = n + q.nc;
  const int K = file <= 48 && a.B > kRfWide ? 4 : file <= 96 && a.B > kWave ? 2 : 1;
  if (K == 4)
    steps(std::integral_constant<int, 4>{});
  else if (K == 2)
    steps(std::integral_constant<int, 2>{});
  else
    steps(std::integral_constant<int, 1>{});
  const int groups = min(kRfGroups, (a.B + K * kWave - 1) / (K * kWave));
  __syncthreads();
  for (int i = tid; i < 4 * n_sums; i += T) {
    float total = 0.0f;
    for (int v = kFold && W == 1 ? max(groups - 2, 0) : 0; v < groups; ++v) {
      const int w = v < W ? v : 2 * W - 1 - v;  // the wavefront of group v
      const float* rows = acc_all + (kFold ? W == 1 ? 0 : w : v) * kRows * kWave;
      const bool before = W == 1 ? v + 1 < groups : v < W && 2 * W - 1 - v < groups;
      total += kFold && before ? rows[kRfSums * kWave + i] : folded(rows, i);
    }
    const int of = sums_of[i >> 2];
    const int2 at = node[of & 0xff];
    const int term = (of >> 8) * 4 + sum_of_quarter(i & 3) - 1;  // -1: the bias
    const int e0 = (at.y & 0xffff) / (int)sizeof(int2), ne = at.y >> 16;
    if (term < 0)
      a.db[nb + order[nb + at.x]] = total;
    else if (term < ne)
      a.dW[cb + edge_row[cb + e0 + term]] = total;
  }
  if (a.loss && tid == 0) {
    float total = 0.0f;
    for (int v = 0; v < groups; ++v) total += part[v];
    a.loss[g] = a.scale * total;
  }
}

}  // namespace

int launch_backward(const tn_population& p, const tn_transformed& t, const float* obs,
                    int64_t obs_stride, int B, const float* dY, int64_t dY_stride,
                    const float* target, int64_t target_stride, float scale, float* loss,
                    float* dW, float* db, hipStream_t stream) {
  // The LDS adjoint holds N_max rows of values and of gradients; above the
  // device's LDS (N_max beyond about 300) it only writes NaN for the genomes
  // the register-file adjoint leaves to it, and the call still succeeds.
  size_t lds = bwd_lds(p.N_max, p.C_max, p.n_in + p.n_out).bytes;
  int rc = allow_lds((const void*)backward_kernel, lds);
  const int lds_ok = rc == TN_OK;
  if (rc == TN_EUNSUPPORTED) {
    lds = 0;
    rc = TN_OK;
  }
  if (rc != TN_OK || p.P == 0) return rc;
  // The low limits hold where the LDS adjoint cannot run (the documented ones: a
  // larger genome's gradients are NaN there), and where genomes may exceed the
  // register file while the LDS adjoint holds the whole population at once: its
  // time is then one genome's, and the register kernel's is added to it (200
  // genomes of 55 to 75 positions, 40 observations: 62 us, 109 with the high
  // limits; 1200 of them, 300 observations: 682 us, 458 with the high limits).
  const bool full = lds_ok && (p.N_max <= kRfPos ||
                               p.P > kComputeUnits * (int64_t)(max_dynamic_lds() / lds));
  BwdArgs a{obs_stride, B, dY, dY_stride, target, target_stride, scale, loss, dW, db,
            full ? kRfPos : kRfPosLow, full ? kRfEdges : kRfEdgesLow};
  // Wavefronts per genome; none of a result's bits follow them. With few genomes
  // one for every tile, up to a group each. Else as many as the usual genomes
  // have steps (of two tiles, of four beyond kRfWide observations), the groups of
  // the others folded in turn: three wavefronts that share four groups took 227 us
  // for 1000 genomes of 600 observations, four 159. One where the genomes alone
  // fill the chip's 2048 several times.
  const int tiles = std::max(1, (B + kWave - 1) / kWave);
  int waves = std::min(kRfWaves, tiles);
  if (p.P > 8192)
    waves = 1;
  else if (p.P > 512 && tiles <= (p.P > 4000 ? 12 : 8))
    waves = tiles <= 2 ? 1 : p.P <= 4000 && (tiles == 5 || tiles == 6) ? 3 : 2;
  const bool fold = waves < std::min(kRfGroups, tiles);
  const auto kern = fold ? backward_rf_kernel<true> : backward_rf_kernel<false>;
  const size_t rf_lds = sizeof(float) * (size_t)waves * (fold ? kRfRows : kRfSums) * kWave;
  rc = allow_lds((const void*)kern, rf_lds);
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(kern, dim3(p.P), dim3(kWave * waves), rf_lds, stream, make_view(p),
                     t.status, t.n_valid, t.order, t.row_ptr, t.edge_src,
                     reinterpret_cast<const int32_t*>(t.edge_w), t.edge_row, t.pos_fn,
                     reinterpret_cast<const int32_t*>(t.pos_bias),
                     reinterpret_cast<const int32_t*>(t.pos_resp), t.io_pos, obs, a);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(backward_kernel, dim3(p.P), dim3(kWave), lds, stream, make_view(p), t.status,
                     t.n_valid, t.order, t.row_ptr, t.edge_src,
                     reinterpret_cast<const int32_t*>(t.edge_w), t.edge_row, t.pos_fn,
                     reinterpret_cast<const int32_t*>(t.pos_bias),
                     reinterpret_cast<const int32_t*>(t.pos_resp), t.io_pos, obs, a, lds_ok);
  return check_launch();
}

}  // namespace tn
