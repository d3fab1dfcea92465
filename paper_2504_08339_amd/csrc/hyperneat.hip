// HyperNEAT over a grid substrate (the indirect encoding among TensorNEAT's
// algorithms, Section 4.4): every CPPN genome is queried at all source /
// target pairs of a grid substrate, the result is thresholded and rounded to
// bfloat16, and the substrate then runs as a dense two-layer network on the
// matrix cores.
//
//   query    one lane = one substrate connection (s -> t): the CPPN's inputs
//            (x_s, y_s, x_t, y_t, 1) are computed from the indices and its
//            program runs in registers, nodes that see only sources or only
//            targets once for many connections; weights are stored transposed, w1t[t][s] and w2t[j][s], so that
//            both GEMM operands are contiguous along the reduction index.
//   hidden   H = tanh(X W1): v_mfma_f32_16x16x32_bf16, a workgroup of four
//            wavefronts per 128 x 128 tile of H with K staged through LDS,
//            fp32 accumulation, tanh in the epilogue.
//   output   Y = bf16(H) W2 with fp32 accumulation in ascending t.
// Geometry: an n x n grid layer has node n*r + c at (-1 + 2c/(n-1),
// -1 + 2r/(n-1)); output j of m sits at (-1 + 2j/(m-1), 0).
#include <algorithm>

#include "fwd_reg.hpp"
#include "rf_file.hpp"
#include "tn_internal.hpp"

namespace tn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

struct SubGeom {
  int grid;    // n: the grid layers are n x n
  int S;       // n * n
  int n_out;   // m
  float thr;   // |w| < thr -> 0
  float step;  // 2 / (n - 1)
  float ostep; // 2 / (m - 1)
};

// float32 -> bfloat16 bits, round to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t bf16_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float bf16_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ------------------------------------------------------------------ query

// Workgroups over (genome, chunk of query units); each wavefront takes
// `per_wave` consecutive units of 4 x 64 queries and runs the CPPN's packed
// program on them with the register engine's walk (a register file of 50 rows
// per tile, four tiles under each index window). Queries 0 .. S*S-1 fill w1t
// (t = q / S, s = q % S), the next S*m fill w2t (j, s); S*S is a multiple of
// 4096, so a unit lies in one of the two.
constexpr int kQueryRows = 50;

__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(TN_RF_BASE))) void
cppn_query_kernel(PopView pop, const int32_t* __restrict__ status,
                  const int32_t* __restrict__ prog_rows, const int32_t* __restrict__ n_valid,
                  const int4* __restrict__ prog_node, const int2* __restrict__ prog_edge,
                  const int32_t* __restrict__ prog_rec, const int32_t* __restrict__ io_pos,
                  SubGeom sg, int n_chunks, int per_wave, uint16_t* __restrict__ w1t,
                  uint16_t* __restrict__ w2t, float* __restrict__ raw1, float* __restrict__ raw2) {
  constexpr int R = kQueryRows, K = rf_tiles(kQueryRows), kUnit = K * kWave;
  rf_reserve<R>();
  const int lane = lane_id();
  const int wave = wave_id();
  const int W = blockDim.x / kWave;
  const int g = blockIdx.x / n_chunks;
  const int chunk = blockIdx.x - g * n_chunks;
  const int Q1 = sg.S * sg.S, Q = Q1 + sg.S * sg.n_out;  // < 2^31 (checked on the host)
  const int n_units = (Q + kUnit - 1) / kUnit;
  const int u0 = (chunk * W + wave) * per_wave;
  const int u1 = min(u0 + per_wave, n_units);
  const bool bad = status[g] != 0 || prog_rows[g] > R;
  const int nn = n_valid[g] - pop.n_in;
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g));
  const int32_t* rec = prog_rec + nb * 16;
  const int2* pe = prog_edge + cb;
  const int nio = pop.n_in + pop.n_out;
  const int out_row =
      bad ? 0 : ((prog_node[nb + io_pos[(int64_t)g * nio + pop.n_in]].y >> 16) & 0x7fff);
  uint16_t* W1 = w1t + (int64_t)g * Q1;
  uint16_t* W2 = w2t + (int64_t)g * sg.S * sg.n_out;
  float* R1 = raw1 ? raw1 + (int64_t)g * Q1 : nullptr;
  float* R2 = raw2 ? raw2 + (int64_t)g * sg.S * sg.n_out : nullptr;
  const int step_r = kWave / sg.grid, step_c = kWave - step_r * sg.grid;  // 64 = step_r grid + step_c
  for (int u = u0; u < u1; ++u) {
    const bool first = u * kUnit < Q1;
    const int base = first ? u * kUnit : u * kUnit - Q1;
    float y[K];
    if (bad) {
#pragma unroll
      for (int k = 0; k < K; ++k) y[k] = __builtin_nanf("");
    } else {
      // the CPPN's inputs (x_s, y_s, x_t, y_t, 1) at rows 0..4 of every tile
      // query qq = tgt * S + src, src = rs * grid + cs, tgt = rt * grid + ct:
      // divided once for the unit's first tile, then stepped by 64 queries
      // per tile (S is a multiple of 64, so src wraps at most once a step)
      float xs[K], ys[K], xt[K], yt[K], one[K];
      const int q0 = base + lane;
      int tgt = q0 / sg.S;
      int src = q0 - tgt * sg.S;
      int rs = src / sg.grid, cs = src - rs * sg.grid;
      int rt = tgt / sg.grid, ct = tgt - rt * sg.grid;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        xs[k] = fmaf((float)cs, sg.step, -1.0f);
        ys[k] = fmaf((float)rs, sg.step, -1.0f);
        if (first) {
          xt[k] = fmaf((float)ct, sg.step, -1.0f);
          yt[k] = fmaf((float)rt, sg.step, -1.0f);
        } else {
          xt[k] = sg.n_out > 1 ? fmaf((float)tgt, sg.ostep, -1.0f) : 0.0f;
          yt[k] = 0.0f;
        }
        one[k] = 1.0f;
        src += kWave;
        rs += step_r;
        cs += step_c;
        if (cs >= sg.grid) {
          cs -= sg.grid;
          ++rs;
        }
        if (src >= sg.S) {
          src -= sg.S;
          rs -= sg.grid;
          ++tgt;
          if (++ct == sg.grid) {
            ct = 0;
            ++rt;
          }
        }
      }
      rfk_set<R>(0, xs);
      rfk_set<R>(1, ys);
      rfk_set<R>(2, xt);
      rfk_set<R>(3, yt);
      rfk_set<R>(4, one);
      walk_records<R>(rec, pe, nn, lane);
      rfk_get<R>(out_row, y);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int qq = base + k * kWave + lane;
      const uint16_t wb = bf16_bits(fabsf(y[k]) < sg.thr ? 0.0f : y[k]);
      if (first) {
        W1[qq] = wb;
        if (R1) R1[qq] = y[k];
      } else if (qq < sg.S * sg.n_out) {
        W2[qq] = wb;
        if (R2) R2[qq] = y[k];
      }
    }
  }
}

// ------------------------------------------------ CPPN over the substrate
//
// The query and its adjoint walk a CPPN at every (source, target) pair. A
// wavefront takes 64 sources (lane = source) and a run of targets, K targets
// (the tiles of a register file) at a time, so a node's in-edges say how often
// it has to be evaluated:
//   fixed    it depends on no target coordinate: once per wavefront;
//   target   on no source coordinate: once for up to 64 targets (lane =
//            target), then read back from LDS, one broadcast per step;
//   both     at every step.
// The same operations in the same order give every value its bits.
struct CppnWave {
  const int2* edge;  // LDS: the source's row, weight; 64 more are readable
  uint64_t fixed, target, both;  // positions
  int l_fn, l_bias, l_resp;      // of position `lane`
  int l_edge;                    // first in-edge | in-edges << 16
  int l_row;                     // row in the file
  int n_rows;                    // rows of computed nodes (inputs come after them), if kGrad
  int in_row[5];                 // rows of the inputs
  int op;                        // the output's position
  int n_kept;                    // target coordinates (2) and target nodes
};

// An activation whose slope needs the pre-activation keeps it in a row.
__device__ __forceinline__ int node_width(int f) { return 2 + (slope_needs_z(f & 7) ? 1 : 0); }

// By all threads of a workgroup; n <= 64 positions. kGrad: a node takes
// node_width rows and the inputs' rows follow; else position p takes row p.
template <bool kGrad>
__device__ __forceinline__ CppnWave cppn_program(int n, int n_edges, const int32_t* rp,
                                                 const int32_t* edge_src, const int32_t* w_bits,
                                                 const int32_t* fn, const int32_t* bias_bits,
                                                 const int32_t* resp_bits, const int32_t* io,
                                                 int slots, int2* edge) {
  const int lane = lane_id(), tid = threadIdx.x, T = blockDim.x;
  CppnWave c;
  c.edge = edge;
  c.l_fn = lane < n ? fn[lane] : -1;
  c.l_bias = lane < n ? bias_bits[lane] : 0;
  c.l_resp = lane < n ? resp_bits[lane] : 0;
  const int start = lane < n ? rp[lane] : 0, end = lane < n ? rp[lane + 1] : 0;
  c.l_edge = start | ((end - start) << 16);
  const uint64_t nodes = __ballot(c.l_fn >= 0);
  const uint64_t inputs = __ballot(lane < n && c.l_fn < 0);
  c.n_rows = 0;
  if (kGrad) {
    const int width = c.l_fn >= 0 ? node_width(c.l_fn) : 0;
    const int upto = wave_inclusive_scan(width);
    c.n_rows = __builtin_amdgcn_readlane(upto, kWave - 1);
    c.l_row = c.l_fn >= 0 ? upto - width : c.n_rows + mbcnt(inputs);
  } else {
    c.l_row = lane;
  }
  for (int e0 = 0; e0 < n_edges; e0 += T) {  // whole wavefronts: the shuffle
    const int e = e0 + tid;
    const int q = e < n_edges ? edge_src[e] : 0;
    const int row = __shfl(c.l_row, q, kWave);
    if (e < n_edges) edge[e] = make_int2(row, w_bits[e]);
  }
  const int first_src = lane < n_edges ? edge_src[lane] : 0;  // the first 64 edges' sources
  uint64_t on_src = 0, on_tgt = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int p = io[i];
    c.in_row[i] = __builtin_amdgcn_readlane(c.l_row, p);
    if (i < 2) on_src |= (uint64_t)1 << p;
    else if (i < 4) on_tgt |= (uint64_t)1 << p;
  }
  c.op = io[5];
  for (uint64_t m = nodes; m; m &= m - 1) {
    const int p = __builtin_ctzll(m);
    const int le = __builtin_amdgcn_readlane(c.l_edge, p);
    const int e0 = le & 0xffff, e1 = e0 + (le >> 16);
    bool s = false, t = false;
    if (lane >= e0 && lane < e1) {
      s = (on_src >> first_src) & 1;
      t = (on_tgt >> first_src) & 1;
    }
    for (int e = max(e0, kWave) + lane; e < e1; e += kWave) {
      const int q = edge_src[e];
      s |= (on_src >> q) & 1;
      t |= (on_tgt >> q) & 1;
    }
    if (__ballot(s)) on_src |= (uint64_t)1 << p;
    if (__ballot(t)) on_tgt |= (uint64_t)1 << p;
  }
  c.fixed = nodes & ~on_tgt;
  c.target = nodes & on_tgt & ~on_src;
  // those that fit the slots, in topological order, are kept in LDS; the others
  // run at every step
  uint64_t kept = 0;
  c.n_kept = 2;
  for (; c.n_kept < slots && c.target; ++c.n_kept) {
    kept |= c.target & -c.target;
    c.target &= c.target - 1;
  }
  c.target = kept;
  c.both = nodes & ~c.fixed & ~c.target;
  return c;
}

__device__ __forceinline__ int2 cppn_edges(const CppnWave& c, int p) {
  return c.edge[(__builtin_amdgcn_readlane(c.l_edge, p) & 0xffff) + lane_id()];
}

// Pre-activations of the computed position p in K tiles; ed: cppn_edges(p).
// kAny: every aggregation and any number of in-edges, else sum or mean of at
// most 64.
template <class F, int K, bool kAny>
__device__ __forceinline__ void cppn_pre(const CppnWave& c, int p, int2 ed, float (&z)[K]) {
  const int f = __builtin_amdgcn_readlane(c.l_fn, p);
  const int le = __builtin_amdgcn_readlane(c.l_edge, p);
  const int ne = le >> 16, agg = (f >> 8) & 0xff;
  auto row = [&](int e) { return __builtin_amdgcn_readlane(ed.x, e); };
  auto weight = [&](int e) { return __int_as_float(__builtin_amdgcn_readlane(ed.y, e)); };
  float s[K];
#pragma unroll
  for (int k = 0; k < K; ++k) s[k] = 0.0f;
  if (!kAny || agg == TN_AGG_SUM) {
    const int n0 = kAny ? min(ne, kWave) : ne;
    if (n0 > 0) {
      F::fma_v(s, weight(0), row(0));
      if (n0 > 1) {
        F::fma_v(s, weight(1), row(1));
        for (int e = 2; e < n0; ++e) F::fma_v(s, weight(e), row(e));
      }
    }
    if (kAny)
      for (int b = kWave; b < ne; b += kWave) {
        ed = c.edge[(le & 0xffff) + b + lane_id()];
        for (int e = 0; e < min(ne - b, kWave); ++e) F::fma_v(s, weight(e), row(e));
      }
    if (!kAny && agg == TN_AGG_MEAN && ne > 0)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        s[k] = s[k] / (float)ne;
        asm volatile("" : "+v"(s[k]));
      }
  } else if (ne > 0) {
    // other aggregations: terms in order
    for (int b = 0; b < ne; b += kWave) {
      if (b) ed = c.edge[(le & 0xffff) + b + lane_id()];
      for (int e = 0; e < min(ne - b, kWave); ++e) {
        float x[K];
        F::get_v(row(e), x);
        const float w = weight(e);
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma clang fp contract(off)
          const float t = w * x[k];
          if (b + e == 0) {
            s[k] = t;
            continue;
          }
          switch (agg) {
            case TN_AGG_PRODUCT: s[k] = s[k] * t; break;
            case TN_AGG_MAX: s[k] = fmaxf(s[k], t); break;
            case TN_AGG_MIN: s[k] = fminf(s[k], t); break;
            case TN_AGG_MEAN: s[k] = s[k] + t; break;
            default: s[k] = fabsf(t) > fabsf(s[k]) ? t : s[k]; break;  // maxabs
          }
        }
      }
    }
    if (agg == TN_AGG_MEAN)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        s[k] = s[k] / (float)ne;
        asm volatile("" : "+v"(s[k]));
      }
  }
  const float rho = __int_as_float(__builtin_amdgcn_readlane(c.l_resp, p));
  const float bias = __int_as_float(__builtin_amdgcn_readlane(c.l_bias, p));
#pragma unroll
  for (int k = 0; k < K; ++k) z[k] = fmaf(rho, s[k], bias);
}

// f(p, its in-edges) for every position of `m`, in topological order, the next
// position's in-edges read ahead.
template <class Fn>
__device__ __forceinline__ void cppn_forward(const CppnWave& c, uint64_t m, Fn f) {
  if (!m) return;
  int p = __builtin_ctzll(m);
  int2 ed = cppn_edges(c, p);
  for (;;) {
    m &= m - 1;
    const int next = m ? __builtin_ctzll(m) : p;
    const int2 en = cppn_edges(c, next);
    f(p, ed);
    if (!m) break;
    p = next;
    ed = en;
  }
}
template <class Fn>
__device__ __forceinline__ void cppn_reverse(const CppnWave& c, uint64_t m, Fn f) {
  if (!m) return;
  int p = 63 - __builtin_clzll(m);
  int2 ed = cppn_edges(c, p);
  for (;;) {
    m ^= (uint64_t)1 << p;
    const int next = m ? 63 - __builtin_clzll(m) : p;
    const int2 en = cppn_edges(c, next);
    f(p, ed);
    if (!m) break;
    p = next;
    ed = en;
  }
}

// Coordinates: source s of the grid, target t of the hidden grid or of the
// output row.
__device__ __forceinline__ void source_xy(const SubGeom& sg, int s, float* x, float* y) {
  const int r = s / sg.grid, c = s - r * sg.grid;
  *x = fmaf((float)c, sg.step, -1.0f);
  *y = fmaf((float)r, sg.step, -1.0f);
}
__device__ __forceinline__ void target_xy(const SubGeom& sg, bool hidden, int t, float* x,
                                          float* y) {
  if (hidden) {
    source_xy(sg, t, x, y);
  } else {
    *x = sg.n_out > 1 ? fmaf((float)t, sg.ostep, -1.0f) : 0.0f;
    *y = 0.0f;
  }
}

// A wavefront's part: sources s0 .. s0 + 63, targets t0 .. t1 - 1 of the
// hidden grid or the outputs. Items of a genome run over the blocks of sources,
// then over the runs of `per` targets.
struct CppnItem {
  bool hidden;
  int s0, t0, t1;
};
__host__ __device__ inline int cppn_items(const SubGeom& sg, int per) {
  return (sg.S / kWave) * ((sg.S + per - 1) / per + (sg.n_out + per - 1) / per);
}
__device__ __forceinline__ CppnItem cppn_item(const SubGeom& sg, int per, int item) {
  const int blocks = sg.S / kWave, runs = (sg.S + per - 1) / per;
  const int run = item / blocks;
  CppnItem it;
  it.s0 = (item - run * blocks) * kWave;
  it.hidden = run < runs;
  it.t0 = (it.hidden ? run : run - runs) * per;
  it.t1 = min(it.t0 + per, it.hidden ? sg.S : sg.n_out);
  return it;
}

// The query for populations of at most kMapRows node rows (one row of the file
// each): four targets a step for genomes of up to 20 positions, else two. Bound
// by instruction issue (activations and in-edge windows). 200 CPPNs (33
// in-edges, 11 computed nodes) over a 32 x 32 grid and 8 outputs: 1348 us; 2181
// us in cppn_query_kernel, which evaluates every node at every pair with two
// wavefronts per SIMD. With this walk on a file of 48 rows for
// four tiles (two wavefronts per SIMD) 1841 us, of 28 rows (three) 1493 us.
constexpr int kMapRows = 32, kMapWaves = 4;
// Targets per wavefront, at most, and the wavefronts that make it fewer: 200 CPPNs
// over a 32 x 32 grid run 64 each (1420 us with 128, 1348 with 64: the last round
// is shorter). Rows of the table.
constexpr int kMapRun = 128, kMapWavesWanted = 32768, kMapSlots = 16;

template <int K>
__device__ __forceinline__ void cppn_map(const CppnWave& c, const SubGeom& sg, const CppnItem& it,
                                         float (*table)[kMapRun], uint16_t* __restrict__ W,
                                         float* __restrict__ R) {
  using F = ShortFiles<K>;
  const int lane = lane_id();
  const int runs = it.t1 - it.t0;
  // Step -2 evaluates the fixed nodes, step -1 (lane = target, in two tiles) the
  // target nodes, the others K targets each: one walk in the code for all.
  for (int step = -2; step * K < runs; ++step) {
    const int t = step * K;
    float v[K];
    uint64_t nodes = c.both;
    if (step < -1) {
      float x0, y0, one = 1.0f;
      asm volatile("" : "+v"(one));
      source_xy(sg, it.s0 + lane, &x0, &y0);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = x0;
      F::set_v(c.in_row[0], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = y0;
      F::set_v(c.in_row[1], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = one;
      F::set_v(c.in_row[4], v);
      nodes = c.fixed;
    } else if (step < 0) {
      float x[2], y[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        target_xy(sg, it.hidden, min(it.t0 + k * kWave + lane, it.t1 - 1), &x[k], &y[k]);
        table[0][k * kWave + lane] = x[k];
        table[1][k * kWave + lane] = y[k];
      }
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = x[k % 2];
      F::set_v(c.in_row[2], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = y[k % 2];
      F::set_v(c.in_row[3], v);
      nodes = c.target;
    } else {
      uint64_t m = c.target;
      for (int slot = 0; slot < c.n_kept; ++slot) {
        const int row = slot == 0 ? c.in_row[2] : slot == 1 ? c.in_row[3] : __builtin_ctzll(m);
        if (slot >= 2) m &= m - 1;
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = table[slot][t + k];
        F::set_v(row, v);
      }
    }
    int slot = 2;
    cppn_forward(c, nodes, [&](int p, int2 ed) __attribute__((always_inline)) {
      float z[K];
      cppn_pre<F, K, true>(c, p, ed, z);
      activate_all<K>(__builtin_amdgcn_readlane(c.l_fn, p) & 7, z, v);
      F::set_v(p, v);
      if (step == -1) {
#pragma unroll
        for (int k = 0; k < 2; ++k) table[slot][k * kWave + lane] = v[k];
        ++slot;
      }
    });
    if (step < 0) continue;
    F::get_v(c.op, v);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (t + k >= runs) break;
      const int64_t q = (int64_t)(t + k) * sg.S + lane;
      W[q] = bf16_bits(fabsf(v[k]) < sg.thr ? 0.0f : v[k]);
      if (R) R[q] = v[k];
    }
  }
}

__global__ __launch_bounds__(kWave * kMapWaves) __attribute__((amdgpu_num_vgpr(TN_RF_SHORT / 2))) void
cppn_map_kernel(PopView pop, const int32_t* __restrict__ status,
                const int32_t* __restrict__ n_valid, const int32_t* __restrict__ row_ptr,
                const int32_t* __restrict__ edge_src,
                const int32_t* __restrict__ w_bits, const int32_t* __restrict__ fn,
                const int32_t* __restrict__ bias_bits, const int32_t* __restrict__ resp_bits,
                const int32_t* __restrict__ io_pos, SubGeom sg, int run, int wg_per_g,
                uint16_t* __restrict__ w1t, uint16_t* __restrict__ w2t, float* __restrict__ raw1,
                float* __restrict__ raw2) {
  short_file_reserve();
  extern __shared__ int2 map_edge[];
  __shared__ __align__(16) float table_all[kMapWaves][kMapSlots][kMapRun];
  const int lane = lane_id(), wave = wave_id();
  const int g = blockIdx.x / wg_per_g;
  const int item = (blockIdx.x - g * wg_per_g) * kMapWaves + wave;
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g)),
                rb = uniform64(pop.rowptr_base(g));
  const bool bad = status[g] != 0;
  const int n = n_valid[g];
  CppnWave c{};
  if (!bad) {
    c = cppn_program<false>(n, row_ptr[rb + n], row_ptr + rb, edge_src + cb, w_bits + cb, fn + nb,
                            bias_bits + nb, resp_bits + nb,
                            io_pos + (int64_t)g * (pop.n_in + pop.n_out), kMapSlots, map_edge);
  }
  __syncthreads();
  if (item >= cppn_items(sg, run)) return;
  const CppnItem it = cppn_item(sg, run, item);
  const int64_t Q1 = (int64_t)sg.S * sg.S, Q2 = (int64_t)sg.S * sg.n_out;
  const int64_t at = (it.hidden ? g * Q1 : g * Q2) + (int64_t)it.t0 * sg.S + it.s0;
  uint16_t* W = (it.hidden ? w1t : w2t) + at;
  float* R = it.hidden ? raw1 : raw2;
  if (R) R += at;
  if (bad) {
    for (int t = 0; t < it.t1 - it.t0; ++t) {
      W[(int64_t)t * sg.S + lane] = bf16_bits(__builtin_nanf(""));
      if (R) R[(int64_t)t * sg.S + lane] = __builtin_nanf("");
    }
  } else if (n <= kShortFileRows / 4) {
    cppn_map<4>(c, sg, it, table_all[wave], W, R);
  } else {
    cppn_map<2>(c, sg, it, table_all[wave], W, R);
  }
}

// ----------------------------------------------------------------- hidden

// Batched C[g][m][n] = sum_k A[g][m][k] * B[g][n][k] (bfloat16 operands, both
// contiguous along k; float32 accumulation). A workgroup of four wavefronts
// computes a 128 x 128 tile of C, each wavefront a 64 x 64 quarter with MFMA
// 16x16x32. K runs in stages of 64: while the wavefronts multiply from one LDS
// buffer, every thread fetches its 16-byte chunks of the next stage's A and B
// rows into registers and then writes them to the other buffer, one barrier
// per stage. Rows m >= M, n >= N and columns k >= K read zeros and are not
// stored; K is a multiple of 32. kTanh applies tanh in the epilogue (the
// substrate's hidden layer). The tiles of one batch entry are consecutive
// workgroups kept on one XCD, so its operands come from HBM once.
struct GemmArgs {
  const uint16_t* a;
  int64_t lda, a_batch;
  const uint16_t* b;
  int64_t ldb, b_batch;
  float* c;
  int64_t ldc, c_batch;
  int M, N, K;
  int m_tiles, n_tiles;
  int64_t n_items;
};

constexpr int kGemmTile = 128;              // rows of C per workgroup, both ways
constexpr int kGemmKs = 64;                 // k per stage
constexpr int kGemmRow = kGemmKs + 8;       // bf16 per LDS row (16 bytes of padding)
constexpr int kGemmBuf = kGemmTile * kGemmRow;  // bf16 per operand buffer
constexpr size_t kGemmLds = sizeof(uint16_t) * 4 * kGemmBuf;  // A and B, two buffers each

// Workgroup b of n runs on XCD b mod 8; returns the item it takes so that
// consecutive items share an XCD (the last n mod 8 in order).
__device__ __forceinline__ int64_t gemm_item(int64_t b, int64_t n) {
  constexpr int kXcd = 8;
  const int64_t per = n / kXcd, full = per * kXcd;
  if (b >= full) return b;
  return (b % kXcd) * per + b / kXcd;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes from global memory (the operands arrive as pointers in a struct
// argument, whose address space the compiler cannot infer)
__device__ __forceinline__ u32x4 load_global16(const uint16_t* q) {
  return *(const __attribute__((address_space(1))) u32x4*)q;
}
__device__ __forceinline__ void store_global(float* q, float v) {
  *(__attribute__((address_space(1))) float*)q = v;
}

// Stores a wavefront's 64 x 64 quarter of C. The fragment of D = C^T holds rows
// 4 (lane / 16) + e, column lane % 16: C row row0 (+ 16 i), columns col0 (+ 16 j)
// + e.
template <bool kTanh>
__device__ __forceinline__ void store_tile(const GemmArgs& p, const f32x4 (&acc)[4][4], float* C,
                                           int row0, int col0) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = row0 + 16 * i, col = col0 + 16 * j;
      if (row >= p.M) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = kTanh ? act_tanh(acc[i][j][e]) : acc[i][j][e];
      float* q = C + (int64_t)row * p.ldc + col;
      if (col + 3 < p.N && (p.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0) {
        f32x4 w = {v[0], v[1], v[2], v[3]};
        *(__attribute__((address_space(1))) f32x4*)q = w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < p.N) store_global(q + e, v[e]);
      }
    }
}

template <bool kTanh>
__global__ __launch_bounds__(256) void gemm_nt_kernel(GemmArgs p) {
  extern __shared__ __align__(16) uint16_t gemm_lds[];
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int64_t item = gemm_item(blockIdx.x, gridDim.x);
  const int per_g = p.m_tiles * p.n_tiles;
  const int g = (int)(item / per_g);
  const int r = (int)(item - (int64_t)g * per_g);
  const int nt = r / p.m_tiles, mt = r - nt * p.m_tiles;
  const int m0 = mt * kGemmTile, n0 = nt * kGemmTile;
  const uint16_t* A = p.a + (int64_t)g * p.a_batch;
  const uint16_t* Bm = p.b + (int64_t)g * p.b_batch;
  uint16_t* sa = gemm_lds;                 // [2][kGemmBuf]
  uint16_t* sb = gemm_lds + 2 * kGemmBuf;  // [2][kGemmBuf]

  // this thread's chunks of a stage: chunk c = tid + 256 u is row c / 8,
  // k (c % 8) * 8 .. + 7 of the stage
  constexpr int kChunks = kGemmTile * kGemmKs / 8 / 256;
  struct Regs {
    u32x4 a[kChunks], b[kChunks];
  };
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  auto fetch = [&](int st, Regs& r) {
    const int k0 = st * kGemmKs;
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
      const int c = tid + 256 * u, row = c >> 3, k = k0 + (c & 7) * 8;
      const bool kin = k < p.K;
      r.a[u] = m0 + row < p.M && kin ? load_global16(A + (int64_t)(m0 + row) * p.lda + k) : zero4;
      r.b[u] = n0 + row < p.N && kin ? load_global16(Bm + (int64_t)(n0 + row) * p.ldb + k) : zero4;
    }
  };
  auto stash = [&](int buf, const Regs& r) {
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
      const int c = tid + 256 * u, at = (c >> 3) * kGemmRow + (c & 7) * 8;
      *reinterpret_cast<u32x4*>(sa + buf * kGemmBuf + at) = r.a[u];
      *reinterpret_cast<u32x4*>(sb + buf * kGemmBuf + at) = r.b[u];
    }
  };

  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;  // this wavefront's quarter
  const int li = lane & 15, kq = (lane >> 4) * 8;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;
  auto multiply = [&](int buf) {
    const uint16_t* pa = sa + buf * kGemmBuf + (wm + li) * kGemmRow + kq;
    const uint16_t* pb = sb + buf * kGemmBuf + (wn + li) * kGemmRow + kq;
#pragma unroll
    for (int kk = 0; kk < kGemmKs; kk += 32) {
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        fa[i] = *reinterpret_cast<const bf16x8*>(pa + 16 * i * kGemmRow + kk);
        fb[i] = *reinterpret_cast<const bf16x8*>(pb + 16 * i * kGemmRow + kk);
      }
      // B as the first operand: the fragment is the 16 x 16 block of C
      // transposed, so a lane ends up with four consecutive columns of a row
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  };
  // Stage st sits in LDS buffer st % 2 while the wavefronts multiply it; the
  // next stage is requested to registers before the multiply and written to
  // the other buffer after it, which was last read before the previous
  // barrier. (Two stages in flight need a second register set: 352 registers,
  // one wavefront per SIMD, or spills when held to two.)
  const int n_stages = (p.K + kGemmKs - 1) / kGemmKs;
  Regs rg;
  fetch(0, rg);
  stash(0, rg);
  __syncthreads();
  for (int st = 0; st < n_stages; ++st) {
    const int buf = st & 1;
    const bool more = st + 1 < n_stages;
    if (more) fetch(st + 1, rg);
    multiply(buf);
    if (more) stash(buf ^ 1, rg);
    __syncthreads();
  }
  store_tile<kTanh>(p, acc, p.c + (int64_t)g * p.c_batch, m0 + wm + li, n0 + wn + (lane >> 4) * 4);
}

// The same product with operands that are 16-byte aligned in every row: stages
// of 32 k (16 KB) arrive by LDS-direct loads, kRing buffers deep, so four
// stages per workgroup are in flight without a register (gemm_nt_kernel: one,
// in registers). A row's 64 bytes of a stage are four lanes' loads, and a
// fragment read of a wavefront then is 1 KB of consecutive LDS: no bank
// conflicts, no padding. One barrier per stage: it tells that every
// wavefront's part of stage st has landed and that stage st - 1 is no longer
// read, so stage st + 4 takes its buffer. Rows past M and N read the last row
// and are not stored. Bound by memory: 200 genomes, 128 x 1024 x 1024 (577 MB)
// 165 us, 177 us by gemm_nt_kernel. Runs of columns instead of tiles (1600 tiles
// make 3.1 rounds of 512 workgroups) measured 184 us, stages in an order of
// their own per workgroup 167. The order of the sums is gemm_nt_kernel's.
constexpr int kRing = 5, kRingKs = 32;
constexpr int kRingBytes = kGemmTile * kRingKs * 2;  // one operand of a stage
constexpr size_t kRingLds = (size_t)kRing * 2 * kRingBytes;

template <bool kTanh>
__global__ __launch_bounds__(256, 2) void gemm_ring_kernel(GemmArgs p) {
  extern __shared__ __align__(16) uint16_t gemm_lds[];
  const int lane = lane_id(), wave = wave_id();
  const int64_t item = gemm_item(blockIdx.x, gridDim.x);
  const int per_g = p.m_tiles * p.n_tiles;
  const int g = (int)(item / per_g);
  const int r = (int)(item - (int64_t)g * per_g);
  const int nt = r / p.m_tiles, mt = r - nt * p.m_tiles;
  const int m0 = mt * kGemmTile, n0 = nt * kGemmTile;
  const uint16_t* A = p.a + (int64_t)g * p.a_batch + (int64_t)m0 * p.lda;
  const uint16_t* Bm = p.b + (int64_t)g * p.b_batch + (int64_t)n0 * p.ldb;
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(gemm_lds);

  // this wavefront's loads of a stage: rows 32 wave .. + 31 of either operand,
  // 16 rows (1 KB) each
  constexpr int kLoads = 4;
  uint32_t off[kLoads];
#pragma unroll
  for (int u = 0; u < kLoads; ++u) {
    const int row = 32 * wave + 16 * (u & 1) + (lane >> 2);
    const int last = (u < 2 ? p.M - m0 : p.N - n0) - 1;
    off[u] = (uint32_t)(min(row, last) * (int)(u < 2 ? p.lda : p.ldb) * 2 + (lane & 3) * 16);
  }
  auto fetch = [&](int st) {
    const uint32_t at = lds0 + (uint32_t)(st % kRing) * (2 * kRingBytes) + (uint32_t)wave * 2048;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const uint32_t to = __builtin_amdgcn_readfirstlane(at + (u >> 1) * kRingBytes + (u & 1) * 1024);
      const uint16_t* from = (u < 2 ? A : Bm) + st * kRingKs;
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off[u]),
                   "s"(from), "s"(to)
                   : "memory", "m0");
    }
  };

  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;  // this wavefront's quarter
  const int li = lane & 15, kq = (lane >> 4) * 8;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;
  auto multiply = [&](int st) {
    const uint16_t* sa = gemm_lds + (st % kRing) * kRingBytes;  // 2 operands of kRingBytes / 2
    const uint16_t* pa = sa + (wm + li) * kRingKs + kq;
    const uint16_t* pb = sa + kRingBytes / 2 + (wn + li) * kRingKs + kq;
    bf16x8 fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[i] = *reinterpret_cast<const bf16x8*>(pa + 16 * i * kRingKs);
      fb[i] = *reinterpret_cast<const bf16x8*>(pb + 16 * i * kRingKs);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };
  const int n_stages = p.K / kRingKs;
  const int ahead = min(kRing - 1, n_stages);
  for (int st = 0; st < ahead; ++st) fetch(st);
  // the wavefront's loads complete in order: at most those of the later
  // stages that were requested may still be on their way
  for (int st = 0; st < n_stages; ++st) {
    switch (min(kRing - 2, n_stages - 1 - st)) {
      case 3: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
      case 2: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
      case 1: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
      default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
    lds_barrier();
    if (st + kRing - 1 < n_stages) fetch(st + kRing - 1);
    multiply(st);
  }
  store_tile<kTanh>(p, acc, p.c + (int64_t)g * p.c_batch, m0 + wm + li, n0 + wn + (lane >> 4) * 4);
}

template <bool kTanh>
int launch_gemm(GemmArgs p, int batch, hipStream_t stream) {
  p.m_tiles = (p.M + kGemmTile - 1) / kGemmTile;
  p.n_tiles = (p.N + kGemmTile - 1) / kGemmTile;
  p.n_items = (int64_t)batch * p.m_tiles * p.n_tiles;
  // LDS-direct loads take 16-byte pieces of every row: both operands aligned
  const bool ring = ((reinterpret_cast<uintptr_t>(p.a) | reinterpret_cast<uintptr_t>(p.b)) & 15) == 0 &&
                    ((p.lda | p.ldb | p.a_batch | p.b_batch) & 7) == 0;
  const auto kern = ring ? gemm_ring_kernel<kTanh> : gemm_nt_kernel<kTanh>;
  const size_t lds = ring ? kRingLds : kGemmLds;
  const int rc = allow_lds((const void*)kern, lds);
  if (rc != TN_OK || p.n_items == 0) return rc;
  if (p.n_items > 0x7fffffff) return TN_EUNSUPPORTED;
  hipLaunchKernelGGL(kern, dim3((unsigned)p.n_items), dim3(256), lds, stream, p);
  return check_launch();
}

// ----------------------------------------------------------------- output

// Y[b][j] = sum_t bf16(H[b][t]) w2t[j][t], fp32 accumulation in ascending t, one
// product after the other: the order is part of the result, so the sums are 4 x 4
// outer products on the matrix cores (16 of them for 64 rows and four outputs;
// bfloat16 MFMA adds 32 products at once). A workgroup takes 64 rows b and 16
// outputs j of one genome, a wavefront four of them; t comes in blocks of 64
// through two LDS buffers, kAhead blocks requested ahead. Rows are padded so that
// 16-byte reads down a column of rows touch every bank once. Bound by reading H
// and, for few genomes, by the chain of products: 200 genomes (128 rows, 1024
// hidden units, 8 outputs; 105 MB) 24 us, 135 us with one thread per output
// straight from memory; vector multiply-adds took 27 us, and 19 us for 60 genomes
// with 10 outputs (13 us so), bound by their reads of weights from LDS.
constexpr int kOutRows = kWave, kOutCols = 16, kOutKs = 64, kOutRow = kOutKs + 4;
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void substrate_output_kernel(
    const float* __restrict__ h, const uint16_t* __restrict__ w2t, int S, int B, int m,
    int b_tiles, int j_tiles, float* __restrict__ y) {
  __shared__ __align__(16) float sh[2][kOutRows * kOutRow];
  __shared__ __align__(16) float sw[2][kOutCols * kOutRow];
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int per_g = b_tiles * j_tiles;
  const int g = blockIdx.x / per_g, r = blockIdx.x - g * per_g;
  const int bt = r / j_tiles, jt = r - bt * j_tiles;
  const int b0 = bt * kOutRows, j0 = jt * kOutCols;
  const float* H = h + ((int64_t)g * B + b0) * S;
  const uint16_t* W = w2t + ((int64_t)g * m + j0) * S;

  // this thread's part of a block: four hidden units of four rows and of one
  // output's weights. Loads without a branch, so that older blocks can be waited
  // for alone: past the last block, row and output they read the last, which is
  // not used.
  constexpr int kAhead = 4, kLoads = kOutRows * kOutKs / 4 / 256;
  struct Block {
    f32x4 h[kLoads];
    uint16_t w[4];
  };
  Block in[kAhead];
  const int n_blocks = S / kOutKs;
  const int tr = tid >> 4, tk = (tid & 15) * 4;
  const uint16_t* Wt = W + (int64_t)min(tr, m - j0 - 1) * S + tk;
  auto fetch = [&](int i, Block& q) {
    const int t0 = min(i, n_blocks - 1) * kOutKs;
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      q.h[u] = *reinterpret_cast<const f32x4_any*>(
          H + (int64_t)min(tr + 16 * u, B - b0 - 1) * S + t0 + tk);
#pragma unroll
    for (int e = 0; e < 4; ++e) q.w[e] = Wt[t0 + e];
  };
  auto stash = [&](int i, const Block& q) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      *reinterpret_cast<f32x4*>(sh[i & 1] + (tr + 16 * u) * kOutRow + tk) =
          __builtin_convertvector(__builtin_convertvector(q.h[u], bf16x4), f32x4);
    f32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = bf16_float(q.w[e]);
    *reinterpret_cast<f32x4*>(sw[i & 1] + tr * kOutRow + tk) = w;
  };
  const int jw = j0 + 4 * wave;  // this wavefront's outputs
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};  // of row `lane`
#pragma unroll
  for (int a = 0; a < kAhead; ++a) fetch(a, in[a]);
  stash(0, in[0]);
  fetch(kAhead, in[0]);
  for (int i0 = 0; i0 < n_blocks; i0 += kAhead) {
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int i = i0 + a;
      if (i >= n_blocks) break;
      lds_barrier();
      if (jw < m) {
        const float* ph = sh[i & 1] + lane * kOutRow;
        const float* pw = sw[i & 1] + (4 * wave + (lane & 3)) * kOutRow;
#pragma unroll
        for (int k = 0; k < kOutKs; k += 4) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(ph + k);
          const f32x4 w = *reinterpret_cast<const f32x4*>(pw + k);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(w[e], x[e], acc, 0, 0, 0);
        }
      }
      // the other buffer was last read before the barrier above
      stash(i + 1, in[(a + 1) % kAhead]);
      fetch(i + 1 + kAhead, in[(a + 1) % kAhead]);
    }
  }
  if (b0 + lane >= B) return;
  float* q = y + ((int64_t)g * B + b0 + lane) * m + jw;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (jw + e < m) q[e] = acc[e];
}

// ---------------------------------------------------------------- backward

constexpr int kMaxOutBwd = 32;

// For L = sum(dY * Y), per hidden unit t of genome g (one thread each):
//   dw2t[j][t] = sum_b H[b][t] dY[b][j]                  (ascending b)
//   dz[b][t]   = (sum_j dY[b][j] w2t[j][t]) (1 - H[b][t]^2)
// dz is stored transposed and rounded to bfloat16, dzt[t][b], rows padded
// with zeros to Kp (a multiple of 32) for the weight-gradient GEMM.
__global__ __launch_bounds__(256) void substrate_grad_out_kernel(
    const float* __restrict__ h, const uint16_t* __restrict__ w2t, const float* __restrict__ dy,
    int S, int B, int Kp, int m, int wg_per_g, uint16_t* __restrict__ dzt,
    float* __restrict__ dw2t) {
  extern __shared__ __align__(16) float dys[];
  const int g = blockIdx.x / wg_per_g;
  const int t = (blockIdx.x - g * wg_per_g) * blockDim.x + threadIdx.x;
  const float* D = dy + (int64_t)g * B * m;
  for (int i = threadIdx.x; i < B * m; i += blockDim.x) dys[i] = D[i];
  __syncthreads();
  if (t >= S) return;
  float w2[kMaxOutBwd], acc[kMaxOutBwd];
#pragma unroll
  for (int j = 0; j < kMaxOutBwd; ++j) {
    w2[j] = j < m ? bf16_float(w2t[((int64_t)g * m + j) * S + t]) : 0.0f;
    acc[j] = 0.0f;
  }
  const float* H = h + (int64_t)g * B * S + t;
  uint16_t* Z = dzt + ((int64_t)g * S + t) * Kp;
  for (int b0 = 0; b0 < Kp; b0 += 8) {
    uint16_t pack[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int b = b0 + u;
      float dz = 0.0f;
      if (b < B) {
        const float hb = H[(int64_t)b * S];
        const float* d = dys + b * m;
        float up = 0.0f;
#pragma unroll
        for (int j = 0; j < kMaxOutBwd; ++j)
          if (j < m) {
            up = fmaf(d[j], w2[j], up);
            acc[j] = fmaf(hb, d[j], acc[j]);
          }
        dz = up * fmaf(-hb, hb, 1.0f);
      }
      pack[u] = bf16_bits(dz);
    }
    uint4 v;
    v.x = pack[0] | ((uint32_t)pack[1] << 16);
    v.y = pack[2] | ((uint32_t)pack[3] << 16);
    v.z = pack[4] | ((uint32_t)pack[5] << 16);
    v.w = pack[6] | ((uint32_t)pack[7] << 16);
    *reinterpret_cast<uint4*>(Z + b0) = v;
  }
  for (int j = 0; j < m; ++j) dw2t[((int64_t)g * m + j) * S + t] = acc[j];
}

// Both gradients of the substrate at once for batches of up to kFusedBatch
// rows, the whole reduction of the weight gradient:
//   dw1t[t][s] = sum_b dz[b][t] x[b][s],  dw2t[j][t] = sum_b H[b][t] dY[b][j].
// A workgroup takes 128 hidden units t of one genome and a range of 128-wide
// tiles of s. It computes dz of its units from H, dY and w2t, rounds it to
// bfloat16 and keeps it, transposed, in LDS; then for each tile of s the rows
// of x come through registers into LDS transposed (the next tile is requested
// before this one's MFMAs). So H is read once, and neither dz nor x^T passes
// through memory. Bound by the stores of dw1t and the reads of H and x: 200 genomes
// (32 x 32 grids, 128 rows; 840 MB written, 160 MB read) 284 us, against 445 us in
// three kernels that wrote dz and x^T out.
constexpr int kFusedBatch = 128;
constexpr int kFusedRow = kFusedBatch + 8;  // bf16 per LDS row
constexpr size_t kFusedLds = sizeof(uint16_t) * 2 * kGemmTile * kFusedRow;

// MO: outputs held per thread (m <= MO).
template <int MO>
__global__ __launch_bounds__(256, 2) void substrate_wgrad_kernel(
    const float* __restrict__ h, const uint16_t* __restrict__ w2t, const float* __restrict__ dy,
    const uint16_t* __restrict__ x, int64_t x_stride, int S, int B, int m, int t_tiles, int parts,
    int tiles_per_part, float* __restrict__ dw1t, float* __restrict__ dw2t) {
  extern __shared__ __align__(16) uint16_t wg_lds[];
  uint16_t* sz = wg_lds;                         // dz^T [128 t][kFusedRow]
  uint16_t* sx = wg_lds + kGemmTile * kFusedRow; // x^T [128 s][kFusedRow]; first dY
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int64_t item = gemm_item(blockIdx.x, gridDim.x);
  const int per_g = t_tiles * parts;
  const int g = (int)(item / per_g), r = (int)(item - (int64_t)g * per_g);
  const int part = r / t_tiles, t0 = (r - part * t_tiles) * kGemmTile;
  const int s_begin = part * tiles_per_part * kGemmTile;
  const int s_end = min(S, s_begin + tiles_per_part * kGemmTile);
  const uint16_t* X = x + (int64_t)g * x_stride;

  // x of one tile of s: item c = tid + 256 u is two columns (c % 64) of eight
  // rows (c / 64)
  constexpr int kItems = 64 * (kFusedBatch / 8) / 256;
  uint32_t rx[kItems][8];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int c = tid + 256 * u, s = s0 + 2 * (c & 63), b = (c >> 6) * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        rx[u][i] = b + i < B && s < S
                       ? *reinterpret_cast<const uint32_t*>(X + (int64_t)(b + i) * S + s)
                       : 0u;
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int c = tid + 256 * u, b = (c >> 6) * 8;
      u32x4 lo, hi;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lo[i] = (rx[u][2 * i] & 0xffffu) | (rx[u][2 * i + 1] << 16);
        hi[i] = (rx[u][2 * i] >> 16) | (rx[u][2 * i + 1] & 0xffff0000u);
      }
      uint16_t* to = sx + 2 * (c & 63) * kFusedRow + b;
      *reinterpret_cast<u32x4*>(to) = lo;
      *reinterpret_cast<u32x4*>(to + kFusedRow) = hi;
    }
  };
  // the tiles in turn from a place of the workgroup's own: workgroups that
  // run side by side store to different parts of their rows
  const int n_tiles = (s_end - s_begin + kGemmTile - 1) / kGemmTile;
  int turn = (int)(item % n_tiles);
  fetch(s_begin + turn * kGemmTile);

  // dz of the workgroup's hidden units and dw2t: thread = hidden unit, two
  // threads per unit. Each reads every other group of eight rows of H and
  // takes dz of these; the pair's 16 rows meet in LDS, and each thread adds them
  // to half of the outputs' sums: one chain per output in ascending b, the sum of
  // the kernel for larger batches. (With both threads reading all rows of H the
  // kernel takes 429 us, with branches around the rows past the last 398.)
  const int tl = tid & (kGemmTile - 1), half = wave >> 1, t = t0 + tl;
  const bool unit = t < S;
  const float* H = h + (int64_t)g * B * S + (unit ? t : 0);
  constexpr int kPair = 16;  // rows that two threads share at once
  float* sdy = reinterpret_cast<float*>(sx);                  // [B][MO]
  float (*sh)[kPair][kGemmTile] =                             // [2][kPair][128]
      reinterpret_cast<float (*)[kPair][kGemmTile]>(sdy + kFusedBatch * MO);
  static_assert(sizeof(float) * (kFusedBatch * MO + 2 * kPair * kGemmTile) <=
                sizeof(uint16_t) * kGemmTile * kFusedRow, "dY and H rows fit the tile of x");
  // rows from B on and outputs from m on are zeros, which add nothing below
  for (int i = tid; i < (B + 31) / 32 * 32 * MO; i += 256) {
    const int b = i / MO, j = i % MO;
    sdy[i] = b < B && j < m ? dy[((int64_t)g * B + b) * m + j] : 0.0f;
  }
  float w2[MO], acc2[MO / 2];
#pragma unroll
  for (int j = 0; j < MO; ++j)
    w2[j] = j < m && unit ? bf16_float(w2t[((int64_t)g * m + j) * S + t]) : 0.0f;
#pragma unroll
  for (int j = 0; j < MO / 2; ++j) acc2[j] = 0.0f;
  // one group of eight rows ahead; not unrolled further, the code has to stay
  // well inside the instruction cache
  float hb[8], hn[8];
  auto rows_of = [&](int b0, float (&v)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = b0 + u < B && unit ? H[(int64_t)(b0 + u) * S] : 0.0f;
  };
  rows_of(half * 8, hb);
#pragma unroll 1
  for (int p0 = 0; p0 < (B + 31) / 32 * 32; p0 += kPair) {
    const int b0 = p0 + half * 8;
    rows_of(b0 + kPair, hn);
    float (*rows)[kGemmTile] = sh[(p0 / kPair) & 1];
#pragma unroll
    for (int u = 0; u < 8; ++u) rows[half * 8 + u][tl] = hb[u];
    lds_barrier();  // the rows, and before the first pair dY
    float dz[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float* d = sdy + (b0 + u) * MO;
      float up = 0.0f;
#pragma unroll
      for (int j = 0; j < MO; ++j) up = fmaf(d[j], w2[j], up);
      dz[u] = b0 + u < B ? up * fmaf(-hb[u], hb[u], 1.0f) : 0.0f;
    }
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = bf16_bits(dz[2 * e]) | ((uint32_t)bf16_bits(dz[2 * e + 1]) << 16);
    *reinterpret_cast<u32x4*>(sz + tl * kFusedRow + b0) = v;
#pragma unroll
    for (int u = 0; u < kPair; ++u) {
      const float* d = sdy + (p0 + u) * MO + half * (MO / 2);
      const float x = rows[u][tl];
#pragma unroll
      for (int j = 0; j < MO / 2; ++j) acc2[j] = fmaf(x, d[j], acc2[j]);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) hb[u] = hn[u];
  }
  if (part == 0 && unit)
#pragma unroll
    for (int j = 0; j < MO / 2; ++j)
      if (half * (MO / 2) + j < m)
        dw2t[((int64_t)g * m + half * (MO / 2) + j) * S + t] = acc2[j];

  // this wavefront's quarter: 64 hidden units x 64 columns of a tile
  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;
  const int li = lane & 15, kq = (lane >> 4) * 8;
  constexpr int kSteps = kFusedBatch / 32;
  const int steps = (B + 31) / 32;
  const uint16_t* pa = sz + (wm + li) * kFusedRow + kq;
  const uint16_t* pb = sx + (wn + li) * kFusedRow + kq;
  float* C = dw1t + (int64_t)g * S * S;
  for (int i_tile = 0; i_tile < n_tiles; ++i_tile) {
    const int s0 = s_begin + turn * kGemmTile;
    turn = turn + 1 == n_tiles ? 0 : turn + 1;
    lds_barrier();  // the previous tile (or dY) is no longer read
    stash();
    lds_barrier();
    if (i_tile + 1 < n_tiles) fetch(s_begin + turn * kGemmTile);
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < kSteps; ++kk) {
      if (kk >= steps) break;
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        fa[i] = *reinterpret_cast<const bf16x8*>(pa + 16 * i * kFusedRow + 32 * kk);
        fb[i] = *reinterpret_cast<const bf16x8*>(pb + 16 * i * kFusedRow + 32 * kk);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    // a lane holds four consecutive columns of one row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = t0 + wm + 16 * i + li;
      if (row >= S) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = s0 + wn + 16 * j + (lane >> 4) * 4;  // S is a multiple of 64
        if (col < S) {
          float* q = C + (int64_t)row * S + col;
          if ((reinterpret_cast<uintptr_t>(C) & 15) == 0) {
            *(__attribute__((address_space(1))) f32x4*)q = acc[i][j];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) store_global(q + e, acc[i][j][e]);
          }
        }
      }
    }
  }
}

// xt[g][s][b] = x[g][b][s] (bfloat16 bits), rows padded with zeros to Kp.
__global__ __launch_bounds__(256) void transpose_x_kernel(const uint16_t* __restrict__ x,
                                                          int64_t x_stride, int S, int B, int Kp,
                                                          int wg_per_g, uint16_t* __restrict__ xt) {
  const int g = blockIdx.x / wg_per_g;
  const int s = (blockIdx.x - g * wg_per_g) * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const uint16_t* X = x + (int64_t)g * x_stride + s;
  uint16_t* T = xt + ((int64_t)g * S + s) * Kp;
  for (int b0 = 0; b0 < Kp; b0 += 8) {
    uint16_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = b0 + u < B ? X[(int64_t)(b0 + u) * S] : (uint16_t)0;
    uint4 q;
    q.x = v[0] | ((uint32_t)v[1] << 16);
    q.y = v[2] | ((uint32_t)v[3] << 16);
    q.z = v[4] | ((uint32_t)v[5] << 16);
    q.w = v[6] | ((uint32_t)v[7] << 16);
    *reinterpret_cast<uint4*>(T + b0) = q;
  }
}

// ----------------------------------------------------------- CPPN adjoint

// Limits of the CPPN adjoint.
constexpr int kCppnNodes = 32, kCppnEdges = 64;
constexpr int kCppnPart = kCppnEdges + kCppnNodes;  // partial sums per workgroup
// rows of four sums: a computed node takes (in-edges + 4) / 4 of them
constexpr int kCppnSums = (kCppnEdges + 4 * (kCppnNodes - 5)) / 4;
// 64 targets per wavefront measured 1287 us, 32 (twice the wavefronts) 1438 us
constexpr int kCppnWaves = 4, kCppnRun = 64, kCppnWavesWanted = 4096, kCppnSlots = 12;

struct CppnLds {
  int2 edge[kCppnEdges + kWave];
  float acc[kCppnWaves][kCppnSums][kWave];
  // values and slopes of the targets' coordinates and target nodes
  __align__(16) float table[kCppnWaves][kCppnSlots][2][kCppnRun];
  float part[kCppnPart];
};

// The gradient of sum_q u_q * w(q) over every query q of the substrate with
// respect to the CPPN's connection weights and node biases, where the upstream
// u_q is dw1t / dw2t at the query when its weight survived the threshold (the
// CPPN value of this very evaluation, float32) and 0 otherwise. A wavefront
// (64 sources, 64 targets, K targets a step: four, or two for genomes whose
// rows do not fit) runs the forward pass as the query does, each value beside
// its gradient in the register file (and its slope, where that needs the
// pre-activation), then the reverse sweep:
//   delta_k = gbar_k act'(z_k);  db_k += delta_k;
//   for in-edge e = (j -> k): dt = delta_k rho_k (/ n for mean);
//   dw_e += dt v_j;  gbar_j += dt w_e
// A fixed node's gradient is linear in its gbar, and its value is the same at
// every step: its gbar adds up over the steps and its own sweep runs once, at
// the end. Sums are folded four at a time into one LDS row (see rf_file.hpp),
// then added over the workgroup in a fixed order, one partial per workgroup.
// Sum and mean aggregation only (the CPPN's); other genomes get NaN.
// Bound by instruction issue; registers hold two wavefronts per SIMD. 50 CPPNs
// (11 computed nodes, 33 in-edges), 32 x 32 grid, 8 outputs: 1287 us; 2479 us
// with every node at every pair, two tiles a step and a slot per sum and lane.
template <int K>
__device__ __forceinline__ void cppn_adjoint(const CppnWave& c, const SubGeom& sg,
                                             const CppnItem& it, int l_sum,
                                             const float* __restrict__ up, float (*acc)[kWave],
                                             float (*table)[2][kCppnRun]) {
  using F = Files<K>;
  const int lane = lane_id();
  auto row_of = [&](int p) { return __builtin_amdgcn_readlane(c.l_row, p); };
  auto act_of = [&](int p) { return __builtin_amdgcn_readlane(c.l_fn, p) & 7; };
  auto back = [&](int p, int2 ed) __attribute__((always_inline)) {
    const int act = act_of(p), row = row_of(p);
    const int le = __builtin_amdgcn_readlane(c.l_edge, p), ne = le >> 16;
    const int f = __builtin_amdgcn_readlane(c.l_fn, p);
    float* sum = acc[__builtin_amdgcn_readlane(l_sum, p)] + lane;
    float old = *sum;
    float g[K], v[K], slope[K], dt[K], db = 0.0f;
    F::get_gv(row, g, v);
    if (slope_needs_z(act))
      F::get_v(row + 2, slope);
    else
      act_slopes_v<K>(act, v, slope);
    const float rho = __int_as_float(__builtin_amdgcn_readlane(c.l_resp, p));
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float d = g[k] * slope[k];
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
      const int j = __builtin_amdgcn_readlane(ed.x, e);
      return j < c.n_rows
                 ? F::dot_v_fma_g(j, dt, __int_as_float(__builtin_amdgcn_readlane(ed.y, e)))
                 : F::dot_v(j, dt);  // an input
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
      const float t0 = term(e);
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
  };
  const int op_row = row_of(c.op);
  const int runs = it.t1 - it.t0;
  // Step -2 evaluates the fixed nodes, step -1 (lane = target) the target
  // nodes, the others K targets each, and the last sweeps the fixed nodes back:
  // one walk each way in the code for all.
  const int last = (runs + K - 1) / K * K;
  for (int t = -2 * K; t <= last; t += K) {
    float v[K], slope[K], u[K];
    uint64_t forth = c.both, back_over = c.both | c.target;
    if (t < -K) {
      float x0, y0, one = 1.0f;
      asm volatile("" : "+v"(one));
      source_xy(sg, it.s0 + lane, &x0, &y0);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = x0;
      F::set_v(c.in_row[0], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = y0;
      F::set_v(c.in_row[1], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = one;
      F::set_v(c.in_row[4], v);
      forth = c.fixed;
    } else if (t < 0) {
      float x0, y0;
      target_xy(sg, it.hidden, min(it.t0 + lane, it.t1 - 1), &x0, &y0);
      table[0][0][lane] = x0;
      table[1][0][lane] = y0;
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = x0;
      F::set_v(c.in_row[2], v);
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = y0;
      F::set_v(c.in_row[3], v);
      forth = c.target;
    } else if (t < last) {
#pragma unroll
      for (int k = 0; k < K; ++k) u[k] = up[(int64_t)min(t + k, runs - 1) * sg.S + lane];
      uint64_t m = c.target;
      for (int slot = 0; slot < c.n_kept; ++slot) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = table[slot][0][t + k];
        if (slot < 2) {
          F::set_v(slot == 0 ? c.in_row[2] : c.in_row[3], v);
        } else {
          const int p = __builtin_ctzll(m), row = row_of(p);
          m &= m - 1;
          F::set_vg(row, v);
          if (slope_needs_z(act_of(p))) {
#pragma unroll
            for (int k = 0; k < K; ++k) slope[k] = table[slot][1][t + k];
            F::set_v(row + 2, slope);
          }
        }
      }
    } else {
      forth = 0;
      back_over = c.fixed;
    }
    int slot = 2;
    cppn_forward(c, forth, [&](int p, int2 ed) __attribute__((always_inline)) {
      float z[K];
      cppn_pre<F, K, false>(c, p, ed, z);
      const int act = act_of(p), row = row_of(p);
      activate_all<K>(act, z, v);
      F::set_vg(row, v);
      slope[0] = 0.0f;
      if (slope_needs_z(act)) {
        act_slopes<K>(act, v, z, slope);
        F::set_v(row + 2, slope);
      }
      if (t == -K) {
        table[slot][0][lane] = v[0];
        table[slot][1][lane] = slope[0];
        ++slot;
      }
    });
    if (t < 0) continue;
    if (t < last) {
      float y[K];
      F::get_v(op_row, y);
#pragma unroll
      for (int k = 0; k < K; ++k)  // NaN y: no gradient
        u[k] = t + k < runs && fabsf(y[k]) >= sg.thr ? u[k] : 0.0f;
      F::fma_g(op_row, u, 1.0f);
    }
    cppn_reverse(c, back_over, back);
  }
}

__global__ __launch_bounds__(kWave * kCppnWaves) __attribute__((amdgpu_num_vgpr(TN_RF_FILE / 2))) void
cppn_backward_kernel(PopView pop, const int32_t* __restrict__ status,
                     const int32_t* __restrict__ n_valid, const int32_t* __restrict__ row_ptr,
                     const int32_t* __restrict__ edge_src, const int32_t* __restrict__ w_bits,
                     const int32_t* __restrict__ fn, const int32_t* __restrict__ bias_bits,
                     const int32_t* __restrict__ resp_bits, const int32_t* __restrict__ io_pos,
                     SubGeom sg, int run, int wg_per_g, const float* __restrict__ dw1t,
                     const float* __restrict__ dw2t, float* __restrict__ part) {
  rf_file_reserve();
  extern __shared__ __align__(16) char cppn_lds[];
  CppnLds& L = *reinterpret_cast<CppnLds*>(cppn_lds);
  const int lane = lane_id(), wave = wave_id(), tid = threadIdx.x;
  const int g = blockIdx.x / wg_per_g;
  const int item = (blockIdx.x - g * wg_per_g) * kCppnWaves + wave;
  const int n = n_valid[g];
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g)),
                rb = uniform64(pop.rowptr_base(g));
  const int n_edges = n > 0 ? row_ptr[rb + n] : 0;
  float* out = part + (int64_t)blockIdx.x * kCppnPart;
  bool ok = status[g] == 0 && n <= kCppnNodes && n_edges <= kCppnEdges;
  if (ok) {
    const int f = lane < n ? fn[nb + lane] : -1;
    const int agg = (f >> 8) & 0xff;
    ok = !__ballot(f >= 0 && agg != TN_AGG_SUM && agg != TN_AGG_MEAN);
  }
  if (!ok) {
    for (int i = tid; i < kCppnPart; i += blockDim.x) out[i] = __builtin_nanf("");
    return;
  }
  const CppnWave c = cppn_program<true>(
      n, n_edges, row_ptr + rb, edge_src + cb, w_bits + cb, fn + nb, bias_bits + nb,
      resp_bits + nb, io_pos + (int64_t)g * (pop.n_in + pop.n_out), kCppnSlots, L.edge);
  const int rows = c.l_fn >= 0 ? sum_rows(c.l_edge >> 16) : 0;
  const int row_end = wave_inclusive_scan(rows), l_sum = row_end - rows;
  const int n_sums = __builtin_amdgcn_readlane(row_end, kWave - 1);
  for (int r = 0; r < n_sums; ++r) L.acc[wave][r][lane] = 0.0f;
  for (int i = tid; i < kCppnPart; i += blockDim.x) L.part[i] = 0.0f;
  __syncthreads();
  if (item < cppn_items(sg, run)) {
    const CppnItem it = cppn_item(sg, run, item);
    const int64_t Q1 = (int64_t)sg.S * sg.S, Q2 = (int64_t)sg.S * sg.n_out;
    const float* up = (it.hidden ? dw1t + g * Q1 : dw2t + g * Q2) + (int64_t)it.t0 * sg.S + it.s0;
    if (c.n_rows + 5 <= kRfFileRows / 4)
      cppn_adjoint<4>(c, sg, it, l_sum, up, L.acc[wave], L.table[wave]);
    else
      cppn_adjoint<2>(c, sg, it, l_sum, up, L.acc[wave], L.table[wave]);
  }
  __syncthreads();
  // each sum's 16 lanes over the wavefronts, in a fixed order; partial sums:
  // in-edge e at e, position p at kCppnEdges + p
  for (int p = 0; p < n; ++p) {
    if (__builtin_amdgcn_readlane(c.l_fn, p) < 0) continue;
    const int le = __builtin_amdgcn_readlane(c.l_edge, p);
    const int r0 = __builtin_amdgcn_readlane(l_sum, p);
    for (int i = tid; i <= (le >> 16); i += blockDim.x) {  // 0: the bias
      const int quarter = sum_of_quarter(i & 3);
      float total = 0.0f;
      for (int w = 0; w < kCppnWaves; ++w) {
        const float* from = L.acc[w][r0 + (i >> 2)] + quarter * 16;
        float t = 0.0f;
#pragma unroll 8
        for (int b = 0; b < 16; ++b) t += from[b];
        total += t;
      }
      L.part[i ? (le & 0xffff) + i - 1 : kCppnEdges + p] = total;
    }
  }
  __syncthreads();
  for (int i = tid; i < kCppnPart; i += blockDim.x) out[i] = L.part[i];
}

// Sums the workgroups' partials of each genome in slot order and scatters them:
// dW[connection row of in-edge e], db[node row of position p]; every other row
// of the genome (disabled, padding, inputs) is 0; NaN where the partials are.
__global__ __launch_bounds__(256) void cppn_grad_reduce_kernel(
    PopView pop, const int32_t* __restrict__ n_valid, const int32_t* __restrict__ row_ptr,
    const int32_t* __restrict__ edge_row, const int32_t* __restrict__ order,
    const int32_t* __restrict__ fn, const float* __restrict__ part, int slots,
    float* __restrict__ dW, float* __restrict__ db) {
  const int g = blockIdx.x;
  const int64_t nb = pop.node_base(g), cb = pop.conn_base(g), rb = pop.rowptr_base(g);
  const int nrows = (int)pop.node_rows(g), crows = (int)pop.conn_rows(g);
  const int n = n_valid[g];
  const int n_edges = n > 0 ? row_ptr[rb + n] : 0;
  const float* pg = part + (int64_t)g * slots * kCppnPart;
  const bool bad = n == 0 || pg[0] != pg[0] || n > kCppnNodes || n_edges > kCppnEdges;
  for (int r = threadIdx.x; r < crows; r += blockDim.x) dW[cb + r] = bad ? __builtin_nanf("") : 0.0f;
  for (int r = threadIdx.x; r < nrows; r += blockDim.x) db[nb + r] = bad ? __builtin_nanf("") : 0.0f;
  __syncthreads();
  if (bad) return;
  for (int i = threadIdx.x; i < n_edges + n; i += blockDim.x) {
    const int col = i < n_edges ? i : kCppnEdges + (i - n_edges);
    float acc = 0.0f;
    for (int w = 0; w < slots; ++w) acc += pg[(int64_t)w * kCppnPart + col];
    if (i < n_edges) {
      dW[cb + edge_row[cb + i]] = acc;
    } else {
      const int p = i - n_edges;
      if (fn[nb + p] >= 0) db[nb + order[nb + p]] = acc;
    }
  }
}

// Targets per wavefront: the most (each wavefront pays for reading its genome
// and for the fixed and target nodes) that still gives `waves` wavefronts.
constexpr int kCppnRunLeast = 8;
int cppn_run(int P, const SubGeom& sg, int most, int waves) {
  int run = most;
  while (run > kCppnRunLeast && (int64_t)P * cppn_items(sg, run) < waves) run /= 2;
  return run;
}

SubGeom geometry(const tn_substrate& sub) {
  SubGeom sg;
  sg.grid = sub.grid;
  sg.S = sub.grid * sub.grid;
  sg.n_out = sub.n_out;
  sg.thr = sub.threshold;
  sg.step = 2.0f / (float)(sub.grid - 1);
  sg.ostep = sub.n_out > 1 ? 2.0f / (float)(sub.n_out - 1) : 0.0f;
  return sg;
}

}  // namespace

int check_substrate(const tn_substrate* sub) {
  if (!sub) return TN_EINVAL;
  if (sub->grid < 2 || sub->n_out < 1 || !(sub->threshold >= 0.0f)) return TN_EINVAL;
  const int64_t S = (int64_t)sub->grid * sub->grid;
  // MFMA tiles of 64 along S; the output weights of one genome fit in LDS
  if (S % 64 != 0 || S > 16384 || S * sub->n_out * 2 > 64 * 1024) return TN_EUNSUPPORTED;
  return TN_OK;
}

int launch_cppn_query(const tn_population& p, const tn_transformed& t, const tn_substrate& sub,
                      uint16_t* w1t, uint16_t* w2t, float* raw1, float* raw2,
                      hipStream_t stream) {
  const SubGeom sg = geometry(sub);
  // Genomes of up to 20 positions run four tiles in a file of 80 rows, larger
  // ones two, so populations of more than kMapRows node rows take the packed
  // program (which reuses rows: four tiles for all) and evaluate every node at
  // every pair: 30 CPPNs of 21 to 38 positions (N_max 40) on a 16 x 16 grid took
  // 76 us there and 85 us here; with N_max 32 and 10 to 21 positions 45 and 44
  // us, 100 of them on a 32 x 32 grid 1112 and 713 us.
  if (p.N_max <= kMapRows) {
    const int run = cppn_run(p.P, sg, kMapRun, kMapWavesWanted);
    const int per_g = (cppn_items(sg, run) + kMapWaves - 1) / kMapWaves;
    const int64_t blocks = (int64_t)p.P * per_g;
    if (blocks == 0) return TN_OK;
    if (blocks > 0x7fffffff) return TN_EUNSUPPORTED;
    const size_t lds = sizeof(int2) * ((size_t)p.C_max + kWave);
    const int rc = allow_lds((const void*)cppn_map_kernel, lds);
    if (rc != TN_OK) return rc;
    hipLaunchKernelGGL(cppn_map_kernel, dim3((unsigned)blocks), dim3(kWave * kMapWaves), lds,
                       stream, make_view(p), t.status, t.n_valid, t.row_ptr, t.edge_src,
                       reinterpret_cast<const int32_t*>(t.edge_w), t.pos_fn,
                       reinterpret_cast<const int32_t*>(t.pos_bias),
                       reinterpret_cast<const int32_t*>(t.pos_resp), t.io_pos, sg, run, per_g, w1t,
                       w2t, raw1, raw2);
    return check_launch();
  }
  const int64_t Q = (int64_t)sg.S * sg.S + (int64_t)sg.S * sg.n_out;  // < 2^31 by check_substrate
  const int64_t unit = (int64_t)rf_tiles(kQueryRows) * kWave;
  const int64_t n_units = (Q + unit - 1) / unit;
  const int waves = 4, per_wave = 4;
  const int n_chunks = (int)((n_units + (int64_t)waves * per_wave - 1) / ((int64_t)waves * per_wave));
  const int64_t grid = (int64_t)p.P * n_chunks;
  if (grid == 0) return TN_OK;
  if (grid > 0x7fffffff) return TN_EUNSUPPORTED;
  hipLaunchKernelGGL(cppn_query_kernel, dim3((unsigned)grid), dim3(kWave * waves), 0, stream,
                     make_view(p), t.status, t.prog_rows, t.n_valid,
                     reinterpret_cast<const int4*>(t.prog_node),
                     reinterpret_cast<const int2*>(t.prog_edge), t.prog_rec, t.io_pos, sg,
                     n_chunks, per_wave, w1t, w2t, raw1, raw2);
  return check_launch();
}

int launch_substrate_forward(const tn_substrate& sub, int P, const uint16_t* w1t,
                             const uint16_t* w2t, const uint16_t* x, int64_t x_stride, int B,
                             float* h, float* y, hipStream_t stream) {
  const int S = sub.grid * sub.grid;
  GemmArgs ga{};
  ga.a = x;
  ga.lda = S;
  ga.a_batch = x_stride;
  ga.b = w1t;
  ga.ldb = S;
  ga.b_batch = (int64_t)S * S;
  ga.c = h;
  ga.ldc = S;
  ga.c_batch = (int64_t)B * S;
  ga.M = B;
  ga.N = S;
  ga.K = S;
  int rc = launch_gemm<true>(ga, P, stream);
  if (rc != TN_OK) return rc;
  const int b_tiles = (B + kOutRows - 1) / kOutRows, j_tiles = (sub.n_out + kOutCols - 1) / kOutCols;
  const int64_t grid = (int64_t)P * b_tiles * j_tiles;
  if (grid > 0x7fffffff) return TN_EUNSUPPORTED;
  hipLaunchKernelGGL(substrate_output_kernel, dim3((unsigned)grid), dim3(256), 0, stream, h, w2t,
                     S, B, sub.n_out, b_tiles, j_tiles, y);
  return check_launch();
}

size_t substrate_workspace_bytes(const tn_substrate& sub, int P, int B, int64_t x_stride) {
  const int64_t S = (int64_t)sub.grid * sub.grid;
  const int64_t Kp = ((int64_t)B + 31) / 32 * 32;
  const int64_t px = x_stride == 0 ? 1 : P;
  return (size_t)(2 * S * Kp * (P + px));
}

int launch_substrate_backward(const tn_substrate& sub, int P, const uint16_t* w2t,
                              const uint16_t* x, int64_t x_stride, int B, const float* h,
                              const float* dy, void* workspace, float* dw1t, float* dw2t,
                              hipStream_t stream) {
  const int S = sub.grid * sub.grid, m = sub.n_out;
  // Up to kFusedBatch rows (the whole reduction in one workgroup's registers)
  // one kernel; a genome's tiles of s are split where its tiles of t alone
  // would leave the chip idle (two workgroups fit a compute unit). It reads x
  // two columns at a time: rows that are not 4-byte aligned take the kernels
  // below, as larger batches do.
  if (B <= kFusedBatch && (reinterpret_cast<uintptr_t>(x) & 3) == 0 && x_stride % 2 == 0) {
    const int tiles = (S + kGemmTile - 1) / kGemmTile;
    const int want = (int)std::min<int64_t>(tiles, std::max<int64_t>(1, 512 / std::max<int64_t>(1, (int64_t)P * tiles)));
    const int per = (tiles + want - 1) / want, parts = (tiles + per - 1) / per;
    const int64_t grid = (int64_t)P * tiles * parts;
    if (grid > 0x7fffffff) return TN_EUNSUPPORTED;
    const auto kern = m <= 8    ? substrate_wgrad_kernel<8>
                      : m <= 16 ? substrate_wgrad_kernel<16>
                                : substrate_wgrad_kernel<kMaxOutBwd>;
    const int rc = allow_lds((const void*)kern, kFusedLds);
    if (rc != TN_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), kFusedLds, stream, h, w2t, dy, x,
                       x_stride, S, B, m, tiles, parts, per, dw1t, dw2t);
    return check_launch();
  }
  const int Kp = (B + 31) / 32 * 32;
  const int px = x_stride == 0 ? 1 : P;
  uint16_t* dzt = static_cast<uint16_t*>(workspace);
  uint16_t* xt = dzt + (int64_t)P * S * Kp;
  const int wg_per_g = (S + 255) / 256;
  const size_t lds = sizeof(float) * (size_t)B * m;
  int rc = allow_lds((const void*)substrate_grad_out_kernel, lds);
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(substrate_grad_out_kernel, dim3((unsigned)(P * wg_per_g)), dim3(256), lds,
                     stream, h, w2t, dy, S, B, Kp, m, wg_per_g, dzt, dw2t);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(transpose_x_kernel, dim3((unsigned)(px * wg_per_g)), dim3(256), 0, stream, x,
                     x_stride, S, B, Kp, wg_per_g, xt);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  // dw1t[t][s] = sum_b dz[b][t] x[b][s]
  GemmArgs ga{};
  ga.a = dzt;
  ga.lda = Kp;
  ga.a_batch = (int64_t)S * Kp;
  ga.b = xt;
  ga.ldb = Kp;
  ga.b_batch = x_stride == 0 ? 0 : (int64_t)S * Kp;
  ga.c = dw1t;
  ga.ldc = S;
  ga.c_batch = (int64_t)S * S;
  ga.M = S;
  ga.N = S;
  ga.K = Kp;
  return launch_gemm<false>(ga, P, stream);
}

namespace {
int adjoint_run(int P, const SubGeom& sg) { return cppn_run(P, sg, kCppnRun, kCppnWavesWanted); }
int adjoint_workgroups(int P, const SubGeom& sg) {  // of a genome
  return (cppn_items(sg, adjoint_run(P, sg)) + kCppnWaves - 1) / kCppnWaves;
}
}  // namespace

// Enough for every population of up to P genomes: fewer genomes take shorter runs,
// so 15 of them (32 x 32 grid, 8 outputs) make more partial sums than 16.
size_t cppn_backward_workspace_bytes(const tn_population& p, const tn_substrate& sub) {
  const SubGeom sg = geometry(sub);
  int64_t groups = 0;
  for (int run = kCppnRun; run >= kCppnRunLeast; run /= 2) {
    // genomes that take this run, at most
    const int64_t genomes =
        run == kCppnRun ? p.P
                        : std::min<int64_t>(p.P, (kCppnWavesWanted - 1) / cppn_items(sg, 2 * run));
    groups = std::max(groups, genomes * ((cppn_items(sg, run) + kCppnWaves - 1) / kCppnWaves));
  }
  return sizeof(float) * (size_t)groups * kCppnPart;
}

int launch_cppn_backward(const tn_population& p, const tn_transformed& t, const tn_substrate& sub,
                         const float* dw1t, const float* dw2t, void* workspace, float* dW,
                         float* db, hipStream_t stream) {
  const SubGeom sg = geometry(sub);
  const int per_g = adjoint_workgroups(p.P, sg);
  const int64_t grid = (int64_t)p.P * per_g;
  if (grid == 0) return TN_OK;
  if (grid > 0x7fffffff) return TN_EUNSUPPORTED;
  float* part = static_cast<float*>(workspace);
  int rc = allow_lds((const void*)cppn_backward_kernel, sizeof(CppnLds));
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(cppn_backward_kernel, dim3((unsigned)grid), dim3(kWave * kCppnWaves),
                     sizeof(CppnLds), stream, make_view(p), t.status, t.n_valid, t.row_ptr,
                     t.edge_src, reinterpret_cast<const int32_t*>(t.edge_w), t.pos_fn,
                     reinterpret_cast<const int32_t*>(t.pos_bias),
                     reinterpret_cast<const int32_t*>(t.pos_resp), t.io_pos, sg, adjoint_run(p.P, sg), per_g,
                     dw1t, dw2t, part);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(cppn_grad_reduce_kernel, dim3((unsigned)p.P), dim3(256), 0, stream,
                     make_view(p), t.n_valid, t.row_ptr, t.edge_row, t.order, t.pos_fn, part,
                     per_g, dW, db);
  return check_launch();
}

}  // namespace tn
