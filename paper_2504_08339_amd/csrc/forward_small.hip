// Calculation stage (TensorNEAT Section 3.3) for small batches: one step of a
// rollout (one observation per genome), the four XOR rows.
//
// The other engines give a lane to an observation, so a batch of one leaves 63
// of 64 lanes idle and walks a genome node after node. Here a wavefront takes
// one genome and its lanes are (node, observation) pairs: with the batch
// rounded up to a power of two, Bp, 64 / Bp nodes of a level of the topological
// order run side by side, and the genome costs its levels, not its nodes.
// The program and every node's values sit in LDS (a row of Bp values per
// position, no reuse); the wavefronts of a workgroup have genomes of their own
// and never wait for each other. Each node's arithmetic is the other engines'
// (ascending in-edges, fused multiply-add), so the outputs are the same bits.
//
// Bound by the latency of two dependent loads of the program and of the LDS
// round trips of a level's longest node (reading the next level's records ahead
// measured the same); enough wavefronts per SIMD (one genome
// of 64 / 256 rows takes 3.6 KB of LDS) hide most of it. 10,000 genomes (17 ->
// 6, 40 nodes, 126 in-edges), one observation each: 17 us (51 us in the two
// launches of the register engine).
#include <algorithm>

#include "fwd_core.hpp"
#include "fwd_launch.hpp"

namespace tn {

namespace {

constexpr int kSmallWaves = 4;  // genomes per workgroup, where the LDS holds them

struct SmallArgs {
  int64_t obs_stride;
  int B, shift;  // observations; Bp = 1 << shift >= B
  int64_t target_stride;
  float scale, offset;
  int rows_cap;     // value rows the LDS engine holds; N_max or more: no limit to report
  int wave_bytes;   // LDS of one wavefront
};

struct SmallLds {
  int node, edge, lvl, io, vals, bytes;
};

__host__ __device__ inline int up16(int x) { return (x + 15) & ~15; }

__host__ __device__ inline SmallLds small_lds(int N, int C, int nio, int shift) {
  SmallLds l;
  l.node = 0;
  l.edge = l.node + 16 * N;
  l.lvl = l.edge + up16(8 * C);
  l.io = l.lvl + up16(4 * (N + 2));  // level starts, the end, the number of levels
  l.vals = l.io + up16(4 * nio);
  l.bytes = l.vals + up16((4 * N) << shift);
  return l;
}

// log2 of B observations rounded up to a power of two.
inline int batch_shift(int B) {
  int shift = 0;
  while ((1 << shift) < B) ++shift;
  return shift;
}

// LDS bytes of one wavefront.
inline size_t small_bytes(const tn_population& p, int B) {
  return (size_t)small_lds(p.N_max, p.C_max, p.n_in + p.n_out, batch_shift(B)).bytes;
}

// One node's aggregate over in-edges e0 .. e1-1 at this lane's observation:
// v[edge.x] is the source's value. In-edges come four at a time, their records
// and then their values requested together.
__device__ __forceinline__ float aggregate(int agg, const int2* edge, int e0, int e1,
                                           const float* v) {
  float s = 0.0f;
  if (agg == TN_AGG_SUM) {
    for (int e = e0; e < e1; e += 4) {
      int2 q[4];
      float x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) q[j] = edge[min(e + j, e1 - 1)];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = v[q[j].x];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (e + j < e1) s = fmaf(__int_as_float(q[j].y), x[j], s);
    }
  } else if (e0 < e1) {
    s = __int_as_float(edge[e0].y) * v[edge[e0].x];
    for (int e = e0 + 1; e < e1; ++e) {
      const float t = __int_as_float(edge[e].y) * v[edge[e].x];
      switch (agg) {
        case TN_AGG_PRODUCT: s = s * t; break;
        case TN_AGG_MAX: s = fmaxf(s, t); break;
        case TN_AGG_MIN: s = fminf(s, t); break;
        case TN_AGG_MEAN: s = s + t; break;
        default: s = fabsf(t) > fabsf(s) ? t : s; break;  // maxabs
      }
    }
    if (agg == TN_AGG_MEAN) s = s / (float)(e1 - e0);
  }
  return s;
}

template <bool kLoss>
__global__ __launch_bounds__(kWave * kSmallWaves) void forward_small_kernel(
    PopView pop, const int32_t* __restrict__ status, const int32_t* __restrict__ n_valid,
    const int32_t* __restrict__ level, const int4* __restrict__ prog_node,
    const int32_t* __restrict__ edge_src, const int32_t* __restrict__ w_bits,
    const int32_t* __restrict__ io_pos, const int32_t* __restrict__ n_rows,
    const int32_t* __restrict__ prog_rows, const float* __restrict__ obs,
    const float* __restrict__ target, float* __restrict__ out, float* __restrict__ loss,
    SmallArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = lane_id();
  const int g = blockIdx.x * (blockDim.x / kWave) + wave_id();
  if (g >= pop.P) return;
  const int I = pop.n_in, O = pop.n_out, nio = I + O;
  const SmallLds L = small_lds(pop.N_max, pop.C_max, nio, a.shift);
  unsigned char* mine = smem + wave_id() * a.wave_bytes;
  int4* node = reinterpret_cast<int4*>(mine + L.node);
  int2* edge = reinterpret_cast<int2*>(mine + L.edge);
  int32_t* lvl = reinterpret_cast<int32_t*>(mine + L.lvl);
  int32_t* io = reinterpret_cast<int32_t*>(mine + L.io);
  float* vals = reinterpret_cast<float*>(mine + L.vals);
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g));
  const int rows = (int)min(pop.node_rows(g), (int64_t)pop.N_max);
  const int64_t out_at = (int64_t)g * a.B * O;

  // everything that needs no size is requested at once: the genome's node
  // rows (the few past its last position are not used) and io positions
  int st = status[g];
  const int n = n_valid[g];
  if (a.rows_cap < pop.N_max && prog_rows[g] > kRegRowsMax && n_rows[g] > a.rows_cap) st = -1;
  for (int k = lane; k < nio; k += kWave) io[k] = io_pos[(int64_t)g * nio + k];
  for (int p = lane; p < rows; p += kWave) {
    node[p] = prog_node[nb + p];
    const int lv = level[nb + p], before = p > 0 ? level[nb + p - 1] : -1;
    if (p < n && lv != before) lvl[lv] = p;
    if (p == n - 1) {
      lvl[lv + 1] = n;
      lvl[pop.N_max + 1] = lv + 1;
    }
  }
  if (st != 0) {
    const float nan = __builtin_nanf("");
    if (out)
      for (int i = lane; i < a.B * O; i += kWave) out[out_at + i] = nan;
    if (kLoss && lane == 0) loss[g] = nan;
    return;
  }
  wave_sync();
  const int n_edges = node[n - 1].x;
  for (int e = lane; e < n_edges; e += kWave)
    edge[e] = make_int2(edge_src[cb + e] << a.shift, w_bits[cb + e]);
  const float* x = obs + (int64_t)g * a.obs_stride;
  {
    DivWalk d(lane, I > 0 ? I : 1, kWave);
    for (int i = lane; i < a.B * I; i += kWave, d.step())
      vals[(io[d.c] << a.shift) + d.b] = x[i];
  }
  wave_sync();
  const int b = lane & ((1 << a.shift) - 1), step = kWave >> a.shift;
  float* v = vals + b;
  const int n_lvl = __builtin_amdgcn_readfirstlane(lvl[pop.N_max + 1]);
  for (int l = 0; l < n_lvl; ++l) {
    const int p1 = __builtin_amdgcn_readfirstlane(lvl[l + 1]);
    for (int p = __builtin_amdgcn_readfirstlane(lvl[l]) + (lane >> a.shift); p < p1; p += step) {
      const int4 q = node[p];
      if (q.y < 0) continue;  // an input: its row holds the observation
      const int e0 = p > 0 ? node[p - 1].x : 0;
      const float s = aggregate((q.y >> 8) & 0xff, edge, e0, q.x, v);
      const float z[1] = {fmaf(__int_as_float(q.w), s, __int_as_float(q.z))};
      float y[1];
      activate_all<1>(q.y & 7, z, y);  // codes below 7, checked by the transformation
      v[p << a.shift] = y[0];
    }
    wave_sync();
  }
  const float* t = kLoss ? target + (int64_t)g * a.target_stride : nullptr;
  float sse = 0.0f;
  DivWalk d(lane, O, kWave);
  for (int i = lane; i < a.B * O; i += kWave, d.step()) {
    const float y = vals[(io[I + d.c] << a.shift) + d.b];
    if (out) out[out_at + i] = y;
    if (kLoss) {
      const float e = y - t[i];
      sse = fmaf(e, e, sse);
    }
  }
  if (kLoss) {
    const float total = wave_sum(sse);
    if (lane == 0) loss[g] = fmaf(a.scale, total, a.offset);
  }
}

template <bool kLoss>
int launch_small(const tn_population& p, const tn_transformed& t, const float* obs,
                 int64_t obs_stride, int B, const float* target, int64_t target_stride,
                 float scale, float offset, float* out, float* loss, hipStream_t stream) {
  SmallArgs a{obs_stride, B, batch_shift(B), target_stride, scale, offset, lds_rows_cap(p),
              (int)small_bytes(p, B)};
  // as many genomes per workgroup as leave two workgroups to a compute unit
  int waves = kSmallWaves;
  while (waves > 1 && (size_t)waves * a.wave_bytes > 80 * 1024) waves /= 2;
  const size_t lds = (size_t)waves * a.wave_bytes;
  int rc = allow_lds((const void*)forward_small_kernel<kLoss>, lds);
  if (rc != TN_OK || p.P == 0) return rc;
  hipLaunchKernelGGL(forward_small_kernel<kLoss>, dim3((p.P + waves - 1) / waves),
                     dim3(kWave * waves), lds, stream, make_view(p), t.status, t.n_valid, t.level,
                     reinterpret_cast<const int4*>(t.prog_node), t.edge_src,
                     reinterpret_cast<const int32_t*>(t.edge_w), t.io_pos, t.n_rows, t.prog_rows,
                     obs, target, out, loss, a);
  return check_launch();
}

}  // namespace

bool small_batch(const tn_population& p, int B) {
  return p.N_max > 32 && B > 0 && (B <= 16 || (B <= 32 && p.P <= 2048)) &&
         small_bytes(p, B) <= max_dynamic_lds();
}

int launch_forward_small(const tn_population& p, const tn_transformed& t, const float* obs,
                         int64_t obs_stride, int B, const float* target, int64_t target_stride,
                         float scale, float offset, float* out, float* loss, hipStream_t stream) {
  return loss ? launch_small<true>(p, t, obs, obs_stride, B, target, target_stride, scale, offset,
                                   out, loss, stream)
              : launch_small<false>(p, t, obs, obs_stride, B, nullptr, 0, 0.0f, 0.0f, out, nullptr,
                                    stream);
}

}  // namespace tn
