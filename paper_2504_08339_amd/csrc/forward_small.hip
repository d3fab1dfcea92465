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
  int n_cap, c_cap;    // node rows and in-edges it holds
  int n_prev, c_prev;  // genomes of at most these are an earlier launch's (-1: there is none)
  int per_wave;        // genomes of a wavefront (class launches; else one)
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

struct SmallIn {
  const int32_t *status, *n_valid, *level;
  const int4* prog_node;
  const int32_t *edge_src, *w_bits, *io_pos, *n_rows, *prog_rows;
  const float *obs, *target;
  float *out, *loss;
};

// Genome g by this wavefront; `mine`: its LDS.
template <bool kLoss>
__device__ __forceinline__ void small_genome(const PopView& pop, const SmallIn& in,
                                             const SmallArgs& a, int g, unsigned char* mine) {
  const int32_t* __restrict__ level = in.level;
  const int4* __restrict__ prog_node = in.prog_node;
  const int32_t* __restrict__ edge_src = in.edge_src;
  const int32_t* __restrict__ w_bits = in.w_bits;
  const int32_t* __restrict__ io_pos = in.io_pos;
  const float* __restrict__ target = in.target;
  float* __restrict__ out = in.out;
  float* __restrict__ loss = in.loss;
  const int lane = lane_id();
  const int I = pop.n_in, O = pop.n_out, nio = I + O;
  const SmallLds L = small_lds(a.n_cap, a.c_cap, nio, a.shift);
  int4* node = reinterpret_cast<int4*>(mine + L.node);
  int2* edge = reinterpret_cast<int2*>(mine + L.edge);
  int32_t* lvl = reinterpret_cast<int32_t*>(mine + L.lvl);
  int32_t* io = reinterpret_cast<int32_t*>(mine + L.io);
  float* vals = reinterpret_cast<float*>(mine + L.vals);
  const int64_t nb = uniform64(pop.node_base(g)), cb = uniform64(pop.conn_base(g));
  const int rows = (int)min(pop.node_rows(g), (int64_t)a.n_cap);
  const int64_t out_at = (int64_t)g * a.B * O;

  // everything that needs no size is requested at once: the genome's node
  // rows (the few past its last position are not used) and io positions
  int st = in.status[g];
  const int n = in.n_valid[g];
  if (a.rows_cap < pop.N_max && in.prog_rows[g] > kRegRowsMax && in.n_rows[g] > a.rows_cap) st = -1;
  for (int k = lane; k < nio; k += kWave) io[k] = io_pos[(int64_t)g * nio + k];
  for (int p = lane; p < rows; p += kWave) {
    node[p] = prog_node[nb + p];
    const int lv = level[nb + p], before = p > 0 ? level[nb + p - 1] : -1;
    if (p < n && lv != before) lvl[lv] = p;
    if (p == n - 1) {
      lvl[lv + 1] = n;
      lvl[a.n_cap + 1] = lv + 1;
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
  const float* x = in.obs + (int64_t)g * a.obs_stride;
  {
    DivWalk d(lane, I > 0 ? I : 1, kWave);
    for (int i = lane; i < a.B * I; i += kWave, d.step())
      vals[(io[d.c] << a.shift) + d.b] = x[i];
  }
  wave_sync();
  const int b = lane & ((1 << a.shift) - 1), step = kWave >> a.shift;
  float* v = vals + b;
  const int n_lvl = __builtin_amdgcn_readfirstlane(lvl[a.n_cap + 1]);
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

// kClasses: this launch's size class of the genomes; else every genome fits.
template <bool kLoss, bool kClasses>
__global__ __launch_bounds__(kWave * kSmallWaves) void forward_small_kernel(
    PopView pop, const int32_t* __restrict__ status, const int32_t* __restrict__ n_valid,
    const int32_t* __restrict__ level, const int4* __restrict__ prog_node,
    const int32_t* __restrict__ edge_src, const int32_t* __restrict__ w_bits,
    const int32_t* __restrict__ io_pos, const int32_t* __restrict__ n_rows,
    const int32_t* __restrict__ prog_rows, const float* __restrict__ obs,
    const float* __restrict__ target, float* __restrict__ out, float* __restrict__ loss,
    SmallArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SmallIn in{status, n_valid,   level, prog_node, edge_src, w_bits, io_pos,
                   n_rows, prog_rows, obs,   target,    out,      loss};
  const int wave = blockIdx.x * (blockDim.x / kWave) + wave_id();
  unsigned char* mine = smem + wave_id() * a.wave_bytes;
  if constexpr (!kClasses) {
    if (wave < pop.P) small_genome<kLoss>(pop, in, a, wave, mine);
    return;
  }
  // the launch's genomes among this wavefront's, lane by lane
  const int lane = lane_id(), g0 = wave * a.per_wave, g = g0 + lane;
  bool take = false;
  if (lane < a.per_wave && g < pop.P) {
    const int n = status[g] == 0 ? n_valid[g] : 0;
    const int edges = n > 0 ? prog_node[pop.node_base(g) + n - 1].x : 0;
    take = n <= a.n_cap && edges <= a.c_cap && (n > a.n_prev || edges > a.c_prev);
  }
  for (uint64_t m = __ballot(take); m; m &= m - 1) {
    small_genome<kLoss>(pop, in, a, g0 + __ffsll((unsigned long long)m) - 1, mine);
    wave_sync();  // the next genome overwrites this one's rows
  }
}

// How a launch for genomes of up to n_cap node rows and c_cap in-edges fills the chip.
struct SmallFit {
  int bytes;   // LDS of one wavefront
  int waves;   // wavefronts per workgroup: as many as leave two workgroups to a compute unit
  int64_t resident;  // wavefronts on the chip
};

SmallFit small_fit(int n_cap, int c_cap, int nio, int shift) {
  SmallFit f;
  f.bytes = small_lds(n_cap, c_cap, nio, shift).bytes;
  f.waves = kSmallWaves;
  while (f.waves > 1 && f.waves * f.bytes > 80 * 1024) f.waves /= 2;
  const int64_t groups = (int64_t)max_dynamic_lds() / (f.waves * f.bytes);
  f.resident = kComputeUnits * std::min<int64_t>(32, groups * f.waves);
  return f;
}

// Whether P genomes of these capacities are worth the launch, whatever they
// hold: rounds of resident wavefronts (11 to 18 us each, measured with 40 nodes in
// up to 1024 rows) against the other engines (33 to 42 us for the first round and
// 5 us for every 1000 genomes).
bool small_pays(int n_cap, const SmallFit& f, int64_t P, int shift) {
  if (f.bytes > 96 * 1024) return false;  // one wavefront per compute unit: large genomes lose
  const int64_t rounds = (P + f.resident - 1) / f.resident;
  return (double)rounds * (11.0 + 0.25 * (1 << shift) + n_cap / 256.0) <= 36.0 + 0.005 * (double)P;
}

// Size classes (node rows, in-edges) of populations that do not pay at their own
// capacities, at up to kClassBatch observations: most genomes are smaller
// than what their rows are sized for, and LDS for 128 / 512 rows lets eight
// wavefronts or more onto a compute unit. The larger genomes take a launch at
// 512 / 2048 rows and one at N_max / C_max; a launch that finds none costs 4 us.
// 10,000 genomes of 40 nodes in 1024 / 4096 rows, 8 observations: 70 us, 99 us in
// the other engines, 609 us in one launch at the capacities. Of 500 to 790 nodes
// 5.0 ms, 6.3 and 4.3 ms.
constexpr int kClassNodes[] = {128, 512}, kClassBatch = 16;

enum class SmallForm { kNone, kOne, kClasses };

SmallForm small_form(const tn_population& p, int B) {
  if (p.N_max <= 32 || B <= 0 || B > 32 || (B > kClassBatch && p.P > 2048)) return SmallForm::kNone;
  const int shift = batch_shift(B), nio = p.n_in + p.n_out;
  const SmallFit whole = small_fit(p.N_max, p.C_max, nio, shift);
  if ((size_t)whole.bytes > max_dynamic_lds()) return SmallForm::kNone;
  if (small_pays(p.N_max, whole, p.P, shift)) return SmallForm::kOne;
  const int n = std::min(p.N_max, kClassNodes[0]), c = std::min(p.C_max, 4 * kClassNodes[0]);
  if (B > kClassBatch || whole.bytes > 96 * 1024 || (n == p.N_max && c == p.C_max))
    return SmallForm::kNone;
  return small_pays(n, small_fit(n, c, nio, shift), p.P, shift) ? SmallForm::kClasses
                                                                : SmallForm::kNone;
}

template <bool kLoss>
int launch_small(const tn_population& p, const tn_transformed& t, const float* obs,
                 int64_t obs_stride, int B, const float* target, int64_t target_stride,
                 float scale, float offset, float* out, float* loss, hipStream_t stream) {
  const bool classes = small_form(p, B) == SmallForm::kClasses;
  const int shift = batch_shift(B);
  SmallArgs a{obs_stride, B, shift, target_stride, scale, offset, lds_rows_cap(p)};
  a.n_prev = a.c_prev = -1;
  auto launch = [&](int n_cap, int c_cap) {
    const SmallFit f = small_fit(n_cap, c_cap, p.n_in + p.n_out, shift);
    a.wave_bytes = f.bytes;
    a.n_cap = n_cap;
    a.c_cap = c_cap;
    // (with four wavefronts for each that fits the chip 2000 genomes of 500 to 790
    // nodes took 345 us at B = 1, 317 with one)
    a.per_wave = classes ? (int)std::min<int64_t>(kWave, (p.P + f.resident - 1) / f.resident) : 1;
    const size_t lds = (size_t)f.waves * f.bytes;
    const auto kern = classes ? forward_small_kernel<kLoss, true> : forward_small_kernel<kLoss, false>;
    const int rc = allow_lds((const void*)kern, lds);
    if (rc != TN_OK || p.P == 0) return rc;
    const int64_t per_group = (int64_t)f.waves * a.per_wave;
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.P + per_group - 1) / per_group)),
                       dim3(kWave * f.waves), lds, stream, make_view(p), t.status, t.n_valid, t.level,
                       reinterpret_cast<const int4*>(t.prog_node), t.edge_src,
                       reinterpret_cast<const int32_t*>(t.edge_w), t.io_pos, t.n_rows, t.prog_rows,
                       obs, target, out, loss, a);
    a.n_prev = n_cap;
    a.c_prev = c_cap;
    return check_launch();
  };
  if (classes)
    for (int n : kClassNodes) {
      if (n >= p.N_max && 4 * n >= p.C_max) break;
      const int rc = launch(std::min(n, p.N_max), std::min(4 * n, p.C_max));
      if (rc != TN_OK) return rc;
    }
  return launch(p.N_max, p.C_max);
}

}  // namespace

bool small_batch(const tn_population& p, int B) { return small_form(p, B) != SmallForm::kNone; }

int launch_forward_small(const tn_population& p, const tn_transformed& t, const float* obs,
                         int64_t obs_stride, int B, const float* target, int64_t target_stride,
                         float scale, float offset, float* out, float* loss, hipStream_t stream) {
  return loss ? launch_small<true>(p, t, obs, obs_stride, B, target, target_stride, scale, offset,
                                   out, loss, stream)
              : launch_small<false>(p, t, obs, obs_stride, B, nullptr, 0, 0.0f, 0.0f, out, nullptr,
                                    stream);
}

}  // namespace tn
