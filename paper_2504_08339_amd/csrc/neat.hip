// One NEAT generation on the device (Algorithm 1's loop body: divide the
// population into species by distance, decide each species' number of
// children from the fitness, make them by crossover and mutation) and the
// initial population (Algorithm 1's first step); hyperparameters of Appendix
// A. The paper names these steps, not their rules; the rules implemented are
// stated at tn_neat_generation in the public header.
//
// Launches of one generation, all on the caller's stream:
//   prep        sorted gene lists of the population and of the species
//               representatives (the node-inclusive distance's genes);
//   reps        every genome against every alive representative: a wavefront
//               per 16 genomes and representative;
//   assign      thread per genome: the nearest representative below the
//               threshold; the first genome without one;
//   found       one round per founded species: the round's founder (the first
//               genome in index order that no earlier founder is near) against
//               every later genome without a species. A genome's choice
//               depends only on the founders before it, so the rounds give
//               what going through the genomes one by one gives;
//   settle      thread per genome: the species of the genomes left;
//   stats       wavefront per slot: members, largest and smallest fitness, sum;
//   counts      one wavefront, lane per slot: stagnation, offspring counts
//               (float32 as specified, sums in slot order);
//   rank        wavefront per four genomes: their ranks in their species,
//               scattered into the member order;
//   parents     thread per child: elites, then two survivor picks;
//   reproduce   the crossover / mutation kernels;
//   table       workgroup per slot: next representatives and slot state.
// Every float decision (distance below the threshold, nearest species,
// counts) uses float32 operations in a fixed order with no contraction.
#include <algorithm>
#include <climits>
#include <cmath>

#include "genes.hpp"
#include "tn_internal.hpp"

#pragma clang fp contract(off)

namespace tn {

size_t reproduce_workspace_bytes(int n);
int launch_reproduce(const tn_population& p, int n, const int32_t* parents, const float* U,
                     const float* Z, const tn_mutation_params& prm, int32_t next_key,
                     const tn_population_arrays& out, int32_t* next_key_out, void* workspace,
                     hipStream_t stream);

namespace {

constexpr int kBlock = 256;
constexpr int kMaxSpecies = TN_NEAT_MAX_SPECIES;

struct NeatWs {
  WsN pop;             // gene lists of the population, genome-major
  WsN reps;            // gene lists of the representatives, genome-major
  float* dist;         // [S][P] distance to the slot's representative or founder
  int32_t* sp;         // [P] species slot of each genome
  int32_t* near;       // [P] a founder before this genome is below the threshold
  int32_t* order;      // [P] genomes by slot, then rank
  int32_t* parents;    // [P][2]
  int32_t* founders;   // [S + 1] founder of each round (INT_MAX: none)
  int32_t* member_off; // [S + 1]
  int32_t* child_off;  // [S + 1]
  int32_t* counts;     // [S]
  int32_t* nmem;       // [S]
  int32_t* surv;       // [S]
  float* smax;         // [S] largest member fitness
  float* smin;         // [S] smallest
  float* ssum;         // [S] sum in ascending genome order
  float* best;         // [S] updated best species fitness
  int32_t* last;       // [S] updated generation of the last improvement
  void* repro;         // workspace of the reproduction kernels
};

struct Table {
  int32_t* alive;
  float* best;
  int32_t* last;
  int32_t* size;
  tn_population_arrays reps;
};

// Carves the workspace at `base` (null: its size alone); *bytes (may be null): its size.
NeatWs carve(void* base, int P, int S, int N, int C, size_t* bytes) {
  const uintptr_t p = (uintptr_t)base;
  size_t o = 0;
  NeatWs w;
  w.pop = carve_nodes((void*)(p + o), P, N, C);
  o += ws_nodes_bytes(P, N, C);
  w.reps = carve_nodes((void*)(p + o), S, N, C);
  o += ws_nodes_bytes(S, N, C);
  auto ints = [&](size_t n) {
    int32_t* q = (int32_t*)(p + o);
    o += gene_align(4 * n);
    return q;
  };
  w.dist = (float*)ints((size_t)S * P);
  w.sp = ints(P);
  w.near = ints(P);
  w.order = ints(P);
  w.parents = ints(2 * (size_t)P);
  w.founders = ints(S + 1);
  w.member_off = ints(S + 1);
  w.child_off = ints(S + 1);
  w.counts = ints(S + 1);
  w.nmem = ints(S + 1);
  w.surv = ints(S + 1);
  w.smax = (float*)ints(S + 1);
  w.smin = (float*)ints(S + 1);
  w.ssum = (float*)ints(S + 1);
  w.best = (float*)ints(S + 1);
  w.last = ints(S + 1);
  w.repro = (void*)(p + o);
  if (bytes) *bytes = o + gene_align(reproduce_workspace_bytes(P));
  return w;
}

__device__ __forceinline__ float draw(float mean, float std_, float z) {
  const float t = std_ * z;
  return mean + t;
}

__global__ __launch_bounds__(kBlock) void init_kernel(int n_in, int n_out, int N, int C,
                                                      const float* Z, int64_t nZ,
                                                      tn_mutation_params m,
                                                      tn_population_arrays out) {
  const int g = blockIdx.x;
  const float* z = Z + (int64_t)g * nZ;
  const int nio = n_in + n_out;
  const int64_t nb = (int64_t)g * N, cb = (int64_t)g * C;
  for (int r = threadIdx.x; r < N; r += kBlock) {
    const bool v = r < nio;
    out.node_key[nb + r] = v ? r : -1;
    out.node_bias[nb + r] = v ? draw(m.bias_init_mean, m.bias_init_std, z[4 + 2 * r]) : 0.0f;
    out.node_resp[nb + r] = v ? draw(m.resp_init_mean, m.resp_init_std, z[4 + 2 * r + 1]) : 0.0f;
    out.node_act[nb + r] = v ? (uint8_t)m.act_default : 0;
    out.node_agg[nb + r] = v ? (uint8_t)m.agg_default : 0;
  }
  for (int r = threadIdx.x; r < C; r += kBlock) {
    const bool v = r < n_in * n_out;
    out.conn_in[cb + r] = v ? r / n_out : -1;
    out.conn_out[cb + r] = v ? n_in + r % n_out : -1;
    out.conn_w[cb + r] =
        v ? draw(m.weight_init_mean, m.weight_init_std, z[4 + 2 * (int64_t)N + r]) : 0.0f;
    out.conn_en[cb + r] = v ? 1 : 0;
  }
}

__global__ __launch_bounds__(kBlock) void clear_table_kernel(Table t, int N, int C) {
  const int s = blockIdx.x;
  if (threadIdx.x == 0) {
    t.alive[s] = 0;
    t.best[s] = -INFINITY;
    t.last[s] = 0;
    t.size[s] = 0;
  }
  const int64_t nb = (int64_t)s * N, cb = (int64_t)s * C;
  for (int r = threadIdx.x; r < N; r += kBlock) {
    t.reps.node_key[nb + r] = -1;
    t.reps.node_bias[nb + r] = t.reps.node_resp[nb + r] = 0.0f;
    t.reps.node_act[nb + r] = t.reps.node_agg[nb + r] = 0;
  }
  for (int r = threadIdx.x; r < C; r += kBlock) {
    t.reps.conn_in[cb + r] = t.reps.conn_out[cb + r] = -1;
    t.reps.conn_w[cb + r] = 0.0f;
    t.reps.conn_en[cb + r] = 0;
  }
}

__global__ __launch_bounds__(kWave) void prep_kernel(PopView pop, WsN pop_ws, PopView reps,
                                                     WsN reps_ws, int SN, int SC) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int g = blockIdx.x;
  if (g < pop.P)
    prep_genes<true>(pop, pop_ws, g, SN, SC, smem);
  else
    prep_genes<true>(reps, reps_ws, g - pop.P, SN, SC, smem);
}

// Distances of many genomes to one target genome, whose sorted keys sit in
// LDS. A wavefront takes kTile genomes: for each, its lanes take 64 genes at a
// time, find them in the target's keys by binary search and put each gene's
// term (0 where it is not shared) into the wavefront's LDS rows; then lane q
// adds genome q's 64 terms in ascending key order. The sum is one serial chain
// per pair (its order is part of the result), so 16 pairs run it side by side,
// and adding the zeros changes no bit of a sum of non-negative terms. Bound by
// the searches' LDS round trips and the serial sums. 5000 genomes of 40 node
// and 164 connection rows against 10 representatives: 84 us, and 8 us for each
// founder. (One workgroup that merged the lists pair by pair and took the
// genomes without a species one after another spent 248 ms on this step.)
constexpr int kTile = 16;
constexpr int kTermRow = kWave + 1;
constexpr int kTermBytes = sizeof(float) * kTile * kTermRow;  // LDS per wavefront

struct Target {
  const long long* nodes;  // LDS
  const long long* conns;  // LDS
  int n_nodes, n_conns;    // -1: no gene set
};

// Copies target genome b's keys into LDS; every thread of the workgroup calls
// it. The caller synchronises before and after.
__device__ __forceinline__ Target load_target(const WsN& B, int N, int C, int b, long long* lds) {
  Target t;
  t.n_nodes = B.cnt_n[b];
  t.n_conns = B.cnt_c[b];
  t.nodes = lds;
  t.conns = lds + N;
  for (int k = threadIdx.x; k < t.n_nodes; k += blockDim.x) lds[k] = B.nodes.keyT[(int64_t)b * N + k];
  for (int k = threadIdx.x; k < t.n_conns; k += blockDim.x)
    lds[N + k] = B.conns.keyT[(int64_t)b * C + k];
  return t;
}

// (c_d * D + c_h * H) / max(n1, n2) of one gene kind for genomes g0 + q (lane
// q < kTile): H summed in ascending key order, each term
// ((|da0| + |da1|) + [c0 differ]) + [c1 differ]. na: this lane's gene count.
__device__ __forceinline__ float kind_term(const GeneList& A, int cap, int g0, int na,
                                           const GeneList& B, int b, const long long* keys, int nb,
                                           float* terms, float c_d, float c_h) {
  const int lane = lane_id();
  int most = na;
#pragma unroll
  for (int off = kTile / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, kWave));
  most = __builtin_amdgcn_readfirstlane(most);
  int top = 1;  // the largest power of two within nb
  while (2 * top <= nb) top *= 2;
  int hom = 0;
  float H = 0.0f;
  for (int base = 0; base < most; base += kWave) {
    const int k = base + lane;
#pragma unroll 4
    for (int q = 0; q < kTile; ++q) {
      const int nq = __builtin_amdgcn_readlane(na, q);
      bool found = false;
      float t = 0.0f;
      if (k < nq) {
        const int64_t oa = (int64_t)(g0 + q) * cap + k;
        const long long key = A.keyT[oa];
        int at = 0;
        for (int step = top; step > 0; step >>= 1)
          if (at + step <= nb && keys[at + step - 1] < key) at += step;
        found = at < nb && keys[at] == key;
        if (found) {
          const int64_t ob = (int64_t)b * cap + at;
          t = fabsf(A.a0T[oa] - B.a0T[ob]) + fabsf(A.a1T[oa] - B.a1T[ob]);
          const uint32_t ca = A.codeT[oa], cb = B.codeT[ob];
          t = t + ((ca & 0xffu) != (cb & 0xffu) ? 1.0f : 0.0f);
          t = t + ((ca >> 8) != (cb >> 8) ? 1.0f : 0.0f);
        }
      }
      const uint64_t m = __ballot(found);
      if (lane == q) hom += __popcll(m);
      terms[q * kTermRow + lane] = t;
    }
    wave_sync();
    const float* mine = terms + (lane & (kTile - 1)) * kTermRow;
#pragma unroll 16
    for (int j = 0; j < kWave; ++j) H = H + mine[j];
    wave_sync();
  }
  const int n = max(na, nb);
  if (n == 0) return 0.0f;
  const float x = c_d * (float)(na + nb - 2 * hom);
  const float y = c_h * H;
  const float num = x + y;
  return num / (float)n;
}

// Node-inclusive distance of genome g0 + q of A and genome b of B on lane q <
// kTile (NaN when either has no gene set; genomes from P on count as empty).
__device__ __forceinline__ float tile_distance(const WsN& A, int P, int N, int C, int g0,
                                               const WsN& B, int b, const Target& t, float* terms,
                                               float c_d, float c_h) {
  const int g = g0 + (lane_id() & (kTile - 1));
  const bool real = lane_id() < kTile && g < P;
  const int an = real ? A.cnt_n[g] : 0, ac = real ? A.cnt_c[g] : 0;
  if (t.n_nodes < 0) return __builtin_nanf("");
  const float tn = kind_term(A.nodes, N, g0, max(an, 0), B.nodes, b, t.nodes, t.n_nodes, terms,
                             c_d, c_h);
  const float tc = kind_term(A.conns, C, g0, max(ac, 0), B.conns, b, t.conns, t.n_conns, terms,
                             c_d, c_h);
  float total = 0.0f;
  total = total + tn;
  total = total + tc;
  return an < 0 ? __builtin_nanf("") : total;
}

struct SpecArgs {
  int P, S, N, C, gen;
  float thr, c_d, c_h;
  int species_elitism, max_stagnation;
  float rate;
};

// dist[s][g] of every genome and alive representative (workgroups of slot s:
// blockIdx.y = s); the founder list is emptied.
__global__ __launch_bounds__(kBlock) void reps_kernel(NeatWs ws, Table t, SpecArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int s = blockIdx.y;
  if (blockIdx.x == 0 && s == 0)
    for (int r = threadIdx.x; r <= a.S; r += kBlock) ws.founders[r] = INT_MAX;
  if (!t.alive[s]) return;
  float* terms = (float*)(smem + sizeof(long long) * (size_t)(a.N + a.C)) +
                 wave_id() * kTile * kTermRow;
  const Target tg = load_target(ws.reps, a.N, a.C, s, (long long*)smem);
  __syncthreads();
  const int W = kBlock / kWave;
  for (int g0 = (blockIdx.x * W + wave_id()) * kTile; g0 < a.P; g0 += gridDim.x * W * kTile) {
    const float d = tile_distance(ws.pop, a.P, a.N, a.C, g0, ws.reps, s, tg, terms, a.c_d, a.c_h);
    const int g = g0 + lane_id();
    if (lane_id() < kTile && g < a.P) ws.dist[(int64_t)s * a.P + g] = d;
  }
}

// The nearest alive representative below the threshold (ties: lowest slot);
// the first genome without one founds the first species if a slot is free.
__global__ __launch_bounds__(kBlock) void assign_kernel(NeatWs ws, Table t, SpecArgs a) {
  const int g = blockIdx.x * kBlock + threadIdx.x;
  if (g >= a.P) return;
  int best = -1;
  float bd = 0.0f;
  for (int s = 0; s < a.S; ++s) {
    if (!t.alive[s]) continue;
    const float d = ws.dist[(int64_t)s * a.P + g];
    if (d < a.thr && (best < 0 || d < bd)) {
      best = s;
      bd = d;
    }
  }
  ws.sp[g] = best;
  ws.near[g] = 0;
  if (best < 0) atomicMin(&ws.founders[0], g);
}

// Slot of founding round r (the r-th free slot), or -1; the same on every lane.
__device__ __forceinline__ int round_slot(const Table& t, int S, int r) {
  const int lane = lane_id();
  const bool open = lane < S && !t.alive[lane];
  const uint64_t m = __ballot(open && mbcnt(__ballot(open)) == r);
  return m ? __ffsll((unsigned long long)m) - 1 : -1;
}

// Founding rounds r0 .. r1 - 1: over the grid for one round, or by a single
// workgroup for all of them. Round r's founder is founders[r]; its distances
// to the later genomes without a species fill its slot's row of dist, and the
// first of them that no founder so far is near becomes founders[r + 1].
__global__ __launch_bounds__(1024) void found_kernel(NeatWs ws, Table t, SpecArgs a, int r0,
                                                     int r1) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* terms = (float*)(smem + sizeof(long long) * (size_t)(a.N + a.C)) +
                 wave_id() * kTile * kTermRow;
  const int W = blockDim.x / kWave, lane = lane_id();
  for (int r = r0; r < r1; ++r) {
    const int slot = round_slot(t, a.S, r);
    const int f = __hip_atomic_load(&ws.founders[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (slot < 0 || f == INT_MAX) return;  // the same on every thread
    const Target tg = load_target(ws.pop, a.N, a.C, f, (long long*)smem);
    __syncthreads();
    for (int g0 = (blockIdx.x * W + wave_id()) * kTile; g0 < a.P; g0 += gridDim.x * W * kTile) {
      const int g = g0 + lane;
      const bool todo = lane < kTile && g < a.P && g > f && ws.sp[g] < 0;
      if (__ballot(todo) == 0) continue;
      const float d = tile_distance(ws.pop, a.P, a.N, a.C, g0, ws.pop, f, tg, terms, a.c_d, a.c_h);
      if (!todo) continue;
      ws.dist[(int64_t)slot * a.P + g] = d;
      if (d < a.thr)
        ws.near[g] = 1;
      else if (!ws.near[g])
        atomicMin(&ws.founders[r + 1], g);
    }
    __threadfence();
    __syncthreads();
  }
}

// The species of the genomes left: a founder's own slot; the nearest founder
// before the genome if below the threshold; past the founder of the last free
// slot the nearest alive species whatever the distance (NaN counts as
// infinite). Ties: lowest slot. Also stored to species_of (may be null).
__global__ __launch_bounds__(kBlock) void settle_kernel(NeatWs ws, Table t, SpecArgs a,
                                                        int32_t* species_of) {
  __shared__ int by_slot[kMaxSpecies];  // founder; -1: a representative; INT_MAX: not alive
  __shared__ int full_from;             // genomes after this one find no free slot
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    const bool open = lane < a.S && !t.alive[lane];
    const int r = mbcnt(__ballot(open));
    const int f = open ? ws.founders[r] : INT_MAX;
    if (lane < a.S) by_slot[lane] = open ? f : -1;
    const uint64_t opens = __ballot(open), took = __ballot(open && f != INT_MAX);
    int last = -1;
    for (int s = 0; s < a.S; ++s)
      if ((took >> s) & 1) last = max(last, __builtin_amdgcn_readlane(f, s));
    if (lane == 0) full_from = opens == took ? last : INT_MAX;
  }
  __syncthreads();
  const int g = blockIdx.x * kBlock + threadIdx.x;
  if (g >= a.P) return;
  int best = ws.sp[g];
  if (best < 0) {
    const bool any = g > full_from;
    float bd = 0.0f;
    for (int s = 0; s < a.S; ++s) {
      const int f = by_slot[s];
      if (f == g) {
        best = s;
        break;
      }
      if (f > g || (!any && f < 0)) continue;  // not alive at this genome's turn, or no founder
      float d = ws.dist[(int64_t)s * a.P + g];
      if (any) d = d != d ? INFINITY : d;
      if ((any || d < a.thr) && (best < 0 || d < bd)) {
        best = s;
        bd = d;
      }
    }
    ws.sp[g] = best;
  }
  if (species_of) species_of[g] = best;
}

// Members, largest and smallest fitness (the first of equal ones) and the sum
// in ascending genome order of slot blockIdx.x. The sum is one serial chain: the
// workgroup first packs a segment's members into LDS in genome order (counts of
// all its chunks in one prefix sum), then a wavefront adds them 16 reads ahead.
// 5000 genomes, 10 species: 23 us; 69 us by one wavefront that took the chain
// over all genomes, members or not, from its lanes.
constexpr int kStatsWaves = 4, kStatsChunks = kWave / kStatsWaves;
constexpr int kStatsSegment = kStatsChunks * kStatsWaves * kWave;

__global__ __launch_bounds__(kWave * kStatsWaves) void stats_kernel(NeatWs ws, const float* fit,
                                                                    int P) {
  constexpr int T = kWave * kStatsWaves;
  __shared__ __align__(16) float member[kStatsSegment];
  __shared__ int start[kWave];  // of a wavefront's part of a chunk: [chunk][wavefront]
  __shared__ float wmx[kStatsWaves], wmn[kStatsWaves];
  __shared__ int wimx[kStatsWaves], wimn[kStatsWaves];
  const int s = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  int total = 0, imx = INT_MAX, imn = INT_MAX;
  float mx = -INFINITY, mn = INFINITY, sum = 0.0f;
  for (int base = 0; base < P; base += kStatsSegment) {
    float f[kStatsChunks];
    uint64_t in[kStatsChunks];
#pragma unroll
    for (int u = 0; u < kStatsChunks; ++u) {
      const int g = base + u * T + tid, gg = min(g, P - 1);
      const int sp = ws.sp[gg];
      f[u] = fit[gg];
      in[u] = __ballot(g < P && sp == s);
    }
#pragma unroll
    for (int u = 0; u < kStatsChunks; ++u) {
      if ((in[u] >> lane) & 1) {
        const int g = base + u * T + tid;
        if (f[u] > mx) {
          mx = f[u];
          imx = g;
        }
        if (f[u] < mn) {
          mn = f[u];
          imn = g;
        }
      }
      if (lane == 0) start[u * kStatsWaves + wave] = __popcll(in[u]);
    }
    lds_barrier();
    const int count = start[lane];
    const int upto = wave_inclusive_scan(count);
    const int n = __builtin_amdgcn_readlane(upto, kWave - 1);
    const int mine = upto - count;
#pragma unroll
    for (int u = 0; u < kStatsChunks; ++u) {
      const int at = __builtin_amdgcn_readlane(mine, u * kStatsWaves + wave);
      if ((in[u] >> lane) & 1) member[at + mbcnt(in[u])] = f[u];
    }
    lds_barrier();
    total += n;
    if (wave == 0) {  // one chain of additions in genome order
      int i = 0;
      for (; i + 16 <= n; i += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = member[i + k];
#pragma unroll
        for (int k = 0; k < 16; ++k) sum = sum + v[k];
      }
      for (; i < n; ++i) sum = sum + member[i];
    }
    lds_barrier();  // the next segment overwrites the members
  }
  // the larger maximum and the smaller minimum, of equal ones the earlier genome's
  auto take = [](float& mx, int& imx, float& mn, int& imn, float omx, int oimx, float omn,
                 int oimn) {
    if (omx > mx || (omx == mx && oimx < imx)) {
      mx = omx;
      imx = oimx;
    }
    if (omn < mn || (omn == mn && oimn < imn)) {
      mn = omn;
      imn = oimn;
    }
  };
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    take(mx, imx, mn, imn, __shfl_xor(mx, off, kWave), __shfl_xor(imx, off, kWave),
         __shfl_xor(mn, off, kWave), __shfl_xor(imn, off, kWave));
  }
  if (lane == 0) {
    wmx[wave] = mx;
    wmn[wave] = mn;
    wimx[wave] = imx;
    wimn[wave] = imn;
  }
  lds_barrier();
  if (tid == 0) {
    for (int w = 1; w < kStatsWaves; ++w) take(mx, imx, mn, imn, wmx[w], wimx[w], wmn[w], wimn[w]);
    ws.nmem[s] = total;
    ws.smax[s] = mx;
    ws.smin[s] = mn;
    ws.ssum[s] = sum;
  }
}

__device__ __forceinline__ float lane_value(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// Stagnation and offspring counts, lane = slot; sums over slots in slot order.
__global__ __launch_bounds__(kWave) void counts_kernel(NeatWs ws, Table t, SpecArgs a) {
  const int s = threadIdx.x, P = a.P, S = a.S;
  const bool slot = s < S;
  const bool open = slot && !t.alive[s];
  const bool founded = open && ws.founders[mbcnt(__ballot(open))] != INT_MAX;
  const int nmem = slot ? ws.nmem[s] : 0;
  const float smax = slot ? ws.smax[s] : -INFINITY, smin = slot ? ws.smin[s] : INFINITY;
  float best = founded ? -INFINITY : (slot ? t.best[s] : -INFINITY);
  int last = founded ? a.gen : (slot ? t.last[s] : 0);
  if (nmem > 0 && smax > best) {
    best = smax;
    last = a.gen;
  }
  // the species_elitism largest species fitnesses are kept (ties: lowest slot)
  int above = 0;
  for (int o = 0; o < S; ++o) {
    const float x = lane_value(smax, o);
    above += __builtin_amdgcn_readlane(nmem, o) > 0 && (x > smax || (x == smax && o < s)) ? 1 : 0;
  }
  const bool surv = nmem > 0 && (above < a.species_elitism || a.gen - last < a.max_stagnation);
  const uint64_t alive = __ballot(surv);
  const int nsurv = __popcll(alive);
  int cnt = 0;
  if (nsurv > 0) {
    float lo = INFINITY, hi = -INFINITY;
    for (int o = 0; o < S; ++o) {
      if (!((alive >> o) & 1)) continue;
      const float l = lane_value(smin, o), h = lane_value(smax, o);
      lo = l < lo ? l : lo;
      hi = h > hi ? h : hi;
    }
    const float d = hi - lo;
    const float rng = d > 1.0f ? d : 1.0f;
    const float mean = (slot ? ws.ssum[s] : 0.0f) / (float)nmem;
    const float af = (mean - lo) / rng;
    float af_sum = 0.0f;
    for (int o = 0; o < S; ++o)
      if ((alive >> o) & 1) af_sum = af_sum + lane_value(af, o);
    const float fP = (float)P, ns = (float)nsurv;
    const float target = af_sum > 0.0f ? (fP * af) / af_sum : fP / ns;
    const float prev = (slot ? (float)t.size[s] : 0.0f) * (founded ? 0.0f : 1.0f);
    const float spawn = prev + (target - prev) * a.rate;
    float sp_sum = 0.0f;
    for (int o = 0; o < S; ++o)
      if ((alive >> o) & 1) sp_sum = sp_sum + lane_value(spawn, o);
    const float share = sp_sum > 0.0f ? (spawn * fP) / sp_sum : fP / ns;
    const bool fine = __builtin_isfinite(share) && share >= 0.0f && share < 1073741824.0f;
    const bool ok = __ballot(surv && !fine) == 0;
    cnt = surv && ok ? (int)floorf(share) : 0;
    const int left = P - wave_sum_int(cnt);
    if (!ok || left < 0 || left > nsurv) {  // non-finite fitness: equal split
      cnt = surv ? P / nsurv + (mbcnt(alive) < P % nsurv ? 1 : 0) : 0;
    } else {  // one more each by largest remainder, ties lowest slot
      const float rest = share - (float)cnt;
      int before = 0;
      for (int o = 0; o < S; ++o) {
        const float x = lane_value(rest, o);
        before += ((alive >> o) & 1) && (x > rest || (x == rest && o < s)) ? 1 : 0;
      }
      if (surv && before < left) ++cnt;
    }
  }
  const int mo = wave_inclusive_scan(nmem), co = wave_inclusive_scan(cnt);
  if (slot) {
    ws.member_off[s] = mo - nmem;
    ws.child_off[s] = co - cnt;
    ws.counts[s] = cnt;
    ws.surv[s] = surv ? 1 : 0;
    ws.best[s] = best;
    ws.last[s] = last;
  }
  if (s == S - 1) {
    ws.member_off[S] = mo;
    ws.child_off[S] = co;
  }
}

// rank of genome g in its species: members of larger fitness, or of equal
// fitness and lower index (a NaN counts as the lowest, so every rank is taken
// once). A wavefront takes kRanks genomes, its lanes the population.
constexpr int kRanks = 4;

__device__ __forceinline__ float ranked(float f) { return f == f ? f : -INFINITY; }

__global__ __launch_bounds__(kBlock) void rank_kernel(NeatWs ws, const float* fit, int P) {
  const int lane = lane_id();
  const int g0 = (blockIdx.x * (kBlock / kWave) + wave_id()) * kRanks;
  if (g0 >= P) return;
  int s[kRanks], rank[kRanks];
  float f[kRanks];
#pragma unroll
  for (int i = 0; i < kRanks; ++i) {
    s[i] = g0 + i < P ? ws.sp[g0 + i] : -1;
    f[i] = g0 + i < P ? ranked(fit[g0 + i]) : 0.0f;
    rank[i] = 0;
  }
#pragma unroll 4
  for (int h = lane; h < P; h += kWave) {
    const int sh = ws.sp[h];
    const float fh = ranked(fit[h]);
#pragma unroll
    for (int i = 0; i < kRanks; ++i)
      rank[i] += sh == s[i] && (fh > f[i] || (fh == f[i] && h < g0 + i)) ? 1 : 0;
  }
#pragma unroll
  for (int i = 0; i < kRanks; ++i) {
    const int r = wave_sum_int(rank[i]);
    if (lane == 0 && g0 + i < P) ws.order[ws.member_off[s[i]] + r] = g0 + i;
  }
}

__device__ __forceinline__ int pick(float u, int n) {
  const int k = (int)floorf(u * (float)n);
  return min(k, n - 1);
}

__global__ __launch_bounds__(kBlock) void parents_kernel(NeatWs ws, const float* fit,
                                                         const float* sel, int P, int S,
                                                         int genome_elitism, float survival,
                                                         int32_t* parents_out) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= P) return;
  int s = 0;
  while (s < S && !(ws.child_off[s] <= c && c < ws.child_off[s] + ws.counts[s])) ++s;
  int pa = -1, pb = -1;
  if (s < S) {
    const int i = c - ws.child_off[s];
    const int n = ws.nmem[s];
    const int* ms = ws.order + ws.member_off[s];
    const int e = min(min(genome_elitism, ws.counts[s]), n);
    if (i < e) {
      pa = ms[i];
    } else {
      const int k = max(1, (int)ceilf(survival * (float)n));
      pa = ms[pick(sel[2 * (int64_t)c], k)];
      pb = ms[pick(sel[2 * (int64_t)c + 1], k)];
      if (fit[pb] > fit[pa] || (fit[pb] == fit[pa] && pb < pa)) {
        const int x = pa;
        pa = pb;
        pb = x;
      }
    }
  }
  ws.parents[2 * (int64_t)c] = pa;
  ws.parents[2 * (int64_t)c + 1] = pb;
  if (parents_out) {
    parents_out[2 * (int64_t)c] = pa;
    parents_out[2 * (int64_t)c + 1] = pb;
  }
}

__global__ __launch_bounds__(kBlock) void table_kernel(NeatWs ws, Table t, PopView pop) {
  const int s = blockIdx.x;
  const bool keep = ws.surv[s] && ws.counts[s] > 0;
  if (threadIdx.x == 0) {
    t.alive[s] = keep ? 1 : 0;
    t.best[s] = keep ? ws.best[s] : -INFINITY;
    t.last[s] = keep ? ws.last[s] : 0;
    t.size[s] = keep ? ws.counts[s] : 0;
  }
  if (!keep) return;
  const int g = ws.order[ws.member_off[s]];
  const int N = pop.N_max, C = pop.C_max;
  const int64_t sb = (int64_t)s * N, gb = (int64_t)g * N;
  for (int r = threadIdx.x; r < N; r += kBlock) {
    t.reps.node_key[sb + r] = pop.node_key[gb + r];
    t.reps.node_bias[sb + r] = pop.node_bias[gb + r];
    t.reps.node_resp[sb + r] = pop.node_resp[gb + r];
    t.reps.node_act[sb + r] = pop.node_act[gb + r];
    t.reps.node_agg[sb + r] = pop.node_agg[gb + r];
  }
  const int64_t sc = (int64_t)s * C, gc = (int64_t)g * C;
  for (int r = threadIdx.x; r < C; r += kBlock) {
    t.reps.conn_in[sc + r] = pop.conn_in[gc + r];
    t.reps.conn_out[sc + r] = pop.conn_out[gc + r];
    t.reps.conn_w[sc + r] = pop.conn_w[gc + r];
    t.reps.conn_en[sc + r] = pop.conn_en[gc + r];
  }
}

Table table_of(const tn_species_table& t) {
  Table x;
  x.alive = t.alive;
  x.best = t.best;
  x.last = t.last_improved;
  x.size = t.size;
  x.reps = t.reps;
  return x;
}

}  // namespace

size_t neat_workspace_bytes(int P, int S, int N, int C) {
  size_t bytes = 0;
  (void)carve(nullptr, P, S, N, C, &bytes);
  return bytes;
}

int launch_neat_init(int P, int n_in, int n_out, int N, int C, const float* Z,
                     const tn_mutation_params& m, const tn_population_arrays& out,
                     const tn_species_table* table, hipStream_t stream) {
  if (P > 0) {
    int nU = 0, nZ = 0;
    tn_reproduce_draws(N, C, &nU, &nZ);
    hipLaunchKernelGGL(init_kernel, dim3(P), dim3(kBlock), 0, stream, n_in, n_out, N, C, Z,
                       (int64_t)nZ, m, out);
    int rc = check_launch();
    if (rc != TN_OK) return rc;
  }
  if (table) {
    hipLaunchKernelGGL(clear_table_kernel, dim3(table->max_species), dim3(kBlock), 0, stream,
                       table_of(*table), N, C);
    return check_launch();
  }
  return TN_OK;
}

int launch_neat_generation(const tn_population& p, const float* fit, int gen,
                           const tn_neat_params& prm, const tn_species_table& table,
                           const float* sel, const float* U, const float* Z, int32_t next_key,
                           const tn_population_arrays& children, int32_t* species_of,
                           int32_t* parents, int32_t* next_key_out, void* workspace,
                           hipStream_t stream) {
  const int P = p.P, S = table.max_species, N = p.N_max, C = p.C_max;
  const size_t prep_lds = prep_nodes_lds(N, C);
  const size_t key_lds = sizeof(long long) * (size_t)(N + C);
  const size_t reps_lds = key_lds + (kBlock / kWave) * (size_t)kTermBytes;
  // Founding rounds: up to kOneBlock genomes one workgroup runs them all (one
  // launch); more genomes take one launch over the grid per free slot at most,
  // which end at once when no founder is left.
  constexpr int kOneBlock = 512;
  const bool one = P <= kOneBlock;
  const int found_waves = one ? (P + kTile - 1) / kTile < 16 ? (P + kTile - 1) / kTile : 16
                              : kBlock / kWave;
  const size_t found_lds = key_lds + found_waves * (size_t)kTermBytes;
  int rc = allow_lds((const void*)prep_kernel, prep_lds);
  if (rc == TN_OK) rc = allow_lds((const void*)reps_kernel, reps_lds);
  if (rc == TN_OK) rc = allow_lds((const void*)found_kernel, found_lds);
  if (rc != TN_OK) return rc;
  NeatWs ws = carve(workspace, P, S, N, C, nullptr);
  const Table t = table_of(table);
  // gene lists of the population and of the representatives
  const PopView pv = make_view(p);
  tn_population rp = p;
  rp.P = S;
  rp.node_key = table.reps.node_key;
  rp.node_bias = table.reps.node_bias;
  rp.node_resp = table.reps.node_resp;
  rp.node_act = table.reps.node_act;
  rp.node_agg = table.reps.node_agg;
  rp.conn_in = table.reps.conn_in;
  rp.conn_out = table.reps.conn_out;
  rp.conn_w = table.reps.conn_w;
  rp.conn_en = table.reps.conn_en;
  hipLaunchKernelGGL(prep_kernel, dim3(P + S), dim3(kWave), prep_lds, stream, pv, ws.pop,
                     make_view(rp), ws.reps, gene_pow2(N), gene_pow2(C));
  rc = check_launch();
  if (rc != TN_OK) return rc;
  SpecArgs a;
  a.P = P;
  a.S = S;
  a.N = N;
  a.C = C;
  a.gen = gen;
  a.thr = prm.compatibility_threshold;
  a.c_d = prm.compatibility_disjoint;
  a.c_h = prm.compatibility_homologous;
  a.species_elitism = prm.species_elitism;
  a.max_stagnation = prm.max_stagnation;
  a.rate = prm.spawn_number_change_rate;
  const int blocks = (P + kBlock - 1) / kBlock;
  const int tiles = (P + kTile * (kBlock / kWave) - 1) / (kTile * (kBlock / kWave));
  hipLaunchKernelGGL(reps_kernel, dim3(tiles, S), dim3(kBlock), reps_lds, stream, ws, t, a);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(assign_kernel, dim3(blocks), dim3(kBlock), 0, stream, ws, t, a);
  rc = check_launch();
  for (int r = 0; r < (one ? 1 : S) && rc == TN_OK; ++r) {
    hipLaunchKernelGGL(found_kernel, dim3(one ? 1 : tiles), dim3(found_waves * kWave), found_lds,
                       stream, ws, t, a, r, one ? S : r + 1);
    rc = check_launch();
  }
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(settle_kernel, dim3(blocks), dim3(kBlock), 0, stream, ws, t, a, species_of);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(stats_kernel, dim3(S), dim3(kWave * kStatsWaves), 0, stream, ws, fit, P);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(counts_kernel, dim3(1), dim3(kWave), 0, stream, ws, t, a);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  const int per = kRanks * (kBlock / kWave);
  hipLaunchKernelGGL(rank_kernel, dim3((P + per - 1) / per), dim3(kBlock), 0, stream, ws, fit, P);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(parents_kernel, dim3(blocks), dim3(kBlock), 0, stream, ws, fit, sel, P, S,
                     prm.genome_elitism, prm.survival_threshold, parents);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  rc = launch_reproduce(p, P, ws.parents, U, Z, prm.mutation, next_key, children, next_key_out,
                        ws.repro, stream);
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(table_kernel, dim3(S), dim3(kBlock), 0, stream, ws, t, pv);
  return check_launch();
}

}  // namespace tn
