// Forward pass of recurrent networks (network type "recurrent" of Appendix
// A). The paper details the calculation only for feedforward networks
// (Section 3.3); a recurrent one has no topological order, so it is evaluated
// by T synchronous sweeps: input nodes hold the observation, every other node
// starts at 0, and sweep t computes every non-input node with the Section 3.3
// node rule (response scaling the aggregate) from the values of sweep t - 1.
//
// One workgroup of four wavefronts per genome, in two forms. Both start with
//   1. checks: node keys and markings hashed in LDS (repeats), input / output
//      keys present, enabled connections' endpoints present and not ending at
//      an input, attribute codes in range; any failure: NaN outputs;
//   2. the enabled in-edges grouped by destination node row in ascending
//      connection row (counted, dropped into buckets, ranked in their bucket).
// recurrent_rf_kernel (genomes whose values fit a register file: n_in + 3 x
// computed nodes <= 200 rows) then gives each wavefront units of 1, 2 or 4 tiles
// of 64 observations with every value in registers, two rows per node (read
// one, write the other each sweep) and no barriers. Two things are not done
// again in every sweep: the terms of a node's leading in-edges from inputs
// (their partial sum is kept in a third row: the same additions in the same
// order), and nodes whose value has settled (all sources inputs, or settled a
// sweep earlier: copied once to the other row, then left alone).
// recurrent_kernel takes the others and short runs: two LDS value buffers of N_max rows x 64,
// the computed rows' records dealt round-robin to the wavefronts, one barrier
// per sweep.
// The sum aggregation accumulates with fused multiply-adds in ascending
// in-edge order and z = fma(response, aggregate, bias), as in the feedforward
// engines, so on an acyclic sum-aggregation genome T sweeps past its largest
// level reproduce the feedforward outputs bit for bit.
#include <algorithm>

#include "fwd_reg.hpp"
#include "tn_internal.hpp"

namespace tn {

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
constexpr int32_t kRowEmpty = 0x40000000;  // node function word of an empty row

int next_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

__device__ __forceinline__ uint32_t hash32(uint32_t k) {
  // lowbias32 (Chris Wellons' integer hash constants)
  k ^= k >> 16;
  k *= 0x7feb352du;
  k ^= k >> 15;
  k *= 0x846ca68bu;
  k ^= k >> 16;
  return k;
}

struct Layout {
  int HN, HM;             // key hash, marking hash (powers of two)
  size_t phase1, vals;    // bytes of the two aliased regions
  size_t persist;         // bytes of the kept tables
  size_t total;
};

size_t up16(size_t x) { return (x + 15) & ~size_t(15); }

Layout layout(int N, int C, int nio) {
  Layout l;
  l.HN = next_pow2(2 * N);
  l.HM = next_pow2(2 * C);
  l.phase1 = up16(8 * (size_t)l.HN + 8 * (size_t)l.HM + 8 * (size_t)(N + 1) + 10 * (size_t)C);
  l.vals = 2 * (size_t)N * kWave * sizeof(float);
  l.persist = up16(16 * (size_t)N + 8 * (size_t)C + 4 * (size_t)N + 4 * (size_t)nio);
  l.total = l.persist + std::max(l.phase1, l.vals);
  return l;
}

// Largest number of computed nodes of the register form, and of its file rows.
constexpr int kRfNodes = 61, kRfRows = 200;

__host__ __device__ constexpr bool rf_takes(int n_in, int computed) {
  return computed <= kRfNodes && n_in + 3 * computed <= kRfRows;
}

// LDS tables of the checks and of the in-edge lists.
struct Checked {
  int32_t* hk;    // [HN] node keys
  int32_t* hr;    // [HN] first row holding the key
  long long* mk;  // [HM] markings
  int32_t* ptr;   // [N + 1] first in-edge of each node row
  int32_t* fill;  // [N + 1]
  float* w;       // [C] weight of connection row r
  int16_t* src;   // [C] its source node row (-1: not an enabled connection)
  int16_t* dst;   // [C] its destination node row
  int16_t* slot;  // [C] connection rows by destination, in any order inside one
  int HN, HM;
  __device__ __forceinline__ int row_of(int32_t k) const {
    uint32_t h = hash32((uint32_t)k) & (uint32_t)(HN - 1);
    while (true) {
      const int32_t kk = hk[h];
      if (kk == k) return hr[h];
      if (kk == -1) return -1;
      h = (h + 1) & (uint32_t)(HN - 1);
    }
  }
};

__device__ __forceinline__ Checked carve_checked(unsigned char* region, int HN, int HM, int N,
                                                 int C) {
  Checked c;
  c.hk = (int32_t*)region;
  c.hr = c.hk + HN;
  c.mk = (long long*)(c.hr + HN);
  c.ptr = (int32_t*)(c.mk + HM);
  c.fill = c.ptr + N + 1;
  c.w = (float*)(c.fill + N + 1);
  c.src = (int16_t*)(c.w + C);
  c.dst = c.src + C;
  c.slot = c.dst + C;
  c.HN = HN;
  c.HM = HM;
  return c;
}

// Steps 1 and 2 of genome g by the whole workgroup: the in-edge lists (ptr, and
// edge(e, source row, weight) called once for each in-edge e of the lists) and
// iorow [n_in + n_out] (node row of key k). *status is in LDS and 0 on entry;
// returns the genome's status bits (a flagged genome has no lists). ptr and
// iorow are ready on return, what `edge` stores after the next barrier.
template <class Edge>
__device__ __forceinline__ int check_genome(const PopView& pop, int g, const Checked& c,
                                            int32_t* iorow, int* status, const Edge& edge) {
  const int tid = threadIdx.x;
  const int N = pop.N_max, C = pop.C_max, n_in = pop.n_in, nio = n_in + pop.n_out;
  const int64_t nb = pop.node_base(g), cb = pop.conn_base(g);
  const int64_t nrows = pop.node_rows(g), crows = pop.conn_rows(g);
  for (int h = tid; h < c.HN; h += kBlock) {
    c.hk[h] = -1;
    c.hr[h] = 0x7fffffff;
  }
  for (int h = tid; h < c.HM; h += kBlock) c.mk[h] = -1;
  for (int r = tid; r <= N; r += kBlock) c.ptr[r] = c.fill[r] = 0;
  __syncthreads();
  const bool oversize = nrows > N || crows > C || nrows < 0 || crows < 0;
  if (oversize) {
    if (tid == 0) *status = TN_OVERSIZE;
  } else {
    // node rows: key hash (first row of each key), repeats, attribute codes
    for (int r = tid; r < N; r += kBlock) {
      const int32_t k = r < nrows ? pop.node_key[nb + r] : -1;
      if (k < 0) continue;
      const int act = pop.node_act[nb + r], agg = pop.node_agg[nb + r];
      int bits = (act > TN_ACT_ABS || agg > TN_AGG_MAXABS) ? TN_BAD_ATTR : 0;
      uint32_t h = hash32((uint32_t)k) & (uint32_t)(c.HN - 1);
      while (true) {
        const int32_t prev = atomicCAS(&c.hk[h], -1, k);
        if (prev == -1) break;
        if (prev == k) {
          bits |= TN_DUP_NODE;
          break;
        }
        h = (h + 1) & (uint32_t)(c.HN - 1);
      }
      atomicMin(&c.hr[h], r);
      if (bits) atomicOr(status, bits);
    }
    // connection rows: repeated markings (enabled or not)
    for (int r = tid; r < (int)crows; r += kBlock) {
      const int32_t a = pop.conn_in[cb + r], b = pop.conn_out[cb + r];
      if (a < 0 || b < 0) continue;
      const long long m = ((long long)a << 32) | (long long)(uint32_t)b;
      uint32_t h = hash32((uint32_t)a ^ hash32((uint32_t)b)) & (uint32_t)(c.HM - 1);
      while (true) {
        const long long prev = (long long)atomicCAS((unsigned long long*)&c.mk[h], ~0ull,
                                                    (unsigned long long)m);
        if (prev == -1) break;
        if (prev == m) {
          atomicOr(status, TN_DUP_CONN);
          break;
        }
        h = (h + 1) & (uint32_t)(c.HM - 1);
      }
    }
  }
  __syncthreads();
  if (!oversize) {
    for (int k = tid; k < nio; k += kBlock) {
      const int r = c.row_of(k);
      iorow[k] = r;
      if (r < 0) atomicOr(status, TN_MISSING_IO);
    }
    // enabled connections: endpoints present, not ending at an input; in-degrees
    for (int r = tid; r < (int)crows; r += kBlock) {
      const int32_t a = pop.conn_in[cb + r], b = pop.conn_out[cb + r];
      const float w = pop.conn_w[cb + r];
      int src = -1, dst = 0;
      if (a >= 0 && b >= 0 && pop.conn_en[cb + r]) {
        const int ra = c.row_of(a), rb = c.row_of(b);
        int bits = 0;
        if (ra < 0 || rb < 0) bits |= TN_DANGLING;
        if (b < n_in) bits |= TN_INPUT_DST;
        if (bits) {
          atomicOr(status, bits);
        } else {
          src = ra;
          dst = rb;
          atomicAdd(&c.ptr[rb + 1], 1);
        }
      }
      c.src[r] = (int16_t)src;
      c.dst[r] = (int16_t)dst;
      c.w[r] = w;
    }
  }
  __syncthreads();
  const int st = *status;
  if (st != 0) return st;
  if (tid < kWave) {  // counts -> starts
    int carry = 0;
    for (int base = 0; base < N; base += kWave) {
      const int r = base + tid;
      const int x = wave_inclusive_scan(r < N ? c.ptr[r + 1] : 0);
      if (r < N) c.ptr[r + 1] = carry + x;
      carry += __shfl(x, kWave - 1, kWave);
    }
  }
  __syncthreads();
  for (int r = tid; r < (int)crows; r += kBlock)
    if (c.src[r] >= 0) {
      const int d = c.dst[r];
      c.slot[c.ptr[d] + atomicAdd(&c.fill[d], 1)] = (int16_t)r;
    }
  __syncthreads();
  const int n_edges = c.ptr[N];
  for (int i = tid; i < n_edges; i += kBlock) {
    const int r = c.slot[i], d = c.dst[r];
    const int lo = c.ptr[d], hi = c.ptr[d + 1];
    int rank = 0;
    for (int j = lo; j < hi; ++j) rank += c.slot[j] < r ? 1 : 0;
    edge(lo + rank, (int)c.src[r], c.w[r]);
  }
  return 0;
}

// NaN outputs and the status word of a flagged genome.
__device__ __forceinline__ void write_flagged(float* out, int64_t base, int64_t n,
                                              int32_t* status_out, int g, int st) {
  const float nan = __builtin_nanf("");
  for (int64_t i = threadIdx.x; i < n; i += kBlock) out[base + i] = nan;
  if (status_out && threadIdx.x == 0) status_out[g] = st;
}

// Computed (non-input) rows of genome g, on every thread; `sh`: an int of LDS
// that is 0 on entry. An oversize genome counts as none; more than N_max - n_in
// (an input is missing or a key repeats: a flagged genome) count as that many.
__device__ __forceinline__ int computed_rows(const PopView& pop, int g, int* sh) {
  const int64_t nrows = pop.node_rows(g), crows = pop.conn_rows(g), nb = pop.node_base(g);
  if (nrows >= 0 && nrows <= pop.N_max && crows >= 0 && crows <= pop.C_max) {
    int mine = 0;
    for (int r = threadIdx.x; r < (int)nrows; r += kBlock)
      mine += pop.node_key[nb + r] >= pop.n_in ? 1 : 0;
    mine = wave_sum_int(mine);
    if (lane_id() == 0 && mine) atomicAdd(sh, mine);
  }
  __syncthreads();
  return min(*sh, max(0, pop.N_max - pop.n_in));
}

// ------------------------------------------------ register form

// The program of one genome in LDS. Nodes are ordered by the sweep they settle
// in, latest first. File rows: inputs 0 .. n_in-1, node i at n_in + i (even
// buffer), n_in + na + i (odd), its partial sum over the leading input
// in-edges at n_in + 2 na + i.
struct RfProgram {
  const int4* hdr;       // [na] act | agg << 3 | leading in-edges << 6, bias, response,
                         //      byte offset of its in-edges | count << 16: the ones after
                         //      the leading ones first, then those
  const int32_t* settle; // [na] sweep its value settles in
  const int2* edge[2];   // [C + 64] source row in the even / odd buffer, weight
  const int16_t* out;    // [n_out] node of output j
  int na;
};

constexpr int kStageTiles = 2;  // tiles of observations staged at once, at most

// Requests the observations b0 .. b0 + n - 1 (contiguous) into this wavefront's
// LDS buffer with LDS-direct loads (16 bytes per lane where the source is
// aligned); the caller waits for vmcnt before it reads them.
__device__ __forceinline__ void stage_obs(const float* src, int total, float* stg, int lane) {
  int j = 0;
  if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {
    const int full = total & ~(4 * kWave - 1), voff = lane * 16;
    for (; j < full; j += 4 * kWave) {
      const uint32_t to =
          __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(stg + j));
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff),
                   "s"(src + j), "s"(to)
                   : "memory", "m0");
    }
  }
  for (; j < total; j += kWave)
    if (j + lane < total) __builtin_amdgcn_global_load_lds(src + j + lane, stg + j, 4, 0, 0);
}

// This wavefront's units of K = rf_tiles(R) tiles. A node's in-edges come
// across the lanes (one LDS read for the next node while this one runs), node
// words by v_readlane; the next unit's first observations are on their way to
// LDS while a unit runs (staged: the first unit's already are; the buffer is
// free once they are in registers). Bound by instruction issue and the
// latency of a node's chain at two wavefronts per SIMD (21k instructions per
// wavefront, about 85 per node and sweep): tiles share one index window per
// in-edge. 1000 genomes (17 -> 6, 40 nodes, 134 in-edges of which 104 lead),
// 1000 observations, 10 sweeps: 346 us; 602 us with the LDS form.
template <int R>
__device__ __forceinline__ void run_units(const RfProgram& pg, int n_in, int n_out, int B, int T,
                                          const float* x_g, float* out_g, float* stg, bool staged) {
  constexpr int K = rf_tiles(R), P = K < kStageTiles ? K : kStageTiles;
  const int lane = lane_id();
  const int na = pg.na;
  const int part = n_in + 2 * na;
  const int4 h = lane < na ? pg.hdr[lane] : make_int4(0, 0, 0, 0);
  const int l_settle = lane < na ? pg.settle[lane] : 0;
  const int l_out = lane < min(n_out, kWave) ? pg.out[lane] : 0;
  const int n_units = (B + K * kWave - 1) / (K * kWave);
  // in-edges of node i across the lanes (lanes past its last hold other words)
  auto edges_of = [&](const int2* base, int i) {
    const int at = __builtin_amdgcn_readlane(h.w, i) & 0xffff;
    return *reinterpret_cast<const int2*>(reinterpret_cast<const char*>(base + lane) + at);
  };
  for (int u = wave_id(); u < n_units; u += kWaves) {
    const int b0 = u * K * kWave;
    if (staged) {
      for (int f0 = 0; f0 < K; f0 += P) {
        if (f0 > 0)
          stage_obs(x_g + (int64_t)(b0 + f0 * kWave) * n_in,
                    max(0, min(P * kWave, B - b0 - f0 * kWave)) * n_in, stg, lane);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        for (int c = 0; c < n_in; ++c) {
          float x[K];
#pragma unroll
          for (int p = 0; p < K; ++p) x[p] = p < P ? stg[(p * kWave + lane) * n_in + c] : 0.0f;
          rf_set_part<R>(P, f0, c, x);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      const int bn = b0 + kWaves * K * kWave;
      if (bn < B)
        stage_obs(x_g + (int64_t)bn * n_in, min(P * kWave, B - bn) * n_in, stg, lane);
    } else {
      for (int c = 0; c < n_in; ++c) {
        float x[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const int b = b0 + k * kWave + lane;
          x[k] = b < B ? x_g[(int64_t)b * n_in + c] : 0.0f;
        }
        rfk_set<R>(c, x);
      }
    }
    float zero[K];
#pragma unroll
    for (int k = 0; k < K; ++k) zero[k] = 0.0f;
    int2 q = edges_of(pg.edge[0], 0);
    for (int i = 0; i < na; ++i) {
      rfk_set<R>(n_in + i, zero);
      const int2 qn = edges_of(pg.edge[0], min(i + 1, na - 1));
      const int np = __builtin_amdgcn_readlane(h.x, i) >> 6;
      if (np > 0) {
        const int er = __builtin_amdgcn_readlane(h.w, i);
        const int e0 = (er & 0xffff) >> 3, first = (er >> 16) - np;
        float s[K];
#pragma unroll
        for (int k = 0; k < K; ++k) s[k] = 0.0f;
        if (first + np > kWave) q = pg.edge[0][e0 + first + lane];
        int at = first + np > kWave ? 0 : first;
        for (int left = np; left > 0;) {
          const int end = min(at + left, kWave);
          left -= end - at;
          for (; at < end; ++at)
            rfk_fma<R>(s, __int_as_float(__builtin_amdgcn_readlane(q.y, at)),
                       __builtin_amdgcn_readlane(q.x, at));
          if (left > 0) {
            q = pg.edge[0][e0 + first + np - left + lane];
            at = 0;
          }
        }
        rfk_set<R>(part + i, s);
      }
      q = qn;
    }
    int active = na;
    for (int t = 1; t <= T; ++t) {
      const int odd = (t & 1) ^ 1;                   // the buffer that is read
      const int2* ed = odd ? pg.edge[1] : pg.edge[0];
      const int from = odd ? n_in + na : n_in, to = odd ? n_in : n_in + na;
      // nodes settled two sweeps ago are in both buffers, one sweep ago in one
      while (active > 0 && __builtin_amdgcn_readlane(l_settle, active - 1) + 1 < t) --active;
      if (active == 0) break;
      while (active > 0 && __builtin_amdgcn_readlane(l_settle, active - 1) < t) {
        --active;
        float v[K];
        rfk_get<R>(from + active, v);
        rfk_set<R>(to + active, v);
      }
      if (active == 0) break;  // every node settled: both buffers hold the values
      q = edges_of(ed, 0);
      for (int i = 0; i < active; ++i) {
        const int2 qn = edges_of(ed, min(i + 1, active - 1));
        const int d0 = __builtin_amdgcn_readlane(h.x, i);
        const int er = __builtin_amdgcn_readlane(h.w, i);
        const int agg = (d0 >> 3) & 7, np = d0 >> 6;
        const int ne = (er >> 16) - np;  // in-edges after the leading ones (np: sum only)
        auto row = [&](int e) { return __builtin_amdgcn_readlane(q.x, e); };
        auto weight = [&](int e) { return __int_as_float(__builtin_amdgcn_readlane(q.y, e)); };
        float s[K];
        if (np > 0)
          rfk_get<R>(part + i, s);
        else
#pragma unroll
          for (int k = 0; k < K; ++k) s[k] = 0.0f;
        if (ne <= 0) {
        } else if (agg == TN_AGG_SUM) {
          rfk_fma<R>(s, weight(0), row(0));
          if (ne > 1) {
            rfk_fma<R>(s, weight(1), row(1));
            if (ne > 2) {
              rfk_fma<R>(s, weight(2), row(2));
              int at = 3;
              for (int left = ne - 3; left > 0;) {
                const int end = min(at + left, kWave);
                left -= end - at;
                for (; at < end; ++at) rfk_fma<R>(s, weight(at), row(at));
                if (left > 0) {
                  q = ed[((er & 0xffff) >> 3) + ne - left + lane];
                  at = 0;
                }
              }
            }
          }
        } else {
          for (int base = 0; base < ne; base += kWave) {
            if (base > 0) q = ed[((er & 0xffff) >> 3) + base + lane];
            const int end = min(ne - base, kWave);
            for (int e = 0; e < end; ++e) {
              float v[K];
              rfk_get<R>(row(e), v);
              const float w = weight(e);
              const bool first = base + e == 0;
#pragma unroll
              for (int k = 0; k < K; ++k) {
                const float tm = w * v[k];
                if (first) {
                  s[k] = tm;
                } else {
                  switch (agg) {
                    case TN_AGG_PRODUCT: s[k] = s[k] * tm; break;
                    case TN_AGG_MAX: s[k] = fmaxf(s[k], tm); break;
                    case TN_AGG_MIN: s[k] = fminf(s[k], tm); break;
                    case TN_AGG_MEAN: s[k] = s[k] + tm; break;
                    default: s[k] = fabsf(tm) > fabsf(s[k]) ? tm : s[k]; break;  // maxabs
                  }
                }
              }
            }
          }
          if (agg == TN_AGG_MEAN)
#pragma unroll
            for (int k = 0; k < K; ++k) s[k] = s[k] / (float)ne;
        }
        const float bias = __int_as_float(__builtin_amdgcn_readlane(h.y, i));
        const float resp = __int_as_float(__builtin_amdgcn_readlane(h.z, i));
        float z[K], v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) z[k] = fmaf(resp, s[k], bias);
        activate_all<K>(d0 & 7, z, v);  // codes below 7: checked in step 1
        rfk_set<R>(to + i, v);
        q = qn;
      }
    }
    const int fin = (T & 1) ? n_in + na : n_in;
    for (int j = 0; j < n_out; ++j) {
      const int i = j < kWave ? __builtin_amdgcn_readlane(l_out, j)
                              : __builtin_amdgcn_readfirstlane(pg.out[j]);
      float y[K];
      rfk_get<R>(fin + i, y);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int b = b0 + k * kWave + lane;
        if (b < B) out_g[(int64_t)b * n_out + j] = y[k];
      }
    }
  }
}

// LDS bytes of the register form without the staging.
size_t rf_tables(const Layout& l, int N, int C, int nio, int n_out) {
  return up16(l.phase1 + 16 * (size_t)(C + kWave) + 4 * (size_t)nio + 2 * (size_t)(N + n_out));
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_num_vgpr(TN_RF_BASE))) void
recurrent_rf_kernel(PopView pop, const float* __restrict__ obs, int64_t obs_stride, int B, int T,
                    float* __restrict__ out, int32_t* __restrict__ status_out, int HN, int HM,
                    int phase1, int tables, int stage, int most_tiles) {
  rf_reserve<kRfRows>();
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int status, n_computed, n_act;
  __shared__ int4 hdr[kWave];
  __shared__ unsigned long long need[kWave];  // computed sources of node j
  __shared__ int32_t lead[kWave];             // first in-edge of node j with a computed source
  __shared__ int32_t node_row[kWave], place[kWave], settle[kWave];
  const int g = blockIdx.x;
  const int tid = threadIdx.x, lane = lane_id();
  const int N = pop.N_max, C = pop.C_max, n_in = pop.n_in, n_out = pop.n_out;
  const Checked ck = carve_checked(smem, HN, HM, N, C);
  int2* even = (int2*)(smem + phase1);               // [C + 64]
  int2* odd = even + C + kWave;                      // [C + 64]
  int32_t* iorow = (int32_t*)(odd + C + kWave);      // [n_in + n_out]
  int16_t* at = (int16_t*)(iorow + n_in + n_out);    // [N] node j of a row; -1 - k for input k
  int16_t* out_node = at + N;                        // [n_out]
  float* stg = (float*)(smem + tables) + wave_id() * stage;
  if (tid == 0) {
    status = 0;
    n_computed = 0;
    n_act = 0;
  }
  if (tid < kWave) {
    need[tid] = 0;
    lead[tid] = 0x7fffffff;
  }
  __syncthreads();
  const int computed = computed_rows(pop, g, &n_computed);
  if (!rf_takes(n_in, computed)) return;  // recurrent_kernel's
  // tiles per wavefront: as many as the launch wants and the file holds; the
  // first unit's observations are requested before the tables are built
  const int rows = n_in + 3 * computed;
  const int K = most_tiles >= 4 && rows <= 50 ? 4 : most_tiles >= 2 && rows <= 100 ? 2 : 1;
  const float* x_g = obs + (int64_t)g * obs_stride;
  const int P = min(K, kStageTiles);
  const bool staged = stage >= P * kWave * n_in;
  if (staged) {
    const int b0 = wave_id() * K * kWave;
    if (b0 < B) stage_obs(x_g + (int64_t)b0 * n_in, min(P * kWave, B - b0) * n_in, stg, lane);
  }
  const int64_t out_n = (int64_t)B * n_out;
  const int st = check_genome(pop, g, ck, iorow, &status, [&](int e, int src, float w) {
    even[e] = make_int2(src, __float_as_int(w));
  });
  if (st != 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load into LDS outlives the workgroup
    write_flagged(out, (int64_t)g * out_n, out_n, status_out, g, st);
    return;
  }
  const int64_t nb = pop.node_base(g);
  const int nrows = (int)pop.node_rows(g);
  // the computed rows (keys are distinct: at most kRfNodes), in any order
  for (int r = tid; r < nrows; r += kBlock) {
    const int32_t k = pop.node_key[nb + r];
    if (k < 0) continue;
    if (k < n_in) {
      at[r] = (int16_t)(-1 - k);
    } else {
      const int j = atomicAdd(&n_act, 1);
      at[r] = (int16_t)j;
      node_row[j] = r;
    }
  }
  __syncthreads();
  const int na = __builtin_amdgcn_readfirstlane(n_act);
  // sources that are computed, and the end of each node's leading input in-edges
  for (int j = wave_id(); j < na; j += kWaves) {
    const int r = node_row[j];
    const int e0 = ck.ptr[r], e1 = ck.ptr[r + 1];
    for (int e = e0 + lane; e < e1; e += kWave) {
      const int src = at[even[e].x];
      if (src >= 0) {
        atomicOr(&need[j], 1ull << src);
        atomicMin(&lead[j], e);
      }
    }
  }
  __syncthreads();
  // the sweep each node's value settles in (T: not before the last), and the
  // nodes' order, latest first
  if (tid < kWave) {
    const bool node = lane < na;
    const unsigned long long from = node ? need[lane] : 0;
    const int r = node ? node_row[lane] : 0;
    unsigned long long done = 0;
    int mine = T;
    bool open = node;
    for (int t = 1; t < T; ++t) {
      const bool ready = open && (from & ~done) == 0;
      const uint64_t m = __ballot(ready);
      if (m == 0) break;
      if (ready) {
        mine = t;
        open = false;
      }
      done |= m;
    }
    int before = 0;
    for (int o = 0; o < na; ++o) {
      const int so = __builtin_amdgcn_readlane(mine, o), ro = __builtin_amdgcn_readlane(r, o);
      before += so > mine || (so == mine && ro < r) ? 1 : 0;
    }
    if (node) {
      place[lane] = before;
      settle[before] = mine;
    }
  }
  __syncthreads();
  // each node's in-edges with file rows: after the leading ones, then those;
  // `even` holds the source rows until every list is in `odd`
  for (int j = wave_id(); j < na; j += kWaves) {
    const int r = node_row[j];
    const int e0 = ck.ptr[r], e1 = ck.ptr[r + 1];
    const int agg = pop.node_agg[nb + r];
    const int np = agg == TN_AGG_SUM ? min(lead[j], e1) - e0 : 0;
    for (int e = e0 + lane; e < e1; e += kWave) {
      const int src = at[even[e].x];
      odd[e - e0 < np ? e + (e1 - e0 - np) : e - np] =
          make_int2(src < 0 ? -1 - src : n_in + na + place[src], even[e].y);
    }
    if (lane == 0)
      hdr[place[j]] = make_int4(pop.node_act[nb + r] | (agg << 3) | (np << 6),
                                __float_as_int(pop.node_bias[nb + r]),
                                __float_as_int(pop.node_resp[nb + r]),
                                (e0 * (int)sizeof(int2)) | ((e1 - e0) << 16));
  }
  for (int j = tid; j < n_out; j += kBlock)
    out_node[j] = (int16_t)place[at[iorow[n_in + j]]];
  if (status_out && tid == 0) status_out[g] = 0;
  __syncthreads();
  for (int e = tid; e < ck.ptr[N]; e += kBlock) {
    const int2 q = odd[e];
    even[e] = make_int2(q.x >= n_in ? q.x - na : q.x, q.y);
  }
  __syncthreads();
  const RfProgram pg{hdr, settle, {even, odd}, out_node, na};
  float* out_g = out + (int64_t)g * out_n;
  if (K == 4)
    run_units<50>(pg, n_in, n_out, B, T, x_g, out_g, stg, staged);
  else if (K == 2)
    run_units<100>(pg, n_in, n_out, B, T, x_g, out_g, stg, staged);
  else
    run_units<200>(pg, n_in, n_out, B, T, x_g, out_g, stg, staged);
}

// ------------------------------------------------ LDS form

__global__ __launch_bounds__(kBlock) void recurrent_kernel(PopView pop, const float* obs,
                                                           int64_t obs_stride, int B, int T,
                                                           float* out, int32_t* status_out,
                                                           int HN, int HM, size_t persist, int rf) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int status;
  __shared__ int n_act;  // entries of crec
  __shared__ int n_computed;
  const int g = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = lane_id(), wv = wave_id();
  const int N = pop.N_max, C = pop.C_max, n_in = pop.n_in, n_out = pop.n_out;
  const int nio = n_in + n_out;
  // kept tables
  int4* crec = (int4*)smem;                     // [N] computed row: act | agg << 8 | row << 16,
                                                //     e0 | e1 << 16, bias bits, response bits
  int2* edge = (int2*)(crec + N);               // [C] in-edge: source row * 64, weight bits
  int32_t* nfn = (int32_t*)(edge + C);          // [N] act | agg << 8; input: bit 31 | index
  int32_t* iorow = nfn + N;                     // [n_in + n_out] node row of key k
  unsigned char* region = smem + persist;
  // phase 1 region
  const Checked ck = carve_checked(region, HN, HM, N, C);
  // phase 2 region
  float* vals = (float*)region;                 // [2][N][64]

  if (tid == 0) {
    status = 0;
    n_act = 0;
    n_computed = 0;
  }
  __syncthreads();
  // the genomes that the register form takes are left to it (rf: it is launched)
  if (rf && rf_takes(n_in, computed_rows(pop, g, &n_computed))) return;
  const int64_t nb = pop.node_base(g);
  const int64_t nrows = pop.node_rows(g);
  const int st = check_genome(pop, g, ck, iorow, &status, [&](int e, int src, float w) {
    edge[e] = make_int2(src * kWave, __float_as_int(w));
  });
  if (st != 0) {
    write_flagged(out, (int64_t)g * B * n_out, (int64_t)B * n_out, status_out, g, st);
    return;
  }
  for (int r = tid; r < N; r += kBlock) {
    const int32_t k = r < nrows ? pop.node_key[nb + r] : -1;
    int32_t f = kRowEmpty;
    if (k >= 0 && k < n_in) f = (int32_t)(kFnInput | (uint32_t)k);
    else if (k >= 0) f = pop.node_act[nb + r] | (pop.node_agg[nb + r] << 8);
    nfn[r] = f;
    // the computed rows' records, in any order (the rows of a sweep are
    // independent); in-edges e0 .. e1-1 of the lists
    if (f >= 0 && f != kRowEmpty) {
      const int e0 = ck.ptr[r], e1 = ck.ptr[r + 1];
      crec[atomicAdd(&n_act, 1)] =
          make_int4(f | (r << 16), e0 | (e1 << 16), __float_as_int(pop.node_bias[nb + r]),
                    __float_as_int(pop.node_resp[nb + r]));
    }
  }
  if (status_out && tid == 0) status_out[g] = 0;
  __syncthreads();  // phase 1 region is reused for the values from here on

  const int na = __builtin_amdgcn_readfirstlane(n_act);
  const float* x_g = obs + (int64_t)g * obs_stride;
  float* out_g = out + (int64_t)g * B * n_out;
  for (int b0 = 0; b0 < B; b0 += kWave) {
    const int b = b0 + lane;
    const bool active = b < B;
    for (int r = wv; r < N; r += kWaves) {
      const int32_t f = nfn[r];
      if (f == kRowEmpty) continue;
      float v = 0.0f;
      if (f < 0) v = active ? x_g[(int64_t)b * n_in + (f & 0xffff)] : 0.0f;
      vals[r * kWave + lane] = v;
      vals[(N + r) * kWave + lane] = v;
    }
    __syncthreads();
    for (int t = 0; t < T; ++t) {
      const float* cur = vals + (size_t)(t & 1) * N * kWave;
      float* nxt = vals + (size_t)((t + 1) & 1) * N * kWave;
      // the computed rows, dealt round-robin to the wavefronts; the row, its
      // function word and in-edge range as wavefront-uniform values (scalar
      // loop control and branches)
      for (int i = wv; i < na; i += kWaves) {
        const int4 q = crec[i];  // one 16-byte read
        const int fr = __builtin_amdgcn_readfirstlane(q.x);
        const int er = __builtin_amdgcn_readfirstlane(q.y);
        const int32_t f = fr & 0xffff;
        const int r = fr >> 16;
        const int e0 = er & 0xffff, e1 = er >> 16;
        const int agg = (f >> 8) & 0xff;
        float s;
        if (agg == TN_AGG_SUM) {
          s = 0.0f;
          int e = e0;
          for (; e + 2 <= e1; e += 2) {  // two in-edges' records, then both values
            const int2 q0 = edge[e], q1 = edge[e + 1];
            const float x0 = cur[q0.x + lane], x1 = cur[q1.x + lane];
            s = fmaf(__int_as_float(q0.y), x0, s);
            s = fmaf(__int_as_float(q1.y), x1, s);
          }
          if (e < e1) {
            const int2 q = edge[e];
            s = fmaf(__int_as_float(q.y), cur[q.x + lane], s);
          }
        } else if (e0 == e1) {
          s = 0.0f;
        } else {
          s = __int_as_float(edge[e0].y) * cur[edge[e0].x + lane];
          for (int e = e0 + 1; e < e1; ++e) {
            const float q = __int_as_float(edge[e].y) * cur[edge[e].x + lane];
            switch (agg) {
              case TN_AGG_PRODUCT: s = s * q; break;
              case TN_AGG_MAX: s = fmaxf(s, q); break;
              case TN_AGG_MIN: s = fminf(s, q); break;
              case TN_AGG_MEAN: s = s + q; break;
              default: s = fabsf(q) > fabsf(s) ? q : s; break;  // maxabs
            }
          }
          if (agg == TN_AGG_MEAN) s = s / (float)(e1 - e0);
        }
        float z[1] = {fmaf(__int_as_float(q.w), s, __int_as_float(q.z))}, v[1];
        activate_all<1>(f & 7, z, v);  // codes below 7: checked above
        nxt[r * kWave + lane] = v[0];
      }
      __syncthreads();
    }
    const float* fin = vals + (size_t)(T & 1) * N * kWave;
    if (active)
      for (int j = wv; j < n_out; j += kWaves)
        out_g[(int64_t)b * n_out + j] = fin[iorow[n_in + j] * kWave + lane];
    __syncthreads();
  }
}

}  // namespace

int recurrent_lds_check(const tn_population& p, size_t* bytes) {
  const Layout l = layout(p.N_max, p.C_max, p.n_in + p.n_out);
  *bytes = l.total;
  return l.total > max_dynamic_lds() ? TN_EUNSUPPORTED : TN_OK;
}

namespace {
// Whether the register form is the faster one. A genome's tables and partial
// sums cost it more, and its wavefronts do not share a tile's nodes: short runs
// stay on the LDS form. 200 genomes (17 -> 6): 10 sweeps of 64 / 128 observations
// 40 / 73 us on the LDS form, 61 / 62 us on registers (256: 137 and 63), one sweep
// 13 / 18 against 32 / 33; 1000 genomes (two rounds of register workgroups): 10
// sweeps of 64 / 128 / 256 45 / 81 / 155 against 90 / 123 / 125, four sweeps of 256
// / 500 72 / 137 against 88 / 124. The first lines lie where genomes of five inputs
// (fewer terms to keep) break even too.
// Genomes of many inputs mostly fill the file with a tile or two. Four wavefronts
// then take `units` tiles each, some of their places
// empty, and a batch of a tile too many is better off on the LDS form: 300 genomes
// (17 -> 6, 22 computed nodes), register / LDS form, 320 observations, two sweeps
// 64 / 53 us, four 72 / 86; 1000 genomes, 512 observations, three sweeps 146 / 116,
// six 156 / 202. The second lines are fitted to 720 calls (8 to 2500 such genomes, 1
// to 24 tiles, 1 to 10 sweeps). Row capacities say nothing of the genomes: in 256
// rows the same 300 take 81 us for 300 observations, 235 on the LDS form.
bool register_form_pays(const tn_population& p, int B, int T) {
  const int64_t tiles = ((int64_t)B + kWave - 1) / kWave;
  if (p.P <= 512 ? tiles * ((int64_t)T + 3) < 28 : tiles * ((int64_t)T - 1) < 32) return false;
  if (p.n_in <= 10) return true;
  const float units = (float)((tiles + kWaves - 1) / kWaves);
  const float places = units * kWaves / (float)tiles;
  const float least = p.P <= 512 ? 4.0f * places + 3.0f / units - 4.0f
                                 : 3.5f * places + 14.0f / (float)tiles - 0.5f;
  return (float)T >= least;
}
}  // namespace

int launch_forward_recurrent(const tn_population& p, const float* obs, int64_t obs_stride, int B,
                             int T, float* out, int32_t* status, hipStream_t stream) {
  const Layout l = layout(p.N_max, p.C_max, p.n_in + p.n_out);
  int rc = allow_lds((const void*)recurrent_kernel, l.total);
  if (rc != TN_OK || p.P == 0) return rc;
  // Tiles per wavefront share an index window per in-edge, but leave fewer
  // wavefronts: several only while the chip's 2048 register-form wavefronts
  // stay busy.
  const int64_t tiles = (int64_t)p.P * ((B + kWave - 1) / kWave);
  const int most = tiles >= 4 * 2048 ? 4 : tiles >= 2 * 2048 ? 2 : 1;
  // Observations are staged through LDS while two workgroups still fit a
  // compute unit (8.7 KB per wavefront at 17 inputs), else loaded directly.
  const size_t tables = rf_tables(l, p.N_max, p.C_max, p.n_in + p.n_out, p.n_out);
  int stage = std::min(most, kStageTiles) * kWave * p.n_in;  // floats per wavefront
  if (tables + kWaves * sizeof(float) * (size_t)stage > 72 * 1024) stage = 0;
  const size_t rf_lds = tables + kWaves * sizeof(float) * (size_t)stage;
  // The register form takes every genome it can hold (connection capacities
  // whose tables exceed the LDS leave it out); the LDS form is launched where
  // a genome of these capacities could be too large for it.
  const bool pays = register_form_pays(p, B, T);
  rc = pays ? allow_lds((const void*)recurrent_rf_kernel, rf_lds) : TN_EUNSUPPORTED;
  const bool rf = rc == TN_OK;
  if (rf) {
    hipLaunchKernelGGL(recurrent_rf_kernel, dim3(p.P), dim3(kBlock), rf_lds, stream, make_view(p),
                       obs, obs_stride, B, T, out, status, l.HN, l.HM, (int)l.phase1, (int)tables,
                       stage, most);
    rc = check_launch();
    if (rc == TN_OK && rf_takes(p.n_in, std::max(0, p.N_max - p.n_in))) return rc;
  } else if (rc == TN_EUNSUPPORTED) {
    rc = TN_OK;
  }
  if (rc != TN_OK) return rc;
  hipLaunchKernelGGL(recurrent_kernel, dim3(p.P), dim3(kBlock), l.total, stream, make_view(p), obs,
                     obs_stride, B, T, out, status, l.HN, l.HM, l.persist, rf ? 1 : 0);
  return check_launch();
}

}  // namespace tn
