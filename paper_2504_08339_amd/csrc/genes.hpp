// Per-genome sorted gene lists for the node-inclusive compatibility distance
// (node genes by key, connection genes by marking, with the attributes the
// distance compares), shared by the distance matrix and the speciation of
// one NEAT generation. Included by one translation unit each: everything here
// has internal linkage.
#pragma once

#include "tn_internal.hpp"

namespace tn {
namespace {

constexpr long long kGenePad = 0x7fffffffffffffffll;

__device__ __forceinline__ uint32_t gene_mix32(uint32_t k) {
  // lowbias32 (Chris Wellons' integer hash constants)
  k ^= k >> 16;
  k *= 0x7feb352du;
  k ^= k >> 15;
  k *= 0x846ca68bu;
  k ^= k >> 16;
  return k;
}

__device__ __forceinline__ uint32_t gene_hash(long long k) {
  return gene_mix32((uint32_t)k ^ gene_mix32((uint32_t)((unsigned long long)k >> 32)));
}

inline size_t gene_align(size_t x) { return (x + 255) & ~size_t(255); }

inline int gene_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

struct GeneList {
  long long* keyT;   // [cap][P], or [P][cap] (see prep_genes), as the others
  int32_t* hT;       // [cap][P] hash of the key (position-major lists only)
  float* a0T;        // [cap][P]
  float* a1T;        // [cap][P]
  uint32_t* codeT;   // [cap][P] c0 | c1 << 8
};

struct WsN {
  int32_t* cnt_n;    // [P] node genes, -1 for a genome without a gene set
  int32_t* cnt_c;    // [P] connection genes, -1 likewise
  GeneList nodes;    // cap N_max
  GeneList conns;    // cap C_max
};

inline size_t gene_list_bytes(int P, int cap) {
  const size_t n = (size_t)P * cap;
  return gene_align(sizeof(long long) * n) + 4 * gene_align(4 * n);
}

// p: the workspace's address (0 to find its size, so no pointer arithmetic).
inline GeneList carve_list(uintptr_t p, size_t& o, int P, int cap) {
  const size_t n = (size_t)P * cap;
  GeneList l;
  l.keyT = (long long*)(p + o);
  o += gene_align(sizeof(long long) * n);
  l.hT = (int32_t*)(p + o);
  o += gene_align(4 * n);
  l.a0T = (float*)(p + o);
  o += gene_align(4 * n);
  l.a1T = (float*)(p + o);
  o += gene_align(4 * n);
  l.codeT = (uint32_t*)(p + o);
  o += gene_align(4 * n);
  return l;
}

inline size_t ws_nodes_bytes(int P, int N, int C) {
  return 2 * gene_align(sizeof(int32_t) * P) + gene_list_bytes(P, N) + gene_list_bytes(P, C);
}

inline WsN carve_nodes(void* base, int P, int N, int C) {
  const uintptr_t p = (uintptr_t)base;
  size_t o = 0;
  WsN w;
  w.cnt_n = (int32_t*)(p + o);
  o += gene_align(sizeof(int32_t) * P);
  w.cnt_c = (int32_t*)(p + o);
  o += gene_align(sizeof(int32_t) * P);
  w.nodes = carve_list(p, o, P, N);
  w.conns = carve_list(p, o, P, C);
  return w;
}

// Bitonic sort of S (a power of two) (key, row) pairs in LDS by key; one
// wavefront.
__device__ void wave_bitonic(long long* key, int32_t* row, int S) {
  const int lane = lane_id();
  for (int k = 2; k <= S; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = lane; i < S; i += kWave) {
        const int ixj = i ^ j;
        if (ixj > i) {
          const long long ki = key[i], kj = key[ixj];
          if ((ki > kj) == ((i & k) == 0)) {
            key[i] = kj;
            key[ixj] = ki;
            const int32_t t = row[i];
            row[i] = row[ixj];
            row[ixj] = t;
          }
        }
      }
      wave_sync();
    }
  }
}

// Sort of n <= 64 NK pairs by counting, one wavefront: every lane ranks NK of
// the keys against all of them, read as broadcasts. Returns whether a key
// occurs twice (the order is then incomplete, the pairs at 0 .. n-1 still are
// some of the given ones).
template <int NK>
__device__ __forceinline__ bool wave_rank_sort(long long* key, int32_t* row, int n) {
  const int lane = lane_id();
  long long mine[NK];
  int32_t r[NK];
  int rank[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int i = min(k * kWave + lane, n - 1);
    mine[k] = key[i];
    r[k] = row[i];
    rank[k] = 0;
  }
#pragma unroll 8
  for (int j = 0; j < n; ++j) {
    const long long other = key[j];
#pragma unroll
    for (int k = 0; k < NK; ++k) rank[k] += other < mine[k] ? 1 : 0;
  }
  wave_sync();
  int total = 0;
#pragma unroll
  for (int k = 0; k < NK; ++k)
    if (k * kWave + lane < n) {
      key[rank[k]] = mine[k];
      row[rank[k]] = r[k];
      total += rank[k];
    }
  wave_sync();
  return wave_sum_int(total) != n * (n - 1) / 2;
}

// Sorts n pairs (room for S, a power of two) by key, one wavefront; returns
// whether a key occurs twice. Up to 256 by counting: no chain of LDS round
// trips (36 of them for 256 keys). 5000 genomes of 40 nodes and 164 connections
// 29 us, 60 us with the bitonic sort.
__device__ __forceinline__ bool wave_sort(long long* key, int32_t* row, int n, int S) {
  const int lane = lane_id();
  if (n <= 1) return false;
  if (n <= kWave) return wave_rank_sort<1>(key, row, n);
  if (n <= 2 * kWave) return wave_rank_sort<2>(key, row, n);
  if (n <= 4 * kWave) return wave_rank_sort<4>(key, row, n);
  for (int i = n + lane; i < S; i += kWave) {
    key[i] = kGenePad;
    row[i] = -1;
  }
  wave_sync();
  wave_bitonic(key, row, S);
  bool dup = false;
  for (int i = lane + 1; i < n; i += kWave) dup |= key[i] == key[i - 1];
  return __ballot(dup) != 0;
}

// Sorted gene lists of consecutive genomes from g0 on, one wavefront of the
// workgroup each (every thread calls it); SN / SC: powers of two holding the
// node / connection row capacities, smem: prep_nodes_lds bytes per genome.
// Position-major lists (entry k of genome g at k * P + g, with each key's
// hash) let 64 genomes' k-th genes be read as consecutive words; they are
// stored with consecutive threads on consecutive genomes. kByGenome stores
// genome-major lists (g * capacity + k, no hashes) for readers that take one
// genome's genes across their lanes.
template <bool kByGenome>
__device__ __forceinline__ void prep_genes(const PopView& pop, const WsN& ws, int g0, int SN, int SC,
                                           unsigned char* smem) {
  __shared__ int count[16];  // genes of each wavefront's genome
  const int S = SN > SC ? SN : SC;
  const int lane = lane_id(), wave = wave_id(), G = blockDim.x / kWave;
  const int P = pop.P, g = g0 + wave;
  long long* keys = (long long*)smem;              // [G][S]
  int32_t* rows = (int32_t*)(keys + (size_t)G * S);  // [G][S]
  long long* key = keys + (size_t)wave * S;
  int32_t* row = rows + (size_t)wave * S;
  const bool real = g < P;
  const int64_t nb = real ? pop.node_base(g) : 0, cb = real ? pop.conn_base(g) : 0;
  const int64_t nrows = real ? pop.node_rows(g) : 0, crows = real ? pop.conn_rows(g) : 0;
  const bool fits = nrows <= pop.N_max && nrows >= 0 && crows <= pop.C_max && crows >= 0;
  // node genes: every valid key is sorted (a repeated input key also leaves
  // the genome without a gene set); the inputs, keys 0 .. n_in-1, sort first
  // and are dropped
  int n = 0;
  for (int base = 0; fits && base < (int)nrows; base += kWave) {
    const int r = base + lane;
    const int32_t k = r < nrows ? pop.node_key[nb + r] : -1;
    const uint64_t m = __ballot(k >= 0);
    if (k >= 0) {
      key[n + mbcnt(m)] = (long long)k;
      row[n + mbcnt(m)] = r;
    }
    n += __popcll(m);
  }
  wave_sync();
  const bool dup_n = wave_sort(key, row, n, SN);
  int n_inputs = 0;
  for (int i = lane; i < n; i += kWave) n_inputs += key[i] < (long long)pop.n_in;
  n_inputs = wave_sum_int(n_inputs);
  const int nn = n - n_inputs;
  __shared__ int skipped[16];
  if (lane == 0) {
    count[wave] = nn;
    skipped[wave] = n_inputs;
  }
  __syncthreads();
  {
    const int gi = kByGenome ? wave : threadIdx.x % G;
    const int gg = g0 + gi;
    const int64_t base = gg < P ? pop.node_base(gg) : 0;
    for (int k = kByGenome ? lane : threadIdx.x / G; k < count[gi]; k += kWave) {
      const size_t at = (size_t)gi * S + skipped[gi] + k;
      const long long kk = keys[at];
      const int64_t r = base + rows[at];
      const int64_t o = kByGenome ? (int64_t)gg * pop.N_max + k : (int64_t)k * P + gg;
      ws.nodes.keyT[o] = kk;
      if (!kByGenome) ws.nodes.hT[o] = (int32_t)gene_hash(kk);
      ws.nodes.a0T[o] = pop.node_bias[r];
      ws.nodes.a1T[o] = pop.node_resp[r];
      ws.nodes.codeT[o] = (uint32_t)pop.node_act[r] | ((uint32_t)pop.node_agg[r] << 8);
    }
  }
  __syncthreads();
  // connection genes
  n = 0;
  for (int base = 0; fits && base < (int)crows; base += kWave) {
    const int r = base + lane;
    int32_t a = -1, b = -1;
    if (r < crows) {
      a = pop.conn_in[cb + r];
      b = pop.conn_out[cb + r];
    }
    const bool valid = a >= 0 && b >= 0;
    const uint64_t m = __ballot(valid);
    if (valid) {
      key[n + mbcnt(m)] = ((long long)a << 32) | (long long)(uint32_t)b;
      row[n + mbcnt(m)] = r;
    }
    n += __popcll(m);
  }
  wave_sync();
  const bool dup_c = wave_sort(key, row, n, SC);
  if (lane == 0) {
    count[wave] = n;
    if (real) {
      const bool bad = dup_n || dup_c || !fits;
      ws.cnt_n[g] = bad ? -1 : nn;
      ws.cnt_c[g] = bad ? -1 : n;
    }
  }
  __syncthreads();
  {
    const int gi = kByGenome ? wave : threadIdx.x % G;
    const int gg = g0 + gi;
    const int64_t base = gg < P ? pop.conn_base(gg) : 0;
    for (int k = kByGenome ? lane : threadIdx.x / G; k < count[gi]; k += kWave) {
      const size_t at = (size_t)gi * S + k;
      const long long kk = keys[at];
      const int64_t r = base + rows[at];
      const int64_t o = kByGenome ? (int64_t)gg * pop.C_max + k : (int64_t)k * P + gg;
      ws.conns.keyT[o] = kk;
      if (!kByGenome) ws.conns.hT[o] = (int32_t)gene_hash(kk);
      ws.conns.a0T[o] = pop.conn_w[r];
      ws.conns.a1T[o] = 0.0f;
      ws.conns.codeT[o] = (uint32_t)(pop.conn_en[r] != 0);
    }
  }
}

// LDS bytes of prep_genes per genome for capacities N, C.
inline size_t prep_nodes_lds(int N, int C) {
  return (sizeof(long long) + sizeof(int32_t)) * (size_t)gene_pow2(N > C ? N : C);
}

}  // namespace
}  // namespace tn
