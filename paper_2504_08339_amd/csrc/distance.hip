// Compatibility distance matrix (NEAT speciation; TensorNEAT Section 2.1,
// Algorithm 1, coefficients of Appendix A), over connection genes identified
// by their marking (in-key, out-key) in lexicographic order.
//
// Two launches:
//   prep  one wavefront per genome, up to eight of them a workgroup: gather the
//         valid connection rows into LDS, sort them by marking (up to 256 by
//         counting, more bitonically), flag repeated markings, and store the
//         sorted list position-major (keysT[k][g]) so that 64 genomes' k-th
//         genes are 64 consecutive words.
//   pairs C_max up to 512: pair_table_kernel, four row genomes (two above 256)
//         x 512 column genomes, the row genes in one LDS table, each column
//         gene read and looked up once for all rows. Above: pair_kernel, up to
//         kMaxRows x 256, a hash per row genome and a probe of each. Either way
//         only the pairs on or above the diagonal are evaluated, each written
//         to both halves.
#include <algorithm>
#include <mutex>

#include "genes.hpp"
#include "tn_internal.hpp"

namespace tn {

namespace {


__device__ __forceinline__ uint32_t mix32(uint32_t k) {
  // lowbias32 (Chris Wellons' integer hash constants)
  k ^= k >> 16;
  k *= 0x7feb352du;
  k ^= k >> 15;
  k *= 0x846ca68bu;
  k ^= k >> 16;
  return k;
}

__device__ __forceinline__ uint32_t hash_mark(long long k) {
  return mix32((uint32_t)k ^ mix32((uint32_t)((unsigned long long)k >> 32)));
}

// Genomes per workgroup of the prep kernels where their LDS allows it.
constexpr int kPrepGenomes = 8;

// That number for `bytes` of LDS per genome (a power of two).
int prep_genomes(size_t bytes) {
  int g = kPrepGenomes;
  while (g > 1 && g * bytes > 64 * 1024) g /= 2;
  return g;
}

struct Ws {
  int32_t* cnt;      // [P] gene count, -1 when a marking repeats
  long long* maxk;   // [P] largest marking, -1 when there are none
  long long* keysT;  // [C_max][P]
  float* wT;         // [C_max][P]
  int32_t* hT;       // [C_max][P] hash of each marking (hash_mark), computed once
};

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

Ws carve(void* base, int P, int C) {
  unsigned char* p = (unsigned char*)base;
  Ws w;
  size_t o = 0;
  w.cnt = (int32_t*)(p + o);
  o += align_up(sizeof(int32_t) * P);
  w.maxk = (long long*)(p + o);
  o += align_up(sizeof(long long) * P);
  w.keysT = (long long*)(p + o);
  o += align_up(sizeof(long long) * (size_t)P * C);
  w.wT = (float*)(p + o);
  o += align_up(sizeof(float) * (size_t)P * C);
  w.hT = (int32_t*)(p + o);
  return w;
}

size_t ws_bytes(int P, int C) {
  return align_up(sizeof(int32_t) * P) + align_up(sizeof(long long) * P) +
         align_up(sizeof(long long) * (size_t)P * C) + align_up(sizeof(float) * (size_t)P * C) +
         align_up(sizeof(int32_t) * (size_t)P * C);
}

int next_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

// One wavefront per genome, several genomes per workgroup (blockDim / 64,
// consecutive ones): the sorted lists meet in LDS and are stored with
// consecutive threads on consecutive genomes, whole memory segments instead of
// one word per cache line. Dynamic LDS: S keys and weights per genome.
__global__ __launch_bounds__(kPrepGenomes * kWave) void prep_kernel(PopView pop, Ws ws, int S) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int count[kPrepGenomes];
  const int wave = wave_id(), lane = lane_id(), G = blockDim.x / kWave;
  long long* keys = (long long*)smem;               // [G][S]
  float* weights = (float*)(keys + (size_t)G * S);  // [G][S]
  long long* key = keys + (size_t)wave * S;
  float* w = weights + (size_t)wave * S;
  const int g0 = blockIdx.x * G, g = g0 + wave;
  const int P = pop.P;
  int n = 0;
  if (g < P) {
    const int64_t cb = pop.conn_base(g);
    const int64_t crows = pop.conn_rows(g);
    const bool fits = crows <= pop.C_max && crows >= 0;
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
        const int at = n + mbcnt(m);
        key[at] = ((long long)a << 32) | (long long)(uint32_t)b;
        w[at] = pop.conn_w[cb + r];
      }
      n += __popcll(m);
    }
    wave_sync();
    const bool bad = wave_sort(key, reinterpret_cast<int32_t*>(w), n, S) || !fits;
    if (lane == 0) {
      ws.cnt[g] = bad ? -1 : n;
      ws.maxk[g] = n > 0 ? key[n - 1] : -1;
    }
  }
  if (lane == 0) count[wave] = n;
  __syncthreads();
  const int gi = threadIdx.x % G;
  for (int k = threadIdx.x / G; k < count[gi]; k += kWave) {
    const int64_t o = (int64_t)k * P + g0 + gi;
    const long long kk = keys[(size_t)gi * S + k];
    ws.keysT[o] = kk;
    ws.wT[o] = weights[(size_t)gi * S + k];
    ws.hT[o] = (int32_t)hash_mark(kk);
  }
}

constexpr int kPairBlock = 256;
constexpr int kMaxRows = 2;  // row genomes per block (measured best of 1, 2, 4, 8)

// Capacities whose shared table does not fit (table_rows below gives 0). Block = up to kMaxRows "row" genomes i0 .. i0+R-1 x 256 "column" genomes.
// Each row genome's genes go into an LDS hash (marking -> weight) plus its
// sorted list. Each lane walks its column genome's sorted list once
// (coalesced across the wavefront), hashes every marking once and probes all
// R tables: matches (|dw| summed in ascending marking order per row), column
// genes beyond each row's largest marking; then per row a binary search for
// the row's genes beyond the column's largest marking. The column genes are
// read from memory once per R rows.
__global__ __launch_bounds__(kPairBlock) void pair_kernel(Ws ws, int P, int HC, int C, int R,
                                                           float c1, float c2, float c3,
                                                           float* dist, int32_t* E_out,
                                                           int32_t* D_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  // per row r: hash keys [HC], hash weights [HC], sorted list [C]
  long long* hk_all = (long long*)smem;                                   // [R][HC]
  long long* si_all = hk_all + (size_t)R * HC;                             // [R][C]
  float* hw_all = (float*)(si_all + (size_t)R * C);                        // [R][HC]
  const int i0 = blockIdx.y * R;
  const int j = blockIdx.x * kPairBlock + threadIdx.x;
  const int nr = min(R, P - i0);
  // the distance is symmetric bit for bit (the matched markings are visited
  // in ascending order from either side): only pairs j >= i are evaluated,
  // each written to both halves of the matrix
  if ((int)(blockIdx.x * kPairBlock + kPairBlock - 1) < i0) return;  // all below the diagonal
  for (int h = threadIdx.x; h < nr * HC; h += kPairBlock) hk_all[h] = -1;
  __syncthreads();
  for (int r = 0; r < nr; ++r) {
    const int i = i0 + r;
    const int ni = ws.cnt[i];
    long long* hk = hk_all + (size_t)r * HC;
    float* hw = hw_all + (size_t)r * HC;
    long long* si = si_all + (size_t)r * C;
    for (int k = threadIdx.x; k < ni; k += kPairBlock) {
      const long long key = ws.keysT[(int64_t)k * P + i];
      si[k] = key;
      uint32_t h = (uint32_t)ws.hT[(int64_t)k * P + i] & (uint32_t)(HC - 1);
      while (atomicCAS((unsigned long long*)&hk[h], ~0ull, (unsigned long long)key) != ~0ull)
        h = (h + 1) & (uint32_t)(HC - 1);
      hw[h] = ws.wT[(int64_t)k * P + i];
    }
  }
  __syncthreads();
  if (j >= P) return;
  const int nj = ws.cnt[j];
  int ni[kMaxRows];
  long long maxi[kMaxRows];
  int M[kMaxRows], ex[kMaxRows];
  float S[kMaxRows];
#pragma unroll
  for (int r = 0; r < kMaxRows; ++r) {
    ni[r] = r < nr ? ws.cnt[i0 + r] : 0;
    maxi[r] = r < nr ? ws.maxk[i0 + r] : -1;
    M[r] = 0;
    ex[r] = 0;
    S[r] = 0.0f;
  }
  for (int k = 0; k < max(nj, 0); ++k) {
    const long long key = ws.keysT[(int64_t)k * P + j];
    const float w = ws.wT[(int64_t)k * P + j];
    const uint32_t h0 = (uint32_t)ws.hT[(int64_t)k * P + j] & (uint32_t)(HC - 1);
#pragma unroll
    for (int r = 0; r < kMaxRows; ++r) {
      if (r >= nr || ni[r] < 0 || j < i0 + r) continue;
      ex[r] += key > maxi[r];
      const long long* hk = hk_all + (size_t)r * HC;
      uint32_t h = h0;
      while (true) {
        const long long kk = hk[h];
        if (kk == key) {
          ++M[r];
          S[r] += fabsf(hw_all[(size_t)r * HC + h] - w);
          break;
        }
        if (kk == -1) break;
        h = (h + 1) & (uint32_t)(HC - 1);
      }
    }
  }
  const long long maxj = ws.maxk[j];
#pragma unroll
  for (int r = 0; r < kMaxRows; ++r) {
    if (r >= nr || j < i0 + r) continue;
    const int64_t o = (int64_t)(i0 + r) * P + j;
    const int64_t ot = (int64_t)j * P + (i0 + r);  // the mirrored entry (o itself on the diagonal)
    if (ni[r] < 0 || nj < 0) {
      dist[o] = __builtin_nanf("");
      dist[ot] = __builtin_nanf("");
      if (E_out) {
        E_out[o] = -1;
        D_out[o] = -1;
        E_out[ot] = -1;
        D_out[ot] = -1;
      }
      continue;
    }
    // row genes beyond the column's largest marking: ni - upper_bound(si, maxj)
    const long long* si = si_all + (size_t)r * C;
    int lo = 0, hi = ni[r];
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (si[mid] <= maxj) lo = mid + 1;
      else hi = mid;
    }
    const int E = ex[r] + (ni[r] - lo);
    const int D = ni[r] + nj - 2 * M[r] - E;
    const int N = max(ni[r], nj);
    float d = 0.0f;
    if (N > 0) {
      const float fN = (float)N;
      d = c1 * (float)E / fN + c2 * (float)D / fN + c3 * (M[r] > 0 ? S[r] / (float)M[r] : 0.0f);
    }
    dist[o] = d;
    dist[ot] = d;
    if (E_out) {
      E_out[o] = E;
      D_out[o] = D;
      E_out[ot] = E;
      D_out[ot] = D;
    }
  }
}


// ------------------------------------------------ node-inclusive distance
//
// delta = sum over the two gene kinds X (node genes, connection genes) of
//   (c_d * D_X + c_h * H_X) / max(|X1|, |X2|)          (0 when both are empty)
// node genes: valid non-input node rows by key; connection genes: valid
// connection rows (enabled or not) by marking. D_X counts the genes only one
// genome holds; H_X sums, over the shared ones in ascending identity order,
// |a0 - a0'| + |a1 - a1'| + [c0 != c0'] + [c1 != c1'] with (a0, a1, c0, c1) =
// (bias, response, act, agg) for a node and (weight, 0, enabled, 0) for a
// connection (the zero terms add exactly nothing).
//
// Same two-launch shape as the connection-gene distance: a prep wavefront per
// genome sorts both gene lists (keys + the row they came from) as above, checks
// repeated keys / markings, and stores them position-major with their
// attributes. The pairs take pair_nodes_table_kernel (node genes first, then
// connections, each kind's row genes in one table) where its LDS allows four
// rows (N_max up to 128, C_max up to 256) or two (512, 1024), else
// pair_nodes_kernel: R row genomes' genes in LDS hashes, each column genome's
// sorted lists walked once.

struct Gene {
  float a0, a1;
  uint32_t code;
};

__device__ __forceinline__ float attr_distance(Gene p, float a0, float a1, uint32_t code) {
  float t = fabsf(p.a0 - a0) + fabsf(p.a1 - a1);
  t += (p.code & 0xffu) != (code & 0xffu) ? 1.0f : 0.0f;
  t += (p.code >> 8) != (code >> 8) ? 1.0f : 0.0f;
  return t;
}

__global__ __launch_bounds__(kPrepGenomes * kWave) void prep_nodes_kernel(PopView pop, WsN ws,
                                                                         int SN, int SC) {
  extern __shared__ __align__(16) unsigned char smem[];
  prep_genes<false>(pop, ws, blockIdx.x * (blockDim.x / kWave), SN, SC, smem);
}

// Inserts row genome i's genes of one kind into an LDS hash of HC slots.
__device__ __forceinline__ void fill_hash(const GeneList& l, int P, int i, int n, int HC,
                                          long long* hk, Gene* hv) {
  for (int k = threadIdx.x; k < n; k += kPairBlock) {
    const int64_t o = (int64_t)k * P + i;
    const long long key = l.keyT[o];
    uint32_t h = (uint32_t)l.hT[o] & (uint32_t)(HC - 1);
    while (atomicCAS((unsigned long long*)&hk[h], ~0ull, (unsigned long long)key) != ~0ull)
      h = (h + 1) & (uint32_t)(HC - 1);
    hv[h] = Gene{l.a0T[o], l.a1T[o], l.codeT[o]};
  }
}

// Walks column genome j's sorted genes of one kind against the row hashes:
// homologous counts and attribute sums per row, in ascending key order.
__device__ __forceinline__ void walk_genes(const GeneList& l, int P, int j, int nj, int nr,
                                           int i0, const int* ni, int HC,
                                           const long long* hk_all, const Gene* hv_all,
                                           int* hom, float* H) {
  for (int k = 0; k < nj; ++k) {
    const int64_t o = (int64_t)k * P + j;
    const long long key = l.keyT[o];
    const float a0 = l.a0T[o], a1 = l.a1T[o];
    const uint32_t code = l.codeT[o];
    const uint32_t h0 = (uint32_t)l.hT[o] & (uint32_t)(HC - 1);
#pragma unroll
    for (int r = 0; r < kMaxRows; ++r) {
      if (r >= nr || ni[r] < 0 || j < i0 + r) continue;
      const long long* hk = hk_all + (size_t)r * HC;
      uint32_t h = h0;
      while (true) {
        const long long kk = hk[h];
        if (kk == key) {
          ++hom[r];
          H[r] += attr_distance(hv_all[(size_t)r * HC + h], a0, a1, code);
          break;
        }
        if (kk == -1) break;
        h = (h + 1) & (uint32_t)(HC - 1);
      }
    }
  }
}

__device__ __forceinline__ float kind_term(int n1, int n2, int hom, float H, float c_d,
                                           float c_h) {
  const int n = max(n1, n2);
  if (n == 0) return 0.0f;
  return (c_d * (float)(n1 + n2 - 2 * hom) + c_h * H) / (float)n;
}

// Block = up to kMaxRows row genomes x 256 column genomes; LDS per row: the
// node hash [HN] and the connection hash [HC] (keys, then attributes).
__global__ __launch_bounds__(kPairBlock) void pair_nodes_kernel(WsN ws, int P, int HN, int HC,
                                                                 int R, float c_d, float c_h,
                                                                 float* dist, int32_t* DN_out,
                                                                 int32_t* DC_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  long long* nk_all = (long long*)smem;                         // [R][HN]
  long long* ck_all = nk_all + (size_t)R * HN;                  // [R][HC]
  Gene* nv_all = (Gene*)(ck_all + (size_t)R * HC);              // [R][HN]
  Gene* cv_all = nv_all + (size_t)R * HN;                       // [R][HC]
  const int i0 = blockIdx.y * R;
  const int j = blockIdx.x * kPairBlock + threadIdx.x;
  const int nr = min(R, P - i0);
  if ((int)(blockIdx.x * kPairBlock + kPairBlock - 1) < i0) return;  // all below the diagonal
  for (int h = threadIdx.x; h < nr * HN; h += kPairBlock) nk_all[h] = -1;
  for (int h = threadIdx.x; h < nr * HC; h += kPairBlock) ck_all[h] = -1;
  __syncthreads();
  for (int r = 0; r < nr; ++r) {
    const int i = i0 + r;
    const int nn = ws.cnt_n[i], nc = ws.cnt_c[i];
    fill_hash(ws.nodes, P, i, nn, HN, nk_all + (size_t)r * HN, nv_all + (size_t)r * HN);
    fill_hash(ws.conns, P, i, nc, HC, ck_all + (size_t)r * HC, cv_all + (size_t)r * HC);
  }
  __syncthreads();
  if (j >= P) return;
  const int nj_n = ws.cnt_n[j], nj_c = ws.cnt_c[j];
  int ni_n[kMaxRows], ni_c[kMaxRows], hom_n[kMaxRows], hom_c[kMaxRows];
  float H_n[kMaxRows], H_c[kMaxRows];
#pragma unroll
  for (int r = 0; r < kMaxRows; ++r) {
    ni_n[r] = r < nr ? ws.cnt_n[i0 + r] : 0;
    ni_c[r] = r < nr ? ws.cnt_c[i0 + r] : 0;
    hom_n[r] = hom_c[r] = 0;
    H_n[r] = H_c[r] = 0.0f;
  }
  walk_genes(ws.nodes, P, j, max(nj_n, 0), nr, i0, ni_n, HN, nk_all, nv_all, hom_n, H_n);
  walk_genes(ws.conns, P, j, max(nj_c, 0), nr, i0, ni_c, HC, ck_all, cv_all, hom_c, H_c);
#pragma unroll
  for (int r = 0; r < kMaxRows; ++r) {
    if (r >= nr || j < i0 + r) continue;
    const int64_t o = (int64_t)(i0 + r) * P + j;
    const int64_t ot = (int64_t)j * P + (i0 + r);
    float d;
    int dn, dc;
    if (ni_n[r] < 0 || nj_n < 0) {
      d = __builtin_nanf("");
      dn = dc = -1;
    } else {
      d = kind_term(ni_n[r], nj_n, hom_n[r], H_n[r], c_d, c_h) +
          kind_term(ni_c[r], nj_c, hom_c[r], H_c[r], c_d, c_h);
      dn = ni_n[r] + nj_n - 2 * hom_n[r];
      dc = ni_c[r] + nj_c - 2 * hom_c[r];
    }
    dist[o] = d;
    dist[ot] = d;
    if (DN_out) {
      DN_out[o] = dn;
      DC_out[o] = dc;
      DN_out[ot] = dn;
      DC_out[ot] = dc;
    }
  }
}

// ------------------------------------------------ shared row tables
//
// The pair kernels of populations whose row genes fit: a block takes R row
// genomes x 512 column genomes. All R genomes' genes go into one LDS table
// (marking -> the attributes of each of the R genomes that hold it, and a
// presence mask), so a column gene is read and looked up once for R rows;
// most genes of a NEAT population are shared by its genomes, so the table is
// little larger than one genome's. A lane walks its column genome's sorted
// list kStep genes at a time: the next kStep genes' loads and this group's first
// probes are in flight together. Each pair's sum runs in ascending gene order,
// one term (0 for an absent gene: a sum of non-negative terms keeps its bits)
// after the other. Bound by instruction issue (about 120 vector instructions
// per gene and four rows) and LDS latency. 1000 genomes of 40 / 164 genes: 167
// us with node genes, 110 us without; 465 and 310 us with one table per row
// genome, two rows a block, and a probe at a time. (Two-slot probes in a loop
// 245 us, loads that were masked as they arrived, so that nothing stayed in
// flight, 317 us.)
constexpr int kStep = 4;
constexpr int kTableBlock = 512;
constexpr int kBucket = 4;  // slots read at once

template <int R>
struct alignas(4 * R) Attr {
  float v[R];
};

template <int R>
struct alignas(4 * R) Codes {
  uint32_t v[R];
};

template <int R>
struct Table {
  long long* key;   // [H], -1: empty
  Attr<R>* a0;      // [H]
  Attr<R>* a1;      // [H] node genes only
  Codes<R>* code;   // [H] node genes only
  uint32_t* meta;   // [H] bit r: row genome r holds the gene; bit 8 + r: its enabled flag
  int H;
  // first slot of a hash's bucket of kBucket; a key sits in its bucket or, where
  // that is full, in the slots after it
  __device__ __forceinline__ uint32_t bucket(int32_t h) const {
    return ((uint32_t)h & (uint32_t)(H / kBucket - 1)) * kBucket;
  }
};

// LDS of one table per slot: markings and weights, or node genes.
constexpr size_t conn_slot(int R) { return 8 + 4 * (size_t)R + 4; }
constexpr size_t node_slot(int R) { return 8 + 12 * (size_t)R + 4; }

template <int R>
__device__ __forceinline__ Table<R> carve_table(unsigned char* p, int H, bool nodes) {
  Table<R> t;
  t.H = H;
  t.key = (long long*)p;
  t.a0 = (Attr<R>*)(t.key + H);
  t.a1 = t.a0 + H;
  t.code = (Codes<R>*)(nodes ? t.a1 + H : t.a1);
  t.meta = (uint32_t*)(nodes ? t.code + H : t.code);
  return t;
}

// Fills the table with rows i0 .. i0 + R - 1 (n[r] genes, <= 0: none). Every
// thread of the workgroup calls it; ends at a barrier. kNodes: node genes
// (a1 and codes); else code (where given) is the enabled flag.
template <int R, bool kNodes>
__device__ __forceinline__ void fill_table(const Table<R>& t, const long long* keyT,
                                           const int32_t* hT, const float* a0T, const float* a1T,
                                           const uint32_t* codeT, int P, int i0,
                                           const int (&n)[R]) {
  for (int h = threadIdx.x; h < t.H; h += kTableBlock) {
    t.key[h] = -1;
    t.meta[h] = 0;
  }
  __syncthreads();
  const int r = threadIdx.x % R;
  int count = 0;
#pragma unroll
  for (int i = 0; i < R; ++i) count = r == i ? n[i] : count;
  for (int k = threadIdx.x / R; k < count; k += kTableBlock / R) {
    const int64_t o = (int64_t)k * P + i0 + r;
    const long long key = keyT[o];
    uint32_t h = t.bucket(hT[o]);
    while (true) {
      const long long old = (long long)atomicCAS((unsigned long long*)&t.key[h], ~0ull,
                                                 (unsigned long long)key);
      if (old == -1 || old == key) break;
      h = (h + 1) & (uint32_t)(t.H - 1);
    }
    t.a0[h].v[r] = a0T[o];
    uint32_t bits = 1u << r;
    if (kNodes) {
      t.a1[h].v[r] = a1T[o];
      t.code[h].v[r] = codeT[o];
    } else if (codeT) {
      bits |= codeT[o] << (8 + r);
    }
    atomicOr(&t.meta[h], bits);
  }
  __syncthreads();
}

// Walks column genome j's nj sorted genes against the table: per row, shared
// genes (hom) and the sum of their terms. kNodes: |da0| + |da1| + [act differs]
// + [agg differs]; else |dw| + [enabled differs] (where codeT is given).
template <int R, bool kNodes>
__device__ __forceinline__ void walk_table(const Table<R>& t, const long long* keyT,
                                           const int32_t* hT, const float* a0T, const float* a1T,
                                           const uint32_t* codeT, int P, int j, int nj,
                                           int (&hom)[R], float (&sum)[R]) {
  // as many steps as the wavefront's longest list takes, so that every load has
  // a wavefront-uniform base (entries past a lane's own last are not used)
  int most = nj;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, kWave));
  most = __builtin_amdgcn_readfirstlane(most);
  struct Group {
    int k;
    long long key[kStep];
    int32_t h[kStep];
    uint32_t code[kStep];
    float a0[kStep], a1[kStep];
  };
  auto load = [&](int k, Group& q) {
    q.k = k;
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      const int64_t row = (int64_t)min(k + u, most - 1) * P;
      q.key[u] = (keyT + row)[j];
      q.h[u] = (hT + row)[j];
      q.a0[u] = (a0T + row)[j];
      if (kNodes) q.a1[u] = (a1T + row)[j];
      if (codeT) q.code[u] = (codeT + row)[j];
    }
  };
  // one group: its probes side by side until the slowest has its answer, then
  // the slots' attributes
  auto work = [&](Group& q) {
    bool mine[kStep], open[kStep], more = false;
    uint32_t h[kStep];
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      // the whole bucket at once: nearly every gene is answered by it
      h[u] = t.bucket(q.h[u]);
      mine[u] = q.k + u < nj;
    }
    typedef long long Keys __attribute__((ext_vector_type(2)));
    Keys lo[kStep], hi[kStep];
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      lo[u] = *reinterpret_cast<const Keys*>(t.key + h[u]);
      hi[u] = *reinterpret_cast<const Keys*>(t.key + h[u] + 2);
    }
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      const long long key = q.key[u];
      int at = 4;
      at = hi[u].y == key ? 3 : at;
      at = hi[u].x == key ? 2 : at;
      at = lo[u].y == key ? 1 : at;
      at = lo[u].x == key ? 0 : at;
      open[u] = mine[u] && at == 4 && hi[u].y != -1;  // full, and not there
      mine[u] = mine[u] && (at < 4 || open[u]);
      h[u] = (h[u] + at) & (uint32_t)(t.H - 1);
      more |= open[u];
    }
    while (__ballot(more)) {
      more = false;
#pragma unroll
      for (int u = 0; u < kStep; ++u) {
        const long long kk = t.key[h[u]];
        // it ends at the key, or at an empty slot, whose presence mask is 0
        open[u] = open[u] && kk != q.key[u] && kk != -1;
        h[u] = open[u] ? (h[u] + 1) & (uint32_t)(t.H - 1) : h[u];
        more |= open[u];
      }
    }
    uint32_t meta[kStep];
    Attr<R> a0[kStep], a1[kStep];
    Codes<R> code[kStep];
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      meta[u] = mine[u] ? t.meta[h[u]] : 0;
      a0[u] = t.a0[h[u]];
      if (kNodes) {
        a1[u] = t.a1[h[u]];
        code[u] = t.code[h[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool has = (meta[u] >> r) & 1;
        float term = fabsf(a0[u].v[r] - q.a0[u]);
        if (kNodes) {
          term += fabsf(a1[u].v[r] - q.a1[u]);
          const uint32_t own = code[u].v[r];
          term += (own & 0xffu) != (q.code[u] & 0xffu) ? 1.0f : 0.0f;
          term += (own >> 8) != (q.code[u] >> 8) ? 1.0f : 0.0f;
        } else if (codeT) {
          term += ((meta[u] >> (8 + r)) & 1) != q.code[u] ? 1.0f : 0.0f;
        }
        hom[r] += has ? 1 : 0;
        sum[r] += has ? term : 0.0f;
      }
    }
  };
  if (most <= 0) return;  // uniform
  // groups in flight: the roles turn, so no load is waited for in a copy
  Group x, y, z;
  load(0, x);
  load(kStep, y);
  for (int k = 0; k < most; k += 3 * kStep) {
    load(k + 2 * kStep, z);
    work(x);
    load(k + 3 * kStep, x);
    work(y);
    load(k + 4 * kStep, y);
    work(z);
  }
}

// pair_kernel on a shared table.
template <int R>
__global__ __launch_bounds__(kTableBlock) void pair_table_kernel(Ws ws, int P, int H, int C,
                                                                float c1, float c2, float c3,
                                                                float* dist, int32_t* E_out,
                                                                int32_t* D_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)(blockIdx.x * kTableBlock + kTableBlock - 1) < (int)blockIdx.y * R) return;  // below the diagonal
  const Table<R> t = carve_table<R>(smem, H, false);
  long long* lists = (long long*)(smem + (size_t)H * conn_slot(R));  // [R][C] sorted markings
  const int i0 = blockIdx.y * R, j = blockIdx.x * kTableBlock + threadIdx.x;
  int ni[R], M[R];
  float S[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ni[r] = i0 + r < P ? ws.cnt[i0 + r] : 0;
    M[r] = 0;
    S[r] = 0.0f;
  }
  for (int k = threadIdx.x / R, r = threadIdx.x % R; k < C; k += kTableBlock / R) {
    int count = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) count = r == i ? ni[i] : count;
    if (k < count) lists[(size_t)r * C + k] = ws.keysT[(int64_t)k * P + i0 + r];
  }
  fill_table<R, false>(t, ws.keysT, ws.hT, ws.wT, nullptr, nullptr, P, i0, ni);
  const int nj = j >= i0 && j < P ? ws.cnt[j] : 0;  // no walk below the diagonal
  walk_table<R, false>(t, ws.keysT, ws.hT, ws.wT, nullptr, nullptr, P, min(j, P - 1), nj, M, S);
  if (j >= P) return;
  const long long maxj = ws.maxk[j];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (i0 + r >= P || j < i0 + r) continue;
    const int64_t o = (int64_t)(i0 + r) * P + j, ot = (int64_t)j * P + (i0 + r);
    float d = __builtin_nanf("");
    int E = -1, D = -1;
    if (ni[r] >= 0 && nj >= 0) {
      // row genes beyond the column's largest marking, column genes beyond
      // the row's
      int lo = 0, hi = ni[r];
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (lists[(size_t)r * C + mid] <= maxj) lo = mid + 1;
        else hi = mid;
      }
      E = ni[r] - lo;
      const long long maxi = ni[r] > 0 ? lists[(size_t)r * C + ni[r] - 1] : -1;
      if (maxj > maxi) {
        lo = 0;
        hi = nj;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (ws.keysT[(int64_t)mid * P + j] <= maxi) lo = mid + 1;
          else hi = mid;
        }
        E += nj - lo;
      }
      D = ni[r] + nj - 2 * M[r] - E;
      const int N = max(ni[r], nj);
      d = 0.0f;
      if (N > 0) {
        const float fN = (float)N;
        d = c1 * (float)E / fN + c2 * (float)D / fN + c3 * (M[r] > 0 ? S[r] / (float)M[r] : 0.0f);
      }
    }
    dist[o] = d;
    dist[ot] = d;
    if (E_out) {
      E_out[o] = E;
      D_out[o] = D;
      E_out[ot] = E;
      D_out[ot] = D;
    }
  }
}

// pair_nodes_kernel on shared tables: node genes first, then connections, in
// the same LDS.
template <int R>
__global__ __launch_bounds__(kTableBlock) void pair_nodes_table_kernel(WsN ws, int P, int HN, int HC,
                                                                      float c_d, float c_h,
                                                                      float* dist, int32_t* DN_out,
                                                                      int32_t* DC_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)(blockIdx.x * kTableBlock + kTableBlock - 1) < (int)blockIdx.y * R) return;  // below the diagonal
  const int i0 = blockIdx.y * R, j = blockIdx.x * kTableBlock + threadIdx.x;
  int ni_n[R], ni_c[R], hom_n[R], hom_c[R];
  float H_n[R], H_c[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ni_n[r] = i0 + r < P ? ws.cnt_n[i0 + r] : 0;
    ni_c[r] = i0 + r < P ? ws.cnt_c[i0 + r] : 0;
    hom_n[r] = hom_c[r] = 0;
    H_n[r] = H_c[r] = 0.0f;
  }
  const bool col = j >= i0 && j < P;  // no walk below the diagonal
  const int nj_n = col ? ws.cnt_n[j] : 0, nj_c = col ? ws.cnt_c[j] : 0;
  {
    const Table<R> t = carve_table<R>(smem, HN, true);
    fill_table<R, true>(t, ws.nodes.keyT, ws.nodes.hT, ws.nodes.a0T, ws.nodes.a1T, ws.nodes.codeT, P,
                        i0, ni_n);
    walk_table<R, true>(t, ws.nodes.keyT, ws.nodes.hT, ws.nodes.a0T, ws.nodes.a1T,
                               ws.nodes.codeT, P, min(j, P - 1), nj_n, hom_n, H_n);
    __syncthreads();
  }
  {
    const Table<R> t = carve_table<R>(smem, HC, false);
    fill_table<R, false>(t, ws.conns.keyT, ws.conns.hT, ws.conns.a0T, nullptr, ws.conns.codeT, P,
                         i0, ni_c);
    walk_table<R, false>(t, ws.conns.keyT, ws.conns.hT, ws.conns.a0T, nullptr,
                                ws.conns.codeT, P, min(j, P - 1), nj_c, hom_c, H_c);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!col || i0 + r >= P || j < i0 + r) continue;
    const int64_t o = (int64_t)(i0 + r) * P + j, ot = (int64_t)j * P + (i0 + r);
    float d = __builtin_nanf("");
    int dn = -1, dc = -1;
    if (ni_n[r] >= 0 && nj_n >= 0) {
      d = kind_term(ni_n[r], nj_n, hom_n[r], H_n[r], c_d, c_h) +
          kind_term(ni_c[r], nj_c, hom_c[r], H_c[r], c_d, c_h);
      dn = ni_n[r] + nj_n - 2 * hom_n[r];
      dc = ni_c[r] + nj_c - 2 * hom_c[r];
    }
    dist[o] = d;
    dist[ot] = d;
    if (DN_out) {
      DN_out[o] = dn;
      DC_out[o] = dc;
      DN_out[ot] = dn;
      DC_out[ot] = dc;
    }
  }
}

// LDS of the table kernels with R rows (tables at most half full).
int table_slots(int R, int rows) { return std::max(2 * kBucket, next_pow2(2 * R * rows)); }
size_t pair_table_lds(int R, int C) {
  return (size_t)table_slots(R, C) * conn_slot(R) + sizeof(long long) * (size_t)R * C;
}
size_t pair_nodes_table_lds(int R, int N, int C) {
  return std::max((size_t)table_slots(R, N) * node_slot(R), (size_t)table_slots(R, C) * conn_slot(R));
}

// Rows per block of the table kernels: four, else two, where two blocks share
// a compute unit's LDS; 0: a table per row genome (the kernels above).
constexpr size_t kTableLds = 80 * 1024;
template <class Lds>
int table_rows(const Lds& lds) {
  for (int R : {4, 2})
    if (lds(R) <= kTableLds) return R;
  return 0;
}

}  // namespace

size_t distance_workspace_bytes(int P, int C_max) { return ws_bytes(P, C_max); }

// ------------------------------------------------ allocation-free variant

// Workspace of tn_distance_noalloc: a fixed device array instead of a caller
// buffer. Each device holds its own copy for the life of the process; every
// call on a device reuses it (the prep kernel rewrites every entry the pair
// kernel reads, so nothing needs clearing between calls).
static __device__ __align__(256) unsigned char scratch[TN_DISTANCE_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device, looked up once per
// device (host code must never use the array's name as an address).
int noalloc_scratch(void** out) {
  int dev = 0;
  int rc = record_hip(hipGetDevice(&dev));
  if (rc != TN_OK) return rc;
  if (dev < 0 || dev >= kMaxDevices) return TN_EUNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    rc = record_hip(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (rc != TN_OK) return rc;
    if (!ptr) return record_hip(hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return TN_OK;
}

int launch_distance(const tn_population& p, float c1, float c2, float c3, void* workspace,
                    float* dist, int32_t* E, int32_t* D, hipStream_t stream) {
  const int S = next_pow2(p.C_max);
  const int G = prep_genomes((sizeof(long long) + sizeof(float)) * (size_t)S);
  const size_t prep_lds = G * (sizeof(long long) + sizeof(float)) * (size_t)S;
  const int HC = next_pow2(2 * p.C_max);
  const size_t per_row = (sizeof(long long) + sizeof(float)) * (size_t)HC +
                         sizeof(long long) * (size_t)p.C_max;
  // row genomes per block: as many as fit 64 KB of LDS (two blocks per CU), >= 1
  const int R = (int)std::max<size_t>(1, std::min<size_t>(kMaxRows, (64 * 1024) / per_row));
  const size_t pair_lds = per_row * R;
  int rc = allow_lds((const void*)prep_kernel, prep_lds);
  if (rc == TN_OK) rc = allow_lds((const void*)pair_kernel, pair_lds);
  if (rc != TN_OK || p.P == 0) return rc;
  Ws ws = carve(workspace, p.P, p.C_max);
  hipLaunchKernelGGL(prep_kernel, dim3((p.P + G - 1) / G), dim3(G * kWave), prep_lds, stream,
                     make_view(p), ws, S);
  rc = check_launch();
  if (rc != TN_OK) return rc;
  const int rows = table_rows([&](int r) { return pair_table_lds(r, p.C_max); });
  if (rows) {
    const size_t lds = pair_table_lds(rows, p.C_max);
    const auto kern = rows == 4 ? pair_table_kernel<4> : pair_table_kernel<2>;
    rc = allow_lds((const void*)kern, lds);
    if (rc != TN_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((p.P + kTableBlock - 1) / kTableBlock, (p.P + rows - 1) / rows),
                       dim3(kTableBlock), lds, stream, ws, p.P, table_slots(rows, p.C_max),
                       p.C_max, c1, c2, c3, dist, E, D);
    return check_launch();
  }
  dim3 grid((p.P + kPairBlock - 1) / kPairBlock, (p.P + R - 1) / R);
  hipLaunchKernelGGL(pair_kernel, grid, dim3(kPairBlock), pair_lds, stream, ws, p.P, HC,
                     p.C_max, R, c1, c2, c3, dist, E, D);
  return check_launch();
}

size_t distance_nodes_workspace_bytes(int P, int N_max, int C_max) {
  return ws_nodes_bytes(P, N_max, C_max);
}

int launch_distance_nodes(const tn_population& p, float c_d, float c_h, void* workspace,
                          float* dist, int32_t* DN, int32_t* DC, hipStream_t stream) {
  const int G = prep_genomes(prep_nodes_lds(p.N_max, p.C_max));
  const size_t prep_lds = G * prep_nodes_lds(p.N_max, p.C_max);
  const int HN = next_pow2(2 * p.N_max), HC = next_pow2(2 * p.C_max);
  const size_t per_row = (sizeof(long long) + sizeof(Gene)) * (size_t)(HN + HC);
  const int R = (int)std::max<size_t>(1, std::min<size_t>(kMaxRows, (64 * 1024) / per_row));
  const size_t pair_lds = per_row * R;
  int rc = allow_lds((const void*)prep_nodes_kernel, prep_lds);
  if (rc == TN_OK) rc = allow_lds((const void*)pair_nodes_kernel, pair_lds);
  if (rc != TN_OK || p.P == 0) return rc;
  WsN ws = carve_nodes(workspace, p.P, p.N_max, p.C_max);
  hipLaunchKernelGGL(prep_nodes_kernel, dim3((p.P + G - 1) / G), dim3(G * kWave), prep_lds, stream,
                     make_view(p), ws, gene_pow2(p.N_max), gene_pow2(p.C_max));
  rc = check_launch();
  if (rc != TN_OK) return rc;
  const int rows = table_rows([&](int r) { return pair_nodes_table_lds(r, p.N_max, p.C_max); });
  if (rows) {
    const size_t lds = pair_nodes_table_lds(rows, p.N_max, p.C_max);
    const auto kern = rows == 4 ? pair_nodes_table_kernel<4> : pair_nodes_table_kernel<2>;
    rc = allow_lds((const void*)kern, lds);
    if (rc != TN_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((p.P + kTableBlock - 1) / kTableBlock, (p.P + rows - 1) / rows),
                       dim3(kTableBlock), lds, stream, ws, p.P, table_slots(rows, p.N_max),
                       table_slots(rows, p.C_max), c_d, c_h, dist, DN, DC);
    return check_launch();
  }
  dim3 grid((p.P + kPairBlock - 1) / kPairBlock, (p.P + R - 1) / R);
  hipLaunchKernelGGL(pair_nodes_kernel, grid, dim3(kPairBlock), pair_lds, stream, ws, p.P, HN,
                     HC, R, c_d, c_h, dist, DN, DC);
  return check_launch();
}

}  // namespace tn
