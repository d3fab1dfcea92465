// Transformation stage (TensorNEAT Section 3.3) of genomes of at most 64 node
// rows and 256 connection rows: the same results as transform_kernel, by one
// wavefront whose lanes are the node rows, then the topological positions.
// Included by transform.hip.
//
// A genome of this size fits the lanes, so the steps that transform_kernel
// makes of LDS round trips become operations on 64-bit masks: a node's sources
// are one mask (a Kahn round is a compare and a ballot), the free value rows
// are one mask, prefix sums over positions or in-edges are population counts of
// ballots, and attributes move between rows and positions by lane shuffles.
// Bound by latency: one round of loads, the key lookups, and the chain of
// rounds (150 genomes of 16 / 32 rows 7.7 us, 1000 of 64 / 256 rows 17.9 us;
// 25.7 and 40.1 us with transform_kernel).
#pragma once

#include "tn_internal.hpp"

namespace tn {
namespace {

constexpr int kSmallNodes = 64, kSmallConns = 256;

// Bits of `mask` below bit n (0 <= n <= 64).
__device__ __forceinline__ uint64_t bits_below(uint64_t mask, int n) {
  return n >= 64 ? mask : mask & ((1ull << n) - 1);
}

template <int KC>
struct SmallMem {
  int2 hash[2 * kSmallNodes];      // key, row; key -1: empty
  uint64_t adj[kSmallNodes];       // destinations of the valid connections of a source row
  uint64_t pred[kSmallNodes];      // sources of the enabled connections into a row
  uint64_t rows[KC][kSmallNodes];  // enabled connection rows (bit: lane of chunk j) into a row
  int2 edge[KC * kWave];           // in-edge list: source position | consumer << 8 | row << 16, weight;
                                   // then source's program row, weight
  int32_t last[kSmallNodes];       // last consumer of a position, -1: none
  int32_t order[kSmallNodes];
  int32_t ev[kSmallNodes];         // position whose program row the u-th free event frees
};

// KC: chunks of 64 connection rows.
template <int KC>
__global__ __launch_bounds__(kWave) void transform_small_kernel(PopView pop, TrView tr, Layout L) {
  __shared__ SmallMem<KC> mem;
  const int g = blockIdx.x, lane = threadIdx.x;
  const int64_t nb = pop.node_base(g), cb = pop.conn_base(g);
  const int64_t nrows64 = pop.node_rows(g), crows64 = pop.conn_rows(g);
  const bool bad = nrows64 > pop.N_max || crows64 > pop.C_max || nrows64 < 0 || crows64 < 0;
  if (bad ? !L.last : nrows64 > L.n_cap || crows64 > L.c_cap) return;  // another launch's genome
  if (bad) {
    write_flagged(pop, tr, g, TN_OVERSIZE, nb, nrows64 > 0 ? nrows64 : 0, cb,
                  crows64 > 0 ? crows64 : 0);
    return;
  }
  const int nrows = (int)nrows64, crows = (int)crows64;
  const int n_in = pop.n_in, nio = n_in + pop.n_out;

  // every row of the genome, one round of loads
  int key = -1, code = 0, bias = 0, resp = 0;
  if (lane < nrows) {
    key = pop.node_key[nb + lane];
    code = pop.node_act[nb + lane] | (pop.node_agg[nb + lane] << 8);
    bias = __float_as_int(pop.node_bias[nb + lane]);
    resp = __float_as_int(pop.node_resp[nb + lane]);
  }
  int ca[KC], cd[KC], w[KC];
  bool on[KC];
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const int r = j * kWave + lane;
    const bool row = r < crows;
    ca[j] = row ? pop.conn_in[cb + r] : -1;
    cd[j] = row ? pop.conn_out[cb + r] : -1;
    w[j] = row ? __float_as_int(pop.conn_w[cb + r]) : 0;
    on[j] = row && pop.conn_en[cb + r] != 0;
  }
  mem.hash[lane].x = mem.hash[kWave + lane].x = -1;
  mem.adj[lane] = mem.pred[lane] = 0;
  mem.last[lane] = -1;
#pragma unroll
  for (int j = 0; j < KC; ++j) mem.rows[j][lane] = 0;
  wave_sync();

  // node keys -> rows
  constexpr uint32_t kMask = 2 * kSmallNodes - 1;
  const bool node_row = key >= 0;
  bool dup_node = false;
  if (node_row) {
    uint32_t h = hash32((uint32_t)key) & kMask;
    while (true) {
      const int32_t old = atomicCAS(&mem.hash[h].x, -1, key);
      if (old == -1) mem.hash[h].y = lane;
      dup_node = old == key;
      if (old == -1 || dup_node) break;
      h = (h + 1) & kMask;
    }
  }
  const bool bad_attr = node_row && ((code & 0xff) > TN_ACT_ABS || (code >> 8) > TN_AGG_MAXABS);
  const int n = __popcll(__ballot(node_row));
  wave_sync();
  // rows of the connections' endpoints and of the input / output keys; the
  // first probes of all of them are requested together
  auto row_of = [&](int k, uint32_t h, int2 q) {
    while (q.x != k) {
      if (q.x == -1) return -1;
      h = (h + 1) & kMask;
      q = mem.hash[h];
    }
    return (int)q.y;
  };
  int sa[KC], sb[KC], io_row;
  {
    int2 qa[KC], qb[KC];
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      qa[j] = mem.hash[hash32((uint32_t)ca[j]) & kMask];
      qb[j] = mem.hash[hash32((uint32_t)cd[j]) & kMask];
    }
    const int2 qi = mem.hash[hash32((uint32_t)lane) & kMask];
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      const bool valid = ca[j] >= 0 && cd[j] >= 0;
      sa[j] = valid ? row_of(ca[j], hash32((uint32_t)ca[j]) & kMask, qa[j]) : -1;
      sb[j] = valid ? row_of(cd[j], hash32((uint32_t)cd[j]) & kMask, qb[j]) : -1;
    }
    io_row = lane < nio ? row_of(lane, hash32((uint32_t)lane) & kMask, qi) : -1;
  }
  const bool missing = (lane < nio && io_row < 0) || nio > kWave;

  // repeated markings, endpoints, the source masks
  bool dup = false, dangling = false, input_dst = false;
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const bool valid = ca[j] >= 0 && cd[j] >= 0, found = sa[j] >= 0 && sb[j] >= 0;
    if (found) {
      const uint64_t old = atomicOr((unsigned long long*)&mem.adj[sa[j]], 1ull << sb[j]);
      dup |= (old >> sb[j]) & 1;
    }
    on[j] = on[j] && valid;
    dangling |= on[j] && !found;
    input_dst |= on[j] && cd[j] < n_in;
    on[j] = on[j] && found;
    if (on[j]) {
      atomicOr((unsigned long long*)&mem.pred[sb[j]], 1ull << sa[j]);
      atomicOr((unsigned long long*)&mem.rows[j][sb[j]], 1ull << lane);
    }
    // a connection with an endpoint that has no row (disabled, or the genome is
    // flagged): its marking against every other row's
    for (uint64_t m = __ballot(valid && !found); m; m &= m - 1) {
      const int l = __ffsll((unsigned long long)m) - 1;
      const int a = __builtin_amdgcn_readlane(ca[j], l), b = __builtin_amdgcn_readlane(cd[j], l);
#pragma unroll
      for (int i = 0; i < KC; ++i) dup |= ca[i] == a && cd[i] == b && !(i == j && lane == l);
    }
  }
  const int st = (__ballot(bad_attr) ? TN_BAD_ATTR : 0) | (__ballot(dup_node) ? TN_DUP_NODE : 0) |
                 (__ballot(missing) ? TN_MISSING_IO : 0) | (__ballot(dup) ? TN_DUP_CONN : 0) |
                 (__ballot(dangling) ? TN_DANGLING : 0) | (__ballot(input_dst) ? TN_INPUT_DST : 0);
  if (st) {
    write_flagged(pop, tr, g, st, nb, nrows, cb, crows);
    return;
  }
  wave_sync();

  // level-synchronous Kahn rounds, rows in ascending order inside a round
  const uint64_t from = mem.pred[lane];
  int pos = -1, lvl_row = -1, placed = 0;
  {
    uint64_t done = 0;
    for (int l = 0;; ++l) {
      const bool ready = node_row && pos < 0 && (from & ~done) == 0;
      const uint64_t m = __ballot(ready);
      if (m == 0) break;
      if (ready) {
        pos = placed + mbcnt(m);
        lvl_row = l;
      }
      placed += __popcll(m);
      done |= m;
    }
  }
  if (placed < n) {
    write_flagged(pop, tr, g, TN_CYCLE, nb, nrows, cb, crows);
    return;
  }
  if (node_row) mem.order[pos] = lane;
  wave_sync();

  // lane = topological position from here on (p < n): its row's attributes
  const int p = lane;
  const bool real = p < n;
  const int s = real ? mem.order[p] : 0;
  const int k = __shfl(key, s, kWave), fn = __shfl(code, s, kWave);
  const int p_bias = __shfl(bias, s, kWave), p_resp = __shfl(resp, s, kWave);
  const int lvl = __shfl(lvl_row, s, kWave);
  const int sources = __shfl(__popcll(from), s, kWave);
  const int deg = real ? sources : 0;
  const int end = wave_inclusive_scan(deg), start = end - deg;
  const int n_edges = __builtin_amdgcn_readlane(end, kWave - 1);

  // in-edge lists: by consumer position, then ascending connection row
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const int to = on[j] ? sb[j] : 0;
    const int ps = __shfl(pos, on[j] ? sa[j] : 0, kWave), pd = __shfl(pos, to, kWave);
    const int first = __shfl(start, pd & (kWave - 1), kWave);
    if (on[j]) {
      int rank = mbcnt(mem.rows[j][to]);
#pragma unroll
      for (int i = 0; i < j; ++i) rank += __popcll(mem.rows[i][to]);
      mem.edge[first + rank] = make_int2(ps | (pd << 8) | ((j * kWave + lane) << 16), w[j]);
      atomicMax(&mem.last[ps], pd);
    }
  }
  wave_sync();
  const int last = mem.last[p];
  int2 e[KC];
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const int i = j * kWave + lane;
    const bool in = i < n_edges;
    e[j] = in ? mem.edge[i] : make_int2(0, 0);
    if (i < crows) {
      tr.edge_row[cb + i] = in ? e[j].x >> 16 : -1;
      tr.edge_src[cb + i] = in ? e[j].x & 0xff : -1;
      tr.edge_w[cb + i] = __int_as_float(e[j].y);
    }
  }
  const int64_t rb = pop.rowptr_base(g);
  for (int i = lane; i <= nrows; i += kWave) tr.row_ptr[rb + i] = i < n ? start : n_edges;
  if (p < nrows) {
    tr.order[nb + p] = real ? s : -1;
    tr.level[nb + p] = real ? lvl : -1;
    tr.pos_bias[nb + p] = real ? __int_as_float(p_bias) : 0.0f;
    tr.pos_resp[nb + p] = real ? __int_as_float(p_resp) : 0.0f;
    tr.pos_fn[nb + p] =
        real ? (k < n_in ? (int32_t)(kFnInput | ((uint32_t)k << 16) | (uint32_t)fn) : fn) : 0;
  }
  const int io_at = __shfl(pos, io_row < 0 ? 0 : io_row, kWave);
  if (lane < nio) tr.io_pos[(int64_t)g * nio + lane] = io_at;

  // value rows of the level-parallel pass: input k takes row k; level by
  // level, in position order, a node takes the lowest free row or a new one,
  // then the rows whose last reader is in the level are free
  const bool input = real && k < n_in, output = real && k >= n_in && k < nio;
  const bool node = real && k >= n_in;
  const int last_lvl = __shfl(lvl, last < 0 ? 0 : last, kWave);
  const int free_lvl = !real || output ? -1 : last >= 0 ? last_lvl : node ? lvl : -1;
  const uint64_t nodes = __ballot(node), unused = __ballot(input && last < 0);
  int row = input ? k : -1, next_row = n_in;
  {
    uint64_t open = 0;
    for (uint64_t m = unused; m; m &= m - 1)
      open |= 1ull << __builtin_amdgcn_readlane(k, __ffsll((unsigned long long)m) - 1);
    const int n_levels = __builtin_amdgcn_readlane(lvl, n - 1) + 1;
    for (int l = 0; l < n_levels; ++l) {
      for (uint64_t m = __ballot(node && lvl == l); m; m &= m - 1) {
        const int r = open ? __ffsll((unsigned long long)open) - 1 : next_row++;
        open &= open - 1;
        row = lane == __ffsll((unsigned long long)m) - 1 ? r : row;
      }
      for (uint64_t m = __ballot(free_lvl == l); m; m &= m - 1)
        open |= 1ull << __builtin_amdgcn_readlane(row, __ffsll((unsigned long long)m) - 1);
    }
  }
  if (p < nrows) tr.pos_row[nb + p] = real ? row : -1;

  // program rows (one position after the other, freed rows first in, first
  // out): the free events in order are the unused inputs; then at each
  // position the dead value before it and the sources it reads last
  const int n_unused = __popcll(unused);
  const uint64_t dead = __ballot(real && k >= nio && last < 0);
  uint64_t frees[KC];
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const int src = e[j].x & 0xff, to = (e[j].x >> 8) & 0xff;
    const int src_last = __shfl(last, src, kWave), src_out = __shfl((int)output, src, kWave);
    frees[j] = __ballot(j * kWave + lane < n_edges && src_last == to && !src_out);
  }
  // in-edges before entry i that free their source
  auto frees_before = [&](int i) {
    int c = 0;
#pragma unroll
    for (int j = 0; j < KC; ++j)
      c += __popcll(bits_below(frees[j], max(0, min(i - j * kWave, kWave))));
    return c;
  };
  if (input && last < 0) mem.ev[mbcnt(unused)] = p;
  if (((dead >> p) & 1) && p + 1 < n) mem.ev[n_unused + mbcnt(dead) + frees_before(end)] = p;
#pragma unroll
  for (int j = 0; j < KC; ++j)
    if ((frees[j] >> lane) & 1) {
      const int to = (e[j].x >> 8) & 0xff;
      mem.ev[n_unused + __popcll(bits_below(dead, to)) + frees_before(j * kWave + lane)] =
          e[j].x & 0xff;
    }
  const int freed = n_unused + mbcnt(dead) + frees_before(end);  // up to this position
  const int taken = mbcnt(nodes) + 1;                            // allocations up to this node
  const int made = max(0, wave_inclusive_max(node ? taken - freed : INT_MIN));  // rows created
  const int made_up = __shfl_up(made, 1, kWave);  // every lane active: lane 0 is read
  const int made_before = lane == 0 ? 0 : made_up;
  const int n_new = __builtin_amdgcn_readlane(made, kWave - 1);
  wave_sync();
  int prog = k;
  if (node) prog = made > made_before ? n_in + made - 1 : -(mem.ev[taken - made - 1] + 1);
  // "same row as position q" links, resolved by pointer jumping
  while (__ballot(node && prog < 0)) {
    const int t = __shfl(prog, prog < 0 && node ? -prog - 1 : lane, kWave);
    if (node && prog < 0) prog = t;
  }

  // the packed program
  if (p < nrows) {
    const int32_t word = input ? (int32_t)(kFnInput | ((uint32_t)k << 16)) : fn | (prog << 16);
    tr.prog_node[nb + p] = real ? make_int4(end, word, p_bias, p_resp) : make_int4(0, 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < KC; ++j) {
    const int i = j * kWave + lane;
    const int2 q = make_int2(__shfl(prog, e[j].x & 0xff, kWave), e[j].y);
    if (i < n_edges) mem.edge[i] = q;
    if (i < crows) tr.prog_edge[cb + i] = i < n_edges ? q : make_int2(0, 0);
  }
  wave_sync();
  int4* recs = reinterpret_cast<int4*>(tr.prog_rec) + nb * 4;
  if (node) {
    int4* rec = recs + mbcnt(nodes) * 4;
    int2 q[6];
#pragma unroll
    for (int i = 0; i < 6; ++i)
      q[i] = i < deg ? mem.edge[start + i] : make_int2(n_in + n_new, 0);
    rec[0] = make_int4((fn & 0xff) | ((fn >> 8) << 3) | (prog << 6) | (deg << 17), p_bias, p_resp,
                       start + 6);
    rec[1] = make_int4(q[0].x, q[0].y, q[1].x, q[1].y);
    rec[2] = make_int4(q[2].x, q[2].y, q[3].x, q[3].y);
    rec[3] = make_int4(q[4].x, q[4].y, q[5].x, q[5].y);
  }
  for (int i = __popcll(nodes) * 4 + lane; i < nrows * 4; i += kWave) recs[i] = make_int4(0, 0, 0, 0);
  if (lane == 0) {
    tr.status[g] = 0;
    tr.n_valid[g] = n;
    tr.n_rows[g] = next_row;
    tr.prog_rows[g] = n_in + n_new;
  }
}

}  // namespace
}  // namespace tn
