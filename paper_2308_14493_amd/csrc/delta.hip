// Edge-local update of the Sigma terms of a one-batch pass: instead of
// counting the region of change in both versions, only the structures that
// contain a changed pair are enumerated (the idea of updating the count from
// where the change is located, Sec. 4.1), giving C(G_a) - C(G_b) exactly.
//
// Input: the union view left by the tombstone merge (rows sorted by id; an
// entry carries GC_F_NEW when it is absent before the batch, GC_F_DEL when
// absent after it), the sorted directed change lists dirA / dirD and the
// touched rows.  Output: the per-graph sums of version 1 of the pass hold
// the deltas of every Sigma term (version 0 stays zero), so the combine
// kernel applies them unchanged; the triangle counts kept per vertex (Tv) and
// per edge (PoolDev::tt) move to the graph after the batch.
//
// A structure (triangle, 4-clique, 4-cycle) that holds several changed pairs
// is counted once, from the changed pair with the smallest key (min << bits |
// max); it adds [present after] - [present before], decided by the OR of its
// entries' flags.  Per term:
//   S1, W, D1   touched vertices (their degrees before and after);
//   S2          edges at touched vertices, each once;
//   T           triangles {u, v, w} through a changed edge (u, v), w in the
//               common neighbours S(e); each moves t of its three edges and T
//               of its three vertices;
//   DIA         sum_e C(t_e, 2): the edges whose t moved (the affected edges),
//               with t before the batch kept per resident entry (PoolDev::tt);
//   PAW         sum_e t_e (d_u + d_v - 4) = 2 sum_v d_v T(v) - 12 T: the vertices
//               whose degree or T (kept per vertex) moved;
//   K4          per changed edge e = (u, v): pairs {w, x} of S(e) joined by an
//               edge, found like the 4-cycles below: the rows of S(e) walked
//               against a bitmap of S(e), or, where that costs more, its pairs
//               searched;
//   C4          per changed edge: paths s - a - b - o closing the cycle with
//               e = (s, o), from the common ids of N(a) and N(o) for each
//               pair (s, a): the rows N(a) walked against an LDS bitmap of
//               N(o), or, where that costs more (little to walk for the edge,
//               or an N(a) far longer than N(o)), the shorter row walked and
//               searched in the other.  What a bitmap leaves out of N(o) or
//               S(e) is searched too, or, where it is much, the edge is walked
//               in layers that leave nothing out.
#include "gc_kernels.h"

#include <algorithm>

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ int64_t gtid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ int64_t ctr(const unsigned long long* c, int k) { return (int64_t)c[k]; }

// flags of an entry as a 2-bit nibble: bit 0 = absent before, bit 1 = absent after
__device__ __forceinline__ uint32_t nib(uint32_t entry) { return (entry >> GC_VSHIFT) & 3u; }
// [present after] - [present before] of a structure whose entries' nibbles OR to f
__device__ __forceinline__ int64_t delta_of(uint32_t f) { return (int64_t)((f & 2u) == 0) - (int64_t)((f & 1u) == 0); }

__device__ __forceinline__ unsigned long long pkey(uint32_t a, uint32_t b, int bits) {
  const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
  return ((unsigned long long)lo << bits) | hi;
}

// The entries of up to 64 row pieces, the wave together: lane l holds piece
// [b, b + n) of col with a payload; f(payload, entry) on some lane for each
// entry.  Pieces of at least 32 entries go one at a time through the wave
// (consecutive lanes, four loads in flight per lane), the others are
// flattened over the lanes with a search for the piece of each index.
template <class F>
__device__ __forceinline__ void wave_rows(const uint32_t* __restrict__ col, int64_t b, int32_t n, uint32_t pay, F f) {
  const int l = lane_id();
  const bool lng = n >= 32;
  for (uint64_t m = __ballot(lng); m; m &= m - 1) {
    const int src = __builtin_ctzll(m);
    const uint32_t* row = col + (((int64_t)__builtin_amdgcn_readlane((uint32_t)((uint64_t)b >> 32), src) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((uint32_t)b, src));
    const int32_t cnt = __builtin_amdgcn_readlane(n, src);
    const uint32_t ps = __builtin_amdgcn_readlane(pay, src);
    int32_t k = l;
    for (; k + 192 < cnt; k += 256) {
      uint32_t y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] = row[k + 64 * q];
#pragma unroll
      for (int q = 0; q < 4; ++q) f(ps, y[q]);
    }
    for (; k < cnt; k += 64) f(ps, row[k]);
  }
  const int32_t ns = lng ? 0 : n;
  const int32_t incl = wave_incl_scan32(ns), tot = __shfl(incl, 63), excl = incl - ns;
  for (int32_t at = 0; at < tot; at += 64) {
    const int32_t idx = at + l;
    int lo = 0, hi = 64;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const int mid = (lo + hi) >> 1;
      if (__shfl(excl, mid) <= idx) lo = mid; else hi = mid;
    }
    const int64_t bb = __shfl(b, lo);
    const int32_t ex = __shfl(excl, lo);
    const uint32_t ps = __shfl(pay, lo);
    if (idx < tot) f(ps, col[bb + (idx - ex)]);
  }
}

// degree of v in version x (0 before, 1 after): touched rows carry flags and
// have their two degrees in dd; the others have none
__device__ __forceinline__ int64_t deg_of(const DeltaArgs& D, uint32_t v, int x) {
  return D.mark[v] ? (int64_t)D.dd[2 * (int64_t)v + x] : (int64_t)D.P.len[v];
}

__device__ __forceinline__ void add_sig(const DeltaArgs& D, int g, int k, int64_t v) {
  v = wave_sum64(v);
  if (lane_id() == 0 && v != 0) atomicAdd(&D.sig[SIG_IDX(g, 1, k)], (unsigned long long)v);
}

// the same where lanes may work for different graphs (g < 0: none)
__device__ __forceinline__ void add_sig_lanes(const DeltaArgs& D, int g, int k, int64_t v) {
  const bool has = g >= 0 && v != 0;
  const uint64_t m = __ballot(has);
  if (!m) return;
  const int gl = __shfl(g, __builtin_ctzll(m));
  if (__ballot(has && g != gl) == 0) add_sig(D, gl, k, has ? v : 0);
  else if (has) atomicAdd(&D.sig[SIG_IDX(g, 1, k)], (unsigned long long)v);
}

}  // namespace

// --------------------------------------------------------------- changed
// The changed pairs (u < v) of the pass from the directed lists, with the
// pair's nibble in bits 60..61.
__global__ void k_delta_edges(DeltaArgs D) {
  const int64_t na = ctr(D.c, C_DIRA), nd = ctr(D.c, C_DIRD);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  for (int64_t i = gtid(); i < na + nd; i += gstride()) {
    const unsigned long long k = i < na ? D.dirA[i] : D.dirD[i - na];
    const unsigned long long key = k & DIR_KEY_MASK;
    const uint32_t r = (uint32_t)(key >> D.bits), c = (uint32_t)(key & idmask);
    if (r >= c) continue;
    const unsigned long long p = atomicAdd(&D.dc[DC_EDGES], 1ull);
    if ((int64_t)p < D.ce_cap) {
      D.ce[p] = key | ((unsigned long long)(i < na ? 1u : 2u) << DIR_MASK_SHIFT);
      D.e_ns[p] = 0;
      D.e_out[p] = 0;
      D.e_dt[p] = 0;
      D.e_kw[p] = 0;
    }
  }
}

// ------------------------------------------------------- touched vertices
// The touched rows are cut in pieces of at most TV_CHUNK entries (a hub row
// in many), numbered by a scan, and each wave takes one piece at a time: no
// wave walks a whole hub row alone.

// pieces per touched row (0 past the touched count, for the scan)
__global__ void k_delta_titems(DeltaArgs D) {
  const int64_t nt = ctr(D.c, C_TOUCH);
  for (int64_t t = gtid(); t < D.tcap; t += gstride()) {
    int32_t n = 0;
    if (t < nt) {
      const int32_t x = D.touched[t];
      n = max(1, (D.P.len[x] + TV_CHUNK - 1) / TV_CHUNK);
      D.dd[2 * (int64_t)x] = 0;
      D.dd[2 * (int64_t)x + 1] = 0;
    }
    D.tv_items[t] = n;
  }
}

// touched row and entry range of piece k (wave-uniform)
__device__ __forceinline__ void touched_piece(const DeltaArgs& D, int64_t nt, int64_t k, uint32_t& x, int32_t& k0,
                                              int32_t& k1) {
  int64_t lo = 0, hi = nt;  // largest t with tv_ioff[t] <= k
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (D.tv_ioff[mid] <= k) lo = mid; else hi = mid;
  }
  x = (uint32_t)D.touched[lo];
  k0 = (int32_t)((k - D.tv_ioff[lo]) * TV_CHUNK);
  k1 = min(D.P.len[x], k0 + TV_CHUNK);
}

// degrees of the touched rows before and after the batch, by pieces
__global__ void k_delta_vertex(DeltaArgs D) {
  const int64_t nt = ctr(D.c, C_TOUCH);
  if (nt == 0) return;
  const int64_t np = D.tv_ioff[nt];
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  for (int64_t k = w0; k < np; k += ws) {
    uint32_t x;
    int32_t k0, k1;
    touched_piece(D, nt, k, x, k0, k1);
    const uint32_t* row = D.P.col + D.P.off[x];
    int32_t db = 0, da = 0;
    for (int32_t q = k0 + l; q < k1; q += 64) {
      const uint32_t f = nib(row[q]);
      db += (f & 1u) == 0;
      da += (f & 2u) == 0;
    }
    db = wave_sum32(db);
    da = wave_sum32(da);
    if (l == 0) {
      if (db) atomicAdd(&D.dd[2 * (int64_t)x], db);
      if (da) atomicAdd(&D.dd[2 * (int64_t)x + 1], da);
    }
  }
}

// S2 = sum_e (d_u - 1)(d_v - 1) changes only on edges at a touched vertex;
// an edge between two touched vertices is taken at the smaller id.
// The 3-star, wedge and degree-sum terms of each touched vertex come with it.
// Sums stay with the lanes while the graph stays the same.
__global__ void k_delta_s2(DeltaArgs D) {
  const int64_t nt = ctr(D.c, C_TOUCH);
  if (nt == 0) return;
  const int64_t np = D.tv_ioff[nt];
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  int64_t acc = 0;
  int cur_g = -1;
  for (int64_t k = w0; k < np; k += ws) {
    uint32_t x;
    int32_t k0, k1;
    touched_piece(D, nt, k, x, k0, k1);
    const int g = D.gid[x];
    if (g != cur_g) {
      if (cur_g >= 0) add_sig(D, cur_g, SG_S2, acc);
      acc = 0;
      cur_g = g;
    }
    const uint32_t* row = D.P.col + D.P.off[x];
    const int64_t dbx = D.dd[2 * (int64_t)x] - 1, dax = D.dd[2 * (int64_t)x + 1] - 1;
    for (int32_t q = k0 + l; q < k1; q += 64) {
      const uint32_t e = row[q], y = e & GC_ID, f = nib(e);
      if (D.mark[y] && y < x) continue;
      if ((f & 2u) == 0) acc += dax * (deg_of(D, y, 1) - 1);
      if ((f & 1u) == 0) acc -= dbx * (deg_of(D, y, 0) - 1);
    }
  }
  if (cur_g >= 0) add_sig(D, cur_g, SG_S2, acc);
  // the vertices' own terms, a lane each
  for (int64_t b0 = w0 * 64; b0 < nt; b0 += ws * 64) {
    int g = -1;
    int64_t s1 = 0, w2 = 0, d1 = 0;
    if (b0 + l < nt) {
      const uint32_t x = (uint32_t)D.touched[b0 + l];
      const int64_t db = D.dd[2 * (int64_t)x], da = D.dd[2 * (int64_t)x + 1];
      g = D.gid[x];
      s1 = c3(da) - c3(db);
      w2 = c2(da) - c2(db);
      d1 = da - db;
    }
    add_sig_lanes(D, g, SG_S1, s1);
    add_sig_lanes(D, g, SG_W, w2);
    add_sig_lanes(D, g, SG_D1, d1);
  }
}

// ------------------------------------------------------------- 4-cycles
// Through a changed edge e = (s, o) run the 4-cycles s - a - b - o with
// a in N(s) - {o}, b in N(a) & N(o) - {s}.  A pair (e, a) is counted in one
// of two ways (pair_walked): its row N(a) is walked against a bitmap of N(o)
// that a workgroup keeps in LDS (k_delta_bits), or the shorter of N(a) and
// N(o) is walked and each entry searched in the other row (k_delta_search).  s is
// the end with the smaller total cost.  The work is balanced over the whole
// chip: every pair gets its walk length, a scan places the walked entries of
// all pairs in one index space, and waves or workgroups take ranges of that
// space (a hub pair is spread over many waves).

// A walked entry costs one LDS probe, a searched one a chain of dependent
// loads: 9.2e11 walked entries a second at scale 22 (2,500 updates, 5.9e9 of
// them) and 4.5e11 at scale 18 (1,000 updates, 1.2e8), against 3.7e10 searched.
// The line lies above their quotient, as the few pairs searched do not hide
// their chains behind each other.  With 16 and 24 in the place of 64: 1,000
// updates at scale 18 10% and 3% slower, on the hub graph 2% and 3%, 100 on
// livejournal's size 5% and 4%, 2,500 at scale 22 1% and as fast.
constexpr int64_t C4B_RATIO = 64;
// An edge whose walks sum to less than this does not earn a bitmap (clearing,
// filling and the queue cost a workgroup about as much as searching so much).
// For the 4-cycles the row of the edge's other end is not among the walks:
// with it, every edge of a hub earned one.  4,096 there instead of 2,048: 1,000
// updates at scale 18 1.5% slower, on the hub graph 1% faster.
constexpr int64_t C4B_MIN = 2048, K4B_MIN = 4096;
constexpr int C4B_T = 1024;
constexpr int C4B_SMALL = 16384, C4B_LARGE = 36864;  // 32-bit words of the two bitmaps: 64 and 144 KB
// Members that a bitmap leaves out (below its window, or with an edge to the
// changed pair that is in the batch too) are searched one by one.  At a hub
// they are as many as the batch's updates there, or as its neighbours among
// the low ids, for every changed edge of the hub: 1,000 deletions at a star of
// 2,000,000 leaves listed 8e8 searched pairs (33 GB of lists, 179 ms; 3.3 now).
// So an edge that leaves out more than C4B_OUT is walked in layers
// (k_delta_layers) where its searches, at C4B_SEARCH walked entries each, cost
// more than the walk, or list more pairs than C4B_OUT_MAX or its share of what
// the lists hold; but for the 4-cycles only in a batch whose searches together
// cost more than C4B_FREE and a quarter of its walks, or list more pairs than
// C4B_OUT_ALL and the walked ones, as a few edges in layers are a tail of long
// chunks: with every edge above C4B_OUT, 2,500 updates at scale 22 took 13.8
// ms a call instead of 8.6, and with the two limits by equal shares alone
// 57,032 updates 220 ms instead of 179.  No batch of 128 updates on ids that
// fit a bitmap leaves out more than C4B_OUT: small passes do not launch the
// kernel of the layers.
constexpr int32_t C4B_OUT = 128;
constexpr int64_t C4B_SEARCH = 16, C4B_FREE = 1ll << 32, C4B_OUT_MAX = 16384, C4B_OUT_ALL = 1 << 22;

// out members of an edge cost more to search (the entries that the searches
// walk) than to walk the edge (cost) and its share of C4B_FREE among ne edges
__device__ __forceinline__ bool search_dear(int64_t out, int64_t entries, int64_t cost, int64_t ne) {
  return out > C4B_OUT && entries * C4B_SEARCH > cost + C4B_FREE / ne;
}
// What the batch says (k_delta_plan_fin's sums): the edges marked dear to
// search, and those marked to list too many, are walked in layers.
struct C4Layers {
  bool dear, many;
  __device__ __forceinline__ explicit C4Layers(const DeltaArgs& D)
      : dear(ctr(D.dc, DC_OUT_WALK) * C4B_SEARCH > C4B_FREE + ctr(D.dc, DC_COST) / 4),
        many(ctr(D.dc, DC_OUT) > C4B_OUT_ALL + D.pair_cap) {}
  __device__ __forceinline__ bool operator()(int32_t side) const {
    return (side & 4) || (dear && (side & 8)) || (many && (side & 16));
  }
};

__device__ __forceinline__ int64_t pair_cost(int32_t al, int32_t ol) {
  return min((int64_t)al, C4B_RATIO * (int64_t)ol);
}
// The bitmap of N(o) covers D.c4_ids ids downwards from N(o)'s last one: ids
// are a degree order, so the ids below that window have few entries.
__device__ __forceinline__ uint32_t c4b_top(const DeltaArgs& D, uint32_t o) {
  return (D.P.col[D.P.off[o] + D.P.len[o] - 1] & GC_ID) + 1u;
}
__device__ __forceinline__ uint32_t c4b_base(const DeltaArgs& D, uint32_t o) {
  const uint32_t top = c4b_top(D, o);
  return top > D.c4_ids ? top - D.c4_ids : 0u;
}
// pairs of an edge with a bitmap that are walked against it
__device__ __forceinline__ bool pair_walked(int32_t al, int32_t ol) { return (int64_t)al <= C4B_RATIO * (int64_t)ol; }

// per changed edge: the end to walk from, whether it earns a bitmap, and its
// number of pairs.  An end u costs sum_{a in N(u) - {v}} pair_cost(d_a, d_v); both rows of every
// changed edge are cut in pieces of at most TV_CHUNK entries (the touched
// rows' arrays hold the numbering; they are free again after the degree
// passes), each wave sums one piece at a time into the edge's two totals
// (kept in pair_off, free until the pair scan), and a last pass picks the
// cheaper end.
__global__ void k_delta_plan_items(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  for (int64_t i = gtid(); i < D.tcap; i += gstride()) {
    int32_t n = 0;
    if (i < ne) {
      const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
      const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
      n = max(1, (D.P.len[u] + TV_CHUNK - 1) / TV_CHUNK) + max(1, (D.P.len[v] + TV_CHUNK - 1) / TV_CHUNK);
      D.pair_off[2 * i] = 0;
      D.pair_off[2 * i + 1] = 0;
    }
    D.tv_items[i] = n;
  }
}

__global__ void k_delta_c4_plan(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  if (ne == 0) return;
  const int64_t np = D.tv_ioff[ne];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  for (int64_t k = w0; k < np; k += ws) {
    int64_t lo = 0, hi = ne;  // the edge holding piece k
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (D.tv_ioff[mid] <= k) lo = mid; else hi = mid;
    }
    const int64_t i = lo;
    const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const int32_t du = D.P.len[u], dv = D.P.len[v];
    const int64_t nu = max(1, (du + TV_CHUNK - 1) / TV_CHUNK);
    const int64_t pk = k - D.tv_ioff[i];
    const bool side_v = pk >= nu;  // pieces of u first, then of v
    const uint32_t x = side_v ? v : u, z = side_v ? u : v;
    const int32_t dx = side_v ? dv : du, other = side_v ? du : dv;
    const int32_t k0 = (int32_t)((side_v ? pk - nu : pk) * TV_CHUNK), k1 = min(dx, k0 + TV_CHUNK);
    const uint32_t* rx = D.P.col + D.P.off[x];
    int64_t c = 0;
    for (int32_t q = k0 + l; q < k1; q += 64) {
      const uint32_t a = rx[q] & GC_ID;
      if (a != z) c += pair_cost(D.P.len[a], other);
    }
    c = wave_sum64(c);
    if (l == 0 && c) atomicAdd((unsigned long long*)&D.pair_off[2 * i + (side_v ? 1 : 0)], (unsigned long long)c);
  }
}

__global__ void k_delta_plan_fin(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  int64_t outs = 0, walks = 0, costs = 0;  // of the edges with a bitmap
  for (int64_t i = gtid(); i < D.ce_cap; i += gstride()) {
    if (i >= ne) {
      D.c4_nch[i] = 0;
      D.c4_side[i] = 0;
      continue;
    }
    const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const bool from_u = D.pair_off[2 * i] <= D.pair_off[2 * i + 1];
    const int64_t cost = from_u ? D.pair_off[2 * i] : D.pair_off[2 * i + 1];
    const bool bitmap = cost >= C4B_MIN;
    const uint32_t s = from_u ? u : v, o = from_u ? v : u;
    int32_t low = 0;  // N(o) below the window
    int32_t layers = 0;
    if (bitmap) {
      const uint32_t base = c4b_base(D, o);
      const int64_t sl = D.P.len[s], flagged = (int64_t)D.na[o] + D.nr[o];
      int64_t entries = flagged * sl;  // walked and searched: the shorter row of each pair
      if (base) {
        low = lower_bound_id(D.P.col + D.P.off[o], D.P.len[o], base);
        entries += low * min(sl, (int64_t)D.P.len[base - 1]);  // ids are a degree order
      }
      const int64_t out = low + flagged, share = (C4B_OUT_ALL + D.pair_cap) / ne;
      if (D.c4_out > 0)
        layers = out > D.c4_out ? 4 : 0;
      else
        layers = (search_dear(out, entries, cost, ne) ? 8 : 0) |
                 (out > max((int64_t)C4B_OUT, min(C4B_OUT_MAX, share)) ? 16 : 0);
      outs += out;
      walks += entries;
      costs += cost;
    }
    D.c4_side[i] = (from_u ? 0 : 1) | (bitmap ? 2 : 0) | layers;
    D.c4_low[i] = low;
    D.c4_nch[i] = D.P.len[s];
  }
  outs = wave_sum64(outs);
  walks = wave_sum64(walks);
  costs = wave_sum64(costs);
  if (lane_id() == 0 && outs) {
    atomicAdd(&D.dc[DC_OUT], (unsigned long long)outs);
    atomicAdd(&D.dc[DC_OUT_WALK], (unsigned long long)walks);
    atomicAdd(&D.dc[DC_COST], (unsigned long long)costs);
  }
}

// The k-th pair (e, b) of an edge with a bitmap of N(o): N(o)'s `low` entries
// below the window (those in the batch are met again among the others), then
// its insertions, then its deletions.
__device__ __forceinline__ void c4_out_pair(const DeltaArgs& D, uint32_t o, int32_t low, int32_t k, uint32_t& b,
                                            uint32_t& fob) {
  const int32_t na = D.na[o];
  if (k < low) {
    const uint32_t e = D.P.col[D.P.off[o] + k];
    b = e & GC_ID;
    fob = nib(e);
    return;
  }
  k -= low;
  const unsigned long long key = k < na ? D.dirA[D.a_beg[o] + k] : D.dirR[D.r_beg[o] + (k - na)];
  b = (uint32_t)(key & ((1ull << D.bits) - 1ull));
  fob = k < na ? 1u : 2u;
}

// Appends a searched pair (edge i, index j, len entries; j < 0: of the
// 4-cliques, at member ~j of S(e)) of the lanes with
// `take` to the list (one atomic per wave).
__device__ __forceinline__ void search_append(const DeltaArgs& D, bool take, int64_t i, int32_t j, int32_t len) {
  const uint64_t m = __ballot(take);
  if (!m) return;
  unsigned long long at = 0;
  if (lane_id() == 0) at = atomicAdd(&D.dc[DC_SEARCH], (unsigned long long)__popcll(m));
  const int64_t q = (int64_t)__shfl((long long)at, 0) + __popcll(m & lanemask_lt());
  if (take && q < 2 * D.pair_cap) {
    D.pair_edge[q] = (int32_t)i;
    D.pair_idx[q] = j;
    D.pair_len[q] = len;
  }
}

// Moves t of the edge whose entry (in the row of its smaller end) is at
// resident position pos by d, in a hash table of the pass; true where the
// edge is met first, with its slot.  A table too full raises DC_AFF_FULL.
__device__ __forceinline__ bool t_move(const DeltaArgs& D, int64_t pos, int32_t d, uint32_t& slot) {
  uint32_t h = (uint32_t)(((unsigned long long)pos * 0x9E3779B97F4A7C15ull) >> 32) & D.hmask;
  const unsigned long long key = (unsigned long long)pos + 1ull;
  for (int k = 0; k < 512; ++k, h = (h + 1) & D.hmask) {
    unsigned long long old = __hip_atomic_load(&D.hk[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0ull) old = atomicCAS(&D.hk[h], 0ull, key);
    if (old != 0ull && old != key) {
      // a table found full is not searched to the end again
      if ((k & 31) == 31 && __hip_atomic_load(&D.dc[DC_AFF_FULL], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
      continue;
    }
    atomicAdd(&D.hd[h], d);
    slot = h;
    return old == 0ull;
  }
  D.dc[DC_AFF_FULL] = 1ull;
  return false;
}

// Appends the affected edges met first (slot, one of their ends) to the list.
__device__ __forceinline__ void aff_append(const DeltaArgs& D, bool take, uint32_t end, uint32_t slot) {
  const uint64_t m = __ballot(take);
  if (!m) return;
  unsigned long long at = 0;
  if (lane_id() == 0) at = atomicAdd(&D.dc[DC_AFF], (unsigned long long)__popcll(m));
  const int64_t q = (int64_t)__shfl((long long)at, 0) + __popcll(m & lanemask_lt());
  if (take && q < D.ae_cap) D.hl[q] = ((unsigned long long)end << 32) | slot;
}

// resident position of the edge (r, w) in the row of its smaller end; at:
// position of w in row r
__device__ __forceinline__ int64_t edge_pos(const DeltaArgs& D, uint32_t r, uint32_t w, int64_t at) {
  if (r < w) return at;
  return D.P.off[w] + lower_bound_id(D.P.col + D.P.off[w], D.P.len[w], r);
}

// A lane per pair (e, a), e = (s, o), a in N(s): the entries it walks against
// the bitmap, in pair order (0 for the others); the searched pairs go to a
// list that holds nothing else, so that the waves of k_delta_search meet no
// empty pairs.  And a in N(o) (searched) is a common neighbour: a triangle,
// counted here unless another of its edges is a changed pair of smaller key.
__global__ void k_delta_pairs(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  if (gtid() == 0) {
    D.dc[DC_WALK] = npairs > D.pair_cap ? 0ull : 2ull * (unsigned long long)npairs;
    if (npairs > D.pair_cap) {
      atomicAdd(&D.bstats[BS_RETRY], 1ull);
      atomicMax(&D.dc[DC_PAIR_NEED], (unsigned long long)npairs);
    }
  }
  if (npairs > D.pair_cap || ne == 0) return;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  for (int64_t b0 = w0 * 64; b0 < npairs; b0 += ws * 64) {
    const int64_t i0 = wave_upper_bound(D.c4_off, ne, b0);
    const int64_t p = b0 + l;
    const bool in = p < npairs;
    const int64_t i = in ? upper_bound_from(D.c4_off, ne, i0, p) : i0;
    const unsigned long long ek = D.ce[i], K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const int32_t side = D.c4_side[i];
    const uint32_t s = (side & 1) ? v : u, o = s == u ? v : u;
    const int32_t k = (int32_t)(p - D.c4_off[i]);
    const int64_t so = D.P.off[s], oo = D.P.off[o];
    const int32_t ol = D.P.len[o];
    const uint32_t es = in ? D.P.col[so + k] : o, a = es & GC_ID;
    const int32_t al = D.P.len[a];
    const bool walked = (side & 2) && a != o && pair_walked(al, ol);
    if (in) D.pair_hlen[p] = walked ? al : 0;
    search_append(D, a != o && !walked, i, k, min(al, ol));
    // a triangle?
    bool hit = false;
    int32_t x = 0;
    uint32_t eo = 0;
    if (a != o) {
      x = lower_bound_id(D.P.col + oo, ol, a);
      if (x < ol) { eo = D.P.col[oo + x]; hit = (eo & GC_ID) == a; }
    }
    const uint64_t hm = __ballot(hit);
    if (!hm) continue;
    if (l == 0) atomicAdd(&D.dc[DC_AFF_INST], 2ull * (unsigned long long)__popcll(hm));
    const uint32_t fs = nib(es), fo = nib(eo);
    const bool outside = hit && ((fs | fo) != 0 || (D.N > (int64_t)D.c4_ids && a < c4b_base(D, o)));
    for (uint64_t m = hm; m;) {  // S(e): one reservation per edge met by the wave
      const int src = __builtin_ctzll(m);
      const int32_t ii = __builtin_amdgcn_readlane((int32_t)i, src);
      const bool mine = hit && (int32_t)i == ii;
      const uint64_t same = __ballot(mine);
      int32_t at = 0;
      if (l == src) at = atomicAdd(&D.e_ns[ii], (int32_t)__popcll(same));
      at = __shfl(at, src);
      const uint64_t om = __ballot(mine && outside);
      if (om && l == src) atomicAdd(&D.e_out[ii], (int32_t)__popcll(om));
      if (mine) D.slist[D.c4_off[i] + at + __popcll(same & lanemask_lt())] = a | (fs << 28) | (fo << 30);
      m &= ~same;
    }
    int32_t d = 0;
    if (hit) {
      atomicAdd((unsigned long long*)&D.e_kw[i], (unsigned long long)al);
      if (!((fs && pkey(s, a, D.bits) < K) || (fo && pkey(o, a, D.bits) < K))) d = (int32_t)delta_of(fe | fs | fo);
    }
    bool n1 = false, n2 = false;
    uint32_t h1 = 0, h2 = 0;
    if (d) {
      atomicAdd(&D.e_dt[i], d);
      atomicAdd(&D.dT[a], (unsigned long long)(long long)d);
      n1 = t_move(D, edge_pos(D, s, a, so + k), d, h1);
      n2 = t_move(D, edge_pos(D, o, a, oo + x), d, h2);
    }
    aff_append(D, n1, a, h1);
    aff_append(D, n2, a, h2);
  }
  // the pairs (e, b), several waves per edge while there are fewer edges than waves
  const C4Layers layers(D);
  const int32_t parts = (int32_t)max(ws / ne, (int64_t)1);
  for (int64_t i = w0 % ne, part = w0 / ne; i < ne && part < parts; i += ws) {
    if (!(D.c4_side[i] & 2) || layers(D.c4_side[i])) continue;
    const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const uint32_t s = (D.c4_side[i] & 1) ? v : u, o = s == u ? v : u;
    const int32_t sl = D.P.len[s];
    const int32_t low = D.c4_low[i], out = low + D.na[o] + D.nr[o];
    for (int32_t k0 = (int32_t)part * 64; k0 < out; k0 += parts * 64) {
      const int32_t k = k0 + l;
      uint32_t b = s, fob = 0;
      if (k < out) c4_out_pair(D, o, low, k, b, fob);
      const bool take = b != s && !(fob != 0 && (k < low || pkey(o, b, D.bits) < K));
      search_append(D, take, i, sl + k, min(D.P.len[b], sl));
    }
  }
}

// The 4-cliques of an edge with ns common neighbours, whose rows hold kw
// entries: walked against a bitmap of S(e), unless searching the ns^2 / 2
// pairs costs less (a search as C4B_RATIO / 4 * 3 walked entries, about 12
// steps) or there is little to walk.
__device__ __forceinline__ bool k4_walked(int32_t ns, int64_t kw) {
  return kw >= K4B_MIN && kw <= 3 * C4B_RATIO / 8 * (int64_t)ns * ns;
}
__device__ __forceinline__ bool k4_layers(const DeltaArgs& D, int64_t i) {
  const int64_t out = D.e_out[i];
  if (D.c4_out > 0) return out > D.c4_out;
  return search_dear(out, out * D.e_ns[i], D.e_kw[i], ctr(D.dc, DC_EDGES));
}
// members of S(e) (id | flags of both edges << 28) that its bitmap leaves out
__device__ __forceinline__ bool k4_outside(uint32_t w, uint32_t base) { return (w & GC_FLAGS) || (w & GC_ID) < base; }

// After the triangles: what they add at the changed edges themselves, and
// the work lists of the 4-cliques, a lane per member w of a list S(e) (the
// lists sit in the pair space).  An edge that walks: each member inside the
// bitmap walks its row above itself; a member outside is searched against
// the whole list (in layers: every member walks).  An edge that searches:
// each member against those listed after it.
__global__ void k_delta_k4_pairs(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  if (npairs > D.pair_cap || ne == 0) return;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  for (int64_t b0 = w0 * 64; b0 < ne; b0 += ws * 64) {
    const int64_t i = b0 + l;
    int g = -1;
    int32_t d = 0;
    uint32_t u = 0, h = 0;
    bool first = false, split = false;
    if (i < ne) {
      const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
      u = (uint32_t)(K >> D.bits);
      const uint32_t v = (uint32_t)(K & idmask);
      d = D.e_dt[i];
      g = D.gid[u];
      split = k4_walked(D.e_ns[i], D.e_kw[i]);
      if (d) {
        atomicAdd(&D.dT[u], (unsigned long long)(long long)d);
        atomicAdd(&D.dT[v], (unsigned long long)(long long)d);
        first = t_move(D, D.P.off[u] + lower_bound_id(D.P.col + D.P.off[u], D.P.len[u], v), d, h);
      }
    }
    aff_append(D, first, u, h);
    add_sig_lanes(D, g, SG_T, 3 * (int64_t)d);
    add_sig_lanes(D, g, SG_PAW, -12 * (int64_t)d);
    const uint64_t sm = __ballot(split);
    if (sm && l == 0) atomicAdd(&D.bstats[BS_K4_SPLIT], (unsigned long long)__popcll(sm));
  }
  for (int64_t b0 = w0 * 64; b0 < npairs; b0 += ws * 64) {
    const int64_t i0 = wave_upper_bound(D.c4_off, ne, b0);
    const int64_t p = b0 + l;
    const bool in = p < npairs;
    const int64_t i = in ? upper_bound_from(D.c4_off, ne, i0, p) : i0;
    const int32_t j = (int32_t)(p - D.c4_off[i]), ns = D.e_ns[i];
    int32_t walk = 0, search = 0;
    if (in && j < ns) {
      if (!k4_walked(ns, D.e_kw[i])) {
        search = ns - 1 - j;
      } else {
        const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
        const uint32_t o = (uint32_t)((D.c4_side[i] & 1) ? K >> D.bits : K & idmask);
        const uint32_t e = D.slist[p], w = e & GC_ID;
        if (!k4_layers(D, i) && k4_outside(e, c4b_base(D, o))) {
          search = ns;
        } else {
          const int32_t wl = D.P.len[w];
          walk = wl - lower_bound_id(D.P.col + D.P.off[w], wl, w + 1);
        }
      }
    }
    if (in) D.pair_hlen[npairs + p] = walk;
    search_append(D, search > 0, i, ~j, search);
  }
}

// A list too short (searched pairs, affected edges): count again with more.
__global__ void k_delta_check(DeltaArgs D) {
  if (gtid() != 0) return;
  const unsigned long long n = D.dc[DC_SEARCH];
  if ((int64_t)n > 2 * D.pair_cap) {
    atomicAdd(&D.bstats[BS_RETRY], 1ull);
    atomicMax(&D.dc[DC_PAIR_NEED], (n + 1) / 2);
  }
  if ((int64_t)D.dc[DC_AFF] > D.ae_cap || D.dc[DC_AFF_FULL]) {
    atomicAdd(&D.bstats[BS_RETRY], 1ull);
    // distinct edges are fewer than the moves (and than the edges: the host)
    atomicMax(&D.dc[DC_AFF_NEED], D.dc[DC_AFF_INST] + D.dc[DC_EDGES]);
  }
}

// A searched pair: what is walked, the row searched, and what a hit needs.
struct SearchRec {
  const uint32_t* walk;   // first entry of this wave's part of the walk
  const uint32_t* row;    // the row searched
  unsigned long long K;   // key of the changed edge
  int32_t len;            // entries of the row searched
  int32_t only;           // 4-cycles: > 0 for a pair (e, b), |N(o)| of the edge; 4-cliques: member of S(e)
  int32_t j0;             // 4-cliques: member at walk[0]
  uint32_t s, o, a;       // 4-cycles: the path s - a - b - o, the walk runs over b; 4-cliques: s, o and the member a
  uint32_t base;          // 4-cliques: first id of the bitmap, 0xFFFFFFFF: every member counts
  uint32_t meta;          // fe | flags of a << 2 | (4-cycles: the row walked is N(a)) << 6 | (4-cliques) << 7
  int32_t g;
};

// The searched pairs.  Each wave takes one contiguous range of the index
// space of their walked entries (equal ranges: balanced by construction),
// 64 pairs at a time: a lane fetches one pair's record into LDS, then the
// entries of all of them are dealt over the lanes, each searching its entry
// in the other row.  Bound by the dependent loads of the searches.
__global__ __launch_bounds__(TPB) void k_delta_search(DeltaArgs D) {
  __shared__ SearchRec recs[TPB / 64][64];
  if (D.bstats[BS_RETRY]) return;
  const int64_t np = ctr(D.dc, DC_SEARCH);
  if (np == 0) return;
  const int64_t total = D.pair_off[np];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  SearchRec* rec = recs[threadIdx.x >> 6];
  const int64_t nw = gstride() >> 6;
  const int64_t per = ((total + nw - 1) / nw + 63) / 64 * 64;
  const int64_t w0 = min(total, (gtid() >> 6) * per), w1 = min(total, w0 + per);
  int64_t acc = 0, acc4 = 0;
  int cur_g = -1;
  for (int64_t p = w0 < w1 ? wave_upper_bound(D.pair_off, np, w0) : np; p < np; p += 64) {
    if (D.pair_off[p] >= w1) break;
    const int64_t pl = p + l;
    int32_t n = 0;
    if (pl < np) {
      const int64_t hb = D.pair_off[pl], c0 = max(hb, w0), c1 = min(D.pair_off[pl + 1], w1);
      if (c0 < c1) {
        n = (int32_t)(c1 - c0);
        const int64_t i = D.pair_edge[pl];
        const int32_t j = D.pair_idx[pl];
        const unsigned long long ek = D.ce[i];
        SearchRec r;
        r.K = ek & DIR_KEY_MASK;
        const uint32_t u = (uint32_t)(r.K >> D.bits), v = (uint32_t)(r.K & idmask);
        r.s = (D.c4_side[i] & 1) ? v : u;
        r.o = r.s == u ? v : u;
        r.only = 0;
        r.j0 = 0;
        r.base = 0;
        r.g = D.gid[u];
        r.meta = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
        if (j < 0) {  // 4-cliques: the members listed after ~j, or all of them
          const uint32_t* S = D.slist + D.c4_off[i];
          const uint32_t e = S[~j];
          const bool all = k4_walked(D.e_ns[i], D.e_kw[i]);
          r.a = e & GC_ID;
          r.meta |= ((e >> 28) << 2) | (1u << 7);
          r.only = ~j;
          r.j0 = (all ? 0 : ~j + 1) + (int32_t)(c0 - hb);
          r.base = all ? c4b_base(D, r.o) : 0xFFFFFFFFu;
          r.walk = S + r.j0;
          r.row = D.P.col + D.P.off[r.a];
          r.len = D.P.len[r.a];
        } else {
          uint32_t fsa;
          const int32_t sl = D.P.len[r.s];
          if (j < sl) {
            const uint32_t e = D.P.col[D.P.off[r.s] + j];
            r.a = e & GC_ID;
            fsa = nib(e);
          } else {  // a pair (e, b): the same with the ends swapped, through walked a only
            c4_out_pair(D, r.o, D.c4_low[i], j - sl, r.a, fsa);
            r.only = D.P.len[r.o];
            const uint32_t t = r.s;
            r.s = r.o;
            r.o = t;
          }
          const uint32_t* arow = D.P.col + D.P.off[r.a];
          const uint32_t* orow = D.P.col + D.P.off[r.o];
          const int32_t al = D.P.len[r.a], ol = D.P.len[r.o];
          const bool wa = al <= ol;
          r.walk = (wa ? arow : orow) + (c0 - hb);
          r.row = wa ? orow : arow;
          r.len = wa ? ol : al;
          r.meta |= (fsa << 2) | ((wa ? 1u : 0u) << 6);
        }
        rec[l] = r;
      }
    }
    const int32_t incl = wave_incl_scan32(n), tot = __shfl(incl, 63), excl = incl - n;
    wave_sync();
    for (int32_t at = 0; at < tot; at += 64) {
      const int32_t idx = at + l;
      int lo = 0, hi = 64;  // the pair of index idx: largest lane with excl <= idx
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const int mid = (lo + hi) >> 1;
        if (__shfl(excl, mid) <= idx) lo = mid; else hi = mid;
      }
      const int32_t ex = __shfl(excl, lo);
      if (idx >= tot) continue;
      const SearchRec& r = rec[lo];
      const uint32_t ew = r.walk[idx - ex], b = ew & GC_ID;
      const uint32_t* row = r.row;
      const int32_t len = r.len, x = lower_bound_id(row, len, b);
      if (x >= len) continue;
      const uint32_t er = row[x];
      if ((er & GC_ID) != b) continue;
      const unsigned long long K = r.K;
      const uint32_t fe = r.meta & 3u;
      int64_t d4 = 0, d = 0;
      if (r.meta >> 7) {  // members a and b of S(e) are joined
        const int32_t j = r.j0 + (idx - ex);
        if (r.base != 0xFFFFFFFFu && (j == r.only || (j < r.only && k4_outside(ew, r.base)))) continue;
        const uint32_t fsa = (r.meta >> 2) & 3u, foa = (r.meta >> 4) & 3u, fsb = (ew >> 28) & 3u, fob = ew >> 30;
        const uint32_t fab = nib(er);
        if ((fsa && pkey(r.s, r.a, D.bits) < K) || (foa && pkey(r.o, r.a, D.bits) < K) ||
            (fsb && pkey(r.s, b, D.bits) < K) || (fob && pkey(r.o, b, D.bits) < K) ||
            (fab && pkey(r.a, b, D.bits) < K))
          continue;
        d4 = delta_of(fe | fsa | foa | fsb | fob | fab);
      } else {
        const bool wa = (r.meta >> 6) & 1u;
        const uint32_t fsa = (r.meta >> 2) & 3u, fab = nib(wa ? ew : er), fob = nib(wa ? er : ew);
        if (b == r.s || (fsa && pkey(r.s, r.a, D.bits) < K) || (fab && pkey(r.a, b, D.bits) < K) ||
            (fob && pkey(r.o, b, D.bits) < K) || (r.only && !pair_walked(D.P.len[b], r.only)))
          continue;
        d = delta_of(fe | fsa | fab | fob);
      }
      if (r.g != cur_g) {
        if (cur_g >= 0 && acc) atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_C4)], (unsigned long long)acc);
        if (cur_g >= 0 && acc4) atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_K4)], (unsigned long long)acc4);
        acc = acc4 = 0;
        cur_g = r.g;
      }
      acc += d;
      acc4 += d4;
    }
    wave_sync();
  }
  add_sig_lanes(D, cur_g, SG_C4, acc);
  add_sig_lanes(D, cur_g, SG_K4, acc4);
}

// Walked entries per chunk of a bitmap edge: enough chunks to fill the chip
// several times over, each long enough to pay for its bitmap (four times
// |N(o)|, and a floor for the fixed cost of a chunk).
__device__ __forceinline__ int64_t c4b_chunk(int64_t total, int64_t ol) {
  const int64_t even = total / 4096;
  return max(min(max(even, (int64_t)16384), (int64_t)131072), 4 * ol);
}

// Walked entries per chunk of an edge in layers with nm members: the members
// of S(e), in no order, are read once per window.
__device__ __forceinline__ int64_t layers_chunk(const DeltaArgs& D, int64_t total, bool k4, int32_t nm, uint32_t top) {
  const int64_t nw = k4 ? ((int64_t)top + D.lay_ids - 1) / D.lay_ids : 1;
  return c4b_chunk(total, nw * nm);
}

// Chunks of the walked entries per changed edge: of its 4-cycles at i, of its
// 4-cliques at ne + i (0 past them, for the scan).  Those in layers go to a
// list of their own, whose entries are taken together with the number of
// their first chunk: one word counts entries (above DC_LAY_SHIFT) and chunks.
__global__ void k_delta_hitems(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  const bool fits = npairs <= D.pair_cap;  // else the pairs were not listed (count again)
  const int64_t total = fits ? D.pair_hoff[2 * npairs] : 0;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const C4Layers layers(D);
  for (int64_t t = gtid(); t < D.tcap; t += gstride()) {
    int32_t n = 0;
    if (t < 2 * ne && fits) {
      const bool k4 = t >= ne;
      const int64_t i = k4 ? t - ne : t, at = k4 ? npairs : 0;
      const int64_t h = D.pair_hoff[at + D.c4_off[i + 1]] - D.pair_hoff[at + D.c4_off[i]];
      if (h > 0) {
        const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
        const uint32_t o = (uint32_t)((D.c4_side[i] & 1) ? K >> D.bits : K & idmask);
        const int32_t nm = k4 ? D.e_ns[i] : D.P.len[o];
        if (k4 ? k4_layers(D, i) : layers(D.c4_side[i])) {
          const int64_t T = layers_chunk(D, total, k4, nm, c4b_top(D, o));
          const unsigned long long at =
              atomicAdd(&D.dc[DC_LAY], (1ull << DC_LAY_SHIFT) | (unsigned long long)((h + T - 1) / T));
          D.lay_list[at >> DC_LAY_SHIFT] = (int32_t)t;
          D.lay_off[at >> DC_LAY_SHIFT] = (int64_t)(at & ((1ull << DC_LAY_SHIFT) - 1ull));
        } else {
          const int64_t T = c4b_chunk(total, nm);
          n = (int32_t)((h + T - 1) / T);
        }
      }
    }
    D.tv_items[t] = n;
  }
}

// The walked entries.  Each workgroup takes chunks from a queue and holds a
// bitmap in LDS (kept while the next chunk is of the same edge and kind).
// 4-cycles of e = (s, o): the bitmap holds the b in N(o) inside the window
// whose edge (o, b) is not in the batch, the rows are those N(a) of the
// walked pairs, and a hit closes the path s - a - b - o.  4-cliques: it holds
// the members of S(e) inside the window with neither edge to e in the batch,
// the rows are those of the same members, above themselves, and a hit joins
// two members.  The waves split the chunk's entries evenly, read them with
// consecutive lanes and probe one bit per entry.  Hits on entries that are in
// the batch themselves take the general rule (rare).
// What bounds it: the rows' loads.  At scale 22 3.7 TB/s come from beyond the
// L2s (a copy reaches 4.7; one entry in ten hits the L2) and 74% of the wave
// cycles wait; the VALU is 39% busy (17 instructions per 64 entries), the LDS
// 13%.  At scale 18, where the rows stay in the caches, latency alone (79%
// waiting).  The bitmap costs little: a chunk is at least four times its
// members.  Before, rows of similar length were merged by a wave (about 35
// instructions and nine lane exchanges per 64 entries of each row), shorter
// rows probed an LDS hash table and the rest was searched: 22 ms in all for
// 2,500 updates at scale 22 (5.9e9 entries walked), 2.1 ms for 1,000 at scale
// 18 (1.2e8); now 6.4 ms and 0.6 for the searched pairs, 0.27 and 0.08.
// WORDS = 16384 (ids up to 2^19) lets two workgroups share a CU.
template <int WORDS>
__global__ __launch_bounds__(C4B_T, WORDS <= 16384 ? 8 : 4) void k_delta_bits(DeltaArgs D) {
  __shared__ uint4 bm4[WORDS / 4];
  __shared__ int64_t item_s, edge_s;
  if (D.bstats[BS_RETRY]) return;
  uint32_t* bm = (uint32_t*)bm4;
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  if (ne == 0) return;
  const int64_t nitems = D.tv_ioff[2 * ne];
  const int64_t npairs = D.c4_off[D.ce_cap];
  const int64_t total = D.pair_hoff[2 * npairs];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int32_t l = lane_id(), wv = (int32_t)(threadIdx.x >> 6);
  constexpr int32_t NW = C4B_T / 64;
  const uint32_t ids = D.c4_ids;  // <= WORDS * 32
  const uint32_t* __restrict__ col = D.P.col;
  int64_t acc[2] = {0, 0};
  int cur_g = -1;
  int64_t cur_t = -1;
  while (true) {
    __syncthreads();
    if (wv == 0) {
      int64_t it0 = 0;
      if (l == 0) it0 = (int64_t)atomicAdd(&D.dc[DC_QH], 1ull);
      it0 = __shfl(it0, 0);
      const int64_t t0 = it0 < nitems ? wave_upper_bound(D.tv_ioff, 2 * ne, it0) : 0;
      if (l == 0) { item_s = it0; edge_s = t0; }
    }
    __syncthreads();
    const int64_t it = item_s, t = edge_s;
    if (it >= nitems) break;
    const bool k4 = t >= ne;
    const int64_t i = k4 ? t - ne : t;
    const unsigned long long ek = D.ce[i];
    const unsigned long long K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const uint32_t s = (D.c4_side[i] & 1) ? v : u, o = s == u ? v : u;
    const int g = D.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) { add_sig(D, cur_g, SG_C4, acc[0]); add_sig(D, cur_g, SG_K4, acc[1]); }
      acc[0] = acc[1] = 0;
      cur_g = g;
    }
    const uint32_t base = c4b_base(D, o);
    const int64_t p0 = D.c4_off[i], so = D.P.off[s];
    // the members: N(o), or S(e) with the flags of both edges
    const uint32_t* mem = k4 ? D.slist + p0 : col + D.P.off[o];
    const int32_t nm = k4 ? D.e_ns[i] : D.P.len[o];  // > 0
    if (t != cur_t) {
      for (int32_t k = (int32_t)threadIdx.x; k < WORDS / 4; k += C4B_T) bm4[k] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
      for (int32_t k0 = wv * 256; k0 < nm; k0 += 4 * C4B_T) {  // four loads in flight per lane
        uint32_t y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = mem[min(k0 + 64 * q + l, nm - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t x = (y[q] & GC_ID) - base;
          if (!(y[q] & GC_FLAGS) && x < ids) atomicOr(&bm[x >> 5], 1u << (x & 31u));
        }
      }
      cur_t = t;
      __syncthreads();
    }
    // the chunk: entries [r0, r1) of the walked index space, this wave's
    // piece of them; 64 rows at a time, a row's part of the piece per lane
    const int64_t* __restrict__ hoff = D.pair_hoff + (k4 ? npairs : 0) + p0;
    const int64_t nr = D.c4_off[i + 1] - p0;
    const int64_t T = c4b_chunk(total, nm);
    const int64_t r0 = hoff[0] + (it - D.tv_ioff[t]) * T, r1 = min(hoff[nr], r0 + T);
    const int64_t per = (r1 - r0 + NW - 1) / NW;
    const int64_t w0 = min(r1, r0 + wv * per), w1 = min(r1, w0 + per);
    uint32_t clean = 0;  // hits with no other edge of the structure in the batch
    int64_t rest = 0;
    if (w0 < w1) {
      for (int64_t p = wave_upper_bound(hoff, nr, w0); p < nr; p += 64) {
        if (hoff[p] >= w1) break;
        const int64_t pl = p + l;
        int64_t sb = 0;
        int32_t sn = 0;
        uint32_t ea = 0;
        if (pl < nr) {
          const int64_t hb = hoff[pl], he = hoff[pl + 1];
          const int64_t c0 = max(hb, w0), c1 = min(he, w1);
          if (c0 < c1) {
            ea = k4 ? mem[pl] : col[so + pl];
            const uint32_t a = ea & GC_ID;
            sb = D.P.off[a] + (k4 ? D.P.len[a] - (he - hb) : 0) + (c0 - hb);
            sn = (int32_t)(c1 - c0);
          }
        }
        wave_rows(col, sb, sn, ea, [&](uint32_t ea_, uint32_t y) {
          const uint32_t x = (y & GC_ID) - base;
          uint32_t hit = 0;
          if (x < ids) hit = (bm[x >> 5] >> (x & 31u)) & 1u;
          if (hit && ((ea_ | y) & GC_FLAGS)) {  // (s, a) or (a, b) in the batch
            const uint32_t a = ea_ & GC_ID, b = y & GC_ID, fsa = nib(ea_), fab = nib(y);
            hit = 0;
            if (!(fsa && pkey(s, a, D.bits) < K) && !(fab && pkey(a, b, D.bits) < K)) rest += delta_of(fe | fsa | fab);
          }
          clean += hit;
        });
      }
    }
    acc[k4 ? 1 : 0] += (int64_t)clean * delta_of(fe) + rest;
  }
  if (cur_g >= 0) { add_sig(D, cur_g, SG_C4, acc[0]); add_sig(D, cur_g, SG_K4, acc[1]); }
}

// The walked entries of the edges in layers: as above, but N(o) or S(e) is
// taken in windows of ids from its largest member downwards (those without a
// member skipped), and every member gets a bit, with a second bit where one
// of its edges to the changed pair is in the batch, so that nothing is left
// to searches.  A piece of a row is cut to the window by two searches; an entry is read in one
// window only.  Members in the batch are looked up again when they are hit.
// Bound like k_delta_bits; per window a chunk also pays for clearing the
// window's words and for three barriers.
__global__ __launch_bounds__(C4B_T, 4) void k_delta_layers(DeltaArgs D) {
  __shared__ uint32_t bm[C4B_LARGE / 2];  // members
  __shared__ uint32_t bf[C4B_LARGE / 2];  // those with an edge in the batch
  __shared__ int64_t item_s, entry_s;
  __shared__ int32_t next_s;
  if (D.bstats[BS_RETRY]) return;
  const unsigned long long lay = D.dc[DC_LAY];
  const int64_t nent = (int64_t)(lay >> DC_LAY_SHIFT), nitems = (int64_t)(lay & ((1ull << DC_LAY_SHIFT) - 1ull));
  if (nent == 0) return;
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  const int64_t total = D.pair_hoff[2 * npairs];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int32_t l = lane_id(), wv = (int32_t)(threadIdx.x >> 6);
  constexpr int32_t NW = C4B_T / 64;
  const uint32_t* __restrict__ col = D.P.col;
  int64_t acc[2] = {0, 0};
  int cur_g = -1;
  while (true) {
    __syncthreads();
    if (wv == 0) {
      int64_t it0 = 0;
      if (l == 0) it0 = (int64_t)atomicAdd(&D.dc[DC_QL], 1ull);
      it0 = __shfl(it0, 0);
      const int64_t q0 = it0 < nitems ? wave_upper_bound(D.lay_off, nent, it0) : 0;
      if (l == 0) { item_s = it0; entry_s = q0; }
    }
    __syncthreads();
    const int64_t it = item_s, q = entry_s;
    if (it >= nitems) break;
    const int64_t t = D.lay_list[q];
    const bool k4 = t >= ne;
    const int64_t i = k4 ? t - ne : t;
    const unsigned long long ek = D.ce[i];
    const unsigned long long K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const uint32_t s = (D.c4_side[i] & 1) ? v : u, o = s == u ? v : u;
    const int g = D.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) { add_sig(D, cur_g, SG_C4, acc[0]); add_sig(D, cur_g, SG_K4, acc[1]); }
      acc[0] = acc[1] = 0;
      cur_g = g;
    }
    const int64_t p0 = D.c4_off[i], so = D.P.off[s], oo = D.P.off[o];
    const int32_t sl = D.P.len[s], ol = D.P.len[o];
    const uint32_t* mem = k4 ? D.slist + p0 : col + oo;
    const int32_t nm = k4 ? D.e_ns[i] : ol;  // > 0
    const uint32_t top0 = c4b_top(D, o);
    const int64_t* __restrict__ hoff = D.pair_hoff + (k4 ? npairs : 0) + p0;
    const int64_t nr = D.c4_off[i + 1] - p0;
    const int64_t T = layers_chunk(D, total, k4, nm, top0);
    const int64_t r0 = hoff[0] + (it - D.lay_off[q]) * T, r1 = min(hoff[nr], r0 + T);
    const int64_t per = (r1 - r0 + NW - 1) / NW;
    const int64_t w0 = min(r1, r0 + wv * per), w1 = min(r1, w0 + per);
    int64_t clean = 0, rest = 0;
    int32_t mhi = nm;  // members not taken yet (N(o): sorted)
    for (uint32_t top = top0;;) {
      const uint32_t base = top > D.lay_ids ? top - D.lay_ids : 0u, wsz = top - base;
      const int32_t words = (int32_t)((wsz + 31u) >> 5);  // <= C4B_LARGE / 2
      __syncthreads();  // the window before is done with
      for (int32_t k = (int32_t)threadIdx.x; k < words; k += C4B_T) { bm[k] = 0u; bf[k] = 0u; }
      if (threadIdx.x == 0) next_s = -1;
      __syncthreads();
      auto put = [&](uint32_t y) {
        const uint32_t x = (y & GC_ID) - base;
        if (x >= wsz || (y & GC_ID) == s) return;
        atomicOr(&bm[x >> 5], 1u << (x & 31u));
        if (y & GC_FLAGS) atomicOr(&bf[x >> 5], 1u << (x & 31u));
      };
      int32_t next = -1;  // largest member below the window
      if (k4) {
        for (int32_t k = (int32_t)threadIdx.x; k < nm; k += C4B_T) {
          const uint32_t y = mem[k];
          put(y);
          if ((y & GC_ID) < base) next = max(next, (int32_t)(y & GC_ID));
        }
        next = wave_max32(next);
        if (l == 0 && next >= 0) atomicMax(&next_s, next);
      } else {
        const int32_t mlo = base ? lower_bound_id(mem, mhi, base) : 0;
        for (int32_t k = mlo + (int32_t)threadIdx.x; k < mhi; k += C4B_T) put(mem[k]);
        if (mlo) next = (int32_t)(mem[mlo - 1] & GC_ID);
        mhi = mlo;
      }
      __syncthreads();
      if (k4) next = next_s;
      if (w0 < w1) {
        for (int64_t p = wave_upper_bound(hoff, nr, w0); p < nr; p += 64) {
          if (hoff[p] >= w1) break;
          const int64_t pl = p + l;
          int64_t sb = 0;
          int32_t sn = 0;
          uint32_t ea = 0;
          if (pl < nr) {
            const int64_t hb = hoff[pl], he = hoff[pl + 1];
            const int64_t c0 = max(hb, w0), c1 = min(he, w1);
            if (c0 < c1) {
              ea = k4 ? mem[pl] : col[so + pl];
              const uint32_t a = ea & GC_ID;
              sb = D.P.off[a] + (k4 ? D.P.len[a] - (he - hb) : 0) + (c0 - hb);
              sn = (int32_t)(c1 - c0);
              if (top < top0) sn = lower_bound_id(col + sb, sn, top);
              if (base) {
                const int32_t b0 = lower_bound_id(col + sb, sn, base);
                sb += b0;
                sn -= b0;
              }
            }
          }
          wave_rows(col, sb, sn, ea, [&](uint32_t ea_, uint32_t y) {
            const uint32_t b = y & GC_ID, x = b - base;
            if (x >= wsz || !((bm[x >> 5] >> (x & 31u)) & 1u)) return;
            const bool fb = (bf[x >> 5] >> (x & 31u)) & 1u;
            if (!fb && !((ea_ | y) & GC_FLAGS)) { ++clean; return; }
            const uint32_t a = ea_ & GC_ID, fsa = (ea_ >> 28) & 3u, foa = ea_ >> 30, fab = nib(y);
            uint32_t fsb = 0, fob = 0;
            if (fb) {
              fob = nib(col[oo + lower_bound_id(col + oo, ol, b)]);
              if (k4) fsb = nib(col[so + lower_bound_id(col + so, sl, b)]);
            }
            if ((fsa && pkey(s, a, D.bits) < K) || (foa && pkey(o, a, D.bits) < K) ||
                (fsb && pkey(s, b, D.bits) < K) || (fob && pkey(o, b, D.bits) < K) ||
                (fab && pkey(a, b, D.bits) < K))
              return;
            rest += delta_of(fe | fsa | foa | fsb | fob | fab);
          });
        }
      }
      if (next < 0) break;
      top = (uint32_t)next + 1u;
    }
    acc[k4 ? 1 : 0] += clean * delta_of(fe) + rest;
  }
  if (cur_g >= 0) { add_sig(D, cur_g, SG_C4, acc[0]); add_sig(D, cur_g, SG_K4, acc[1]); }
}

// ---------------------------------------------- triangles, diamonds, paws
// The affected edges take their new t (their slots of the table are cleared),
// the vertices their new T: every vertex whose T moved is touched or the
// listed end of an affected edge.  Runs only when no list was short.
__global__ void k_delta_t(DeltaArgs D) {
  if (D.bstats[BS_RETRY]) return;
  const int64_t n = ctr(D.dc, DC_AFF), nt = ctr(D.c, C_TOUCH);
  int64_t dia = 0, paw = 0;
  int cur_g = -1;
  auto graph = [&](uint32_t x) {
    const int g = D.gid[x];
    if (g == cur_g) return;
    if (cur_g >= 0) {
      if (dia) atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_DIA)], (unsigned long long)dia);
      if (paw) atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_PAW)], (unsigned long long)paw);
    }
    dia = paw = 0;
    cur_g = g;
  };
  for (int64_t q = gtid(); q < n; q += gstride()) {
    const unsigned long long e = D.hl[q];
    const uint32_t h = (uint32_t)e, x = (uint32_t)(e >> 32);
    graph(x);
    const int64_t pos = (int64_t)D.hk[h] - 1;
    const int64_t d = D.hd[h], t = D.P.tt[pos];
    D.hk[h] = 0ull;
    D.hd[h] = 0;
    D.P.tt[pos] = (uint32_t)(t + d);
    dia += c2(t + d) - c2(t);
    if (!D.mark[x]) {
      const long long dt = (long long)atomicExch(&D.dT[x], 0ull);
      if (dt) {
        atomicAdd((unsigned long long*)&D.Tv[x], (unsigned long long)dt);
        paw += 2 * (int64_t)D.P.len[x] * dt;
      }
    }
  }
  for (int64_t k = gtid(); k < nt; k += gstride()) {
    const uint32_t x = (uint32_t)D.touched[k];
    graph(x);
    const int64_t db = D.dd[2 * (int64_t)x], da = D.dd[2 * (int64_t)x + 1];
    const int64_t dt = (long long)D.dT[x], T = D.Tv[x];
    D.dT[x] = 0ull;
    D.Tv[x] = T + dt;
    paw += 2 * (da * (T + dt) - db * T);
  }
  add_sig_lanes(D, cur_g, SG_DIA, dia);
  add_sig_lanes(D, cur_g, SG_PAW, paw);
}

// ------------------------------------------------ T(v) in the region path
// After the triangle kernels of a region (or whole-graph) pass, t holds the
// triangles of every upper entry (id order) of the region per version.  A
// changed triangle lies inside the region, so the resident t of an edge moves
// by the change of its t; and it sits on two edges at v, so T(v) moves by
// half the change of t summed over the edges at v: each upper entry hands its
// change to both ends, then each region vertex takes its half once.
//
// A hub is the larger end of very many edges: per workgroup the changes at
// the larger ends first meet in an LDS table of the ids it meets first (the
// rest go to memory), those at the row's own vertex in the wave.  With an
// atomic per end and entry the hubs' words queued (0.37 ms at scale 18).
constexpr int TVC = 2048;

template <int NV>
__global__ __launch_bounds__(TPB) void k_tv_entries(PoolDev P, RegionDev R, const int32_t* __restrict__ level,
                                                    int32_t radius, const unsigned long long* c,
                                                    unsigned long long* __restrict__ dT,
                                                    const unsigned long long* bstats) {
  __shared__ int32_t tag[TVC];
  __shared__ unsigned long long val[TVC];
  if (bstats[BS_RETRY]) return;
  for (int k = threadIdx.x; k < TVC; k += TPB) { tag[k] = -1; val[k] = 0ull; }
  __syncthreads();
  const int64_t ne = ctr(c, C_ER);
  const int l = lane_id();
  for (int64_t b0 = gtid() - l; b0 < ne; b0 += gstride()) {
    const int64_t p = b0 + l;
    int32_t v = -1;
    uint32_t w = 0;
    int64_t d = 0;
    if (p < ne) {
      w = R.rcol[p] & GC_ID;
      v = R.rrow[p];
      if ((int64_t)w > (int64_t)v) {
        if constexpr (NV == 2) {
          d = R.td[p];
        } else {
          // t_x = t[p] + field x of tp[2p] (x = 0, 1) and tp[2p + 1] (x = 2, 3)
          d = (int64_t)(R.tp[2 * p + 1] >> 32) - (int64_t)(R.tp[2 * p] & 0xFFFFFFFFull);
        }
      }
    }
    if (!__ballot(d != 0)) continue;
    // own vertex: the lanes of one row are consecutive
    const int32_t before = __shfl_up(v, 1), after = __shfl_down(v, 1);
    const uint64_t heads = __ballot(l == 0 || before != v);
    const int head = 63 - __clzll((long long)(heads & (lanemask_lt() | (1ull << l))));
    const int64_t incl = wave_incl_scan64(d);
    const int64_t sum = incl - __shfl(incl - d, head);
    if (v >= 0 && sum && (l == 63 || after != v)) atomicAdd(&dT[v], (unsigned long long)sum);
    if (!d) continue;
    const uint32_t h = (w * 2654435761u) >> 21;
    int32_t k = tag[h];
    if (k == -1) {
      k = atomicCAS(&tag[h], -1, (int32_t)w);
      if (k == -1) k = (int32_t)w;
    }
    if (k == (int32_t)w) atomicAdd(&val[h], (unsigned long long)d);
    else atomicAdd(&dT[w], (unsigned long long)d);
    // rows inside the radius are whole in the region, the outermost ones are not
    int64_t at = p - R.roff[v];
    if (radius >= 0 && level[v] >= radius) at = lower_bound_id(P.col + P.off[v], P.len[v], w);
    P.tt[P.off[v] + at] += (uint32_t)d;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < TVC; k += TPB)
    if (val[k]) atomicAdd(&dT[tag[k]], val[k]);
}

__global__ void k_tv_apply(const int32_t* __restrict__ rlist, const unsigned long long* c,
                           unsigned long long* __restrict__ dT, long long* __restrict__ Tv,
                           unsigned long long* bstats) {
  if (bstats[BS_RETRY]) return;
  const int64_t nr = ctr(c, C_RLIST);
  for (int64_t i = gtid(); i < nr; i += gstride()) {
    const int32_t v = rlist[i];
    const long long d2 = (long long)atomicExch(&dT[v], 0ull);
    if (d2) {
      if (d2 & 1) atomicAdd(&bstats[BS_ERR], 1ull);
      Tv[v] += d2 / 2;
    }
  }
}

// ---------------------------------------------------------- launchers
void launch_delta(const DeltaArgs& D_, hipStream_t s) {
  DeltaArgs D = D_;
  const bool small_bits = D.N <= C4B_SMALL * 32;
  const uint32_t ids = (small_bits ? C4B_SMALL : C4B_LARGE) * 32;
  if (D.c4_ids == 0 || D.c4_ids > ids) D.c4_ids = ids;
  // two bits per id: half as many ids per window
  D.lay_ids = std::min<uint32_t>(D.c4_ids, C4B_LARGE * 16);
  hipLaunchKernelGGL(k_delta_edges, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_titems, dim3(1024), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_vertex, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_s2, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_plan_items, dim3(1024), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_c4_plan, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_plan_fin, dim3(256), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.c4_nch, D.c4_off, D.ce_cap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_pairs, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_k4_pairs, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_check, dim3(1), dim3(64), 0, s, D);
  // every walked and every searched pair below their counts gets a length,
  // and only offsets up to the counts are read: no clearing, scans up to them
  exclusive_scan_i32_to_i64_count(D.pair_len, D.pair_off, 2 * D.pair_cap, (const int64_t*)(D.dc + DC_SEARCH), D.scan_tmp, s);
  exclusive_scan_i32_to_i64_count(D.pair_hlen, D.pair_hoff, 2 * D.pair_cap, (const int64_t*)(D.dc + DC_WALK), D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_hitems, dim3(256), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  // every kernel that can find a buffer too small (and raise BS_RETRY) ran
  // before the first one that moves the kept triangle counts
  hipLaunchKernelGGL(k_delta_t, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_search, dim3(4096), dim3(TPB), 0, s, D);
  if (small_bits)
    hipLaunchKernelGGL(k_delta_bits<C4B_SMALL>, dim3(512), dim3(C4B_T), 0, s, D);
  else
    hipLaunchKernelGGL(k_delta_bits<C4B_LARGE>, dim3(256), dim3(C4B_T), 0, s, D);
  // an edge's members outside its bitmap: flagged ones, at most one per
  // changed pair (and two ends for S(e)), and ids below the window
  if (D.ce_cap > C4B_OUT || D.N > (int64_t)D.c4_ids || D.c4_out > 0)
    hipLaunchKernelGGL(k_delta_layers, dim3(256), dim3(C4B_T), 0, s, D);
}

void launch_tv_region(int nv, const PoolDev& P, const RegionDev& R, const int32_t* level, int32_t radius,
                      const int32_t* rlist, const unsigned long long* c, unsigned long long* dT, long long* Tv,
                      unsigned long long* bstats, hipStream_t s) {
  if (nv == 2)
    hipLaunchKernelGGL(k_tv_entries<2>, dim3(1024), dim3(TPB), 0, s, P, R, level, radius, c, dT,
                       (const unsigned long long*)bstats);
  else
    hipLaunchKernelGGL(k_tv_entries<4>, dim3(1024), dim3(TPB), 0, s, P, R, level, radius, c, dT,
                       (const unsigned long long*)bstats);
  hipLaunchKernelGGL(k_tv_apply, dim3(2048), dim3(TPB), 0, s, rlist, c, dT, Tv, bstats);
}
