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
// kernel applies them unchanged; the per-vertex triangle counts Tv move to
// the graph after the batch.
//
// A structure (triangle, 4-clique, 4-cycle) that holds several changed pairs
// is counted once, from the changed pair with the smallest key (min << bits |
// max); it adds [present after] - [present before], decided by the OR of its
// entries' flags.  Per term:
//   S1, W, D1   touched vertices (their degrees before and after);
//   S2          edges at touched vertices, each once;
//   T, DIA      the affected edges -- changed edges and the other two edges
//               of every triangle on a changed edge (deduplicated): t before
//               and after by row intersection, sum of [p] t and [p] C(t, 2);
//   PAW         sum_e t_e (d_u + d_v - 4): affected edges directly; for the
//               other edges at a vertex x whose degree changed, their t sum
//               is 2 T(x) minus the affected ones (T(x) kept per vertex);
//   K4          per changed edge e = (u, v): pairs {w, x} of common
//               neighbours S(e) joined by an edge;
//   C4          per changed edge: paths s - a - b - o closing the cycle with
//               e = (s, o), from the common ids of N(a) and N(o) for each
//               pair (s, a): the rows N(a) walked against an LDS bitmap of
//               N(o), or, where that costs more (little to walk for the edge,
//               or an N(a) far longer than N(o)), the shorter row walked and
//               searched in the other.
#include "gc_kernels.h"

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

// Position of id in row r (sorted, flags ignored) or -1.
__device__ __forceinline__ int64_t find_in_row(const PoolDev& P, uint32_t r, uint32_t id) {
  const uint32_t* row = P.col + P.off[r];
  const int32_t n = P.len[r];
  const int32_t p = lower_bound_id(row, n, id);
  return (p < n && (row[p] & GC_ID) == id) ? P.off[r] + p : -1;
}

// The common ids of two id-sorted rows, the wave together: each step loads
// the next 64 entries of both rows (one per lane), finds each a entry in the
// b window by a search over the lanes, and consumes the window with the
// smaller last id together with the entries of the other window up to that
// id.  No common id is ever consumed on one side only, so each is met once,
// in the step that consumes it, with both of its entries in the windows.
// f(entry of a, entry of b) per common id, on the lane holding the a entry.
// The step bookkeeping is wave-uniform (scalar registers and branches): lanes
// past a row's end load its last entry again instead of branching, the
// windows' last ids are read from lane 63, and the lane exchanges address
// ds_bpermute by byte (lane * 4) directly.
__device__ __forceinline__ uint32_t bperm4(uint32_t byte_lane, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute((int)byte_lane, (int)v);
}

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  return (int64_t)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32)) << 32) |
                   __builtin_amdgcn_readfirstlane((uint32_t)x));
}

// Rows a = col + oa (na entries) and b = col + ob (nb entries), the same on
// every lane of the wave.
template <class F>
__device__ __forceinline__ void wave_window_common(const uint32_t* __restrict__ col, int64_t oa_, int32_t na_,
                                                   int64_t ob_, int32_t nb_, F f) {
  const int64_t oa = uniform64(oa_), ob = uniform64(ob_);
  const int32_t na = __builtin_amdgcn_readfirstlane(na_), nb = __builtin_amdgcn_readfirstlane(nb_);
  const int32_t l = lane_id();
  int32_t i0 = 0, j0 = 0;
  while (i0 < na && j0 < nb) {
    const int32_t ra = na - i0, rb = nb - j0;  // > 0
    const bool va = l < ra, vb = l < rb;
    const uint32_t* aw = col + (oa + i0);
    const uint32_t* bw = col + (ob + j0);
    const uint32_t ea = aw[(uint32_t)min(l, ra - 1)], eb = bw[(uint32_t)min(l, rb - 1)];
    const uint32_t ida = ea & GC_ID, idb = eb & GC_ID;
    // last ids of the windows (lane 63 holds the last entry of a short one)
    const uint32_t amax = __builtin_amdgcn_readlane(ida, 63), bmax = __builtin_amdgcn_readlane(idb, 63);
    const uint32_t ia = va ? ida : 0xFFFFFFFFu, ib = vb ? idb : 0xFFFFFFFFu;
    // 4 x (number of window ids of b below ia): the window ascends and is
    // padded above; a count of 64 reads lane 0 (ds_bpermute wraps), whose
    // id is below ia, so it never matches
    uint32_t lo4 = 0;
#pragma unroll
    for (uint32_t sp = 32; sp >= 1; sp >>= 1) lo4 = bperm4(lo4 + 4 * (sp - 1), ib) < ia ? lo4 + 4 * sp : lo4;
    const uint32_t ibp = bperm4(lo4, ib), ebp = bperm4(lo4, eb);
    if (va && ibp == ia) f(ea, ebp);
    if (amax <= bmax) {
      j0 += (int32_t)__popcll(__ballot(ib <= amax));
      i0 += 64;
    } else {
      i0 += (int32_t)__popcll(__ballot(ia <= bmax));
      j0 += 64;
    }
  }
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

// Work items for the waves of a grid: each wave's first item is its own
// index (no atomic, so a small input costs no contention: waves without an
// item leave at once), and a wave that finished one takes the next from a
// shared counter counting on from the grid's wave count, so that waves which
// met light items take more (a fixed share per wave leaves the kernel
// waiting for the wave that drew the heaviest ones).  One item at a time:
// the items in flight stay a moving window of consecutive ones, whose rows
// (one changed edge's opposite row, one vertex's row) the waves share in L2
// (chunks of 16 spread the waves over the item space: both kernels slower by
// half and more).  Returns the same item on every lane.
__device__ __forceinline__ int64_t wave_next(unsigned long long* ctr_, int64_t nwaves) {
  unsigned long long c = 0;
  if (lane_id() == 0) c = atomicAdd(ctr_, 1ull);
  return nwaves + (int64_t)__shfl(c, 0);
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
    if ((int64_t)p < D.ce_cap) D.ce[p] = key | ((unsigned long long)(i < na ? 1u : 2u) << DIR_MASK_SHIFT);
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

// the 3-star, wedge and degree-sum terms of each touched vertex
__global__ void k_delta_vertex_fin(DeltaArgs D) {
  const int64_t nt = ctr(D.c, C_TOUCH);
  for (int64_t t = gtid(); t < nt; t += gstride()) {
    const uint32_t x = (uint32_t)D.touched[t];
    const int64_t db = D.dd[2 * (int64_t)x], da = D.dd[2 * (int64_t)x + 1];
    const int g = D.gid[x];
    const int64_t s1 = c3(da) - c3(db), w2 = c2(da) - c2(db), d1 = da - db;
    if (s1) atomicAdd(&D.sig[SIG_IDX(g, 1, SG_S1)], (unsigned long long)s1);
    if (w2) atomicAdd(&D.sig[SIG_IDX(g, 1, SG_W)], (unsigned long long)w2);
    if (d1) atomicAdd(&D.sig[SIG_IDX(g, 1, SG_D1)], (unsigned long long)d1);
  }
}

// S2 = sum_e (d_u - 1)(d_v - 1) changes only on edges at a touched vertex;
// an edge between two touched vertices is taken at the smaller id.
__global__ void k_delta_s2(DeltaArgs D) {
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
    const int64_t dbx = D.dd[2 * (int64_t)x] - 1, dax = D.dd[2 * (int64_t)x + 1] - 1;
    int64_t acc = 0;
    for (int32_t q = k0 + l; q < k1; q += 64) {
      const uint32_t e = row[q], y = e & GC_ID, f = nib(e);
      if (D.mark[y] && y < x) continue;
      if ((f & 2u) == 0) acc += dax * (deg_of(D, y, 1) - 1);
      if ((f & 1u) == 0) acc -= dbx * (deg_of(D, y, 0) - 1);
    }
    add_sig(D, D.gid[x], SG_S2, acc);
  }
}

// ---------------------------------------------- triangles and 4-cliques
// One workgroup per changed edge e = (u, v) at a time (a queue over the
// changed edges).  S(e) = N(u) & N(v) in the union view: the shorter row's
// entries are searched in the longer row.  Each w in S(e) gives the affected
// edges (u, w), (v, w) and is marked in the workgroup's dense slot with the
// nibbles of (u, w) and (v, w).  Then every pair {w, x} of S(e) joined by an
// edge closes a 4-clique {u, v, w, x}: for each w, the shorter of its row
// above w and S(e) is tested against the other.
// 4-cliques {u, v, w, x} through the changed edge (u, v) (key K, nibble fe)
// for the common neighbours w = S[i], i in [i0, i1) (one wave per w, the
// workgroup's waves in turn): x runs over S(e) above w, joined to w by an
// edge; S(e) is marked in `mark` (a byte per vertex: bit 7, the nibble of
// (u, x) in bits 0-1 and of (v, x) in bits 2-3) and listed in S (ids, flag
// bits above them ignored).  Returns this lane's share of the sum.
__device__ int64_t k4_through(const DeltaArgs& D, const uint8_t* mark, const uint32_t* S, int32_t ns, int32_t i0,
                              int32_t i1, uint32_t u, uint32_t v, unsigned long long K, uint32_t fe) {
  int64_t k4 = 0;
  for (int32_t i = i0 + (int32_t)(threadIdx.x >> 6); i < i1; i += (int32_t)(blockDim.x >> 6)) {
    const uint32_t w = S[i] & GC_ID;
    const uint32_t mw = mark[w];
    const uint32_t* wrow = D.P.col + D.P.off[w];
    const int32_t wl = D.P.len[w];
    const int32_t above = lower_bound_id(wrow, wl, w + 1);
    const int32_t nab = wl - above;
    int64_t acc = 0;
    auto clique = [&](uint32_t x, uint32_t fwx, uint32_t mx) {
      const uint32_t fuw = mw & 3u, fvw = (mw >> 2) & 3u;
      const uint32_t fux = mx & 3u, fvx = (mx >> 2) & 3u;
      // counted from the changed edge of smallest key only
      if ((fuw && pkey(u, w, D.bits) < K) || (fvw && pkey(v, w, D.bits) < K) || (fux && pkey(u, x, D.bits) < K) ||
          (fvx && pkey(v, x, D.bits) < K) || (fwx && pkey(w, x, D.bits) < K))
        return;
      acc += delta_of(fe | fuw | fvw | fux | fvx | fwx);
    };
    if (nab <= ns) {
      for (int32_t k = above + lane_id(); k < wl; k += 64) {
        const uint32_t ex = wrow[k], x = ex & GC_ID;
        const uint32_t mx = mark[x];
        if (mx) clique(x, nib(ex), mx);
      }
    } else {
      for (int32_t j = lane_id(); j < ns; j += 64) {
        const uint32_t x = S[j] & GC_ID;
        if (x <= w) continue;
        const int32_t p = lower_bound_id(wrow, wl, x);
        if (p < wl && (wrow[p] & GC_ID) == x) clique(x, nib(wrow[p]), mark[x]);
      }
    }
    k4 += acc;
  }
  return k4;
}

__global__ __launch_bounds__(TPB) void k_delta_tri(DeltaArgs D) {
  __shared__ int64_t item_s, split_s;
  __shared__ int32_t ns_s;
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  // marks of S(e), one byte per vertex (bit 7 set, the nibbles of (u, w) and
  // (v, w) in bits 0-1 and 2-3) in the first N bytes of the workgroup's
  // slot (denser than a word per vertex for the random reads of the
  // 4-clique step); all zero again when the kernel ends
  uint8_t* mark = (uint8_t*)(D.slot_mark + (int64_t)blockIdx.x * D.N);
  uint32_t* S = D.slot_list + (int64_t)blockIdx.x * D.slot_cap;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  int64_t k4acc = 0;
  int cur_g = -1;
  while (true) {
    __syncthreads();
    if (threadIdx.x == 0) { item_s = (int64_t)atomicAdd(&D.dc[DC_QTRI], 1ull); ns_s = 0; }
    __syncthreads();
    const int64_t it = item_s;
    if (it >= ne) break;
    const unsigned long long ek = D.ce[it];
    const unsigned long long K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const int g = D.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) add_sig(D, cur_g, SG_K4, k4acc);
      k4acc = 0;
      cur_g = g;
    }
    const uint32_t s = D.P.len[u] <= D.P.len[v] ? u : v, o = s == u ? v : u;
    const uint32_t* srow = D.P.col + D.P.off[s];
    const int32_t sl = D.P.len[s];
    if (sl > D.slot_cap) {  // more common neighbours possible than the slot holds: count again with more
      if (threadIdx.x == 0) { atomicAdd(&D.bstats[BS_RETRY], 1ull); atomicMax(&D.dc[DC_SLOT_NEED], (unsigned long long)sl); }
      continue;
    }
    for (int32_t k = threadIdx.x; k < sl; k += blockDim.x) {
      const uint32_t es = srow[k], w = es & GC_ID;
      if (w == o) continue;
      const int64_t p = find_in_row(D.P, o, w);
      if (p < 0) continue;
      const uint32_t eo = D.P.col[p];
      const uint32_t fu = nib(s == u ? es : eo), fv = nib(s == u ? eo : es);
      mark[w] = (uint8_t)(0x80u | fu | (fv << 2));
      S[atomicAdd(&ns_s, 1)] = w;
      // affected edges (u, w), (v, w)
      const unsigned long long q = atomicAdd(&D.dc[DC_AFF], 2ull);
      if ((int64_t)q + 1 < D.ae_cap) { D.ae[q] = pkey(u, w, D.bits); D.ae[q + 1] = pkey(v, w, D.bits); }
    }
    __syncthreads();
    const int32_t ns = ns_s;
    // an edge with many common neighbours hands its 4-cliques to
    // k_delta_k4_split in chunks (when the fixed buffers hold it)
    if (ns >= K4_HEAVY_MIN) {
      if (threadIdx.x == 0) {
        const int32_t nch = (ns + K4_CHUNK - 1) / K4_CHUNK;
        int64_t off = (int64_t)atomicAdd(&D.dc[DC_HS], (unsigned long long)ns);
        bool ok = off + ns <= K4_HS_CAP;
        int64_t first = -1;
        if (ok) {
          first = (int64_t)atomicAdd(&D.dc[DC_HITEMS], (unsigned long long)nch);
          if (first + nch > K4_IT_CAP) {
            for (int64_t t = first; t < min(first + nch, K4_IT_CAP); ++t) D.k4_item[2 * t] = -1;
            ok = false;
          }
        }
        if (ok) {
          const int64_t h = (int64_t)atomicAdd(&D.dc[DC_HEAVY], 1ull);
          if (h >= K4_HE_CAP) {
            for (int64_t t = first; t < first + nch; ++t) D.k4_item[2 * t] = -1;
            ok = false;
          } else {
            D.k4_edge[3 * h] = it;
            D.k4_edge[3 * h + 1] = off;
            D.k4_edge[3 * h + 2] = ns;
            for (int32_t c = 0; c < nch; ++c) {
              D.k4_item[2 * (first + c)] = (int32_t)h;
              D.k4_item[2 * (first + c) + 1] = c;
            }
            atomicAdd(&D.bstats[BS_K4_SPLIT], 1ull);
          }
        }
        split_s = ok ? off : -1;
      }
      __syncthreads();
    } else if (threadIdx.x == 0) {
      split_s = -1;
    }
    __syncthreads();
    const int64_t off = split_s;
    if (off >= 0) {
      for (int32_t i = threadIdx.x; i < ns; i += blockDim.x) {
        const uint32_t w = S[i], m = mark[w];
        D.k4_s[off + i] = w | ((m & 3u) << 28) | (((m >> 2) & 3u) << 30);
      }
    } else {
      k4acc += k4_through(D, mark, S, ns, 0, ns, u, v, K, fe);
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < ns; i += blockDim.x) mark[S[i]] = 0;
  }
  if (cur_g >= 0) add_sig(D, cur_g, SG_K4, k4acc);
}

// The 4-cliques of the edges k_delta_tri split: each workgroup takes chunks
// of K4_CHUNK common neighbours from a queue, marks the edge's common
// neighbours in its own slot (kept while the next chunk is of the same
// edge) and counts the chunk's 4-cliques; the slot is clear on return.
__global__ __launch_bounds__(TPB) void k_delta_k4_split(DeltaArgs D) {
  if (D.bstats[BS_RETRY]) return;
  __shared__ int64_t item_s;
  const int64_t nit = min((int64_t)ctr(D.dc, DC_HITEMS), K4_IT_CAP);
  uint8_t* mark = (uint8_t*)(D.slot_mark + (int64_t)blockIdx.x * D.N);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  int64_t k4acc = 0;
  int cur_g = -1;
  int32_t cur_h = -1, cur_ns = 0;
  const uint32_t* cur_S = nullptr;
  while (true) {
    __syncthreads();
    if (threadIdx.x == 0) item_s = (int64_t)atomicAdd(&D.dc[DC_QK4], 1ull);
    __syncthreads();
    const int64_t t = item_s;
    if (t >= nit) break;
    const int32_t h = D.k4_item[2 * t], c = D.k4_item[2 * t + 1];
    if (h < 0) continue;
    const int64_t i = D.k4_edge[3 * h], off = D.k4_edge[3 * h + 1];
    const int32_t ns = (int32_t)D.k4_edge[3 * h + 2];
    const uint32_t* Sh = D.k4_s + off;
    if (h != cur_h) {
      for (int32_t j = threadIdx.x; j < cur_ns; j += blockDim.x) mark[cur_S[j] & GC_ID] = 0;
      __syncthreads();
      for (int32_t j = threadIdx.x; j < ns; j += blockDim.x) {
        const uint32_t e = Sh[j];
        mark[e & GC_ID] = (uint8_t)(0x80u | ((e >> 28) & 3u) | (((e >> 30) & 3u) << 2));
      }
      __syncthreads();
      cur_h = h;
      cur_ns = ns;
      cur_S = Sh;
    }
    const unsigned long long ek = D.ce[i];
    const unsigned long long K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const int g = D.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) add_sig(D, cur_g, SG_K4, k4acc);
      k4acc = 0;
      cur_g = g;
    }
    k4acc += k4_through(D, mark, Sh, ns, c * K4_CHUNK, min(ns, (c + 1) * K4_CHUNK), u, v, K, fe);
  }
  __syncthreads();
  for (int32_t j = threadIdx.x; j < cur_ns; j += blockDim.x) mark[cur_S[j] & GC_ID] = 0;
  if (cur_g >= 0) add_sig(D, cur_g, SG_K4, k4acc);
}

// ------------------------------------------------------- affected edges
// The changed edges join the affected list (after the triangle kernel, so
// its count is final), then the list is sorted and each distinct edge
// (x, y) is taken by one wave: t before / after from the intersection of
// its rows, presence from its own entry.
__global__ void k_delta_aff_changed(DeltaArgs D) {
  if (D.bstats[BS_RETRY]) return;
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t base = (int64_t)D.dc[DC_AFF];
  for (int64_t i = gtid(); i < ne; i += gstride()) {
    const int64_t q = base + i;
    if (q < D.ae_cap) D.ae[q] = D.ce[i] & DIR_KEY_MASK;
  }
  if (gtid() == 0) {
    const int64_t tot = base + ne;
    D.dc[DC_AFF_TOTAL] = (unsigned long long)(tot < D.ae_cap ? tot : D.ae_cap);
    if (tot > D.ae_cap) {
      atomicAdd(&D.bstats[BS_RETRY], 1ull);
      atomicMax(&D.dc[DC_AFF_NEED], (unsigned long long)tot);
    }
  }
}

__global__ void k_delta_aff(DeltaArgs D, const unsigned long long* __restrict__ keys) {
  if (D.bstats[BS_RETRY]) return;
  const int64_t na = ctr(D.dc, DC_AFF_TOTAL);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  int64_t s3 = 0, s4 = 0, s5 = 0;
  int cur_g = -1;
  const int64_t nwv = gstride() >> 6;
  for (int64_t i = gtid() >> 6; i < na; i = wave_next(&D.dc[DC_QAFF], nwv)) {
    const unsigned long long key = keys[i];
    if (i > 0 && keys[i - 1] == key) continue;
    const uint32_t x = (uint32_t)(key >> D.bits), y = (uint32_t)(key & idmask);
    const int g = D.gid[x];
    if (g != cur_g) {
      if (cur_g >= 0) { add_sig(D, cur_g, SG_T, s3); add_sig(D, cur_g, SG_DIA, s4); add_sig(D, cur_g, SG_PAW, s5); }
      s3 = s4 = s5 = 0;
      cur_g = g;
    }
    const uint32_t a = D.P.len[x] <= D.P.len[y] ? x : y, b = a == x ? y : x;
    const uint32_t* arow = D.P.col + D.P.off[a];
    const int32_t al = D.P.len[a], bl = D.P.len[b];
    int32_t tb = 0, ta = 0;
    if (al > 0 && (int64_t)bl <= (int64_t)al * ((30 - __clz(max(bl, 1))) / 2)) {
      // rows of similar length (as for the 4-cycle pairs): both walked
      // together, 64 entries of each a step, instead of a search of the
      // longer row per entry of the shorter
      wave_window_common(D.P.col, D.P.off[a], al, D.P.off[b], bl, [&](uint32_t ea, uint32_t eb) {
        const uint32_t f = nib(ea) | nib(eb);
        tb += (f & 1u) == 0;
        ta += (f & 2u) == 0;
      });
    } else {
      // the shorter row's entries searched in the longer
      for (int32_t k = l; k < al; k += 64) {
        const uint32_t ea = arow[k], w = ea & GC_ID;
        if (w == b) continue;
        const int64_t p = find_in_row(D.P, b, w);
        if (p < 0) continue;
        const uint32_t f = nib(ea) | nib(D.P.col[p]);
        tb += (f & 1u) == 0;
        ta += (f & 2u) == 0;
      }
    }
    tb = wave_sum32(tb);
    ta = wave_sum32(ta);
    if (l == 0) {
      const int64_t p = find_in_row(D.P, x, y);
      const uint32_t f = p >= 0 ? nib(D.P.col[p]) : 3u;
      const int64_t pb = (f & 1u) == 0, pa = (f & 2u) == 0;
      const int64_t tbp = pb * tb, tap = pa * ta;
      s3 += tap - tbp;
      s4 += pa * c2(ta) - pb * c2(tb);
      s5 += tap * (deg_of(D, x, 1) + deg_of(D, y, 1) - 4) - tbp * (deg_of(D, x, 0) + deg_of(D, y, 0) - 4);
      // twice the change of T at both ends; t before on the affected edges at a touched end
      if (tap != tbp) { atomicAdd(&D.dT[x], (unsigned long long)(tap - tbp)); atomicAdd(&D.dT[y], (unsigned long long)(tap - tbp)); }
      if (tbp) {
        if (D.mark[x]) atomicAdd(&D.sbt[x], (unsigned long long)tbp);
        if (D.mark[y]) atomicAdd(&D.sbt[y], (unsigned long long)tbp);
      }
    }
  }
  if (cur_g >= 0) {
    // sums are held by lane 0 only: the wave sums add zeros from the others
    add_sig(D, cur_g, SG_T, s3); add_sig(D, cur_g, SG_DIA, s4); add_sig(D, cur_g, SG_PAW, s5);
  }
}

// At a touched vertex x whose degree changed, the edges that are not
// affected keep their t and present in both versions; their share of the
// paw term changes by t (d_a(x) - d_b(x)), and their t sum is 2 T(x) minus
// the t before of the affected edges at x.
__global__ void k_delta_vertex2(DeltaArgs D) {
  if (D.bstats[BS_RETRY]) return;
  const int64_t nt = ctr(D.c, C_TOUCH);
  for (int64_t t = gtid(); t < nt; t += gstride()) {
    const uint32_t x = (uint32_t)D.touched[t];
    const int64_t dd = (int64_t)D.dd[2 * (int64_t)x + 1] - D.dd[2 * (int64_t)x];
    const int64_t sb = (int64_t)D.sbt[x];
    D.sbt[x] = 0ull;
    if (dd) {
      const int64_t v = dd * (2 * D.Tv[x] - sb);
      atomicAdd(&D.sig[SIG_IDX(D.gid[x], 1, SG_PAW)], (unsigned long long)v);
    }
  }
}

// T(v) after the batch: every affected edge's ends take their share once.
__global__ void k_delta_tv(DeltaArgs D, const unsigned long long* __restrict__ keys) {
  if (D.bstats[BS_RETRY]) return;
  const int64_t na = ctr(D.dc, DC_AFF_TOTAL);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  for (int64_t i = gtid(); i < na; i += gstride()) {
    const unsigned long long key = keys[i];
    const uint32_t ends[2] = {(uint32_t)(key >> D.bits), (uint32_t)(key & idmask)};
    for (uint32_t x : ends) {
      const long long d2 = (long long)atomicExch(&D.dT[x], 0ull);
      if (d2) {
        if (d2 & 1) atomicAdd(&D.bstats[BS_ERR], 1ull);
        atomicAdd((unsigned long long*)&D.Tv[x], (unsigned long long)(d2 / 2));
      }
    }
  }
}

// ------------------------------------------------------------- 4-cycles
// Through a changed edge e = (s, o) run the 4-cycles s - a - b - o with
// a in N(s) - {o}, b in N(a) & N(o) - {s}.  A pair (e, a) is counted in one
// of two ways (pair_kind): its row N(a) is walked against a bitmap of N(o)
// that a workgroup keeps in LDS (k_delta_c4_bits), or the shorter of N(a) and
// N(o) is walked and each entry searched in the other row (k_delta_c4).  s is
// the end with the smaller total cost.  The work is balanced over the whole
// chip: every pair gets its walk length, a scan places the walked entries of
// all pairs in one index space, and waves or workgroups take ranges of that
// space (a hub pair is spread over many waves).

// A walked entry costs one LDS probe; a search step is a dependent global
// load.  Measured at scale 22: 9.9 ms for 0.6e9 searched entries (about 15
// steps each) against 3.5e12 probes a second for the walk, so a search of
// N(o) in N(a) pays only when N(a) is longer by more than this factor.
constexpr int64_t C4B_RATIO = 64;
// An edge whose walks sum to less than this does not earn a bitmap (clearing,
// filling and the queue cost a workgroup about as much as searching so much).
constexpr int64_t C4B_MIN = 4096;
constexpr int C4B_T = 1024;
constexpr int C4B_SMALL = 16384, C4B_LARGE = 36864;  // 32-bit words of the two bitmaps: 64 and 144 KB

__device__ __forceinline__ int64_t pair_cost(int32_t al, int32_t ol) {
  return min((int64_t)al, C4B_RATIO * (int64_t)ol);
}
// The bitmap of N(o) covers D.c4_ids ids downwards from N(o)'s last one: ids
// are a degree order, so the ids below that window have few entries.
__device__ __forceinline__ uint32_t c4b_base(const DeltaArgs& D, uint32_t o) {
  const uint32_t top = (D.P.col[D.P.off[o] + D.P.len[o] - 1] & GC_ID) + 1u;
  return top > D.c4_ids ? top - D.c4_ids : 0u;
}
// pairs of an edge with a bitmap that are walked against it
__device__ __forceinline__ bool pair_walked(int32_t al, int32_t ol) { return (int64_t)al <= C4B_RATIO * (int64_t)ol; }

// per changed edge: the end to walk from, whether it earns a bitmap, and its
// number of pairs.  An end u costs sum_{a in N(u)} pair_cost(d_a, d_v); both rows of every
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
    const uint32_t x = side_v ? v : u;
    const int32_t dx = side_v ? dv : du, other = side_v ? du : dv;
    const int32_t k0 = (int32_t)((side_v ? pk - nu : pk) * TV_CHUNK), k1 = min(dx, k0 + TV_CHUNK);
    const uint32_t* rx = D.P.col + D.P.off[x];
    int64_t c = 0;
    for (int32_t q = k0 + l; q < k1; q += 64) c += pair_cost(D.P.len[rx[q] & GC_ID], other);
    c = wave_sum64(c);
    if (l == 0 && c) atomicAdd((unsigned long long*)&D.pair_off[2 * i + (side_v ? 1 : 0)], (unsigned long long)c);
  }
}

__global__ void k_delta_plan_fin(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
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
    if (bitmap) {
      const uint32_t base = c4b_base(D, o);
      if (base) low = lower_bound_id(D.P.col + D.P.off[o], D.P.len[o], base);
    }
    D.c4_side[i] = (from_u ? 0 : 1) | (bitmap ? 2 : 0);
    D.c4_low[i] = low;
    D.c4_nch[i] = D.P.len[s];
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

// Appends a searched pair (edge i, index j, len entries) of the lanes with
// `take` to the list (one atomic per wave).
__device__ __forceinline__ void c4_search_append(const DeltaArgs& D, bool take, int64_t i, int32_t j, int32_t len) {
  const uint64_t m = __ballot(take);
  if (!m) return;
  unsigned long long at = 0;
  if (lane_id() == 0) at = atomicAdd(&D.dc[DC_SEARCH], (unsigned long long)__popcll(m));
  const int64_t q = (int64_t)__shfl((long long)at, 0) + __popcll(m & lanemask_lt());
  if (take && q < D.pair_cap) {
    D.pair_edge[q] = (int32_t)i;
    D.pair_idx[q] = j;
    D.pair_len[q] = len;
  }
}

// Per changed edge, a wave: the entries each pair (e, a) walks against the
// bitmap (0 for the others), in pair order; the searched pairs go to a list
// that holds nothing else, so that the waves of k_delta_c4 meet no empty
// pairs.
__global__ void k_delta_c4_pairs(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  if (gtid() == 0 && npairs > D.pair_cap) {
    atomicAdd(&D.bstats[BS_RETRY], 1ull);
    atomicMax(&D.dc[DC_PAIR_NEED], (unsigned long long)npairs);
  }
  if (npairs > D.pair_cap) return;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  const int64_t w0 = gtid() >> 6, ws = gstride() >> 6;
  for (int64_t i = w0; i < ne; i += ws) {
    const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const uint32_t s = (D.c4_side[i] & 1) ? v : u, o = s == u ? v : u;
    const uint32_t* srow = D.P.col + D.P.off[s];
    const int32_t sl = D.P.len[s], ol = D.P.len[o];
    const int64_t base = D.c4_off[i];
    const bool bitmap = (D.c4_side[i] & 2) != 0;
    for (int32_t k0 = 0; k0 < sl; k0 += 64) {
      const int32_t k = k0 + l;
      const uint32_t a = k < sl ? srow[k] & GC_ID : o;
      const int32_t al = D.P.len[a];
      const bool walked = bitmap && a != o && pair_walked(al, ol);
      if (k < sl) D.pair_hlen[base + k] = walked ? al : 0;
      c4_search_append(D, a != o && !walked, i, k, min(al, ol));
    }
    if (!bitmap) continue;
    const int32_t low = D.c4_low[i], out = low + D.na[o] + D.nr[o];  // pairs (e, b)
    for (int32_t k0 = 0; k0 < out; k0 += 64) {
      const int32_t k = k0 + l;
      uint32_t b = s, fob = 0;
      if (k < out) c4_out_pair(D, o, low, k, b, fob);
      const bool take = b != s && !(fob != 0 && (k < low || pkey(o, b, D.bits) < K));
      c4_search_append(D, take, i, sl + k, min(D.P.len[b], sl));
    }
  }
}

// More searched pairs than the list holds: count again with more.
__global__ void k_delta_c4_check(DeltaArgs D) {
  const unsigned long long n = D.dc[DC_SEARCH];
  if (gtid() == 0 && (int64_t)n > D.pair_cap) {
    atomicAdd(&D.bstats[BS_RETRY], 1ull);
    atomicMax(&D.dc[DC_PAIR_NEED], n);
  }
}

// largest i in [0, n) with pre[i] <= x, the wave together: 63 samples a round
__device__ __forceinline__ int64_t wave_upper_bound(const int64_t* __restrict__ pre, int64_t n, int64_t x) {
  int64_t lo = 0, hi = n;  // pre[lo] <= x, pre[hi] > x (or hi == n)
  while (hi - lo > 1) {
    const int64_t st = (hi - lo + 63) / 64;
    const int64_t at = lo + st * (lane_id() + 1);
    const int k = __popcll(__ballot(at < hi && pre[min(at, hi - 1)] <= x));
    hi = min(hi, lo + st * (k + 1));
    lo = lo + st * k;
  }
  return lo;
}

// A searched pair: the row walked, the row searched, and what a hit needs.
struct C4Search {
  int64_t walk;           // first entry of this wave's part of the row walked
  int64_t row;            // the row searched
  unsigned long long K;   // key of the changed edge
  int32_t len;            // entries of the row searched
  int32_t only;           // > 0: a pair (e, b), |N(o)| of the edge
  uint32_t s, o, a;       // the path s - a - b - o; the walk runs over b
  uint32_t meta;          // fe | fsa << 2 | (the row walked is N(a)) << 4
  int32_t g;
};

// The searched pairs.  Each wave takes one contiguous range of the index
// space of their walked entries (equal ranges: balanced by construction),
// 64 pairs at a time: a lane fetches one pair's record into LDS, then the
// entries of all of them are dealt over the lanes, each searching its entry
// in the other row.  Bound by the dependent loads of the searches.
__global__ __launch_bounds__(TPB) void k_delta_c4(DeltaArgs D) {
  __shared__ C4Search recs[TPB / 64][64];
  if (D.bstats[BS_RETRY]) return;
  const int64_t np = ctr(D.dc, DC_SEARCH);
  if (np == 0) return;
  const int64_t total = D.pair_off[np];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int l = lane_id();
  C4Search* rec = recs[threadIdx.x >> 6];
  const int64_t nw = gstride() >> 6;
  const int64_t per = ((total + nw - 1) / nw + 63) / 64 * 64;
  const int64_t w0 = min(total, (gtid() >> 6) * per), w1 = min(total, w0 + per);
  int64_t acc = 0;
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
        C4Search r;
        r.K = ek & DIR_KEY_MASK;
        const uint32_t u = (uint32_t)(r.K >> D.bits), v = (uint32_t)(r.K & idmask);
        r.s = (D.c4_side[i] & 1) ? v : u;
        r.o = r.s == u ? v : u;
        r.only = 0;
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
        const int64_t ao = D.P.off[r.a], oo = D.P.off[r.o];
        const int32_t al = D.P.len[r.a], ol = D.P.len[r.o];
        const bool wa = al <= ol;
        r.walk = (wa ? ao : oo) + (c0 - hb);
        r.row = wa ? oo : ao;
        r.len = wa ? ol : al;
        r.meta = ((uint32_t)(ek >> DIR_MASK_SHIFT) & 3u) | (fsa << 2) | ((wa ? 1u : 0u) << 4);
        r.g = D.gid[u];
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
      const C4Search& r = rec[lo];
      const uint32_t ew = D.P.col[r.walk + (idx - ex)], b = ew & GC_ID;
      const uint32_t* row = D.P.col + r.row;
      const int32_t len = r.len, x = lower_bound_id(row, len, b);
      if (x >= len) continue;
      const uint32_t er = row[x];
      if ((er & GC_ID) != b || b == r.s) continue;
      const bool wa = (r.meta >> 4) & 1u;
      const uint32_t fe = r.meta & 3u, fsa = (r.meta >> 2) & 3u, fab = nib(wa ? ew : er), fob = nib(wa ? er : ew);
      if ((fsa && pkey(r.s, r.a, D.bits) < r.K) || (fab && pkey(r.a, b, D.bits) < r.K) ||
          (fob && pkey(r.o, b, D.bits) < r.K) || (r.only && !pair_walked(D.P.len[b], r.only)))
        continue;
      if (r.g != cur_g) {
        if (cur_g >= 0 && acc) atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_C4)], (unsigned long long)acc);
        acc = 0;
        cur_g = r.g;
      }
      acc += delta_of(fe | fsa | fab | fob);
    }
    wave_sync();
  }
  // one atomic per wave when its lanes hold sums of one graph
  const uint64_t has = __ballot(cur_g >= 0 && acc != 0);
  if (has) {
    const int gl = __shfl(cur_g, __builtin_ctzll(has));
    if (__ballot(acc != 0 && cur_g != gl) == 0) {
      const int64_t t = wave_sum64(acc);
      if (lane_id() == 0 && t) atomicAdd(&D.sig[SIG_IDX(gl, 1, SG_C4)], (unsigned long long)t);
    } else if (acc) {
      atomicAdd(&D.sig[SIG_IDX(cur_g, 1, SG_C4)], (unsigned long long)acc);
    }
  }
}

// Walked entries per chunk of a bitmap edge: enough chunks to fill the chip
// several times over, each long enough to pay for its bitmap (four times
// |N(o)|, and a floor for the fixed cost of a chunk).
__device__ __forceinline__ int64_t c4b_chunk(int64_t total, int32_t ol) {
  const int64_t even = total / 4096;
  return max(min(max(even, (int64_t)16384), (int64_t)131072), 4 * (int64_t)ol);
}

// Chunks of the walked pairs per changed edge (0 past the edge count, for
// the scan).
__global__ void k_delta_hitems(DeltaArgs D) {
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  const int64_t npairs = D.c4_off[D.ce_cap];
  const bool fits = npairs <= D.pair_cap;  // else the pairs were not listed (count again)
  const int64_t total = fits ? D.pair_hoff[npairs] : 0;
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  for (int64_t i = gtid(); i < D.tcap; i += gstride()) {
    int32_t n = 0;
    if (i < ne && fits) {
      const int64_t h = D.pair_hoff[D.c4_off[i + 1]] - D.pair_hoff[D.c4_off[i]];
      if (h > 0) {
        const unsigned long long K = D.ce[i] & DIR_KEY_MASK;
        const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
        const int64_t T = c4b_chunk(total, D.P.len[(D.c4_side[i] & 1) ? u : v]);
        n = (int32_t)((h + T - 1) / T);
      }
    }
    D.tv_items[i] = n;
  }
}

// The walked pairs (e, a), e = (s, o).  Each workgroup takes chunks from a
// queue and holds a bitmap in LDS (kept while the next chunk is of the same
// edge) of the b in N(o) inside the window whose edge (o, b) is not in the
// batch.  Its waves split the chunk's entries of the rows N(a) evenly, read
// them with consecutive lanes and probe one bit per entry: a hit closes the
// path s - a - b - o.  Hits on entries that are in the batch themselves take
// the general rule (rare).
// What bounds it: instruction issue, about 13 per 64 entries, while the
// bitmap costs little (a chunk is at least four times |N(o)|).  Before, rows
// of similar length were merged by a wave (about 35 instructions and nine
// lane exchanges per 64 entries of each row), shorter rows probed an LDS hash
// table and the rest was searched: 22 ms in all for 2,500 updates at scale 22
// (7e9 entries walked), 2.1 ms for 1,000 at scale 18 (1.3e8); now 6.3 + 0.3 ms
// and 0.25 + 0.02 ms.  WORDS = 16384 (ids up to 2^19) lets two workgroups
// share a CU.
template <int WORDS>
__global__ __launch_bounds__(C4B_T, WORDS <= 16384 ? 8 : 4) void k_delta_c4_bits(DeltaArgs D) {
  __shared__ uint4 bm4[WORDS / 4];
  __shared__ int64_t item_s, edge_s;
  if (D.bstats[BS_RETRY]) return;
  uint32_t* bm = (uint32_t*)bm4;
  const int64_t ne = min(ctr(D.dc, DC_EDGES), D.ce_cap);
  if (ne == 0) return;
  const int64_t nitems = D.tv_ioff[ne];
  const int64_t total = D.pair_hoff[D.c4_off[D.ce_cap]];
  const unsigned long long idmask = (1ull << D.bits) - 1ull;
  const int32_t l = lane_id(), wv = (int32_t)(threadIdx.x >> 6);
  constexpr int32_t NW = C4B_T / 64;
  const uint32_t ids = D.c4_ids;  // <= WORDS * 32
  const uint32_t* __restrict__ col = D.P.col;
  int64_t acc = 0;
  int cur_g = -1;
  int64_t cur_i = -1;
  while (true) {
    __syncthreads();
    if (wv == 0) {
      int64_t it0 = 0;
      if (l == 0) it0 = (int64_t)atomicAdd(&D.dc[DC_QH], 1ull);
      it0 = __shfl(it0, 0);
      const int64_t i0 = it0 < nitems ? wave_upper_bound(D.tv_ioff, ne, it0) : 0;
      if (l == 0) { item_s = it0; edge_s = i0; }
    }
    __syncthreads();
    const int64_t it = item_s, i = edge_s;
    if (it >= nitems) break;
    const unsigned long long ek = D.ce[i];
    const unsigned long long K = ek & DIR_KEY_MASK;
    const uint32_t fe = (uint32_t)(ek >> DIR_MASK_SHIFT) & 3u;
    const uint32_t u = (uint32_t)(K >> D.bits), v = (uint32_t)(K & idmask);
    const uint32_t s = (D.c4_side[i] & 1) ? v : u, o = s == u ? v : u;
    const int64_t so = D.P.off[s], oo = D.P.off[o];
    const int32_t ol = D.P.len[o];  // > 0: row o holds s
    const uint32_t base = c4b_base(D, o);
    const int g = D.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) add_sig(D, cur_g, SG_C4, acc);
      acc = 0;
      cur_g = g;
    }
    const int64_t T = c4b_chunk(total, ol);
    const int64_t ch = it - D.tv_ioff[i];
    if (i != cur_i) {
      for (int32_t k = (int32_t)threadIdx.x; k < WORDS / 4; k += C4B_T) bm4[k] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
      for (int32_t k0 = wv * 256; k0 < ol; k0 += 4 * C4B_T) {  // four loads in flight per lane
        uint32_t y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = col[oo + min(k0 + 64 * q + l, ol - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t x = (y[q] & GC_ID) - base;
          if (!(y[q] & GC_FLAGS) && x < ids) atomicOr(&bm[x >> 5], 1u << (x & 31u));
        }
      }
      cur_i = i;
      __syncthreads();
    }
    // the chunk: entries [r0, r1) of the walked index space, this wave's
    // piece of them; 64 pairs at a time, a pair's part of the piece per lane
    const int64_t p0 = D.c4_off[i], p1 = D.c4_off[i + 1];
    const int64_t r0 = D.pair_hoff[p0] + ch * T, r1 = min(D.pair_hoff[p1], r0 + T);
    const int64_t per = (r1 - r0 + NW - 1) / NW;
    const int64_t w0 = min(r1, r0 + wv * per), w1 = min(r1, w0 + per);
    uint32_t clean = 0;  // hits with no other edge of the path in the batch
    if (w0 < w1) {
      for (int64_t p = p0 + wave_upper_bound(D.pair_hoff + p0, p1 - p0, w0); p < p1; p += 64) {
        if (D.pair_hoff[p] >= w1) break;
        const int64_t pl = p + l;
        int64_t sb = 0;
        int32_t sn = 0;
        uint32_t esa = 0;
        if (pl < p1) {
          const int64_t hb = D.pair_hoff[pl], he = D.pair_hoff[pl + 1];
          const int64_t c0 = max(hb, w0), c1 = min(he, w1);
          if (c0 < c1) {
            esa = col[so + (pl - p0)];
            sb = D.P.off[esa & GC_ID] + (c0 - hb);
            sn = (int32_t)(c1 - c0);
          }
        }
        wave_rows(col, sb, sn, esa, [&](uint32_t ea, uint32_t y) {
          const uint32_t x = (y & GC_ID) - base;
          uint32_t hit = 0;
          if (x < ids) hit = (bm[x >> 5] >> (x & 31u)) & 1u;
          if (hit && ((ea | y) & GC_FLAGS)) {  // (s, a) or (a, b) in the batch
            const uint32_t a = ea & GC_ID, b = y & GC_ID, fsa = nib(ea), fab = nib(y);
            hit = 0;
            if (!(fsa && pkey(s, a, D.bits) < K) && !(fab && pkey(a, b, D.bits) < K)) acc += delta_of(fe | fsa | fab);
          }
          clean += hit;
        });
      }
    }
    acc += (int64_t)clean * delta_of(fe);
  }
  if (cur_g >= 0) add_sig(D, cur_g, SG_C4, acc);
}

// ------------------------------------------------ T(v) in the region path
// After the triangle kernels of a region (or whole-graph) pass, t holds the
// triangles of every upper entry (id order) of the region per version.  A
// changed triangle at v lies inside the region and sits on two edges at v,
// so T(v) moves by half the change of t summed over the edges at v: each
// upper entry hands its change to both ends, then each region vertex takes
// its half once.
template <int NV>
__global__ void k_tv_entries(RegionDev R, const unsigned long long* c, unsigned long long* __restrict__ dT,
                             const unsigned long long* bstats) {
  if (bstats[BS_RETRY]) return;
  const int64_t ne = ctr(c, C_ER);
  for (int64_t p = gtid(); p < ne; p += gstride()) {
    const uint32_t w = R.rcol[p] & GC_ID;
    const int32_t v = R.rrow[p];
    if ((int64_t)w <= (int64_t)v) continue;
    int64_t d;
    if constexpr (NV == 2) {
      const unsigned long long x = R.t[p];
      d = (int64_t)(x >> 32) - (int64_t)(x & 0xFFFFFFFFull);
    } else {
      // t_x = t[p] + field x of tp[2p] (x = 0, 1) and tp[2p + 1] (x = 2, 3)
      d = (int64_t)(R.tp[2 * p + 1] >> 32) - (int64_t)(R.tp[2 * p] & 0xFFFFFFFFull);
    }
    if (d) {
      atomicAdd(&dT[v], (unsigned long long)d);
      atomicAdd(&dT[w], (unsigned long long)d);
    }
  }
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
void launch_delta(const DeltaArgs& D_, int slots, hipStream_t s) {
  DeltaArgs D = D_;
  const bool small_bits = D.N <= C4B_SMALL * 32;
  const uint32_t ids = (small_bits ? C4B_SMALL : C4B_LARGE) * 32;
  if (D.c4_ids == 0 || D.c4_ids > ids) D.c4_ids = ids;
  fill_u64(D.dc, 0ull, DC_COUNT, s);
  hipLaunchKernelGGL(k_delta_edges, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_titems, dim3(1024), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_vertex, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_vertex_fin, dim3(256), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_s2, dim3(2048), dim3(TPB), 0, s, D);
  // every kernel that can find a buffer too small (and raise BS_RETRY)
  // runs before the first one that moves T(v) or clears scratch
  hipLaunchKernelGGL(k_delta_tri, dim3(slots), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_k4_split, dim3(slots), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_aff_changed, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_plan_items, dim3(1024), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_c4_plan, dim3(2048), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_plan_fin, dim3(256), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.c4_nch, D.c4_off, D.ce_cap, D.scan_tmp, s);
  // every walked and every searched pair below their counts gets a length,
  // and only offsets up to the counts are read: no clearing, scans up to them
  hipLaunchKernelGGL(k_delta_c4_pairs, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_c4_check, dim3(1), dim3(64), 0, s, D);
  exclusive_scan_i32_to_i64_count(D.pair_len, D.pair_off, D.pair_cap, (const int64_t*)(D.dc + DC_SEARCH), D.scan_tmp, s);
  exclusive_scan_i32_to_i64_count(D.pair_hlen, D.pair_hoff, D.pair_cap, D.c4_off + D.ce_cap, D.scan_tmp, s);
  hipLaunchKernelGGL(k_delta_hitems, dim3(256), dim3(TPB), 0, s, D);
  exclusive_scan_i32_to_i64(D.tv_items, D.tv_ioff, D.tcap, D.scan_tmp, s);
  unsigned long long* sorted =
      radix_sort_u64(D.ae, D.ae_alt, D.sort_tmp, D.ae_cap, D.dc + DC_AFF_TOTAL, 2 * D.bits, s);
  hipLaunchKernelGGL(k_delta_aff, dim3(4096), dim3(TPB), 0, s, D, (const unsigned long long*)sorted);
  hipLaunchKernelGGL(k_delta_vertex2, dim3(1024), dim3(TPB), 0, s, D);
  hipLaunchKernelGGL(k_delta_tv, dim3(1024), dim3(TPB), 0, s, D, (const unsigned long long*)sorted);
  hipLaunchKernelGGL(k_delta_c4, dim3(4096), dim3(TPB), 0, s, D);
  if (small_bits)
    hipLaunchKernelGGL(k_delta_c4_bits<C4B_SMALL>, dim3(512), dim3(C4B_T), 0, s, D);
  else
    hipLaunchKernelGGL(k_delta_c4_bits<C4B_LARGE>, dim3(256), dim3(C4B_T), 0, s, D);
}

void launch_tv_region(int nv, const RegionDev& R, const int32_t* rlist, const unsigned long long* c,
                      unsigned long long* dT, long long* Tv, unsigned long long* bstats, hipStream_t s) {
  if (nv == 2)
    hipLaunchKernelGGL(k_tv_entries<2>, dim3(4096), dim3(TPB), 0, s, R, c, dT, (const unsigned long long*)bstats);
  else
    hipLaunchKernelGGL(k_tv_entries<4>, dim3(4096), dim3(TPB), 0, s, R, c, dT, (const unsigned long long*)bstats);
  hipLaunchKernelGGL(k_tv_apply, dim3(2048), dim3(TPB), 0, s, rlist, c, dT, Tv, bstats);
}
