// Counting kernels: the local static counter applied to the region, fused
// over the versions of the pass (Alg. 2 counts G_b and G_a and adds
// C_a - C_b; a pass over several queued batches counts every intermediate
// graph as well).  Every structure is enumerated once in the union view and
// the versions it exists in are read off the flags of its entries.  Kernels
// are instantiated for NV = 2 versions (one batch) and NV = 4 (up to three
// batches of one graph).
//
// Per-edge counting (the PGD approach of Sec. 3: iterate over edges, count
// triangles, 4-cliques and 4-cycles, derive the rest by combinatorics):
//   triangles  oriented by id: u < v < w found at u, with v in N+(u) and
//              w in N+(u) & N+(v).  Each triangle adds 1 to t of its three
//              edges (t_e = common neighbours of the endpoints of e).
//   4-cliques  u < v < w < x, x in N+(u) & N+(v) & N+(w).
//   4-cycles   counted once, at the largest vertex v, through the opposite
//              vertex w < v: c(v,w) = #{u < v adjacent to both}, and
//              sum_w C(c(v,w), 2).
//   the non-induced counts follow:
//     N_K13 = sum_v C(d,3)        N_P4 = sum_e (d_u-1)(d_v-1) - 3T
//     N_paw = sum_tri (d_u + d_v + d_w - 6)   N_dia = sum_e C(t_e, 2)
//     N_K4, N_C4 as enumerated.
//
// Tiers (work lists built by the per-vertex pass):
//   tri  S: out-degree <= 64, one wave per vertex, bit matrices in LDS
//   tri  L: larger out-degree, one workgroup per vertex, LDS hash; tiers of
//           out-degree <= 128, 256, 512, 1024, 1280, and global-memory
//           scratch above
//   c4   S / M: wedge bound <= 256 / <= 4096, LDS hash per wave / workgroup
//   c4   L: one workgroup per vertex, windows of dense counters in LDS,
//           then dense counters in global memory
#include "gc_kernels.h"

#include <type_traits>

namespace {

__device__ __forceinline__ int64_t gtid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }

__device__ __forceinline__ uint32_t hash32(uint32_t x) { return x * 2654435761u; }

__device__ __forceinline__ int32_t ld_relaxed(int32_t* p) { return __atomic_load_n(p, __ATOMIC_RELAXED); }

// Open addressing, linear probing; -1 marks a free slot.
struct HashLook {
  const int32_t* keys;
  uint32_t mask;
  int shift;
  __device__ __forceinline__ int find(uint32_t key) const {  // position or -1
    for (uint32_t h = hash32(key) >> shift;; h = (h + 1) & mask) {
      const int32_t k = keys[h];
      if (k == (int32_t)key) return (int)h;
      if (k == -1) return -1;
    }
  }
};

// add `add` to the counter of key (insert on first use)
template <class V>
__device__ __forceinline__ void hash_add(int32_t* keys, V* vals, uint32_t mask, int shift, uint32_t key, V add) {
  uint32_t h = hash32(key) >> shift;
  while (true) {
    int32_t k = ld_relaxed(&keys[h]);
    if (k == (int32_t)key) { atomicAdd(&vals[h], add); return; }
    if (k == -1) {
      int32_t old = atomicCAS(&keys[h], -1, (int32_t)key);
      if (old == -1 || old == (int32_t)key) { atomicAdd(&vals[h], add); return; }
    }
    h = (h + 1) & mask;
  }
}

__device__ __forceinline__ int log2i(uint32_t x) { return 31 - __clz(x); }

// Segment search for wave-flattened loops: every lane holds one segment
// with exclusive prefix `excl`; returns the lane whose segment holds idx
// (largest lane with excl <= idx).  All 64 lanes must call it.
__device__ __forceinline__ int seg_of(int32_t excl, int32_t idx) {
  int lo = 0, hi = 64;
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    int mid = (lo + hi) >> 1;
    int32_t e = __shfl(excl, mid);
    if (e <= idx) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int32_t rdl32(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

// Vertices of a per-wave tier in chunks of up to QV_CHUNK (as many as the
// list holds per wave of the grid, so that a short list still uses every
// wave): a wave's first chunk is its own index (no atomic: waves without one
// leave at once), later ones come from a shared counter counting on from the
// grid's wave count, so that the waves that drew light vertices take more
// than a fixed stride would give them.  Returns the same chunk on every lane.
constexpr int64_t QV_CHUNK = 16;
__device__ __forceinline__ int64_t qv_chunk(int64_t n, int64_t nwaves) {
  return max((int64_t)1, min(QV_CHUNK, n / max(nwaves, (int64_t)1)));
}
__device__ __forceinline__ int64_t wave_next_chunk(const unsigned long long* ctr_, int64_t nwaves) {
  unsigned long long c = 0;
  if ((__lane_id()) == 0) c = atomicAdd((unsigned long long*)ctr_, 1ull);
  return nwaves + (int64_t)__shfl(c, 0);
}
__device__ __forceinline__ int64_t rdl64(int64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Walk the lists of a wave's lanes (lane l: positions [sb, sb + sl) of the
// entry array col, with a 32-bit payload pl) calling f(list lane, position,
// payload of that lane, entry).  Lists of at least WALK_LONG entries go one
// at a time through the whole wave (consecutive lanes read consecutive
// entries, D loads in flight per lane; the list's lane is read with scalar
// reads); the others are flattened over the lanes with a segment search per
// step.  Most entries sit in long lists, which then cost no cross-lane
// traffic.  All lanes must call it.
constexpr int32_t WALK_LONG = 32;

template <int D = 4, class F>
__device__ __forceinline__ void wave_walk(const uint32_t* col, int64_t sb, int32_t sl, uint32_t pl, F f) {
  const int l = lane_id();
  const bool lng = sl >= WALK_LONG;
  uint64_t lm = __ballot(lng);
  while (lm) {
    const int s = __builtin_ctzll(lm);
    lm &= lm - 1;
    const int64_t b = rdl64(sb, s);
    const int32_t n = rdl32(sl, s);
    const uint32_t ps = (uint32_t)rdl32((int32_t)pl, s);
    for (int32_t k = l; k < n; k += 64 * D) {
      uint32_t y[D];
#pragma unroll
      for (int u = 0; u < D; ++u) y[u] = k + 64 * u < n ? col[b + k + 64 * u] : 0u;
#pragma unroll
      for (int u = 0; u < D; ++u)
        if (k + 64 * u < n) f(s, b + k + 64 * u, ps, y[u]);
    }
  }
  const int32_t ss = lng ? 0 : sl;
  const int32_t incl = wave_incl_scan32(ss);
  const int32_t tot = __shfl(incl, 63);
  const int32_t excl = incl - ss;
  for (int32_t base = 0; base < tot; base += 64) {
    const int32_t idx = base + l;
    const int s = seg_of(excl, idx);
    const int64_t sbs = __shfl(sb, s);
    const int32_t exs = __shfl(excl, s);
    const uint32_t ps = (uint32_t)__shfl((int32_t)pl, s);
    if (idx < tot) {
      const int64_t pos = sbs + (idx - exs);
      f(s, pos, ps, col[pos]);
    }
  }
}

// The entries of the lists of a wave's lanes (lane l: [sb, sb + sl) of col)
// that are in a set of ids: f(s, pos, y) for every entry y at pos of lane s's
// list whose bit in `filt` is set -- a superset of those in the set, which f
// looks up.  filt holds 2^(32 - fsh) bits, one per hash value; about one id in
// ten passes in the triangle tiers, so the ids that pass are packed into a
// list in LDS (q, 256 words of the wave) and 64 at a time take a lane each:
// the lookup and what a hit does, some 100 instructions, ran for nearly every
// 64 entries before, for the few lanes that hit.  Long lists go one at a time
// through the whole wave, 128 entries a step with the next step's loads in
// flight (also across lists); short ones are flattened over the lanes.
// Bound by issue (about 30 instructions per 64 entries) and, in dense graphs,
// by the atomics of the hits.  Scale 22, a count: k_tri_small 12.1 -> 7.6 ms,
// <128> 9.5 -> 6.5, <256> 13.3 -> 9.7, <512> 14.9 -> 12.9, <1024> 18.7 -> 18.2.
template <class F>
__device__ __forceinline__ void wave_probe(const uint32_t* __restrict__ col, int64_t sb, int32_t sl,
                                           const uint32_t* filt, int fsh, uint32_t* q, F f) {
  const int l = lane_id();
  int32_t n = 0;  // listed entries
  auto run = [&](int32_t k, bool in) {
    const uint32_t y = in ? q[k] : 0u, at = in ? q[128 + k] : 0u;
    const int s = (int)(at >> 26);
    const int64_t b = __shfl(sb, s);
    f(s, b + (int64_t)(at & 0x3FFFFFFu), y, in);
  };
  // offsets in a list take 26 bits: the bit matrix of a vertex with more
  // out-neighbours would not fit the memory
  auto probe = [&](uint32_t y, bool in, uint32_t at) {
    const uint32_t h = hash32(y & GC_ID) >> fsh;
    const bool pass = in && ((filt[h >> 5] >> (h & 31u)) & 1u);
    const uint64_t m = __ballot(pass);
    if (!m) return;
    if (pass) {
      const int32_t k = n + __popcll(m & lanemask_lt());
      q[k] = y;
      q[128 + k] = at;
    }
    n += __popcll(m);
    if (n >= 64) {
      n -= 64;
      wave_sync();
      run(n + l, true);
      wave_sync();
    }
  };
  uint64_t lm = __ballot(sl >= WALK_LONG);
  if (lm) {
    int s = __builtin_ctzll(lm);
    int64_t b = rdl64(sb, s);
    int32_t len = rdl32(sl, s), k = 0;
    uint32_t y0 = col[b + min(l, len - 1)], y1 = col[b + min(64 + l, len - 1)];
    while (true) {
      const int sc = s;
      const int32_t kc = k, lc = len;
      const uint32_t c0 = y0, c1 = y1;
      bool more = true;
      if (k + 128 < len) {
        k += 128;
      } else {
        lm &= lm - 1;
        more = lm != 0;
        if (more) {
          s = __builtin_ctzll(lm);
          b = rdl64(sb, s);
          len = rdl32(sl, s);
          k = 0;
        }
      }
      if (more) {
        y0 = col[b + min(k + l, len - 1)];
        y1 = col[b + min(k + 64 + l, len - 1)];
      }
      const uint32_t at = ((uint32_t)sc << 26) | (uint32_t)(kc + l);
      probe(c0, kc + l < lc, at);
      if (kc + 64 < lc) probe(c1, kc + 64 + l < lc, at + 64u);
      if (!more) break;
    }
  }
  const int32_t ss = sl >= WALK_LONG ? 0 : sl;
  const int32_t incl = wave_incl_scan32(ss);
  const int32_t tot = __shfl(incl, 63), excl = incl - ss;
  for (int32_t base = 0; base < tot; base += 64) {
    const int32_t idx = base + l;
    const int s = seg_of(excl, idx);
    const int64_t sbs = __shfl(sb, s);
    const int32_t k = idx - __shfl(excl, s);
    const bool in = idx < tot;
    probe(in ? col[sbs + k] : 0u, in, ((uint32_t)s << 26) | (uint32_t)(in ? k : 0));
  }
  wave_sync();
  if (n) run(l, l < n);
  wave_sync();
}

__device__ __forceinline__ unsigned long long pack2(uint32_t b, uint32_t a) {
  return (unsigned long long)b | ((unsigned long long)a << 32);
}

// Per-version counters packed in one word: NF fields of FB bits each.
template <int NF, int FB>
struct Fields {
  using T = typename std::conditional<(NF * FB <= 32), uint32_t, unsigned long long>::type;
  // 1 in field x for every bit x of pm
  __device__ static __forceinline__ T spread(uint32_t pm) {
    T r = 0;
#pragma unroll
    for (int x = 0; x < NF; ++x) r |= (T)((pm >> x) & 1u) << (FB * x);
    return r;
  }
  __device__ static __forceinline__ int64_t get(T c, int x) {
    return (int64_t)((c >> (FB * x)) & (T)((1ull << FB) - 1ull));
  }
};

// flush lane-private per-version sums of a wave whose lanes all work for graph g
template <int NV>
__device__ __forceinline__ void flushv(unsigned long long* sig, int g, int k, int64_t (&a)[NV]) {
#pragma unroll
  for (int x = 0; x < NV; ++x) {
    flush_sig(sig, g, x, k, a[x]);
    a[x] = 0;
  }
}

template <int NV>
__device__ __forceinline__ void zerov(int64_t (&a)[NV]) {
#pragma unroll
  for (int x = 0; x < NV; ++x) a[x] = 0;
}

// t of entry pos: one triangle (or c of them) present in the versions of pm
// (at least one).  These atomics are what the dense tiers wait for: 32-bit
// instead of 64-bit words with a field per version took k_tri_large<1024> from
// 24.8 to 22.9 ms at scale 22 and <512> from 17.4 to 16.7 (without the
// 4-cliques, during which the queue drains, 20.5 to 12.1 and 16.1 to 11.2);
// later changes brought them to 18.2 and 13.0.
template <int NV>
__device__ __forceinline__ void t_add(const RegionDev& R, int64_t pos, uint32_t pm, uint32_t c = 1u) {
  if constexpr (NV == 2) {
    if (pm & 1u) atomicAdd(&R.t[pos], c);
    if (pm != 3u) atomicAdd(&R.td[pos], pm == 2u ? (int32_t)c : -(int32_t)c);
  } else {
    if (pm == 0xFu) { atomicAdd(&R.t[pos], c); return; }
    if (pm & 3u) atomicAdd(&R.tp[2 * pos], pack2((pm & 1u) * c, ((pm >> 1) & 1u) * c));
    if (pm & 12u) atomicAdd(&R.tp[2 * pos + 1], pack2(((pm >> 2) & 1u) * c, ((pm >> 3) & 1u) * c));
  }
}

// t of entry pos: c[x] triangles in version x
template <int NV>
__device__ __forceinline__ void t_addv(const RegionDev& R, int64_t pos, const uint32_t (&c)[NV]) {
  if constexpr (NV == 2) {
    if (c[0]) atomicAdd(&R.t[pos], c[0]);
    if (c[1] != c[0]) atomicAdd(&R.td[pos], (int32_t)(c[1] - c[0]));
  } else {
    const uint32_t m = min(min(c[0], c[1]), min(c[2], c[3]));
    if (m) atomicAdd(&R.t[pos], m);
    if ((c[0] - m) | (c[1] - m)) atomicAdd(&R.tp[2 * pos], pack2(c[0] - m, c[1] - m));
    if ((c[2] - m) | (c[3] - m)) atomicAdd(&R.tp[2 * pos + 1], pack2(c[2] - m, c[3] - m));
  }
}

template <int NV>
__device__ __forceinline__ void t_read(const RegionDev& R, int64_t pos, int64_t (&t)[NV]) {
  const unsigned long long a = R.t[pos];
  if constexpr (NV == 2) {
    t[0] = (int64_t)a;
    t[1] = (int64_t)a + R.td[pos];
  } else {
    const ulonglong2 p = *(const ulonglong2*)(R.tp + 2 * pos);
    t[0] = (int64_t)(a + (p.x & 0xFFFFFFFFull));
    t[1] = (int64_t)(a + (p.x >> 32));
    t[2] = (int64_t)(a + (p.y & 0xFFFFFFFFull));
    t[3] = (int64_t)(a + (p.y >> 32));
  }
}

// The triangle counts of the region's entries, cleared 16 bytes at a time.
template <int NV>
__global__ __launch_bounds__(256) void k_t_clear(CountArgs A) {
  const int64_t E = min((int64_t)A.c[C_ER], A.e_max), n4 = (E + 3) / 4;
  const uint4 z = make_uint4(0u, 0u, 0u, 0u);
  uint4* t = (uint4*)A.R.t;
  uint4* td = (uint4*)A.R.td;
  uint4* tp = (uint4*)A.R.tp;
  for (int64_t i = gtid(); i < n4; i += gstride()) {
    t[i] = z;
    if (NV == 2) td[i] = z;
  }
  if (NV == 4)
    for (int64_t i = gtid(); i < E; i += gstride()) tp[i] = z;
}

template <int NV>
__device__ __forceinline__ void d_read(const RegionDev& R, int64_t v, int32_t (&d)[NV]) {
  if constexpr (NV == 2) {
    const int2 q = *(const int2*)(R.d + v * 2);
    d[0] = q.x; d[1] = q.y;
  } else {
    const int4 q = *(const int4*)(R.d + v * 4);
    d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
  }
}

__device__ __forceinline__ bool absent_in(uint32_t flags, int x) { return (flags >> (GC_VSHIFT + x)) & 1u; }

// ------------------------------------------------------ triangles, tier S
// One wave per vertex u with out-degree <= 64.  Bit matrices over the slots
// of N+(u): EU[i] has bit j (j > i) when v_i -> v_j is an edge of the union
// view, TU its transpose, and EX[x] / TX[x] the same for the edges absent
// from version x (only edges with flags land there).  A wave that met no
// flag at all counts version 0 once and copies it to the others.
constexpr int TS_WAVES = 4;

template <int NV>
__global__ __launch_bounds__(256) void k_tri_small(CountArgs A) {
  __shared__ int32_t hkey[TS_WAVES][128];   // load factor <= 1/2: few ids that are not there are looked up
  __shared__ uint32_t hval[TS_WAVES][128];  // slot | its flags
  __shared__ uint32_t filt[TS_WAVES][128];  // 4096 bits
  __shared__ uint32_t queue[TS_WAVES][256];
  __shared__ unsigned long long EU[TS_WAVES][64], TU[TS_WAVES][64];
  __shared__ unsigned long long EX[TS_WAVES][NV][64], TX[TS_WAVES][NV][64];
  __shared__ uint32_t dirty[TS_WAVES];
  const int w = threadIdx.x >> 6, l = lane_id();
  const RegionDev& R = A.R;
  const int64_t n = (int64_t)A.c[C_LIST0 + L_TRI_S];
  const int32_t* list = A.lists + L_TRI_S * A.list_stride;
  int cur_g = -1;
  int64_t kacc[NV];
  zerov<NV>(kacc);
  int64_t ent = 0;  // entries of N+(u) and of the lists probed (algorithmic reads)
  const int64_t nwv = (int64_t)gridDim.x * TS_WAVES, cq = qv_chunk(n, nwv);
  for (int64_t ch = (int64_t)blockIdx.x * TS_WAVES + w; ch * cq < n; ch = wave_next_chunk(A.c + C_QTS, nwv))
  for (int64_t it = ch * cq; it < min(n, (ch + 1) * cq); ++it) {
    const int32_t u = list[it];
    const int g = A.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_K4, kacc);
      cur_g = g;
    }
    const int64_t ub = R.roff[u] + R.rlow[u];
    const int32_t dp = (int32_t)(R.roff[u + 1] - ub);
    uint32_t vi = 0, fi = 0;
    if (l < dp) { const uint32_t x = R.rcol[ub + l]; vi = x & GC_ID; fi = x & GC_FLAGS; }
#pragma unroll
    for (int q = 0; q < 2; ++q) { hkey[w][l + 64 * q] = -1; filt[w][l + 64 * q] = 0u; }
    EU[w][l] = 0; TU[w][l] = 0;
#pragma unroll
    for (int x = 0; x < NV; ++x) { EX[w][x][l] = 0; TX[w][x][l] = 0; }
    if (l == 0) dirty[w] = 0;
    wave_sync();
    if (l < dp) {
      const uint32_t fh = hash32(vi) >> 20;
      atomicOr(&filt[w][fh >> 5], 1u << (fh & 31u));
      uint32_t h = hash32(vi) >> 25;
      while (atomicCAS(&hkey[w][h], -1, (int32_t)vi) != -1) h = (h + 1) & 127u;
      hval[w][h] = (uint32_t)l | fi;
    }
    wave_sync();
    int64_t sb = 0;
    int32_t sl = 0;
    if (l < dp) { sb = R.roff[vi] + R.rlow[vi]; sl = (int32_t)(R.roff[vi + 1] - sb); ent += 1 + sl; }
    // a hit of list i (slot j with flags, jv) is the triangle (u, v_i, v_j)
    const HashLook hl{hkey[w], 127u, 25};
    wave_probe(R.rcol, sb, sl, filt[w], 20, queue[w], [&](int i, int64_t pos, uint32_t y, bool in) {
      const uint32_t fs = (uint32_t)__shfl((int32_t)fi, i);
      if (!in) return;
      const int p = hl.find(y & GC_ID);
      if (p < 0) return;
      const uint32_t jv = hval[w][p], fy = y & GC_FLAGS;
      const int j = (int)(jv & GC_ID);
      const unsigned long long bj = 1ull << j, bi = 1ull << i;
      atomicOr(&EU[w][i], bj);
      atomicOr(&TU[w][j], bi);
      if (fy) {
        dirty[w] = 1u;
#pragma unroll
        for (int x = 0; x < NV; ++x)
          if (absent_in(fy, x)) { atomicOr(&EX[w][x][i], bj); atomicOr(&TX[w][x][j], bi); }
      }
      const uint32_t pm = vpresent<NV>(fs | (jv & GC_FLAGS) | fy);
      if (pm) t_add<NV>(R, pos, pm);
    });
    wave_sync();
    const bool clean = __ballot(l < dp && fi != 0) == 0ull && dirty[w] == 0u;
    uint64_t Px[NV];
#pragma unroll
    for (int x = 0; x < NV; ++x) Px[x] = __ballot(l < dp && !absent_in(fi, x));
    if (l < dp) {
      uint32_t tu[NV];
      int64_t kv[NV];
#pragma unroll
      for (int x = 0; x < NV; ++x) {
        tu[x] = 0;
        kv[x] = 0;
        if (x > 0 && clean) { tu[x] = tu[0]; kv[x] = kv[0]; continue; }
        if (!((Px[x] >> l) & 1ull)) continue;
        const unsigned long long e = EU[w][l] & ~EX[w][x][l] & Px[x];
        const unsigned long long tt = TU[w][l] & ~TX[w][x][l] & Px[x];
        tu[x] = (uint32_t)__popcll(e | tt);
        int64_t k4 = 0;
        for (unsigned long long m = e; m; m &= m - 1) {
          const int j = __builtin_ctzll(m);
          k4 += __popcll(e & EU[w][j] & ~EX[w][x][j] & Px[x]);
        }
        kv[x] = k4;
      }
#pragma unroll
      for (int x = 0; x < NV; ++x) kacc[x] += kv[x];
      t_addv<NV>(R, ub + l, tu);
    }
    wave_sync();
  }
  if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_K4, kacc);
  ent = wave_sum64(ent);
  if (l == 0 && ent) atomicAdd(&A.bstats[BS_TRI_E], (unsigned long long)ent);
}

// ------------------------------------------------------ triangles, tier L
// One workgroup per vertex u with out-degree above 64, twice as many threads
// as slots up to 512: fewer vertices at a time, each done sooner, so the last
// round of a tier is shorter.  Scale 18, <256> with 256 and 512 threads 0.54
// and 0.42 ms, <512> 0.20 and 0.12, <128> 0.46 and 0.43; scale 22, where the
// rounds are many, 9.1 and 9.7, 12.3 and 12.9, 6.3 and 6.5 ms.  N+(u) goes into a
// hash (slot = position in the sorted suffix, i.e. id order).  The waves
// walk the lists N+(v_i) of 64 slots i at a time, flattened over lanes: a
// hit j is a triangle (u, v_i, w_j); it updates t of the three edges and
// records the edge v_i -> w_j as bit j of row i of the bit matrix E (the
// graph induced on N+(u), union view).  4-cliques u < v_i < v_j < v_k then
// follow from AND-popcounts of rows:
//   K4_x(u) = sum_{i in P_x} sum_{j in E[i] & P_x} |E[i] & E[j] & P_x|
// with P_x the slots whose edge from u exists in version x (versions with
// equal P_x share one count).  Edges among N+(u) that are absent from some
// version are few; the triangles of E that contain such an edge absent from
// version x are removed from K4_x one by one (each once, at its first such
// edge in list order), or the edges are taken out of the matrix and K4_x
// counted for each version alone.  If the list overflows, the matrix is
// rebuilt per version instead.
constexpr int TL_EXC = 256;       // edges with flags tracked per vertex (twice as many above 128 slots)
constexpr int32_t EXC_DP = 1 << 14;  // largest out-degree they are tracked for

// Words of the triangular bit matrix of n slots with W words per full row:
// row i keeps only words (i >> 6) .. W - 1 (its bits j > i).
__host__ __device__ __forceinline__ int64_t tri_words(int64_t n, int64_t W) {
  const int64_t b = n >> 6;
  return n * W - (32 * b * (b - 1) + (n - 64 * b) * b);
}

template <int NV>
struct TriL {
  using TU = typename Fields<NV, 16>::T;  // per-slot triangle counts, 16-bit field per version
  unsigned long long* E;    // triangular row bitsets, tri_words(dp, W) words
  // word w >= (i >> 6) of row i is erow(i)[w]
  // (32 bits hold the index: a slot of 2^31 words would not fit the memory)
  __device__ __forceinline__ unsigned long long* erow(int32_t i) const {
    const int32_t b = i >> 6;
    return E + (uint32_t)(i * W - (32 * b * (b - 1) + (i - 64 * b) * b) - b);
  }
  unsigned long long* P;    // [NV][W] slot masks per version
  uint32_t* ids;            // [dp]
  int32_t* hkey;            // [H]
  uint32_t* hval;           // [H] slot | its flags
  int32_t hcap;             // slots of hkey / hval (a power of two)
  uint32_t* filt;           // [2^(27 - fsh)] bits of the ids in the table (wave_probe)
  int32_t fsh;
  uint32_t* queue;          // [256] per wave: entries that passed, then edges (k4_edges)
  TU* tuc;                  // [dp]
  int32_t xcap;             // entries of exc
  uint32_t* exc;            // [xcap] i << 18 | j << 4 | absence mask
  int32_t* nexc;            // [1]
  int32_t W;                // words per row
};

__device__ __forceinline__ bool bit_of(const unsigned long long* m, int32_t k) { return (m[k >> 6] >> (k & 63)) & 1ull; }

// One wave: slots g0 + gs * l (lane l) of N+(u), their out-lists walked
// together.  The slots of a vertex are dealt to the waves of the block in
// turn, so every wave gets a share whatever the out-degree.  only = 0: union
// matrix plus all triangle bookkeeping; only = x+1: matrix of version x alone.
template <int NV>
__device__ __forceinline__ void tri_large_probe(const CountArgs& A, const TriL<NV>& S, uint32_t hmask, int shift,
                                                int32_t g0, int32_t gs, int32_t dp, int only, int64_t& ent) {
  const RegionDev& R = A.R;
  const int l = lane_id();
  const int32_t i0 = g0 + gs * l;
  int64_t sb = 0;
  int32_t sl = 0;
  uint32_t fi = 0;
  if (i0 < dp) {
    const uint32_t xi = S.ids[i0];
    const uint32_t v = xi & GC_ID;
    fi = xi & GC_FLAGS;
    sb = R.roff[v] + R.rlow[v];
    sl = (int32_t)(R.roff[v + 1] - sb);
    if (only == 0) ent += sl;
  }
  using TU = typename TriL<NV>::TU;
  // a hit of list i (slot j with flags, jv) is the triangle (u, v_i, w_j)
  const HashLook hl{S.hkey, hmask, shift};
  wave_probe(R.rcol, sb, sl, S.filt, S.fsh, S.queue + (threadIdx.x >> 6) * 256,
             [&](int s, int64_t pos, uint32_t y, bool in) {
    const uint32_t fs = (uint32_t)__shfl((int32_t)fi, s);
    if (!in) return;
    const int p = hl.find(y & GC_ID);
    if (p < 0) return;
    const uint32_t jv = S.hval[p], fy = y & GC_FLAGS;
    const int32_t i = g0 + gs * s, j = (int32_t)(jv & GC_ID);
    unsigned long long* at = S.erow(i) + (j >> 6);
    if (only) {
      if (!absent_in(fy, only - 1)) atomicOr(at, 1ull << (j & 63));
      return;
    }
    atomicOr(at, 1ull << (j & 63));
    if (fy) {
      const int32_t e = atomicAdd(S.nexc, 1);
      if (e < S.xcap) S.exc[e] = ((uint32_t)i << 18) | ((uint32_t)j << 4) | (fy >> GC_VSHIFT);
    }
    const uint32_t pm = vpresent<NV>(fs | (jv & GC_FLAGS) | fy);
    if (!pm) return;
    t_add<NV>(R, pos, pm);
    const TU add = Fields<NV, 16>::spread(pm);
    atomicAdd(&S.tuc[j], add);
    // the hits of the first lane's list (in a dense graph: most of the wave)
    // add to the same word: one atomic for them
    const bool mine = i == __builtin_amdgcn_readfirstlane(i);
    TU tot = 0;
#pragma unroll
    for (int x = 0; x < NV; ++x) tot |= (TU)__popcll(__ballot(mine && ((pm >> x) & 1u))) << (16 * x);
    const uint64_t act = __ballot(mine);
    if (!mine) atomicAdd(&S.tuc[i], add);
    else if (lane_id() == __builtin_ctzll(act)) atomicAdd(&S.tuc[i], tot);
  });
}

// kv[x] += sum over i in P_x, j in E[i] & P_x of |E[i] & E[j] & P_x|, for the
// versions x of `vers` (one wave's rows).  Most bits of a row's words are 0:
// the edges i -> j are packed into a list first, and 64 of them at a time take a lane each, whose AND-popcounts serve every
// version.  With a lane per bit of a word and a pass per version (and the
// exceptions below searched slot by slot) k_tri_large<128> took 1.01 ms on a
// scale-18 graph with 5% of the edges in the batch, all tiers 81 ms at scale
// 22; now 0.54 and 70 ms.
//
// DENSE, the tiers above 512 slots, whose counts take longest in dense graphs:
// a word with at least K4_DENSE of its edges is not packed (row i and the
// first word are then the same for every lane), and ONE version alone, the
// usual case there, masks the words as they are read and keeps one sum.
// MEM, the matrix in memory (the global tier): the waves meet once per row
// each, as four waves that drift apart read 64 rows each, all that the vector
// cache holds, and in step the same ones (6.4e9 instead of 6.0e10 reads of the
// L2 for the complete graph of 3,000 vertices); and a dense word's lanes take
// row i, the same for all, from registers.  Whole counts with 20,000 edges in
// the batch, complete graphs of 1,500 and 3,000 vertices: a lane per bit
// throughout 84 ms and 1.54 s, every word packed 87 ms and 2.05 s, dense words
// by bit 74 ms and 1.74 s, waves in step 72 ms and 1.54 s, row i in registers
// 67 ms and 1.33 s.  (With the matrix in LDS, registers took 4% longer.)
constexpr int K4_DENSE = 48;

template <int NV, bool DENSE, bool MEM, bool ONE>
__device__ __forceinline__ void k4_edges_(const TriL<NV>& S, int32_t dp, int nwaves, int vers, int64_t (&kv)[NV]) {
  const int w = threadIdx.x >> 6, l = lane_id();
  const int32_t W = S.W;
  uint32_t* qi = S.queue + w * 256;
  uint32_t* qj = qi + 128;
  int32_t n = 0;  // listed edges
  const unsigned long long* Pm = S.P + (__ffs(vers) - 1) * W;  // ONE: the version's slots
  int64_t one = 0;
  auto edge = [&](int32_t i, int32_t j, int32_t q0) {
    const unsigned long long* Ei = S.erow(i);
    const unsigned long long* Ej = S.erow(j);
    if constexpr (ONE) {
      uint32_t c = 0;
      for (int32_t q = q0; q < W; ++q) c += (uint32_t)__popcll(Ei[q] & Ej[q] & Pm[q]);
      one += c;
      return;
    }
    uint32_t c[NV];
#pragma unroll
    for (int x = 0; x < NV; ++x) c[x] = 0;
    for (int32_t q = q0; q < W; ++q) {
      const unsigned long long e = Ei[q] & Ej[q];
#pragma unroll
      for (int x = 0; x < NV; ++x)
        if ((vers >> x) & 1) c[x] += (uint32_t)__popcll(e & S.P[x * W + q]);
    }
#pragma unroll
    for (int x = 0; x < NV; ++x)
      if (((vers >> x) & 1) && bit_of(S.P + x * W, i) && bit_of(S.P + x * W, j)) kv[x] += c[x];
  };
  auto run = [&](int32_t k) {
    const int32_t j = (int32_t)qj[k];
    edge((int32_t)qi[k], j, j >> 6);
  };
  // MEM: every wave takes as many turns, and a barrier in each
  for (int32_t i = w; (MEM ? i - w : i) < dp; i += nwaves) {
    if constexpr (MEM) __syncthreads();
    if ((MEM && i >= dp) || (ONE && !bit_of(Pm, i))) continue;
    const unsigned long long* Ei = S.erow(i);
    for (int32_t w0 = i >> 6; w0 < W; ++w0) {
      const unsigned long long word = ONE ? Ei[w0] & Pm[w0] : Ei[w0];
      const bool in = (word >> l) & 1ull;
      const uint64_t m = __ballot(in);
      if (!m) continue;
      if (DENSE && __popcll(m) >= K4_DENSE) {
        if constexpr (MEM && ONE) {
          const unsigned long long* Ej = S.erow(in ? w0 * 64 + l : i);
          uint32_t c = 0;
          for (int32_t b = w0; b < W; b += 64) {
            const int32_t words = min(64, W - b);
            const int64_t ei = l < words ? (int64_t)(Ei[b + l] & Pm[b + l]) : 0;
            for (int32_t k = 0; k < words; ++k) c += (uint32_t)__popcll((uint64_t)rdl64(ei, k) & Ej[b + k]);
          }
          one += in ? c : 0u;
        } else if (in) {
          edge(i, w0 * 64 + l, w0);
        }
        continue;
      }
      if (in) {
        const int32_t k = n + __popcll(m & lanemask_lt());
        qi[k] = (uint32_t)i;
        qj[k] = (uint32_t)(w0 * 64 + l);
      }
      n += __popcll(m);
      if (n >= 64) {
        n -= 64;
        wave_sync();
        run(n + l);
        wave_sync();
      }
    }
  }
  wave_sync();
  if (l < n) run(l);
  if constexpr (ONE) {
#pragma unroll
    for (int x = 0; x < NV; ++x) kv[x] += (vers >> x) & 1 ? one : 0;
  }
}

template <int NV, bool DENSE, bool MEM>
__device__ __forceinline__ void k4_edges(const TriL<NV>& S, int32_t dp, int nwaves, int vers, int64_t (&kv)[NV]) {
  if (DENSE && (vers & (vers - 1)) == 0) k4_edges_<NV, DENSE, MEM, true>(S, dp, nwaves, vers, kv);
  else k4_edges_<NV, DENSE, MEM, false>(S, dp, nwaves, vers, kv);
}

template <int NV, bool DENSE, bool MEM>
__device__ void tri_large_vertex(const CountArgs& A, const TriL<NV>& S, int64_t ub, int32_t dp,
                                 int64_t (&kacc)[NV], int64_t& ent) {
  const RegionDev& R = A.R;
  const int w = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const int32_t W = S.W;
  // load factor <= 1/4 where the table has room, else as low as it allows
  int H = 1;
  while (H < 4 * dp) H <<= 1;
  while (H > S.hcap) H >>= 1;
  const uint32_t hmask = (uint32_t)H - 1u;
  const int shift = 32 - log2i((uint32_t)H);
  for (int32_t k = threadIdx.x; k < dp; k += blockDim.x) { S.ids[k] = R.rcol[ub + k]; S.tuc[k] = 0; }
  for (int32_t k = threadIdx.x; k < H; k += blockDim.x) S.hkey[k] = -1;
  const int32_t fw = 1 << (27 - S.fsh);
  for (int32_t k = threadIdx.x; k < fw; k += blockDim.x) S.filt[k] = 0u;
  const int64_t ew = tri_words(dp, W);
  for (int64_t k = threadIdx.x; k < ew; k += blockDim.x) S.E[k] = 0ull;
  for (int32_t k = threadIdx.x; k < NV * W; k += blockDim.x) S.P[k] = 0ull;
  if (threadIdx.x == 0) *S.nexc = 0;
  __syncthreads();
  for (int32_t k = threadIdx.x; k < dp; k += blockDim.x) {
    const uint32_t x = S.ids[k];
    const uint32_t id = x & GC_ID;
    const uint32_t fh = hash32(id) >> S.fsh;
    atomicOr(&S.filt[fh >> 5], 1u << (fh & 31u));
    uint32_t h = hash32(id) >> shift;
    while (atomicCAS(&S.hkey[h], -1, (int32_t)id) != -1) h = (h + 1) & hmask;
    S.hval[h] = (uint32_t)k | (x & GC_FLAGS);
#pragma unroll
    for (int q = 0; q < NV; ++q)
      if (!absent_in(x, q)) atomicOr(&S.P[q * W + (k >> 6)], 1ull << (k & 63));
  }
  __syncthreads();
  if (threadIdx.x == 0) ent += dp;
  for (int32_t g0 = w; g0 < dp; g0 += nwaves * 64) tri_large_probe<NV>(A, S, hmask, shift, g0, nwaves, dp, 0, ent);
  __syncthreads();
  // more slots than an exception can name: as many exceptions as none could hold
  const int32_t ne = dp <= EXC_DP || *S.nexc == 0 ? *S.nexc : INT32_MAX;
  if (ne <= S.xcap && 4 * ne > (NV - 1) * dp) {
    // Many of them: per version, the bits of the absent edges are taken out of
    // E for its count and put back.  One by one each costs a few dozen
    // instructions per 64 slots, a further count about as much as dp / 4 of
    // them.  Scale 18 with 5% of the edges in the batch, <128> and <256>: 0.91
    // and 0.67 ms all one by one, 0.54 and 0.54 with this; four versions with
    // 0.5%: <256> 0.44 ms one by one, 0.54 with this from dp / 4 on.
    auto flip = [&](int x, bool out) {
      for (int32_t e = threadIdx.x; e < ne; e += blockDim.x) {
        const uint32_t ex = S.exc[e];
        const int32_t i = (int32_t)(ex >> 18), j = (int32_t)((ex >> 4) & 0x3FFFu);
        if (!((ex >> x) & 1u)) continue;
        unsigned long long* at = S.erow(i) + (j >> 6);
        if (out) atomicAnd(at, ~(1ull << (j & 63)));
        else atomicOr(at, 1ull << (j & 63));
      }
    };
    for (int x = 0; x < NV; ++x) {
      flip(x, true);
      __syncthreads();
      k4_edges<NV, DENSE, MEM>(S, dp, nwaves, 1 << x, kacc);
      __syncthreads();
      if (x < NV - 1) flip(x, false);
    }
  } else if (ne <= S.xcap) {
    // versions with the same slot mask share one count
    int64_t kv[NV];
    int same[NV], vers = 0;
#pragma unroll
    for (int x = 0; x < NV; ++x) {
      kv[x] = 0;
      same[x] = x;
#pragma unroll
      for (int y = 0; y < x; ++y) {
        bool eq = same[x] == x;
        for (int32_t q = 0; q < W && eq; ++q) eq = S.P[x * W + q] == S.P[y * W + q];
        if (eq) same[x] = y;
      }
      if (same[x] == x) vers |= 1 << x;
    }
    k4_edges<NV, DENSE, MEM>(S, dp, nwaves, vers, kv);
#pragma unroll
    for (int x = 1; x < NV; ++x)
#pragma unroll
      for (int y = 0; y < x; ++y)
        if (same[x] == y) kv[x] = kv[y];
    if (ne > 0) {
      // The exceptions by slot pair, in the probe hash table (not read again
      // for this vertex): key min << 16 | max, value the exception's index.
      // Pairs are unique (each found from its lower slot's list only).
      for (int32_t k = threadIdx.x; k < H; k += blockDim.x) S.hkey[k] = -1;
      __syncthreads();
      for (int32_t e = threadIdx.x; e < ne; e += blockDim.x) {
        const uint32_t ex = S.exc[e], a = ex >> 18, b = (ex >> 4) & 0x3FFFu;
        const uint32_t key = (a << 16) | b;  // a < b: found from the lower slot's list
        uint32_t h = hash32(key) >> shift;
        while (atomicCAS(&S.hkey[h], -1, (int32_t)key) != -1) h = (h + 1) & hmask;
        S.hval[h] = (uint32_t)e;
      }
      __syncthreads();
      // index of the exception on slot pair (a, b), or -1
      auto exc_of = [&](int32_t a, int32_t b) -> int32_t {
        const uint32_t key = ((uint32_t)min(a, b) << 16) | (uint32_t)max(a, b);
        uint32_t h = hash32(key) >> shift;
        for (;;) {
          const int32_t q = S.hkey[h];
          if (q == -1) return -1;
          if ((uint32_t)q == key) return (int32_t)S.hval[h];
          h = (h + 1) & hmask;
        }
      };
      // Triangles of E (inside P_x) holding an edge i -> j absent from version
      // x: the slots adjacent to both, 64 at a time.  Above i they are the words
      // of row i, below it bit i of their own rows.
      const int l = lane_id();
      for (int32_t e = w; e < ne; e += nwaves) {
        const uint32_t ex = S.exc[e];
        const int32_t i = (int32_t)(ex >> 18), j = (int32_t)((ex >> 4) & 0x3FFFu);
        int av = 0;
#pragma unroll
        for (int x = 0; x < NV; ++x)
          if (((ex >> x) & 1u) && bit_of(S.P + x * W, i) && bit_of(S.P + x * W, j)) av |= 1 << x;
        if (!av) continue;
        const unsigned long long* Ei = S.erow(i);
        const unsigned long long* Ej = S.erow(j);
        for (int32_t c = 0; c < W; ++c) {
          const int32_t k = 64 * c + l;
          unsigned long long mi = 0, mj = 0, pm = 0;
          if (c >= (i >> 6)) mi = Ei[c];
          if (c <= (i >> 6)) mi |= __ballot(k < i && bit_of(S.erow(min(k, i)), i));
          if (c >= (j >> 6)) mj = Ej[c];
          if (c <= (j >> 6)) mj |= __ballot(k < j && bit_of(S.erow(min(k, j)), j));
#pragma unroll
          for (int x = 0; x < NV; ++x)
            if ((av >> x) & 1) pm |= S.P[x * W + c];
          if (!((mi & mj & pm) >> l & 1ull)) continue;
          // count once: not where an earlier listed edge of this triangle is absent too
          uint32_t early = 0;
          const int32_t f1 = exc_of(i, k), f2 = exc_of(j, k);
          if (f1 >= 0 && f1 < e) early |= S.exc[f1];
          if (f2 >= 0 && f2 < e) early |= S.exc[f2];
#pragma unroll
          for (int x = 0; x < NV; ++x)
            if (((av >> x) & 1) && ((S.P[x * W + c] >> l) & 1ull) && !((early >> x) & 1u)) --kv[x];
        }
      }
    }
#pragma unroll
    for (int x = 0; x < NV; ++x) kacc[x] += kv[x];
  } else {
    // too many version-specific edges: rebuild E per version and count
    if (threadIdx.x == 0) atomicAdd(&A.bstats[BS_TRI_REBUILD], 1ull);
    for (int x = 0; x < NV; ++x) {
      __syncthreads();
      for (int64_t k = threadIdx.x; k < ew; k += blockDim.x) S.E[k] = 0ull;
      __syncthreads();
      for (int32_t g0 = w; g0 < dp; g0 += nwaves * 64) tri_large_probe<NV>(A, S, hmask, shift, g0, nwaves, dp, x + 1, ent);
      __syncthreads();
      k4_edges<NV, DENSE, MEM>(S, dp, nwaves, 1 << x, kacc);
    }
  }
  __syncthreads();
  for (int32_t k = threadIdx.x; k < dp; k += blockDim.x) {
    const typename TriL<NV>::TU c = S.tuc[k];
    if (c) {
      uint32_t cv[NV];
#pragma unroll
      for (int x = 0; x < NV; ++x) cv[x] = (uint32_t)Fields<NV, 16>::get(c, x);
      t_addv<NV>(R, ub + k, cv);
    }
  }
  __syncthreads();
}

// global-scratch slot layout (u64 words): E [tri_words(cap, W)] | P [NV*W] |
// tuc [cap] | then u32 words: exc [2 TL_EXC] | ids [cap] | hkey [4 cap] |
// hval [4 cap] | nexc [2]
template <int NV>
__host__ __device__ inline int64_t tri_slot_words64(int64_t cap) {
  const int64_t W = (cap + 63) / 64;
  return tri_words(cap, W) + NV * W + cap + TL_EXC + (cap + 4 * cap + 4 * cap + 2 + 1) / 2 + 8;
}

constexpr int pow2_at_least(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

// The vertices of work list L (out-degree at most CAP; CAP = 0 selects the
// global-memory scratch), taken one at a time from the queue whose head is
// qhead.
// Registers: the tiers up to 256 hide their latencies with 6 waves per SIMD (5
// with four versions, which spill below 96 registers); without the bound they
// took 17.8 against 13.3 ms (<256>) and 12.5 against 9.5 ms (<128>) at scale 22.
constexpr int TG_HASH = 8192;
template <int CAP, int THREADS, int NV>
__global__ __launch_bounds__(THREADS, CAP == 0 || CAP > 256 ? 4 : (NV == 2 ? 6 : 5)) void k_tri_large(CountArgs A, int L, unsigned long long* qhead) {
  const RegionDev& R = A.R;
  const int64_t n = (int64_t)A.c[C_LIST0 + L];
  const int32_t* list = A.lists + L * A.list_stride;
  __shared__ int64_t item_s;
  int cur_g = -1;
  int64_t kacc[NV];
  zerov<NV>(kacc);
  int64_t ent = 0;  // entries of N+(u) and of the lists probed (algorithmic reads)
  TriL<NV> S;
  using TU = typename TriL<NV>::TU;
  // CAP = 0: the hash in LDS up to TG_HASH / 2 slots, else in the scratch (a
  // lookup waits for its loads: 79 instead of 74 ms for the graph of 1,500)
  __shared__ int32_t tkey[CAP == 0 ? TG_HASH : 1];
  __shared__ uint32_t tval[CAP == 0 ? TG_HASH : 1];
  int32_t* gkey = nullptr;
  uint32_t* gval = nullptr;
  int32_t ghc = 0;
  if constexpr (CAP == 0) {
    // slot layout for capacity tri_cap (no slot is touched while tri_cap == 0)
    const int64_t cap = A.tri_cap > 0 ? A.tri_cap : 1;
    const int64_t W = (cap + 63) / 64;
    unsigned long long* base = A.tri_scratch + (int64_t)blockIdx.x * tri_slot_words64<NV>(cap);
    S.W = (int32_t)W;
    S.E = base;
    S.P = base + tri_words(cap, W);
    S.tuc = (TU*)(S.P + NV * W);
    S.exc = (uint32_t*)(S.P + NV * W + cap);
    S.xcap = 2 * TL_EXC;
    uint32_t* u32 = S.exc + 2 * TL_EXC;
    S.ids = u32;
    gkey = (int32_t*)(u32 + cap);
    gval = u32 + 5 * cap;
    S.nexc = (int32_t*)(u32 + 9 * cap);
    int32_t hc = 1;
    while (2 * hc <= 4 * cap) hc <<= 1;
    ghc = hc;
    __shared__ uint32_t filt[8192];
    __shared__ uint32_t queue[THREADS / 64 * 256];
    S.filt = filt;
    S.fsh = 14;
    S.queue = queue;
  } else {
    constexpr int CW = CAP / 64;
    constexpr int HC = CAP <= 1024 ? pow2_at_least(4 * CAP) : pow2_at_least(CAP);
    // 64 filter bits per slot, 32 in the last tier (LDS)
    constexpr int FSH = CAP <= 128 ? 19 : CAP <= 256 ? 18 : CAP <= 512 ? 17 : CAP <= 1024 ? 16 : 17;
    __shared__ uint32_t filt[1 << (27 - FSH)];
    __shared__ uint32_t queue[THREADS / 64 * 256];
    __shared__ unsigned long long E[32 * CW * CW + 32 * CW];  // tri_words(CAP, CW)
    __shared__ unsigned long long P[NV * CW];
    __shared__ uint32_t ids[CAP];
    __shared__ TU tuc[CAP];
    __shared__ int32_t hkey[HC];
    __shared__ uint32_t hval[HC];
    constexpr int XC = CAP > 128 ? 2 * TL_EXC : TL_EXC;
    static_assert(CAP <= EXC_DP, "exceptions hold slots in 14 bits");
    __shared__ uint32_t exc[XC];
    __shared__ int32_t nexc;
    S.E = E; S.P = P; S.ids = ids; S.tuc = tuc; S.hkey = hkey; S.hval = hval; S.exc = exc; S.nexc = &nexc;
    S.filt = filt; S.fsh = FSH; S.queue = queue;
    S.xcap = XC;
    S.W = CW;
    S.hcap = HC;
  }
  while (true) {
    __syncthreads();  // every thread has read the previous item before it is replaced
    if (threadIdx.x == 0) item_s = (int64_t)atomicAdd(qhead, 1ull);
    __syncthreads();
    const int64_t it = item_s;
    if (it >= n) break;
    const int32_t u = list[it];
    const int64_t ub = R.roff[u] + R.rlow[u];
    const int32_t dp = (int32_t)(R.roff[u + 1] - ub);
    if (CAP != 0 && dp > CAP) {  // cannot happen: the lists are cut at the tier capacities
      if (threadIdx.x == 0) atomicAdd(&A.bstats[BS_ERR], 1ull);
      continue;
    }
    if (CAP == 0 && dp > A.tri_cap) {  // scratch too small: the host counts again with more
      if (threadIdx.x == 0) atomicAdd(&A.bstats[BS_RETRY], 1ull);
      continue;
    }
    if (CAP == 0 && threadIdx.x == 0) atomicAdd(&A.bstats[BS_TRI_GLOBAL], 1ull);
    const int g = A.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_K4, kacc);
      cur_g = g;
    }
    if constexpr (CAP != 0) {
      S.W = (dp + 63) / 64;
    } else {
      const bool lds = 2 * dp <= TG_HASH;
      S.hkey = lds ? tkey : gkey;
      S.hval = lds ? tval : gval;
      S.hcap = lds ? TG_HASH : ghc;
    }
    tri_large_vertex<NV, (CAP == 0 || CAP > 512), CAP == 0>(A, S, ub, dp, kacc, ent);
  }
  if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_K4, kacc);
  ent = wave_sum64(ent);
  if (lane_id() == 0 && ent) atomicAdd(&A.bstats[BS_TRI_E], (unsigned long long)ent);
}

template <int NV> constexpr int tl_max() { return TRI_LDS_MAX; }

// ------------------------------------------------------------ edge pass
// After all triangles, per upper entry u -> w present in version x, with
// t = t_x(u, w) and d = d_x:
//   S2  += (d_u - 1)(d_w - 1)      DIA += C(t, 2)
//   T3  += t                        (= 3 T)
//   PAW2 += t (d_u + d_w - 4)       (= 2 N_paw: a triangle on the edge plus a
//                                    pendant edge at one of its ends)
// One thread per entry: each workgroup takes one contiguous range of the
// entries, consecutive lanes read consecutive entries (row ids come from the
// region build), and a lane meets a new graph of a pool only at a graph
// boundary of its range, so its per-graph sums are flushed rarely.
template <int NV>
__device__ __forceinline__ void edge_flush_lane(unsigned long long* sig, int g, int64_t (&acc)[4][NV]) {
  const int keys[4] = {SG_S2, SG_DIA, SG_T, SG_PAW};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int x = 0; x < NV; ++x) {
      if (acc[k][x]) atomicAdd(&sig[SIG_IDX(g, x, keys[k])], (unsigned long long)acc[k][x]);
      acc[k][x] = 0;
    }
}

template <int NV>
__global__ __launch_bounds__(256) void k_edge_pass(CountArgs A) {
  const RegionDev& R = A.R;
  const int64_t E = (int64_t)A.c[C_ER];
  int cur_g = -1;
  int64_t acc[4][NV];  // s2, dia, t3, paw2 per version
#pragma unroll
  for (int k = 0; k < 4; ++k) zerov<NV>(acc[k]);
  const int64_t per = ((E + gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
  const int64_t end = min(E, per * (blockIdx.x + 1));
  for (int64_t p = per * blockIdx.x + threadIdx.x; p < end; p += 256) {
    const uint32_t x = R.rcol[p];
    const uint32_t wv = x & GC_ID;
    const int32_t u = R.rrow[p];
    if (wv <= (uint32_t)u) continue;
    const int g = A.gid[u];
    if (g != cur_g) {
      if (cur_g >= 0) edge_flush_lane<NV>(A.sig, cur_g, acc);
      cur_g = g;
    }
    const uint32_t pm = vpresent<NV>(x);
    int64_t t[NV];
    int32_t du[NV], dw[NV];
    t_read<NV>(R, p, t);
    d_read<NV>(R, u, du);
    d_read<NV>(R, wv, dw);
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      if (!((pm >> q) & 1u)) continue;
      acc[0][q] += (int64_t)(du[q] - 1) * (dw[q] - 1);
      acc[1][q] += c2(t[q]);
      acc[2][q] += t[q];
      acc[3][q] += t[q] * (du[q] + dw[q] - 4);
    }
  }
  // Sums of a wave that worked for one graph (or none) go through a block
  // reduction: one atomic per value and block when every wave of the block
  // has the same graph (many atomics on the few words of one graph would
  // queue at one L2 channel), else one per value and wave.  Lanes that saw
  // several graphs flush on their own.
  __shared__ int64_t red[4][4 * NV];
  __shared__ int wg[4];
  const int wv_ = threadIdx.x >> 6;
  int g0 = __shfl(cur_g, 0);
  for (int l = 1; l < 64 && g0 < 0; ++l) g0 = __shfl(cur_g, l);
  const bool wuni = __ballot(cur_g == g0 || cur_g < 0) == ~0ull;
  if (!wuni && cur_g >= 0) edge_flush_lane<NV>(A.sig, cur_g, acc);
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int64_t v = wave_sum64(wuni ? acc[k][q] : 0);
      if (lane_id() == 0) red[wv_][k * NV + q] = v;
    }
  if (lane_id() == 0) wg[wv_] = wuni ? g0 : -1;
  __syncthreads();
  if (threadIdx.x < 4 * NV) {
    const int keys[4] = {SG_S2, SG_DIA, SG_T, SG_PAW};
    const int k = threadIdx.x / NV, q = threadIdx.x % NV;
    int gb = -1;
    bool same = true;
    for (int w = 0; w < 4; ++w) {
      if (wg[w] < 0) continue;
      if (gb < 0) gb = wg[w];
      else if (wg[w] != gb) same = false;
    }
    if (same) {
      int64_t v = 0;
      for (int w = 0; w < 4; ++w) v += red[w][threadIdx.x];
      if (gb >= 0 && v) atomicAdd(&A.sig[SIG_IDX(gb, q, keys[k])], (unsigned long long)v);
    } else {
      for (int w = 0; w < 4; ++w)
        if (wg[w] >= 0 && red[w][threadIdx.x])
          atomicAdd(&A.sig[SIG_IDX(wg[w], q, keys[k])], (unsigned long long)red[w][threadIdx.x]);
    }
  }
}

// ------------------------------------------------------------ 4-cycles
// Segment of the wedges through u for apex v: entries of row u below v.
__device__ __forceinline__ void c4_segment(const RegionDev& R, uint32_t v, uint32_t u, int64_t& sb, int32_t& sl) {
  sb = R.roff[u];
  const int32_t L = (int32_t)(R.roff[u + 1] - sb);
  sl = lower_bound_id(R.rcol + sb, L, v);
}

// Wave-flattened walk over the wedges (v, u, w) for the lower neighbours
// u in positions [g0, g0 + 64) of row v; calls f(w, flags of both entries).
template <class F>
__device__ __forceinline__ void c4_group(const RegionDev& R, uint32_t v, int64_t rb, int32_t nlow, int32_t g0, F f) {
  const int l = lane_id();
  const int32_t q = g0 + l;
  int64_t sb = 0;
  int32_t sl = 0;
  uint32_t fvu = 0;
  if (q < nlow) {
    const uint32_t x = R.rcol[rb + q];
    fvu = x & GC_FLAGS;
    c4_segment(R, v, x & GC_ID, sb, sl);
  }
  wave_walk(R.rcol, sb, sl, fvu, [&](int, int64_t, uint32_t fs, uint32_t y) { f(y & GC_ID, fs | (y & GC_FLAGS)); });
}

constexpr int C4S_SLOTS = 512;
constexpr int C4S_WAVES = 4;

// c(v, w) <= wedges of v <= 4096 in the small and mid tiers: 16-bit fields
template <int NV>
__global__ __launch_bounds__(256) void k_c4_small(CountArgs A) {
  using F = Fields<NV, 16>;
  using T = typename F::T;
  __shared__ int32_t hkey[C4S_WAVES][C4S_SLOTS];
  __shared__ T hcnt[C4S_WAVES][C4S_SLOTS];
  const int w = threadIdx.x >> 6, l = lane_id();
  const RegionDev& R = A.R;
  const int64_t n = (int64_t)A.c[C_LIST0 + L_C4_S];
  const int32_t* list = A.lists + L_C4_S * A.list_stride;
  int cur_g = -1;
  int64_t acc[NV];
  zerov<NV>(acc);
  for (int s = l; s < C4S_SLOTS; s += 64) { hkey[w][s] = -1; hcnt[w][s] = 0; }
  wave_sync();
  // a fixed stride: the vertices of this tier are uniformly light (a shared
  // counter costs more than it balances)
  for (int64_t it = (int64_t)blockIdx.x * C4S_WAVES + w; it < n; it += (int64_t)gridDim.x * C4S_WAVES) {
    const int32_t v = list[it];
    const int g = A.gid[v];
    if (g != cur_g) { if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc); cur_g = g; }
    const int64_t rb = R.roff[v];
    const int32_t nlow = R.rlow[v];
    int32_t* hk = hkey[w];
    T* hc = hcnt[w];
    for (int32_t g0 = 0; g0 < nlow; g0 += 64)
      c4_group(R, (uint32_t)v, rb, nlow, g0, [&](uint32_t wid, uint32_t fl) {
        const uint32_t pm = vpresent<NV>(fl);
        if (pm) hash_add<T>(hk, hc, C4S_SLOTS - 1, 23, wid, F::spread(pm));
      });
    wave_sync();
    for (int s = l; s < C4S_SLOTS; s += 64) {
      if (hk[s] != -1) {
        const T c = hc[s];
#pragma unroll
        for (int x = 0; x < NV; ++x) acc[x] += c2(F::get(c, x));
        hk[s] = -1; hc[s] = 0;
      }
    }
    wave_sync();
  }
  if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc);
}

constexpr int C4M_SLOTS = 8192;

template <int NV>
__global__ __launch_bounds__(256) void k_c4_mid(CountArgs A) {
  using F = Fields<NV, 16>;
  using T = typename F::T;
  __shared__ int32_t hkey[C4M_SLOTS];
  __shared__ T hcnt[C4M_SLOTS];
  const int w = threadIdx.x >> 6;
  const RegionDev& R = A.R;
  const int64_t n = (int64_t)A.c[C_LIST0 + L_C4_M];
  const int32_t* list = A.lists + L_C4_M * A.list_stride;
  int cur_g = -1;
  int64_t acc[NV];
  zerov<NV>(acc);
  for (int s = threadIdx.x; s < C4M_SLOTS; s += blockDim.x) { hkey[s] = -1; hcnt[s] = 0; }
  __syncthreads();
  // first vertex by block index (no atomic: blocks without one leave at
  // once), later ones from the shared counter counting on from the grid size
  __shared__ int64_t item_s;
  for (int64_t it = blockIdx.x; it < n; it = item_s) {
    const int32_t v = list[it];
    const int g = A.gid[v];
    if (g != cur_g) { if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc); cur_g = g; }
    const int64_t rb = R.roff[v];
    const int32_t nlow = R.rlow[v];
    for (int32_t g0 = w * 64; g0 < nlow; g0 += 64 * 4)
      c4_group(R, (uint32_t)v, rb, nlow, g0, [&](uint32_t wid, uint32_t fl) {
        const uint32_t pm = vpresent<NV>(fl);
        if (pm) hash_add<T>(hkey, hcnt, C4M_SLOTS - 1, 19, wid, F::spread(pm));
      });
    __syncthreads();
    for (int s = threadIdx.x; s < C4M_SLOTS; s += blockDim.x) {
      if (hkey[s] != -1) {
        const T c = hcnt[s];
#pragma unroll
        for (int x = 0; x < NV; ++x) acc[x] += c2(F::get(c, x));
        hkey[s] = -1; hcnt[s] = 0;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) item_s = (int64_t)gridDim.x + (int64_t)atomicAdd((unsigned long long*)(A.c + C_QC4M), 1ull);
    __syncthreads();
  }
  if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc);
}

// Large tier: one workgroup per hub v at a time, hubs in decreasing order of
// wedge work.  The opposite vertices w < v are taken in windows of ids from
// v downwards, each with dense LDS counters: one field per w for the wedges
// present in every version (8 bits where no row of the window exceeds 255
// entries, else 16 bits while c(v, w) <= 65535 can be guaranteed, else 32),
// the other wedges in per-version global counters.  Hits concentrate just
// below v because ids are a degree order and a wedge reaches w with odds
// growing with deg w.  Once a window is sparse, all wedges below it go to
// the global counters (one array per resident workgroup, with a touched
// list).  Each lower neighbour u keeps a cursor in its row, starting at v's
// position, and walks it backwards window by window, so rows are read about
// once.  Four versions with 32-bit fields would not fit a 64-bit counter:
// such hubs are walked twice, for versions 0-1 and 2-3.
constexpr int C4W_WIN = 18432;  // 144 KB of 64-bit words
constexpr int C4W_T = 1024;
constexpr int C4_BLK_LOG = 10;  // ids per entry of the row-length maxima: 1024
constexpr int C4_BLK = 1 << C4_BLK_LOG;

struct C4Chunk {
  long long red[C4W_T / 64][2];
};

struct C4Smem {
  unsigned long long win[C4W_WIN];
  C4Chunk C;
  int64_t item;
  int64_t cut[2];
  int32_t nt;
};

// block maximum (all threads call; result valid in every thread)
__device__ __forceinline__ int32_t block_max32(C4Chunk& C, int32_t x) {
  const int wv = threadIdx.x >> 6;
  x = wave_max32(x);
  if (lane_id() == 0) C.red[wv][0] = x;
  __syncthreads();
  x = 0;
  for (int k = 0; k < C4W_T / 64; ++k) x = max(x, (int32_t)C.red[k][0]);
  __syncthreads();
  return x;
}

// block sum of two values (all threads call; result valid in every thread)
__device__ __forceinline__ void block_sum2(C4Chunk& C, long long& x, long long& y) {
  const int t = threadIdx.x, wv = t >> 6;
  x = wave_sum64(x); y = wave_sum64(y);
  if (lane_id() == 0) { C.red[wv][0] = x; C.red[wv][1] = y; }
  __syncthreads();
  x = 0; y = 0;
  for (int k = 0; k < C4W_T / 64; ++k) { x += C.red[k][0]; y += C.red[k][1]; }
  __syncthreads();
}

// Walk the wedges (v, u_q, w) for q in [0, nlow) with w in row u_q at
// positions [urow[q] + p0(q), urow[q] + p1(q)); f(w, flags of both entries).
// Thread q takes u_q: short slices (the common case: u_q has few entries in
// the id range) are walked by their own thread, long ones by their whole
// wave, one at a time (wave_walk).
constexpr int32_t C4W_LANE = 128;  // entries a thread walks itself

template <class P0, class P1, class F>
__device__ __forceinline__ void c4_block_walk(const RegionDev& R, int64_t rb, int32_t nlow, const int64_t* urow,
                                              P0 p0f, P1 p1f, F f) {
  const int t = threadIdx.x;
  for (int32_t c0 = 0; c0 < nlow; c0 += C4W_T) {
    const int32_t q = c0 + t;
    int64_t sb = 0;
    int32_t sl = 0;
    uint32_t fl = 0;
    int32_t p0 = 0, p1 = 0;
    if (q < nlow) { p0 = p0f(q); p1 = p1f(q); }
    if (p1 > p0) {
      sb = urow[q] + p0;
      fl = R.rcol[rb + q] & GC_FLAGS;
      if (p1 - p0 <= C4W_LANE) {
        const int32_t len = p1 - p0;
        for (int32_t k = 0; k < len; k += 4) {  // four loads in flight
          uint32_t y[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) y[u] = k + u < len ? R.rcol[sb + k + u] : 0u;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (k + u < len) f(y[u] & GC_ID, fl | (y[u] & GC_FLAGS));
        }
      } else {
        sl = p1 - p0;
      }
    }
    if (__ballot(sl > 0))
      wave_walk(R.rcol, sb, sl, fl, [&](int, int64_t, uint32_t fs, uint32_t y) { f(y & GC_ID, fs | (y & GC_FLAGS)); });
  }
  __syncthreads();
}

// sum over each group of LANES (4 or 16) consecutive lanes
template <int LANES>
__device__ __forceinline__ int32_t lanes_sum(int32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);  // quad_perm [1, 0, 3, 2]
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);  // quad_perm [2, 3, 0, 1]
  if constexpr (LANES == 16) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, true);  // row_ror:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);  // row_ror:8
  }
  return x;
}

// One window of ids [lo, lo + wsz) of hub v: every lower neighbour u_q walks
// its row backwards from its cursor while the ids stay >= lo and leaves the
// cursor at the first position below the window, so the slice is read once
// and no search precedes it.  wc: the window's counters (FW bits each), cf:
// the flags of an entry that counts there; slow(take, id, flags of both
// entries) gets the others.  wtot += entries walked, rest += entries left below
// the window (per thread).
//
// An entry y counts in the window exactly when y - (lo | cf) is below wsz as
// an unsigned number: one subtract and one compare test the range and the
// flags, entries past the cursor included (their ids are lo + wsz or more).
// What bounds it is the latency of the rows' loads: 144 KB of counters leave
// one workgroup per CU.  So the lanes read adjacent aligned 16-byte groups of
// a row, four lanes a row for its first C4W_SHORT entries, then 16 lanes a
// row, and each step's groups are loaded one step ahead.  (A lane per row for
// 128 entries, then a gallop and the whole wave, took 100.5 ms at scale 22;
// this 86, at 3.5 TB/s of lines from beyond the L2s for 1.6e11 bytes of
// entries.  Unrolling the slow path costs more than it gives: beyond 128
// registers the walk spills.)
constexpr int32_t C4W_SHORT = 64;

// one more in the counter of FW bits at offset o (FW = 0: 2^sh of them a word)
template <int FW>
__device__ __forceinline__ void window_add(uint32_t* wc, uint32_t o, int sh = 0) {
  if constexpr (FW == 0) { atomicAdd(&wc[o >> sh], 1u << ((o << (5 - sh)) & 31u)); return; }
  if constexpr (FW == 8) atomicAdd(&wc[o >> 2], 1u << ((o << 3) & 31u));
  else if constexpr (FW == 16) atomicAdd(&wc[o >> 1], 1u << ((o << 4) & 31u));
  else atomicAdd(&wc[o], 1u);
}

// LANES lanes walk the row at R.rcol + base (cursor k, flags of its own entry
// fl) for at most `steps` steps of 4 LANES entries; k moves to the first
// position not taken.  True while the row has more entries in the window.
// The same base, k, fl on the lanes of a group; all lanes of the wave call it.
template <int LANES, int FW, class S>
__device__ __forceinline__ bool window_row(const uint32_t* __restrict__ rcol, int64_t base, int32_t& k, uint32_t fl,
                                           bool open, int32_t steps, uint32_t lo, uint32_t wsz, uint32_t cf,
                                           uint32_t* wc, int sh, S& slow) {
  const int32_t gl = (int32_t)threadIdx.x & (LANES - 1);
  const uint32_t lob = lo | cf;
  const uint32_t* row = rcol + base;
  const int32_t a0 = (int32_t)(base & 3);  // row start within its 16-byte group
  // first entry of the topmost group: the one holding position k - 1; this
  // lane's group is the gl-th below it
  int32_t g0 = ((k - 1 + a0) & ~3) - a0, top = k - 1;
  uint4 y = make_uint4(cf, cf, cf, cf);
  if (open && g0 - 4 * gl > -4) y = *(const uint4*)(row + (g0 - 4 * gl));
  for (int32_t step = 0; step < steps && __ballot(open); ++step) {
    const int32_t g = g0 - 4 * gl;
    const bool mine = open && g > -4;
    uint4 yn = make_uint4(cf, cf, cf, cf);  // the next step's, if this one is taken whole
    if (open && g - 4 * LANES > -4) yn = *(const uint4*)(row + (g - 4 * LANES));
    const bool odd = mine && (((y.x ^ cf) | (y.y ^ cf) | (y.z ^ cf) | (y.w ^ cf) | (fl ^ cf)) & GC_FLAGS) != 0u;
    int32_t took = 0;
    if (__ballot(odd) == 0ull) {
      uint32_t o[4] = {y.x - lob, y.y - lob, y.z - lob, y.w - lob};
      if (step == 0) {  // entries past the cursor may be another row's
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = g + u > top ? 0xFFFFFFFFu : o[u];
      }
      if (__ballot(g < 0)) {  // and those before the row's start
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = g + u < 0 ? 0xFFFFFFFFu : o[u];
      }
      if (mine) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (o[u] < wsz) {
            window_add<FW>(wc, o[u], sh);
            ++took;
          }
      }
    } else {  // entries in the batch somewhere in the step
#pragma unroll 1
      for (int u = 0; u < 4; ++u) {
        const uint32_t e = u == 0 ? y.x : (u == 1 ? y.y : (u == 2 ? y.z : y.w)), id = e & GC_ID;
        const uint32_t f = fl | (e & GC_FLAGS);
        const bool in = mine && g + u >= 0 && g + u <= top && id >= lo;
        if (in) {
          ++took;
          if (f == cf) window_add<FW>(wc, id - lo, sh);
        }
        slow(in && f != cf, id, f);
      }
    }
    took = lanes_sum<LANES>(took);
    // entries the groups hold of [0, top]: all taken, and more below?
    const int32_t low = g0 - 4 * (LANES - 1);
    if (open) {
      k = top + 1 - took;
      open = low > 0 && k == low;
      top = low - 1;
      g0 = low - 4;
    }
    y = yn;
  }
  return open;
}

template <int FW, class S>
__device__ __forceinline__ void c4_window_walk(const RegionDev& R, int64_t rb, int32_t nlow, const int64_t* urow,
                                               int32_t* ucur, uint32_t lo, uint32_t wsz, uint32_t cf, uint32_t* wc,
                                               int sh, S slow, long long& wtot, long long& rest) {
  const int32_t l = lane_id();
  for (int32_t c0 = 0; c0 < nlow; c0 += C4W_T / 4) {
    const int32_t q = c0 + ((int32_t)threadIdx.x >> 2);
    uint32_t fl = cf;
    int32_t c = 0, k = 0;  // positions [k, c) are walked
    int64_t base = 0;
    if (q < nlow) {
      c = k = ucur[q];
      base = urow[q];
      fl = R.rcol[rb + q] & GC_FLAGS;
    }
    const bool open = window_row<4, FW>(R.rcol, base, k, fl, k > 0, C4W_SHORT / 16, lo, wsz, cf, wc, sh, slow);
    // rows that go on: four at a time, 16 lanes each
    for (uint64_t m = __ballot(open && (l & 3) == 0); m;) {
      int src = -1;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = m ? __builtin_ctzll(m) : -1;
        m &= m - 1;  // (0 stays 0)
        if ((l >> 4) == r) src = at;
      }
      const int from = max(src, 0);
      const int64_t b2 = __shfl(base, from);
      int32_t k2 = __shfl(k, from);
      const uint32_t f2 = (uint32_t)__shfl((int32_t)fl, from);
      (void)window_row<16, FW>(R.rcol, b2, k2, f2, src >= 0, 1 << 30, lo, wsz, cf, wc, sh, slow);
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // the cursor goes back to the row's quad
        const int to = __shfl(src, 16 * r);
        const int32_t kr = __shfl(k2, 16 * r);
        if (to >= 0 && (l >> 2) == (to >> 2)) k = kr;
      }
    }
    if ((l & 3) == 0 && q < nlow) {
      ucur[q] = k;
      wtot += c - k;
      rest += k;
    }
  }
}

// Pair sums of one 16-byte piece of single-field window counters of FB bits:
// s += c(c - 1) for every counter c, with no branch on zero counters.  The
// scan of a window is as long as a few thousand wedges' walk, and there are
// 40 windows per million wedges at scale 22: sums of squares and of counters
// by dot products (a word of four 8-bit counters in two instructions).
template <int FB>
__device__ __forceinline__ void window_pairs(const uint4 q, uint64_t& s) {
  const uint32_t wv[4] = {q.x, q.y, q.z, q.w};
  if constexpr (FB == 8) {
    uint32_t sq = 0, sm = 0;  // at most 16 x 255^2
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      sq = __builtin_amdgcn_udot4(wv[k], wv[k], sq, false);
      sm = __builtin_amdgcn_udot4(wv[k], 0x01010101u, sm, false);
    }
    s += sq - sm;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (FB == 16) {
        const uint32_t a = wv[k] & 0xFFFFu, b = wv[k] >> 16;
        s += (uint64_t)(a * (a - 1u));  // < 2^32 for a < 2^16, and 0 for a = 0
        s += (uint64_t)(b * (b - 1u));
      } else {
        s += (uint64_t)wv[k] * (uint64_t)(wv[k] - 1u);
      }
    }
  }
}

// One hub v, versions [vsh, vsh + NF) of an NV-version pass.  The window
// counts, per opposite vertex w, the wedges present in exactly the reference
// versions (c_A(w), one field of FBW bits, or of 8 bits over twice the ids
// where every row of the window's blocks has at most 255 entries, which
// bounds c_A; the reference set M is every
// version, or every version but 0 when version 0 is the empty graph); the
// other wedges (few: they hold a flagged entry) go to the block's global
// counters (e_x(w) per version x, one u64 of NF fields of 64 / NF bits, by
// atomics whose result nobody waits for, with w listed once per wedge, or
// the whole id range read back when the list would outgrow it).  With
// c_x = [x in M] c_A + e_x,
//   sum_w C(c_x(w), 2) = [x in M] sum_w C(c_A(w), 2)
//                        + sum_{w with exceptions} ([x in M] c_A e_x + C(e_x, 2)),
// so one scan of the window serves every version of M and the exceptions add
// the rest.  The tail uses the same global counters.  The window and the
// global counters are clear on entry and on return (each pass clears what it
// read).
template <int NV, int NF, int FBW>
__device__ void c4_hub(const CountArgs& A, C4Smem& S, int32_t v, int64_t top, int64_t bot, int vsh,
                       int64_t (&acc)[NV], int64_t& tail_) {
  using TFd = Fields<NF, 64 / NF>;
  constexpr int IPW = 32 / FBW;  // ids per 32-bit window word
  const RegionDev& R = A.R;
  const int t = threadIdx.x;
  unsigned long long* cnt = A.c4_dense + (int64_t)blockIdx.x * A.N;
  int32_t* touch = A.c4_touch + (int64_t)blockIdx.x * A.N;
  int64_t* urow = A.c4_cur + (int64_t)blockIdx.x * 2 * A.c4_maxlow;
  int32_t* ucur = (int32_t*)(urow + A.c4_maxlow);
  const int64_t rb = R.roff[v];
  const int32_t nlow = R.rlow[v];
  const uint32_t fmask = (1u << NF) - 1u;
  const uint32_t ref = (A.c4_ref >> vsh) & fmask;
  const int64_t ws = (int64_t)A.c4_win * 2 * IPW;  // ids per window
  uint32_t* wc = (uint32_t*)S.win;
  // field layout of the current window: 2^sh ids of fw bits per 32-bit word
  int sh = FBW == 16 ? 1 : 0, fw = FBW;
  auto count_of = [&](uint32_t o) -> uint32_t {  // c_A of the id at offset o in the window
    const uint32_t im = (1u << sh) - 1u;
    return (uint32_t)(((uint64_t)wc[o >> sh] >> (fw * (o & im))) & ((1ull << fw) - 1ull));
  };
  if (t == 0) S.nt = 0;
  for (int32_t q = t; q < nlow; q += C4W_T) {
    const int64_t ub = R.roff[R.rcol[rb + q] & GC_ID];
    int32_t c = R.vpos[rb + q];
    if (top < v) c = lower_bound_id(R.rcol + ub, c, (uint32_t)top);
    urow[q] = ub;
    ucur[q] = c;
  }
  __syncthreads();
  int64_t hi = top;
  while (hi > bot) {
    int64_t wsz = ws;
    sh = FBW == 16 ? 1 : 0;
    fw = FBW;
    if constexpr (FBW == 16) {
      // 8-bit fields over twice the ids when c(v, w) <= 255: v has no more
      // lower neighbours, or no row there is longer
      int32_t m = nlow;
      if (nlow > 255) {
        const int64_t lo8 = hi - 2 * ws > bot ? hi - 2 * ws : bot;
        const int64_t b0 = lo8 >> C4_BLK_LOG, b1 = (hi - 1) >> C4_BLK_LOG;
        m = 0;
        for (int64_t b = b0 + t; b <= b1; b += C4W_T) m = max(m, A.c4_blk[b]);
        m = block_max32(S.C, m);
      }
      if (m <= 255) { sh = 2; fw = 8; wsz = 2 * ws; }
    }
    const uint32_t lo = (uint32_t)(hi - wsz > bot ? hi - wsz : bot);
    const int32_t wcap = (int32_t)(hi - lo);  // list capacity: ids of the window (<= N)
    if (t == 0) {
      atomicAdd(&A.bstats[BS_C4_SEARCH], (unsigned long long)nlow);
      atomicAdd(&A.bstats[BS_C4_WINDOWS], 1ull);
    }
    long long wtot = 0, rest = 0;
    // the window walk with the field layout as constants (8-bit fields, or FBW)
    // wedges with an entry in the batch, on the lanes with `take` (all lanes call it)
    auto other = [&](bool take, uint32_t wid, uint32_t fl) {
      const uint32_t sub = (vpresent<NV>(fl) >> vsh) & fmask;
      if (take && sub == ref) {
        const uint32_t o = wid - lo;
        window_add<0>(wc, o, sh);
      }
      const bool some = take && sub != 0u && sub != ref;  // present in some versions only
      const uint64_t m = __ballot(some);
      if (!m) return;
      // no wait for the global atomic: the id is listed once per
      // exception wedge (while the list is shorter than the window)
      int32_t at = 0;
      if (lane_id() == 0) at = atomicAdd(&S.nt, (int32_t)__popcll(m));
      at = rdl32(at, 0) + (int32_t)__popcll(m & lanemask_lt());
      if (some) {
        atomicAdd(&cnt[wid], (unsigned long long)TFd::spread(sub));
        if (at < wcap) touch[at] = (int32_t)wid;
      }
    };
    // flags of the wedges the window counts (versions outside this walk's
    // differing send an entry through other(), which counts it all the same)
    const uint32_t cf = ((~ref & fmask) << vsh) << GC_VSHIFT;
    auto walk = [&](auto fwc) {
      c4_window_walk<decltype(fwc)::value>(R, rb, nlow, urow, ucur, lo, (uint32_t)wcap, cf, wc, sh, other, wtot, rest);
    };
    // (four versions: one copy of the walk for either width, to stay within the registers)
    if constexpr (NV == 4) walk(std::integral_constant<int, 0>{});
    else if (fw == 8) walk(std::integral_constant<int, 8>{});
    else walk(std::integral_constant<int, FBW>{});
    block_sum2(S.C, wtot, rest);  // also orders the window's counter updates before the passes below
    if (const int32_t nt = S.nt) {  // the window's exceptions
      auto one = [&](int32_t k, unsigned long long e) {
        const int64_t c = (int64_t)count_of((uint32_t)k - lo);
#pragma unroll
        for (int x = 0; x < NF; ++x) {
          const int64_t ex = TFd::get(e, x);
          acc[vsh + x] += ((ref >> x) & 1u ? c * ex : 0) + c2(ex);
        }
      };
      if (nt <= wcap) {
        // an id listed several times: the first exchange takes its counter
        for (int32_t q = t; q < nt; q += C4W_T) {
          const int32_t k = touch[q];
          const unsigned long long e = atomicExch(&cnt[k], 0ull);
          if (e) one(k, e);
        }
      } else {
        // more exception wedges than ids in the window: every counter of it
        for (int64_t k = lo + t; k < hi; k += C4W_T) {
          const unsigned long long e = __hip_atomic_load(&cnt[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (e) {
            cnt[k] = 0ull;
            one((int32_t)k, e);
          }
        }
      }
      __syncthreads();
      if (t == 0) S.nt = 0;
    }
    {
      uint4* w4 = (uint4*)S.win;
      uint64_t s2 = 0;
      const int nq = min(((wcap >> sh) + 4) >> 2, A.c4_win / 2);  // 16-byte pieces that hold the window's ids
      for (int qi = t; qi < nq; qi += C4W_T) {
        const uint4 q = w4[qi];
        w4[qi] = make_uint4(0u, 0u, 0u, 0u);
        if (fw == 8) window_pairs<8>(q, s2);
        else window_pairs<FBW>(q, s2);
      }
#pragma unroll
      for (int x = 0; x < NF; ++x)
        if ((ref >> x) & 1u) acc[vsh + x] += (int64_t)(s2 >> 1);  // sum of c(c - 1), all even
    }
    __syncthreads();
    hi = lo;
    if (rest == 0) break;
    if (wtot < A.c4_dense_min && bot == 0) {  // (a range above others is dense throughout)
      // sparse from here down: every remaining wedge in global memory
      const int32_t tcap = (int32_t)lo;  // list capacity: the ids below the windows (<= N)
      c4_block_walk(R, rb, nlow, urow, [&](int32_t) { return 0; }, [&](int32_t q) { return ucur[q]; },
                    [&](uint32_t wid, uint32_t fl) {
                      const uint32_t sub = (vpresent<NV>(fl) >> vsh) & fmask;
                      if (!sub) return;
                      ++tail_;
                      // as in the windows: no wait for the global atomic, the id
                      // listed once per wedge while the list is shorter than [0, lo)
                      atomicAdd(&cnt[wid], (unsigned long long)TFd::spread(sub));
                      const int32_t p = atomicAdd(&S.nt, 1);
                      if (p < tcap) touch[p] = (int32_t)wid;
                    });
      const int32_t nt = S.nt;
      if (nt <= tcap) {
        for (int32_t q = t; q < nt; q += C4W_T) {
          const unsigned long long c = atomicExch(&cnt[touch[q]], 0ull);
#pragma unroll
          for (int x = 0; x < NF; ++x) acc[vsh + x] += c2(TFd::get(c, x));
        }
      } else {
        for (int64_t k = t; k < (int64_t)lo; k += C4W_T) {
          const unsigned long long c = __hip_atomic_load(&cnt[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (c) {
            cnt[k] = 0ull;
#pragma unroll
            for (int x = 0; x < NF; ++x) acc[vsh + x] += c2(TFd::get(c, x));
          }
        }
      }
      __syncthreads();
      if (t == 0) S.nt = 0;
      break;
    }
  }
  __syncthreads();
}

template <int NV>
__global__ __launch_bounds__(C4W_T) void k_c4_large(CountArgs A, unsigned long long* qhead) {
  __shared__ C4Smem S;
  const RegionDev& R = A.R;
  const int64_t n = (int64_t)A.c[C_C4I];
  const int t = threadIdx.x;
  int cur_g = -1;
  int64_t acc[NV];
  zerov<NV>(acc);
  int64_t tail_ = 0;
  for (int s = t; s < A.c4_win; s += C4W_T) S.win[s] = 0ull;  // kept clear between windows
  while (true) {
    __syncthreads();  // every thread has read the previous item before it is replaced
    if (t == 0) S.item = (int64_t)atomicAdd(qhead, 1ull);
    __syncthreads();
    const int64_t item = S.item;
    if (item >= n) break;
    const unsigned long long e = A.c4_keys_alt[item];
    const int32_t v = (int32_t)(uint32_t)e;
    const int g = A.gid[v];
    if (g != cur_g) { if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc); cur_g = g; }
    if (R.rlow[v] > A.c4_maxlow) {  // cursor scratch too small: the host counts again with more
      if (t == 0) atomicAdd(&A.bstats[BS_RETRY], 1ull);
      continue;
    }
    // the item's ids [bot, top): all below v, or one of `cut` ranges that hold
    // about equal shares of the graph's entries below v
    const int part = (int)(e >> 32) & 0xFF, cut = (int)(e >> 40);
    int64_t top = v, bot = 0;
    if (cut > 1) {
      if (t < 64) {  // the graph's first vertex, then the two cuts
        int64_t lo = 0, hi = v;  // gid[hi] == g
        while (hi > lo) {
          const int64_t st = (hi - lo + 63) / 64, at = min(lo + st * lane_id(), hi);
          const int k = __popcll(__ballot(A.gid[at] < g));  // samples before the graph
          hi = min(hi, lo + st * k);
          lo = k ? min(lo + st * (k - 1) + 1, hi) : lo;
        }
        const int64_t r0 = R.roff[hi], all = R.roff[v] - r0;
        const int64_t x = part == 0 ? v : wave_upper_bound(R.roff, v, r0 + all / cut * (cut - part));
        const int64_t y = part == cut - 1 ? 0 : wave_upper_bound(R.roff, v, r0 + all / cut * (cut - part - 1));
        if (lane_id() == 0) { S.cut[0] = x; S.cut[1] = y; }
      }
      __syncthreads();
      top = S.cut[0];
      bot = S.cut[1];
    }
    if (top <= bot) continue;
    // c(v, w) <= nlow: 16-bit fields suffice up to 65535 lower neighbours
    const bool narrow = R.rlow[v] <= A.c4_narrow_max;
    if constexpr (NV == 2) {
      if (narrow) c4_hub<2, 2, 16>(A, S, v, top, bot, 0, acc, tail_);
      else c4_hub<2, 2, 32>(A, S, v, top, bot, 0, acc, tail_);
    } else {
      if (narrow) {
        c4_hub<4, 4, 16>(A, S, v, top, bot, 0, acc, tail_);
      } else {
        c4_hub<4, 2, 32>(A, S, v, top, bot, 0, acc, tail_);
        c4_hub<4, 2, 32>(A, S, v, top, bot, 2, acc, tail_);
      }
    }
  }
  if (cur_g >= 0) flushv<NV>(A.sig, cur_g, SG_C4, acc);
  tail_ = wave_sum64(tail_);
  if (lane_id() == 0 && tail_) atomicAdd(&A.bstats[BS_TRIPROBE], (unsigned long long)tail_);
}

// Largest union row length in each block of C4_BLK ids: bounds c(v, w) for
// every w of the block, so a hub window over blocks whose rows are all at
// most 255 long can count in 8-bit fields.  blk must be zero on entry.
__global__ void k_c4_blkmax(const int64_t* __restrict__ roff, int64_t N, int32_t* __restrict__ blk) {
  for (int64_t v0 = (int64_t)blockIdx.x * 256 * 4; v0 < N; v0 += (int64_t)gridDim.x * 256 * 4) {
    int32_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t v = v0 + threadIdx.x + 256 * k;
      if (v < N) m = max(m, (int32_t)(roff[v + 1] - roff[v]));
    }
    // the 1024 ids of one iteration form one block (v0 is block aligned)
    m = wave_max32(m);
    if (lane_id() == 0 && m) atomicMax(&blk[v0 >> C4_BLK_LOG], m);
  }
}

// Items of the large tier: a hub, or one of the id ranges a large hub is cut
// into (the opposite vertices of different ranges are counted apart), in
// decreasing order of wedge work: the workgroups then walk hubs of about the
// same size through the same windows at the same time, and find the rows in
// the shared cache (in loose order the count at scale 22 took 115 ms instead
// of 90).  One workgroup walks about 1.5e9 wedges a second, so a hub with
// more than 1/1024 of all wedges sets the time of a small graph's count.
constexpr int64_t C4_ITEMS = 1024;        // pieces the whole work is cut to
constexpr int64_t C4_ITEM_MIN = 65536;    // wedges that pay for a range's cursor searches
constexpr int64_t C4_CUT_MAX = 32;        // ranges per hub

__global__ __launch_bounds__(1024) void k_c4_items(const unsigned long long* sorted, unsigned long long* cc,
                                                   const unsigned long long* bstats, int64_t N,
                                                   unsigned long long* items) {
  __shared__ int32_t ws[2][16];
  const int64_t n = (int64_t)cc[C_LIST0 + L_C4_L];
  const int64_t target = max((int64_t)bstats[BS_C4_L] / C4_ITEMS, C4_ITEM_MIN);
  const int64_t most = max((int64_t)1, min(C4_CUT_MAX, N / max(n, (int64_t)1)));  // the list holds N items
  const int l = lane_id(), w = threadIdx.x >> 6;
  int64_t base = 0;
  int ph = 0;
  for (int64_t b0 = 0; b0 < n; b0 += 1024, ph ^= 1) {
    int32_t cut = 0;
    unsigned long long v = 0;
    if (b0 + threadIdx.x < n) {
      const unsigned long long key = sorted[b0 + threadIdx.x];
      v = key >> 16;
      const int q = 65535 - (int)(key & 65535ull), e = q >> 11;  // work: (2048 + q % 2048) 2^(e - 11)
      const int64_t work = ((int64_t)(2048 + (q & 2047)) << e) >> 11;
      cut = (int32_t)max((int64_t)1, min(most, (work + target - 1) / target));
    }
    const int32_t incl = wave_incl_scan32(cut);
    if (l == 63) ws[ph][w] = incl;
    __syncthreads();  // the other phase's sums are read no more once all are here
    int64_t at = base + incl - cut;
    for (int k = 0; k < 16; ++k) {
      at += k < w ? ws[ph][k] : 0;
      base += ws[ph][k];
    }
    for (int32_t k = 0; k < cut; ++k)
      items[at + k] = v | ((unsigned long long)k << 32) | ((unsigned long long)cut << 40);
  }
  if (threadIdx.x == 0) cc[C_C4I] = (unsigned long long)base;
}

// --------------------------------------------------------------- combine
// C' = C_x - C_0 on the six connected classes for every later version x
// (Alg. 2), through the non-induced counts of each version and the
// triangular relation between non-induced and induced counts (copies of
// pattern X inside class Y).
template <int NV>
__global__ void k_combine(const unsigned long long* sig, long long* state, long long* vout, int32_t k,
                          const unsigned long long* bstats) {
  const int64_t g = gtid();
  if (g >= k || bstats[BS_RETRY]) return;
  int64_t N[NV][6], T[NV], W[NV], D1[NV];
  int bad = 0;
  for (int x = 0; x < NV; ++x) {
    const unsigned long long* s = sig + SIG_IDX(g, x, 0);
    const int64_t t3 = (int64_t)s[SG_T], paw2 = (int64_t)s[SG_PAW];
    bad |= (t3 % 3 != 0) | (paw2 % 2 != 0);
    const int64_t t = t3 / 3;
    N[x][0] = (int64_t)s[SG_S2] - 3 * t;      // 3-paths
    N[x][1] = (int64_t)s[SG_S1];              // 3-stars
    N[x][2] = (int64_t)s[SG_C4];              // 4-cycles
    N[x][3] = paw2 / 2;                       // paws
    N[x][4] = (int64_t)s[SG_DIA];             // diamonds
    N[x][5] = (int64_t)s[SG_K4];              // 4-cliques
    T[x] = t; W[x] = (int64_t)s[SG_W]; D1[x] = (int64_t)s[SG_D1];
    bad |= (D1[x] % 2 != 0);
  }
  long long* st = state + g * ST_STRIDE;
  long long base[ST_STRIDE];
  for (int c = 0; c < ST_STRIDE; ++c) base[c] = st[c];
  for (int x = 1; x < NV; ++x) {
    int64_t d[6];
    for (int c = 0; c < 6; ++c) d[c] = N[x][c] - N[0][c];
    int64_t I[6];
    I[5] = d[5];
    I[4] = d[4] - 6 * I[5];
    I[3] = d[3] - 4 * I[4] - 12 * I[5];
    I[2] = d[2] - I[4] - 3 * I[5];
    I[0] = d[0] - 2 * I[3] - 4 * I[2] - 6 * I[4] - 12 * I[5];
    I[1] = d[1] - I[3] - 2 * I[4] - 4 * I[5];
    long long* o = vout + ((int64_t)(x - 1) * k + g) * ST_STRIDE;
    for (int c = 0; c < ST_STRIDE; ++c) o[c] = base[c];
    for (int c = 0; c < 6; ++c) o[ST_F0 + c] += I[c];
    o[ST_T] += T[x] - T[0];
    o[ST_W] += W[x] - W[0];
    o[ST_M] += (D1[x] - D1[0]) / 2;
    if (bad) o[ST_ERR] += 1;
    if (x == NV - 1)
      for (int c = 0; c < ST_STRIDE; ++c) st[c] = o[c];
  }
}

inline unsigned cap_grid(int64_t want, unsigned cap) {
  if (want < 1) want = 1;
  return (unsigned)(want > cap ? cap : want);
}

template <int NV>
void launch_count_t(const CountArgs& A, hipStream_t s, hipEvent_t* ev) {
  constexpr int TLM = tl_max<NV>();
  const int64_t N = A.N;
  if (ev) (void)hipEventRecord(ev[0], s);
  hipLaunchKernelGGL(k_t_clear<NV>, dim3(cap_grid((A.e_max + 1023) / 1024, 4096)), dim3(256), 0, s, A);
  hipLaunchKernelGGL(k_tri_small<NV>, dim3(cap_grid((N + 3) / 4, 8192)), dim3(256), 0, s, A);
  // out-degree tiers (64,128] (256] (512] (1024] (TLM] and above, one list each
  unsigned long long* qt = (unsigned long long*)(A.c + C_QTRI) - L_TRI_1;
  hipLaunchKernelGGL((k_tri_large<128, 256, NV>), dim3(cap_grid(N, 8192)), dim3(256), 0, s, A, (int)L_TRI_1,
                     qt + L_TRI_1);
  hipLaunchKernelGGL((k_tri_large<256, 512, NV>), dim3(cap_grid(N, 4096)), dim3(512), 0, s, A, (int)L_TRI_2,
                     qt + L_TRI_2);
  hipLaunchKernelGGL((k_tri_large<512, 1024, NV>), dim3(cap_grid(N, 2048)), dim3(1024), 0, s, A, (int)L_TRI_3,
                     qt + L_TRI_3);
  hipLaunchKernelGGL((k_tri_large<1024, 1024, NV>), dim3(cap_grid(N, 1024)), dim3(1024), 0, s, A, (int)L_TRI_4,
                     qt + L_TRI_4);
  hipLaunchKernelGGL((k_tri_large<TLM, 1024, NV>), dim3(cap_grid(N, 1024)), dim3(1024), 0, s, A, (int)L_TRI_5,
                     qt + L_TRI_5);
  hipLaunchKernelGGL((k_tri_large<0, 256, NV>), dim3(cap_grid(N, (unsigned)A.tri_slots)), dim3(256), 0, s, A,
                     (int)L_TRI_G, qt + L_TRI_G);
  if (ev) (void)hipEventRecord(ev[1], s);
  // at least 4096 entries per workgroup: few flushes of per-graph sums
  hipLaunchKernelGGL(k_edge_pass<NV>, dim3(cap_grid((A.e_max + 4095) / 4096, 2048)), dim3(256), 0, s, A);
  if (ev) (void)hipEventRecord(ev[2], s);
  hipLaunchKernelGGL(k_c4_small<NV>, dim3(cap_grid((N + 3) / 4, 8192)), dim3(256), 0, s, A);
  if (ev) (void)hipEventRecord(ev[3], s);
  hipLaunchKernelGGL(k_c4_mid<NV>, dim3(cap_grid(N, 4096)), dim3(256), 0, s, A);
  if (ev) (void)hipEventRecord(ev[4], s);
  // order the hubs by decreasing wedge work (keys written by the per-vertex pass)
  unsigned long long* sk = radix_sort_u64(A.c4_keys, A.c4_keys_alt, A.sort_tmp, N, A.c + C_LIST0 + L_C4_L, 16, s);
  // two digits: the keys are back where they were written, the other buffer takes the items
  hipLaunchKernelGGL(k_c4_items, dim3(1), dim3(1024), 0, s, (const unsigned long long*)sk, (unsigned long long*)A.c,
                     (const unsigned long long*)A.bstats, N, A.c4_keys_alt);
  fill_u32((uint32_t*)A.c4_blk, 0u, N / C4_BLK + 2, s);
  hipLaunchKernelGGL(k_c4_blkmax, dim3(cap_grid((N + 1023) / 1024, 4096)), dim3(256), 0, s, A.R.roff, N, A.c4_blk);
  hipLaunchKernelGGL(k_c4_large<NV>, dim3(cap_grid(N, (unsigned)A.slots)), dim3(C4W_T), 0, s, A,
                     (unsigned long long*)(A.c + C_QHEAD));
  if (ev) (void)hipEventRecord(ev[5], s);
}

}  // namespace

int32_t c4_window_max() { return C4W_WIN; }
int32_t c4_block_ids() { return C4_BLK; }
int64_t tri_scratch_words64(int nv, int64_t cap) {
  return nv == 2 ? tri_slot_words64<2>(cap) : tri_slot_words64<4>(cap);
}
int32_t tri_lds_max(int nv) { return nv == 2 ? tl_max<2>() : tl_max<4>(); }

void launch_count(int nv, const CountArgs& A, hipStream_t s, hipEvent_t* ev) {
  if (nv == 2) launch_count_t<2>(A, s, ev);
  else launch_count_t<4>(A, s, ev);
}

void launch_combine(int nv, const unsigned long long* sig, long long* state, long long* vout, int32_t k,
                    const unsigned long long* bstats, hipStream_t s) {
  if (nv == 2) hipLaunchKernelGGL(k_combine<2>, dim3((k + 63) / 64), dim3(64), 0, s, sig, state, vout, k, bstats);
  else hipLaunchKernelGGL(k_combine<4>, dim3((k + 63) / 64), dim3(64), 0, s, sig, state, vout, k, bstats);
}
