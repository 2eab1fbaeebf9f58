// Launcher declarations shared by the kernel files and the host code.
#pragma once
#include "gc_internal.h"

// device counters (u64) of one batch
enum {
  C_DIRA = 0,     // directed entries of pairs absent before the pass and present in a later version
  C_DIRD,         // directed entries of existing edges absent from a later version
  C_DIRR,         // directed entries absent from the last version (removed by the purge)
  C_TOUCH,        // rows touched by the pass
  C_NKEYS,        // update entries of the pass (set by the ingest kernel)
  C_RLIST,        // region vertices (first counter of the counting stage)
  C_LVL0,         // C_LVL0 + k: end of level-k vertices in the region list (k = 0..4)
  C_ER = C_LVL0 + 6,  // region entries
  C_MAXDP,        // max oriented out-degree
  C_MAXW,         // max wedge bound
  C_MAXLOW,       // max lower degree in the large 4-cycle tier
  C_LIST0,        // C_LIST0 + L_*: work list sizes
  C_QHEAD = C_LIST0 + 12,  // dynamic queue head of the large 4-cycle tier
  C_QTRI,                  // C_QTRI + k: queue head of list L_TRI_1 + k (k < 6)
  C_QTS = C_QTRI + 6,      // queue heads of the small triangle tier and of the mid 4-cycle tier
  C_QC4M,
  C_C4I,                   // items of the large 4-cycle tier
  C_COUNT
};
// Work lists: triangles by out-degree (<= 64 one wave per vertex, then the
// workgroup tiers (64,128] (128,256] (256,512] (512,1024] (1024,TRI_LDS_MAX]
// in LDS and the global-scratch tier above), 4-cycles by wedge bound.
enum { L_TRI_S = 0, L_TRI_1, L_TRI_2, L_TRI_3, L_TRI_4, L_TRI_5, L_TRI_G, L_C4_S, L_C4_M, L_C4_L, L_NUM };
constexpr int TRI_LDS_MAX = 1280;
static_assert(L_NUM <= 12, "list counters");

__host__ __device__ inline int tri_list_of(int32_t dplus, int32_t small) {
  if (dplus <= small) return L_TRI_S;
  if (dplus <= 128) return L_TRI_1;
  if (dplus <= 256) return L_TRI_2;
  if (dplus <= 512) return L_TRI_3;
  if (dplus <= 1024) return L_TRI_4;
  if (dplus <= TRI_LDS_MAX) return L_TRI_5;
  return L_TRI_G;
}

// Directed entry keys of the merge lists: row << bits | col, with the
// absence mask of the edge (bit x = absent from version x) in bits 60..63.
#define DIR_MASK_SHIFT 60
#define DIR_KEY_MASK ((1ull << DIR_MASK_SHIFT) - 1ull)

// Segments of the update arrays: one per graph of a pool (seq = 0), or one
// per successive batch of graph 0 (seq = 1).
struct BatchIn {
  const int32_t* iu; const int32_t* iv; const int32_t* du; const int32_t* dv;
  int64_t n_ins, n_del;
  const int64_t* ins_seg;  // [k+1] insertion segment bounds
  const int64_t* del_seg;  // [k+1]
  const int64_t* gbase;    // [graphs] first vertex of each graph
  const int64_t* gn;       // [graphs] vertex count of each graph
  int32_t k;               // segments
  int32_t seq;
  const uint8_t* dead;     // [N] 1 for a vertex taken out of its graph (nullptr: none)
};

struct BatchWork {
  unsigned long long* c;       // counters
  unsigned long long* dirA;    // directed entry keys (see DIR_MASK_SHIFT), sorted
  unsigned long long* dirD;    // in any order
  unsigned long long* dirR;    // sorted
  // per row: segment of dirA (a_beg, na) and of dirR (r_beg, nr)
  int32_t* a_beg; int32_t* na; int32_t* r_beg; int32_t* nr; int32_t* mark; int32_t* tix;  // [N]
  int32_t* touched;            // [max_touched]
  int64_t* dest; int32_t* newcap; int32_t* tlen; int64_t* tpre;  // [max_touched (+1)]
  uint32_t* scratch;           // copy of the touched rows (col)
  uint32_t* scratch_t;         // and of their tt
};

// graph.hip
// The update counts live on the device (ins_seg[k], del_seg[k]); cap_total
// bounds their sum and sizes the grid.  Sets c[C_NKEYS].
void launch_ingest_keys(const PoolDev& P, const BatchIn& B, int bits, unsigned long long* keys, unsigned long long* c,
                        unsigned long long* bstats, int64_t cap_total, hipStream_t s);
// keys: pair << 3 | batch << 1 | op (c[C_NKEYS] of them); nb batches in the
// pass, nv versions
void launch_ingest_classify(const PoolDev& P, const unsigned long long* keys, int64_t cap_total, int bits, int nb,
                            int nv, unsigned long long* dirA, unsigned long long* dirD, unsigned long long* dirR,
                            unsigned long long* c, unsigned long long* bstats, hipStream_t s);
// max_n bounds the entries of dirA, dirD and dirR together
void launch_mark_rows(const BatchWork& W, int64_t max_n, int bits, hipStream_t s);
void launch_merge(const PoolDev& P, const BatchWork& W, int64_t max_touched, int64_t max_dirA, int bits, float slack,
                  unsigned long long* bstats, void* scan_tmp, hipStream_t s);
void launch_flag_rows(const PoolDev& P, const BatchWork& W, int64_t max_dirD, int bits, unsigned long long* bstats,
                      hipStream_t s);
// removes the entries carrying `fin` (absent from the last version), clears
// all flags (rows that lose nothing: in place, max_dir bounds the
// flagged entries); does nothing while *skip != 0.  undo: removes the entries new
// in the pass instead (GC_F_NEW, listed in W.dirA), which restores the graph
// as it was before a one-batch pass whose counting did not complete
void launch_purge(const PoolDev& P, const BatchWork& W, int64_t max_touched, int64_t max_dir, int bits, uint32_t fin,
                  const unsigned long long* skip, void* scan_tmp, hipStream_t s, bool undo = false);
// the purge of a pass without deletions: the flags of the new entries are
// cleared in place (max_dirA bounds their count)
void launch_purge_insert_only(const PoolDev& P, const BatchWork& W, int64_t max_touched, int64_t max_dirA, int bits,
                              const unsigned long long* skip, hipStream_t s);
void launch_region(const PoolDev& P, const BatchWork& W, int radius, int32_t* level, int32_t* rlist, int32_t* rlen,
                   hipStream_t s);
// wsum [N]: wedge sums of the region vertices (cleared by launch_region_fill,
// summed by launch_degrees)
void launch_region_fill(int nv, const PoolDev& P, const RegionDev& R, const BatchWork& W, int radius,
                        const int32_t* level, const int32_t* rlist, const int32_t* rlen, unsigned long long* wsum,
                        void* scan_tmp, hipStream_t s);
void launch_degrees(int nv, const RegionDev& R, const int32_t* gid, const int32_t* rlist, unsigned long long* c,
                    unsigned long long* sig, int32_t* lists, int64_t list_stride, int32_t tri_small, int32_t c4_small,
                    int32_t c4_mid, unsigned long long* bstats, unsigned long long* c4_keys, unsigned long long* wsum,
                    hipStream_t s);
void launch_init_keys(const int32_t* src, const int32_t* dst, int64_t m, const int64_t* seg, const int64_t* gbase,
                      int32_t k, int bits, unsigned long long* keys, hipStream_t s);
void launch_init_unique(const unsigned long long* keys, int64_t m, int bits, unsigned long long* uniq,
                        unsigned long long* c, int32_t* deg, hipStream_t s);
void launch_rank(const int32_t* deg, const int32_t* gid, const int64_t* gbase, int64_t N, int lbits, int total_bits,
                 unsigned long long* keys, unsigned long long* alt, void* sort_tmp, int32_t* ext2int, int32_t* int2ext,
                 int32_t* len, hipStream_t s);
void launch_init_dir(const unsigned long long* uniq, int64_t max_m, unsigned long long* c, int bits,
                     const int32_t* ext2int, unsigned long long* dir, hipStream_t s);
void launch_init_csr(const PoolDev& P, const unsigned long long* dir, int64_t max_dir, unsigned long long* c, int bits,
                     int64_t* rstart, float slack, void* scan_tmp, uint32_t flag, hipStream_t s);
void launch_caps(const PoolDev& P, float slack, hipStream_t s);  // P.cap <- len + slack
void launch_all_flags(const PoolDev& P, uint32_t set, uint32_t keep, hipStream_t s);
void launch_compact(const PoolDev& P, int64_t* noff, uint32_t* ncol, uint32_t* ntt, hipStream_t s);
void launch_upper_count(const PoolDev& P, int32_t* cnt, hipStream_t s);
// rows of k vertices of a single graph (external ids): lengths, then the
// edges (x, neighbour) in external ids at the exclusive prefix pre
void launch_row_len(const PoolDev& P, const int32_t* ids, int64_t k, int32_t* out, hipStream_t s);
void launch_row_gather(const PoolDev& P, const int32_t* int2ext, const int32_t* ids, int64_t k, const int64_t* pre,
                       int32_t* u, int32_t* v, hipStream_t s);
// a[ids[i]] = val
void launch_set_bytes(uint8_t* a, const int32_t* ids, int64_t k, uint8_t val, hipStream_t s);
void launch_export(const PoolDev& P, const int32_t* int2ext, const int64_t* gbase, const int64_t* pre, int32_t* src,
                   int32_t* dst, hipStream_t s);

// count.hip
struct CountArgs {
  RegionDev R;
  const int32_t* gid;
  const int32_t* lists;     // L_NUM lists of list_stride entries
  int64_t list_stride;
  const unsigned long long* c;
  unsigned long long* sig;
  unsigned long long* bstats;
  // per-slot scratch of the large tiers
  unsigned long long* c4_dense;   // [slots][N] (two versions, or four with 16-bit fields)
  int32_t* c4_touch;              // [slots][N]
  int64_t N;
  int32_t slots;                  // workgroups of the large 4-cycle tier
  int32_t c4_win;                 // 64-bit words of the LDS window of the large tier (<= c4_window_max())
  int32_t c4_narrow_max;          // up to this many lower neighbours, 16-bit counters (2x window)
  int64_t c4_dense_min;           // hits that earn a window dense LDS counters
  uint32_t c4_ref;                // versions whose common wedges the hub windows count (the rest are exceptions)
  int64_t* c4_cur;                // [slots][2 * c4_maxlow]: row starts, cursors
  int32_t* c4_blk;                // [N / C4_BLK + 1] largest union row length per block of C4_BLK ids
  int64_t c4_maxlow;              // largest lower degree of a large-tier vertex
  unsigned long long* c4_keys;    // [N] sort keys of the large tier (written by the per-vertex pass)
  unsigned long long* c4_keys_alt;  // [N] wedge sums, then the sort's buffer, then the tier's items
  void* sort_tmp;
  int32_t tri_slots;              // workgroups of the global-scratch triangle tier
  unsigned long long* tri_scratch;  // [tri_slots][tri_scratch_words64(tri_cap)] above the LDS tier
  int64_t tri_cap;                  // out-degree capacity of a scratch slot (0: no scratch)
  int64_t e_max;                    // capacity of the region arrays (entries)
};
// nv = 2 or 4 versions.  Grids come from host bounds (A.N, A.e_max, the
// scratch sizes); work sizes from the device counters.
void launch_count(int nv, const CountArgs& A, hipStream_t s,
                  hipEvent_t* ev /* nullable: 6 events between the kernel phases */);
int64_t tri_scratch_words64(int nv, int64_t cap);  // u64 words of one triangle scratch slot
int32_t tri_lds_max(int nv);                        // largest out-degree of the LDS triangle tiers
int32_t c4_window_max();                            // u64 words of the LDS window of the large 4-cycle tier
int32_t c4_block_ids();                             // ids per entry of CountArgs::c4_blk
// Per graph g: the state after version x (x = 1 .. nv-1) goes to
// vout[((x - 1) * k + g) * ST_STRIDE ...]; state becomes the one of version nv-1.
// nothing is written while bstats[BS_RETRY] != 0
void launch_combine(int nv, const unsigned long long* sig, long long* state, long long* vout, int32_t k,
                    const unsigned long long* bstats, hipStream_t s);

// capi.cpp: thread-local error text read by gc_last_error()
// delta.hip: edge-local update of the Sigma terms of a one-batch pass
enum {
  DC_EDGES = 0,  // changed pairs
  DC_AFF,        // affected edges listed
  DC_AFF_INST,   // moves of t of an affected edge (at least as many)
  DC_AFF_FULL,   // the table of the affected edges was too full
  DC_AFF_NEED, DC_PAIR_NEED,
  DC_SEARCH,     // searched pairs
  DC_WALK,       // walk lengths (twice the pairs)
  DC_QH,         // queue of the walked chunks
  DC_LAY,        // edges walked in layers (above DC_LAY_SHIFT) and their chunks
  DC_QL,         // queue of those chunks
  DC_OUT,        // members of N(o) that the bitmaps leave out
  DC_OUT_WALK,   // entries that searching them walks, at most
  DC_COST,       // entries walked against the bitmaps, or searched in their place
  DC_COUNT
};
constexpr int DC_LAY_SHIFT = 36;
constexpr int32_t TV_CHUNK = 4096;      // entries of a touched row per piece in the edge-local degree passes
struct DeltaArgs {
  PoolDev P;                          // union view left by the tombstone merge
  int64_t N;
  int bits;
  const unsigned long long* dirA;     // directed change lists, dirA sorted (counts in c)
  const unsigned long long* dirD;
  const unsigned long long* dirR;     // the deletions again, with a segment per row (r_beg, nr)
  const int32_t *a_beg, *na, *r_beg, *nr;  // [N] segments of dirA and dirR
  const unsigned long long* c;        // batch counters (C_DIRA, C_DIRD, C_TOUCH)
  const int32_t* touched;             // touched rows
  const int32_t* mark;                // [N] 1 on touched rows
  const int32_t* gid;                 // [N] graph of each vertex
  unsigned long long* sig;            // per-graph sums; version 1 receives the deltas
  unsigned long long* bstats;         // BS_RETRY when a buffer below is too small
  int32_t* dd;                        // [N][2] degrees before / after of the touched rows
  long long* Tv;                      // [N] triangles at each vertex (moved to the graph after the batch)
  unsigned long long* dT;             // [N] scratch, zero between passes: the change of T(v)
  unsigned long long* ce;             // changed pairs (u < v) | nibble << 60
  int64_t ce_cap;
  int32_t *e_ns, *e_dt;               // [ce_cap] per changed pair: common neighbours, change of t
  int32_t* e_out;                     // [ce_cap] common neighbours that the pair's bitmap leaves out
  int64_t* e_kw;                      // [ce_cap] and the entries of the common neighbours' rows
  // affected edges: a hash table of resident positions + 1 (0: free; all free
  // between passes) with the change of t, and the slots taken (slot | an end << 32)
  unsigned long long* hk;             // [hmask + 1]
  int32_t* hd;                        // [hmask + 1]
  uint32_t hmask;
  unsigned long long* hl;             // [ae_cap]
  int64_t ae_cap;
  unsigned long long* dc;             // [DC_COUNT] counters of the stage, zero on entry
  int32_t* c4_nch;                    // [ce_cap] pairs (e, a) per changed edge: degree of the end walked from
  int32_t* c4_side;                   // [ce_cap] bit 0: walk from v instead of u; bit 1: against a bitmap; bits 2 to 4: in
                                      // layers (for certain; when searches are dear; when they list too many)
  int32_t* c4_low;                    // [ce_cap] entries of the other end's row below the bitmap's window
  uint32_t c4_ids;                    // ids a bitmap covers (0 or too many: launch_delta sets the most)
  int32_t c4_out;                     // > 0: an edge whose bitmap leaves out more members is walked in layers (tests)
  uint32_t lay_ids;                   // ids a window of the layers covers (set by launch_delta)
  // edges walked in layers: their index (4-cliques: after all 4-cycles) and first chunk
  int32_t* lay_list;                  // [2 ce_cap]
  int64_t* lay_off;                   // [2 ce_cap]
  int64_t* c4_off;                    // [ce_cap + 1] exclusive scan of c4_nch
  // searched pairs (DC_SEARCH of them): changed edge, index (below the degree
  // of the end walked from: pair (e, a), else (e, b)) and entries walked
  int32_t *pair_edge, *pair_idx, *pair_len;  // [2 pair_cap]
  uint32_t* slist;                    // [pair_cap] S(e) at c4_off of e: id | nibble(s, w) << 28 | nibble(o, w) << 30
  int32_t* tv_items;                  // [tcap] pieces of each touched row (rows split in TV_CHUNK entries)
  int64_t* tv_ioff;                   // [tcap + 1] exclusive scan of tv_items
  int64_t tcap;                       // touched rows the two arrays cover (>= the touched count)
  int64_t* pair_off;                  // [2 pair_cap + 1] exclusive scan of pair_len
  // entries walked against a bitmap: of N(a) per pair (e, a), then of the row
  // of each member of the lists S(e) (same places)
  int32_t* pair_hlen;                 // [2 pair_cap]
  int64_t* pair_hoff;                 // [2 pair_cap + 1] exclusive scan of pair_hlen
  int64_t pair_cap;
  void* scan_tmp;                     // scan scratch for max(ce_cap, 2 pair_cap) + 1 entries
};
void launch_delta(const DeltaArgs& D, hipStream_t s);
// T(v) of the region vertices and the resident t of its edges after a region
// pass (t of the last version minus t of version 0); dT zero before and after
void launch_tv_region(int nv, const PoolDev& P, const RegionDev& R, const int32_t* level, int32_t radius,
                      const int32_t* rlist, const unsigned long long* c, unsigned long long* dT, long long* Tv,
                      unsigned long long* bstats, hipStream_t s);

void gc_set_error(const char* msg);
// device bytes a single-graph handle reaches (capi.cpp); used by the server's admission
int64_t gc_footprint_estimate(int64_t n, int64_t m, double slack, int64_t max_deg, int64_t max_out, bool local);
