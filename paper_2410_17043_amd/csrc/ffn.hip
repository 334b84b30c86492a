// Expert FFN of Sec. 2.1 over the rows a GPU received: a ragged grouped GEMM pair.
//
//   GEMM1  Hmid[R,F] = act(recv . W1^T)            (SwiGLU: silu(recv . W1^T) * (recv . Wu^T))
//   GEMM2  out[R,H]  = Hmid . Wd^T
//
// Both operands of both GEMMs are K-contiguous ([rows,K] activations, [out,in]
// weights), which is exactly the operand layout of the CDNA MFMA instructions.
// Rows are grouped in segments, one local expert per segment; a small device kernel
// turns the segment list into a list of M-tiles (adjacent segments of the same
// expert are merged, tiles never straddle experts), so nothing waits for the host.
//
// bf16 path: 256x256 block tile (192x256 or 128x128 where that fills the chip better, see take_shapes), 32-wide
// k-tiles, 4 waves in 2x2, each wave 128x128 = 8x8
// tiles of v_mfma_f32_16x16x32_bf16 with fp32 accumulators (256 accumulator registers per
// lane); operands go global -> LDS directly (no register staging) through a 5-stage ring that
// fills the whole 160 KB LDS, in an XOR-swizzled layout that makes every ds_read_b128 of an
// MFMA operand conflict-free on the 64 LDS banks.  Loads, LDS reads and MFMAs are software
// pipelined by hand (see the kernel).  For SwiGLU the B tile holds 128 gate rows and 128 up
// rows arranged so that a wave owns the gate and the up product of the same 64 columns: the
// activation is applied on registers and the intermediate is written once, in bf16, as whole
// 128-byte lines after a transpose through LDS.  Tiles are numbered so that the blocks that
// share an XCD's L2 form a compact patch and all XCDs sweep the N-tiles in step (see
// tile_of_block); the tiles of a mostly empty last round are cut along K (see plan_tail).
//
// Shares of at most 64 rows (bf16) take a pair of weight-streaming kernels instead (gemm_bf16_skinny_kernel):
// 32- or 64-row tiles, 256-byte bursts per weight row, the LDS ring given to loads in flight.  Either GEMM of a bf16 share of
// up to 128 rows per expert, those of at most 64 rows included, takes narrow tiles where they are modelled faster
// (gemm_bf16_narrow_kernel: 32 to 128 rows x 32 or 64 weight rows over the whole of K, see take_narrow).
//
// Experts of up to 192 KB (bf16; fp32: 128 KB) and few blocks: both GEMMs in one kernel, without a tile map (ffn_small_kernel, see takes_small).
//
// fp32 path: 128 x 128 tiles of three bf16 parts per element on the bf16 matrix cores (gemm_f32_parts_kernel); where there are
// too few of them, 64 x 64 tiles on the fp32 matrix cores (gemm_f32_kernel).
#include "common.h"
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstddef>
#include <type_traits>
#include <vector>

namespace {

constexpr int kMaxSeg = 1024;

struct TileMap {
    int32_t* n_tiles;   // [1]
    int32_t* row0;      // [max_tiles] first row of the tile
    int32_t* nrows;     // [max_tiles] valid rows (1..BM)
    int32_t* expert;    // [max_tiles] local expert
    int32_t* gather;    // [max_tiles] 0: the tile is rows row0 .. row0 + nrows - 1; 1: row r is row0 + rel[tile][r]
    int32_t* rel;       // [max_tiles][kRelPitch] row offsets of the gathered tiles (written for those only)
    int32_t* done;      // [kMaxSplitTiles] pieces that have arrived, per tile cut along K (zeroed with the map)
};
constexpr int kMaxSplitTiles = 256;
constexpr int kRelPitch = 256;

struct ExpertTable {
    const void* w1[MOE_MAX_LOCAL];
    const void* w_up[MOE_MAX_LOCAL];
    const void* w_down[MOE_MAX_LOCAL];
};

__host__ __device__ inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
inline int max_tiles_for(int R) { return R / 64 + 1 + kMaxSeg; }
inline size_t tilemap_bytes(int R) {
    return align256(256 + 4 * sizeof(int32_t) * (size_t)max_tiles_for(R)) + (size_t)max_tiles_for(R) * kRelPitch * sizeof(int32_t);
}

// the map whose tiles are the workspace's records from `first` on; `which` (0, 1) has a tile count of its own
TileMap tilemap_at(void* ws, int R, int which = 0, int first = 0) {
    TileMap m;
    char* p = reinterpret_cast<char*>(ws);
    const size_t n = (size_t)max_tiles_for(R);
    m.n_tiles = reinterpret_cast<int32_t*>(p) + which;
    m.row0 = reinterpret_cast<int32_t*>(p + 256);
    m.nrows = m.row0 + n;
    m.expert = m.nrows + n;
    m.gather = m.expert + n;
    m.rel = reinterpret_cast<int32_t*>(p + align256(256 + 4 * sizeof(int32_t) * n));
    m.row0 += first; m.nrows += first; m.expert += first; m.gather += first;
    m.rel += (size_t)first * kRelPitch;
    m.done = nullptr;
    return m;
}
inline int max_tiles_of(int R, int bm, int nseg) { return std::min((R + bm - 1) / bm + nseg, R); }   // a tile has a row at least

// Tile map.  The received rows come as segments (rows seg_offset[i] .. seg_offset[i+1] - 1 belong to local
// expert seg_expert[i]); with several sources and several local experts the segments of one expert are not
// adjacent, and a segment can be much shorter than a tile (160 rows per source and expert under the
// capacity rule of the Switch-shape workload), so cutting every segment into tiles of its own would leave
// most tiles half empty.  With `gather` the segments of an expert are chained in index order into one
// list of rows that is cut into full tiles: a tile whose rows are not consecutive in memory carries a
// table of row offsets (rel), which the GEMM uses for its A-operand addresses and its output rows.
// Without `gather` only adjacent segments of the same expert are merged (every tile is consecutive rows).
//
// Items are the clamped, non-empty segments in processing order; a group is a maximal chain of items of
// one expert whose rows increase (so offsets from the tile's first row are never negative); tiles never
// straddle groups.  Both constructions - this one, and the one of lists of up to 64 segments below - are written once
// for the device kernel and for the host self check.
struct SegWork {
    int lo[kMaxSeg], hi[kMaxSeg], exp[kMaxSeg];                            // items (rows lo .. hi - 1 of one expert)
    int v0[kMaxSeg];                                                       // position of the item's first row in its group
    int grp[kMaxSeg];                                                      // group of the item
    int gaps[kMaxSeg];                                                     // items up to and including this one that do not follow their predecessor in memory
    int g_first[kMaxSeg + 1], g_tile0[kMaxSeg + 1], g_rows[kMaxSeg];       // groups: first item, first tile, rows
    int raw_off[kMaxSeg + 1], raw_exp[kMaxSeg];                            // the caller's segment list (raw_off: scratch once the items exist)
    int cnt[MOE_MAX_LOCAL], pos[MOE_MAX_LOCAL];
    int n_items, n_groups, n_tiles;
};
constexpr int kMapThreads = 1024;       // one block: a thread per segment / item, 16 waves to hide the LDS latency of the searches

// The steps take (tid, nth) = this thread and the thread count where they run in parallel; a barrier
// separates them.  The host self check runs the same per-element functions with plain loops in place
// of the block-wide ballots and prefix sums of the device kernel.
// 1: an expert outside [0, n_local) (-1) or an empty row range (-2) marks a segment to be skipped
__host__ __device__ inline void tilemap_clean(SegWork& w, int nseg, int R, int n_local, int tid, int nth) {
    for (int i = tid; i < nseg; i += nth) {
        const int lo = w.raw_off[i] > 0 ? w.raw_off[i] : 0;
        const int hi = w.raw_off[i + 1] < R ? w.raw_off[i + 1] : R;
        const int e = w.raw_exp[i];
        if (!(e >= 0 && e < n_local)) w.raw_exp[i] = -1;
        else if (!(hi > lo)) w.raw_exp[i] = -2;             // no rows: neither an item nor the end of a run
    }
    for (int e = tid; e < n_local; e += nth) w.cnt[e] = 0;
}
// 2 (gather), host form: rank of every segment among the segments of its expert, and the count per expert
inline void tilemap_rank_host(SegWork& w, int nseg) {
    for (int i = 0; i < nseg; ++i) {
        const int e = w.raw_exp[i];
        if (e < 0) continue;
        w.v0[i] = w.cnt[e]++;                        // the rank is parked in v0 until step 4
    }
}
// 3 (gather), host form: where the items of every expert start
inline void tilemap_starts_host(SegWork& w, int n_local) {
    int p = 0;
    for (int e = 0; e < n_local; ++e) { w.pos[e] = p; p += w.cnt[e]; }
    w.n_items = p;
}
// 4 (gather): segment i becomes item pos[e] + rank
__host__ __device__ inline void tilemap_place(SegWork& w, int nseg, int R, int tid, int nth) {
    for (int i = tid; i < nseg; i += nth) {
        const int e = w.raw_exp[i];
        if (e < 0) continue;
        const int k = w.pos[e] + w.v0[i];
        w.lo[k] = w.raw_off[i] > 0 ? w.raw_off[i] : 0;
        w.hi[k] = w.raw_off[i + 1] < R ? w.raw_off[i + 1] : R;
        w.exp[k] = e;
    }
}
// 2-4 without gathering (one thread): adjacent segments of the same expert merged
__host__ __device__ inline void tilemap_merge(SegWork& w, int nseg, int R) {
    int ni = 0, i = 0;
    while (i < nseg) {
        const int e = w.raw_exp[i];
        if (e < 0) { ++i; continue; }
        int j = i + 1;
        while (j < nseg && (w.raw_exp[j] == e || w.raw_exp[j] == -2)) ++j;
        const int lo = w.raw_off[i] > 0 ? w.raw_off[i] : 0;
        const int hi = w.raw_off[j] < R ? w.raw_off[j] : R;
        if (hi > lo) { w.lo[ni] = lo; w.hi[ni] = hi; w.exp[ni] = e; ++ni; }
        i = j;
    }
    w.n_items = ni;
}
// 5: does item k open a group / does it leave a gap behind its predecessor
__host__ __device__ inline bool tilemap_opens(const SegWork& w, int k, bool gather) {
    return !(gather && k > 0 && w.exp[k] == w.exp[k - 1] && w.lo[k] >= w.hi[k - 1]);
}
__host__ __device__ inline bool tilemap_gap(const SegWork& w, int k, bool gather) {
    return !tilemap_opens(w, k, gather) && w.lo[k] != w.hi[k - 1];
}
// 5, host form: groups and their tiles
inline void tilemap_groups_host(SegWork& w, int BM, bool gather) {
    const int ni = w.n_items;
    int ng = 0, nt = 0, rows = 0, gaps = 0;
    for (int k = 0; k < ni; ++k) {
        if (tilemap_opens(w, k, gather)) {
            if (ng > 0) { w.g_rows[ng - 1] = rows; nt += (rows + BM - 1) / BM; }
            w.g_first[ng] = k; w.g_tile0[ng] = nt; rows = 0;
            ++ng;
        }
        gaps += tilemap_gap(w, k, gather) ? 1 : 0;
        w.gaps[k] = gaps;
        w.v0[k] = rows;
        w.grp[k] = ng - 1;
        rows += w.hi[k] - w.lo[k];
    }
    if (ng > 0) { w.g_rows[ng - 1] = rows; nt += (rows + BM - 1) / BM; }
    w.g_first[ng] = ni; w.g_tile0[ng] = nt;
    w.n_groups = ng;
    w.n_tiles = nt;
}

// item of group g that holds group row v: the largest item with v0 <= v
__host__ __device__ inline int tilemap_item_of(const SegWork& w, int g, int v) {
    int c = w.g_first[g], d = w.g_first[g + 1];
    while (d - c > 1) { const int mid = (c + d) >> 1; if (w.v0[mid] <= v) c = mid; else d = mid; }
    return c;
}
struct TileSpan { int v_lo, v_hi, first_item, row0, gather; };
// tile q of group g: its range of group rows, its first row in memory, whether its rows have gaps
__host__ __device__ inline TileSpan tilemap_span(const SegWork& w, int g, int q, int BM) {
    TileSpan s;
    s.v_lo = q * BM;
    s.v_hi = w.g_rows[g] < s.v_lo + BM ? w.g_rows[g] : s.v_lo + BM;
    s.first_item = tilemap_item_of(w, g, s.v_lo);
    const int last_item = tilemap_item_of(w, g, s.v_hi - 1);
    s.row0 = w.lo[s.first_item] + (s.v_lo - w.v0[s.first_item]);
    s.gather = (w.gaps[last_item] - w.gaps[s.first_item] > 0) ? 1 : 0;   // a gap in front of an item that starts inside the tile
    return s;
}
// 6: the record of tile t
__host__ __device__ inline void tilemap_tile(const SegWork& w, int t, int BM, const TileMap& m) {
    int a = 0, b = w.n_groups;                       // largest group with g_tile0 <= t
    while (b - a > 1) { const int mid = (a + b) >> 1; if (w.g_tile0[mid] <= t) a = mid; else b = mid; }
    const TileSpan s = tilemap_span(w, a, t - w.g_tile0[a], BM);
    m.row0[t] = s.row0;
    m.nrows[t] = s.v_hi - s.v_lo;
    m.expert[t] = w.exp[s.first_item];
    m.gather[t] = s.gather;
}
// 7: the offset tables, item by item.  Only the first and the last tile of an item can have gaps (the
// tiles in between lie inside the item); for each of the two, if it has gaps, the item's rows in it are a
// run of consecutive table entries with consecutive values: rel[dst + r] = val + r for r < cnt.
struct RelJob { int dst, cnt, val; };
__host__ __device__ inline void tilemap_rel_jobs(const SegWork& w, int k, int BM, int n_tiles, RelJob (&job)[2]) {
    job[0] = job[1] = RelJob{0, 0, 0};
    const int g = w.grp[k], len = w.hi[k] - w.lo[k];
    const int q_a = w.v0[k] / BM, q_b = (w.v0[k] + len - 1) / BM;
    for (int pass = 0; pass < 2; ++pass) {
        const int q = pass == 0 ? q_a : q_b;
        if (pass == 1 && q_b == q_a) break;
        const int tile = w.g_tile0[g] + q;
        if (tile >= n_tiles) continue;
        const TileSpan s = tilemap_span(w, g, q, BM);
        if (!s.gather) continue;
        const int v_a = w.v0[k] > s.v_lo ? w.v0[k] : s.v_lo;                 // the item's rows inside the tile
        const int v_b = w.v0[k] + len < s.v_hi ? w.v0[k] + len : s.v_hi;
        job[pass].dst = tile * kRelPitch + (v_a - s.v_lo);
        job[pass].cnt = v_b - v_a;
        job[pass].val = w.lo[k] + (v_a - w.v0[k]) - s.row0;
    }
}

// Barrier that orders LDS traffic only (lgkmcnt(0), then s_barrier): the steps of the map exchange data
// through LDS alone, and __syncthreads() would also wait for every global store to land.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0); vmcnt and expcnt untouched
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// exclusive prefix sums of three values per thread over the block; totals to every thread
struct Int3 { int a, b, c; };
__device__ __forceinline__ Int3 block_scan3(Int3 v, Int3* excl, int* wave_tot /* LDS [3][16] */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    Int3 incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int ua = __shfl_up(incl.a, o, 64), ub = __shfl_up(incl.b, o, 64), uc = __shfl_up(incl.c, o, 64);
        if (lane >= o) { incl.a += ua; incl.b += ub; incl.c += uc; }
    }
    lds_barrier();                                 // wave_tot may still be read from an earlier scan
    if (lane == 63) { wave_tot[wave] = incl.a; wave_tot[16 + wave] = incl.b; wave_tot[32 + wave] = incl.c; }
    lds_barrier();
    Int3 before = {0, 0, 0}, total = {0, 0, 0};
#pragma unroll
    for (int wv = 0; wv < nw; ++wv) {
        const int ta = wave_tot[wv], tb = wave_tot[16 + wv], tc = wave_tot[32 + wv];
        if (wv < wave) { before.a += ta; before.b += tb; before.c += tc; }
        total.a += ta; total.b += tb; total.c += tc;
    }
    excl->a = before.a + incl.a - v.a; excl->b = before.b + incl.b - v.b; excl->c = before.c + incl.c - v.c;
    return total;
}

// How the tiles of a GEMM are numbered over the XCDs (see tile_of_block)
constexpr int kFewestStripTiles = 192, kStripTiles = 3000;
struct Strips { int wide, more; };                           // `more` strips of wide + 1 columns, then strips of `wide`; wide = 0: bands
__host__ __device__ __forceinline__ Strips plan_strips(int tiles_m, int tiles_n) {
    const int total = tiles_m * tiles_n;
    if (total < kFewestStripTiles || total > kStripTiles || (tiles_m / 8 < 4 && tiles_n / 8 > tiles_m / 8)) return Strips{0, 0};
    const float patch = fminf(total * 0.125f, 32.f), width = fmaxf(sqrtf(patch), patch / tiles_m);
    const int strips = max(1, min(tiles_n, (int)(tiles_n / width + 0.5f)));
    return Strips{tiles_n / strips, tiles_n % strips};
}
// One block per map, a thread per segment.  The segment list is read into LDS in one round trip; the stable order
// by expert comes from wave ballots (segments of the same expert inside a wave) plus a scan over the 16
// waves; groups, positions inside the groups and the tiles of the groups come from two block-wide prefix
// sums; then one thread per tile writes the tile records and the items fill the offset tables.
struct MapJob { int bm, max_tiles; TileMap m; };
struct MapJobs { MapJob job[2]; int32_t* done; int32_t* strips; int tiles_n[2]; };   // the two GEMMs may take tiles of different heights; done: both GEMMs' counters or NULL; strips: two numbers per GEMM (see Strips); tiles_n: column tiles of the GEMMs that are numbered by tile_of_block, else 0
// lane g < 2 writes the strips of GEMM g if map `job` of `maps` is its map
__device__ __forceinline__ void write_strips(const MapJobs& jobs, int job, int maps, int n_tiles, int lane) {
    if (lane >= 2 || (maps == 2 && lane != job) || jobs.tiles_n[lane] == 0) return;
    const Strips p = plan_strips(n_tiles, jobs.tiles_n[lane]);
    int32_t* to = jobs.strips + 2 * lane;
    to[0] = p.wide;
    to[1] = p.more;
}
__device__ __forceinline__ void zero_done(int32_t* done, int tid, int nth) {
    if (done)
        for (int i = tid; i < 2 * kMaxSplitTiles; i += nth) done[i] = 0;
}

// Up to 64 segments (every local expert of every source of a layer of up to 64 experts): lane k of EVERY wave holds
// segment k and works out the whole list for itself with ballots, lane permutations and prefix sums - no LDS, no
// barrier - and the waves share out the tiles.  10 -> 4.7 us at 64 segments against the block-wide kernel below.
// The steps are written once over W, the 64 lanes: WaveLanes on the device, ArrayLanes in the host self check.
constexpr int kSmallMapSegs = 64;
struct SmallItem {
    int off0, off1, e;               // in: seg_offset[k], seg_offset[k + 1], seg_expert[k]; e: then the item's expert
    int lo, len, hi;                 // rows lo .. hi - 1
    int rank;                        // position of the segment among the items
    int incl, excl;                  // rows of the items up to and in front of this one
    int prev_e, prev_hi;
    int v0;                          // position of the item's first row in its group
    int end, rows, tiles, tincl;     // of the group that the item opens: one past its last item, rows, tiles; tiles up to it
    bool ok, opens;
};
struct WaveLanes {
    SmallItem mine;
    int lane;
    template <class F> __device__ __forceinline__ void each(F f) { f(mine, lane); }
    template <class F> __device__ __forceinline__ unsigned long long ballot(F f) const { return __ballot(f(mine, lane)); }
    __device__ __forceinline__ int at(int SmallItem::*v, int k) const { return __builtin_amdgcn_readlane(mine.*v, k); }
    __device__ __forceinline__ void move_to_rank(int SmallItem::*v) { mine.*v = __builtin_amdgcn_ds_permute(mine.rank * 4, mine.*v); }
    __device__ __forceinline__ int from(int SmallItem::*v, int l, const SmallItem&) const { return __shfl(mine.*v, l, 64); }
    // by data-parallel moves: a few clocks each, where a shuffle takes the way through the LDS crossbar
    __device__ __forceinline__ void from_below(int SmallItem::*v, int SmallItem::*to) { mine.*to = __builtin_amdgcn_update_dpp(mine.*v, mine.*v, 0x138, 0xf, 0xf, false); }   // wave_shr:1
    __device__ __forceinline__ void prefix(int SmallItem::*v, int SmallItem::*to) {   // inclusive
        int x = mine.*v;
        x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8: inside rows of 16 lanes
        x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
        x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
        x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
        x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15: the row below into rows 1 and 3
        x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31: the lower half into rows 2 and 3
        mine.*to = x;
    }
};
struct ArrayLanes {
    SmallItem it[64];
    template <class F> void each(F f) { for (int l = 0; l < 64; ++l) f(it[l], l); }
    template <class F> unsigned long long ballot(F f) const {
        unsigned long long m = 0;
        for (int l = 0; l < 64; ++l) m |= (unsigned long long)(f(it[l], l) ? 1 : 0) << l;
        return m;
    }
    int at(int SmallItem::*v, int k) const { return it[k].*v; }
    void move_to_rank(int SmallItem::*v) {
        int old[64];
        for (int l = 0; l < 64; ++l) old[l] = it[l].*v;
        for (int l = 0; l < 64; ++l) it[it[l].rank].*v = old[l];
    }
    int from(int SmallItem::*v, int l, const SmallItem&) const { return it[l].*v; }
    void from_below(int SmallItem::*v, int SmallItem::*to) { for (int l = 0; l < 64; ++l) it[l].*to = it[l > 0 ? l - 1 : 0].*v; }
    void prefix(int SmallItem::*v, int SmallItem::*to) {
        int x = 0;
        for (int l = 0; l < 64; ++l) it[l].*to = (x += it[l].*v);
    }
};
struct SmallMap {
    unsigned long long gaps;         // items that leave a gap behind their predecessor in the group
    int n_tiles;
};
template <class W>
__host__ __device__ __forceinline__ SmallMap small_map(W& w, int nseg, int R, int n_local, int gather, int BM, int max_tiles) {
    using U = unsigned long long;
    using S = SmallItem;
    w.each([&](S& s, int lane) {
        s.lo = s.off0 > 0 ? s.off0 : 0;
        const int hi = s.off1 < R ? s.off1 : R;
        s.len = hi > s.lo ? hi - s.lo : 0;                             // (of offsets that fall by 2^31 the difference would wrap)
        s.ok = lane < nseg && s.e >= 0 && s.e < n_local && s.len > 0;  // others are skipped
    });
    // items: the segments by (expert, index) - without gathering by index - first, the skipped ones behind them
    const U okm = w.ballot([](const S& s, int) { return s.ok; });
    const int ni = __builtin_popcountll(okm);
    U bit[6];                                                          // MOE_MAX_LOCAL = 64 experts: six bits
#pragma unroll
    for (int b = 0; b < 6; ++b) bit[b] = w.ballot([&](const S& s, int) { return s.ok && ((s.e >> b) & 1); });
    w.each([&](S& s, int lane) {
        const U below = (1ull << lane) - 1ull;
        U eq = okm, lt = 0;                                            // the items of this expert, of lower experts
#pragma unroll
        for (int b = 5; b >= 0; --b) {
            if ((s.e >> b) & 1) { lt |= eq & ~bit[b]; eq &= bit[b]; }
            else eq &= ~bit[b];
        }
        s.rank = gather ? __builtin_popcountll(lt) + __builtin_popcountll(eq & below) : __builtin_popcountll(okm & below);
        if (!s.ok) { s.rank = ni + __builtin_popcountll(~okm & below); s.len = 0; s.e = -1; }
    });
    w.move_to_rank(&S::lo);
    w.move_to_rank(&S::len);
    w.move_to_rank(&S::e);
    // groups: chains of items of one expert whose rows increase (without gathering: follow each other)
    w.prefix(&S::len, &S::incl);
    w.each([](S& s, int) { s.excl = s.incl - s.len; s.hi = s.lo + s.len; });
    const int total = w.at(&S::incl, 63);
    w.from_below(&S::e, &S::prev_e);
    w.from_below(&S::hi, &S::prev_hi);
    w.each([&](S& s, int lane) {
        s.opens = lane < ni && (lane == 0 || s.e != s.prev_e || (gather ? s.lo < s.prev_hi : s.lo != s.prev_hi));
    });
    SmallMap m;
    const U heads = w.ballot([](const S& s, int) { return s.opens; });
    m.gaps = w.ballot([&](const S& s, int lane) { return lane < ni && !s.opens && s.lo != s.prev_hi; });
    w.each([&](S& s, int lane) {
        const U upto = (2ull << lane) - 1ull, above = heads & ~upto;
        const int head = 63 - __builtin_clzll((heads & upto) | 1ull);  // bit 0 is set whenever there is an item
        s.v0 = s.excl - w.from(&S::excl, head, s);
        s.end = above ? __builtin_ctzll(above) : ni;
        const int excl_end = w.from(&S::excl, s.end < 63 ? s.end : 63, s);
        s.rows = (s.end < ni ? excl_end : total) - s.excl;
        s.tiles = s.opens ? (s.rows + BM - 1) / BM : 0;
    });
    w.prefix(&S::tiles, &S::tincl);
    // a well-formed list (non-decreasing offsets) stays below the bound; overlapping segments are cut off here
    const int nt = w.at(&S::tincl, 63);
    m.n_tiles = nt < max_tiles ? nt : max_tiles;
    return m;
}
// tile t: its record, the items that have rows in it and its range of group rows
struct SmallTile { int row0, nrows, expert, gather, v_lo; unsigned long long in; };
template <class W> __host__ __device__ __forceinline__ SmallTile small_tile(const W& w, const SmallMap& m, int t, int BM) {
    using S = SmallItem;
    SmallTile r;
    const int g = 63 - __builtin_clzll(w.ballot([&](const S& s, int) { return s.opens && s.tincl - s.tiles <= t; }));
    const int v_lo = (t - (w.at(&S::tincl, g) - w.at(&S::tiles, g))) * BM, rows = w.at(&S::rows, g), g_end = w.at(&S::end, g);
    const int v_hi = rows < v_lo + BM ? rows : v_lo + BM;
    r.in = w.ballot([&](const S& s, int lane) { return lane >= g && lane < g_end && s.v0 < v_hi && s.v0 + s.len > v_lo; });
    const int f = __builtin_ctzll(r.in);
    r.row0 = w.at(&S::lo, f) + v_lo - w.at(&S::v0, f);
    r.nrows = v_hi - v_lo;
    r.expert = w.at(&S::e, f);
    r.gather = (m.gaps & r.in & ~(1ull << f)) != 0 ? 1 : 0;            // a gap in front of an item that starts inside the tile
    r.v_lo = v_lo;
    return r;
}
// the table entries of item k of a gathered tile: rel[v] = val + v for lo <= v < hi
struct SmallRun { int lo, hi, val; };
template <class W> __host__ __device__ __forceinline__ SmallRun small_run(const W& w, const SmallTile& r, int k) {
    using S = SmallItem;
    const int v0 = w.at(&S::v0, k) - r.v_lo, hi = v0 + w.at(&S::len, k);
    return SmallRun{v0 > 0 ? v0 : 0, hi < r.nrows ? hi : r.nrows, w.at(&S::lo, k) - v0 - r.row0};
}

// STRIPS: a GEMM may be numbered in strips.  Without, the kernel is 0.5 us shorter, which shows in shares of 17 to 40 us.
template <bool STRIPS>
__global__ __launch_bounds__(256) void tilemap_small_kernel(const int32_t* __restrict__ seg_offset,
                                                            const int32_t* __restrict__ seg_expert, int nseg, int R,
                                                            int n_local, int gather, MapJobs jobs) {
    const MapJob& job = jobs.job[blockIdx.y];
    const TileMap m = job.m;
    const int wave_id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WaveLanes w;
    w.lane = threadIdx.x & 63;
    const int i = min(w.lane, nseg - 1);
    w.mine.off0 = seg_offset[i];
    w.mine.off1 = seg_offset[i + 1];
    w.mine.e = seg_expert[i];
    if (blockIdx.x == 0 && blockIdx.y == 0) zero_done(jobs.done, threadIdx.x, 256);
    const SmallMap sm = small_map(w, nseg, R, n_local, gather, job.bm, job.max_tiles);
    if (blockIdx.x == 0 && threadIdx.x == 0) *m.n_tiles = sm.n_tiles;
    if (STRIPS && wave_id == (int)gridDim.x * 4 - 1) write_strips(jobs, blockIdx.y, gridDim.y, sm.n_tiles, w.lane);   // often without a tile
    for (int t = wave_id; t < sm.n_tiles; t += gridDim.x * 4) {
        const SmallTile r = small_tile(w, sm, t, job.bm);
        if (w.lane == 0) {
            m.row0[t] = r.row0;
            m.nrows[t] = r.nrows;
            m.expert[t] = r.expert;
            m.gather[t] = r.gather;
        }
        if (!r.gather) continue;
        for (unsigned long long in = r.in; in; in &= in - 1) {
            const SmallRun run = small_run(w, r, __builtin_ctzll(in));
            for (int v = run.lo + w.lane; v < run.hi; v += 64) m.rel[(size_t)t * kRelPitch + v] = run.val + v;
        }
    }
}

// The segment list itself, for shares that take gemm_f32_kernel twice: its blocks take one tile each and every wave works it
// out from the list, instead of a map by a launch of its own.  A small fp32 share (256 tokens, 517 rows of 64 -> 128 -> 64) is
// bound by its launches: 32.1 -> 27.9 us with six instead of seven.  In the narrow tiles of decode steps the same gained
// nothing: the list is cold in every kernel, and what the map's launches cost (2 x 4.7 us) the four GEMMs took longer.  Up to 64
// segments, and few tiles (see kListTiles).
struct SegList { const int32_t *offset, *expert; int nseg, R, n_local, gather, max_tiles; };
__device__ __forceinline__ SmallMap load_segments(const SegList& g, int bm, WaveLanes& w) {
    w.lane = threadIdx.x & 63;
    const int i = min(w.lane, g.nseg - 1);
    w.mine.off0 = g.offset[i];
    w.mine.off1 = g.offset[i + 1];
    w.mine.e = g.expert[i];
    return small_map(w, g.nseg, g.R, g.n_local, g.gather, bm, g.max_tiles);
}
// rows of a tile (in it: 0 .. nrows - 1) -> offsets from its first row
template <int N> __device__ __forceinline__ void segment_rows(const WaveLanes& w, const SmallTile& r, int (&row)[N]) {
    if (!r.gather) return;
    int off[N];
#pragma unroll
    for (int i = 0; i < N; ++i) off[i] = 0;
    for (unsigned long long in = r.in; in; in &= in - 1) {
        const SmallRun run = small_run(w, r, __builtin_ctzll(in));
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (row[i] >= run.lo && row[i] < run.hi) off[i] = run.val + row[i];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) row[i] = off[i];
}

__global__ __launch_bounds__(kMapThreads) void tilemap_kernel(const int32_t* __restrict__ seg_offset,
                                                              const int32_t* __restrict__ seg_expert, int nseg, int R,
                                                              int n_local, int gather, MapJobs jobs) {
    const int BM = jobs.job[blockIdx.x].bm, max_tiles = jobs.job[blockIdx.x].max_tiles;
    const TileMap m = jobs.job[blockIdx.x].m;
    if (blockIdx.x == 0) zero_done(jobs.done, threadIdx.x, blockDim.x);
    __shared__ SegWork w;
    __shared__ int wave_cnt[kMapThreads / 64][MOE_MAX_LOCAL];
    __shared__ int wave_tot[3 * 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nth = blockDim.x, nw = nth >> 6;       // at least as many threads as segments (the launch sees to that)
    for (int i = tid; i <= nseg; i += nth) {
        w.raw_off[i] = seg_offset[i];
        if (i < nseg) w.raw_exp[i] = seg_expert[i];
    }
    for (int i = tid; i < (kMapThreads / 64) * MOE_MAX_LOCAL; i += nth) (&wave_cnt[0][0])[i] = 0;
    lds_barrier();
    tilemap_clean(w, nseg, R, n_local, tid, nth);
    lds_barrier();
    if (gather) {
        // rank among the segments of the same expert: inside the wave from ballots over the bits of the expert id
        const int e = tid < nseg ? w.raw_exp[tid] : -1;
        unsigned long long peers = __ballot(e >= 0);
#pragma unroll
        for (int b = 0; b < 6; ++b) {                // MOE_MAX_LOCAL = 64 experts: six bits
            const unsigned long long mb = __ballot((e >> b) & 1);
            peers &= ((e >> b) & 1) ? mb : ~mb;
        }
        const int rank_in_wave = __popcll(peers & ((1ull << lane) - 1ull));
        if (e >= 0 && rank_in_wave == 0) wave_cnt[wave][e] = __popcll(peers);
        lds_barrier();
        if (tid < n_local) {                         // exclusive scan over the waves, total per expert
            int run = 0;
#pragma unroll
            for (int wv = 0; wv < nw; ++wv) {
                const int c = wave_cnt[wv][tid];
                wave_cnt[wv][tid] = run;
                run += c;
            }
            w.cnt[tid] = run;
        }
        lds_barrier();
        if (e >= 0) w.v0[tid] = wave_cnt[wave][e] + rank_in_wave;
        if (wave == 0) {                             // where the items of every expert start
            const int c = lane < n_local ? w.cnt[lane] : 0;
            int incl = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(incl, o, 64);
                if (lane >= o) incl += up;
            }
            if (lane < n_local) w.pos[lane] = incl - c;
            if (lane == 63) w.n_items = incl;
        }
        lds_barrier();
        tilemap_place(w, nseg, R, tid, nth);
    } else if (tid == 0) {
        tilemap_merge(w, nseg, R);
    }
    lds_barrier();
    // groups: item tid opens one or not; prefix sums give the group of every item, the rows in front of it
    // and the gaps up to it
    const int ni = w.n_items;
    const bool live = tid < ni;
    const bool opens = live && tilemap_opens(w, tid, gather != 0);
    const bool gap = live && tilemap_gap(w, tid, gather != 0);
    const int len = live ? w.hi[tid] - w.lo[tid] : 0;
    Int3 ex;
    const Int3 tot = block_scan3(Int3{opens ? 1 : 0, len, gap ? 1 : 0}, &ex, wave_tot);
    const int ng = tot.a;
    int* rows_before = w.raw_off;                    // rows in front of each group (the raw list is no longer needed)
    if (live) {
        w.grp[tid] = ex.a + (opens ? 1 : 0) - 1;
        w.gaps[tid] = ex.c + (gap ? 1 : 0);
        if (opens) { w.g_first[ex.a] = tid; rows_before[ex.a] = ex.b; }
    }
    if (tid == 0) { w.g_first[ng] = ni; rows_before[ng] = tot.b; w.n_groups = ng; }
    lds_barrier();
    if (live) w.v0[tid] = ex.b - rows_before[w.grp[tid]];
    const int g_rows = tid < ng ? rows_before[tid + 1] - rows_before[tid] : 0;
    Int3 ex2;
    const Int3 tot2 = block_scan3(Int3{tid < ng ? (g_rows + BM - 1) / BM : 0, 0, 0}, &ex2, wave_tot);
    if (tid < ng) { w.g_rows[tid] = g_rows; w.g_tile0[tid] = ex2.a; }
    // a well-formed list (non-decreasing offsets) stays below the bound; overlapping segments are cut off here
    const int nt = tot2.a < max_tiles ? tot2.a : max_tiles;
    if (tid == 0) { w.g_tile0[ng] = tot2.a; w.n_tiles = nt; *m.n_tiles = nt; }
    write_strips(jobs, blockIdx.x, gridDim.x, nt, tid);
    lds_barrier();
    for (int t = tid; t < nt; t += nth) tilemap_tile(w, t, BM, m);
    if (!gather) return;
    // offset tables: every item works out its (at most two) runs of table entries; the runs are then parked
    // in LDS, over the item arrays that nobody needs any more, and written by whole waves, 64 entries a time
    RelJob job[2] = {{0, 0, 0}, {0, 0, 0}};
    if (live) tilemap_rel_jobs(w, tid, BM, nt, job);
    lds_barrier();
    static_assert(offsetof(SegWork, gaps) == 5 * kMaxSeg * sizeof(int), "the six item arrays must be contiguous");
    int* jd = &w.lo[0];                              // [2 * kMaxSeg] each
    int* jc = jd + 2 * kMaxSeg;
    int* jv = jc + 2 * kMaxSeg;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        jd[2 * tid + pass] = job[pass].dst;
        jc[2 * tid + pass] = job[pass].cnt;
        jv[2 * tid + pass] = job[pass].val;
    }
    lds_barrier();
    // the runs go round the waves (run j to wave j % nw) so that a short list still uses all of them; lane l of
    // wave w holds runs w + nw * l and w + nw * (64 + l), and the wave walks through them one at a time
    int d_reg[2], c_reg[2], v_reg[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int j = wave + nw * (64 * h + lane);
        d_reg[h] = jd[j];
        c_reg[h] = jc[j];
        v_reg[h] = jv[j];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        unsigned long long todo = __ballot(c_reg[h] > 0);
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int dst = __builtin_amdgcn_readlane(d_reg[h], src), cnt = __builtin_amdgcn_readlane(c_reg[h], src);
            const int val = __builtin_amdgcn_readlane(v_reg[h], src);
            for (int r = lane; r < cnt; r += 64) m.rel[(size_t)dst + r] = val + r;
        }
    }
}

enum { EPI_PLAIN = 0, EPI_SILU = 1, EPI_GELU = 2, EPI_SWIGLU = 3 };

__device__ __forceinline__ float silu_f(float a) { return a / (1.f + __expf(-a)); }
__device__ __forceinline__ float gelu_tanh_f(float a) {
    const float u = 0.7978845608028654f * (a + 0.044715f * a * a * a);
    return 0.5f * a * (1.f + tanhf(u));
}
template <int EPI> __device__ __forceinline__ float epilogue(float a, float b) {
    if (EPI == EPI_SILU) return silu_f(a);
    if (EPI == EPI_GELU) return gelu_tanh_f(a);
    if (EPI == EPI_SWIGLU) return silu_f(a) * b;
    return a;
}

// Tile number `id` of `total` = tiles_m * tiles_n -> (tile_m, tile_n); a bijection for every shape.
// Blocks are handed to the 8 XCDs round-robin (XCD = id % 8), each XCD has its own L2, and all of them
// share the memory-side cache.  The map gives XCD x a band of tiles_m / 8 consecutive M-tiles and lets it
// walk ALL N-tiles for that band, in groups of 8 (then 4, 2, 1) M-tiles, M fastest: the blocks resident on an
// XCD form a patch of a few M-tiles by a few N-tiles (few distinct operand tiles in its L2), and the 8 XCDs
// sweep the N-tiles in step with each other, so a B tile fetched for one XCD is in the memory-side cache
// when the other seven ask for it and the A bands stay there for the whole sweep.  The tiles_m % 8
// M-tiles that do not fill a band come last, cut evenly over the XCDs.
__host__ __device__ __forceinline__ void tile_of_block_bands(int id, int tiles_m, int tiles_n, int* tm, int* tn) {
    const int x = id % 8, j = id / 8;                        // XCD and position in that XCD's sequence
    const int q = tiles_m / 8;                               // M-tiles per band
    const int band = q * tiles_n;                            // tiles of a band
    if (j < band) {
        // group heights: 8 as often as it fits, then the binary digits of the rest, so that a height always
        // divides the 32 blocks resident on an XCD (a 8 x 4, 4 x 8, ... patch with no straddling rows)
        int in_g = j, h = 8, first = 0, rest = q;
        while (true) {
            while (h > rest) h >>= 1;
            const int sz = h * tiles_n;
            if (in_g < sz) break;
            in_g -= sz; first += h; rest -= h;
        }
        *tm = q * x + first + in_g % h;
        *tn = in_g / h;
        return;
    }
    const int lm = tiles_m - 8 * q;                          // left-over M-tiles (lm >= 1 here)
    const int left = lm * tiles_n;
    const int v = x * (left / 8) + min(x, left % 8) + (j - band);
    *tm = 8 * q + v % lm;
    *tn = v / lm;
}
// With fewer than 32 M-tiles a band is at most three rows of tiles (patches of 1 x 32 or 2 x 16 tiles: 33 or
// 18 operand tiles for the 32 resident blocks instead of 12); when the N side has thicker bands the same
// numbering is used with the roles of M and N exchanged: XCD x owns a band of N-tiles and all XCDs sweep
// the M-tiles in step.  Measured at the 4096 -> 14336 -> 4096 shape: +7 % on both GEMMs at 2000 rows (bands
// of one row), +2.5 % at 6745 and 7900 rows (three rows), +1 % at 4147 and 5000 (two rows); with bands of
// four to seven rows the exchange gains or loses less than 1 %, so those keep the M bands.
//
// bf16 grids of kFewestStripTiles to kStripTiles tiles that N does not band (see plan_strips), of GEMMs with K of least_strip_k and more, are
// numbered in strips instead: XCD x gets
// the x-th eighth of the tiles in an order that cuts N into strips and goes through a strip row by row, so that the tiles resident
// on an XCD form a patch about as high as it is wide.  Bands -> strips on the kernels as they are, one FFN after the other: left-over
// M-tiles and low bands, 2741 rows of 1152 -> 2304 -> 1152 for four experts 48.1 -> 47.2 us, 12000 of 1408 -> 2048 -> 1408 SwiGLU for
// eight 208.3 -> 205.3, 2476 of 3584 -> 2560 -> 3584 111.2 -> 105.2; thick M bands, 16384 of 2048 -> 2816 -> 2048 SwiGLU 420.8 -> 409.8, 16318 of
// 1664 -> 2816 -> 1664 253.0 -> 249.8, 20571 of 4096 -> 14336 -> 4096 (second GEMM) the same.  33 shares 1.009 in the geometric mean, three of
// them 0.984 to 0.991.  (Where N has the thicker bands, each XCD reads weights of its own, which strips do not keep up: up to 7 %
// slower.  Outside the two limits nothing was gained.)  fp32: 11 shares of 128 x 128 tiles 0.997 to 1.005, so those keep the bands.
// Working the numbers below out in every block costs 0.4 us of a GEMM that takes 12 to 17, so the tile map holds them.
__host__ __device__ __forceinline__ void tile_of_block_strips(int id, int total, int tiles_m, Strips p, int* tm, int* tn) {
    const int x = id % 8, base = total / 8, extra = total % 8;
    const int v = x * base + min(x, extra) + id / 8;         // place in the order
    const int head = p.more * (p.wide + 1) * tiles_m;        // tiles of the wider strips
    const unsigned w = p.wide + (v < head ? 1 : 0), u = v < head ? v : v - head;
    const unsigned row = u / w, strip = row / (unsigned)tiles_m;
    *tm = (int)(row - strip * (unsigned)tiles_m);
    *tn = (v < head ? 0 : p.more * (p.wide + 1)) + (int)(strip * w + (u - row * w));
}
__host__ __device__ __forceinline__ void tile_of_block(int id, int total, int tiles_m, int tiles_n, Strips strips, int* tm, int* tn) {
    if (strips.wide > 0) tile_of_block_strips(id, total, tiles_m, strips, tm, tn);
    else if (tiles_m / 8 < 4 && tiles_n / 8 > tiles_m / 8) tile_of_block_bands(id, tiles_n, tiles_m, tn, tm);
    else tile_of_block_bands(id, tiles_m, tiles_n, tm, tn);
}

// Tail splitting.  The grid runs in rounds of `ncu` tiles (one block per CU); the tiles of a last,
// mostly empty round would leave most CUs idle for a whole tile time.  When that round has at most
// ncu / 2 tiles, each of them is cut along K into `parts` pieces that run as separate blocks
// (1/parts of a tile time) and write fp32 partial tiles, which are added in piece order before the
// epilogue - at 128 x 128 by the piece that arrives last (see last_piece), else by gemm_bf16_tail_kernel.
// Everything here depends only on the shapes, so results do not vary from run to run; another tile
// height or another cut adds the products of a row in another order, i.e. may round the last bit differently.
struct TailPlan {
    int n_full;        // tiles handled whole: ids [0, n_full)
    int n_tail;        // tiles cut in pieces: ids [n_full, n_full + n_tail)
    int parts;         // pieces per tail tile (1: no tail)
    int pairs_per;     // k-tile pairs per piece
};
__host__ __device__ __forceinline__ TailPlan plan_tail(int total, int ncu, int nk) {
    TailPlan p;
    p.n_full = total; p.n_tail = 0; p.parts = 1; p.pairs_per = nk / 2;
    const int rem = total % ncu;
    const int npairs = nk / 2;
    if (rem == 0) return p;
    // up to 8 pieces of at least 16 k-tiles (more only add partial tiles) but for the last one, which has four at least: of p <= 8
    // pieces of ceil(npairs / p) pairs, npairs >= 8 p, the last has (npairs - (p - 1)^2) / p > 1 of them.  2 or 3 pieces pay for the extra
    // pass only when a piece is still long (64 k-tiles)
    const int parts = min(min(ncu / rem, npairs / 8), 8);
    if (parts < 2 || (parts < 4 && npairs / parts < 32)) return p;
    p.pairs_per = (npairs + parts - 1) / parts;
    p.parts = (npairs + p.pairs_per - 1) / p.pairs_per;
    p.n_tail = rem;
    p.n_full = total - rem;
    return p;
}
// ... with a tail of at most `most_tail` tiles, which the launch has made room for; else none
__host__ __device__ __forceinline__ TailPlan plan_tail_upto(int most_tail, int total, int ncu, int nk) {
    const TailPlan p = plan_tail(total, ncu, nk);
    return p.n_tail <= most_tail ? p : TailPlan{total, 0, 1, nk / 2};
}

// Which items (tiles, then pieces) a block of the bf16 GEMM walks through: item, item + ncu, ... below end.  Place p of the
// ncu places works through items p, p + ncu, ... in runs of `walk`, a block for each.  The places' runs end one after the
// other, not all at once: whenever a run ends its CU is free for what other streams have queued.  Blocks start in the
// order of their numbers, and so do the runs of a generation end.  No cut when there are no more than `walk` rounds.
struct WalkRun { int item, end; };
__host__ __device__ __forceinline__ WalkRun walk_run(int block, int ncu, int walk, int n_items) {
    const int gen = block / ncu, place = block % ncu;
    const int ahead = n_items <= walk * ncu ? 0 : (ncu - 1 - place) * walk / ncu;   // rounds that this place's runs end early
    const int r0 = gen * walk - ahead, r1 = r0 + walk;
    const int first = (r0 > 0 ? r0 : 0) * ncu + place, end = r1 * ncu;
    return WalkRun{first, end < n_items ? end : n_items};
}

// ------------------------------------------------------------------------------------ fp32
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// C[r, n] = epi( sum_k A[r,k] * B0[n,k], sum_k A[r,k] * B1[n,k] ) on v_mfma_f32_32x32x2_f32 (fp32 operands and
// accumulation, like a chain of fmaf).  64 x 64 block tile, 4 waves 2 x 2 of one 32 x 32 tile each, k-tiles of 32.
// The matrix core's fp32 rate (256 flop per clock and CU; 155 TFLOP/s from registers alone) is the bound, and the tile
// is small so that three blocks (48 KB of LDS each) share a CU, which hides prologues and epilogues and keeps the last
// round short: 3001 rows of 1024 -> 2816 -> 1024 SwiGLU are 16.5 + 3 tiles per CU.  Operands go global -> LDS directly
// through a ring of three k-tiles, one wave-load per k-step between the MFMAs, fragments are read one k-step ahead,
// one barrier per k-tile.  The pair of GEMMs of that layer: 500 us with the operands staged through registers one
// k-tile ahead, 475 with direct loads issued together, 415 with them spread over the k-steps on scalar bases
// (125 TFLOP/s); tiles of 128 x 64 and 128 x 128 take 455 and 480 (4.1 rounds, and 0.75 of one).
//
// Operands: the order of the sum over k is free, so lane half h takes k-chunk 2 s + h (four floats, one
// ds_read_b128) of k-step s and feeds float v of both operands to MFMA v.  LDS: 8 chunks of 16 bytes per row,
// slot(r, c) = 8 r + (c ^ ((r >> 1) & 7)): the 16 consecutive rows that a read serves at a time fall on all 64 banks,
// and a wave-load fills 8 rows with 128 contiguous bytes each.
// SwiGLU: a wave's 32 weight rows are 16 gate rows and the 16 up rows of the same columns (accumulator elements
// 0-7 and 8-15), so the activation needs no exchange.  D = B . A^T: a lane ends with 4 consecutive columns of a row.
constexpr int FM = 64, FN = 64, FK = 32;
constexpr int kF32TileBytes = FM * FK * 4;     // one operand tile: 8 KB
constexpr int kF32Stages = 3;
__device__ __forceinline__ int f32_slot(int r, int c) { return (r << 3) + (c ^ ((r >> 1) & 7)); }

template <int EPI, bool SEG>
__global__ __launch_bounds__(256, 3) void gemm_f32_kernel(const float* __restrict__ A, int lda, TileMap m, SegList seg,
                                                          ExpertTable tab, int which0, int which1, int N, int K,
                                                          float* __restrict__ C, int ldc, int tiles_n) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kF32Stages * 2 * kF32TileBytes];
    constexpr int NOUT = (EPI == EPI_SWIGLU) ? FN / 2 : FN;                 // output columns per block
    WaveLanes lanes;
    SmallMap map;
    if constexpr (SEG) map = load_segments(seg, FM, lanes);
    const int n_tiles_m = SEG ? __builtin_amdgcn_readfirstlane(map.n_tiles) : *m.n_tiles;
    const int total = n_tiles_m * tiles_n;
    for (int id = blockIdx.x; id < total; id += gridDim.x) {   // one: always with a map, else unless the list has more runs than experts
        int tile_m, tile_n;
        tile_of_block(id, total, n_tiles_m, tiles_n, Strips{0, 0}, &tile_m, &tile_n);
        SmallTile t{};
        const int32_t* rel = nullptr;
        if constexpr (SEG) {
            tile_m = __builtin_amdgcn_readfirstlane(tile_m);
            t = small_tile(lanes, map, tile_m, FM);
        } else {
            t.row0 = m.row0[tile_m]; t.nrows = m.nrows[tile_m]; t.expert = m.expert[tile_m];
            rel = m.gather[tile_m] ? m.rel + (size_t)tile_m * kRelPitch : nullptr;
        }
        const int row0 = t.row0, nrows = t.nrows, ex = t.expert;
        auto pick = [&](int which) -> const float* {
            return reinterpret_cast<const float*>(which == 0 ? tab.w1[ex] : which == 1 ? tab.w_up[ex] : tab.w_down[ex]);
        };
        const float* B0 = pick(which0);
        const float* B1 = (EPI == EPI_SWIGLU) ? pick(which1) : B0;
        const int n0 = tile_n * NOUT;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int wm = wave >> 1, wn = wave & 1;

        // wave-load i (of 2 per operand) fills rows 8 (wave + 4 i) .. + 7: this lane fetches one chunk of one row.  Addresses
        // are a scalar base plus a 32-bit offset per lane.  Chunks past K are fetched clamped to the row's last one and
        // zeroed when they are read.
        const int nchunk = K / 4, nk = (K + FK - 1) / FK;   // K is a multiple of 4
        // byte offset of the lane's chunk inside a k-tile's 128 bytes: row r = 8 (wave + 4 i) + lane / 8, so (r >> 1) & 7 does not depend on i
        const uint32_t chunk = (uint32_t)(((lane & 7) ^ (((wave & 1) << 2) + (lane >> 4))) * 16);
        const uint32_t chunk_last = min(chunk, (uint32_t)((nchunk - 1) * 16 - (nk - 1) * (FK * 4)));
        const char* a_base = reinterpret_cast<const char*>(A + (size_t)row0 * lda);
        const char* b_base[2];
        uint32_t a_voff[2], b_voff[2];
        // rows that this lane fetches, and the one whose products it ends up with
        int rows[3] = {min(wave * 8 + (lane >> 3), nrows - 1), min((wave + 4) * 8 + (lane >> 3), nrows - 1), min(wm * 32 + (lane & 31), nrows - 1)};
        if constexpr (SEG) segment_rows(lanes, t, rows);
        else if (rel) {                                // gathered tile: offsets below 2^32 bytes (checked on the host)
#pragma unroll
            for (int i = 0; i < 3; ++i) rows[i] = rel[rows[i]];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r0 = (wave + 4 * i) * 8;         // wave-uniform
            a_voff[i] = (uint32_t)rows[i] * (uint32_t)lda * 4u;
            const int col0 = (EPI == EPI_SWIGLU) ? (r0 >> 5) * 16 + (r0 & 15) : r0;
            b_base[i] = reinterpret_cast<const char*>(((EPI == EPI_SWIGLU && (r0 & 16)) ? B1 : B0) + (size_t)n0 * K);
            b_voff[i] = (uint32_t)min(col0 + (lane >> 3), N - 1 - n0) * (uint32_t)K * 4u;
            asm volatile("" : "+v"(a_voff[i]), "+v"(b_voff[i]));   // stay 32-bit lane offsets next to a scalar base
        }
        // loads [lo, hi) of the four of k-tile kt; past the end the last k-tile is fetched again: their count stays uniform
        auto issue = [&](int kt, int stage, int lo, int hi) {
            kt = min(kt, nk - 1);
            const uint32_t ch = kt == nk - 1 ? chunk_last : chunk;
            unsigned char* st = lds + stage * 2 * kF32TileBytes + wave * 1024;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                if (it < lo || it >= hi) continue;
                const bool is_a = it < 2;
                const int i = it & 1;
                const char* p = (is_a ? a_base : b_base[i]) + (size_t)kt * (FK * 4);
                uint32_t v = (is_a ? a_voff[i] : b_voff[i]) + ch;
                asm volatile("" : "+s"(p), "+v"(v));
                __builtin_amdgcn_global_load_lds(p + v, (__attribute__((address_space(3))) void*)(st + (is_a ? 0 : kF32TileBytes) + i * 4096), 16, 0, 0);
            }
        };
        issue(0, 0, 0, 4);
        issue(1, 1, 0, 3);                             // the fourth goes out in the first k-step below
        const int fr = lane & 31, fk = lane >> 5;
        int a_off[4], b_off[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            a_off[s] = f32_slot(wm * 32 + fr, 2 * s + fk) * 16;
            b_off[s] = kF32TileBytes + f32_slot(wn * 32 + fr, 2 * s + fk) * 16;
        }
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        f32x4 af[2], bf[2];
        auto read = [&](const unsigned char* st, int s) {
            af[s & 1] = *reinterpret_cast<const f32x4*>(st + a_off[s]);
            bf[s & 1] = *reinterpret_cast<const f32x4*>(st + b_off[s]);
        };
        // the MFMAs of k-step s of k-tile kt; behind the first the fragments of the next k-step are read, behind the second
        // load `it` of k-tile t_load goes out
        auto step = [&](const unsigned char* st_next, int kt, int s, bool ragged, int t_load, int slot, int it) {
            __builtin_amdgcn_sched_barrier(0);
            if (ragged && kt * (FK / 4) + 2 * s + fk >= nchunk)   // zero in both: 0 * a stray infinity would be a NaN
                af[s & 1] = bf[s & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
            read(st_next, (s + 1) & 3);
            issue(t_load, slot, it, it + 1);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf[s & 1][v], af[s & 1][v], acc, 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        int cur = 0;                                   // ring slot of k-tile kt
        auto trip = [&](int kt, bool ragged) {
            const int nxt = cur == kF32Stages - 1 ? 0 : cur + 1, prev = cur == 0 ? kF32Stages - 1 : cur - 1;
            const unsigned char* st = lds + cur * 2 * kF32TileBytes;
            // slot `prev` was last read in trip kt - 1, whose barrier every wave has passed: k-tile kt + 2 goes there
            step(st, kt, 0, ragged, kt + 1, nxt, 3);
            step(st, kt, 1, ragged, kt + 2, prev, 0);
            step(st, kt, 2, ragged, kt + 2, prev, 1);
            __builtin_amdgcn_s_waitcnt(0x0070 | 2);    // vmcnt(2) lgkmcnt(0): k-tile kt + 1 is in LDS, this wave has read all of kt
            __builtin_amdgcn_s_barrier();
            step(lds + nxt * 2 * kF32TileBytes, kt, 3, ragged, kt + 2, prev, 2);
            cur = nxt;
        };
        __builtin_amdgcn_s_waitcnt(0x0F70 | 3);        // vmcnt(3): k-tile 0 is in LDS
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read(lds, 0);
        for (int kt = 0; kt < K / FK; ++kt) trip(kt, false);
        if (K % FK != 0) trip(nk - 1, true);
        __builtin_amdgcn_s_waitcnt(0x0070);            // no load may still target LDS when the block ends
        if (wm * 32 + fr < nrows) {
            float* crow = C + (size_t)(row0 + rows[2]) * ldc;
#pragma unroll
            for (int g = 0; g < ((EPI == EPI_SWIGLU) ? 2 : 4); ++g) {
                f32x4 v;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = epilogue<EPI>(acc[4 * g + t], (EPI == EPI_SWIGLU) ? acc[4 * (g & 1) + 8 + t] : 0.f);
                const int col = n0 + wn * (NOUT / 2) + g * 8 + fk * 4;
                if (col < N) *reinterpret_cast<f32x4*>(crow + col) = v;            // N is a multiple of 4
            }
        }
        if constexpr (!SEG) return;
        __builtin_amdgcn_s_barrier();              // the next item's loads go to the same LDS
    }
}

// ------------------------------------------------------------------------------------ bf16 MFMA
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 32, STAGES = 5;
// Block tile of MI x NJ: the 4 waves are 2 x 2, a wave holds 32 MI rows by 32 NJ weight rows.
//   4 x 4  256 x 256, all 160 KB of LDS, one block per CU: the fewest operand bytes per flop
//   3 x 4  192 x 256, 140 KB, one block per CU
//   2 x 2  128 x 128, 80 KB, two blocks per CU
// The last two are for grids that 256 x 256 tiles do not fill (see choose_shape).
template <int MI, int NJ> struct TileGeom {
    static constexpr int BM = 64 * MI, BN = 64 * NJ;
    static constexpr int A_BYTES = BM * BK * 2;              // A tile of a stage (one 32-wide k-tile); the B tile follows
    static constexpr int STAGE = A_BYTES + BN * BK * 2;
    static constexpr int LDS = STAGES * STAGE;
    static constexpr int PER_CU = (160 * 1024) / LDS;        // blocks that share a CU
    static constexpr size_t PARTIAL = (size_t)BM * BN * sizeof(float);   // one fp32 partial tile
    static constexpr bool SUM_IN_PLACE = PARTIAL <= 64 * 1024;           // how the pieces of a cut tile are added (see last_piece)
};
constexpr int BM = TileGeom<4, 4>::BM;         // rows of the largest tile

// An operand tile is stored as blocks of 16 rows; a block is 1 KB = 64 slots of
// 16 bytes and is filled by ONE wave-wide direct-to-LDS load (lane l fills slot l).
// Inside a block the rows are kept row-major (4 slots per row, so 4 neighbouring
// lanes fetch 64 contiguous bytes of one row from memory), with the 16-byte chunk
// index XOR-ed by -row/4:
//     slot(r, c) = 4*r + (c ^ (-(r >> 2) & 3)),   r = 0..15, c = 0..3.
// The LDS has 64 banks and serves a ds_read_b128 sixteen lanes at a time: lanes 0-3, 12-15 and 20-27 of the
// lower half, its others, and the same of the upper half.  Those of an MFMA operand read - one chunk of 16 rows, or chunk l / 16
// of row l % 16 - fall on 16 different values of slot % 16, i.e. on all 64 banks once.  (With r >> 2 in place of its
// negative the second kind of read takes twice as long: 256 x 256 tiles 5 % slower.)
__device__ __forceinline__ int slot_of(int r, int c) { return (r << 2) + (c ^ (-(r >> 2) & 3)); }
// inverse for the loading lane: which (row, chunk) of the block lane l must fetch
__device__ __forceinline__ void rc_of_slot(int l, int* r, int* c) {
    *r = l >> 2;
    *c = (l & 3) ^ (-(l >> 4) & 3);
}
// byte offset of (row, chunk) inside an operand tile
__device__ __forceinline__ int tile_off(int row, int c) { return ((row >> 4) << 10) + (slot_of(row & 15, c) << 4); }

__device__ __forceinline__ float fast_silu(float a) {
    return a * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896f * a));
}
// tanh-form GELU: 0.5 a (1 + tanh(u)) = a * sigmoid(2u), u = sqrt(2/pi) (a + 0.044715 a^3); one exp2 and one rcp
// (the exponent -log2(e) * 2u = a * (k1 + k2 a^2) is formed with the constants folded: five plain operations around the two slow ones)
__device__ __forceinline__ float fast_gelu(float a) {
    const float k1 = -1.44269504088896f * 1.5957691216057308f, k2 = k1 * 0.044715f;
    const float arg = a * __builtin_fmaf(k2, a * a, k1);
    return a * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(arg));
}
template <int EPI> __device__ __forceinline__ float epilogue_bf16(float a, float b) {
    if (EPI == EPI_SILU) return fast_silu(a);
    if (EPI == EPI_GELU) return fast_gelu(a);
    if (EPI == EPI_SWIGLU) return fast_silu(a) * b;
    return a;
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    const bf16x2 b = __builtin_convertvector(v, bf16x2);      // round to nearest even in hardware
    return *reinterpret_cast<const uint32_t*>(&b);
}

// The pieces of a tile that is cut along K.  Every piece writes its fp32 accumulators; at 128 x 128 (and in the
// weight-streaming kernels) the block that arrives last (a counter per tile, nobody waits) adds all pieces in piece
// order - its own is read back like the others, so the result does not depend on who was last - and finishes the
// tile.  A kernel of its own for the sums costs 4.5 us where there is nothing to add and 5-16 us where there is, each
// time behind a launch gap; the last block reads up to half a megabyte (32 pieces of a weight-streaming tile: 1 MB) in
// about as long, without the gap.  The larger tiles have 0.8 to 2 MB of pieces, which take one block 20 us and more (93
// against 108 us for the second GEMM at 4096 -> 14336 -> 4096 and 701 rows): those are added by gemm_bf16_tail_kernel,
// spread over the chip.
// The writers may sit on other XCDs, whose L2s do not see each other: pieces are stored and read with accesses of
// agent scope (sc1: written through, read past the L2), the counter is an agent-scope atomic, and a wave's stores have
// completed (vmcnt(0)) before its block counts.  The same with plain accesses between __threadfence()s was far
// slower: every fence writes back the whole L2 (54 against 17 us at 110 tiles of four pieces).
constexpr int kAgentScope = 16;                              // cache policy bits of a buffer access: sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pieces_rsrc(const float* partial, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(partial), 0, bytes, 0x00027000);
}
__device__ __forceinline__ void store_piece(__amdgpu_buffer_rsrc_t r, int quad, const f32x4& v) {   // 16 bytes at quad * 16
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, quad * 16, 0, kAgentScope);
}
__device__ __forceinline__ f32x4 load_piece(__amdgpu_buffer_rsrc_t r, int quad) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, quad * 16, 0, kAgentScope));
}
__device__ __forceinline__ bool last_piece(int32_t* done, int parts, int* lds_flag) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);                        // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    if (threadIdx.x == 0) *lds_flag = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
    __syncthreads();
    asm volatile("" ::: "memory");
    return *lds_flag != 0;
}

// The same products on the bf16 matrix cores, for grids that fill the chip with 128 x 128 tiles (see take_f32_kernels).
//
// A float of 24 bits is the sum of three bf16 numbers of 8 bits and a sign, x = x0 + x1 + x2, each the rest rounded to nearest
// (the differences are exact), and x w = x0 w0 + (x0 w1 + x1 w0) + (x1 w1 + x0 w2 + x2 w0) + terms below 2^-24 of it: six
// products of v_mfma_f32_32x32x16_bf16 in 192 clocks per 16 elements of K instead of 512 for v_mfma_f32_32x32x2_f32.  (The
// splitting and the six products are those of G. Henry, P. Tang and A. Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019.)  bf16 has the exponents of fp32, so no element needs a scale
// and none hides behind a larger one.  Products of parts are exact, and the small ones are accumulated apart from x0 w0, so
// that they are not rounded to its last bit: against 64 bits the FFN is off by a quarter of what the chain of fp32 products is (3001
// rows of 1024 -> 2816 -> 1024, normal, uniform, heavy-tailed and unevenly scaled operands: 1.4e-7 ... 2.8e-7 against 7.4e-7 ...
// 1.16e-6, also behind elements of 2^20 to 2^60 that meet zeros).  A single product is off by 0.43 x 2^-24 rms and below 2^-23, one
// of fp32 by 0.42 x 2^-24 and up to 2^-24: for rows with one nonzero element both FFNs are off by 5.7e-8.
//
// What parts cannot give is taken from the fp32 matrix cores, element by element (multiply_exactly): a sum that is not finite
// (infinities, NaN, and elements that bf16 rounds to infinity), and one so small that what lies below the range of the parts
// could count in it: less than K 2^-100 times the largest element of its row or weight row, and 1 (rows of zeros have
// nothing to lose).  Small are then the sums of both groups of waves below: one that merely cancels, which one in 10^8 does, has
// lost nothing that counts.  The other elements of the tile stay as they are: no row depends on its neighbours.
//
// 128 x 128 block tile, k-tiles of 32, 8 waves: two groups of 2 x 2 waves, 64 x 64 each, group g taking half g of every
// k-tile; the groups' sums are exchanged through LDS at the end and each group finishes half of the rows: two waves per
// SIMD on one tile per CU.  Every element is split once per block: loaded to registers three k-tiles
// ahead, split between the products and written to LDS as three planes one ahead (two stages of 48 KB).
// A k-tile takes about 2450 clocks at 2 GHz for 1536 of products: without the vector work of splitting 2050, and a third stage with
// the next fragments read in front of the barrier left it where it is (power: the clock rises by what the units do less).
// The pair of GEMMs of 3001 rows of 1024 -> 2816 -> 1024 SwiGLU takes 410 us with gemm_f32_kernel and 330 here; 20000 rows,
// SiLU: 1750 -> 1290 (179 TFLOP/s; the fp32 instruction reaches 155 from registers).  With all results of a GEMM below the limit: 3001
// rows, SiLU, 283 -> 490 for one GEMM of the two, 730 for both (234 above it).
// Blocks walk through tiles like those of gemm_bf16_kernel: the loads run on into the next tile.
//
// Plane of an operand tile: 128 rows x 32 elements as blocks of 16 rows x 4 chunks of 16 bytes (tile_off, conflict-free).
// The order of the sum over k is free: chunk c holds elements 4 c .. 4 c + 3 and 16 + 4 c .. + 3 of the k-tile, so that
// four lanes fetch 64 contiguous bytes of a row per load.
constexpr int XM = 128, XN = 128, XK = 32;
constexpr int kXPlane = XM * XK * 2;                     // 8 KB
constexpr int kXOperand = 3 * kXPlane;
constexpr int kXStage = 2 * kXOperand;                   // A, then B
constexpr int kXGive = 32 * 1024;                        // sums of a group that the other one finishes; both groups' begin in the second stage
constexpr int kXLargest = kXStage + 2 * kXGive;          // largest elements of the rows and weight rows of a tile
constexpr int kXFlag = kXLargest + (XM + XN) * 4;        // whether this block adds the pieces of a tile
constexpr int kXLds = kXFlag + 16;
static_assert(2 * kXGive >= kXStage, "");
constexpr int kXMinK = 4 * XK;                           // a walk reads three k-tiles ahead: at most into the next tile
constexpr float kPartsFloor = 0x1p-100f;

// The tiles of a last round that leaves most CUs idle are cut along K into `parts` pieces of at least kXCutMin k-tiles, one per
// block.  A piece writes its sums (fp32, 64 KB) and the largest elements of its rows and weight rows; the block whose
// piece of a tile arrives last adds them in order and finishes the tile.
// A k-tile takes 0.93 us on an empty chip and 0.3 more on a full one, and pieces on all CUs cost 17 us (fit over 36 of 120
// shares of 300 to 16000 rows); a round is cut where that leaves a gain: 8355 rows of 512 -> 2048 -> 512 (8 of 264 tiles in the second
// GEMM's last round, K = 2048) 293 -> 252 us, 7064 of 768 -> 2304 -> 768 332 -> 301, 3001 of 1024 -> 2816 -> 1024 SwiGLU (32 of 1056
// tiles, K = 1024) first GEMM 229 -> 218.  Shares that cross from one tile into the next, for rounds that are more than half full (192
// tiles of K = 2816), gained nothing: the chip is slower by about what it is fuller.
constexpr int kXCutMin = 8;
constexpr size_t kXPiece = (size_t)(XM * XN + XM + XN) * sizeof(float);
struct PartsCut {
    int n_full;        // tiles taken whole: ids [0, n_full)
    int n_cut;         // the others, each as
    int parts, per;    // ... parts pieces of per k-tiles (the last one may be shorter)
};
__host__ __device__ __forceinline__ PartsCut plan_parts(int total, int ncu, int nk) {
    const PartsCut whole{total, 0, 1, nk};
    const int rest = total % ncu;
    if (2 * rest > ncu || rest == 0) return whole;
    const int most = min(ncu / rest, nk / kXCutMin);
    if (most < 2) return whole;
    const int per = ((nk + most - 1) / most + 1) & ~1;     // pieces begin at even k-tiles
    const int parts = (nk + per - 1) / per, places = rest * parts;
    // in nanoseconds: the round as it is, as pieces, and what those cost, half as much again
    if (nk * (932 + 299 * rest / ncu) - per * (932 + 299 * places / ncu) < 26000 * places / ncu) return whole;
    return PartsCut{total - rest, rest, parts, per};
}

// m or the larger of |a| and |b| (neither is taken for a NaN)
__device__ __forceinline__ float largest_of(float m, float a, float b) {
    asm("v_max3_f32 %0, %0, abs(%1), abs(%2)" : "+v"(m) : "v"(a), "v"(b));
    return m;
}

// A lane's part of an operand pair on its way from floats to planes: 2 x 4 elements of A and of B, taken in pairs u = 0 .. 7,
// each in three phases.
struct Splitter {
    u32x4 part[2][3];                                      // [A, B][plane]
    f32x2 rest;
    __device__ __forceinline__ uint32_t take() {           // nearest bf16 of the rest, which it leaves
        const bf16x2 b = __builtin_convertvector(rest, bf16x2);
        return __builtin_bit_cast(uint32_t, b);
    }
    __device__ __forceinline__ void phase(const f32x4 (&q)[4], float (&largest)[2], int p, unsigned char* st) {
        const int u = p / 3, n = p % 3, op = u >> 2;
        if (n == 0) {
            rest = f32x2{q[u >> 1][2 * (u & 1)], q[u >> 1][2 * (u & 1) + 1]};
            largest[op] = largest_of(largest[op], rest.x, rest.y);
        }
        const uint32_t b = take();
        part[op][n][u & 3] = b;
        if (n < 2) rest = f32x2{rest.x - bf16_bits_to_f32(b & 0xffffu), rest.y - __uint_as_float(b & 0xffff0000u)};
        if ((u & 3) == 3) *reinterpret_cast<u32x4*>(st + op * kXOperand + n * kXPlane) = part[op][n];
    }
};
__device__ __forceinline__ void split_parts(const f32x4 (&q)[4], float (&largest)[2], unsigned char* st) {
    Splitter s;
#pragma unroll
    for (int p = 0; p < 24; ++p) s.phase(q, largest, p, st);
}
// 64 x 64 x 16 ([row tile][weight-row tile], D^T: rows n, columns m) while the next k-tile is split: a product, then a
// handful of vector instructions, held together (the scheduler left to itself puts all products first)
typedef f32x16 Acc22[2][2];
__device__ __forceinline__ void multiply_parts(const unsigned char* pa, const unsigned char* pb, Acc22& hi, Acc22& lo, const f32x4 (&q)[4],
                                               float (&largest)[2], unsigned char* then) {
    bf16x8 a[3][2], b[3][2];
    auto read = [&](bf16x8 (&f)[3][2], const unsigned char* p, int n) {
#pragma unroll
        for (int i = 0; i < 2; ++i) f[n][i] = *reinterpret_cast<const bf16x8*>(p + n * kXPlane + i * 2048);
    };
    read(a, pa, 0);
    read(b, pb, 0);
    read(b, pb, 1);
    read(a, pa, 1);
    Splitter s;
    constexpr int term[6][2] = {{0, 0}, {0, 1}, {1, 1}, {1, 0}, {2, 0}, {0, 2}};   // part of A, of B
#pragma unroll
    for (int t = 0; t < 24; ++t) {
        const int i = (t >> 1) & 1, j = t & 1;
        __builtin_amdgcn_sched_barrier(0);
        f32x16& acc = t < 4 ? hi[i][j] : lo[i][j];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[term[t >> 2][1]][j], a[term[t >> 2][0]][i], acc, 0, 0, 0);
        if (t == 9) read(a, pa, 2);
        if (t == 13) read(b, pb, 2);
        // 24 phases behind the first 22 products: the last of them are in LDS by the barrier
        if (t < 20) s.phase(q, largest, t, then);
        if (t == 20 || t == 21) {
            s.phase(q, largest, 2 * t - 20, then);
            s.phase(q, largest, 2 * t - 19, then);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}
// one 32 x 32 tile and its neighbour (rows of b[1]) on the fp32 matrix cores, straight from memory
__device__ __forceinline__ void multiply_exactly(const float* pa, const float* pb0, const float* pb1, int fk, int K, f32x16 (&acc)[2]) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
    // where few waves need it, bound by the round trips of the loads: those of four steps of 8 elements go out at once, under no
    // condition (past K, a multiple of 4, the last quad again, which does not count).  3001 rows of 1024 -> 2816 -> 1024 with the largest
    // floats in two rows 346 -> 327 us, without them 234; where all need it the 32-byte loads of each row count, not their latency.
    constexpr int STEPS = 4;
    for (int k0 = 0; k0 < K; k0 += 8 * STEPS) {
        f32x4 a[STEPS], b0[STEPS], b1[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int kc = min(k0 + 8 * s + 4 * fk, K - 4);
            a[s] = *reinterpret_cast<const f32x4*>(pa + kc);
            b0[s] = *reinterpret_cast<const f32x4*>(pb0 + kc);
            b1[s] = *reinterpret_cast<const f32x4*>(pb1 + kc);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const bool in = k0 + 8 * s + 4 * fk < K;
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};       // in all three: 0 * a stray infinity would be a NaN
            a[s] = in ? a[s] : zero;
            b0[s] = in ? b0[s] : zero;
            b1[s] = in ? b1[s] : zero;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(b0[s][v], a[s][v], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(b1[s][v], a[s][v], acc[1], 0, 0, 0);
            }
        }
    }
}

// CUT: the last round's tiles may be cut along K (see plan_parts).  The code for pieces costs short tiles 2 to 4 % (scalar registers
// on their way from one tile to the next), so shares that have none run without it.
template <int EPI, bool CUT>
__global__ __launch_bounds__(512, 2) void gemm_f32_parts_kernel(const float* __restrict__ A, int lda, TileMap m, ExpertTable tab,
                                                                int which0, int which1, int N, int K, float* __restrict__ C, int ldc,
                                                                int tiles_n, int ncu, int walk, float* partial) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int NOUT = (EPI == EPI_SWIGLU) ? XN / 2 : XN;
    const int n_tiles_m = *reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(m.n_tiles));
    const int total = n_tiles_m * tiles_n;
    const int nk_all = ((K + XK - 1) / XK + 1) & ~1;       // even; k-tiles past K count as zeros
    PartsCut cut = {total, 0, 1, nk_all};
    if (CUT) {
        cut = plan_parts(total, ncu, nk_all);
        cut.n_full = __builtin_amdgcn_readfirstlane(cut.n_full);
        cut.n_cut = __builtin_amdgcn_readfirstlane(cut.n_cut);
        cut.parts = __builtin_amdgcn_readfirstlane(cut.parts);
        cut.per = __builtin_amdgcn_readfirstlane(cut.per);
    }
    const WalkRun run = walk_run(blockIdx.x, ncu, walk, cut.n_full + cut.n_cut * cut.parts);   // whole tiles, then pieces
    int item = __builtin_amdgcn_readfirstlane(run.item);
    const int end_item = __builtin_amdgcn_readfirstlane(run.end);
    if (item >= end_item) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int fr = lane & 31, fk = lane >> 5;
    const int k_full = K / XK;                             // k-tiles without an end of K in them

    struct Tile { int row0, nrows, n0, ex, nk, piece; const int32_t* rel; };   // nk: k-tiles of it that this block takes; piece < 0: all
    struct Source { __amdgpu_buffer_rsrc_t a, b; uint32_t a_voff, b_voff; int k0; };
    constexpr uint32_t kNoOffset = 0xFFFFFFF0u;               // past the end of the buffer (row offsets end below it, see ffn_impl)
    // what this lane fetches: chunk `lc` of tile row 16 wave + lane / 4, of A and of B; it goes to slot `lane` of block `wave`
    const int lc = (lane & 3) ^ (-(lane >> 4) & 3);
    auto weights = [&](int which, int ex) { return reinterpret_cast<const char*>(which == 0 ? tab.w1[ex] : which == 1 ? tab.w_up[ex] : tab.w_down[ex]); };
    auto describe = [&](int id, Tile& t, Source& s) {
        int tile_m, tile_n;
        s.k0 = 0;
        t.nk = nk_all;
        t.piece = -1;
        if (CUT && id >= cut.n_full) {
            t.piece = __builtin_amdgcn_readfirstlane((id - cut.n_full) / cut.n_cut);
            id -= t.piece * cut.n_cut;
            s.k0 = t.piece * cut.per;
            t.nk = min(cut.per, nk_all - s.k0);
        }
        tile_of_block(id, total, n_tiles_m, tiles_n, Strips{0, 0}, &tile_m, &tile_n);
        tile_m = __builtin_amdgcn_readfirstlane(tile_m);
        auto rec = [&](const int32_t* p) { return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p))[tile_m]; };
        t.row0 = rec(m.row0);
        t.nrows = rec(m.nrows);
        t.ex = rec(m.expert);
        t.rel = rec(m.gather) ? m.rel + (size_t)tile_m * kRelPitch : nullptr;
        t.n0 = __builtin_amdgcn_readfirstlane(tile_n * NOUT);
        const int r = 16 * wave + (lane >> 2);
        int ar = min(r, t.nrows - 1);
        if (t.rel) ar = t.rel[ar];                         // gathered tile: offsets below 2^32 bytes (checked on the host)
        s.a = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A + (size_t)t.row0 * lda), 0, kNoOffset, 0x00027000);
        s.a_voff = (uint32_t)ar * (uint32_t)lda * 4u;
        // SwiGLU: the 64 weight rows of a wave-column are 32 gate rows and the 32 up rows of the same columns
        s.b = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(weights((EPI == EPI_SWIGLU && (wave & 2)) ? which1 : which0, t.ex) + (size_t)t.n0 * K * 4), 0, kNoOffset, 0x00027000);
        const int col = (EPI == EPI_SWIGLU) ? (wave >> 2) * 32 + (r & 31) : r;
        s.b_voff = (uint32_t)min(col, N - 1 - t.n0) * (uint32_t)K * 4u;
        asm volatile("" : "+v"(s.a_voff), "+v"(s.b_voff));  // stay 32-bit lane offsets next to a scalar base
    };
    Tile cur, next;
    Source src, src_next;
    bool more = item + ncu < end_item;
    // Byte offsets of the lane's two quads inside a k-tile.  Past K nothing counts: those lanes' offsets lie past the end of
    // the buffer, which reads as zero.
    const uint32_t quad0 = (uint32_t)lc * 16u, quad1 = quad0 + 64u;
    auto fetch = [&](f32x4 (&q)[4], int kt) {
        kt += src.k0;
        const int at = kt * (XK * 4);
        const bool in0 = kt < k_full || kt * XK + lc * 4 < K, in1 = kt < k_full || kt * XK + 16 + lc * 4 < K;
        auto load = [&](__amdgpu_buffer_rsrc_t r, uint32_t off, bool in) { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, in ? off : kNoOffset, at, 0)); };
        q[0] = load(src.a, src.a_voff + quad0, in0);
        q[1] = load(src.a, src.a_voff + quad1, in1);
        q[2] = load(src.b, src.b_voff + quad0, in0);
        q[3] = load(src.b, src.b_voff + quad1, in1);
    };
    f32x4 even[4], odd[4];                                 // k-tiles in flight: two quads of A, two of B
    float largest[2] = {0.f, 0.f};                         // of the elements that this lane has split, of A and of B
    Acc22 hi, lo;
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) hi[i][j][e] = lo[i][j][e] = 0.f;
    };
    const int a_off = tile_off(wm * 64 + fr, 2 * grp + fk), b_off = kXOperand + tile_off(wn * 64 + fr, 2 * grp + fk);
    const int w_off = wave * 1024 + lane * 16;
    float* tile_largest = reinterpret_cast<float*>(lds + kXLargest);
    auto note_largest = [&] {                              // of the tile's rows, whose four lanes are neighbours; starts the next tile's
#pragma unroll
        for (int op = 0; op < 2; ++op) {
            float m = largest[op];
            m = fmaxf(m, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(m), 0xB1, 0xf, 0xf, true)));   // quad_perm 1 0 3 2
            m = fmaxf(m, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(m), 0x4E, 0xf, 0xf, true)));   // 2 3 0 1
            if ((lane & 3) == 0) tile_largest[op * XM + 16 * wave + (lane >> 2)] = m;
            largest[op] = 0.f;
        }
    };
    // k-tile kt is in `now`; the one behind it goes to `then`
    auto step = [&](int kt, unsigned char* now, unsigned char* then, f32x4 (&q)[4]) {
        if (kt + 3 == cur.nk && more) src = src_next;
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 1 == cur.nk) note_largest();                  // what is split now is the next tile's first k-tile
        __builtin_amdgcn_sched_barrier(0);
        multiply_parts(now + a_off, now + b_off, hi, lo, q, largest, then + w_off);
        fetch(q, kt + 3 >= cur.nk ? kt + 3 - cur.nk : kt + 3);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0): this wave has read `now` and written `then`
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    describe(item, cur, src);
    fetch(even, 0);
    fetch(odd, 1);
    if (more) describe(item + ncu, next, src_next);
    clear();
    unsigned char *st0 = lds, *st1 = lds + kXStage, *sums = st1;
    split_parts(even, largest, st0 + w_off);
    fetch(even, 2);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    while (true) {
        for (int kt = 0; kt < cur.nk; kt += 2) {
            step(kt, st0, st1, odd);
            step(kt + 1, st1, st0, even);
        }
        // sums of the group, and what of them the other group finishes (the second stage is free: the next tile's first k-tile is in st0)
        unsigned char* give = sums + grp * kXGive + (wave & 3) * 8192 + lane * 16;
        const unsigned char* take = sums + (grp ^ 1) * kXGive + (wave & 3) * 8192 + lane * 16;
        f32x16 fin[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 other;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int e = 4 * q + t;
                    const float x0 = hi[0][j][e] + lo[0][j][e], x1 = hi[1][j][e] + lo[1][j][e];
                    fin[j][e] = grp == 0 ? x0 : x1;
                    other[t] = grp == 0 ? x1 : x0;
                }
                *reinterpret_cast<f32x4*>(give + (j * 4 + q) * 1024) = other;
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int gr = wm * 64 + grp * 32 + fr;
        const float small = (float)K * kPartsFloor;
        float row_largest = tile_largest[gr];
        uint32_t bad[2] = {0, 0};
        auto judge = [&](int e, int j, float larger, float w_largest) {
            const float limit = row_largest > 0.f && w_largest > 0.f ? small * fmaxf(fmaxf(row_largest, w_largest), 1.f) : 0.f;
            if (!(larger >= limit && fabsf(fin[j][e]) <= FLT_MAX)) bad[j] |= 1u << e;
        };
        const int w_at = wn * 64 + fk * 4;                 // the weight rows of fin[j][4 q + t]: w_at + 32 j + 8 q + t
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(take + (j * 4 + q) * 1024);
                const f32x4 w = *reinterpret_cast<const f32x4*>(&tile_largest[XM + w_at + j * 32 + q * 8]);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int e = 4 * q + t;
                    const float larger = fmaxf(fabsf(fin[j][e]), fabsf(v[t]));
                    fin[j][e] += v[t];
                    judge(e, j, larger, w[t]);
                }
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();                      // the sums have been read: the next tile's second k-tile may be written
        asm volatile("" ::: "memory");
        bool finish = true;                                // this block writes the tile
        if (CUT && cur.piece >= 0) {
            const int tid = threadIdx.x, tile = (item - cut.n_full) % cut.n_cut;
            auto slot = [&](int p) { return p * (int)(kXPiece / 16); };
            const __amdgpu_buffer_rsrc_t pieces = pieces_rsrc(partial + (size_t)tile * cut.parts * (kXPiece / 4), (uint32_t)(cut.parts * kXPiece));
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    store_piece(pieces, slot(cur.piece) + (j * 4 + q) * 512 + tid, f32x4{fin[j][4 * q], fin[j][4 * q + 1], fin[j][4 * q + 2], fin[j][4 * q + 3]});
            if (tid < (XM + XN) / 4) store_piece(pieces, slot(cur.piece) + XM * XN / 4 + tid, reinterpret_cast<const f32x4*>(tile_largest)[tid]);
            finish = last_piece(m.done + tile, cut.parts, reinterpret_cast<int*>(lds + kXFlag));
            if (finish) {
                // all pieces in order, this one as well: the sum does not depend on who was last.  What counts as small is judged by the
                // pieces' sums as by the groups' above; of the largest elements all pieces have their own.
                f32x4 sum[8], w[8];
                float top[2][16];                          // largest of the pieces' sums
                row_largest = 0.f;
#pragma unroll
                for (int q = 0; q < 8; ++q) sum[q] = w[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) top[j][e] = 0.f;
                for (int i = 0; i < cut.parts; ++i) {
                    const int from = slot(i), larg = from + XM * XN / 4;
                    f32x4 v[8], u[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = load_piece(pieces, from + q * 512 + tid);
                    const f32x4 r = load_piece(pieces, larg + gr / 4);
#pragma unroll
                    for (int q = 0; q < 8; ++q) u[q] = load_piece(pieces, larg + (XM + w_at + q / 4 * 32 + q % 4 * 8) / 4);
                    row_largest = fmaxf(row_largest, r[gr & 3]);
#pragma unroll
                    for (int q = 0; q < 8; ++q)
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            sum[q][t] += v[q][t];
                            w[q][t] = fmaxf(w[q][t], u[q][t]);
                            float& big = top[q / 4][q % 4 * 4 + t];
                            big = fmaxf(big, fabsf(v[q][t]));
                        }
                }
                bad[0] = bad[1] = 0;
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int j = q / 4, e = q % 4 * 4 + t;
                        fin[j][e] = sum[q][t];
                        judge(e, j, top[j][e], w[q][t]);
                    }
            }
        }
        if (finish && __ballot((bad[0] | bad[1]) != 0)) {
            int ar = min(gr, cur.nrows - 1);
            if (cur.rel) ar = cur.rel[ar];
            const int c0 = cur.n0 + wn * (NOUT / 2) + fr;
            const float* w0 = reinterpret_cast<const float*>(weights(which0, cur.ex));
            const float* w1 = (EPI == EPI_SWIGLU) ? reinterpret_cast<const float*>(weights(which1, cur.ex)) : w0;
            f32x16 exact[2];
            multiply_exactly(A + (size_t)(cur.row0 + ar) * lda, w0 + (size_t)min(c0, N - 1) * K,
                             w1 + (size_t)min((EPI == EPI_SWIGLU) ? c0 : c0 + 32, N - 1) * K, fk, K, exact);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (bad[j] >> e & 1) fin[j][e] = exact[j][e];
        }
        if (finish && gr < cur.nrows) {
            float* crow = C + (size_t)(cur.row0 + (cur.rel ? cur.rel[gr] : gr)) * ldc;
#pragma unroll
            for (int j = 0; j < ((EPI == EPI_SWIGLU) ? 1 : 2); ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v;
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = epilogue<EPI>(fin[j][4 * g + t], (EPI == EPI_SWIGLU) ? fin[1][4 * g + t] : 0.f);
                    const int col = cur.n0 + wn * (NOUT / 2) + j * 32 + g * 8 + fk * 4;
                    if (col < N) *reinterpret_cast<f32x4*>(crow + col) = v;     // N is a multiple of 4
                }
        }
        if (!more) return;
        item += ncu;
        cur = next;
        more = item + ncu < end_item;
        if (more) describe(item + ncu, next, src_next);
        clear();
    }
}

template <int EPI, int MI, int NJ> struct EpiGeom {
    static constexpr int NOUT = (EPI == EPI_SWIGLU) ? 32 * NJ : 64 * NJ;   // output columns per block
    static constexpr int NW = NOUT / 2;                            // output columns per wave
    static constexpr int NJO = NW / 32;                            // 32-wide output column tiles per wave
    static constexpr int ROWS = 32 * MI;                           // rows per wave
};
// Activation and store of a wave's part of a tile: acc[i][j][e] is output row 16 i + lane % 16 and output column
// 16 j + lane / 16 * 4 + e.  32 rows of up to 64 columns at a time are packed to bf16, transposed through
// `region` (4 KB of LDS of this wave's own; LDS accesses of a wave execute in order) and stored as whole lines: stores
// of 32 bytes per row straight from the registers took 13 us per 256 x 256 tile instead of 4.
// Region: rows of CH 16-byte chunks, chunk c of row r at slot c ^ (r / (16 / CH)) % CH: both the 8-byte writes (half a wave:
// 16 rows, one chunk) and the 16-byte reads touch all 64 banks once.
// An accumulator element on its way to the vector unit.  The large tiles' accumulators fill the accumulation registers;
// left to itself the register allocator moves whole 16-element tuples out of them at every use and spills.
template <bool IN_AGPR> __device__ __forceinline__ float read_acc(float a) {
    if (!IN_AGPR) return a;
    float v;
    asm("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
    return v;
}
template <int EPI, int MI, int NJ, bool IN_AGPR, bool GATHER>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[2 * MI][2 * NJ], int lane0, unsigned char* region, __amdgpu_buffer_rsrc_t dst,
                                           int first_row, int nrows, const int32_t* __restrict__ rel, int ldc) {
    constexpr int NJO = EpiGeom<EPI, MI, NJ>::NJO;
    constexpr int JP = NJO == 1 ? 1 : 2, CH = 4 * JP, RPI = 64 / CH, STEPS = 32 / RPI;   // column tiles per pass, chunks per row, rows per store
    constexpr int PER_ROW = NJO / JP;                        // passes per 32-row tile
    static_assert(TileGeom<MI, NJ>::STAGE / 4 >= 32 * CH * 16, "32 rows of a pass");
    int lane = lane0;                                        // opaque: what follows from it is not worth registers during the loop
    asm volatile("" : "+v"(lane));
    const int fr = lane & 15;
    unsigned char* wr = region + fr * (CH * 16) + (lane >> 4 & 1) * 8;
    const int w_swz = (fr / (16 / CH)) % CH;                 // (the same 16 rows further)
    auto write = [&](int p) {
        const int i0 = p / PER_ROW * 2, j0 = p % PER_ROW * JP * 2;
#pragma unroll
        for (int i = i0; i < i0 + 2; ++i)
#pragma unroll
            for (int j = j0; j < j0 + 2 * JP; ++j) {
                float v[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    v[t] = epilogue_bf16<EPI>(read_acc<IN_AGPR>(acc[i][j][t]),
                                              (EPI == EPI_SWIGLU) ? read_acc<IN_AGPR>(acc[i][(j + NJ) % (2 * NJ)][t]) : 0.f);
                *reinterpret_cast<u32x2*>(wr + (i - i0) * (16 * CH * 16) + ((((j - j0) * 2) + (lane >> 5)) ^ w_swz) * 16) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
    };
    write(0);
#pragma unroll
    for (int p = 0; p < MI * PER_ROW; ++p) {
        // the wave's LDS accesses execute in order, so the region can be written again behind the reads: what the next
        // pass computes hides their latency
        asm volatile("" ::: "memory");
        u32x4 q[STEPS];
        uint32_t row_off[STEPS];
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {
            const int r = it * RPI + lane / CH;
            q[it] = *reinterpret_cast<const u32x4*>(region + r * (CH * 16) + ((lane % CH) ^ ((r / (16 / CH)) % CH)) * 16);
            const int gr = first_row + p / PER_ROW * 32 + r;
            const int mr = GATHER ? rel[min(gr, nrows - 1)] : gr;
            row_off[it] = gr < nrows ? (uint32_t)mr * (uint32_t)ldc * 2u + (uint32_t)(lane % CH) * 16u : 0xFFFFFF00u;   // else past the end of dst: not stored
        }
        asm volatile("" ::: "memory");
        if (p + 1 < MI * PER_ROW) write(p + 1);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int it = 0; it < STEPS; ++it)
            __builtin_amdgcn_raw_buffer_store_b128(q[it], dst, row_off[it] + p % PER_ROW * JP * 64, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Sum of the pieces of one tile and its epilogue for units [unit_lo, unit_hi) of 32 x 32 outputs per wave.  Four pieces are requested before
// the first is added, without conditions (past the last piece the last one is read again and not added): a load under
// a condition waits for the one before it.
template <int EPI, int MI, int NJ>
__device__ __forceinline__ void sum_pieces(int unit_lo, int unit_hi, const float* partial, int parts, int row0, int nrows,
                                           const int32_t* __restrict__ rel, int n0, int N, uint16_t* __restrict__ C, int ldc) {
    using G = EpiGeom<EPI, MI, NJ>;
    using TG = TileGeom<MI, NJ>;
    constexpr int NP = (EPI == EPI_SWIGLU) ? 2 : 1;            // products behind an output
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const __amdgpu_buffer_rsrc_t src = pieces_rsrc(partial, (uint32_t)(parts * TG::PARTIAL));
#pragma unroll 1
    for (int unit = unit_lo; unit < unit_hi; ++unit) {
        const int i = unit / G::NJO, jo = unit % G::NJO;
        f32x4 sum[NP][4];
#pragma unroll
        for (int n = 0; n < NP; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[n][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < parts; p0 += 4) {
            f32x4 v[4][NP][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int n = 0; n < NP; ++n)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[u][n][q] = load_piece(src, min(p0 + u, parts - 1) * (int)(TG::PARTIAL / 16) + ((2 * i + (q >> 1)) * (2 * NJ) + 2 * jo + (q & 1) + n * NJ) * 256 + (int)threadIdx.x);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p0 + u < parts) {
#pragma unroll
                    for (int n = 0; n < NP; ++n)
#pragma unroll
                        for (int q = 0; q < 4; ++q) sum[n][q] += v[u][n][q];
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int gr = (wave >> 1) * G::ROWS + i * 32 + h * 16 + (lane & 15);
            if (gr >= nrows) continue;
            uint16_t* crow = C + (size_t)(row0 + (rel ? rel[gr] : gr)) * ldc;
#pragma unroll
            for (int q = 2 * h; q < 2 * h + 2; ++q) {
                float v[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = epilogue_bf16<EPI>(sum[0][q][t], sum[NP - 1][q][t]);
                const int col = n0 + (wave & 1) * G::NW + jo * 32 + (q & 1) * 16 + (lane >> 4) * 4;
                if (col < N) *reinterpret_cast<u32x2*>(crow + col) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
        }
    }
}

// 16 bytes per lane, from lane_off + off on, into the KB of LDS at `to`
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, unsigned char* to, uint32_t lane_off, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)to, 16, lane_off, off, 0, 0);
}

// C[r, n] = epi(sum_k A[r,k] B0[n,k] , sum_k A[r,k] B1[n,k]) for one M-tile of 64 MI rows and one
// N-tile of 64 NJ weight rows.  SwiGLU: the B tile's rows are, per wave-column wn (16 NJ output columns), 16 NJ rows
// of W1 followed by the 16 NJ rows of Wu for the same columns, so the gate and the up product of
// a column live in the same lane and the activation needs no exchange.
//
// Pipeline: 5 LDS stages of one 32-wide k-tile each (160 KB at 4 x 4).  Loads are direct-to-LDS and
// issued in PAIRS of k-tiles (2q, 2q+1) every second iteration, interleaved so that the two
// halves of every 128-byte memory line are requested close together (a few products apart): half-line requests
// that come a whole k-tile apart cost about twice the L2 bandwidth.  The pair (kt+4, kt+5) is issued
// from iteration kt on (kt even) and has to be there before iteration kt+3.
// The MFMAs are issued as D = B . A^T (operands swapped), so a lane ends up with 4 consecutive
// output COLUMNS of one row (see store_tile).
//
// A block walks through several tiles, and the pipeline runs across them: the loads that go out in a tile's last two
// trips are the next tile's first k-tiles (its addresses are prepared during the epilogue before), and the last
// fragment reads are its first fragments.  So a tile costs its loop and its epilogue; with a block per tile each also
// paid 3.4 us from the block's start to its first operands and 1.3 us of launch.  Per 256 x 256 tile at K = 1408: 41.6
// -> 39.5 us, at K = 2048 SwiGLU 54.6 -> 53; 612329 rows of 2048 -> 1408 -> 2048 with shared experts, the whole share:
// 9.33 -> 9.13 ms; 10199 rows of 1024 -> 4096 -> 1024 238 -> 233 us; two models at once 1.75 -> 1.70 ms.  (A tile whose
// loop is long is bound by power instead: K = 14336 is unchanged.)  The walk is bounded (`walk` tiles, see walk_tiles): a
// CU that comes free is where work of another stream gets in.
//
// TIMED (diagnostics, moe_diag_ffn_phases): the same kernel with the 100 MHz wall clock read by lane 0 of every wave
// into marks[item][wave][4]: 0 start, 1 first operands in LDS (loop about to start), 2 loop done, 3 end; an item is a
// tile or a piece of one (there is room for all of them: see max_items).  The ordinary instantiation contains none of it.
struct WorkItem {
    int tile_id, piece;      // piece < 0: the whole K range
    int nk;                  // k-tiles (even: K is a multiple of 64)
    int row0, nrows, n0;     // output rows and first output column
    const int32_t* rel;      // row offsets of a gathered tile, else NULL
};
template <int EPI, int MI, int NJ, bool SOON, bool TIMED>
__global__ __launch_bounds__(256, (TileGeom<MI, NJ>::PER_CU)) void gemm_bf16_kernel(const uint16_t* __restrict__ A, int lda, TileMap m,
                                                           ExpertTable tab, int which0, int which1, int N, int K,
                                                           uint16_t* __restrict__ C, int ldc, int tiles_n, const int32_t* __restrict__ strips_at, int ncu, int walk, int most_tail,
                                                           float* partial, long long* __restrict__ marks,
                                                           uint32_t mark_items) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
#define MOE_MARK(i)                                                                                                 \
    do {                                                                                                            \
        if (TIMED && (uint32_t)item < mark_items && (threadIdx.x & 63) == 0)                                        \
            marks[((size_t)item * 4 + (threadIdx.x >> 6)) * 4 + (i)] = (long long)wall_clock64();                    \
    } while (0)
    const long long t_start = TIMED ? (long long)wall_clock64() : 0;
    using TG = TileGeom<MI, NJ>;
    using EG = EpiGeom<EPI, MI, NJ>;
    constexpr int NOUT = EG::NOUT;                                          // output columns per block
    auto word = [](const int32_t* p) { return *reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p)); };
    const int n_tiles_m = word(m.n_tiles);
    const Strips strips = strips_at ? Strips{word(strips_at), word(strips_at + 1)} : Strips{0, 0};
    const int total = n_tiles_m * tiles_n;
    TailPlan plan = plan_tail_upto(most_tail, total, ncu, K / BK);
    // the same for all blocks; the compiler does not see it through the divisions
    plan.n_full = __builtin_amdgcn_readfirstlane(plan.n_full);
    plan.n_tail = __builtin_amdgcn_readfirstlane(plan.n_tail);
    plan.parts = __builtin_amdgcn_readfirstlane(plan.parts);
    plan.pairs_per = __builtin_amdgcn_readfirstlane(plan.pairs_per);
    const int n_items = plan.n_full + (plan.parts > 1 ? plan.n_tail * plan.parts : 0);
    const WalkRun run = walk_run(blockIdx.x, ncu, walk, n_items);
    int item = run.item;
    const int end_item = run.end;
    if (item >= end_item) return;
    if (TIMED && (uint32_t)item < mark_items && (threadIdx.x & 63) == 0) marks[((size_t)item * 4 + (threadIdx.x >> 6)) * 4] = t_start;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction; tell the compiler
    const int wm = wave >> 1, wn = wave & 1;

    // Direct-to-LDS staging.  A stage is 4 (MI + NJ) blocks of 1 KB (4 MI of A, 4 NJ of B); wave w
    // fills blocks w, w+4, ...: MI of A and NJ of B per stage.  A load's address is a buffer descriptor per operand, a
    // fixed 32-bit byte offset per lane and the byte offset of the k-tile in one scalar register, so it costs no address arithmetic.
    struct Source { __amdgpu_buffer_rsrc_t a, b0, b1; uint32_t a_voff[MI], b_voff[NJ]; };
    // in two parts, so that the loads of the first are under way during an epilogue
    auto describe = [&](int id, WorkItem& w, Source& src, int (&a_row)[MI]) {
        int lr, lc, ln = lane;
        asm volatile("" : "+v"(ln));                         // (opaque: not worth registers during the loop)
        rc_of_slot(ln, &lr, &lc);
        w.tile_id = id;
        w.piece = -1;
        int kt_lo = 0;
        w.nk = K / BK;
        if (id >= plan.n_full) {
            const int j = id - plan.n_full;
            w.tile_id = plan.n_full + j % plan.n_tail;
            w.piece = j / plan.n_tail;
            kt_lo = w.piece * plan.pairs_per * 2;
            w.nk = min(plan.pairs_per * 2, K / BK - kt_lo);
        }
        int tile_m, tile_n;
        tile_of_block(w.tile_id, total, n_tiles_m, tiles_n, strips, &tile_m, &tile_n);
        tile_m = __builtin_amdgcn_readfirstlane(tile_m);
        // the same for the whole block, written by an earlier kernel: scalar loads, which do not queue behind the operands
        auto rec = [&](const int32_t* p) { return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p))[tile_m]; };
        w.row0 = rec(m.row0);
        w.nrows = rec(m.nrows);
        const int ex = rec(m.expert);
        w.rel = rec(m.gather) ? m.rel + (size_t)tile_m * kRelPitch : nullptr;
        w.n0 = __builtin_amdgcn_readfirstlane(tile_n * NOUT);
        auto pick = [&](int which) -> const char* {
            return reinterpret_cast<const char*>(which == 0 ? tab.w1[ex] : which == 1 ? tab.w_up[ex] : tab.w_down[ex]) + (size_t)kt_lo * BK * 2;
        };
        const char *b0 = pick(which0), *b1 = (EPI == EPI_SWIGLU) ? pick(which1) : b0;
        // SwiGLU: the second half of a wave-column's 2 NJ 16-row blocks are up rows; this wave fetches blocks wave + 4 i
        if (NJ == 2 && (wave & 2)) b0 = b1;
        auto rsrc = [](const char* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, 0xFFFFFFFFu, 0x00027000); };
        src.b0 = rsrc(b0);
        src.b1 = rsrc(b1);
        src.a = rsrc(reinterpret_cast<const char*>(A + (size_t)w.row0 * lda) + (size_t)kt_lo * BK * 2);
#pragma unroll
        for (int i = 0; i < MI; ++i) a_row[i] = min((wave + 4 * i) * 16 + lr, w.nrows - 1);   // row (relative to row0) of the tile rows this lane fetches
        if (w.rel) {                                         // gathered tile: offsets from row0, below 2^32 bytes (checked
            int t[MI];                                       // on the host); the loads go out together
#pragma unroll
            for (int i = 0; i < MI; ++i) t[i] = w.rel[a_row[i]];
#pragma unroll
            for (int i = 0; i < MI; ++i) a_row[i] = t[i];
        }
    };
    auto describe_lanes = [&](const WorkItem& w, Source& src, const int (&a_row)[MI]) {
        int lr, lc, ln = lane;
        asm volatile("" : "+v"(ln));
        rc_of_slot(ln, &lr, &lc);
#pragma unroll
        for (int i = 0; i < MI; ++i) src.a_voff[i] = (uint32_t)a_row[i] * (uint32_t)lda * 2u + (uint32_t)lc * 16u;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const int r = (wave + 4 * i) * 16 + lr;          // tile row this lane fetches
            int col = w.n0 + r;
            if (EPI == EPI_SWIGLU) {
                constexpr int WB = 32 * NJ;                  // weight rows per wave-column, the first half gate, the second up
                col = w.n0 + r / WB * (WB / 2) + r % (WB / 2);
            }
            src.b_voff[i] = (uint32_t)min(col, N - 1) * (uint32_t)K * 2u + (uint32_t)lc * 16u;
        }
    };
    WorkItem cur, next;
    Source src, src_next;
    int t_first = 0, t_last = 0;                             // loads: the k-tile number at which `src` starts, and the last pair it has
    // byte offset inside a row of the pair of k-tiles t and t+1 (t even).  Past the end of the last tile its last pair is fetched
    // again (into stages nobody reads any more) so that the count of outstanding loads stays uniform.
    auto pair_offset = [&](int t) { return min(t - t_first, t_last) * (BK * 2); };
    // Load l of the 2 (MI + NJ) by which this wave fetches its 16-row blocks of such a pair, A and B in turn, each for both
    // k-tiles, into the stages at LDS byte offsets so0 and so1
    auto issue_one = [&](int kb, int so0, int so1, int l) {
        static_assert(MI <= NJ, "A and B blocks alternate while there are A blocks");
        const int it = l >> 1;
        if (it >= MI + NJ) return;
        const bool is_a = it < 2 * MI && (it & 1) == 0;
        const int i = it < 2 * MI ? it >> 1 : it - MI;
        unsigned char* to = lds + ((l & 1) ? so1 : so0) + (wave + 4 * i) * 1024 + (is_a ? 0 : TG::A_BYTES);
        const __amdgpu_buffer_rsrc_t r = is_a ? src.a : (EPI == EPI_SWIGLU && (i & (NJ / 4))) ? src.b1 : src.b0;
        load_to_lds(r, to, is_a ? src.a_voff[i] : src.b_voff[i], kb + (l & 1) * (BK * 2));
    };
    constexpr int GI = (MI + NJ + 3) / 4;                    // 16-row blocks per quarter of a pair (the last may have fewer)
    // SOON: loads as early as they can go out, else evenly spread (see below)
    constexpr int FIRST_LOADS = SOON ? 8 * GI : 4 * GI;      // of the loads of a pair, 4 or 8 GI go out during the first k-tile of a trip

    // A fragment is 16 rows x 32 elements, one 16-row block of the stage; block i of the wave lies i KB further
    const int a_off = tile_off(wm * 32 * MI + (lane & 15), lane >> 4), b_off = TG::A_BYTES + tile_off(wn * 32 * NJ + (lane & 15), lane >> 4);
    f32x4 acc[2 * MI][2 * NJ];                               // [16 rows i][16 columns j], holds D^T: rows n, columns m
    // Fragment r of the 2 MI + 2 NJ of a k-tile, in the order in which the products need them
    auto read = [&](bf16x8 (&af)[2 * MI], bf16x8 (&bfr)[2 * NJ], const unsigned char* st, int r) {
        if (r == 0) bfr[0] = *reinterpret_cast<const bf16x8*>(st + b_off);
        else if (r <= 2 * MI) af[r - 1] = *reinterpret_cast<const bf16x8*>(st + a_off + (r - 1) * 1024);
        else bfr[r - 2 * MI] = *reinterpret_cast<const bf16x8*>(st + b_off + (r - 2 * MI) * 1024);
    };
    // The MFMAs of a k-tile, with the reads of the next one's fragments and `load` 0 .. LOADS - 1 between them.
    // Power bounds the large tiles, so the instruction is the one that takes the least of it per product: from registers alone
    // v_mfma_f32_16x16x32_bf16 sustained 2.06 PFLOP/s on a whole chip (1.96 GHz), v_mfma_f32_32x32x16_bf16 1.81 (1.73 GHz) - and in
    // runs that have the weight fragment in common (1.66 to 1.79 PFLOP/s where both operands change from product to product).  (The first
    // and the last of these by a loop that is not in the library: moe_diag_mfma_only runs the larger instruction.)
    // The results are the same bits.  The order is that of the source (see the barriers): the scheduler left to itself
    // moves all reads together and mixes the runs.  20571 rows of 4096 -> 14336 -> 4096: 3590 + 1780 -> 3360 + 1650 us.
    auto k_tile = [&](auto from_zero, const bf16x8 (&af)[2 * MI], const bf16x8 (&bfr)[2 * NJ], bf16x8 (&an)[2 * MI], bf16x8 (&bn)[2 * NJ], const unsigned char* next_stage, auto n_loads, auto load) {
        constexpr int READS = 2 * MI + 2 * NJ, LOADS = decltype(n_loads)::value, M = 4 * MI * NJ, EVERY = M >= 48 ? 3 : 1;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j)
#pragma unroll
            for (int i = 0; i < 2 * MI; ++i) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], decltype(from_zero)::value ? zero : acc[i][j], 0, 0, 0);
                const int n = j * 2 * MI + i + 1;            // products so far
                const int r = SOON ? n - 2 : n % EVERY == 0 ? n / EVERY - 1 : -1, l = SOON ? n - 1 : (n + 1) * LOADS / M > n * LOADS / M ? n * LOADS / M : -1;
                const bool reads_now = r >= 0 && r < READS, loads_now = l >= 0 && l < LOADS;
                if (reads_now || loads_now) __builtin_amdgcn_sched_barrier(0);
                if (loads_now) load(l);
                if (reads_now) read(an, bn, next_stage, r);
                if (reads_now || loads_now) __builtin_amdgcn_sched_barrier(0);
            }
    };

    // Software pipeline, two k-tiles per trip; the fragments of a k-tile are read during the one before it:
    //   barrier: every wave has read the fragments of kt, so the stages of kt-1 and kt are free
    //   MFMAs of kt   | read the fragments of kt+1 | load the first half of pair (kt+4, kt+5), or all of it
    //   wait until only those loads (4 or 8 GI per wave) are outstanding: pair (kt+2, kt+3) is in LDS; barrier
    //   MFMAs of kt+1 | read the fragments of kt+2 | load the second half
    // A half is 2 GI 16-row blocks, both k-tiles of the pair: 8 loads per wave at 4 x 4.  These
    // loads are spread evenly, at 4 x 4 one per eight MFMAs: a CU sustains roughly one wave-load per 40 clocks
    // when the lines come from HBM, and a load that cannot be accepted stalls the wave's MFMA issue too (loads one after the
    // other, in front of the reads: 2 to 5 % slower).  128 x 128 tiles of long loops (SOON, see kSoonK) are bound by what is in flight
    // instead: a k-tile of a block is 0.12 us of products, a round trip 0.7, and the other block of the CU fills a stall.  There the whole
    // pair goes out in the first k-tile as soon as its stages are free, in front of the reads: 2741 rows of 1152 -> 2304 -> 1152 for four
    // experts 59.9 -> 56.9 us, 800 of 2048 -> 1408 -> 2048 SwiGLU 53.1 -> 46.9 (in halves, one after the other: 59.2 and 51.9).
    // A bare s_barrier is used: __syncthreads() would add a fence that waits for ALL outstanding loads.  In front of it a
    // wave waits for its own LDS reads: a read that is only issued is not ordered against what other waves write behind
    // the barrier.  They are the first fragments that the MFMAs behind it need.
    // so[j] is the LDS byte offset of the stage that holds k-tile kt + j; the five values rotate by two per
    // trip, which keeps modulo arithmetic out of the instruction stream
    int so[STAGES];
#pragma unroll
    for (int j = 0; j < STAGES; ++j) so[j] = j * TG::STAGE;
    bf16x8 a0[2 * MI], a1[2 * MI], b0[2 * NJ], b1[2 * NJ];   // of even and odd k-tiles

    int a_row[MI];
    describe(item, cur, src, a_row);
    describe_lanes(cur, src, a_row);
    t_last = cur.nk - 2;
#pragma unroll
    for (int l = 0; l < 8 * GI; ++l) issue_one(0, so[0], so[1], l);
#pragma unroll
    for (int l = 0; l < 8 * GI; ++l) issue_one(pair_offset(2), so[2], so[3], l);
    bool more = item + ncu < end_item;
    if (more) {
        describe(item + ncu, next, src_next, a_row);
        describe_lanes(next, src_next, a_row);
    }
    // vmcnt(2 (MI + NJ)): pair (0, 1) is in LDS
    __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * (MI + NJ)) & 15) | ((2 * (MI + NJ)) >> 4) << 14);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int r = 0; r < 2 * (MI + NJ); ++r) read(a0, b0, lds + so[0], r);
    // One trip.  FIRST: of a tile (the products start from zero); SWITCH: the loads of this tile have all
    // gone out, those of the next one follow.
    auto trip = [&](int kt, auto first, auto switches) {
        constexpr bool FIRST = decltype(first)::value, SWITCH = decltype(switches)::value;
        const unsigned char *s1 = lds + so[1], *s2 = lds + so[2];
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0): this wave has read stage so[0], which is refilled below
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if ((SWITCH || (FIRST && cur.nk == 4)) && more) { src = src_next; t_first = cur.nk; t_last = next.nk - 2; }
        const int kb = pair_offset(kt + 4);
        k_tile(first, a0, b0, a1, b1, s1, std::integral_constant<int, FIRST_LOADS>{}, [&](int l) { issue_one(kb, so[4], so[0], l); });
        __builtin_amdgcn_sched_barrier(0);
        // vmcnt(FIRST_LOADS): only what has gone out of the next pair may be outstanding; lgkmcnt(0): this wave has read stage so[1],
        // which the epilogue writes behind a tile's last trip
        static_assert(FIRST_LOADS < 16, "");
        __builtin_amdgcn_s_waitcnt(0x0070 | FIRST_LOADS);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        k_tile(std::false_type{}, a1, b1, a0, b0, s2, std::integral_constant<int, 8 * GI - FIRST_LOADS>{}, [&](int l) { issue_one(kb, so[4], so[0], FIRST_LOADS + l); });
        __builtin_amdgcn_sched_barrier(0);
        const int t0 = so[0], t1 = so[1];
        so[0] = so[2]; so[1] = so[3]; so[2] = so[4]; so[3] = t0; so[4] = t1;
    };
    while (true) {
        MOE_MARK(1);
        trip(0, std::true_type{}, std::false_type{});
        if (cur.nk > 2) {                                    // (a tile that another one follows is whole: at least four k-tiles)
            int kt = 2;
            for (; kt < cur.nk - 4; kt += 2) trip(kt, std::false_type{}, std::false_type{});
            if (cur.nk > 4) {
                trip(kt, std::false_type{}, std::true_type{});
                kt += 2;
            }
            trip(kt, std::false_type{}, std::false_type{});
        }
        if (TG::PER_CU == 1) {                               // the accumulators stay where they are until they are stored
            asm volatile("s_nop 15\n\ts_nop 15");            // the last product has left the matrix core before read_acc
#pragma unroll
            for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
                for (int j = 0; j < 2 * NJ; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
        MOE_MARK(2);
        if (cur.piece >= 0) break;                           // the last item of its block: a round holds all pieces
        const WorkItem done = cur;
        const bool had_next = more;
        if (more) {
            cur = next;
            t_first = 0;
            more = item + 2 * ncu < end_item;
            if (more) describe(item + 2 * ncu, next, src_next, a_row);
        }
        const int col0 = __builtin_amdgcn_readfirstlane(done.n0 + wn * EG::NW);
        if (col0 < N) {                                      // N is a multiple of 128: all columns of the wave or none
            const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(C + (size_t)__builtin_amdgcn_readfirstlane(done.row0) * ldc + col0, 0, 0xFFFFFF00u, 0x00027000);
            unsigned char* region = lds + so[4] + wave * (TG::STAGE / 4);   // the only stage that no load is on its way to
            // two copies: the common one keeps its plain row arithmetic
            if (done.rel) store_tile<EPI, MI, NJ, TG::PER_CU == 1, true>(acc, lane, region, dst, wm * EG::ROWS, done.nrows, done.rel, ldc);
            else store_tile<EPI, MI, NJ, TG::PER_CU == 1, false>(acc, lane, region, dst, wm * EG::ROWS, done.nrows, nullptr, ldc);
        }
        if (more) describe_lanes(next, src_next, a_row);
        MOE_MARK(3);
        if (!had_next) {
            __builtin_amdgcn_s_waitcnt(0x0070);              // no load may still target LDS when the block ends
            return;
        }
        item += ncu;
        MOE_MARK(0);
    }
    // a piece of a tail tile: the raw accumulators, 16 bytes per lane and store (whole 4 KB per store)
    __builtin_amdgcn_s_waitcnt(0x0070);                      // vmcnt(0) lgkmcnt(0): no load may still target LDS below
    const int tail = __builtin_amdgcn_readfirstlane(cur.tile_id - plan.n_full), piece = __builtin_amdgcn_readfirstlane(cur.piece);
    float* pieces = partial + (size_t)tail * plan.parts * (TG::PARTIAL / 4);   // of this tile
    const __amdgpu_buffer_rsrc_t dst = pieces_rsrc(pieces, (uint32_t)(plan.parts * TG::PARTIAL));
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j) store_piece(dst, piece * (int)(TG::PARTIAL / 16) + (i * 2 * NJ + j) * 256 + tid, acc[i][j]);
    if (TG::SUM_IN_PLACE && last_piece(m.done + tail, plan.parts, reinterpret_cast<int*>(lds)))
        sum_pieces<EPI, MI, NJ>(0, MI * EG::NJO, pieces, plan.parts, cur.row0, cur.nrows, cur.rel, cur.n0, N, C, ldc);
    MOE_MARK(3);
#undef MOE_MARK
}

// Adds and finishes the tail tiles of the larger shapes: a block per unit of a tile, so that a few tail tiles make
// hundreds of blocks.
template <int EPI, int MI, int NJ>
__global__ __launch_bounds__(256) void gemm_bf16_tail_kernel(TileMap m, int N, int K, uint16_t* __restrict__ C, int ldc,
                                                             int tiles_n, const int32_t* __restrict__ strips_at, int ncu, int most_tail, const float* __restrict__ partial) {
    using G = EpiGeom<EPI, MI, NJ>;
    constexpr int UNITS = MI * G::NJO;
    const int n_tiles_m = *m.n_tiles;
    const int total = n_tiles_m * tiles_n;
    const TailPlan plan = plan_tail_upto(most_tail, total, ncu, K / BK);
    const int tt = blockIdx.x / UNITS, unit = blockIdx.x % UNITS;
    if (tt >= plan.n_tail) return;
    int tile_m, tile_n;
    tile_of_block(plan.n_full + tt, total, n_tiles_m, tiles_n, strips_at ? Strips{strips_at[0], strips_at[1]} : Strips{0, 0}, &tile_m, &tile_n);
    const int32_t* rel = m.gather[tile_m] ? m.rel + (size_t)tile_m * kRelPitch : nullptr;
    sum_pieces<EPI, MI, NJ>(unit, unit + 1, partial + (size_t)tt * plan.parts * (TileGeom<MI, NJ>::PARTIAL / 4), plan.parts, m.row0[tile_m],
                            m.nrows[tile_m], rel, tile_n * G::NOUT, N, C, ldc);
}

// ------------------------------------------------------------------------------------------------
// Shares of at most 64 rows (decode-sized).  The FLOPs are negligible and every weight is used once: the job
// is to stream the weights at HBM speed, which takes bytes in flight.  The big kernel keeps only 32 KB of
// weight loads outstanding per CU (the other half of its ring is the mostly empty 256-row A tile) and streams
// at a third of HBM speed.  Here a tile is 32 or 64 rows x 128 weight rows and a stage of the LDS ring is 128
// elements of K: a wave-load fetches 4 rows x 256 contiguous bytes, a stage is 8 or 16 KB of A and 32 KB of
// weights, four or three stages fit and all but one of them (96 or 64 KB of weights) are always in flight.
// Wave w owns weight rows 32 w .. 32 w + 31 of the tile (SwiGLU: 16 gate rows, then the 16 up rows of the
// same output columns) and all rows of A: MT x 1 tiles of v_mfma_f32_32x32x16_bf16, eight k-steps per stage.
// A wave loads the weight rows it reads itself; the A tile is shared (one barrier per stage).  With fewer
// tiles than CUs every tile is cut along K into `parts` pieces (fp32 partial tiles, added in piece order by the last
// block to arrive: results do not depend on the run).
//
// LDS layout of a stage: blocks of 1 KB = 4 rows x 16 chunks of 16 bytes, filled by ONE wave-wide
// direct-to-LDS load (lane l fills slot l).  Inside a block slot(r, c) = 16 r + (c ^ (4 r + blk % 4)):
// the 16 lanes that an MFMA operand read serves at a time (16 consecutive rows = 4 blocks, same chunk) then
// fall on 16 different values of slot % 16, i.e. on all 64 banks once.
// MT = 1 or 2 MFMA row tiles: shares of at most 32 rows take 32-row tiles, whose smaller A part leaves room for a
// fourth stage (96 KB of weights in flight).
constexpr int SBN = 128;                                 // weight rows per tile
constexpr int SKW = 128;                                 // elements of K per stage (256 bytes of a row)
template <int MT> struct SkinnyGeom {
    static constexpr int BM_ = 32 * MT;                  // rows per tile
    static constexpr int A_BYTES = BM_ * SKW * 2;        // 8 or 16 KB
    static constexpr int STAGE = A_BYTES + SBN * SKW * 2;   // 40 or 48 KB
    static constexpr int STAGES = (MT == 1) ? 4 : 3;
    static constexpr int LDS = STAGES * STAGE;           // 160 or 144 KB
    static constexpr int LOADS = 2 * MT + 8;             // wave-loads per stage and wave
    static constexpr size_t PARTIAL = (size_t)BM_ * SBN * sizeof(float);   // one fp32 partial tile
};

struct SkinnyPlan {
    int parts;     // pieces per tile
    int per;       // stages per piece (the last piece may be shorter)
};
__host__ __device__ __forceinline__ SkinnyPlan plan_skinny(int total, int ncu, int ns) {
    SkinnyPlan p{1, ns};
    if (total <= 0 || total >= ncu) return p;
    // At least 4 stages per piece: the last block adds the pieces at about 0.4 us each, half a stage's time.  64 rows of
    // 2048 -> 2816 -> 2048 30.0 us (pieces of 2 stages: 32.3, of 6: 32.8), 60 of 1152 -> 2304 -> 1152 25.6 (28.7, 26.5)
    int parts = min(min(ncu / total, ns / 4), 32);
    if (parts < 2) return p;
    p.per = (ns + parts - 1) / parts;
    p.parts = (ns + p.per - 1) / p.per;
    return p;
}

// Block `id` of `total` -> tile (M fastest).  Blocks go to the 8 XCDs round-robin; every XCD gets a run of consecutive
// tiles, so that the M-tiles of an expert which share weight rows find them in one L2.
__host__ __device__ __forceinline__ int skinny_tile(int id, int total) {
    const int x = id % 8, base = total / 8, extra = total % 8;
    return x * base + (x < extra ? x : extra) + id / 8;
}

// byte offset of (row, 16-byte chunk c of the stage's 256 bytes) inside a tile region
__device__ __forceinline__ int skinny_off(int row, int c) {
    const int blk = row >> 2, r = row & 3;
    return (blk << 10) + (((r << 4) + (c ^ ((r << 2) | (blk & 3)))) << 4);
}

// Activation and store of a wave's (32 MT) x 32 block of products held in the MFMA result layout: acc[i][e] is
// row i * 32 + lane % 32 of the tile and weight row 32 w + (e / 4) * 8 + (lane / 32) * 4 + e % 4.
template <int EPI, int MT>
__device__ __forceinline__ void skinny_store(const f32x16 (&acc)[MT], int wave, int lane, int row0, int nrows,
                                             const int32_t* __restrict__ rel, int n0, int N, uint16_t* __restrict__ C, int ldc) {
    const int fr = lane & 31, fk = lane >> 5;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int gr = i * 32 + fr;
        if (gr >= nrows) continue;
        uint16_t* crow = C + (size_t)(row0 + (rel ? rel[gr] : gr)) * ldc;
#pragma unroll
        for (int g = 0; g < ((EPI == EPI_SWIGLU) ? 2 : 4); ++g) {
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float up = (EPI == EPI_SWIGLU) ? acc[i][4 * (g + 2) + t] : 0.f;
                v[t] = epilogue_bf16<EPI>(acc[i][4 * g + t], up);
            }
            const int col = n0 + ((EPI == EPI_SWIGLU) ? wave * 16 : wave * 32) + g * 8 + fk * 4;
            if (col < N) *reinterpret_cast<u32x2*>(crow + col) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        }
    }
}

template <int EPI, int MT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_skinny_kernel(const uint16_t* __restrict__ A, int lda, TileMap m,
                                                                  ExpertTable tab, int which0, int which1, int N, int K,
                                                                  uint16_t* __restrict__ C, int ldc, int tiles_n, int ncu,
                                                                  float* partial) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    using G = SkinnyGeom<MT>;
    constexpr int NOUT = (EPI == EPI_SWIGLU) ? SBN / 2 : SBN;
    const int n_tiles_m = *m.n_tiles;
    const int total = n_tiles_m * tiles_n;
    const int ns_all = K / SKW;
    const SkinnyPlan plan = plan_skinny(total, ncu, ns_all);
    if ((int)blockIdx.x >= total * plan.parts) return;
    const int piece = blockIdx.x / total, tile_id = skinny_tile(blockIdx.x % total, total);
    const int tile_m = tile_id % n_tiles_m, tile_n = tile_id / n_tiles_m;
    const int row0 = __builtin_amdgcn_readfirstlane(m.row0[tile_m]);
    const int nrows = __builtin_amdgcn_readfirstlane(m.nrows[tile_m]);
    const int ex = __builtin_amdgcn_readfirstlane(m.expert[tile_m]);
    const int32_t* rel = __builtin_amdgcn_readfirstlane(m.gather[tile_m]) ? m.rel + (size_t)tile_m * kRelPitch : nullptr;
    auto pick = [&](int which) -> const uint16_t* {
        return reinterpret_cast<const uint16_t*>(which == 0 ? tab.w1[ex] : which == 1 ? tab.w_up[ex] : tab.w_down[ex]);
    };
    const uint16_t* B0 = pick(which0);
    const uint16_t* B1 = (EPI == EPI_SWIGLU) ? pick(which1) : B0;
    const int n0 = tile_n * NOUT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s_lo = piece * plan.per;
    const int ns = min(plan.per, ns_all - s_lo);

    // What this lane fetches.  A: blocks NA wave .. NA wave + NA - 1 of the 4 NA (NA = 2 MT); weights: blocks
    // 8 wave .. 8 wave + 7 of the 32 (the rows this wave reads).  In block blk the lane has row lane / 16 and
    // chunk (lane % 16) ^ (4 row + blk % 4).
    constexpr int NA = 2 * MT;
    const int lrow = lane >> 4;
    const char* a_ptr[NA];
    const char* b_ptr[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < NA) {
            const int blk = NA * wave + i;
            const int lc = (lane & 15) ^ ((lrow << 2) | (blk & 3));
            int ar = min(blk * 4 + lrow, nrows - 1);
            if (rel) ar = rel[ar];
            a_ptr[i] = reinterpret_cast<const char*>(A + (size_t)row0 * lda) + (size_t)ar * lda * 2 + lc * 16 + (size_t)s_lo * SKW * 2;
        }
        const int lc = (lane & 15) ^ ((lrow << 2) | (i & 3));
        const int rr = (8 * wave + i) * 4 + lrow;           // row of the 128-row weight tile
        int col;
        const uint16_t* base;
        if (EPI == EPI_SWIGLU) {
            base = (i >= 4) ? B1 : B0;                      // rows 16 .. 31 of a wave's 32 are the up rows
            col = n0 + wave * 16 + (rr & 15);
        } else {
            base = B0;
            col = n0 + rr;
        }
        b_ptr[i] = reinterpret_cast<const char*>(base) + (size_t)min(col, N - 1) * K * 2 + lc * 16 + (size_t)s_lo * SKW * 2;
    }
    auto issue = [&](int t) {                               // stage t of this piece into ring slot t % STAGES
        const int tc = min(t, ns - 1);                      // past the end: the last stage again, into a slot nobody reads
        unsigned char* st = lds + (t % G::STAGES) * G::STAGE;
        const size_t kb = (size_t)tc * SKW * 2;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const char* ap = a_ptr[i] + kb;
            __builtin_amdgcn_global_load_lds(ap, (__attribute__((address_space(3))) void*)(st + (NA * wave + i) * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const char* bp = b_ptr[i] + kb;
            __builtin_amdgcn_global_load_lds(bp, (__attribute__((address_space(3))) void*)(st + G::A_BYTES + (8 * wave + i) * 1024), 16, 0, 0);
        }
    };

    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

#pragma unroll
    for (int t = 0; t < G::STAGES - 1; ++t) issue(t);
    const int fr = lane & 31, fk = lane >> 5;
    for (int t = 0; t < ns; ++t) {
        // LOADS loads per stage and wave; stages t .. t + STAGES - 2 are outstanding: stage t has landed when at
        // most (STAGES - 2) * LOADS remain: 12 (MT = 2: three stages of 12) or 20 (MT = 1: four stages of 10)
        if (MT == 2) __builtin_amdgcn_s_waitcnt(0x0F7C);    // vmcnt(12)
        else __builtin_amdgcn_s_waitcnt(0x4F74);            // vmcnt(20): low four bits 4, high two bits 1
        __builtin_amdgcn_s_barrier();                       // everybody's part of stage t is in LDS; the slot of stage t - 1 is free
        issue(t + G::STAGES - 1);
        const unsigned char* st = lds + (t % G::STAGES) * G::STAGE;
#pragma unroll
        for (int s2 = 0; s2 < SKW / 16; ++s2) {
            const bf16x8 bfr = *reinterpret_cast<const bf16x8*>(st + G::A_BYTES + skinny_off(wave * 32 + fr, 2 * s2 + fk));
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const bf16x8 af = *reinterpret_cast<const bf16x8*>(st + skinny_off(i * 32 + fr, 2 * s2 + fk));
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr, af, acc[i], 0, 0, 0);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070);                      // no load may still be on its way to LDS when the block ends
    if (plan.parts > 1) {
        const __amdgpu_buffer_rsrc_t pieces = pieces_rsrc(partial + (size_t)tile_id * plan.parts * (G::PARTIAL / 4), (uint32_t)(plan.parts * G::PARTIAL));
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                store_piece(pieces, piece * (int)(G::PARTIAL / 16) + (i * 4 + q) * 256 + tid,
                            f32x4{acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]});
        if (!last_piece(m.done + tile_id, plan.parts, reinterpret_cast<int*>(lds))) return;
        f32x4 sum[4 * MT];
#pragma unroll
        for (int q = 0; q < 4 * MT; ++q) sum[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < plan.parts; p0 += 4) {         // four pieces in flight; past the last one it is read again and not added
            f32x4 v[4][4 * MT];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4 * MT; ++q) v[u][q] = load_piece(pieces, min(p0 + u, plan.parts - 1) * (int)(G::PARTIAL / 16) + q * 256 + tid);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p0 + u < plan.parts) {
#pragma unroll
                    for (int q = 0; q < 4 * MT; ++q) sum[q] += v[u][q];
                }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[i][4 * q + t] = sum[i * 4 + q][t];
    }
    skinny_store<EPI, MT>(acc, wave, lane, row0, nrows, rel, n0, N, C, ldc);
}

// Shares of up to a tile of rows per expert (see narrow_form): every weight is used once or twice, and what counts is how
// many CUs stream and what each has to fetch - a CU gets about 58 GB/s of operands that are not in its L2, whether 90 or 130
// KB of loads are in flight, what a tile costs besides included (55 to 110 GB/s without it, see kNarrowForms).  So a tile is 32 MT rows x only 32 NT weight rows over the whole of K: enough tiles for the
// chip without cutting K, which costs the 128 x 128 tiles and the kernel above 64 KB of partial sums per block, a counter and a
// last block that adds them.  Weights 2048 -> 1408 -> 2048 for four experts and 403 rows, weights from cold memory: 29.4 + 22.1
// -> 18.8 + 12.5 us; 64 rows of 2048 -> 2816 -> 2048 13.3 + 15.0 -> 11.2 + 10; a decode step with both 130 -> 95.
// 8 waves (4 for 32-row tiles), of which KP share a row tile and take a part of every stage each, added through LDS at the end:
// two waves per SIMD hide each other's LDS reads (19.4 + 12.9 us with one).  Rows fetched straight to the registers of the
// wave that multiplies them, which leaves the LDS to the weights, took 26.8 + 19.6: a load of 32 bytes from each of 32
// rows occupies the address unit four times as long as one of 256 bytes from each of 4.
template <int MT, int NT> struct NarrowGeom {
    static constexpr int BM_ = 32 * MT, BN_ = 32 * NT;
    static constexpr int KW = (MT == 4 && NT == 2) ? 64 : 128;   // elements of K per stage: smaller where a stage takes much of the ring
    static constexpr int RPL = 512 / KW;                 // rows that a wave-load (1 KB) fetches
    static constexpr int A_BYTES = BM_ * KW * 2;
    static constexpr int STAGE = A_BYTES + BN_ * KW * 2;
    static constexpr int WAVES = MT == 1 ? 4 : 8;
    static constexpr int NA = BM_ / RPL / WAVES, NB = BN_ / RPL / WAVES;   // wave-loads per stage and wave
    static constexpr int STAGES = 160 * 1024 / STAGE < 8 ? 160 * 1024 / STAGE : 8;
    static constexpr int LDS = STAGES * STAGE;
    static constexpr int AHEAD = (STAGES - 2) * (NA + NB);   // loads that may be outstanding when a stage is needed
    static constexpr int WAIT = 0x0070 | (AHEAD & 15) | (AHEAD >> 4) << 14;   // vmcnt(AHEAD) lgkmcnt(0)
    static constexpr int KP = WAVES / MT;                    // waves that share a row tile, each with a part of every stage
    static constexpr int STEPS = KW / 16 / KP;           // k-steps of a wave per stage
    static_assert(NB >= 1 && AHEAD < 64 && STEPS >= 1 && LDS >= WAVES * NT * 4096, "");
    // byte offset of (row, 16-byte chunk) inside an operand's part of a stage: blocks of one wave-load, conflict-free
    static __device__ __forceinline__ int off(int row, int c) { return KW == 64 ? f32_slot(row, c) * 16 : skinny_off(row, c); }
    // the chunk that lane l of a wave-load fetches, which goes to its slot l: row l / (64 / RPL) of block blk
    static __device__ __forceinline__ int chunk(int l, int blk) {
        return KW == 64 ? (l & 7) ^ ((l >> 4) | (blk & 1) << 2) : (l & 15) ^ ((l >> 4) << 2 | (blk & 3));
    }
};

// ONE: the list has one segment, whose tiles need no map (see ffn_impl).  An instantiation of its own: as a branch on the pointers it
// cost the lists that have a map 1.5 % (300 expert FFNs, from cold memory as from warm), and itself 1 %.
struct OneSegment { const int32_t *offset, *expert; int R, n_local; };
template <int EPI, int MT, int NT, bool ONE>
__global__ __launch_bounds__((64 * NarrowGeom<MT, NT>::WAVES), (NarrowGeom<MT, NT>::WAVES / 4)) void gemm_bf16_narrow_kernel(const uint16_t* __restrict__ A, int lda, TileMap m, ExpertTable tab,
                                                                  int which0, int which1, int N, int K, uint16_t* __restrict__ C, int ldc, int tiles_n, OneSegment one) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    using G = NarrowGeom<MT, NT>;
    constexpr int NOUT = (EPI == EPI_SWIGLU) ? G::BN_ / 2 : G::BN_;
    auto word = [](const int32_t* p, int i) { return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p))[i]; };
    int n_tiles_m, one_lo = 0, one_len = 0, one_expert = 0;
    if (ONE) {
        one_expert = word(one.expert, 0);
        one_lo = max(word(one.offset, 0), 0);
        const int hi = min(word(one.offset, 1), one.R);
        one_len = one_expert >= 0 && one_expert < one.n_local && hi > one_lo ? hi - one_lo : 0;
        n_tiles_m = (one_len + G::BM_ - 1) / G::BM_;
    } else {
        n_tiles_m = word(m.n_tiles, 0);
    }
    // The row tiles of a column tile on one XCD.  A grid of row and column tiles would let a block read its record without waiting
    // for the number of tiles, which gives nothing (300 expert FFNs from cold memory: 1.001), but where weights are still in
    // the L2s, or an expert has several row tiles, they come to several L2s: up to 14 % slower (182 rows of 1920 -> 4096 -> 1920 for two experts 28.9 -> 33.2 us).
    const int total = ONE ? n_tiles_m : n_tiles_m * tiles_n;
    for (int item = ONE ? blockIdx.y : blockIdx.x; item < total; item += ONE ? gridDim.y : gridDim.x) {   // one, unless the list has more runs than experts
        const int tile_id = ONE ? 0 : skinny_tile(item, total);
        const int tile_m = ONE ? item : __builtin_amdgcn_readfirstlane(tile_id % n_tiles_m);
        const int tile_n = ONE ? blockIdx.x : __builtin_amdgcn_readfirstlane(tile_id / n_tiles_m);
        int row0 = one_lo + tile_m * G::BM_, nrows = min(G::BM_, one_len - tile_m * G::BM_), ex = one_expert;
        const int32_t* rel = nullptr;
        if (!ONE) {
            row0 = word(m.row0, tile_m);
            nrows = word(m.nrows, tile_m);
            ex = word(m.expert, tile_m);
            if (word(m.gather, tile_m)) rel = m.rel + (size_t)tile_m * kRelPitch;
        }
        auto pick = [&](int which) { return reinterpret_cast<const char*>(which == 0 ? tab.w1[ex] : which == 1 ? tab.w_up[ex] : tab.w_down[ex]); };
        const int n0 = tile_n * NOUT;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int ns = K / G::KW;
        const int lrow = lane / (64 / G::RPL);
        const char* a_base = reinterpret_cast<const char*>(A + (size_t)row0 * lda);
        const char *b_base = pick(which0) + (size_t)n0 * K * 2, *u_base = (EPI == EPI_SWIGLU) ? pick(which1) + (size_t)n0 * K * 2 : b_base;
        uint32_t a_voff[G::NA], b_voff[G::NB];
        int ar[G::NA];
#pragma unroll
        for (int i = 0; i < G::NA; ++i) ar[i] = min((G::NA * wave + i) * G::RPL + lrow, nrows - 1);
        if (rel) {
            int t[G::NA];
#pragma unroll
            for (int i = 0; i < G::NA; ++i) t[i] = rel[ar[i]];
#pragma unroll
            for (int i = 0; i < G::NA; ++i) ar[i] = t[i];
        }
#pragma unroll
        for (int i = 0; i < G::NA; ++i) a_voff[i] = (uint32_t)ar[i] * (uint32_t)lda * 2u + (uint32_t)G::chunk(lane, G::NA * wave + i) * 16u;
#pragma unroll
        for (int i = 0; i < G::NB; ++i) {
            const int blk = G::NB * wave + i, rr = blk * G::RPL + lrow;
            const int col = (EPI == EPI_SWIGLU) ? (rr >> 5) * 16 + (rr & 15) : rr;   // rows 16 .. 31 of each 32 are up rows
            b_voff[i] = (uint32_t)min(col, N - 1 - n0) * (uint32_t)K * 2u + (uint32_t)G::chunk(lane, blk) * 16u;
        }
        auto issue = [&](int t) {                            // stage t into ring slot t % STAGES; past the end the last one again
            unsigned char* st = lds + (t % G::STAGES) * G::STAGE;
            const size_t kb = (size_t)min(t, ns - 1) * G::KW * 2;
#pragma unroll
            for (int i = 0; i < G::NB; ++i) {
                const int blk = G::NB * wave + i;
                const char* p = ((EPI == EPI_SWIGLU && (blk * G::RPL & 16)) ? u_base : b_base) + kb;
                unsigned char* to = st + G::A_BYTES + blk * 1024;
                uint32_t& v = b_voff[i];
                asm volatile("" : "+s"(p), "+v"(v));
                __builtin_amdgcn_global_load_lds(p + v, (__attribute__((address_space(3))) void*)to, 16, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < G::NA; ++i) {
                const char* p = a_base + kb;
                unsigned char* to = st + (G::NA * wave + i) * 1024;
                uint32_t& v = a_voff[i];
                asm volatile("" : "+s"(p), "+v"(v));
                __builtin_amdgcn_global_load_lds(p + v, (__attribute__((address_space(3))) void*)to, 16, 0, 0);
            }
        };
        f32x16 acc[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
#pragma unroll
        for (int t = 0; t < G::STAGES - 1; ++t) issue(t);
        const int fr = lane & 31, fk = lane >> 5;
        const int rt = wave % MT, kp = wave / MT;            // row tile of this wave, its part of a stage
        for (int t = 0; t < ns; ++t) {
            __builtin_amdgcn_s_waitcnt(G::WAIT);             // stage t has landed
            __builtin_amdgcn_s_barrier();                    // everybody's part of it; the slot of stage t - 1 is free
            asm volatile("" ::: "memory");
            const unsigned char* st = lds + (t % G::STAGES) * G::STAGE;
            bf16x8 af[G::STEPS], bf[G::STEPS][NT];
#pragma unroll
            for (int s = 0; s < G::STEPS; ++s) {
                const int c = 2 * (kp * G::STEPS + s) + fk;
                af[s] = *reinterpret_cast<const bf16x8*>(st + G::off(rt * 32 + fr, c));
#pragma unroll
                for (int j = 0; j < NT; ++j) bf[s][j] = *reinterpret_cast<const bf16x8*>(st + G::A_BYTES + G::off(j * 32 + fr, c));
            }
            issue(t + G::STAGES - 1);
#pragma unroll
            for (int s = 0; s < G::STEPS; ++s)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[s][j], af[s], acc[j], 0, 0, 0);
        }
        __builtin_amdgcn_s_waitcnt(0x0070);                  // no load may still be on its way to LDS
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // the parts of a row tile are added in order by the wave of the first one
        f32x4* parts = reinterpret_cast<f32x4*>(lds);
        if (kp > 0)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    parts[((kp * MT + rt) * NT + j) * 256 + q * 64 + lane] = f32x4{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
        __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int gr = rt * 32 + fr;
        if (kp == 0 && gr < nrows) {
#pragma unroll
            for (int k2 = 1; k2 < G::KP; ++k2)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = parts[((k2 * MT + rt) * NT + j) * 256 + q * 64 + lane];
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[j][4 * q + t] += v[t];
                    }
            uint16_t* crow = C + (size_t)(row0 + (rel ? rel[gr] : gr)) * ldc;
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int g = 0; g < ((EPI == EPI_SWIGLU) ? 2 : 4); ++g) {
                    float v[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = epilogue_bf16<EPI>(acc[j][4 * g + t], (EPI == EPI_SWIGLU) ? acc[j][4 * ((g + 2) & 3) + t] : 0.f);
                    const int col = n0 + j * (NOUT / NT) + g * 8 + fk * 4;
                    if (col < N) *reinterpret_cast<u32x2*>(crow + col) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                }
        }
        __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();                        // the next item's loads go to the same LDS
    }
}

// ------------------------------------------------------------------------------------------------
// Experts of a few hundred KB (see takes_small): both GEMMs of 32 rows by one block, in one launch and without a tile map.  Such a
// share is bound by its launches - 2 to 3 us each at their shortest, where the products take one - so a block works its tile
// out from the segment list (see SegList), takes the weights straight from the caches to registers and keeps its rows of the
// intermediate in LDS.  Rows of operands are read as fragments of 16 rows x 64 bytes: 32 elements of bf16 for one
// v_mfma_f32_16x16x32_bf16, 16 of fp32 for four v_mfma_f32_16x16x4_f32 (lane group g has elements 4 g .. 4 g + 3 and feeds one to
// each: the order of the sum over k is free).  D = B . A^T: a lane ends with 4 consecutive columns of a row.
constexpr int kSmallRows = 32, kSmallSteps = 4;              // rows per block; fragments of K that are loaded together
template <int DT> __device__ __forceinline__ f32x4 small_mma(const u32x4& w, const u32x4& a, f32x4 acc) {
    if (DT == MOE_BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), acc, 0, 0, 0);
    const f32x4 wf = __builtin_bit_cast(f32x4, w), af = __builtin_bit_cast(f32x4, a);
#pragma unroll
    for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[v], af[v], acc, 0, 0, 0);
    return acc;
}
// CT column tiles of 16, from column c0 on, of both row tiles: acc[m] += W_m[c0 + 16 c + ..] . rows over `steps` fragments of K, for
// NM matrices at once.  a(i, s): fragment s of row tile i
template <int DT, int NM, int CT, typename Rows>
__device__ __forceinline__ void small_product(const char* (&w)[NM], size_t w_pitch, int c0, int steps, Rows a, f32x4 (&acc)[NM][CT][2]) {
    const int lane = threadIdx.x & 63;
    const size_t w_off = (size_t)(c0 + (lane & 15)) * w_pitch + (lane >> 4) * 16;
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[m][c][0] = acc[m][c][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < steps; s0 += kSmallSteps) {
        u32x4 wf[NM][CT][kSmallSteps], af[2][kSmallSteps];
#pragma unroll
        for (int s = 0; s < kSmallSteps; ++s) {
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int c = 0; c < CT; ++c) wf[m][c][s] = *reinterpret_cast<const u32x4*>(w[m] + w_off + c * 16 * w_pitch + (s0 + s) * 64);
#pragma unroll
            for (int i = 0; i < 2; ++i) af[i][s] = a(i, s0 + s);
        }
#pragma unroll
        for (int s = 0; s < kSmallSteps; ++s)
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int i = 0; i < 2; ++i) acc[m][c][i] = small_mma<DT>(wf[m][c][s], af[i][s], acc[m][c][i]);
    }
}
template <int DT> __device__ __forceinline__ void small_store(char* p, const float (&v)[4]) {
    if (DT == MOE_BF16) *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    else *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
}
template <int DT, int EPI>
__global__ __launch_bounds__(256) void ffn_small_kernel(const char* __restrict__ x, SegList seg, ExpertTable tab, int H, int F, char* __restrict__ out) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int ES = DT == MOE_BF16 ? 2 : 4;
    WaveLanes wl;
    const SmallMap map = load_segments(seg, kSmallRows, wl);
    const int n_tiles = __builtin_amdgcn_readfirstlane(map.n_tiles);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fr = lane & 15, g = lane >> 4;
    for (int item = blockIdx.x; item < n_tiles; item += gridDim.x) {   // one, unless the list has more runs than experts
        const SmallTile t = small_tile(wl, map, item, kSmallRows);
        int row[2] = {min(fr, t.nrows - 1), min(16 + fr, t.nrows - 1)};
        segment_rows(wl, t, row);
        const char* xr[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) xr[i] = x + (size_t)(t.row0 + row[i]) * H * ES + g * 16;
        const int ex = __builtin_amdgcn_readfirstlane(t.expert);
        const char *w1 = reinterpret_cast<const char*>(tab.w1[ex]), *wu = reinterpret_cast<const char*>(tab.w_up[ex]), *wd = reinterpret_cast<const char*>(tab.w_down[ex]);
        const int pitch = F * ES + 16;                           // of a row of the intermediate: spreads the rows over the banks
        auto first = [&](auto tiles) {
            constexpr int CT = decltype(tiles)::value;
            for (int ct = wave * CT; ct < F / 16; ct += 4 * CT) {
                constexpr int NM = EPI == EPI_SWIGLU ? 2 : 1;
                const char* w[NM];
                w[0] = w1;
                if (NM == 2) w[NM - 1] = wu;
                f32x4 acc[NM][CT][2];
                auto rows = [&](int i, int s) { return *reinterpret_cast<const u32x4*>(xr[i] + s * 64); };
                small_product<DT, NM, CT>(w, (size_t)H * ES, ct * 16, H * ES / 64, rows, acc);
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        float v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = DT == MOE_BF16 ? epilogue_bf16<EPI>(acc[0][c][i][q], acc[NM - 1][c][i][q]) : epilogue<EPI>(acc[0][c][i][q], acc[NM - 1][c][i][q]);
                        small_store<DT>(reinterpret_cast<char*>(lds) + (i * 16 + fr) * pitch + ((ct + c) * 16 + g * 4) * ES, v);
                    }
            }
        };
        auto second = [&](auto tiles) {
            constexpr int CT = decltype(tiles)::value;
            for (int ct = wave * CT; ct < H / 16; ct += 4 * CT) {
                const char* w[1] = {wd};
                f32x4 acc[1][CT][2];
                auto rows = [&](int i, int s) { return *reinterpret_cast<const u32x4*>(lds + (i * 16 + fr) * pitch + s * 64 + g * 16); };
                small_product<DT, 1, CT>(w, (size_t)F * ES, ct * 16, F * ES / 64, rows, acc);
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const float v[4] = {acc[0][c][i][0], acc[0][c][i][1], acc[0][c][i][2], acc[0][c][i][3]};
                        if (i * 16 + fr < t.nrows) small_store<DT>(out + ((size_t)(t.row0 + row[i]) * H + (ct + c) * 16 + g * 4) * ES, v);
                    }
            }
        };
        if (F % 128 == 0) first(std::integral_constant<int, 2>{});
        else first(std::integral_constant<int, 1>{});
        __syncthreads();
        if (H % 256 == 0) second(std::integral_constant<int, 4>{});
        else second(std::integral_constant<int, 1>{});
        __syncthreads();                                     // the next tile's intermediate goes to the same LDS
    }
}

constexpr int kMaxCU = 256;                    // tail pieces per launch, at most: sizes the partial-tile workspace

// number of CUs of the current device (a round of the grid), at most kMaxCU
int round_size() {
    static int ncu = 0;
    if (ncu == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = kMaxCU;
        ncu = n < kMaxCU ? n : kMaxCU;
    }
    return ncu;
}

// Tiles that a block walks through.  A block holds its CU - all of its LDS and registers - until it ends, and what another
// stream has queued (a decode step of a second model, its gate, its send buffer) waits for that, at every kernel of its
// chain.  A decode share of 16 tokens (150 us alone) beside a prefill, one block per CU to the end of the GEMM -> runs of
// 210 us that end one after the other (-> a block per tile): gate to send buffer beside 20571 rows of 4096 -> 14336 -> 4096
// 3.0 -> 0.39 (0.27) ms, the whole share 4.8 -> 2.3 (1.35) ms; beside 200000 rows of 2048 -> 1408 -> 2048 1.26 -> 0.16
// (0.14) and 2.3 -> 1.4 (0.76) ms; beside 40000 rows of 1024 -> 4096 -> 1024 0.89 -> 0.53 (0.53) ms.  What a new block
// costs (4.7 us) shows as 0.5 to 1.4 % of those GEMMs; runs of 100 us cost 1.5 to 3.8 %.  (The k-tiles below are of loops with 32 x 32 x 16
// products; those of 256 rows take 0.69 to 0.75 us today.)
constexpr double kWalkUs = 210.0;
int walk_tiles(int rows, int K) {
    const double k_tile_us = rows == TileGeom<2, 2>::BM ? 0.53 : rows == TileGeom<3, 4>::BM ? 0.61 : 0.75;   // on a full chip
    return std::max(1, (int)(kWalkUs / (5.0 + k_tile_us * (K / BK))));
}
// blocks for up to max_items tiles and pieces, of which only the device knows the number
int walk_blocks(int max_items, int walk, int ncu) {
    const int rounds = (max_items + ncu - 1) / ncu;
    return (rounds <= walk ? 1 : (rounds + 2 * walk - 2) / walk) * ncu;
}

enum TileShape { TS_128, TS_192, TS_256 };
// When the loads of 128 x 128 tiles go out as early as they can.  Time with spread loads over time with early ones, operands in the caches /
// from memory, by the number of tiles, 1000 GEMMs of 100 to 14000 rows, K and N up to 2048: K up to 384 0.94 to 0.99 / 0.97 to 1.01, 512 to 1024
// 0.96 to 1.01 / 0.97 to 1.05, from 1152 on 0.98 to 1.03 / 0.99 to 1.05; 235 of K from 512 to 7168 1.016 / 1.038.  Between 512 and 1024 it depends
// on where the operands are, and the spread loads are the ones that lose less (early ones: 7 to 10 % of a GEMM of 12 to 20 us).
// From 1152 on, grids of 257 to 450 tiles, where some CUs have two blocks and others one, take 1.01 to 1.04 times as long as with the
// 32 x 32 x 16 loop before this one, up to 1.16 times; with one block per CU, or two on all, early loads are 1.02 to 1.08 times as fast.
constexpr int kSoonK = 1152;
bool loads_soon(TileShape t, int K) { return t == TS_128 && K >= kSoonK; }
template <int EPI, int MI, int NJ, bool SOON, bool TIMED>
int launch_bf16(const void* A, int lda, const TileMap& m, const int32_t* strips, const ExpertTable& tab, int which0, int which1, int N, int K,
                void* C, int ldc, int R, int nseg, int n_used, float* partial, hipStream_t st, long long* marks,
                size_t marks_len) {
    using TG = TileGeom<MI, NJ>;
    using G = EpiGeom<EPI, MI, NJ>;
    const int tiles_n = (N + G::NOUT - 1) / G::NOUT;
    const int ncu = round_size() * TG::PER_CU;             // tiles per round of the grid
    static bool attr_done = false;
    if (!attr_done) {
        MOE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<EPI, MI, NJ, SOON, TIMED>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, TG::LDS));
        attr_done = true;
    }
    // The tile count is only known on the device: the most tail tiles over every count that n_used runs of rows which
    // share no tile can give.  A list that leaves rows out may have fewer tiles; its tail is cut if it fits as well.
    int most_tail = 0;
    for (int t = (R + TG::BM - 1) / TG::BM, hi = (R + n_used * (TG::BM - 1)) / TG::BM; t <= hi; ++t)
        most_tail = std::max(most_tail, plan_tail(t * tiles_n, ncu, K / BK).n_tail);
    const int walk = walk_tiles(TG::BM, K);
    hipLaunchKernelGGL((gemm_bf16_kernel<EPI, MI, NJ, SOON, TIMED>), dim3(walk_blocks(max_tiles_of(R, TG::BM, nseg) * tiles_n + ncu, walk, ncu)), dim3(256), TG::LDS, st,
                       reinterpret_cast<const uint16_t*>(A), lda, m, tab, which0, which1, N, K,
                       reinterpret_cast<uint16_t*>(C), ldc, tiles_n, strips, ncu, walk, most_tail, partial, marks,
                       (uint32_t)std::min<size_t>(marks_len / 16, 0xFFFFFFFFu));
    MOE_LAUNCH_CHECK("gemm_bf16_kernel");
    if constexpr (!TG::SUM_IN_PLACE) {
        if (most_tail > 0) {
            hipLaunchKernelGGL((gemm_bf16_tail_kernel<EPI, MI, NJ>), dim3(most_tail * MI * G::NJO), dim3(256), 0, st, m, N, K,
                               reinterpret_cast<uint16_t*>(C), ldc, tiles_n, strips, ncu, most_tail, partial);
            MOE_LAUNCH_CHECK("gemm_bf16_tail_kernel");
        }
    }
    return MOE_OK;
}

template <int EPI>
int launch_bf16_shape(TileShape t, const void* A, int lda, const TileMap& m, const int32_t* strips, const ExpertTable& tab, int which0, int which1, int N, int K,
                      void* C, int ldc, int R, int nseg, int n_used, float* partial, hipStream_t st, bool timed, long long* marks, size_t marks_len) {
#define MOE_GEMM(...) launch_bf16<EPI, __VA_ARGS__>(A, lda, m, strips, tab, which0, which1, N, K, C, ldc, R, nseg, n_used, partial, st, marks, marks_len)
    if (loads_soon(t, K)) return timed ? MOE_GEMM(2, 2, true, true) : MOE_GEMM(2, 2, true, false);
    if (t == TS_128) return timed ? MOE_GEMM(2, 2, false, true) : MOE_GEMM(2, 2, false, false);
    if (t == TS_192) return timed ? MOE_GEMM(3, 4, false, true) : MOE_GEMM(3, 4, false, false);
    return timed ? MOE_GEMM(4, 4, false, true) : MOE_GEMM(4, 4, false, false);
#undef MOE_GEMM
}

// Which tiles a bf16 GEMM takes.  The number of tiles is only known on the device, so the choice is made from an
// estimate of it: half a tile of padding per expert.  Every shape's time is modelled as rounds of the grid, a round
// costing a + b * (k-tiles of 32), and a tail as plan_tail cuts it; the first round of the large shapes starts cold; the
// shape with the least time is preferred, and taken if it holds up (see confirm_shape).  The
// constants (microseconds) are from GEMMs of K = 1024 ... 14336 with whole rounds, in loops of 32 x 32 x 16 products (2 to 9 % slower
// than today's, 5 to 12 at 128 x 128; see below for how the choice does on today's): 256 x 256 100 us per round at
// K = 4096, 37 at 1024; 192 x 256 80 us at 4096; 128 x 128, two blocks per CU, 66 us at 4096 and 36 at 2048, and
// about two thirds of that when the round has one block per CU.  So 256 x 256 is the best rate (1.35 PFLOP/s against
// 1.3 and 1.0) and the others win where it leaves CUs idle or rows empty: at 2048 -> 1408 -> 2048 with four experts
// and 400 rows 35 + 33 us against 27 + 18 for 128 x 128; at 1024 -> 4096 -> 1024 and 10199 rows the second GEMM 93
// against 80 us for 192 x 256 (220 tiles for 256 CUs instead of 160).
constexpr int kShapeRows[] = {TileGeom<2, 2>::BM, TileGeom<3, 4>::BM, TileGeom<4, 4>::BM};
constexpr int kSkinnyRows = 64;                          // shares up to this many rows take the streaming kernels where narrow tiles do not win
inline double estimated_tiles_m(int R, int bm, int n_used) {
    if (n_used <= 1) return (R + bm - 1) / bm;
    return std::max((double)n_used, (double)R / bm + 0.5 * n_used);
}
double modelled_us(TileShape t, int R, int n_used, int N, int K, int act, int cus) {
    struct Cost { double first, a, b, a1, b1, piece; };    // start, round, round of at most one block per CU, pass over a partial tile
    static const Cost cost[] = {{0.0, 6.5, 0.467, 6.0, 0.33, 0.026}, {3.0, 4.6, 0.565, 4.6, 0.565, 0.079}, {3.0, 6.6, 0.71, 6.6, 0.71, 0.105}};
    Cost c = cost[t];
    if (act == MOE_ACT_GELU_MLP) c.a += (t == TS_128) ? 1.0 : 4.0;   // its exp2 and rcp of twice SwiGLU's columns, hidden where two blocks share a CU
    const int per_cu = (t == TS_128) ? TileGeom<2, 2>::PER_CU : 1, slots = cus * per_cu;
    const int out_cols = ((t == TS_128) ? TileGeom<2, 2>::BN : TileGeom<4, 4>::BN) / (act == MOE_ACT_SWIGLU ? 2 : 1);
    const int tiles = (int)(estimated_tiles_m(R, kShapeRows[t], n_used) * ((N + out_cols - 1) / out_cols) + 0.5);
    const TailPlan p = plan_tail(tiles, slots, K / BK);
    const int rest = p.n_full % slots;                     // tiles of a last round that is not cut
    double us = c.first + (double)(p.n_full / slots) * (c.a + c.b * (K / BK));
    if (rest > 0) us += (rest <= cus) ? c.a1 + c.b1 * (K / BK) : c.a + c.b * (K / BK);
    if (p.n_tail > 0) {
        const int pieces = p.n_tail * p.parts;
        us += ((pieces <= cus) ? c.a1 + c.b1 * 2 * p.pairs_per : c.a + c.b * 2 * p.pairs_per) + 5.0 + pieces * c.piece;
    }
    return us;
}
TileShape choose_shape(int R, int n_used, int N, int K, int act, int cus) {
    TileShape best = TS_256;
    double best_us = modelled_us(TS_256, R, n_used, N, K, act, cus);
    for (TileShape t : {TS_192, TS_128}) {
        const double us = modelled_us(t, R, n_used, N, K, act, cus);
        if (us < best_us) { best = t; best_us = us; }
    }
    return best;
}

// A height other than 256 has to hold up.  The choice above rests on a mean tile count and on rates of full rounds; where
// either is off, the smaller tiles cost up to a third (210 rows for each of 32 experts, 1664 -> 6656 -> 1664: 192 and 128
// rows per tile 645 us, 256 478).  So a chosen height is played once more, with
//   - rates that follow the occupancy: a k-tile of a 256 x 256 tile takes 0.57 us on a nearly empty chip and 0.75 on a full
//     one, at 128 x 128 0.38 with a block to itself and 0.53 beside another;
//   - the bytes of weights and rows at the rate a GEMM streams them (5.5 - 6 TB/s), combined with the compute time by
//     their 4-norm: near the crossing both count;
//   - five ways in which the rows may be spread over the experts: even shares, even popularity (shares that differ by
//     chance), popularity 1 / rank, and half a tile of padding per expert give or take its standard deviation;
// each against 256 x 256 tiles played the same way.  What counts is the mean of the five quotients and the worst of them,
// half each; a height at which that exceeds 1.04 is given up for the one with the least (256 has 1).  The constants are
// fitted to 430000 GEMMs of 65 to 20000 rows, 1 to 64 experts, H and F of 128 to 14336, weights from cold memory (median
// error 5 %).  Over those the expert FFN is more than 3 % slower than one block per 256 x 256 tile was in 0.4 % of the
// shares, in 2.9 % without this check; the mean gain is 1.249, 1.230 without.  (All of this is of the loops with 32 x 32 x 16
// products.  On today's, 460 shares of 65 to 20000 rows that take another height than 256 and no narrow tiles, one after the other with operands
// in the caches where they fit: 1.37 times as fast in the geometric mean as with 256 x 256 tiles, three more than 3 % slower.  Fitted again to
// 68000 GEMMs of today's the rule would be 0.5 % faster in the mean and more than 3 % slower in 4 % of them; tiles of 192 x 128 beside the three,
// 2.2 % faster and 1.1 %.)
struct ShapeCost { double start, a, b, a2, pair, b_pair, piece0, piece, gelu, tb_s, first_bytes; };
double played_us(TileShape t, int tiles_m, int R, int n_used, int N, int K, int act, int cus) {
    // start of the launch; per round and per k-tile of it (at no occupancy, and what full occupancy adds); rounds with two
    // blocks per CU: extra per round, and their k-tile; K cuts: per launch and piece; GELU per round; bytes
    static const ShapeCost cost[] = {{6.5, -0.1, 0.374, 2.2, 0.441, 0.094, 9.8, 0.030, 1.6, 5.5, 3.0},
                                     {3.6, 4.8, 0.527, 0.0, 0.0, 0.083, 9.3, 0.054, 3.7, 5.6, 9.4},
                                     {4.3, 6.0, 0.555, 0.0, 0.0, 0.191, 10.0, 0.057, 4.4, 6.0, 9.8}};
    const ShapeCost& c = cost[t];
    const int per_cu = (t == TS_128) ? TileGeom<2, 2>::PER_CU : 1, slots = cus * per_cu, nk = K / BK, mats = (act == MOE_ACT_SWIGLU) ? 2 : 1;
    const int out_cols = ((t == TS_128) ? TileGeom<2, 2>::BN : TileGeom<4, 4>::BN) / mats;
    const TailPlan p = plan_tail(tiles_m * ((N + out_cols - 1) / out_cols), slots, nk);
    const double a = c.a + (act == MOE_ACT_GELU_MLP ? c.gelu : 0.0);
    auto k_tile = [&](double q) { return (per_cu == 2 && q <= 0.5) ? c.b + 0.074 * q : (per_cu == 2 ? c.pair : c.b) + c.b_pair * q; };
    auto round = [&](double q) { return a + (q > 0.5 ? c.a2 : 0.0) + k_tile(q) * nk; };   // of q * slots tiles
    double us = (p.n_full / slots) * round(1.0);
    if (p.n_full % slots > 0) us += round((double)(p.n_full % slots) / slots);
    if (p.n_tail > 0) us += c.piece0 + k_tile((double)(p.n_tail * p.parts) / slots) * 2 * p.pairs_per + p.n_tail * p.parts * c.piece;
    const double bytes = ((double)n_used * N * K * mats + (double)R * (K + N)) * 2.0;
    const double mem = c.first_bytes + bytes * 1e-6 / c.tb_s;
    us = std::max(us, 0.1);
    return c.start + std::sqrt(std::sqrt(us * us * us * us + mem * mem * mem * mem));
}
// M-tiles of bm rows when R rows are spread over n_used experts in way 0 .. 4
int spread_tiles_m(int R, int bm, int n_used, int way) {
    if (n_used <= 1) return (R + bm - 1) / bm;
    if (way == 0) return n_used * (((R + n_used - 1) / n_used + bm - 1) / bm);
    if (way == 1) {
        double ranks = 0.0;
        for (int e = 1; e <= n_used; ++e) ranks += 1.0 / e;
        int tiles = 0;
        for (int e = 1; e <= n_used; ++e) tiles += (int)std::ceil(R / (e * ranks * bm));
        return tiles;
    }
    if (way == 2) {                                        // an expert has more than j tiles with the chance that its rows exceed j * bm
        const double share = (double)R / n_used, sd = std::sqrt(share);
        int j = std::max(1, (int)((share - 6.0 * sd) / bm));
        double tiles = j;
        for (; j * bm < share + 6.0 * sd; ++j) tiles += 0.5 * std::erfc((j * bm - share) / (sd * 1.4142135623730951));
        return std::max(n_used, (int)std::lround(n_used * tiles));
    }
    const double mean = (double)R / bm + 0.5 * n_used, sd = std::sqrt(n_used / 12.0);
    return std::max(n_used, (int)(way == 3 ? std::ceil(mean + sd) : std::floor(mean - sd)));
}
// time of height t over that of 256 rows when the rows are spread in way `way`
double against_256(TileShape t, int way, int R, int n_used, int N, int K, int act, int cus) {
    return played_us(t, spread_tiles_m(R, kShapeRows[t], n_used, way), R, n_used, N, K, act, cus) /
           played_us(TS_256, spread_tiles_m(R, kShapeRows[TS_256], n_used, way), R, n_used, N, K, act, cus);
}
double held_up(TileShape t, int R, int n_used, int N, int K, int act, int cus) {
    const int ways = n_used <= 1 ? 1 : 5;
    double sum = 0.0, worst = 0.0;
    for (int way = 0; way < ways; ++way) {
        const double q = against_256(t, way, R, n_used, N, K, act, cus);
        sum += q;
        worst = std::max(worst, q);
    }
    return 0.5 * (sum / ways + worst);
}
// A height that is 12 % faster at even shares (57 % of those that are preferred to 256) is taken without the other four:
// nothing is lost by it, and the call's host time stays (1.5 us of playing where a whole share of the layer takes 76).
TileShape confirm_shape(TileShape t, int R, int n_used, int N, int K, int act, int cus) {
    if (t == TS_256 || against_256(t, 0, R, n_used, N, K, act, cus) <= 0.88 || held_up(t, R, n_used, N, K, act, cus) <= 1.04) return t;
    const TileShape other = t == TS_128 ? TS_192 : TS_128;
    return held_up(other, R, n_used, N, K, act, cus) < 1.0 ? other : TS_256;
}
// column tiles of a GEMM of N output columns and tiles of bn weight rows
int tiled_columns(int N, bool swiglu, int bn) { return swiglu ? (2 * N + bn - 1) / bn : (N + bn - 1) / bn; }
// Short loops gain nothing from operands that an XCD's tiles share and lose more than that.  First GEMMs with bands / with strips, 128 x 128
// tiles: at K = 128 and 256 0.78 to 1.04, 0.94 in the geometric mean of 41 (4065 rows of 256 -> 1664 14.5 -> 17.7 us), at 384 and 512 0.99,
// from 640 on 1.01 to 1.03.  Larger tiles: at 256 and 384 FFNs of 0.99 to 1.00, at 512 1.013 and 1.016.
int least_strip_k(int bm) { return bm == TileGeom<2, 2>::BM ? 640 : 512; }
// tiles_n, or 0 if none of the tile counts that n_used runs of R rows can have is numbered in strips
int columns_in_strips(int R, int bm, int n_used, int tiles_n, int K) {
    if (K < least_strip_k(bm)) return 0;
    const int hi = (int)((R + (int64_t)n_used * (bm - 1)) / bm);
    for (int t = (R + bm - 1) / bm; t <= hi; ++t)
        if (plan_strips(t, tiles_n).wide > 0) return tiles_n;
    return 0;
}
// Items (tiles and pieces) that a GEMM of N output columns over R rows in nseg segments can have at most.
size_t max_items(TileShape t, int R, int nseg, int N, int act, int cus) {
    const int out_cols = ((t == TS_128) ? TileGeom<2, 2>::BN : TileGeom<4, 4>::BN) / (act == MOE_ACT_SWIGLU ? 2 : 1);
    return (size_t)max_tiles_of(R, kShapeRows[t], nseg) * ((N + out_cols - 1) / out_cols) + (size_t)cus * (t == TS_128 ? TileGeom<2, 2>::PER_CU : 1);
}
// The records that the maps of two heights take of the workspace, which has room for one map of 64-row tiles, and whether
// two more stay free: the counters of the tiles that are cut along K (2 x 256) lie there.
static_assert(2 * kMaxSplitTiles == 2 * kRelPitch, "two rows of the offset table");
bool maps_fit(int R, int nseg, int bm0, int bm1) {
    return max_tiles_of(R, bm0, nseg) + (bm0 == bm1 ? 0 : max_tiles_of(R, bm1, nseg)) + 2 <= max_tiles_for(R);
}
// The heights that both GEMMs of a share take.  With too many segments for two maps: one height, the first GEMM's if it
// holds up for the second as well, else 256.  (The map of one height always fits: up to 255 rows there are fewer tiles than rows,
// from 256 on at least two records more than ceil(R / 128) + 1024.)
void take_shapes(int R, int n_used, int nseg, int H, int F, int act, int cus, TileShape (&shape)[2]) {
    shape[0] = confirm_shape(choose_shape(R, n_used, F, H, act, cus), R, n_used, F, H, act, cus);
    shape[1] = confirm_shape(choose_shape(R, n_used, H, F, -1, cus), R, n_used, H, F, -1, cus);
    if (!maps_fit(R, nseg, kShapeRows[shape[0]], kShapeRows[shape[1]])) {
        if (confirm_shape(shape[0], R, n_used, H, F, -1, cus) != shape[0]) shape[0] = TS_256;
        shape[1] = shape[0];
    }
}

// Shares of at most kSkinnyRows rows (the tile map is then made of 32 MT-row tiles).
inline int skinny_tile_rows(int R) { return R <= 32 ? 32 : 64; }
template <int EPI, int MT>
int launch_bf16_skinny_mt(const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                          void* C, int ldc, int R, int nseg, float* partial, hipStream_t st) {
    using G = SkinnyGeom<MT>;
    const int nout = (EPI == EPI_SWIGLU) ? SBN / 2 : SBN;
    const int tiles_n = (N + nout - 1) / nout;
    const int max_total = max_tiles_of(R, G::BM_, nseg) * tiles_n;
    const int ncu = round_size();
    static bool attr_done = false;
    if (!attr_done) {
        MOE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_skinny_kernel<EPI, MT>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS));
        attr_done = true;
    }
    // a tile count below the CU count is multiplied by its pieces up to at most ncu blocks
    hipLaunchKernelGGL((gemm_bf16_skinny_kernel<EPI, MT>), dim3(std::max(max_total, ncu)), dim3(256), G::LDS, st,
                       reinterpret_cast<const uint16_t*>(A), lda, m, tab, which0, which1, N, K,
                       reinterpret_cast<uint16_t*>(C), ldc, tiles_n, ncu, partial);
    MOE_LAUNCH_CHECK("gemm_bf16_skinny_kernel");
    return MOE_OK;
}
// Which shares take narrow tiles, and of which form.  The time of a form is modelled as what a CU has to fetch, round of tiles by round
// (the last one at a higher rate where it leaves CUs idle), together with the weights at the rate they stream and with all that is
// fetched, again and again for every tile, from caches (the 4-norm of the three); that of the weight-streaming kernels likewise, with
// their pieces; that of the tiled kernels as in played_us; all with what the start of a kernel costs.  A form has to be 13 % faster in
// the mean of the five ways in which rows spread over experts (spread_tiles_m), 12 % beside the streaming kernels; even popularity alone
// decides where it says less than 0.6 or more than the other kernel's time.  Only up to 128 rows per expert: beyond, the
// weights are fetched again for every tile of rows.  The constants are fitted to the kernel durations of 2000 GEMMs, each with every form
// and without: shares of 1 to 2000 rows, 1 to 16 experts, H of 128 to 4096 and F of 128 to 14336, rows in even shares, by chance,
// by popularity and cut at random, weights from cold memory (median error 8 %).  Over 1200 other shares the expert FFN is 1.322
// times faster in the mean than without narrow tiles, two are more than 3 % slower (4 %); with one spread of the rows and equal
// starts of all kernels 39 of 900 were, by up to 20 %.  2500 shares by their kernel durations: 1.390 faster, 1.424 with the best form
// always known, 12 more than 3 % slower; with 10 and 8 % 1.395 and 19, with 18 % 1.372 and 4.  (All beside tiled kernels of 32 x 32 x 16 products.
// Beside today's, 260 shares with narrow tiles, of up to 32 experts and with operands in the caches where they fit: 1.34 times as fast as
// without, eleven more than 3 % slower, ten of them by 3 to 9 %, shares of 14 experts and more.)
struct NarrowForm { int mt, nt; };                       // mt = 0: none
struct NarrowCost { NarrowForm form; double start, gb_s, per_round, tb_s, all_tb_s, alone; };   // alone: what an otherwise idle chip adds to gb_s
constexpr NarrowCost kNarrowForms[] = {{{4, 2}, 1.45, 57.2, 2.95, 10.0, 100.0, 0.70}, {{2, 2}, 1.66, 46.6, 2.96, 10.0, 24.2, 1.18},
                                       {{2, 1}, 1.25, 65.0, 2.82, 10.0, 21.0, 0.68}, {{1, 2}, 1.62, 51.5, 2.97, 5.16, 100.0, 0.98},
                                       {{1, 1}, 1.72, 60.1, 2.43, 6.01, 17.9, 0.88}};
constexpr double kNarrowGain = 0.87, kNarrowGainStreaming = 0.88;
double norm4(double a, double b, double c = 0.0) { return std::sqrt(std::sqrt(a * a * a * a + b * b * b * b + c * c * c * c)); }
double weights_us(int n_used, int N, int K, int act, double tb_s) { return (double)n_used * N * K * (act == MOE_ACT_SWIGLU ? 4.0 : 2.0) * 1e-6 / tb_s; }
double narrow_us(const NarrowCost& c, int tiles_m, int n_used, int N, int K, int act, int cus) {
    const int cols = 32 * c.form.nt / (act == MOE_ACT_SWIGLU ? 2 : 1);
    const int tiles = tiles_m * ((N + cols - 1) / cols), last = tiles % cus;
    const double kb = 64e-3 * (c.form.mt + c.form.nt) * K;
    double cu = tiles / cus * (kb / c.gb_s + c.per_round);
    if (last > 0) cu += kb / (c.gb_s * (1.0 + c.alone * (1.0 - (double)last / cus))) + c.per_round;
    return c.start + norm4(cu, weights_us(n_used, N, K, act, c.tb_s), tiles * kb * 1e-3 / c.all_tb_s);
}
double skinny_us(int R, int n_used, int N, int K, int act, int cus) {
    const int rows = skinny_tile_rows(R), cols = SBN / (act == MOE_ACT_SWIGLU ? 2 : 1), ns = K / SKW;
    const int tiles = spread_tiles_m(R, rows, n_used, 2) * ((N + cols - 1) / cols);
    const SkinnyPlan p = plan_skinny(tiles, cus, ns);
    const double rounds = (tiles * p.parts + cus - 1) / cus, kb = (rows + SBN) * 2e-3 * SKW * p.per;
    if (rows == 32) return 4.88 + norm4(rounds * (kb / 69.6 - 0.82), weights_us(n_used, N, K, act, 6.41)) + (p.parts > 1 ? 1.69 + 0.28 * p.parts : 0.0);
    return 2.25 + norm4(rounds * (kb / 60.7 + 2.79), weights_us(n_used, N, K, act, 5.31)) + (p.parts > 1 ? 2.32 + 0.50 * p.parts : 0.0);
}
// other_tiles(way): tiles of rows of the kernel that would run otherwise; other_us(tiles): its time; tiles_m(mt, way): tiles of 32 mt rows.
// Host time counts in small shares (1 us of the call's 7): a time is worked out once per tile count, and the other four ways are
// played only for forms that come within 15 % of the best one.
template <typename OtherTiles, typename OtherUs, typename Tiles>
NarrowForm narrow_form(int n_used, int N, int K, int act, int cus, double gain, OtherTiles other_tiles, OtherUs other_us, Tiles tiles_m) {
    constexpr int FORMS = sizeof kNarrowForms / sizeof kNarrowForms[0];
    const int likely = n_used <= 1 ? 0 : 2, likely_tiles = other_tiles(likely);
    const double likely_us = other_us(likely_tiles);
    double us[FORMS];
    int best = -1;
    for (int f = 0; f < FORMS; ++f) {
        us[f] = narrow_us(kNarrowForms[f], tiles_m(kNarrowForms[f].form.mt, likely), n_used, N, K, act, cus);
        if (us[f] < (best < 0 ? likely_us : us[best])) best = f;
    }
    if (best < 0) return NarrowForm{0, 0};
    if (us[best] < 0.6 * likely_us || (n_used <= 1 && us[best] < gain * likely_us)) return kNarrowForms[best].form;
    if (n_used <= 1) return NarrowForm{0, 0};
    double others[5];
    for (int way = 0; way < 5; ++way) {
        const int t = other_tiles(way);
        others[way] = t == likely_tiles ? likely_us : other_us(t);
    }
    const double near = 1.15 * us[best];
    best = -1;
    double best_q = gain;
    for (int f = 0; f < FORMS; ++f) {
        if (us[f] > near) continue;
        const NarrowCost& c = kNarrowForms[f];
        double q = 0.0;
        for (int way = 0; way < 5; ++way) {
            const int t = tiles_m(c.form.mt, way);
            q += 0.2 * (t == tiles_m(c.form.mt, likely) ? us[f] : narrow_us(c, t, n_used, N, K, act, cus)) / others[way];
        }
        if (q < best_q) { best = f; best_q = q; }
    }
    return best < 0 ? NarrowForm{0, 0} : kNarrowForms[best].form;
}
// both GEMMs of a share that would take `rows` rows per tile otherwise (of the streaming kernels up to kSkinnyRows rows)
void take_narrow_forms(int R, int n_used, int H, int F, int act, int cus, const int (&rows)[2], NarrowForm (&form)[2]) {
    int counted[5][5] = {};                              // [mt][way]
    auto tiles_m = [&](int mt, int way) {
        int& t = counted[mt][way];
        if (t == 0) t = spread_tiles_m(R, 32 * mt, n_used, way);
        return t;
    };
    const bool streaming = R <= kSkinnyRows;
    for (int g = 0; g < 2; ++g) {
        const int N = g == 0 ? F : H, K = g == 0 ? H : F, a = g == 0 ? act : -1;
        const TileShape t = rows[g] == kShapeRows[TS_128] ? TS_128 : rows[g] == kShapeRows[TS_192] ? TS_192 : TS_256;
        auto other_tiles = [&](int way) { return streaming ? 0 : t == TS_128 ? tiles_m(4, way) : spread_tiles_m(R, rows[g], n_used, way); };
        auto other_us = [&](int tiles) {
            if (streaming) return skinny_us(R, n_used, N, K, a, cus);
            return std::max(1.0, 1.068 * played_us(t, tiles, R, n_used, N, K, a, cus) - 4.88);
        };
        form[g] = narrow_form(n_used, N, K, a, cus, streaming ? kNarrowGainStreaming : kNarrowGain, other_tiles, other_us, tiles_m);
    }
}
// the same, unless their maps do not fit; rows: then theirs
void take_narrow(int R, int n_used, int nseg, int H, int F, int act, int cus, int (&rows)[2], NarrowForm (&form)[2]) {
    form[0] = form[1] = NarrowForm{0, 0};
    if (R > 128 * n_used) return;
    take_narrow_forms(R, n_used, H, F, act, cus, rows, form);
    const int new_rows[2] = {form[0].mt ? 32 * form[0].mt : rows[0], form[1].mt ? 32 * form[1].mt : rows[1]};
    if (!maps_fit(R, nseg, new_rows[0], new_rows[1])) { form[0] = form[1] = NarrowForm{0, 0}; return; }
    rows[0] = new_rows[0];
    rows[1] = new_rows[1];
}

template <int EPI, int MT, int NT, bool ONE>
int launch_bf16_narrow_one(const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                          void* C, int ldc, int R, int nseg, int n_used, const SegList& one, hipStream_t st) {
    using G = NarrowGeom<MT, NT>;
    const int nout = (EPI == EPI_SWIGLU) ? G::BN_ / 2 : G::BN_;
    const int tiles_n = (N + nout - 1) / nout;
    static bool attr_done = false;
    if (!attr_done) {
        MOE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_narrow_kernel<EPI, MT, NT, ONE>), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS));
        attr_done = true;
    }
    const int tiles_m = std::min(max_tiles_of(R, G::BM_, nseg), (R + n_used * (G::BM_ - 1)) / G::BM_);
    hipLaunchKernelGGL((gemm_bf16_narrow_kernel<EPI, MT, NT, ONE>), ONE ? dim3(tiles_n, tiles_m) : dim3(tiles_m * tiles_n), dim3(64 * G::WAVES), G::LDS, st,
                       reinterpret_cast<const uint16_t*>(A), lda, m, tab, which0, which1, N, K, reinterpret_cast<uint16_t*>(C), ldc, tiles_n, OneSegment{one.offset, one.expert, one.R, one.n_local});
    MOE_LAUNCH_CHECK("gemm_bf16_narrow_kernel");
    return MOE_OK;
}
template <int EPI, int MT, int NT>
int launch_bf16_narrow_nt(const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                          void* C, int ldc, int R, int nseg, int n_used, const SegList& one, hipStream_t st) {
    return one.offset ? launch_bf16_narrow_one<EPI, MT, NT, true>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, n_used, one, st)
                      : launch_bf16_narrow_one<EPI, MT, NT, false>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, n_used, one, st);
}
template <int EPI>
int launch_bf16_narrow(NarrowForm f, const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                       void* C, int ldc, int R, int nseg, int n_used, const SegList& one, hipStream_t st) {
#define MOE_NARROW(a, b) if (f.mt == a && f.nt == b) return launch_bf16_narrow_nt<EPI, a, b>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, n_used, one, st)
    MOE_NARROW(4, 2); MOE_NARROW(2, 2); MOE_NARROW(2, 1); MOE_NARROW(1, 2); MOE_NARROW(1, 1);
#undef MOE_NARROW
    return moe_set_error(MOE_EINTERNAL, "no narrow tiles of %d x %d", f.mt, f.nt);
}
template <int EPI>
int launch_bf16_skinny(const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                       void* C, int ldc, int R, int nseg, float* partial, hipStream_t st) {
    if (skinny_tile_rows(R) == 32) return launch_bf16_skinny_mt<EPI, 1>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, partial, st);
    return launch_bf16_skinny_mt<EPI, 2>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, partial, st);
}

// Tiles of gemm_f32_parts_kernel that a block walks through (see kWalkUs).
int parts_walk_tiles(int K) { return std::max(1, (int)(kWalkUs / (5.1 + 1.23 * ((K + XK - 1) / XK)))); }
// Which kernels an fp32 share takes: the 64 x 64 tiles of gemm_f32_kernel keep more CUs busy where there are few tiles and
// need no map by a launch of its own, the 128 x 128 ones of gemm_f32_parts_kernel have the higher rate.  The times of both are modelled
// from the number of tiles, of which the host knows one for every n_used runs of rows only roughly (half a tile of padding
// per run, 0.29 sqrt(n_used) of them standard deviation): the older kernel is given two deviations on its side, the other
// one two against it, and 3 % besides, each GEMM by itself and both together with the map.  The constants (us) are fitted to 260
// shares of 150 to 20000 rows, 1 to 8 experts, H of 128 to 1024 and F of 128 to 2816, all four combinations of kernels one
// after the other without a pause (median error 2.3 %, 19 of 20 within 7.4 %): a third of the shares takes 128 x 128 tiles and is 1.18
// times faster.  Over 120 shares that were not fitted none with 128 x 128 tiles is slower than without.
double f32_us(bool in_parts, int R, int n_used, int N, int K, int act, int cus) {
    const int side = in_parts ? XM : FM, cols = side / (act == MOE_ACT_SWIGLU ? 2 : 1);
    double tiles_m = (R + side - 1) / side;
    if (n_used > 1) tiles_m = std::max((double)n_used, (double)R / side + 0.5 * n_used + (in_parts ? 0.58 : -0.58) * std::sqrt((double)n_used));
    const double per_cu = tiles_m * ((N + cols - 1) / cols) / cus, rounds = std::ceil(per_cu);
    const int nk = in_parts ? ((K + XK - 1) / XK + 1) / 2 * 2 : (K + FK - 1) / FK;
    if (in_parts) return 3.75 + rounds * (5.96 + 0.932 * nk) + per_cu * (0.299 * nk - 0.905);
    return 5.0 + rounds * (0.504 + 0.505 * nk);
}
constexpr double kF32MapUs = 1.8, kF32Gain = 0.97;
// Without room for two maps the small tiles, unless the large ones win for both.
void take_f32_kernels(int R, int n_used, int nseg, int H, int F, int act, int cus, bool (&in_parts)[2]) {
    double older = 0.0, taken = kF32MapUs;
    for (int g = 0; g < 2; ++g) {
        const int N = g == 0 ? F : H, K = g == 0 ? H : F, a = g == 0 ? act : -1;
        const double small = f32_us(false, R, n_used, N, K, a, cus), large = f32_us(true, R, n_used, N, K, a, cus);
        in_parts[g] = K >= kXMinK && large < kF32Gain * small;
        older += small;
        taken += in_parts[g] ? large : small;
    }
    if (taken >= kF32Gain * older || (in_parts[0] != in_parts[1] && !maps_fit(R, nseg, FM, XM))) in_parts[0] = in_parts[1] = false;
}
// Shares that take gemm_f32_kernel twice work their tiles out from the segment list (see SegList) up to this many tiles of both GEMMs
// per CU: the launch of the map, 1.5 us, is saved once, working a tile out costs every block.  1200 tiles on 256 CUs 1.02 to 1.07
// times faster, 2000 0.97 to 1.06, 4000 0.93 to 0.95, 9000 (20480 rows of 64 -> 1600 -> 64) 0.92.
constexpr int kListTiles = 5;
bool f32_needs_map(int R, int n_used, int nseg, int H, int F, int act, int cus, const bool (&in_parts)[2]) {
    if (nseg > kSmallMapSegs || in_parts[0] || in_parts[1]) return true;
    const int cols = act == MOE_ACT_SWIGLU ? FN / 2 : FN;
    const int64_t tiles_m = std::min<int64_t>(max_tiles_of(R, FM, nseg), (R + (int64_t)n_used * (FM - 1)) / FM);
    return tiles_m * ((F + cols - 1) / cols + (H + FN - 1) / FN) > (int64_t)kListTiles * cus;
}
// Whether most of the tile counts that n_used runs of R rows can have (the device knows which it is) leave tiles that are cut.
bool cuts_parts(int R, int n_used, int N, int K, int act, int cus) {
    const int cols = act == MOE_ACT_SWIGLU ? XN / 2 : XN, tiles_n = (N + cols - 1) / cols, nk = ((K + XK - 1) / XK + 1) & ~1;
    const int lo = (R + XM - 1) / XM, hi = std::max(lo, (int)std::min<int64_t>(R, (R + (int64_t)n_used * (XM - 1)) / XM));
    int cut = 0;
    for (int t = lo; t <= hi; ++t) cut += plan_parts(t * tiles_n, cus, nk).n_cut > 0 ? 1 : -1;
    return cut >= 0;
}
// The GEMMs of a share whose tiles may be cut; the counters of the pieces lie behind the tile maps.
void take_cuts(int R, int n_used, int nseg, int H, int F, int act, int cus, const bool (&in_parts)[2], bool (&cuts)[2]) {
    const bool fit = maps_fit(R, nseg, in_parts[0] ? XM : FM, in_parts[1] ? XM : FM);
    cuts[0] = fit && in_parts[0] && cuts_parts(R, n_used, F, H, act, cus);
    cuts[1] = fit && in_parts[1] && cuts_parts(R, n_used, H, F, -1, cus);
}
// What is launched for up to max_items tiles; pieces of a last round take one round more at most.
int parts_blocks(int max_items, int walk, int ncu, bool may_cut) { return walk_blocks(max_items + (may_cut ? ncu : 0), walk, ncu); }
template <int EPI>
int launch_f32_parts(const void* A, int lda, const TileMap& m, const ExpertTable& tab, int which0, int which1, int N, int K,
                     void* C, int ldc, int R, int nseg, float* partial, hipStream_t st) {
    const int nout = (EPI == EPI_SWIGLU) ? XN / 2 : XN;
    const int tiles_n = (N + nout - 1) / nout, ncu = round_size(), walk = parts_walk_tiles(K);
    auto launch = [&](auto kernel, bool& attr_done) -> int {
        if (!attr_done) {
            MOE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kXLds));
            attr_done = true;
        }
        hipLaunchKernelGGL(kernel, dim3(parts_blocks(max_tiles_of(R, XM, nseg) * tiles_n, walk, ncu, partial != nullptr)), dim3(512), kXLds, st,
                           reinterpret_cast<const float*>(A), lda, m, tab, which0, which1, N, K, reinterpret_cast<float*>(C), ldc, tiles_n, ncu, walk, partial);
        return MOE_OK;
    };
    static bool attr_cut = false, attr_whole = false;
    const int rc = partial ? launch(gemm_f32_parts_kernel<EPI, true>, attr_cut) : launch(gemm_f32_parts_kernel<EPI, false>, attr_whole);
    if (rc != MOE_OK) return rc;
    MOE_LAUNCH_CHECK("gemm_f32_parts_kernel");
    return MOE_OK;
}

template <int EPI>
int launch_f32(bool in_parts, bool need_map, const void* A, int lda, const TileMap& m, SegList seg, const ExpertTable& tab, int which0, int which1,
               int N, int K, void* C, int ldc, int R, int nseg, int n_used, float* partial, hipStream_t st) {
    if (in_parts) return launch_f32_parts<EPI>(A, lda, m, tab, which0, which1, N, K, C, ldc, R, nseg, partial, st);
    const int nout = (EPI == EPI_SWIGLU) ? FN / 2 : FN;
    const int tiles_n = (N + nout - 1) / nout;
    seg.max_tiles = max_tiles_of(R, FM, nseg);
    auto launch = [&](auto kernel, int tiles_m) {
        hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(256), 0, st,
                           reinterpret_cast<const float*>(A), lda, m, seg, tab, which0, which1, N, K, reinterpret_cast<float*>(C), ldc, tiles_n);
    };
    if (need_map) launch(gemm_f32_kernel<EPI, false>, seg.max_tiles);
    else launch(gemm_f32_kernel<EPI, true>, std::min(seg.max_tiles, (R + n_used * (FM - 1)) / FM));
    MOE_LAUNCH_CHECK("gemm_f32_kernel");
    return MOE_OK;
}

// Which shares take ffn_small_kernel: those whose weights a block fetches in about the time of the launches that are saved.  The figures are
// one call with its map and two GEMMs over one call in one kernel, called again and again / with the caches flushed before each call.
// - Up to one block per CU: 192 KB of weights per expert in bf16, 128 KB in fp32, whose products take longer.  bf16 192 KB SwiGLU
//   1.10 to 1.29 / 1.10 to 1.25, GELU 1.11 to 1.34 (256 KB 0.90 to 1.14); fp32 128 KB 1.10 to 1.44 / 0.98 to 1.37 (192 KB 0.92 to 1.4).
// - bf16 with at most kSmallFewRows rows per expert, where narrow tiles of few weight rows spread the weights over more CUs: 128 KB
//   (1.16 to 1.45 / 0.95 to 1.19; 192 KB 0.91 to 1.25 / 0.72 to 0.98), and 64 KB for a list of one segment, which needs no map there
//   (1.16 to 1.30 / 1.06 to 1.26; 96 KB 1.00 to 1.09 / 0.86 to 1.04, 192 KB 0.61 to 0.77 / 0.54 to 0.66).
// - A second block per CU fetches the weights again, and its rows are then a good part of what it moves: weights, rows and outputs
//   together at most 144 KB in bf16, 160 KB in fp32.  bf16 128 -> 256 (144 KB) 1.02 to 1.13 / 1.16 to 1.28, 256 -> 128 (160 KB) 0.91 to
//   1.03, SwiGLU of 128 -> 128 (112 KB) 1.18 to 1.31, of 256 -> 128 (224 KB) 0.71 to 0.80; fp32 128 -> 128 (160 KB) 1.06 to 1.14, SwiGLU of
//   64 -> 192 (160 KB) 1.12 to 1.21, 256 -> 64 (192 KB) 0.85 to 1.02.  With a third one 96 KB of bf16 are at 0.80.
constexpr int kSmallBytesBf16 = 192 << 10, kSmallBytesF32 = 128 << 10;
constexpr int kSmallFewRows = 128, kSmallFewBytes = 128 << 10, kSmallOneSegmentBytes = 64 << 10;
constexpr int kSmallMovedBf16 = 144 << 10, kSmallMovedF32 = 160 << 10, kSmallPerCU = 2;
bool takes_small(int R, int n_used, int nseg, int H, int F, int act, int dtype, int cus) {
    const int es = elem_size(dtype), mats = act == MOE_ACT_SWIGLU ? 3 : 2;
    if (nseg > kSmallMapSegs || (int64_t)H * es % (64 * kSmallSteps) != 0 || (int64_t)F * es % (64 * kSmallSteps) != 0) return false;
    const bool bf16 = dtype == MOE_BF16, few = bf16 && R <= (int64_t)kSmallFewRows * n_used;
    const double weights = (double)mats * H * F * es, rows = 2.0 * kSmallRows * H * es;   // bytes
    if (weights > (!bf16 ? kSmallBytesF32 : !few ? kSmallBytesBf16 : nseg == 1 ? kSmallOneSegmentBytes : kSmallFewBytes)) return false;
    const int64_t tile_rows = R + (int64_t)n_used * (kSmallRows - 1), round = (int64_t)cus * kSmallRows;
    return tile_rows <= round || (tile_rows <= kSmallPerCU * round && weights + rows <= (bf16 ? kSmallMovedBf16 : kSmallMovedF32));
}
// whether two arrays of `bytes` have a byte in common
bool share_memory(const void* a, const void* b, size_t bytes) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y ? y - x < bytes : x - y < bytes;
}
template <int DT, int EPI>
int launch_small(const void* x, const ExpertTable& tab, SegList seg, int R, int n_used, int H, int F, void* out, hipStream_t st) {
    seg.max_tiles = max_tiles_of(R, kSmallRows, seg.nseg);
    const int tiles = std::min<int64_t>(seg.max_tiles, (R + (int64_t)n_used * (kSmallRows - 1)) / kSmallRows);
    hipLaunchKernelGGL((ffn_small_kernel<DT, EPI>), dim3(tiles), dim3(256), kSmallRows * (F * (DT == MOE_BF16 ? 2 : 4) + 16), st,
                       reinterpret_cast<const char*>(x), seg, tab, H, F, reinterpret_cast<char*>(out));
    MOE_LAUNCH_CHECK("ffn_small_kernel");
    return MOE_OK;
}

}  // namespace

// Host-side self check of the tile numbering and of the tail plan for a tiles_m x tiles_n grid with nk k-tiles
// (not part of the published interface; used by the CPU tests): every tile is produced exactly once, whole
// or as `parts` pieces that cover its k-tiles exactly once.
extern "C" int moe_selfcheck_tile_order(int32_t tiles_m, int32_t tiles_n, int32_t ncu, int32_t nk) {
    if (tiles_m < 1 || tiles_n < 1 || ncu < 1 || nk < 2 || (nk & 1)) return moe_set_error(MOE_EINVAL, "moe_selfcheck_tile_order: bad argument");
    const int total = tiles_m * tiles_n;
    const Strips numberings[2] = {Strips{0, 0}, plan_strips(tiles_m, tiles_n)};   // fp32, bf16
    for (const Strips& strips : numberings) {
        std::vector<int> seen((size_t)total, 0);
        for (int id = 0; id < total; ++id) {
            int tm = -1, tn = -1;
            tile_of_block(id, total, tiles_m, tiles_n, strips, &tm, &tn);
            if (tm < 0 || tm >= tiles_m || tn < 0 || tn >= tiles_n) return moe_set_error(MOE_EINTERNAL, "tile %d maps outside the grid", id);
            if (seen[(size_t)tm * tiles_n + tn]++) return moe_set_error(MOE_EINTERNAL, "tile (%d, %d) is produced twice", tm, tn);
        }
    }
    const TailPlan p = plan_tail(total, ncu, nk);
    if (p.n_full + p.n_tail != total || p.n_full % ncu != 0 && p.n_tail != 0) return moe_set_error(MOE_EINTERNAL, "tail plan does not partition the tiles");
    if (p.n_tail * p.parts > ncu && p.parts > 1) return moe_set_error(MOE_EINTERNAL, "more pieces than CUs");
    if (p.parts > 1) {
        int covered = 0;
        for (int piece = 0; piece < p.parts; ++piece) {
            const int lo = piece * p.pairs_per * 2, n = std::min(p.pairs_per * 2, nk - lo);
            if (lo != covered || n < 4) return moe_set_error(MOE_EINTERNAL, "pieces do not tile the k range by four k-tiles at least");
            covered += n;
        }
        if (covered != nk) return moe_set_error(MOE_EINTERNAL, "pieces do not cover the k range");
    }
    return p.parts;
}

extern "C" int moe_selfcheck_tile_shape(int32_t R, int32_t n_used, int32_t N, int32_t K, int32_t act, int32_t ncu) {
    if (R < 1 || n_used < 1 || N < 1 || K < 64 || K % 64 != 0 || ncu < 1) return moe_set_error(MOE_EINVAL, "moe_selfcheck_tile_shape: bad argument");
    return kShapeRows[choose_shape(R, n_used, N, K, act, ncu)];
}

extern "C" int moe_selfcheck_tile_shapes(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t ncu, int32_t* rows2) {
    if (R < 1 || n_used < 1 || nseg < n_used || nseg > kMaxSeg || H < 64 || H % 64 != 0 || F < 64 || F % 64 != 0 || act < 0 || act > 2 || ncu < 1 || !rows2)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_tile_shapes: bad argument");
    if (R <= kSkinnyRows) {
        rows2[0] = rows2[1] = skinny_tile_rows(R);
    } else {
        TileShape shape[2];
        take_shapes(R, n_used, nseg, H, F, act, ncu, shape);
        for (int i = 0; i < 2; ++i) rows2[i] = kShapeRows[shape[i]];
    }
    if (!maps_fit(R, nseg, rows2[0], rows2[1])) return moe_set_error(MOE_EINTERNAL, "tile maps of %d and %d rows leave no room for the counters", rows2[0], rows2[1]);
    return MOE_OK;
}

// 1: the share takes the kernel of both GEMMs at once
extern "C" int moe_selfcheck_small(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t dtype, int32_t ncu) {
    if (R < 1 || n_used < 1 || nseg < n_used || H < 1 || F < 1 || act < 0 || act > 2 || (dtype != MOE_F32 && dtype != MOE_BF16) || ncu < 1)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_small: bad argument");
    return takes_small(R, n_used, nseg, H, F, act, dtype, ncu) ? 1 : 0;
}

// 1: the loads of a pair of k-tiles go out together as soon as its stages are free
extern "C" int moe_selfcheck_early_loads(int32_t rows, int32_t K) {
    for (const TileShape t : {TS_128, TS_192, TS_256})
        if (kShapeRows[t] == rows && K > 0) return loads_soon(t, K) ? 1 : 0;
    return moe_set_error(MOE_EINVAL, "moe_selfcheck_early_loads: bad argument");
}

// strips2: 1 where a GEMM that takes tiles of rows2 rows (see moe_selfcheck_tile_shapes) may be numbered in strips
extern "C" int moe_selfcheck_strips(int32_t R, int32_t n_used, int32_t H, int32_t F, int32_t act, const int32_t* rows2, int32_t* strips2) {
    if (R < 1 || n_used < 1 || H < 64 || F < 64 || act < 0 || act > 2 || !rows2 || !strips2) return moe_set_error(MOE_EINVAL, "moe_selfcheck_strips: bad argument");
    for (int g = 0; g < 2; ++g) {
        if (rows2[g] != 128 && rows2[g] != 192 && rows2[g] != 256) return moe_set_error(MOE_EINVAL, "moe_selfcheck_strips: no tiles of %d rows", rows2[g]);
        const int tiles_n = tiled_columns(g == 0 ? F : H, g == 0 && act == MOE_ACT_SWIGLU, rows2[g] == 128 ? TileGeom<2, 2>::BN : TileGeom<4, 4>::BN);
        strips2[g] = columns_in_strips(R, rows2[g], n_used, tiles_n, g == 0 ? H : F) > 0;
    }
    return MOE_OK;
}

extern "C" int moe_selfcheck_narrow(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t ncu, int32_t* forms2) {
    if (R < 1 || n_used < 1 || nseg < n_used || nseg > kMaxSeg || H < 128 || H % 128 != 0 || F < 128 || F % 128 != 0 || act < 0 || act > 2 || ncu < 1 || !forms2)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_narrow: bad argument");
    int32_t rows2[2];
    const int rc = moe_selfcheck_tile_shapes(R, n_used, nseg, H, F, act, ncu, rows2);
    if (rc != MOE_OK) return rc;
    int rows[2] = {rows2[0], rows2[1]};
    NarrowForm form[2];
    take_narrow(R, n_used, nseg, H, F, act, ncu, rows, form);
    for (int i = 0; i < 2; ++i) forms2[i] = 10 * form[i].mt + form[i].nt;
    if (!maps_fit(R, nseg, rows[0], rows[1])) return moe_set_error(MOE_EINTERNAL, "no room for tile maps of %d and %d rows", rows[0], rows[1]);
    return MOE_OK;
}

extern "C" int moe_selfcheck_f32_kernels(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t ncu, int32_t* rows2) {
    if (R < 1 || n_used < 1 || nseg < n_used || nseg > kMaxSeg || H < 4 || H % 4 != 0 || F < 4 || F % 4 != 0 || act < 0 || act > 2 || ncu < 1 || !rows2)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_f32_kernels: bad argument");
    bool in_parts[2];
    take_f32_kernels(R, n_used, nseg, H, F, act, ncu, in_parts);
    for (int i = 0; i < 2; ++i) rows2[i] = in_parts[i] ? XM : FM;
    if (rows2[0] != rows2[1] && !maps_fit(R, nseg, rows2[0], rows2[1])) return moe_set_error(MOE_EINTERNAL, "no room for tile maps of %d and %d rows", rows2[0], rows2[1]);
    return MOE_OK;
}

extern "C" int moe_selfcheck_f32_map(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t ncu) {
    int32_t rows2[2];
    const int rc = moe_selfcheck_f32_kernels(R, n_used, nseg, H, F, act, ncu, rows2);
    if (rc != MOE_OK) return rc;
    const bool in_parts[2] = {rows2[0] == XM, rows2[1] == XM};
    return f32_needs_map(R, n_used, nseg, H, F, act, ncu, in_parts) ? 1 : 0;
}

extern "C" int moe_selfcheck_f32_cuts(int32_t R, int32_t n_used, int32_t nseg, int32_t H, int32_t F, int32_t act, int32_t ncu, int32_t tiles_m, int32_t* parts2) {
    int32_t rows2[2];
    const int rc = moe_selfcheck_f32_kernels(R, n_used, nseg, H, F, act, ncu, rows2);
    if (rc != MOE_OK) return rc;
    if (tiles_m < 0 || !parts2) return moe_set_error(MOE_EINVAL, "moe_selfcheck_f32_cuts: bad argument");
    const bool in_parts[2] = {rows2[0] == XM, rows2[1] == XM};
    bool cuts[2];
    take_cuts(R, n_used, nseg, H, F, act, ncu, in_parts, cuts);
    for (int g = 0; g < 2; ++g) {
        const int N = g == 0 ? F : H, K = g == 0 ? H : F, cols = g == 0 && act == MOE_ACT_SWIGLU ? XN / 2 : XN;
        parts2[g] = cuts[g] ? plan_parts(tiles_m * ((N + cols - 1) / cols), ncu, ((K + XK - 1) / XK + 1) & ~1).parts : 0;
    }
    return MOE_OK;
}

extern "C" int moe_selfcheck_f32_walk(int32_t tiles_m, int32_t max_tiles_m, int32_t tiles_n, int32_t K, int32_t ncu) {
    if (tiles_m < 0 || max_tiles_m < std::max(tiles_m, 1) || tiles_n < 1 || K < kXMinK || K % 4 != 0 || ncu < 1)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_f32_walk: bad argument");
    const int walk = parts_walk_tiles(K), total = tiles_m * tiles_n, nk = ((K + XK - 1) / XK + 1) / 2 * 2;
    const PartsCut cuts[2] = {PartsCut{total, 0, 1, nk}, plan_parts(total, ncu, nk)};
    for (int may_cut = 0; may_cut < 2; ++may_cut) {       // either instantiation, by the grid that it is launched with
        const PartsCut& c = cuts[may_cut];
        const int n_items = c.n_full + c.n_cut * c.parts;
        std::vector<int> seen((size_t)n_items, 0);
        for (int b = 0; b < parts_blocks(max_tiles_m * tiles_n, walk, ncu, may_cut != 0); ++b) {
            const WalkRun run = walk_run(b, ncu, walk, n_items);
            int taken = 0;
            for (int item = run.item; item < run.end; item += ncu, ++taken) {
                if (item >= n_items || taken == walk) return moe_set_error(MOE_EINTERNAL, "run of block %d", b);
                if (item >= c.n_full && c.n_cut > 0 && item + ncu < run.end) return moe_set_error(MOE_EINTERNAL, "piece %d is not the last item of block %d", item, b);
                ++seen[item];
            }
        }
        for (int i = 0; i < n_items; ++i)
            if (seen[i] != 1) return moe_set_error(MOE_EINTERNAL, "item %d is taken %d times", i, seen[i]);
        if (c.n_cut == 0) continue;
        if (c.n_full + c.n_cut != total || c.n_cut * c.parts > ncu)
            return moe_set_error(MOE_EINTERNAL, "%d pieces of %d tiles", c.parts, c.n_cut);
        if (c.parts < 2 || c.per % 2 != 0 || c.per < kXCutMin || c.parts * c.per < nk || (c.parts - 1) * c.per >= nk)
            return moe_set_error(MOE_EINTERNAL, "%d pieces of %d k-tiles for %d", c.parts, c.per, nk);
    }
    return walk;
}

extern "C" int moe_selfcheck_walk(int32_t rows, int32_t tiles_m, int32_t max_tiles_m, int32_t tiles_n, int32_t K, int32_t ncu) {
    if ((rows != 128 && rows != 192 && rows != 256) || tiles_m < 1 || max_tiles_m < tiles_m || tiles_n < 1 || K < 64 || K % 64 != 0 || ncu < 1)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_walk: bad argument");
    const int slots = rows == 128 ? 2 * ncu : ncu, walk = walk_tiles(rows, K);
    const TailPlan p = plan_tail(tiles_m * tiles_n, slots, K / BK);
    const int n_items = p.n_full + (p.parts > 1 ? p.n_tail * p.parts : 0);
    std::vector<int> seen((size_t)n_items, 0);
    const int blocks = walk_blocks(max_tiles_m * tiles_n + slots, walk, slots);
    for (int b = 0; b < blocks; ++b) {
        const WalkRun run = walk_run(b, slots, walk, n_items);
        for (int item = run.item; item < run.end; item += slots) {
            if (item >= n_items || (run.end - run.item + slots - 1) / slots > walk) return moe_set_error(MOE_EINTERNAL, "run of block %d", b);
            ++seen[item];
            // a block stops behind a piece
            if (item >= p.n_full && item + slots < run.end) return moe_set_error(MOE_EINTERNAL, "piece %d is not the last item of block %d", item, b);
        }
    }
    for (int i = 0; i < n_items; ++i)
        if (seen[i] != 1) return moe_set_error(MOE_EINTERNAL, "item %d is taken %d times", i, seen[i]);
    return walk;
}

extern "C" int moe_selfcheck_skinny_plan(int32_t total, int32_t ncu, int32_t ns) {
    if (total < 1 || ncu < 1 || ns < 1) return moe_set_error(MOE_EINVAL, "moe_selfcheck_skinny_plan: total, ncu and ns must be positive");
    const SkinnyPlan p = plan_skinny(total, ncu, ns);
    // every stage in exactly one piece, no empty piece, no more blocks than max(total, ncu), pieces of at least 4 stages
    if (p.parts < 1 || p.per < 1 || (int64_t)p.parts * p.per < ns || (int64_t)(p.parts - 1) * p.per >= ns)
        return moe_set_error(MOE_EINTERNAL, "skinny plan: %d pieces of %d stages do not cover %d stages once", p.parts, p.per, ns);
    if ((int64_t)total * p.parts > std::max(total, ncu))
        return moe_set_error(MOE_EINTERNAL, "skinny plan: %d tiles x %d pieces exceed the launch", total, p.parts);
    if (p.parts > 1 && (p.per < 4 || total >= ncu)) return moe_set_error(MOE_EINTERNAL, "skinny plan: pieces too short or not needed");
    return p.parts;
}

// A tile map on the host, and whether it is the one that the segment list asks for.
struct MapArrays {
    std::vector<int32_t> row0, nrows, expert, gather, rel;
    int32_t n_tiles;
    TileMap m;
    explicit MapArrays(int nt) : row0(nt), nrows(nt), expert(nt), gather(nt), rel((size_t)nt * kRelPitch, -1), n_tiles(nt) {
        m = TileMap{&n_tiles, row0.data(), nrows.data(), expert.data(), gather.data(), rel.data(), nullptr};
    }
    bool enter(size_t at, int32_t value) {
        if (at >= rel.size() || rel[at] != -1) {
            (void)moe_set_error(MOE_EINTERNAL, "offset table entry %zu is outside the table or written twice", at);
            return false;
        }
        rel[at] = value;
        return true;
    }
};
static int check_map(const MapArrays& map, int nt, const int32_t* seg_offset, const int32_t* seg_expert, int nseg, int R, int bm, int n_local, int gather) {
    const TileMap& m = map.m;
    std::vector<int> owner((size_t)R, -1);
    for (int i = 0; i < nseg; ++i) {
        const int lo = std::max(seg_offset[i], 0), hi = std::min(seg_offset[i + 1], R);
        if (hi > lo && seg_expert[i] >= 0 && seg_expert[i] < n_local)
            for (int r = lo; r < hi; ++r) owner[r] = seg_expert[i];
    }
    std::vector<int> hits((size_t)R, 0);
    for (int t = 0; t < nt; ++t) {
        if (m.nrows[t] < 1 || m.nrows[t] > bm) return moe_set_error(MOE_EINTERNAL, "tile %d has %d rows", t, m.nrows[t]);
        if (m.gather[t] && !gather) return moe_set_error(MOE_EINTERNAL, "tile %d is gathered but gathering is off", t);
        int prev = -1;
        bool gaps = false;
        for (int r = 0; r < m.nrows[t]; ++r) {
            const int off = m.gather[t] ? m.rel[(size_t)t * kRelPitch + r] : r;
            if (!m.gather[t] && m.rel[(size_t)t * kRelPitch + r] != -1) return moe_set_error(MOE_EINTERNAL, "tile %d has no gaps but an offset table", t);
            const int row = m.row0[t] + off;
            if (off < 0 || row < 0 || row >= R) return moe_set_error(MOE_EINTERNAL, "tile %d row %d maps to %d", t, r, row);
            if (r == 0 && off != 0) return moe_set_error(MOE_EINTERNAL, "tile %d does not start at its first row", t);
            if (row <= prev) return moe_set_error(MOE_EINTERNAL, "tile %d: rows do not increase", t);
            if (prev >= 0 && row != prev + 1) gaps = true;
            if (owner[row] != m.expert[t]) return moe_set_error(MOE_EINTERNAL, "tile %d of expert %d holds row %d of expert %d", t, m.expert[t], row, owner[row]);
            ++hits[row];
            prev = row;
        }
        if (gaps != (m.gather[t] != 0)) return moe_set_error(MOE_EINTERNAL, "tile %d: gather flag %d but gaps %d", t, m.gather[t], (int)gaps);
    }
    for (int r = 0; r < R; ++r)
        if (hits[r] != (owner[r] >= 0 ? 1 : 0)) return moe_set_error(MOE_EINTERNAL, "row %d is in %d tiles", r, hits[r]);
    return MOE_OK;
}

// Host-side self check of the tile map (not part of the published interface; used by the CPU tests): runs
// the steps that the device kernels run, on the host, and verifies that every row of every non-empty
// segment of a known expert lies in exactly one tile of that expert, that tile rows increase, that exactly
// the tiles with gaps are marked as gathered and that their offset tables are complete.  Returns the
// number of tiles, or a negative status.  Up to 64 segments the same goes for the map that such lists take.
extern "C" int moe_selfcheck_tile_map(const int32_t* seg_offset, const int32_t* seg_expert, int32_t nseg, int32_t R,
                                      int32_t bm, int32_t n_local, int32_t gather) {
    if (!seg_offset || !seg_expert || nseg < 0 || nseg > kMaxSeg || R < 0 || bm < 1 || bm > kRelPitch || n_local < 1 || n_local > MOE_MAX_LOCAL)
        return moe_set_error(MOE_EINVAL, "moe_selfcheck_tile_map: bad argument");
    std::vector<SegWork> store(1);
    SegWork& w = store[0];
    for (int i = 0; i <= nseg; ++i) w.raw_off[i] = seg_offset[i];
    for (int i = 0; i < nseg; ++i) w.raw_exp[i] = seg_expert[i];
    const int nth = 7;                                    // any thread count and order must give the same map
    for (int t = 0; t < nth; ++t) tilemap_clean(w, nseg, R, n_local, t, nth);
    if (gather) {
        tilemap_rank_host(w, nseg);
        tilemap_starts_host(w, n_local);
        for (int t = nth - 1; t >= 0; --t) tilemap_place(w, nseg, R, t, nth);
    } else {
        tilemap_merge(w, nseg, R);
    }
    tilemap_groups_host(w, bm, gather != 0);
    const int max_tiles = max_tiles_of(R, bm, nseg), nt = w.n_tiles;
    if (nt > max_tiles) return moe_set_error(MOE_EINTERNAL, "%d tiles exceed the bound %d", nt, max_tiles);
    MapArrays map(nt);
    for (int t = nt - 1; t >= 0; --t) tilemap_tile(w, t, bm, map.m);
    if (gather)
        for (int k = 0; k < w.n_items; ++k) {
            RelJob job[2];
            tilemap_rel_jobs(w, k, bm, nt, job);
            for (int pass = 0; pass < 2; ++pass)
                for (int r = 0; r < job[pass].cnt; ++r)
                    if (!map.enter((size_t)job[pass].dst + r, job[pass].val + r)) return MOE_EINTERNAL;
        }
    int rc = check_map(map, nt, seg_offset, seg_expert, nseg, R, bm, n_local, gather);
    if (rc != MOE_OK || nseg < 1 || nseg > kSmallMapSegs) return rc != MOE_OK ? rc : nt;
    // the map of up to 64 segments
    std::vector<ArrayLanes> lanes(1);
    ArrayLanes& l = lanes[0];
    for (int k = 0; k < 64; ++k) {
        const int i = std::min(k, nseg - 1);
        l.it[k].off0 = seg_offset[i];
        l.it[k].off1 = seg_offset[i + 1];
        l.it[k].e = seg_expert[i];
    }
    const SmallMap sm = small_map(l, nseg, R, n_local, gather, bm, max_tiles);
    // (without gathering an empty segment of no known expert ends a run above, but not here)
    if (sm.n_tiles > nt || (gather && sm.n_tiles != nt)) return moe_set_error(MOE_EINTERNAL, "%d tiles, and %d from the map of few segments", nt, sm.n_tiles);
    MapArrays small(sm.n_tiles);
    for (int t = 0; t < sm.n_tiles; ++t) {
        const SmallTile r = small_tile(l, sm, t, bm);
        small.m.row0[t] = r.row0;
        small.m.nrows[t] = r.nrows;
        small.m.expert[t] = r.expert;
        small.m.gather[t] = r.gather;
        if (!r.gather) continue;
        for (unsigned long long in = r.in; in; in &= in - 1) {
            const SmallRun run = small_run(l, r, __builtin_ctzll(in));
            for (int v = run.lo; v < run.hi; ++v)
                if (!small.enter((size_t)t * kRelPitch + v, run.val + v)) return MOE_EINTERNAL;
        }
    }
    rc = check_map(small, sm.n_tiles, seg_offset, seg_expert, nseg, R, bm, n_local, gather);
    return rc != MOE_OK ? rc : nt;
}

// without room for the pieces of cut tiles
static size_t least_workspace(int R, int F, int dtype) { return tilemap_bytes(R) + align256((size_t)R * F * elem_size(dtype)) + 256; }

extern "C" size_t moe_ffn_workspace_bytes(int32_t R_max, int32_t H, int32_t F, int32_t act, int32_t dtype) {
    if (R_max < 0 || H <= 0 || F <= 0 || act < 0 || act > 2 || (dtype != MOE_F32 && dtype != MOE_BF16)) return 0;
    const size_t partial = (dtype == MOE_BF16) ? (size_t)kMaxCU * TileGeom<4, 4>::PARTIAL : (size_t)kMaxCU * kXPiece;   // pieces of cut tiles
    return least_workspace(R_max, F, dtype) + partial;
}

// around the kernels: in front of the tile map, the first GEMM, the second, and behind it; at[1] and at[2] around one kernel of both GEMMs
struct FfnEvents { hipEvent_t at[4]; bool one_kernel; };
// timed_gemm: 0 none, 1 / 2: that GEMM runs as its TIMED instantiation and writes marks (bf16, more than 64 rows)
static int ffn_impl(const void* recv, int32_t R, const int32_t* seg_offset, const int32_t* seg_expert, int32_t nseg,
                    const moe_expert_w* experts, int32_t n_local, int32_t H, int32_t F, int32_t act, int32_t dtype,
                    void* out, void* workspace, size_t workspace_bytes, hipStream_t st, FfnEvents* ev,
                    int timed_gemm = 0, long long* marks = nullptr, size_t marks_len = 0) {
    if (!recv || !seg_offset || !seg_expert || !experts || !out || !workspace)
        return moe_set_error(MOE_EINVAL, "moe_expert_ffn: NULL argument");
    if (R < 0 || nseg < 0 || H <= 0 || F <= 0) return moe_set_error(MOE_EINVAL, "moe_expert_ffn: negative size");
    if (dtype != MOE_F32 && dtype != MOE_BF16) return moe_set_error(MOE_EDTYPE, "moe_expert_ffn: unknown dtype %d", dtype);
    if (act < 0 || act > 2) return moe_set_error(MOE_EDTYPE, "moe_expert_ffn: unknown act %d", act);
    if (n_local < 1 || n_local > MOE_MAX_LOCAL || nseg > kMaxSeg)
        return moe_set_error(MOE_ESHAPE, "moe_expert_ffn: need 1 <= n_local <= %d and nseg <= %d", MOE_MAX_LOCAL, kMaxSeg);
    if (dtype == MOE_BF16 && (H % 128 != 0 || F % 128 != 0))
        return moe_set_error(MOE_ESHAPE, "moe_expert_ffn: bf16 needs H and F to be multiples of 128");
    if (dtype == MOE_BF16 && (size_t)H * (size_t)F * 2 > 0xFFFFFFFFull)
        return moe_set_error(MOE_ESHAPE, "moe_expert_ffn: bf16 weight matrices are limited to 4 GiB each (32-bit lane offsets)");
    if (dtype == MOE_F32 && (H % 4 != 0 || F % 4 != 0))
        return moe_set_error(MOE_EALIGN, "moe_expert_ffn: fp32 needs H and F to be multiples of 4");
    if (!aligned16(recv) || !aligned16(out) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return moe_set_error(MOE_EALIGN, "moe_expert_ffn: recv/out need 16-byte, workspace 256-byte alignment");
    const bool pieces_fit = workspace_bytes >= moe_ffn_workspace_bytes(R, H, F, act, dtype);
    // (fp32 tiles are not cut in a workspace that was sized for the tile map and the intermediate alone)
    if (!pieces_fit && (dtype != MOE_F32 || workspace_bytes < least_workspace(R, F, dtype)))
        return moe_set_error(MOE_ESHAPE, "moe_expert_ffn: workspace too small (%zu < %zu)", workspace_bytes,
                             moe_ffn_workspace_bytes(R, H, F, act, dtype));
    ExpertTable tab;
    for (int e = 0; e < n_local; ++e) {
        if (!experts[e].w1 || !experts[e].w_down || (act == MOE_ACT_SWIGLU && !experts[e].w_up))
            return moe_set_error(MOE_EINVAL, "moe_expert_ffn: expert %d has a NULL weight", e);
        if (!aligned16(experts[e].w1) || !aligned16(experts[e].w_down) || !aligned16(experts[e].w_up))
            return moe_set_error(MOE_EALIGN, "moe_expert_ffn: expert %d weights must be 16-byte aligned", e);
        tab.w1[e] = experts[e].w1;
        tab.w_up[e] = experts[e].w_up;
        tab.w_down[e] = experts[e].w_down;
    }
    if (R == 0 || nseg == 0) {
        if (ev) for (int i = 0; i < 4; ++i) MOE_HIP(hipEventRecord(ev->at[i], st));
        return MOE_OK;
    }
    void* hmid = reinterpret_cast<char*>(workspace) + tilemap_bytes(R);
    float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(hmid) + align256((size_t)R * F * elem_size(dtype)));
    const bool skinny = dtype == MOE_BF16 && R <= kSkinnyRows;
    if (timed_gemm != 0 && (dtype != MOE_BF16 || skinny))
        return moe_set_error(MOE_ESHAPE, "moe_diag_ffn_phases: bf16 and more than %d rows needed", kSkinnyRows);
    // gathered tiles address their rows by 32-bit byte offsets from the tile's first row
    const int gather = (size_t)R * (size_t)std::max(H, F) * elem_size(dtype) <= 0xFFFFFFFFull ? 1 : 0;
    const int n_used = std::min(gather ? std::min(n_local, nseg) : nseg, R);   // runs of rows that share no tile
    // a block of the kernel of both GEMMs writes its rows of `out` while others still read theirs of `recv`; the GEMMs apart do not
    if (timed_gemm == 0 && !share_memory(recv, out, (size_t)R * H * elem_size(dtype)) && takes_small(R, n_used, nseg, H, F, act, dtype, round_size())) {
        const SegList list = {seg_offset, seg_expert, nseg, R, n_local, gather, 0};
        if (ev) MOE_HIP(hipEventRecord(ev->at[1], st));
        int rc;
#define MOE_SMALL(DT, EPI) launch_small<DT, EPI>(recv, tab, list, R, n_used, H, F, out, st)
        if (dtype == MOE_BF16) rc = act == MOE_ACT_SWIGLU ? MOE_SMALL(MOE_BF16, EPI_SWIGLU) : act == MOE_ACT_GELU_MLP ? MOE_SMALL(MOE_BF16, EPI_GELU) : MOE_SMALL(MOE_BF16, EPI_SILU);
        else rc = act == MOE_ACT_SWIGLU ? MOE_SMALL(MOE_F32, EPI_SWIGLU) : act == MOE_ACT_GELU_MLP ? MOE_SMALL(MOE_F32, EPI_GELU) : MOE_SMALL(MOE_F32, EPI_SILU);
#undef MOE_SMALL
        if (rc != MOE_OK || !ev) return rc;
        ev->one_kernel = true;
        MOE_HIP(hipEventRecord(ev->at[2], st));
        return MOE_OK;
    }
    TileShape shape[2] = {TS_256, TS_256};
    bool in_parts[2] = {false, false};
    int bm[2] = {FM, FM};
    if (dtype == MOE_F32) {
        take_f32_kernels(R, n_used, nseg, H, F, act, round_size(), in_parts);
        for (int i = 0; i < 2; ++i) bm[i] = in_parts[i] ? XM : FM;
    } else if (skinny) {
        bm[0] = bm[1] = skinny_tile_rows(R);
    } else {
        take_shapes(R, n_used, nseg, H, F, act, round_size(), shape);
        if (timed_gemm != 0) {
            const int g = timed_gemm - 1, N = g == 0 ? F : H, a = g == 0 ? act : -1;
            const size_t need = max_items(TS_256, R, nseg, N, a, round_size()) * 16;
            if (marks_len < need) return moe_set_error(MOE_ESHAPE, "moe_diag_ffn_phases: marks needs %zu elements", need);
            if (marks_len < max_items(shape[g], R, nseg, N, a, round_size()) * 16) {   // no room for every tile of the smaller height
                shape[g] = TS_256;
                if (!maps_fit(R, nseg, kShapeRows[shape[0]], kShapeRows[shape[1]])) shape[0] = shape[1] = TS_256;
            }
        }
        for (int i = 0; i < 2; ++i) bm[i] = kShapeRows[shape[i]];
    }
    NarrowForm form[2] = {{0, 0}, {0, 0}};
    if (dtype == MOE_BF16 && timed_gemm == 0) take_narrow(R, n_used, nseg, H, F, act, round_size(), bm, form);
    if ((dtype == MOE_BF16 || bm[0] != bm[1]) && !maps_fit(R, nseg, bm[0], bm[1])) return moe_set_error(MOE_EINTERNAL, "moe_expert_ffn: tile maps of %d rows in %d segments", R, nseg);
    if (ev) MOE_HIP(hipEventRecord(ev->at[0], st));
    MapJobs jobs;
    jobs.job[0] = MapJob{bm[0], max_tiles_of(R, bm[0], nseg), tilemap_at(workspace, R)};
    jobs.job[1] = (bm[1] == bm[0]) ? jobs.job[0] : MapJob{bm[1], max_tiles_of(R, bm[1], nseg), tilemap_at(workspace, R, 1, jobs.job[0].max_tiles)};
    bool cuts[2] = {false, false};
    if (dtype == MOE_F32 && pieces_fit) take_cuts(R, n_used, nseg, H, F, act, round_size(), in_parts, cuts);
    float* const f32_pieces[2] = {cuts[0] ? partial : nullptr, cuts[1] ? partial : nullptr};   // where an fp32 GEMM's tiles are cut
    jobs.done = (dtype == MOE_BF16 || f32_pieces[0] || f32_pieces[1]) ? tilemap_at(workspace, R, 0, max_tiles_for(R) - 2).rel : nullptr;
    for (int g = 0; g < 2; ++g)
        jobs.tiles_n[g] = form[g].mt || skinny || dtype == MOE_F32 ? 0 : columns_in_strips(R, bm[g], n_used,
            tiled_columns(g == 0 ? F : H, g == 0 && act == MOE_ACT_SWIGLU, shape[g] == TS_128 ? TileGeom<2, 2>::BN : TileGeom<4, 4>::BN), g == 0 ? H : F);
    if (jobs.done) {
        jobs.job[0].m.done = jobs.done;
        jobs.job[1].m.done = jobs.done + kMaxSplitTiles;
    }
    const TileMap &m = jobs.job[0].m, &m2 = jobs.job[1].m;
    jobs.strips = jobs.job[0].m.n_tiles + 4;                  // behind the two tile counts
    const int32_t* const strips[2] = {jobs.tiles_n[0] ? jobs.strips : nullptr, jobs.tiles_n[1] ? jobs.strips + 2 : nullptr};
    const int n_maps = bm[1] == bm[0] ? 1 : 2;
    // A list of one segment (a dense MLP, shared experts) whose GEMMs both take narrow tiles needs no map either: a tile follows from the
    // segment's two offsets, which cost the GEMMs one round trip instead of the two to the number of tiles and a record.
    // Shared experts of a decode step, 64 rows of 2048 -> 2816 -> 2048: 24.7 -> 22.9 us, 16 rows 21.8 -> 19.8.
    const bool one_segment = nseg == 1 && form[0].mt && form[1].mt;
    const bool need_map = dtype == MOE_BF16 ? !one_segment : f32_needs_map(R, n_used, nseg, H, F, act, round_size(), in_parts);   // else see SegList
    const SegList seg = {seg_offset, seg_expert, nseg, R, n_local, gather, 0};
    const SegList one = one_segment ? seg : SegList{};
    if (!need_map) {
    } else if (nseg <= kSmallMapSegs) {                           // about a tile per wave
        const int blocks = std::min(64, (R / std::min(bm[0], bm[1]) + std::min(nseg, n_local) + 3) / 4);
        if (jobs.tiles_n[0] || jobs.tiles_n[1]) hipLaunchKernelGGL(tilemap_small_kernel<true>, dim3(blocks, n_maps), dim3(256), 0, st, seg_offset, seg_expert, nseg, R, n_local, gather, jobs);
        else hipLaunchKernelGGL(tilemap_small_kernel<false>, dim3(blocks, n_maps), dim3(256), 0, st, seg_offset, seg_expert, nseg, R, n_local, gather, jobs);
    } else {
        hipLaunchKernelGGL(tilemap_kernel, dim3(n_maps), dim3(kMapThreads), 0, st, seg_offset, seg_expert, nseg, R, n_local, gather, jobs);
    }
    if (need_map) MOE_LAUNCH_CHECK("tilemap_kernel");
    if (ev) MOE_HIP(hipEventRecord(ev->at[1], st));
    int rc = MOE_OK;
    if (form[0].mt) {
        if (act == MOE_ACT_SWIGLU) rc = launch_bf16_narrow<EPI_SWIGLU>(form[0], recv, H, m, tab, 0, 1, F, H, hmid, F, R, nseg, n_used, one, st);
        else if (act == MOE_ACT_GELU_MLP) rc = launch_bf16_narrow<EPI_GELU>(form[0], recv, H, m, tab, 0, 0, F, H, hmid, F, R, nseg, n_used, one, st);
        else rc = launch_bf16_narrow<EPI_SILU>(form[0], recv, H, m, tab, 0, 0, F, H, hmid, F, R, nseg, n_used, one, st);
    } else if (skinny) {
        if (act == MOE_ACT_SWIGLU) rc = launch_bf16_skinny<EPI_SWIGLU>(recv, H, m, tab, 0, 1, F, H, hmid, F, R, nseg, partial, st);
        else if (act == MOE_ACT_GELU_MLP) rc = launch_bf16_skinny<EPI_GELU>(recv, H, m, tab, 0, 0, F, H, hmid, F, R, nseg, partial, st);
        else rc = launch_bf16_skinny<EPI_SILU>(recv, H, m, tab, 0, 0, F, H, hmid, F, R, nseg, partial, st);
    } else if (dtype == MOE_BF16) {
        if (act == MOE_ACT_SWIGLU)
            rc = launch_bf16_shape<EPI_SWIGLU>(shape[0], recv, H, m, strips[0], tab, 0, 1, F, H, hmid, F, R, nseg, n_used, partial, st, timed_gemm == 1, marks, marks_len);
        else if (act == MOE_ACT_GELU_MLP)
            rc = launch_bf16_shape<EPI_GELU>(shape[0], recv, H, m, strips[0], tab, 0, 0, F, H, hmid, F, R, nseg, n_used, partial, st, timed_gemm == 1, marks, marks_len);
        else
            rc = launch_bf16_shape<EPI_SILU>(shape[0], recv, H, m, strips[0], tab, 0, 0, F, H, hmid, F, R, nseg, n_used, partial, st, timed_gemm == 1, marks, marks_len);
    } else {
        if (act == MOE_ACT_SWIGLU) rc = launch_f32<EPI_SWIGLU>(in_parts[0], need_map, recv, H, m, seg, tab, 0, 1, F, H, hmid, F, R, nseg, n_used, f32_pieces[0], st);
        else if (act == MOE_ACT_GELU_MLP) rc = launch_f32<EPI_GELU>(in_parts[0], need_map, recv, H, m, seg, tab, 0, 0, F, H, hmid, F, R, nseg, n_used, f32_pieces[0], st);
        else rc = launch_f32<EPI_SILU>(in_parts[0], need_map, recv, H, m, seg, tab, 0, 0, F, H, hmid, F, R, nseg, n_used, f32_pieces[0], st);
    }
    if (rc != MOE_OK) return rc;
    if (ev) MOE_HIP(hipEventRecord(ev->at[2], st));
    if (form[1].mt) rc = launch_bf16_narrow<EPI_PLAIN>(form[1], hmid, F, m2, tab, 2, 2, H, F, out, H, R, nseg, n_used, one, st);
    else if (skinny) rc = launch_bf16_skinny<EPI_PLAIN>(hmid, F, m2, tab, 2, 2, H, F, out, H, R, nseg, partial, st);
    else if (dtype == MOE_BF16) rc = launch_bf16_shape<EPI_PLAIN>(shape[1], hmid, F, m2, strips[1], tab, 2, 2, H, F, out, H, R, nseg, n_used, partial, st, timed_gemm == 2, marks, marks_len);
    else rc = launch_f32<EPI_PLAIN>(in_parts[1], need_map, hmid, F, m2, seg, tab, 2, 2, H, F, out, H, R, nseg, n_used, f32_pieces[1], st);
    if (rc != MOE_OK) return rc;
    if (ev) MOE_HIP(hipEventRecord(ev->at[3], st));
    return MOE_OK;
}

extern "C" int moe_expert_ffn(const void* recv, int32_t R, const int32_t* seg_offset, const int32_t* seg_expert,
                              int32_t nseg, const moe_expert_w* experts, int32_t n_local, int32_t H, int32_t F,
                              int32_t act, int32_t dtype, void* out, void* workspace, size_t workspace_bytes,
                              void* stream) {
    return ffn_impl(recv, R, seg_offset, seg_expert, nseg, experts, n_local, H, F, act, dtype, out, workspace,
                    workspace_bytes, reinterpret_cast<hipStream_t>(stream), nullptr);
}

extern "C" int moe_expert_ffn_timed(const void* recv, int32_t R, const int32_t* seg_offset, const int32_t* seg_expert,
                                    int32_t nseg, const moe_expert_w* experts, int32_t n_local, int32_t H, int32_t F,
                                    int32_t act, int32_t dtype, void* out, void* workspace, size_t workspace_bytes,
                                    void* stream, float* ms_out) {
    if (!ms_out) return moe_set_error(MOE_EINVAL, "moe_expert_ffn_timed: ms_out is NULL");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    FfnEvents ev = {{nullptr, nullptr, nullptr, nullptr}, false};
    int rc = MOE_OK;
    for (int i = 0; i < 4 && rc == MOE_OK; ++i)
        if (hipEventCreate(&ev.at[i]) != hipSuccess) rc = moe_set_error(MOE_EHIP, "hipEventCreate failed");
    if (rc == MOE_OK)
        rc = ffn_impl(recv, R, seg_offset, seg_expert, nseg, experts, n_local, H, F, act, dtype, out, workspace,
                      workspace_bytes, st, &ev);
    if (rc == MOE_OK && hipEventSynchronize(ev.at[ev.one_kernel ? 2 : 3]) != hipSuccess) rc = moe_set_error(MOE_EHIP, "hipEventSynchronize failed");
    for (int i = 0; i < 3 && rc == MOE_OK; ++i) {
        if (ev.one_kernel && i != 1) ms_out[i] = 0.f;
        else if (hipEventElapsedTime(&ms_out[i], ev.at[i], ev.at[i + 1]) != hipSuccess) rc = moe_set_error(MOE_EHIP, "hipEventElapsedTime failed");
    }
    for (int i = 0; i < 4; ++i)
        if (ev.at[i]) (void)hipEventDestroy(ev.at[i]);
    return rc;
}

extern "C" int moe_diag_ffn_phases(const void* recv, int32_t R, const int32_t* seg_offset, const int32_t* seg_expert,
                                   int32_t nseg, const moe_expert_w* experts, int32_t n_local, int32_t H, int32_t F,
                                   int32_t act, int32_t dtype, void* out, void* workspace, size_t workspace_bytes,
                                   int32_t which_gemm, int64_t* marks, size_t marks_len, void* stream) {
    if (!marks || (which_gemm != 1 && which_gemm != 2))
        return moe_set_error(MOE_EINVAL, "moe_diag_ffn_phases: marks is NULL or which_gemm is not 1 or 2");
    static_assert(sizeof(long long) == sizeof(int64_t), "marks are 64-bit");
    return ffn_impl(recv, R, seg_offset, seg_expert, nseg, experts, n_local, H, F, act, dtype, out, workspace,
                    workspace_bytes, reinterpret_cast<hipStream_t>(stream), nullptr, which_gemm,
                    reinterpret_cast<long long*>(marks), marks_len);
}
