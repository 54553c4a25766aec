// a3 -- tile binning and depth sort.
//
// Every projected Gaussian is listed once per kept screen tile of its
// rectangle (the 3DGS tile rasteriser the paper names, Sec. 3; the projection
// drops tiles the ellipse q <= 9 cannot reach), and each tile's
// list is ordered front to back by camera-space depth (depth sort per camera,
// supplementary viewer section), equal depths by ascending Gaussian id.
//
// The order is built in two stable radix sorts instead of one sort of
// (tile, depth) keys over all instances:
//   1. the surviving (view, Gaussian) records -- far fewer than instances --
//      are compacted in (view, id) order and stably sorted by their fp32
//      depth bits alone (all views mixed);
//   2. instances are emitted in that order (each record lists the kept tiles
//      of its rectangle) and stably sorted by global tile id alone.
// Because the second sort is stable and every tile belongs to one view, each
// tile's list comes out ordered by (depth, id): equal depths keep the
// compaction order, which inside one view is ascending id.  That is the order
// of sorting (tile, depth, id) keys, with 32-bit keys in both sorts.  Many
// records are sorted view by view (plan_for): both sorts then run over the
// views' runs of the arrays, in the same kernels' launches.
//
// Kernels (all HBM-bound):
//   k_valid_count / k_compact   records with n_tiles > 0 -> (depth bits, gv);
//                               inst_first[gv] = instances of all records before
//                               gv in (view, id) order: the record's gradient
//                               slots, one per kept tile in rectangle order
//   k_seg_tiles                 the views' runs, when they are sorted apart
//   radix passes (32-bit keys)  LSD, four 8-bit digits of the depth bits
//   k_sorted_count / k_emit     tiles per sorted record -> instance offsets ->
//                               work-group-cooperative emission (coalesced writes)
//   radix passes (32-bit keys)  tile ids, 5- to 7-bit digits
//   k_ranges                    [start, end) of every tile
//   k_order_count/_scan/_place  the compositing kernels' tile dispatch order
// Radix passes: one histogram kernel counts every digit of the sort in one
// read of the keys; then one kernel per digit ranks each 4096-key tile with a
// wave-level multisplit (one ballot per digit bit), takes each digit's output
// offset from the counts of the tiles before it (decoupled look-back), and
// scatters through LDS so each digit's run is written contiguously.  Counts
// that only the device knows are read from device memory, so the chain needs
// no host synchronisation.
#include "pg_internal.h"

namespace pg {

namespace {

constexpr int kBlk = 1024;           // records per compaction / emission work-group

int64_t n_blocks(const pg_views* v) { return imax(ceil_div(v->n_gv, kBlk), 1); }

struct DigitPlan {
    int passes, digit;      // LSD passes of equal width digit bits
};
constexpr int kOsMaxBits = 8;                // digit width the radix pass kernels are built for
constexpr int kDepthDigitBits = 8, kDepthPasses = 4;   // digit width caps of the record (depth) and instance (tile) sorts
constexpr int kTileDigitBits = 7;            // 18-bit tile ids: 3 x 6 bits; 19-21 bits: 3 x 7 instead of 4 x 5

DigitPlan digit_plan(int bits, int max_bits) {
    DigitPlan p;
    p.passes = (int)imax((bits + max_bits - 1) / max_bits, 1);
    p.digit = (bits + p.passes - 1) / p.passes;
    return p;
}

// Pairs per work-group of a radix pass: 4,096 keep the scattered runs long and the
// look-back short; 1,024 spread a sort of few pairs over the chip and let a group
// finish sooner (pg_bin_sort, 4,096 / 1,024 pairs: 10 k records 97 / 75 us, 131 k
// 119 / 113; 524 k records and 1 M instances 158 / 196).
constexpr int64_t kSmallSort = 1 << 18;

struct SortPlan {
    DigitPlan depth, tile;  // record sort (32-bit depth keys), instance sort (tile ids)
    int32_t segs;           // views sorted apart, 0: all views in one sort
};

constexpr int kMaxSegs = 1024;                   // views sorted apart: a thread of k_seg_tiles each
constexpr int64_t kSegRecords = 1 << 18;         // records from which views are sorted apart
constexpr int64_t kSegRecordsPass = 1 << 17;     // ... where it saves a tile pass

int view_bits(const pg_views* v) {
    int64_t most = 1;
    for (int32_t k = 0; k < v->n_views; k++) most = imax(most, v->h_tile_base[k + 1] - v->h_tile_base[k]);
    int bits = 1;
    while (((int64_t)1 << bits) < most) bits++;
    return bits;
}

// Views sorted apart: the tile ids inside one view need fewer bits than those of all
// views (two passes of 6 bits instead of three at 50 views of 1024 x 768), the records
// in (view, depth) order gather their tile sets from one view's array at a time, and
// their digits are counted in the compaction.  It costs the launches that small sorts
// fold into other kernels, and a partly filled radix tile per view.  pg_bin_sort, one
// sort / views apart, us: 2 x 1 M records 388 / 367, 16 x 65 k 201 / 166, 4 x 65 k
// 166 / 140, 200 x 1.6 k 167 / 128; 3 x 65 k 153 / 137 and 3 x 32 k 129 / 125 with a pass
// saved, 3 x 65 k 122 / 124, 8 x 16 k 117 / 121 and 2 x 16 k 129 / 147 without; one view
// of 293 k 154 / 164, of 4.2 M 499 / 499.  The large ones with the digits still counted in
// a pass of their own: 50 views x 293 k (38 M instances) 1731 / 1370, 8 x 4 frames of
// 1080p (78 M) 2972 / 2490, 10 x 3.1 M (65 M) 3274 / 3046.
SortPlan plan_for(const pg_views* v, int64_t cap) {
    SortPlan p;
    p.segs = 0;
    p.depth = digit_plan(32, kDepthDigitBits);
    p.tile = digit_plan(v->key_bits, kTileDigitBits);   // ceil(log2(n_tiles)), >= 1
    if (v->n_gv >= kSegRecordsPass && cap > kSmallSort && v->n_gauss >= kBlk && v->n_views > 1 &&
        v->n_views <= kMaxSegs) {
        const DigitPlan apart = digit_plan(view_bits(v), kTileDigitBits);   // ... of the largest view
        if (apart.passes < p.tile.passes || v->n_gv >= kSegRecords) {
            p.segs = v->n_views;
            p.tile = apart;
        }
    }
    return p;
}

size_t os_ws_bytes(int64_t cap, DigitPlan pl, int32_t segs = 0);

// One view's pairs in a sort of views apart: a run of the arrays, its radix tiles
// counted from tile_first over all runs, its keys less `base`.
struct SortSeg {
    uint32_t tile_first, start, len, base;
};

struct SortWs {
    int64_t* blk_a;          // per-block sums (compaction / emission)
    int64_t* blk_a_off;
    int64_t* blk_b;          // per-block tile sums in (view, id) order (slot offsets)
    int64_t* blk_b_off;
    int64_t* scan_tmp;
    int64_t* misc;           // [0] valid records, [1] instances to sort (0 on overflow), [4] instances (slot scan),
                             // [5] the record sort's last pass moved nothing
    uint32_t* rk0;           // record sort ping-pong
    uint32_t* rk1;
    int32_t* rv0;
    int32_t* rv1;
    uint4* stiles;           // the records' tile sets gathered in depth order (read by the emission)
    uint32_t* tk_alt;        // tile sort ping-pong partner of the caller's arrays
    int32_t* tv_alt;
    SortSeg* rec_seg;        // the views' records and instances, when views are sorted apart
    SortSeg* inst_seg;
    char* os;                // radix pass state (histograms, look-back status), shared by both sorts
    int32_t* order_cnt;      // tile dispatch order: per (tile group, length class) counts
    int32_t* order_base;     // ... and their class-major exclusive scan
    int32_t* order_cls;      // ... first slot and size of each class
};

constexpr int kOrderClasses = 64; // length classes of the tile dispatch order (four per octave)
constexpr int kOrderBlk = 256;

SortWs carve(const pg_views* v, int64_t cap, void* ws, size_t* total) {
    const SortPlan pl = plan_for(v, cap);
    SortWs w{};
    const int64_t nb = n_blocks(v);
    const int64_t ngv = imax(v->n_gv, 1);
    char* p = (char*)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* q = p + off;
        off += align256(bytes);
        return q;
    };
    w.blk_a = (int64_t*)take(nb * 8);
    w.blk_a_off = (int64_t*)take(nb * 8);
    w.blk_b = (int64_t*)take(nb * 8);
    w.blk_b_off = (int64_t*)take(nb * 8);
    w.scan_tmp = (int64_t*)take(kScanTmpWords * 8);
    w.misc = (int64_t*)take(8 * 8);
    w.rk0 = (uint32_t*)take(ngv * 4);
    w.rk1 = (uint32_t*)take(ngv * 4);
    w.rv0 = (int32_t*)take(ngv * 4);
    w.rv1 = (int32_t*)take(ngv * 4);
    w.stiles = (uint4*)take(ngv * 16);
    w.tk_alt = (uint32_t*)take(imax(cap, 1) * 4);
    w.tv_alt = (int32_t*)take(imax(cap, 1) * 4);
    w.rec_seg = (SortSeg*)take(pl.segs * sizeof(SortSeg));
    w.inst_seg = (SortSeg*)take(pl.segs * sizeof(SortSeg));
    // (views apart may sort by fewer tile digits than the one sort of a smaller table or capacity)
    w.os = take(std::max({os_ws_bytes(ngv, pl.depth, pl.segs), os_ws_bytes(cap, pl.tile, pl.segs),
                          os_ws_bytes(cap, digit_plan(v->key_bits, kTileDigitBits))}));
    const int64_t order_words = ceil_div(imax(v->n_tiles, 1), kOrderBlk) * kOrderClasses;
    w.order_cnt = (int32_t*)take(order_words * 4);
    w.order_base = (int32_t*)take(order_words * 4);
    w.order_cls = (int32_t*)take(2 * kOrderClasses * 4);
    if (total) *total = off;
    return w;
}

// Inclusive scan of one int per thread over a kBlk work-group.
__device__ __forceinline__ int32_t block_incl_1024(int32_t v, int32_t* s_warp) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    if (lane == 63) s_warp[wid] = v;
    __syncthreads();
    int32_t before = 0;
    for (int k = 0; k < wid; k++) before += s_warp[k];
    return v + before;
}

__device__ __forceinline__ int64_t block_sum_1024(int64_t c, int64_t* s) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = c;
    __syncthreads();
    int64_t t = 0;
    for (int k = 0; k < kBlk / 64; k++) t += s[k];
    return t;
}

// The kernels that walk the records (k_valid_count, k_compact) take a
// group's kBlk records with four per lane, 64 apart, so that four loads are in flight in
// each; with one, in groups of 1,024 threads, they waited on it and on the barriers of
// sixteen waves (k_valid_count and k_compact, us: 14.6 M records 88 and 100 -> 78 and
// 68, 31 M records 177 and 215 -> 125 and 144).
constexpr int kWalk = 256;
constexpr int kWalkItems = kBlk / kWalk;

__global__ __launch_bounds__(kWalk) void k_valid_count(const pg_bin* __restrict__ bins, int64_t n_gv, int64_t n_blk,
                                                       int64_t* __restrict__ blk_cnt, int64_t* __restrict__ blk_nt,
                                                       SortClear clear, uint32_t* __restrict__ ranges,
                                                       int64_t range_words) {
    __shared__ int64_t s[2][kWalk / 64];
    const int64_t i0 = (int64_t)blockIdx.x * kWalk + threadIdx.x, stride = (int64_t)gridDim.x * kWalk;
    clear.run(clear.status_words, i0, stride);
    for (int64_t i = i0; i < range_words; i += stride) ranges[i] = 0u;
    if (blockIdx.x >= n_blk) return;      // groups that only clear
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t gv = (int64_t)blockIdx.x * kBlk + wid * (kBlk / 4) + lane;
    int32_t nt[kWalkItems];
#pragma unroll
    for (int j = 0; j < kWalkItems; j++) nt[j] = gv + j * 64 < n_gv ? bins[gv + j * 64].n_tiles : 0;
    int32_t c = 0;
    int64_t t = 0;
#pragma unroll
    for (int j = 0; j < kWalkItems; j++) {
        c += (int32_t)__popcll(__ballot(nt[j] > 0));
        t += nt[j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) {
        s[0][wid] = c;
        s[1][wid] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        blk_cnt[blockIdx.x] = s[0][0] + s[0][1] + s[0][2] + s[0][3];
        blk_nt[blockIdx.x] = s[1][0] + s[1][1] + s[1][2] + s[1][3];
    }
}

// One key's digits into a wave's LDS histogram sw[p NB + d].  A wave whose active
// lanes share a digit adds once (depth keys share their high bits, which would
// otherwise serialise the LDS atomics).
template <int BITS>
__device__ __forceinline__ void count_key(uint32_t key, bool active, int passes, uint32_t* __restrict__ sw) {
    constexpr int NB = 1 << BITS;
    const uint64_t act = __ballot(active);
    if (act == 0) return;
    const int lane = threadIdx.x & 63, lead = __builtin_ctzll(act);
    for (int p = 0; p < passes; p++) {
        const uint32_t d = (key >> (p * BITS)) & (NB - 1);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, lead);
        if (__ballot(active && d == d0) == act) {
            if (lane == lead) atomicAdd(&sw[p * NB + d0], (uint32_t)__popcll(act));   // counts only: order-free
        } else if (active) {
            atomicAdd(&sw[p * NB + d], 1u);
        }
    }
}

// Compaction of the surviving records (key: depth bits, value: gv) and the
// instance-slot offsets in (view, id) order: inst_first[gv] = number of
// instances of all records before gv.  HIST (views sorted apart): a group takes
// `run` consecutive groups of records, counts their depth digits into
// hist[view][pass][digit] on the way, and notes where the views begin.  The
// counts are bound by LDS atomics and the compaction by memory, so counting here
// costs less than a pass over the keys (us, compaction and counting pass / both here:
// 14.6 M records 68 + 68 / 104, 31 M 144 + 135 / 220).
template <bool HIST>
__global__ __launch_bounds__(kWalk) void k_compact(const pg_bin* __restrict__ bins, int64_t n_gv,
                                                   const int64_t* __restrict__ blk_off,
                                                   const int64_t* __restrict__ blk_nt_off, uint32_t* __restrict__ rk,
                                                   int32_t* __restrict__ rv, int32_t* __restrict__ inst_first,
                                                   int64_t n_blk, int32_t run, SortSeg* __restrict__ rec_seg,
                                                   SortSeg* __restrict__ inst_seg, int64_t N,
                                                   uint32_t* __restrict__ hist) {
    constexpr int kWords = kDepthPasses << kDepthDigitBits;
    __shared__ int64_t s[2][kWalk / 64];
    __shared__ uint32_t s_hist[HIST ? kWalk / 64 : 1][HIST ? kWords : 1];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t g0 = HIST ? (int64_t)blockIdx.x * run : blockIdx.x, g1 = HIST ? imin(g0 + run, n_blk) : g0 + 1;
    int64_t v = 0;              // HIST: the view being counted
    auto flush = [&]() {        // its counts, and a clean histogram for the next
        __syncthreads();
        for (int i = threadIdx.x; i < kWords; i += kWalk) {
            uint32_t c = 0;
#pragma unroll
            for (int w = 0; w < kWalk / 64; w++) {
                c += s_hist[w][i];
                s_hist[w][i] = 0u;
            }
            if (c) atomicAdd(&hist[v * kWords + i], c);
        }
        __syncthreads();
    };
    if (HIST) {
        v = g0 > 0 ? (g0 * kBlk - 1) / N : 0;       // the view of the record before this run
        for (int i = threadIdx.x; i < kWords; i += kWalk) {
#pragma unroll
            for (int w = 0; w < kWalk / 64; w++) s_hist[w][i] = 0u;
        }
        __syncthreads();
    }
    for (int64_t g = g0; g < g1; g++) {
        const int64_t gv0 = g * kBlk + wid * (kBlk / 4) + lane;
        uint4 b[kWalkItems];
#pragma unroll
        for (int j = 0; j < kWalkItems; j++) {
            b[j] = make_uint4(0u, 0u, 0u, 0u);
            if (gv0 + j * 64 < n_gv) b[j] = reinterpret_cast<const uint4*>(bins)[gv0 + j * 64];
        }
        int64_t nt_excl[kWalkItems], nt_run = 0;    // instances of the wave's records before this one
        int32_t excl[kWalkItems], kept = 0;         // ... and its surviving records
#pragma unroll
        for (int j = 0; j < kWalkItems; j++) {
            const uint64_t m = __ballot((int32_t)b[j].w > 0);
            excl[j] = kept + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
            kept += (int32_t)__popcll(m);
            int64_t incl = b[j].w;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t u = __shfl_up(incl, o, 64);
                if (lane >= o) incl += u;
            }
            nt_excl[j] = nt_run + incl - b[j].w;
            nt_run += __shfl(incl, 63, 64);
        }
        if (HIST) __syncthreads();      // the group before has read s
        if (lane == 0) {
            s[0][wid] = kept;
            s[1][wid] = nt_run;
        }
        __syncthreads();
        int64_t pos0 = blk_off[g], inst0 = blk_nt_off[g];
        for (int w = 0; w < wid; w++) {
            pos0 += s[0][w];
            inst0 += s[1][w];
        }
#pragma unroll
        for (int j = 0; j < kWalkItems; j++) {
            const int64_t gv = gv0 + j * 64;
            if (gv >= n_gv) continue;
            inst_first[gv] = (int32_t)(inst0 + nt_excl[j]);
            if ((int32_t)b[j].w > 0) {
                const int64_t pos = pos0 + excl[j];
                rk[pos] = b[j].z;
                rv[pos] = (int32_t)gv;
            }
        }
        if (!HIST) continue;
        // N >= kBlk: at most one view begins in these records (the first one's at gv 0)
        const int64_t first = g == 0 ? 0 : (v + 1) * N, vn = g == 0 ? 0 : v + 1;
        const bool begins = first < imin((g + 1) * kBlk, n_gv);
#pragma unroll
        for (int j = 0; j < kWalkItems; j++) {
            if (begins && gv0 + j * 64 == first) {
                rec_seg[vn].start = (uint32_t)(pos0 + excl[j]);
                inst_seg[vn].start = (uint32_t)(inst0 + nt_excl[j]);
            }
        }
        const int64_t end = begins && vn > v ? first : (g + 1) * kBlk;      // of view v's records here
#pragma unroll
        for (int j = 0; j < kWalkItems; j++)
            count_key<kDepthDigitBits>(b[j].z, (int32_t)b[j].w > 0 && gv0 + j * 64 < end, kDepthPasses,
                                             s_hist[wid]);
        if (begins && vn > v) {
            flush();
            v = vn;
#pragma unroll
            for (int j = 0; j < kWalkItems; j++)
                count_key<kDepthDigitBits>(b[j].z, (int32_t)b[j].w > 0 && gv0 + j * 64 >= end, kDepthPasses,
                                                 s_hist[wid]);
        }
    }
    if (HIST) flush();
}

// The views' runs of records and instances from their starts (k_compact).
__global__ __launch_bounds__(kMaxSegs) void k_seg_tiles(const ViewDev* __restrict__ views, int32_t n_segs,
                                                        const int64_t* __restrict__ misc, int32_t tile,
                                                        SortSeg* __restrict__ rec_seg,
                                                        SortSeg* __restrict__ inst_seg) {
    __shared__ int32_t s_warp[2][kMaxSegs / 64];
    const int32_t v = threadIdx.x;
#pragma unroll
    for (int q = 0; q < 2; q++) {
        SortSeg* seg = q == 0 ? rec_seg : inst_seg;
        uint32_t len = 0;
        if (v < n_segs) len = (v + 1 < n_segs ? seg[v + 1].start : (uint32_t)misc[q == 0 ? 0 : 4]) - seg[v].start;
        const int32_t nt = (int32_t)ceil_div((int64_t)len, tile);
        const int32_t incl = block_incl_1024(nt, s_warp[q]);
        if (v < n_segs) {
            seg[v].tile_first = (uint32_t)(incl - nt);
            seg[v].len = len;
            seg[v].base = q == 0 ? 0u : (uint32_t)views[v].tile_base;
        }
    }
}

// The run that radix tile b belongs to (wave-uniform; -1 beyond the last one).
__device__ __forceinline__ int32_t find_seg(const SortSeg* __restrict__ segs, int32_t n_segs, uint32_t b, int32_t tile,
                                            SortSeg& out) {
    const int lane = threadIdx.x & 63;
    for (int32_t c = 0; c < n_segs; c += 64) {
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if (c + lane < n_segs) q = reinterpret_cast<const uint4*>(segs)[c + lane];
        const uint64_t hit = __ballot(b >= q.x && b - q.x < (q.z + (uint32_t)tile - 1u) / (uint32_t)tile);
        if (hit) {
            const int l = __builtin_ctzll(hit);
            out.tile_first = (uint32_t)__builtin_amdgcn_readlane((int)q.x, l);
            out.start = (uint32_t)__builtin_amdgcn_readlane((int)q.y, l);
            out.len = (uint32_t)__builtin_amdgcn_readlane((int)q.z, l);
            out.base = (uint32_t)__builtin_amdgcn_readlane((int)q.w, l);
            return c + l;
        }
    }
    return -1;
}

// Tile sets gathered into depth order (one 16-byte read per record) and the
// group sums of the kept-tile counts.
// The sorted records are in rv_moved, or in rv_stayed when the depth sort's
// last pass had one digit for every key and moved nothing (*stayed).
__global__ __launch_bounds__(kBlk) void k_sorted_count(const pg_tile_set* __restrict__ tiles,
                                                       const int32_t* __restrict__ rv_moved,
                                                       const int32_t* __restrict__ rv_stayed,
                                                       const uint32_t* __restrict__ stayed,
                                                       const int64_t* __restrict__ misc, int64_t* __restrict__ blk,
                                                       uint4* __restrict__ stiles) {
    __shared__ int64_t s[kBlk / 64];
    const int32_t* __restrict__ rv = *stayed ? rv_stayed : rv_moved;
    const int64_t p = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    int64_t c = 0;
    if (p < misc[0]) {
        const uint4 ts = reinterpret_cast<const uint4*>(tiles)[rv[p]];
        stiles[p] = ts;
        c = (int64_t)kept_count(ts);
    }
    const int64_t t = block_sum_1024(c, s);
    if (threadIdx.x == 0) blk[blockIdx.x] = t;
}

__global__ void k_sort_count(SortCount post) { post.finish(post.n_inst[0]); }

// Emission in sorted-record order.  The group's records own consecutive output
// ranges (their kept-tile counts scanned over the group); each lane walks its
// own record's kept-tile bits in increasing order (row-major over the
// rectangle), so an instance costs a bit scan and one small division.  The 64
// records of a wave own one window of the output, of a few hundred instances:
// the lanes write it to LDS, and the wave copies it out in whole lines (written
// straight from the lanes, every instance was a store address of its own: 160,
// 344 and 264 us for 38, 78 and 65 M instances, now 129, 226 and 242; two groups
// fit a CU, and a buffer that leaves room for one is slower).  It then issues VALU
// work in 87 % of its cycles, so a tile of a mask is found by one 24-bit multiply
// and shift instead of a corrected float division: 106, 173 and 203.  Windows longer
// than the buffer are written directly, as are records keeping every tile of a
// rectangle larger than 64 tiles, which are rare and long: their waves emit them
// one after another, all 64 lanes on one record.
constexpr int kEmitStage = 608;      // instances of a wave's window that LDS holds
__device__ __forceinline__ void rect_tile(int32_t k, int32_t w, float rw, int32_t& row, int32_t& col) {
    // row = k / w from a float estimate (k < 2^24), corrected to the exact quotient
    row = (int32_t)((float)k * rw);
    col = k - row * w;
    if (col < 0) { row--; col += w; }
    else if (col >= w) { row++; col -= w; }
}

__global__ __launch_bounds__(kBlk) void k_emit(const uint4* __restrict__ stiles, const int32_t* __restrict__ rv_moved,
                                               const int32_t* __restrict__ rv_stayed, int64_t N,
                                               const ViewDev* __restrict__ views,
                                               const int64_t* __restrict__ blk_off, const int64_t* __restrict__ misc,
                                               uint32_t* __restrict__ tkeys, int32_t* __restrict__ tvals,
                                               SortClear clear, int32_t passes, int32_t nb, int32_t tile) {
    const int32_t* __restrict__ rv = misc[5] ? rv_stayed : rv_moved;   // as in k_sorted_count
    __shared__ int32_t s_warp[kBlk / 64];
    __shared__ uint2 s_out[kBlk / 64][kEmitStage];
    // the tile sort's words (its workspace overlaps the record sort's, which is done): status
    // is [pass][tile][nb], of which the device-side count needs the first tiles
    if (clear.err) {
        const int64_t words = ceil_div(misc[1], tile) * nb, plane = clear.status_words / passes;
        const int64_t i0 = (int64_t)blockIdx.x * kBlk + threadIdx.x, stride = (int64_t)gridDim.x * kBlk;
        for (int32_t q = 1; q < passes; q++)
            for (int64_t i = i0; i < words; i += stride) clear.status[q * plane + i] = 0ull;
        clear.run(words, i0, stride);
    }
    if (misc[1] == 0) return;   // overflow (or nothing to emit): uniform exit
    const int t = threadIdx.x, lane = t & 63;
    const int64_t p = (int64_t)blockIdx.x * kBlk + t;
    int32_t nt = 0, gv = 0, w = 1, tx = 0;
    uint32_t tile0 = 0u;
    uint64_t mask = 0;
    if (p < misc[0]) {
        gv = rv[p];
        const uint4 ts = stiles[p];
        nt = kept_count(ts);
        const int32_t xlo = (int32_t)(ts.z & 0xffff), ylo = (int32_t)(ts.z >> 16);
        const ViewDev& V = views[(uint32_t)gv / (uint32_t)N];
        w = (int32_t)(ts.w & 0xffff);
        tx = V.TX;
        tile0 = (uint32_t)(V.tile_base + (int64_t)ylo * V.TX + xlo);
        mask = (uint64_t)ts.x | ((uint64_t)ts.y << 32);
    }
    const int32_t incl = block_incl_1024(nt, s_warp);
    const int32_t o0 = incl - nt;                                      // first output in the group
    const int32_t w0 = __builtin_amdgcn_readfirstlane(o0);             // ... of the wave's window
    const int32_t total = __builtin_amdgcn_readlane(incl, 63) - w0;
    const int64_t base = blk_off[blockIdx.x];
    // masks: rectangles of at most 64 tiles, so bit / w is (bit inv) >> 16 with inv the next
    // integer above 2^16 / w (the excess, below 2, times 63 stays under 2^16 / w)
    const uint32_t inv = (uint32_t)(65536.0f * __builtin_amdgcn_rcpf((float)w)) + 1u;
    const uint32_t skip = (uint32_t)(tx - w);         // tiles between the rectangle's rows
    auto key_of = [&](uint32_t bit) __attribute__((always_inline)) {
        return tile0 + bit + __umul24(__umul24(bit, inv) >> 16, skip);
    };
    uint64_t big = __ballot(mask == 0 && nt > 0);
    if (big == 0 && total <= kEmitStage) {
        uint2* out = s_out[t >> 6];
        int32_t e = o0 - w0;
        for (uint64_t m = mask; m != 0; e++) {
            out[e] = make_uint2(key_of((uint32_t)__builtin_ctzll(m)), (uint32_t)gv);
            m &= m - 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // the buffer is the wave's own
        for (int32_t i = lane; i < total; i += 64) {
            const uint2 kv = out[i];
            tkeys[base + w0 + i] = kv.x;
            tvals[base + w0 + i] = (int32_t)kv.y;
        }
        return;
    }
    const int64_t e0 = base + o0;
    if (mask != 0) {
        uint64_t m = mask;
        for (int64_t e = e0; m != 0; e++) {
            tkeys[e] = key_of((uint32_t)__builtin_ctzll(m));
            tvals[e] = gv;
            m &= m - 1;
        }
    }
    // records that keep every tile of their rectangle, one at a time per wave
    while (big) {
        const int src = __builtin_ctzll(big);
        big &= big - 1;
        const int32_t bn = __shfl(nt, src, 64), bw = __shfl(w, src, 64), btx = __shfl(tx, src, 64);
        const int32_t bgv = __shfl(gv, src, 64);
        const uint32_t bt0 = (uint32_t)__shfl((int)tile0, src, 64);
        const int64_t be0 = __shfl(e0, src, 64);
        const float brw = 1.0f / (float)bw;
        for (int32_t k = lane; k < bn; k += 64) {
            int32_t row, col;
            rect_tile(k, bw, brw, row, col);
            tkeys[be0 + k] = bt0 + (uint32_t)(row * btx + col);
            tvals[be0 + k] = bgv;
        }
    }
}

// Peers of this lane: active lanes holding the same BITS-bit digit.  Per
// bit, the ballot of the lanes that have it set, flipped where this lane's
// bit is clear, marks the lanes that differ from it in that bit; a peer
// differs in none.  Each half of the 64-lane mask costs an exclusive-or with
// the lane's sign-extended bit and an or per bit.
template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool active) {
    uint32_t diff_lo = 0u, diff_hi = 0u;
#pragma unroll
    for (int b = 0; b < BITS; b++) {
        const uint32_t s = (uint32_t)__builtin_amdgcn_sbfe((int32_t)d, b, 1);   // all ones where this lane's bit is set
        const uint64_t m = __ballot(s != 0u);
        diff_lo |= (uint32_t)m ^ s;
        diff_hi |= (uint32_t)(m >> 32) ^ s;
    }
    const uint64_t eq = ~(((uint64_t)diff_hi << 32) | diff_lo);
    return eq & __ballot(active);
}

// ------------------------------------------------------------------ onesweep LSD radix passes
// One kernel per digit.  Work-group b ranks the keys of radix tile b (4096
// pairs) with the wave multisplit, publishes its digit counts, and finds
// each digit's output offset by looking back over the tiles before it
// (decoupled look-back): a tile's status word per digit holds either its own
// count (AGG) or the count of that digit over every tile up to and including
// it (PRE).  The digit offsets over the whole input come from one histogram
// pass over the keys for every digit of the sort.  A pass reads and writes
// each pair once.
// Waiting on lower-numbered work-groups cannot deadlock because every XCD
// starts its share of the grid in index order: the lowest-numbered unfinished
// work-group has no unfinished predecessor, and if it had not started, its
// XCD would hold only finished lower-numbered groups and so have room for it.
// (An atomic ticket per work-group, which does not rely on that order, made
// the passes 15 % slower.)  The wait is bounded anyway: a look-back that
// polls kLookbackSpins times gives up, and the sort reports it.
constexpr uint32_t kStAgg = 1u, kStPre = 2u;
constexpr int kLookbackSpins = 1 << 22;      // a bound that a working chain never reaches (~1 s of polling)
constexpr int kMaxSortPasses = 4;
constexpr int kLookWindow = 6;               // predecessors read at once by the look-back (4 to 8 alike, 16 and 2 slower)

__device__ __forceinline__ void st_publish(unsigned long long* p, uint32_t flag, uint32_t value) {
    __hip_atomic_store(p, ((unsigned long long)flag << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long st_read(unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Decoupled look-back: the sum of the values of work-groups 0 .. b-1 (b > 0)
// from their status words (work-group k's at p[k * stride]), read
// kLookWindow at a time from b - 1 backwards (a first wave of work-groups
// starts together, and one dependent load per predecessor would make its
// walks long) and added until a word flagged kStPre (an inclusive prefix).  A
// word not yet published is read again; after kLookbackSpins waits the walk
// gives up and sets *err (never in a working chain: report, do not hang).
__device__ __forceinline__ uint32_t lookback_excl(unsigned long long* p, int64_t stride, int64_t b, int32_t* err) {
    uint32_t excl = 0;
    int64_t k = b - 1;          // newest predecessor not yet added
    int spins = 0;
    bool done = false;
    while (!done) {
        unsigned long long w[kLookWindow];
#pragma unroll
        for (int j = 0; j < kLookWindow; j++) w[j] = k - j >= 0 ? st_read(&p[(k - j) * stride]) : 0ull;
        // newest first: add counts until a PRE word; stop at a word not published yet
        int adv = 0;
        bool stop = false;
#pragma unroll
        for (int j = 0; j < kLookWindow; j++) {
            const uint32_t flag = (uint32_t)(w[j] >> 32);
            if (!stop && !done) {
                if (k - j < 0 || flag == 0u) {
                    stop = true;
                } else {
                    excl += (uint32_t)w[j];
                    adv = j + 1;
                    done = flag == kStPre || k - j == 0;
                }
            }
        }
        if (done) break;
        k -= adv;
        if (adv < kLookWindow) {      // waiting on an unpublished word
            if (++spins > kLookbackSpins) {
                atomicOr(err, 1);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return excl;
}

// Exclusive scan of each pass's digit counts, a wave per pass; uni[p] = 1 when one
// digit of pass p holds every key (the pass is then the identity permutation).
// The counts were added at the device's coherence point and are read there.
__device__ void os_scan(uint32_t* __restrict__ hist, int passes, int nb, int64_t n, uint32_t start,
                        uint32_t* __restrict__ uni, uint32_t* __restrict__ all) {
    constexpr int kPer = (1 << kOsMaxBits) / 64;
    const int lane = threadIdx.x & 63, p = threadIdx.x >> 6;
    if (p >= passes) return;
    const int per = nb > 64 ? nb / 64 : 1;
    uint32_t c[kPer], sum = 0;
    bool whole = false;
#pragma unroll
    for (int e = 0; e < kPer; e++) {
        const int d = lane * per + e;
        c[e] = e < per && d < nb ? __hip_atomic_load(&hist[p * nb + d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        whole |= n > 0 && (int64_t)c[e] == n;
        sum += c[e];
    }
    const bool one = __ballot(whole) != 0;
    if (lane == 0) uni[p] = one ? 1u : 0u;
    if (lane == 0 && all && n > 0 && !one) all[p] = 0u;
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    uint32_t x = start + incl - sum;
#pragma unroll
    for (int e = 0; e < kPer; e++) {
        const int d = lane * per + e;
        if (e < per && d < nb) hist[p * nb + d] = x;
        x += c[e];
    }
}

__global__ __launch_bounds__(64 * kMaxSortPasses) void k_os_scan(uint32_t* __restrict__ hist, int passes, int nb,
                                                                const int64_t* __restrict__ n_ptr,
                                                                const SortSeg* __restrict__ segs,
                                                                uint32_t* __restrict__ uni) {
    if (!segs) return os_scan(hist, passes, nb, *n_ptr, 0u, uni, nullptr);
    const int32_t v = blockIdx.x;
    os_scan(hist + (int64_t)v * passes * nb, passes, nb, segs[v].len, segs[v].start,
            uni + (1 + v) * kMaxSortPasses, uni);
}

// Digit counts of every pass of a sort in one read of the keys (and, with
// `finished`, their scan by the last group to finish):
// hist[p NB + d] = keys whose bits [p BITS, (p + 1) BITS) equal d.  Each wave
// counts into its own LDS histogram; with UNIFORM, a wave whose active lanes
// share a digit adds once (depth keys share their high bits, which would
// otherwise serialise the LDS atomics).
template <int BITS, bool UNIFORM, int KPT>
__device__ __forceinline__ void os_count(const uint32_t* __restrict__ keys, int64_t base, int64_t n, uint32_t key0,
                                         int passes, uint32_t* __restrict__ sw) {
    constexpr int NB = 1 << BITS;
    uint32_t k[KPT];
#pragma unroll
    for (int j = 0; j < KPT; j++) {
        const int64_t i = base + (int64_t)j * 256 + threadIdx.x;
        k[j] = i < n ? keys[i] - key0 : 0u;
    }
#pragma unroll
    for (int j = 0; j < KPT; j++) {
        const bool active = base + (int64_t)j * 256 + threadIdx.x < n;
        if (UNIFORM) {
            count_key<BITS>(k[j], active, passes, sw);
        } else if (active) {
            for (int p = 0; p < passes; p++) atomicAdd(&sw[p * NB + ((k[j] >> (p * BITS)) & (NB - 1))], 1u);
        }
    }
}

template <int BITS, bool UNIFORM, int KPT>
__global__ __launch_bounds__(256) void k_os_hist(const uint32_t* __restrict__ keys, const int64_t* __restrict__ n_ptr,
                                                 int passes, uint32_t* __restrict__ hist, uint32_t* __restrict__ uni,
                                                 int32_t* __restrict__ finished) {
    constexpr int NB = 1 << BITS;
    __shared__ uint32_t s[4][kMaxSortPasses * NB];
    for (int i = threadIdx.x; i < passes * NB; i += 256) {
#pragma unroll
        for (int w = 0; w < 4; w++) s[w][i] = 0;
    }
    __syncthreads();
    const int64_t n = *n_ptr;
    if (n == 0) return;       // the passes read nothing either
    for (int64_t base = (int64_t)blockIdx.x * 256 * KPT; base < n; base += (int64_t)gridDim.x * 256 * KPT)
        os_count<BITS, UNIFORM, KPT>(keys, base, n, 0u, passes, s[threadIdx.x >> 6]);
    __syncthreads();
    for (int i = threadIdx.x; i < passes * NB; i += 256) {
        const uint32_t c = s[0][i] + s[1][i] + s[2][i] + s[3][i];
        if (c) atomicAdd(&hist[i], c);
    }
    if (!finished) return;
    // The last group to finish turns the counts into offsets.  The counts were added by
    // atomics at the device's coherence point, so they only have to have completed before the
    // group reports: a device fence would also write back the whole L2 (280 us a sort at
    // 38 M instances).
    __shared__ int32_t s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(finished, 1) == (int32_t)gridDim.x - 1;
    __syncthreads();
    if (s_last) os_scan(hist, passes, NB, n, 0u, uni, nullptr);
}

// The digit counts of views sorted apart, hist[(v passes + p) NB + d]: a group takes a
// run of consecutive radix tiles and adds its counts whenever the view changes.
template <int BITS, int KPT>
__global__ __launch_bounds__(256) void k_os_hist_seg(const uint32_t* __restrict__ keys,
                                                     const int64_t* __restrict__ n_ptr,
                                                     const SortSeg* __restrict__ segs, int32_t n_segs, int passes,
                                                     uint32_t* __restrict__ hist) {
    constexpr int NB = 1 << BITS;
    constexpr int kTile = 256 * KPT;
    __shared__ uint32_t s[4][kMaxSortPasses * NB];
    for (int i = threadIdx.x; i < passes * NB; i += 256) {
#pragma unroll
        for (int w = 0; w < 4; w++) s[w][i] = 0;
    }
    __syncthreads();
    if (*n_ptr == 0) return;
    const SortSeg last = segs[n_segs - 1];
    const uint32_t tiles = last.tile_first + (last.len + kTile - 1) / kTile;
    const uint32_t per = (tiles + gridDim.x - 1) / gridDim.x;
    const uint32_t b1 = min((blockIdx.x + 1) * per, tiles);
    SortSeg seg{0u, 0u, 0u, 0u};
    int32_t cur = -1;
    for (uint32_t b = blockIdx.x * per; b < b1;) {
        cur = find_seg(segs, n_segs, b, kTile, seg);
        if (cur < 0) return;      // never with a whole table: every tile below `tiles` has its run
        const uint32_t e = min(b1, seg.tile_first + (seg.len + kTile - 1) / kTile);
        for (; b < e; b++)
            os_count<BITS, false, KPT>(keys, seg.start + (int64_t)(b - seg.tile_first) * kTile,
                                       (int64_t)seg.start + seg.len, seg.base, passes, s[threadIdx.x >> 6]);
        __syncthreads();
        for (int i = threadIdx.x; i < passes * NB; i += 256) {
            const uint32_t c = s[0][i] + s[1][i] + s[2][i] + s[3][i];
            if (c) atomicAdd(&hist[(int64_t)cur * passes * NB + i], c);
            if (b < b1) {
#pragma unroll
                for (int w = 0; w < 4; w++) s[w][i] = 0;
            }
        }
        __syncthreads();
    }
}

// Clears what the passes of one sort count on: the histograms, the look-back
// error flag, the histogram's count of finished groups (the word after it) and the status words of the tiles the device-side
// count needs (status is [pass][tile][NB], tile stride NB, pass stride
// tiles_max NB).
__global__ void k_os_clear(const int64_t* __restrict__ n_ptr, int tile, int passes, int nb, int64_t tiles_max,
                           unsigned long long* __restrict__ status, uint32_t* __restrict__ hist,
                           uint32_t* __restrict__ all, int32_t n_segs, int32_t* __restrict__ err) {
    const int64_t ntile = imin(ceil_div(*n_ptr, tile) + n_segs, tiles_max);
    const int64_t words = ntile * nb;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int p = 0; p < passes; p++)
        for (int64_t i = i0; i < words; i += stride) status[p * tiles_max * nb + i] = 0ull;
    for (int64_t i = i0; i < (int64_t)imax(n_segs, 1) * passes * nb; i += stride) hist[i] = 0u;
    if (i0 < kMaxSortPasses) all[i0] = 1u;
    if (i0 < 2) err[i0] = 0;
}

template <int BITS, int ITEMS, bool SEG>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_onesweep(const uint32_t* __restrict__ keys_in,
                                                           const int32_t* __restrict__ vals_in,
                                                           uint32_t* __restrict__ keys_out,
                                                           int32_t* __restrict__ vals_out,
                                                           const int64_t* __restrict__ n_ptr,
                                                           const SortSeg* __restrict__ segs, int32_t n_segs, int shift,
                                                           const uint32_t* __restrict__ digit_base, int seg_words,
                                                           const uint32_t* __restrict__ uniform,
                                                           const uint32_t* __restrict__ stay,
                                                           unsigned long long* __restrict__ status,
                                                           int32_t* __restrict__ err) {
    constexpr int NB = 1 << BITS;
    constexpr int kTile = kSortThreads * ITEMS;
    constexpr int PER = NB >= kSortThreads ? NB / kSortThreads : 1;   // digits per thread
    constexpr int ACT = NB / PER;                                     // threads owning digits
    __shared__ uint32_t s_hist[4][NB];      // per-wave digit counts, then each wave's offset inside the digit
    __shared__ uint32_t s_lstart[NB];       // first position of each digit in the tile
    __shared__ int32_t s_glob[NB];          // output index of a digit's first pair, less s_lstart
    __shared__ uint32_t s_part[kSortThreads / 64];
    __shared__ uint32_t s_keys[kTile];
    __shared__ int32_t s_vals[kTile];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    for (int d = t; d < NB; d += kSortThreads) {
#pragma unroll
        for (int w = 0; w < 4; w++) s_hist[w][d] = 0;
    }
    __syncthreads();
    int64_t n = *n_ptr;                  // end of the run
    const int64_t b = blockIdx.x;
    int64_t first = b * kTile, lb = b;   // the tile's first pair; its number in the run
    uint32_t key0 = 0u;
    if (SEG) {
        if (n == 0) return;
        SortSeg seg;
        const int32_t v = find_seg(segs, n_segs, (uint32_t)b, kTile, seg);
        if (v < 0) return;
        lb = b - seg.tile_first;
        first = seg.start + lb * kTile;
        n = (int64_t)seg.start + seg.len;
        key0 = seg.base;
        digit_base += v * seg_words;
        uniform += (1 + v) * kMaxSortPasses;
    } else if (first >= n) {
        return;
    }
    if (*uniform) {     // every key has the same digit: the stable order is the input order
        if (stay && *stay) return;   // the caller reads the input buffers when this pass moves nothing
        const int64_t e = imin(n, first + kTile);
        for (int64_t i = first + t; i < e; i += kSortThreads) {
            keys_out[i] = keys_in[i];
            vals_out[i] = vals_in[i];
        }
        return;
    }
    uint32_t key[ITEMS];
    int32_t val[ITEMS];
    uint32_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const int64_t idx = first + (int64_t)wid * (kTile / 4) + r * 64 + lane;
        const bool active = idx < n;
        key[r] = active ? keys_in[idx] : 0u;
        val[r] = active ? vals_in[idx] : 0;
    }
    const int64_t start = first + (int64_t)wid * (kTile / 4);
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const int64_t idx = start + r * 64 + lane;
        const bool active = idx < n;
        const uint32_t d = ((key[r] - key0) >> shift) & (NB - 1);
        const uint64_t peers = match_digit<BITS>(d, active);
        const uint64_t below = peers & ((1ull << lane) - 1ull);
        const uint32_t base = s_hist[wid][d];
        rank[r] = base + (uint32_t)__popcll(below);
        if (active && below == 0) s_hist[wid][d] = base + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: offsets of the waves inside the digit, the tile's count, and its status word
    uint32_t tot[PER];
    uint32_t mine = 0;
    if (t < ACT) {
#pragma unroll
        for (int e = 0; e < PER; e++) {
            const int d = t * PER + e;
            uint32_t run = 0;
#pragma unroll
            for (int w = 0; w < 4; w++) {
                const uint32_t c = s_hist[w][d];
                s_hist[w][d] = run;
                run += c;
            }
            tot[e] = run;
            mine += run;
            st_publish(&status[b * NB + d], lb == 0 ? kStPre : kStAgg, run);
        }
    }
    // exclusive scan of the tile's digit counts -> s_lstart
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) s_part[wid] = incl;
    __syncthreads();
    uint32_t pre = 0;
    for (int w = 0; w < wid; w++) pre += s_part[w];
    if (t < ACT) {
        uint32_t x = pre + incl - mine;
#pragma unroll
        for (int e = 0; e < PER; e++) {
            s_lstart[t * PER + e] = x;
            x += tot[e];
        }
    }
    __syncthreads();
    // the tile's pairs in digit order in LDS (stable: waves, then rounds, then lanes)
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const int64_t idx = start + r * 64 + lane;
        if (idx < n) {
            const uint32_t d = ((key[r] - key0) >> shift) & (NB - 1);
            const uint32_t pos = s_lstart[d] + s_hist[wid][d] + rank[r];
            s_keys[pos] = key[r];
            s_vals[pos] = val[r];
        }
    }
    // look-back: this digit's count over the run's tiles before this one
    if (t < ACT) {
#pragma unroll
        for (int e = 0; e < PER; e++) {
            const int d = t * PER + e;
            uint32_t excl = 0;
            if (lb > 0) {
                excl = lookback_excl(status + (b - lb) * NB + d, NB, lb, err);
                st_publish(&status[b * NB + d], kStPre, excl + tot[e]);
            }
            s_glob[d] = (int32_t)(digit_base[d] + excl) - (int32_t)s_lstart[d];
        }
    }
    __syncthreads();
    const int64_t tile_n = imin(kTile, n - first);
    for (int64_t i = t; i < tile_n; i += kSortThreads) {
        const uint32_t k = s_keys[i];
        const int64_t o = (int64_t)s_glob[((k - key0) >> shift) & (NB - 1)] + i;
        keys_out[o] = k;
        vals_out[o] = s_vals[i];
    }
}

// Workspace of the onesweep passes of one sort of at most `cap` pairs.
struct OsWs {
    unsigned long long* status;
    uint32_t* hist;
    uint32_t* uni;       // per pass: one digit holds every key (of views apart: in each view, then per view)
    int32_t* err;        // look-back error, then the histogram's finished groups
    int64_t tiles_max;
    int32_t tile;        // pairs per work-group of a pass
    const SortSeg* segs; // the runs of views sorted apart
    int32_t n_segs;
};
constexpr int kSmallItems = 4;
int32_t sort_tile(int64_t cap) { return kSortThreads * (cap <= kSmallSort ? kSmallItems : kSortItems); }

// Views apart add a partly filled tile each, and a histogram and a flag per pass each.
OsWs os_layout(int64_t cap, DigitPlan pl, const SortSeg* segs, int32_t n_segs, char* p, size_t* bytes) {
    OsWs w{};
    w.tile = n_segs ? kSortTile : sort_tile(cap);
    w.segs = n_segs ? segs : nullptr;
    w.n_segs = n_segs;
    w.tiles_max = imax(ceil_div(imax(cap, 1), w.tile), 1) + n_segs;
    size_t off = 0;
    w.status = (unsigned long long*)(p + off);
    off += align256((size_t)pl.passes * w.tiles_max * ((size_t)1 << pl.digit) * 8);
    w.hist = (uint32_t*)(p + off);
    off += align256((size_t)imax(n_segs, 1) * kMaxSortPasses * ((size_t)1 << kOsMaxBits) * 4);
    w.uni = (uint32_t*)(p + off);
    off += align256((size_t)(1 + n_segs) * kMaxSortPasses * 4);
    w.err = (int32_t*)(p + off);
    off += align256(2 * 4);
    if (bytes) *bytes = off;
    return w;
}
// Bytes for any sort of at most cap pairs: small radix tiles need four times the status
// words of large ones, so the largest of the layouts up to cap (a workspace sized once for
// the largest sort serves the smaller ones).
size_t os_ws_bytes(int64_t cap, DigitPlan pl, int32_t segs) {
    size_t bytes = 0, small = 0;
    os_layout(cap, pl, nullptr, segs, nullptr, &bytes);
    os_layout(imin(cap, kSmallSort), pl, nullptr, 0, nullptr, &small);
    return std::max(bytes, small);
}
OsWs os_carve(int64_t cap, DigitPlan pl, char* p, const SortSeg* segs = nullptr, int32_t n_segs = 0) {
    return os_layout(cap, pl, segs, n_segs, p, nullptr);
}

SortClear sort_clear(const OsWs& w, DigitPlan pl) {
    const int nb = 1 << pl.digit;
    return {w.status, (int64_t)pl.passes * w.tiles_max * nb, w.hist, pl.passes * nb, w.err};
}

void os_clear(DigitPlan pl, const int64_t* n_ptr, const OsWs& w, hipStream_t s) {
    k_os_clear<<<1024, 256, 0, s>>>(n_ptr, w.tile, pl.passes, 1 << pl.digit, w.tiles_max, w.status, w.hist, w.uni,
                                    w.n_segs, w.err);
}

// Stable LSD sort of the *n_ptr (<= cap) pairs in (ka, va) by their low
// pl.passes * pl.digit key bits, ping-ponging with (kb, vb); the result
// lands in (ka, va) for an even number of passes, else in (kb, vb).
// uniform_high: keys whose high digits mostly agree (depth bits), counted with
// the wave-uniform shortcut.  last_may_stay: when the last pass's digit is one
// value for every key, that pass moves nothing and the result stays where the
// pass before left it; w.uni[passes - 1] tells the caller which.  few: the words are
// cleared and the histogram is scanned by kernels around it; counted: they are cleared
// and the digits are counted.
hipError_t onesweep_sort(DigitPlan pl, uint32_t* ka, int32_t* va, uint32_t* kb, int32_t* vb, const int64_t* n_ptr,
                         int64_t cap, OsWs w, bool uniform_high, bool last_may_stay, bool few, bool counted,
                         hipStream_t s) {
    const int nb = 1 << pl.digit;
    int32_t* finished = few ? w.err + 1 : nullptr;
    if (!few && !counted) os_clear(pl, n_ptr, w, s);
    const bool small = w.tile == kSortThreads * kSmallItems;
    const unsigned hgrid = (unsigned)imax(1, imin(2048, ceil_div(imax(cap, 1), w.tile)));
    if (!counted) switch (pl.digit) {
#define PG_HIST_AS(B, U, K) \
    k_os_hist<B, U, K><<<hgrid, 256, 0, s>>>(ka, n_ptr, pl.passes, w.hist, w.uni, finished)
// (views apart count tile digits only: their depth digits are counted in the compaction)
#define PG_HIST_SEG(B)                                                     \
    if (B > kTileDigitBits) return hipErrorInvalidValue;                   \
    k_os_hist_seg<(B < kTileDigitBits ? B : kTileDigitBits), kSortItems>   \
        <<<hgrid, 256, 0, s>>>(ka, n_ptr, w.segs, w.n_segs, pl.passes, w.hist)
#define PG_HIST(B)                                                  \
    case B:                                                         \
        if (w.n_segs) {                                             \
            PG_HIST_SEG(B);                                         \
        } else if (uniform_high) {                                  \
            if (small) PG_HIST_AS(B, true, kSmallItems);            \
            else PG_HIST_AS(B, true, kSortItems);                   \
        } else {                                                    \
            if (small) PG_HIST_AS(B, false, kSmallItems);           \
            else PG_HIST_AS(B, false, kSortItems);                  \
        }                                                           \
        break;
        PG_HIST(1) PG_HIST(2) PG_HIST(3) PG_HIST(4) PG_HIST(5) PG_HIST(6) PG_HIST(7) PG_HIST(8)
#undef PG_HIST
#undef PG_HIST_AS
#undef PG_HIST_SEG
        default: return hipErrorInvalidValue;
    }
    if (!few)
        k_os_scan<<<(unsigned)imax(w.n_segs, 1), 64 * kMaxSortPasses, 0, s>>>(w.hist, pl.passes, nb, n_ptr, w.segs,
                                                                              w.uni);
    const unsigned grid = (unsigned)w.tiles_max;
    for (int p = 0; p < pl.passes; p++) {
        unsigned long long* st = w.status + (int64_t)p * w.tiles_max * nb;
        const uint32_t* stay = last_may_stay && p == pl.passes - 1 ? w.uni + p : nullptr;
        switch (pl.digit) {
#define PG_PASS_AS(B, K, SEG)                                                                              \
    k_onesweep<B, K, SEG><<<grid, kSortThreads, 0, s>>>(ka, va, kb, vb, n_ptr, w.segs, w.n_segs,            \
                                                        p * pl.digit, w.hist + p * nb, pl.passes * nb,      \
                                                        w.uni + p, stay, st, w.err)
#define PG_PASS(B)                                         \
    case B:                                                \
        if (w.n_segs) PG_PASS_AS(B, kSortItems, true);     \
        else if (small) PG_PASS_AS(B, kSmallItems, false); \
        else PG_PASS_AS(B, kSortItems, false);             \
        break;
            PG_PASS(1) PG_PASS(2) PG_PASS(3) PG_PASS(4) PG_PASS(5) PG_PASS(6) PG_PASS(7) PG_PASS(8)
#undef PG_PASS
#undef PG_PASS_AS
            default: return hipErrorInvalidValue;
        }
        uint32_t* tk = ka; ka = kb; kb = tk;
        int32_t* tv = va; va = vb; vb = tv;
    }
    return hipGetLastError();
}

// [start, end) of every tile from the sorted keys: a tile starts where the key
// differs from its predecessor, which is also where the previous tile ends.
// Four consecutive keys per thread, over a fixed grid that strides through
// the device-side count (a grid sized for the capacity was mostly empty
// groups); the predecessor of a thread's first key is the neighbouring lane's
// last (only the first lane of a wave loads it), so every key is read once.
constexpr int kRangeGrid = 4096;
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ keys, const int64_t* __restrict__ misc,
                                                int32_t* __restrict__ ranges, const int32_t* __restrict__ err,
                                                int32_t* __restrict__ overflow) {
    const int64_t I = misc[1];
    // bit 1 of the caller's overflow word: a look-back of the tile sort gave up (results undefined)
    if (blockIdx.x == 0 && threadIdx.x == 0 && *err) *overflow |= 2;
    const int64_t nq = (I + 3) / 4;
    for (int64_t base = (int64_t)blockIdx.x * 256; base < nq; base += (int64_t)gridDim.x * 256) {
        const int64_t i0 = 4 * (base + threadIdx.x);
        uint32_t k[4];
#pragma unroll
        for (int j = 0; j < 4; j++) k[j] = i0 + j < I ? keys[i0 + j] : 0u;
        uint32_t prev = __shfl_up(k[3], 1, 64);
        if ((threadIdx.x & 63) == 0 && i0 > 0 && i0 < I) prev = keys[i0 - 1];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t i = i0 + j;
            if (i >= I) break;
            const uint32_t p = j == 0 ? prev : k[j - 1];
            if (i == 0) {
                ranges[2 * (int64_t)k[j]] = 0;
            } else if (p != k[j]) {
                ranges[2 * (int64_t)k[j]] = (int32_t)i;
                ranges[2 * (int64_t)p + 1] = (int32_t)i;
            }
            if (i == I - 1) ranges[2 * (int64_t)k[j] + 1] = (int32_t)I;
        }
    }
}

// ---------------------------------------------------------------- tile dispatch order
// The compositing kernels run one work-group per tile, and tiles differ in
// cost by their list lengths.  Dispatching the longest lists first (a
// longest-processing-time-first schedule) shortens the tail of those
// launches, where a few long tiles would otherwise run on an emptying chip.
// The order is coarse: 64 classes of list length, four per octave, longest
// class first.  Inside a class, tiles keep their index order and are dealt to
// the XCDs in contiguous runs: the dispatcher hands work-group b to XCD b mod
// 8, so the slots of a class that land on XCD x receive one run of
// neighbouring tiles, which share Gaussians and so their records in that
// XCD's L2.  The order is deterministic and results do not depend on it.
__device__ __forceinline__ int order_class(int32_t len) {
    const uint32_t b = __float_as_uint((float)(len > 0 ? len : 0) + 1.0f);
    const int c = 4 * ((int)((b >> 23) & 0xffu) - 127) + (int)((b >> 21) & 3u);   // 4 log2(len + 1), floored
    return kOrderClasses - 1 - (c < 0 ? 0 : (c < kOrderClasses - 1 ? c : kOrderClasses - 1));
}

// Per work-group of kOrderBlk consecutive tiles: the tile count of each class.
__global__ __launch_bounds__(kOrderBlk) void k_order_count(const int2* __restrict__ ranges, int64_t n_tiles,
                                                           int32_t* __restrict__ cnt) {
    __shared__ int32_t s_cnt[kOrderClasses];
    if (threadIdx.x < kOrderClasses) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kOrderBlk + threadIdx.x;
    if (t < n_tiles) {
        const int2 r = ranges[t];
        atomicAdd(&s_cnt[order_class(r.y - r.x)], 1);     // counts only: order-free
    }
    __syncthreads();
    if (threadIdx.x < kOrderClasses) cnt[(int64_t)blockIdx.x * kOrderClasses + threadIdx.x] = s_cnt[threadIdx.x];
}

// Class-major exclusive scan of the counts (one work-group of 1024 threads):
// base[w][c] = tiles of the classes before c + tiles of class c in groups
// before w; cls[c] = first slot of class c, cls[kOrderClasses + c] = its size.
constexpr int kOrderSeg = 1024 / kOrderClasses;     // threads per class in the scan
__global__ __launch_bounds__(1024) void k_order_scan(const int32_t* __restrict__ cnt, int64_t n_groups,
                                                     int32_t* __restrict__ base, int32_t* __restrict__ cls) {
    __shared__ int32_t s_part[kOrderClasses][kOrderSeg];
    __shared__ int32_t s_first[kOrderClasses];
    // thread (c, k): class c of the k-th run of groups; a wave reads whole rows
    // of 64 class counts, and the loads of a run are independent
    const int c = threadIdx.x % kOrderClasses, k = threadIdx.x / kOrderClasses;
    const int64_t per = ceil_div(n_groups, kOrderSeg);
    const int64_t w0 = imin(n_groups, k * per), w1 = imin(n_groups, w0 + per);
    int32_t sum = 0;
#pragma unroll 8
    for (int64_t w = w0; w < w1; w++) sum += cnt[w * kOrderClasses + c];
    s_part[c][k] = sum;
    __syncthreads();
    if (threadIdx.x < 64) {     // one wave: class totals and their exclusive scan
        int32_t tot = 0;
        for (int j = 0; j < kOrderSeg; j++) tot += s_part[threadIdx.x][j];
        int32_t incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t u = __shfl_up(incl, o, 64);
            if ((int)threadIdx.x >= o) incl += u;
        }
        s_first[threadIdx.x] = incl - tot;
        cls[threadIdx.x] = incl - tot;
        cls[kOrderClasses + threadIdx.x] = tot;
    }
    __syncthreads();
    int32_t run = s_first[c];
    for (int j = 0; j < k; j++) run += s_part[c][j];
#pragma unroll 8
    for (int64_t w = w0; w < w1; w++) {
        base[w * kOrderClasses + c] = run;
        run += cnt[w * kOrderClasses + c];
    }
}

// Dispatch slot of the rank-r tile (in index order) of a class holding slots
// [o, o + n): XCD x receives the ranks [R_x, R_x + m_x), where m_x counts the
// class's slots s with s mod 8 = x and R_x those of the XCDs before x.
__device__ __forceinline__ int64_t order_slot(int64_t o, int64_t n, int64_t r) {
    int64_t R = 0;
    for (int x = 0; x < 8; x++) {
        const int64_t f = o + ((x - (o & 7)) & 7);        // first slot of the class on XCD x
        const int64_t m = f < o + n ? (o + n - f + 7) / 8 : 0;
        if (r < R + m) return f + 8 * (r - R);
        R += m;
    }
    return -1;     // r >= n: not reached for ranks of the class
}

__global__ __launch_bounds__(kOrderBlk) void k_order_place(const int2* __restrict__ ranges, int64_t n_tiles,
                                                           const int32_t* __restrict__ base,
                                                           const int32_t* __restrict__ cls,
                                                           int32_t* __restrict__ order) {
    __shared__ uint32_t s_hist[kOrderBlk / 64][kOrderClasses];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int c = lane; c < kOrderClasses; c += 64) s_hist[wid][c] = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kOrderBlk + threadIdx.x;
    const bool active = t < n_tiles;
    int c = 0;
    if (active) {
        const int2 r = ranges[t];
        c = order_class(r.y - r.x);
    }
    // rank among the lanes of this wave with the same class, then among earlier waves
    const uint64_t peers = match_digit<6>((uint32_t)c, active);
    const uint32_t below = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
    if (active && below == 0) s_hist[wid][c] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (!active) return;
    uint32_t rank = below;
    for (int w = 0; w < wid; w++) rank += s_hist[w][c];
    const int64_t o = cls[c], n = cls[kOrderClasses + c];
    const int64_t r = (int64_t)base[(int64_t)blockIdx.x * kOrderClasses + c] - o + rank;
    const int64_t slot = order_slot(o, n, r);
    if (slot >= 0 && slot < n_tiles) order[slot] = (int32_t)t;
}

hipError_t launch_tile_order(const int32_t* ranges, int64_t n_tiles, int32_t* cnt, int32_t* base, int32_t* cls,
                             int32_t* order, hipStream_t s) {
    if (!order || n_tiles == 0) return hipSuccess;
    const int64_t groups = ceil_div(n_tiles, kOrderBlk);
    const int2* rg = reinterpret_cast<const int2*>(ranges);
    k_order_count<<<(unsigned)groups, kOrderBlk, 0, s>>>(rg, n_tiles, cnt);
    k_order_scan<<<1, 1024, 0, s>>>(cnt, groups, base, cls);
    k_order_place<<<(unsigned)groups, kOrderBlk, 0, s>>>(rg, n_tiles, base, cls, order);
    return hipGetLastError();
}

}  // namespace

// ---------------------------------------------------------------- generic stable pair sort
// The same LSD passes for other parts of the library: n (read on the device,
// at most cap) uint32 keys whose low `bits` bits matter, with int32 values,
// ping-ponged between the two buffer pairs; *out_keys / *out_vals name the
// pair that holds the result.  cleared: an earlier kernel has run the words'
// SortClear (sort_pairs_clear), where there is anything to sort.
size_t sort_pairs_ws_bytes(int64_t cap, int bits) {
    return os_ws_bytes(cap, digit_plan(bits, kDepthDigitBits));
}

SortClear sort_pairs_clear(int64_t cap, int bits, void* ws) {
    const DigitPlan pl = digit_plan(bits, kDepthDigitBits);
    return sort_clear(os_carve(cap, pl, (char*)ws), pl);
}

hipError_t sort_pairs(uint32_t* keys, int32_t* vals, uint32_t* keys_alt, int32_t* vals_alt, const int64_t* n_dev,
                      int64_t cap, int bits, void* ws, bool cleared, uint32_t** out_keys, int32_t** out_vals,
                      hipStream_t s) {
    const DigitPlan pl = digit_plan(bits, kDepthDigitBits);
    const OsWs w = os_carve(cap, pl, (char*)ws);
    const hipError_t e = onesweep_sort(pl, keys, vals, keys_alt, vals_alt, n_dev, cap, w, true, false, cleared, false, s);
    const bool even = pl.passes % 2 == 0;
    *out_keys = even ? keys : keys_alt;
    *out_vals = even ? vals : vals_alt;
    return e;
}

size_t sort_ws_bytes(const pg_views* v, int64_t cap) {
    size_t total = 0;
    carve(v, cap, nullptr, &total);
    return total;
}

hipError_t launch_bin_sort(const pg_views* v, const pg_bin* bins, const pg_tile_set* tiles, int64_t cap,
                           uint32_t* keys, int32_t* values,
                           int32_t* ranges, int32_t* tile_order, int32_t* inst_first, int64_t* n_inst_dev,
                           int32_t* overflow_dev, void* ws, hipStream_t s) {
    const SortPlan pl = plan_for(v, cap);
    SortWs w = carve(v, cap, ws, nullptr);
    const int64_t nb = n_blocks(v);
    hipError_t e = hipSuccess;
    const SortCount post{n_inst_dev, cap, overflow_dev, w.misc, nullptr, nullptr};
    if (v->n_gv == 0) {
        e = fill_u32(ranges, 0u, 2 * v->n_tiles, s);
        if (e != hipSuccess) return e;
        e = fill_u32(n_inst_dev, 0u, 2, s);
        if (e != hipSuccess) return e;
        k_sort_count<<<1, 1, 0, s>>>(post);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_tile_order(ranges, v->n_tiles, w.order_cnt, w.order_base, w.order_cls, tile_order, s);
    }
    // 1. compact surviving records in (view, id) order, keyed by depth; slot offsets in the same order
    // (the count clears the tile ranges on its way and, with few records, the record sort's
    // words, with groups of its own when there is more to clear than the records' groups would)
    const bool short_scan = nb <= kScanShort, few = short_scan && !pl.segs;
    const OsWs dws = os_carve(v->n_gv, pl.depth, w.os, w.rec_seg, pl.segs);
    const SortClear dclear = few ? sort_clear(dws, pl.depth) : SortClear{};
    const int64_t clear_groups = imin(ceil_div(2 * v->n_tiles + dclear.status_words, 4 * kBlk), 256);
    k_valid_count<<<(unsigned)imax(nb, clear_groups), kWalk, 0, s>>>(bins, v->n_gv, nb, w.blk_a, w.blk_b, dclear,
                                                                    reinterpret_cast<uint32_t*>(ranges),
                                                                    2 * v->n_tiles);
    if (short_scan) {
        e = scan_short_i64({w.blk_a, w.blk_a_off, w.misc + 0}, {w.blk_b, w.blk_b_off, w.misc + 4}, nb, {}, s);
    } else {
        e = scan_i64(w.blk_a, w.blk_a_off, nullptr, 0, nb, w.misc + 0, w.scan_tmp, s);
        if (e != hipSuccess) return e;
        e = scan_i64(w.blk_b, w.blk_b_off, nullptr, 0, nb, w.misc + 4, w.scan_tmp, s);
    }
    if (e != hipSuccess) return e;
    if (pl.segs) {
        os_clear(pl.depth, w.misc + 0, dws, s);
        const int32_t run = (int32_t)imax(2, ceil_div(nb, 2048));    // groups of records per work-group
        k_compact<true><<<(unsigned)ceil_div(nb, run), kWalk, 0, s>>>(
            bins, v->n_gv, w.blk_a_off, w.blk_b_off, w.rk0, w.rv0, inst_first, nb, run, w.rec_seg, w.inst_seg,
            v->n_gauss, dws.hist);
        k_seg_tiles<<<1, kMaxSegs, 0, s>>>(v->d_views, pl.segs, w.misc, kSortTile, w.rec_seg, w.inst_seg);
    } else {
        k_compact<false><<<(unsigned)nb, kWalk, 0, s>>>(bins, v->n_gv, w.blk_a_off, w.blk_b_off, w.rk0, w.rv0,
                                                        inst_first, nb, 1, nullptr, nullptr, v->n_gauss, nullptr);
    }
    // 2. stable LSD sort of the records by depth
    // (when the last digit is one value for every key, that pass moves nothing: the
    // records stay in the buffer the pass before wrote, and its flag says so)
    e = onesweep_sort(pl.depth, w.rk0, w.rv0, w.rk1, w.rv1, w.misc + 0, v->n_gv, dws, true, true, few, pl.segs != 0, s);
    if (e != hipSuccess) return e;
    const int32_t* rva = pl.depth.passes % 2 == 0 ? w.rv0 : w.rv1;
    const int32_t* rvb = pl.depth.passes % 2 == 0 ? w.rv1 : w.rv0;
    const uint32_t* stayed = dws.uni + pl.depth.passes - 1;
    // 3. instance offsets in sorted-record order; overflow check
    k_sorted_count<<<(unsigned)nb, kBlk, 0, s>>>(tiles, rva, rvb, stayed, w.misc, w.blk_a, w.stiles);
    SortCount count = post;
    count.err = dws.err;
    count.stayed = stayed;
    if (short_scan) {
        e = scan_short_i64({w.blk_a, w.blk_a_off, nullptr}, {}, nb, count, s);
        if (e != hipSuccess) return e;
    } else {
        e = scan_i64(w.blk_a, w.blk_a_off, nullptr, 0, nb, n_inst_dev, w.scan_tmp, s);
        if (e != hipSuccess) return e;
        k_sort_count<<<1, 1, 0, s>>>(count);
    }
    // 4. emit (tile, gv) in record order into the buffer that makes the last tile pass land in the caller's arrays
    const bool even = pl.tile.passes % 2 == 0;
    uint32_t* ta = even ? keys : w.tk_alt;
    int32_t* tva = even ? values : w.tv_alt;
    uint32_t* tb = even ? w.tk_alt : keys;
    int32_t* tvb = even ? w.tv_alt : values;
    // (and clear the tile sort's words when few: its workspace overlaps the record sort's, whose
    // error and flag the count has taken)
    const OsWs tws = os_carve(cap, pl.tile, w.os, w.inst_seg, pl.segs);
    k_emit<<<(unsigned)nb, kBlk, 0, s>>>(w.stiles, rva, rvb, v->n_gauss, v->d_views, w.blk_a_off, w.misc, ta, tva,
                                         few ? sort_clear(tws, pl.tile) : SortClear{}, pl.tile.passes,
                                         1 << pl.tile.digit, tws.tile);
    // 5. stable LSD sort of the instances by tile id
    e = onesweep_sort(pl.tile, ta, tva, tb, tvb, w.misc + 1, cap, tws, false, false, few, false, s);
    if (e != hipSuccess) return e;
    k_ranges<<<(unsigned)imax(1, imin(kRangeGrid, ceil_div(cap, 256))), 256, 0, s>>>(keys, w.misc, ranges, tws.err,
                                                                                     overflow_dev);
    return launch_tile_order(ranges, v->n_tiles, w.order_cnt, w.order_base, w.order_cls, tile_order, s);
}

}  // namespace pg
