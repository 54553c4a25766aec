// UV-based pruning (Sec. 4.2 "UV-Based Pruning"; UV projection equation of
// Sec. 3).  A Gaussian's position in spherical coordinates gives its UV pixel
//   u = floor((pi + atan2(y, x)) / (2 pi) M),  v = floor(acos(z / rho) / pi N)
// (FP64; theta = pi wraps to u = 0, phi = pi stays in the last row, rho = 0
// is invalid).  Valid UV projection: with the pixel of the storing texel
// given, a Gaussian that maps elsewhere is invalid.  Max-K: per frame and
// pixel, the K valid Gaussians of highest opacity are kept (by the logit,
// which orders like the opacity; ties by ascending id).
//
// Pixel lists: the key kernel counts each pixel's Gaussians and gives each a place in
// its pixel's list (in any order), a running count places the lists, and a
// Gaussian's rank is the number of entries of its list that come before it.
// That is one pass over the Gaussians instead of seven, as long as lists are
// short.  Maps on which they are not expected to be are left to the sorts, and where
// the counts show it a flag is raised on the device and the sorts take over:
//
// a segmented top-K by two stable radix sorts of (key, index) pairs, first by
// the opacity (largest first), then by (frame, pixel), so each pixel's run
// comes out ordered by opacity and then id; a Gaussian's rank is its distance
// from the start of its run.  Without the flag they find no pairs and each of
// their launches ends at once (about 2 us).  1.26 M Gaussians of two frames, 5 a
// pixel: 160 us against 234 by the sorts, 4 k to 90 k Gaussians 48 to 52 against 60
// to 101 (the sorts with their words cleared by the kernels before them; 240, and 87
// to 121 without).
#include "pg_internal.h"

namespace pg {

namespace {

constexpr int kT = 256;
// A Gaussian compares itself with its whole list, so the lists cost a base and the sum of
// the squares of their lengths, about 4.5 us a million comparisons; the sorts cost the
// same for any lengths.  Limits from even maps of 1 to 128 Gaussians a pixel, lists / sorts,
// us: 4 k Gaussians 32 a pixel 46 / 55, 64 56 / 55, 128 70 / 56; 90 k 64 69 / 92, 128
// 94 / 92; 260 k 32 85 / 130; 1.26 M 16 210 / 235, 20 233 / 213; 2 M 5 264 / 313, 10
// 314 / 314; 4 M 1 531 / 506.  Empty pixels are cleared and placed too: 90 k Gaussians on
// 2.9 M pixels 82 / 105, on 5.8 M 115 / 104; 1.26 M on 3.8 M 212 / 240, on 10 M 286 / 248.
// Once the lists are counted the way to the sorts costs 15 to 60 us more (150 where
// hundreds of pixels are crowded), so that limit
// allows twice as many comparisons for few Gaussians.
constexpr int kUvList = 256;                            // longest list that one Gaussian walks
constexpr int64_t kUvWork = (1 << 24) + (1 << 23);      // most comparisons in all
constexpr int64_t kUvWorkEach = 64, kUvWorkCounted = 128;  // ... and per Gaussian, as expected and as counted
constexpr int64_t kUvMost = 1 << 21;                    // most Gaussians of all frames ...
constexpr int64_t kUvPixels = 1 << 22;                  // ... and most pixels of all frames

__host__ __device__ __forceinline__ int64_t uv_work(int64_t n, int64_t each) {
    return each * n < kUvWork ? each * n : kUvWork;
}

// float -> uint32 whose ascending order is the float's descending order
// (-0 counts as +0, as in a float comparison)
__device__ __forceinline__ uint32_t desc_key(float x) {
    if (x == 0.0f) x = 0.0f;
    const uint32_t b = __float_as_uint(x);
    const uint32_t asc = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return ~asc;
}

// cnt[0]: records; cnt[1]: records to sort (lists: none until a list is too long);
// cnt[2]: list entries given out (low word) and the lists' comparisons (high word).  And
// the pixels' counts, cleared.
__global__ __launch_bounds__(kT) void k_uv_init(const int64_t* __restrict__ n_dev, int64_t n_cap, int32_t F, int lists,
                                                int64_t* __restrict__ cnt, int32_t* __restrict__ count,
                                                int64_t pixels) {
    const int64_t i0 = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (i0 == 0) {
        const int64_t n = (int64_t)F * imin(*n_dev, n_cap);
        cnt[0] = n;
        cnt[1] = lists ? 0 : n;
        cnt[2] = 0;
    }
    if (lists)
        for (int64_t i = i0; i < pixels; i += (int64_t)gridDim.x * kT) count[i] = 0;
}

// A work-group counts its Gaussians in an LDS table of pixels first and adds each pixel's
// number to the pixel's count once: additions to one address take 11 ns each, and a map
// may have most of its Gaussians in a few pixels (1.26 M Gaussians, all in one pixel:
// 13,960 -> 260 us for the call, half of them in 200: 620 -> 398; the sorts alone 209 and
// 236; with 1,024 Gaussians a group 235 and 390, but 164 against 160 on an even map).  Once a
// list is known to be too long the counts are of no use and are left alone.
constexpr int kKey = 256;
__global__ __launch_bounds__(kKey) void k_uv_key(const float* __restrict__ params, const int64_t* __restrict__ n_dev,
                                               int64_t n_cap, int32_t F, int32_t C, int32_t M, int32_t Nv,
                                               const int32_t* __restrict__ expected, int32_t* __restrict__ uv,
                                               uint32_t* __restrict__ okey, int32_t* __restrict__ oval,
                                               int32_t* __restrict__ count, int32_t* __restrict__ slot,
                                               int64_t* __restrict__ cnt) {
    constexpr int kTable = 2 * kKey;
    __shared__ int32_t s_pixel[kTable], s_count[kTable];
    __shared__ int32_t s_listed, s_long;
    const int64_t n = imin(*n_dev, n_cap);
    const int64_t j = (int64_t)blockIdx.x * kKey + threadIdx.x;
    if ((int64_t)blockIdx.x * kKey >= (int64_t)F * n) return;
    const bool has = j < (int64_t)F * n;
    if (count) {
        if (threadIdx.x == 0) s_long = 0;
        for (int k = threadIdx.x; k < kTable; k += kKey) {
            s_pixel[k] = -1;
            s_count[k] = 0;
        }
    }
    int32_t key = -1, f = 0;
    int64_t g = 0;
    if (has) {
        f = (int32_t)(j / n);
        const int64_t i = j - (int64_t)f * n;
        const float* P = params + (int64_t)f * C * n_cap + i;
        const double x = P[0], y = P[n_cap], z = P[2 * n_cap];
        const double rho = sqrt((x * x + y * y) + z * z);
        if (rho > 0.0) {
            const double theta = atan2(y, x);
            double c = z / rho;
            c = c > 1.0 ? 1.0 : (c < -1.0 ? -1.0 : c);
            const double phi = acos(c);
            int64_t u = (int64_t)floor((3.141592653589793 + theta) / (2.0 * 3.141592653589793) * (double)M);
            int64_t v = (int64_t)floor(phi / 3.141592653589793 * (double)Nv);
            if (u >= M) u -= M;
            if (v >= Nv) v = Nv - 1;
            key = (int32_t)(v * M + u);
            if (expected && expected[(int64_t)f * n_cap + i] != key) key = -1;
        }
        g = (int64_t)f * n_cap + i;
        uv[g] = key;
        okey[j] = key >= 0 ? desc_key(P[10 * n_cap]) : 0xFFFFFFFFu;
        oval[j] = (int32_t)g;
    }
    if (!count) return;
    if (threadIdx.x == 0) s_listed = __hip_atomic_load(&cnt[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    __syncthreads();
    if (!s_listed) return;
    // the Gaussian's place in its pixel's list: which one it gets does not matter
    const int32_t pixel = f * M * Nv + key;
    uint32_t h = 0;
    int32_t at = 0;
    if (key >= 0) {
        // at most kKey of the table's entries are ever taken, so the walk ends
        h = ((uint32_t)pixel * 2654435761u) % kTable;
        for (;; h = (h + 1) % kTable) {
            const int32_t was = atomicCAS(&s_pixel[h], -1, pixel);
            if (was == -1 || was == pixel) break;
        }
        at = atomicAdd(&s_count[h], 1);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kTable; k += kKey) {
        const int32_t mine = s_count[k];
        if (mine == 0) continue;
        const int32_t before = atomicAdd(&count[s_pixel[k]], mine);
        s_count[k] = before;
        if (before + mine > kUvList) s_long = 1;
    }
    __syncthreads();
    if (key >= 0) slot[g] = at + s_count[h];
    if (threadIdx.x == 0 && s_long)      // every writer stores the same value
        __hip_atomic_store(&cnt[1], cnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Each pixel's list: its first entry and its length.  Which pixels' lists lie first does
// not matter, so a group of pixels takes its entries from a running count and no scan over
// all pixels is needed (three launches).
constexpr int kPlace = 1024;
__global__ __launch_bounds__(kPlace) void k_uv_place(int64_t* __restrict__ cnt, const int32_t* __restrict__ count,
                                                     int64_t pixels, int2* __restrict__ place) {
    __shared__ int32_t s_wave[kPlace / 64], s_work[kPlace / 64];
    __shared__ int32_t s_base;
    if (cnt[1]) return;
    const int64_t p = (int64_t)blockIdx.x * kPlace + threadIdx.x;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t c = p < pixels ? count[p] : 0;
    int32_t incl = c, sq = c * c;       // c <= kUvList here, so the words do not overflow
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t x = __shfl_up(incl, o, 64);
        if (lane >= o) incl += x;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 63) {
        s_wave[wid] = incl;
        s_work[wid] = sq;
    }
    __syncthreads();
    int32_t before = 0, total = 0;
    uint32_t work = 0;
    for (int w = 0; w < kPlace / 64; w++) {
        if (w < wid) before += s_wave[w];
        total += s_wave[w];
        work += (uint32_t)s_work[w];
    }
    if (threadIdx.x == 0)
        s_base = total ? (int32_t)atomicAdd(reinterpret_cast<unsigned long long*>(&cnt[2]),
                                            (unsigned long long)work << 32 | (uint32_t)total) : 0;
    __syncthreads();
    if (p < pixels) place[p] = make_int2(s_base + before + incl - c, c);
}

// The lists: opacity key (high) and Gaussian of every valid record at its place, so
// that entries in ascending order are in rank order (ties by ascending id).
// Where they would take too many comparisons, the ranks are left to the sorts.
__global__ __launch_bounds__(kT) void k_uv_scatter(int64_t* __restrict__ cnt, int64_t n_cap, int32_t M,
                                                   int32_t Nv, const uint32_t* __restrict__ okey,
                                                   const int32_t* __restrict__ oval, const int32_t* __restrict__ uv,
                                                   const int32_t* __restrict__ slot, const int2* __restrict__ place,
                                                   uint64_t* __restrict__ list) {
    const int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (j >= cnt[0]) return;
    if ((int64_t)((uint64_t)cnt[2] >> 32) > uv_work(cnt[0], kUvWorkCounted)) {
        if (j == 0) cnt[1] = cnt[0];
        return;
    }
    if (cnt[1]) return;      // a list is too long (nobody sets it here then)
    const int32_t g = oval[j], u = uv[g];
    if (u < 0) return;
    list[(int64_t)place[(g / n_cap) * M * Nv + u].x + slot[g]] = (uint64_t)okey[j] << 32 | (uint32_t)g;
}

__global__ __launch_bounds__(kT) void k_uv_list_rank(const int64_t* __restrict__ cnt, int64_t n_cap, int32_t M,
                                                     int32_t Nv, const uint32_t* __restrict__ okey,
                                                     const int32_t* __restrict__ oval, const int32_t* __restrict__ uv,
                                                     const int2* __restrict__ place,
                                                     const uint64_t* __restrict__ list, int32_t K, SortClear clear,
                                                     int32_t* __restrict__ rank, uint8_t* __restrict__ keep) {
    const int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (cnt[1]) {       // left to the sorts: their first one's words
        clear.run(clear.status_words, j, (int64_t)gridDim.x * kT);
        return;
    }
    if (j >= cnt[0]) return;
    const int32_t g = oval[j], u = uv[g];
    int32_t r = -1;
    if (u >= 0) {
        const int2 at = place[(g / n_cap) * M * Nv + u];
        const uint64_t mine = (uint64_t)okey[j] << 32 | (uint32_t)g;
        const int32_t e0 = at.x, end = at.x + at.y;
        r = 0;
        for (int32_t e = e0; e < end; e += 4) {         // four entries in flight
            uint64_t x[4];
#pragma unroll
            for (int q = 0; q < 4; q++) x[q] = e + q < end ? list[e + q] : ~0ull;
#pragma unroll
            for (int q = 0; q < 4; q++) r += x[q] < mine ? 1 : 0;
        }
    }
    rank[g] = r;
    keep[g] = r >= 0 && r < K ? 1 : 0;
}

// records in opacity order -> (frame, pixel) keys; invalid ones get F M Nv
__global__ __launch_bounds__(kT) void k_uv_emit(const int32_t* __restrict__ oval, const int64_t* __restrict__ cnt,
                                                int64_t n_cap, int32_t M, int32_t Nv, int32_t F,
                                                const int32_t* __restrict__ uv, SortClear clear,
                                                uint32_t* __restrict__ pkey, int32_t* __restrict__ pval) {
    const int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (cnt[0] && clear.err) clear.run(clear.status_words, j, (int64_t)gridDim.x * kT);    // the second sort's words
    if (j >= cnt[0]) return;
    const int32_t g = oval[j];
    const int32_t f = (int32_t)(g / n_cap);
    const int32_t u = uv[g];
    pkey[j] = u >= 0 ? (uint32_t)((int64_t)f * M * Nv + u) : (uint32_t)((int64_t)F * M * Nv);
    pval[j] = g;
}

__global__ __launch_bounds__(kT) void k_uv_start(const uint32_t* __restrict__ pkey, const int64_t* __restrict__ cnt,
                                                 int32_t* __restrict__ start) {
    const int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (j >= cnt[0]) return;
    if (j == 0 || pkey[j] != pkey[j - 1]) start[pkey[j]] = (int32_t)j;
}

__global__ __launch_bounds__(kT) void k_uv_rank(const uint32_t* __restrict__ pkey, const int32_t* __restrict__ pval,
                                                const int64_t* __restrict__ cnt, const int32_t* __restrict__ start,
                                                uint32_t sentinel, int32_t K, int32_t* __restrict__ rank,
                                                uint8_t* __restrict__ keep) {
    const int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (j >= cnt[0]) return;
    const uint32_t key = pkey[j];
    const int32_t g = pval[j];
    if (key == sentinel) {
        rank[g] = -1;
        keep[g] = 0;
        return;
    }
    const int32_t r = (int32_t)j - start[key];
    rank[g] = r;
    keep[g] = r < K ? 1 : 0;
}

int key_bits_for(int64_t n_keys) {
    int b = 1;
    while (((int64_t)1 << b) < n_keys) b++;
    return b;
}

struct UvWs {
    int64_t* cnt;
    uint32_t *ka, *kb;
    int32_t *va, *vb, *start;
    int2* place;
    void* sort_ws;
};

UvWs carve_uv(int64_t n_cap, int32_t F, int32_t M, int32_t Nv, void* ws, size_t* total) {
    const int64_t n = imax((int64_t)F * n_cap, 1);
    char* p = (char*)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* q = p + off;
        off += align256(bytes);
        return q;
    };
    UvWs w{};
    w.cnt = (int64_t*)take(24);
    w.ka = (uint32_t*)take(n * 4);
    w.va = (int32_t*)take(n * 4);
    w.kb = (uint32_t*)take(n * 4);      // kb and vb together also hold the lists' 8-byte entries
    w.vb = (int32_t*)take(n * 4);
    w.start = (int32_t*)take(((int64_t)F * M * Nv + 1) * 4);
    w.place = (int2*)take((int64_t)F * M * Nv * 8);     // also where lists are not tried: fewer Gaussians need no more
    const int bits = imax(32, key_bits_for((int64_t)F * M * Nv + 1));
    w.sort_ws = take(sort_pairs_ws_bytes(n, bits));
    if (total) *total = off;
    return w;
}

}  // namespace

size_t uv_prune_ws_bytes(int64_t n_cap, int32_t F, int32_t M, int32_t Nv) {
    size_t total = 0;
    carve_uv(n_cap, F, M, Nv, nullptr, &total);
    return total;
}

hipError_t launch_uv_prune(const float* params, const int64_t* n_dev, int64_t n_cap, int32_t F, int32_t C, int32_t M,
                           int32_t Nv, int32_t K, const int32_t* expected, int32_t* uv, int32_t* rank, uint8_t* keep,
                           void* ws, hipStream_t s) {
    UvWs w = carve_uv(n_cap, F, M, Nv, ws, nullptr);
    const int64_t n = (int64_t)F * n_cap;
    const int64_t pixels = (int64_t)F * M * Nv;
    // lists where they are expected to pay: Gaussians spread evenly over the pixels
    const bool lists = n <= kUvMost && pixels <= kUvPixels && n + n * n_cap / ((int64_t)M * Nv) <= uv_work(n, kUvWorkEach);
    k_uv_init<<<lists ? (unsigned)imin(ceil_div(pixels, kT), 1024) : 1u, kT, 0, s>>>(n_dev, n_cap, F, lists, w.cnt,
                                                                                     w.start, pixels);
    if (n == 0) return hipGetLastError();
    const unsigned grid = (unsigned)ceil_div(n, kT);
    const int pixel_bits = key_bits_for(pixels + 1);
    hipError_t e = hipSuccess;
    k_uv_key<<<(unsigned)ceil_div(n, kKey), kKey, 0, s>>>(params, n_dev, n_cap, F, C, M, Nv, expected, uv, w.ka, w.va,
                                                          lists ? w.start : nullptr, rank, w.cnt);
    if (lists) {
        k_uv_place<<<(unsigned)ceil_div(pixels, kPlace), kPlace, 0, s>>>(w.cnt, w.start, pixels, w.place);
        k_uv_scatter<<<grid, kT, 0, s>>>(w.cnt, n_cap, M, Nv, w.ka, w.va, uv, rank, w.place, (uint64_t*)w.kb);
        k_uv_list_rank<<<grid, kT, 0, s>>>(w.cnt, n_cap, M, Nv, w.ka, w.va, uv, w.place, (const uint64_t*)w.kb, K,
                                           sort_pairs_clear(n, 32, w.sort_ws), rank, keep);
    }
    // records to sort: all of them, or none when the lists have ranked them
    const int64_t* left = w.cnt + 1;
    uint32_t* ok;
    int32_t* ov;
    e = sort_pairs(w.ka, w.va, w.kb, w.vb, left, n, 32, w.sort_ws, lists, &ok, &ov, s);
    if (e != hipSuccess) return e;
    // the pixel keys go to the pair the opacity order does not occupy
    uint32_t* pk = ok == w.ka ? w.kb : w.ka;
    int32_t* pv = ov == w.va ? w.vb : w.va;
    k_uv_emit<<<grid, kT, 0, s>>>(ov, left, n_cap, M, Nv, F, uv,
                                  lists ? sort_pairs_clear(n, pixel_bits, w.sort_ws) : SortClear{}, pk, pv);
    const uint32_t sentinel = (uint32_t)pixels;
    uint32_t* sk;
    int32_t* sv;
    e = sort_pairs(pk, pv, ok, ov, left, n, pixel_bits, w.sort_ws, lists, &sk, &sv, s);
    if (e != hipSuccess) return e;
    k_uv_start<<<grid, kT, 0, s>>>(sk, left, w.start);
    k_uv_rank<<<grid, kT, 0, s>>>(sk, sv, left, w.start, sentinel, K, rank, keep);
    return hipGetLastError();
}

}  // namespace pg
