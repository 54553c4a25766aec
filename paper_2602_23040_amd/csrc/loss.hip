// Objective terms of Sec. 4.2 "Objective": the photometric blend and the
// scale / opacity regularisers.
//
// Photometric objective:
//   L = (1 - lambda) mean |I - T| + lambda (1 - mean SSIM(I, T))
// over every view, pixel and channel, and its cotangent dL/dI, in one pass.
//
// SSIM per channel plane: local statistics under an 11 x 11 Gaussian window
// (sigma 1.5, weights summing to 1) with zero padding outside the view,
//   S = (2 a b + C1) (2 s_xy + C2) / ((a^2 + b^2 + C1) (s_x + s_y + C2)),
// a, b the window means, s_x, s_y, s_xy the window (co)variances,
// C1 = 0.01^2, C2 = 0.03^2.  Its gradient with respect to the image is the
// window correlation (the window is symmetric, so its own adjoint) of the
// partials P_a = dS/da, P_c = dS/dE[x^2], P_e = dS/dE[xy]:
//   dS/dx_q = (w * P_a)_q + 2 x_q (w * P_c)_q + y_q (w * P_e)_q.
//
// A wave streams down a strip of kStripCols columns of one channel, one row per
// step, and everything between the input and the cotangent stays in registers:
//  - the row's (x, y) goes to LDS, and each lane adds its 11 horizontal taps of x,
//    d = x - y, d^2 and x y (four window sums instead of five: s_x + s_y - 2 s_xy
//    is the variance of d; the products are formed per tap, since 16-byte rows
//    of them made LDS reads the limit, a fifth slower);
//  - vertical windows are running sums: a new row adds its term to the ten
//    windows under way and completes the oldest (acc[k] = acc[k + 1] + w h, one
//    multiply-add and no shift);
//  - the completed row's partial maps (zero outside the view, where no S is
//    taken) go through the same two steps and give the cotangent ten rows
//    above the input row.
// With s_d the variance of d and m its mean, D1 = N1 + m^2 and D2 = N2 + s_d for the
// numerators N1, N2 and denominators D1, D2 of S, so 1 - S = (N1 s_d + m^2 D2) / (D1 D2),
// 2 P_c + P_e = P_e s_d / D2 and
//   P_a = 2 ((N2 - N1) (a (1 - S) - m) - a S (s_d - m^2)) / (D1 D2),
//   dS/dx_q = (w * P_a)_q + x_q (w * (2 P_c + P_e))_q - d_q (w * P_e)_q:
// no term is a difference of large ones where the images are close, which is
// where a fit spends its time.
// x, y and d are shifted before they are multiplied (E[x~ y~] - a~ b~ with x~ = x - k
// equals the covariance, padding included, since the window sums to 1), which
// keeps FP32 cancellation small: d too, which is constant where both images are flat
// (with d as it is, a flat 0.2 against a flat 0.8 had 1e-4 of error in the SSIM term,
// 2e-8 shifted, and one view's loss at 2.0 against 0.5 5e-4).  Each lane's shift is a
// pixel of its own column, eight rows ahead, and moves every kRebase rows; the windows
// under way are then re-expressed in the new one.  (With 32 rows bands of flat colours
// up to 2 have seven times the error of 16.  One shift for the whole strip spares 33
// instructions a row and loses a digit in flat areas beside texture.)  Three waves, one per channel, share a work-group; per-strip sums
// of S and |I - T| (FP64) go to a small partial array that k_photo_final reduces.
//
// Bound by FP32 VALU issue, about 310 instructions per lane and row: the strip's
// 64 lanes give 54 columns and its rows run 20 ahead of the first output, 1.3
// times the work without halos.  16 views of 1024x768: 754 us by 32 x 32 blocks in
// LDS (every tap of both passes read from there), 433 by strips (414 before d was
// shifted); error against FP64 on images 0.05 from their targets 2e-6 and 7.7e-7.
#include "pg_internal.h"

#include <algorithm>
#include <utility>

namespace pg {

namespace {

constexpr int kR = 5;                       // window half-width
constexpr int kK = 2 * kR + 1;
constexpr int kLanes = 64;
constexpr int kStripCols = kLanes - 2 * kR; // output columns of a strip: a wave less the window's reach on both sides
constexpr int kStripMin = 16;               // least rows of a strip
constexpr int kChannels = 3;
constexpr int kRebase = 16;                 // rows between shifts of the base
constexpr int kB = 32;                      // output block side
constexpr int kIW = kB + 4 * kR;            // input patch side (42 + 10 = 52 with 2 halos)
constexpr int kMW = kB + 2 * kR;            // partial-map region side (42)
constexpr int kBlockThreads = 512;          // two output pixels per thread in the last pass
constexpr int64_t kBlockRound = 512;        // blocks the chip takes at once (two work-groups per CU)
static_assert(kB % kStripMin == 0 && kB <= kStripCols, "photo_sums");
constexpr float kC1 = 0.01f * 0.01f, kC2 = 0.03f * 0.03f;

struct Win {
    float w[kK];
};

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// LDS written by this wave's lanes is read by its other lanes: LDS operations of
// a wave run in order, so only the compiler has to keep them so.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// strips: kStripCols x rows pixels of every view, numbered per view row-major
// (ceil(W / kStripCols) x ceil(H / rows)) from strip_base[v]; a wave per channel.
__global__ __launch_bounds__(kChannels * kLanes) __attribute__((amdgpu_waves_per_eu(4))) void k_photo(
    const ViewDev* __restrict__ views, int nv, const int64_t* __restrict__ strip_base, int32_t rows,
    const float* __restrict__ image, const float* __restrict__ target, Win win, float lambda, double inv_n,
    float* __restrict__ dimg, double* __restrict__ partial) {
    constexpr int kIn = kLanes + 2 * kR;                     // input columns of a strip (74)
    __shared__ float2 s_in_all[kChannels][kIn];              // x, y
    __shared__ float4 s_map_all[kChannels][kIn];             // P_a, 2 P_c + P_e, P_e of lane l at l + kR
    __shared__ double s_sums[kChannels][2];
    const int64_t strip = blockIdx.x;
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (strip_base[mid] <= strip) lo = mid; else hi = mid - 1;
    }
    const ViewDev& V = views[lo];
    const int32_t W = V.W, H = V.H;
    const int32_t across = (W + kStripCols - 1) / kStripCols;
    const int64_t local = strip - strip_base[lo];
    const int32_t xs = (int32_t)(local % across) * kStripCols;
    const int lane = threadIdx.x % kLanes, ch = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int32_t y0 = (int32_t)(local / across) * rows;
    const int32_t y1 = min(y0 + rows, H);
    const int64_t HW = (int64_t)W * H;
    const float* X = image + 3 * V.pix_base + ch * HW;
    const float* Y = target + 3 * V.pix_base + ch * HW;
    float* D = dimg + 3 * V.pix_base + ch * HW;
    float2* s_in = s_in_all[ch];
    float4* s_map = s_map_all[ch];
    // lane l: input column xs - 10 + l (and, for l < 10, xs + 54 + l), map column
    // cx = xs - 5 + l; lanes 5 .. 58 own an output column, their cx
    const int32_t cx = xs - kR + lane;
    const int32_t ca = xs - 2 * kR + lane, cb = ca + kLanes;
    const bool in_a = ca >= 0 && ca < W, in_b = lane < 2 * kR && cb < W, in_map = cx >= 0 && cx < W;
    const bool own = lane >= kR && lane < kR + kStripCols && cx < W;
    // the next row's inputs, and the pixels whose cotangent completes there, loaded a row ahead
    float xa = 0.f, ya = 0.f, xb = 0.f, yb = 0.f, xo = 0.f, yo = 0.f;
    auto load_row = [&](int32_t r) __attribute__((always_inline)) {
        if (own && r - 2 * kR >= y0 && r - 2 * kR < y1) {
            const int64_t p = (int64_t)(r - 2 * kR) * W + cx;
            xo = X[p];
            yo = Y[p];
        }
        xa = ya = xb = yb = 0.f;
        if (r < 0 || r >= H) return;
        const int64_t p = (int64_t)r * W;
        if (in_a) {
            xa = X[p + ca];
            ya = Y[p + ca];
        }
        if (in_b) {
            xb = X[p + cb];
            yb = Y[p + cb];
        }
    };
    // running vertical windows: [k] completes after k + 1 more rows
    float va[2 * kR], vd[2 * kR], vq[2 * kR], vr[2 * kR];      // means of x, d, x y, d^2, shifted
    float ga[2 * kR], gf[2 * kR], ge[2 * kR];                  // blurred partial maps
#pragma unroll
    for (int k = 0; k < 2 * kR; k++) va[k] = vd[k] = vq[k] = vr[k] = ga[k] = gf[k] = ge[k] = 0.f;
    // a row's term into the running windows; returns the window it completes
    auto push = [&](float* v, float h) __attribute__((always_inline)) {
        const float out = fmaf(win.w[2 * kR], h, v[0]);
#pragma unroll
        for (int k = 0; k < 2 * kR - 1; k++)
            // three-operand form: the compiler's accumulate form leaves the sum in v[k + 1]'s register, and
            // every row then copies all seventy windows back
            asm("v_fma_f32 %0, %1, %2, %3" : "=v"(v[k]) : "s"(win.w[2 * kR - 1 - k]), "v"(h), "v"(v[k + 1]));
        v[2 * kR - 1] = win.w[0] * h;
        return out;
    };
    double s_sum = 0.0, l1_sum = 0.0;
    float kx = 0.f, kd = 0.f;        // the lane's shifts of x and d (of y: kx - kd)
    const double w_l1 = (double)(1.0f - lambda) * inv_n, w_ssim = (double)lambda * inv_n;
    auto rebase = [&](int32_t r) __attribute__((always_inline)) {
        const int64_t p = (int64_t)min(max(r + kRebase / 2, 0), H - 1) * W + min(max(cx, 0), W - 1);
        float nx = X[p], nd = nx - Y[p];
        // a pixel that is not finite spoils the windows that hold it; as a shift it would spoil all
        const bool finite = fabsf(nx) < INFINITY && fabsf(nd) < INFINITY;
        nx = finite ? nx : kx;
        nd = finite ? nd : kd;
        const float dx = nx - kx, dd = nd - kd, dy = dx - dd;
        // sum w (x~ - dx)(y~ - dy) = sum w x~ y~ - dx sum w y~ - dy sum w x~ + dx dy sum w,
        // and the square of d~ alike
        float wsum = 0.f;      // weights taken by window k
#pragma unroll
        for (int k = 2 * kR - 1; k >= 0; k--) {
            wsum += win.w[2 * kR - 1 - k];
            const float wx = va[k], wd = vd[k], wy = wx - wd;
            vq[k] = fmaf(dx, fmaf(dy, wsum, -wy), fmaf(-dy, wx, vq[k]));
            vr[k] = fmaf(dd, fmaf(dd, wsum, -2.0f * wd), vr[k]);
            vd[k] = fmaf(-dd, wsum, wd);
            va[k] = fmaf(-dx, wsum, wx);
        }
        kx = nx;
        kd = nd;
    };
    // input row r: the windows it completes (row r - 5)
    float ma, md, mq, mr, xv = 0.f, yv = 0.f;
    auto input_row = [&](int32_t r) __attribute__((always_inline)) {
        xv = xo;
        yv = yo;
        s_in[lane] = make_float2(xa, ya);
        if (lane < 2 * kR) s_in[kLanes + lane] = make_float2(xb, yb);
        wave_lds_order();
        load_row(r + 1);
        float ha = 0.f, hd = 0.f, hq = 0.f, hr = 0.f;
#pragma unroll
        for (int j = 0; j < kK; j++) {
            const float2 v = s_in[lane + j];
            const float w = win.w[j], x = v.x - kx, d = (v.x - v.y) - kd;
            ha = fmaf(w, x, ha);
            hd = fmaf(w, d, hd);
            hq = fmaf(w * x, x - d, hq);
            hr = fmaf(w, d * d, hr);
        }
        ma = push(va, ha);
        md = push(vd, hd);
        mq = push(vq, hq);
        mr = push(vr, hr);
    };
    // the completed windows' S and partial maps, and the cotangent they complete (row r - 10)
    auto output_row = [&](int32_t r) __attribute__((always_inline)) {
        const int32_t r1 = r - kR, r2 = r - 2 * kR;
        const bool out = own && r2 >= y0;
        float pa = 0.f, pf = 0.f, pe = 0.f;
        if (in_map && r1 >= 0 && r1 < H) {
            const float sd = mr - md * md, sxy = mq - ma * (ma - md);      // of the shifted means
            const float a = ma + kx, m = md + kd, b = a - m, m2 = m * m;
            const float N1 = 2.0f * a * b + kC1, N2 = 2.0f * sxy + kC2;
            const float D1 = N1 + m2, D2 = N2 + sd;
            const float DD = D1 * D2, rcp = __builtin_amdgcn_rcpf(DD);
            const float iD = fmaf(rcp, fmaf(-DD, rcp, 1.0f), rcp);        // one Newton step
            const float S = N1 * N2 * iD, U = fmaf(N1, sd, m2 * D2) * iD;     // S, 1 - S
            pe = 2.0f * N1 * iD;
            pf = pe * sd * (D1 * iD);
            pa = 2.0f * iD * fmaf(N2 - N1, fmaf(a, U, -m), -(a * S) * (sd - m2));
            if (own && r1 >= y0 && r1 < y1) s_sum += (double)S;
        }
        s_map[kR + lane] = make_float4(pa, pf, pe, 0.f);
        wave_lds_order();
        float ba = 0.f, bf = 0.f, be = 0.f;
#pragma unroll
        for (int j = 0; j < kK; j++) {
            const float4 v = s_map[lane + j];              // the outer lanes' taps are not theirs; they own no column
            const float w = win.w[j];
            ba = fmaf(w, v.x, ba);
            bf = fmaf(w, v.y, bf);
            be = fmaf(w, v.z, be);
        }
        const float qa = push(ga, ba), qf = push(gf, bf), qe = push(ge, be);
        if (out) {
            const float df = xv - yv;
            const float gs = fmaf(xv, qf, fmaf(-df, qe, qa));
            const float sg = df > 0.f ? 1.f : (df < 0.f ? -1.f : 0.f);
            D[(int64_t)r2 * W + cx] = (float)(w_l1 * (double)sg - w_ssim * (double)gs);
            l1_sum += (double)fabsf(df);
        }
    };
    const int32_t first = y0 - 2 * kR, last = y1 + 2 * kR;
    load_row(first);
    for (int32_t c0 = first; c0 < last; c0 += kRebase) {
        rebase(c0);
        int32_t r = c0;
        for (; r < y0; r++) {                              // windows of the first map row still under way
            input_row(r);
            wave_lds_order();      // its reads before the next row's store (in the rows below s_map's stand between)
        }
        for (; r < min(c0 + kRebase, last); r++) {
            input_row(r);
            output_row(r);
        }
    }
    const double ts = wave_sum_d(s_sum), tl = wave_sum_d(l1_sum);
    if (lane == 0) {
        s_sums[ch][0] = ts;
        s_sums[ch][1] = tl;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        partial[2 * strip + threadIdx.x] = (s_sums[0][threadIdx.x] + s_sums[1][threadIdx.x]) + s_sums[2][threadIdx.x];
}

// ---- small tables: one work-group of 512 threads per 32 x 32 pixel block of a
// view and one channel at a time (the next channel's inputs load while one is
// computed).  Everything stays in LDS: the inputs with a 10-pixel halo, their
// separable window sums over the 42 x 42 region the adjoint needs, the three
// partial maps there, and their separable blur back to the block.  The shift is
// the block's first pixel.
__device__ __forceinline__ double block_sum_d(double v, double* s_w) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) s_w[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < kBlockThreads / 64; k++) t += s_w[k];
    return t;
}

// blocks: one per 32 x 32 block of every view, numbered per view row-major
// (ceil(W/32) x ceil(H/32)) from blk_base[v].
__global__ __launch_bounds__(kBlockThreads) void k_photo_blocks(const ViewDev* __restrict__ views, int nv,
                                                                const int64_t* __restrict__ blk_base,
                                                                const float* __restrict__ image,
                                                                const float* __restrict__ target, Win win, float lambda,
                                                                double inv_n, float* __restrict__ dimg,
                                                                double* __restrict__ partial) {
    // LDS by lifetime: the input patch, then (over it) the partial maps; the
    // window sums, then (over them) the adjoint's horizontal blur.  65 KB, so
    // two work-groups share a CU.
    __shared__ float s_in[2 * kIW * kIW];
    __shared__ float s_h5[5 * kIW * kMW];
    __shared__ double s_w[kBlockThreads / 64];
    static_assert(3 * kMW * kMW <= 2 * kIW * kIW && 3 * kMW * kB <= 5 * kIW * kMW, "LDS aliasing");
    float* sx = s_in;
    float* sy = s_in + kIW * kIW;
    float (*h5)[kIW * kMW] = reinterpret_cast<float (*)[kIW * kMW]>(s_h5);
    float (*sm)[kMW * kMW] = reinterpret_cast<float (*)[kMW * kMW]>(s_in);
    float (*h3)[kMW * kB] = reinterpret_cast<float (*)[kMW * kB]>(s_h5);
    // view of this block (binary search over the per-view block bases)
    const int64_t blk = blockIdx.x;
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (blk_base[mid] <= blk) lo = mid; else hi = mid - 1;
    }
    const ViewDev& V = views[lo];
    const int32_t BX = (V.W + kB - 1) / kB;
    const int64_t local = blk - blk_base[lo];
    const int32_t x0 = (int32_t)(local % BX) * kB, y0 = (int32_t)(local / BX) * kB;
    const int64_t HW = (int64_t)V.W * V.H;
    const int t = threadIdx.x;
    double s_sum = 0.0, l1_sum = 0.0;
    // each thread's share of a channel's input patch, loaded one channel ahead
    constexpr int kPer = (kIW * kIW + kBlockThreads - 1) / kBlockThreads;
    float px[kPer], py[kPer];
    auto fetch = [&](int ch) __attribute__((always_inline)) {
        const float* X = image + 3 * V.pix_base + ch * HW;
        const float* Y = target + 3 * V.pix_base + ch * HW;
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            const int k = t + u * kBlockThreads;
            const int gx = x0 - 2 * kR + k % kIW, gy = y0 - 2 * kR + k / kIW;
            const bool in = k < kIW * kIW && gx >= 0 && gx < V.W && gy >= 0 && gy < V.H;
            const int64_t p = (int64_t)gy * V.W + gx;
            px[u] = in ? X[p] : 0.0f;
            py[u] = in ? Y[p] : 0.0f;
        }
    };
    fetch(0);
    for (int ch = 0; ch < 3; ch++) {
        const float* X = image + 3 * V.pix_base + ch * HW;
        const float* Y = target + 3 * V.pix_base + ch * HW;
        const float kx = X[(int64_t)y0 * V.W + x0], ky = Y[(int64_t)y0 * V.W + x0];
        __syncthreads();   // the previous channel is done with the LDS
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            const int k = t + u * kBlockThreads;
            if (k < kIW * kIW) {
                sx[k] = px[u] - kx;
                sy[k] = py[u] - ky;
            }
        }
        __syncthreads();
        if (ch < 2) fetch(ch + 1);   // in flight while this channel is computed
        // horizontal window sums: input rows x partial-map columns, two adjacent
        // columns per item (12 loads per input plane for 22 taps)
        for (int k = t; k < kIW * (kMW / 2); k += kBlockThreads) {
            const int r = k / (kMW / 2), c = 2 * (k % (kMW / 2));
            float a0 = 0.f, b0 = 0.f, c0 = 0.f, d0 = 0.f, e0 = 0.f;
            float a1 = 0.f, b1 = 0.f, c1 = 0.f, d1 = 0.f, e1 = 0.f;
            float xp = sx[r * kIW + c], yp = sy[r * kIW + c];
#pragma unroll
            for (int j = 0; j < kK; j++) {
                const float xn = sx[r * kIW + c + j + 1], yn = sy[r * kIW + c + j + 1], w = win.w[j];
                a0 = fmaf(w, xp, a0);
                b0 = fmaf(w, yp, b0);
                c0 = fmaf(w, xp * xp, c0);
                d0 = fmaf(w, yp * yp, d0);
                e0 = fmaf(w, xp * yp, e0);
                a1 = fmaf(w, xn, a1);
                b1 = fmaf(w, yn, b1);
                c1 = fmaf(w, xn * xn, c1);
                d1 = fmaf(w, yn * yn, d1);
                e1 = fmaf(w, xn * yn, e1);
                xp = xn;
                yp = yn;
            }
            const int o = r * kMW + c;
            h5[0][o] = a0;
            h5[1][o] = b0;
            h5[2][o] = c0;
            h5[3][o] = d0;
            h5[4][o] = e0;
            h5[0][o + 1] = a1;
            h5[1][o + 1] = b1;
            h5[2][o + 1] = c1;
            h5[3][o + 1] = d1;
            h5[4][o + 1] = e1;
        }
        __syncthreads();
        // vertical window sums on the partial-map region -> S and its partials,
        // two adjacent rows per item
        for (int k = t; k < (kMW / 2) * kMW; k += kBlockThreads) {
            const int r0 = 2 * (k / kMW), c = k % kMW;
            float m0[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, m1[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
            float prev[5];
#pragma unroll
            for (int q = 0; q < 5; q++) prev[q] = h5[q][r0 * kMW + c];
#pragma unroll
            for (int j = 0; j < kK; j++) {
                const float w = win.w[j];
#pragma unroll
                for (int q = 0; q < 5; q++) {
                    const float nx = h5[q][(r0 + j + 1) * kMW + c];
                    m0[q] = fmaf(w, prev[q], m0[q]);
                    m1[q] = fmaf(w, nx, m1[q]);
                    prev[q] = nx;
                }
            }
#pragma unroll
            for (int half = 0; half < 2; half++) {
                const float* m = half ? m1 : m0;
                const int r = r0 + half;
                const int gx = x0 - kR + c, gy = y0 - kR + r;
                float pa = 0.f, pc = 0.f, pe = 0.f;
                if (gx >= 0 && gx < V.W && gy >= 0 && gy < V.H) {
                    const float a = m[0] + kx, b = m[1] + ky;
                    const float vx = m[2] - m[0] * m[0], vy = m[3] - m[1] * m[1], cxy = m[4] - m[0] * m[1];
                    const float N1 = 2.0f * a * b + kC1, N2 = 2.0f * cxy + kC2;
                    const float D1 = a * a + b * b + kC1, D2 = vx + vy + kC2;
                    const float iD = 1.0f / (D1 * D2);
                    const float S = N1 * N2 * iD;
                    pa = 2.0f * b * (N2 - N1) * iD - S * (2.0f * a / D1 - 2.0f * a / D2);
                    pc = -S / D2;
                    pe = 2.0f * N1 * iD;
                    if (r >= kR && r < kR + kB && c >= kR && c < kR + kB) s_sum += (double)S;
                }
                sm[0][r * kMW + c] = pa;
                sm[1][r * kMW + c] = pc;
                sm[2][r * kMW + c] = pe;
            }
        }
        __syncthreads();
        // adjoint: blur the partial maps back to the block (horizontal, then
        // vertical), two adjacent columns per item
        for (int k = t; k < kMW * (kB / 2); k += kBlockThreads) {
            const int r = k / (kB / 2), c = 2 * (k % (kB / 2));
            float a0 = 0.f, c0 = 0.f, e0 = 0.f, a1 = 0.f, c1 = 0.f, e1 = 0.f;
            float pa = sm[0][r * kMW + c], pc = sm[1][r * kMW + c], pe = sm[2][r * kMW + c];
#pragma unroll
            for (int j = 0; j < kK; j++) {
                const float w = win.w[j];
                const int o = r * kMW + c + j + 1;
                const float na = sm[0][o], nc = sm[1][o], ne = sm[2][o];
                a0 = fmaf(w, pa, a0);
                c0 = fmaf(w, pc, c0);
                e0 = fmaf(w, pe, e0);
                a1 = fmaf(w, na, a1);
                c1 = fmaf(w, nc, c1);
                e1 = fmaf(w, ne, e1);
                pa = na;
                pc = nc;
                pe = ne;
            }
            const int o = r * kB + c;
            h3[0][o] = a0;
            h3[1][o] = c0;
            h3[2][o] = e0;
            h3[0][o + 1] = a1;
            h3[1][o + 1] = c1;
            h3[2][o + 1] = e1;
        }
        __syncthreads();
        for (int o = t; o < kB * kB; o += kBlockThreads) {
            const int tx = o % kB, ty = o / kB;
            float ga = 0.f, gc = 0.f, ge = 0.f;
#pragma unroll
            for (int j = 0; j < kK; j++) {
                const float w = win.w[j];
                ga = fmaf(w, h3[0][(ty + j) * kB + tx], ga);
                gc = fmaf(w, h3[1][(ty + j) * kB + tx], gc);
                ge = fmaf(w, h3[2][(ty + j) * kB + tx], ge);
            }
            const int gx = x0 + tx, gy = y0 + ty;
            if (gx < V.W && gy < V.H) {
                const int64_t p = (int64_t)gy * V.W + gx;
                const float xv = X[p], yv = Y[p];
                const float gs = ga + 2.0f * xv * gc + yv * ge;
                const float df = xv - yv;
                const float sg = df > 0.f ? 1.f : (df < 0.f ? -1.f : 0.f);
                dimg[3 * V.pix_base + ch * HW + p] =
                    (float)(((double)(1.0f - lambda) * sg - (double)lambda * gs) * inv_n);
                l1_sum += (double)fabsf(df);
            }
        }
    }
    const double ts = block_sum_d(s_sum, s_w);
    const double tl = block_sum_d(l1_sum, s_w);
    if (t == 0) {
        partial[2 * blk] = ts;
        partial[2 * blk + 1] = tl;
    }
}

__global__ __launch_bounds__(1024) void k_photo_final(const double* __restrict__ partial, int64_t n_blk,
                                                      float lambda, double inv_n, float* __restrict__ loss) {
    __shared__ double s_s[16], s_l[16];
    double ss = 0.0, sl = 0.0;
    for (int64_t i = threadIdx.x; i < n_blk; i += 1024) {
        ss += partial[2 * i];
        sl += partial[2 * i + 1];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        ss += __shfl_xor(ss, o, 64);
        sl += __shfl_xor(sl, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_s[threadIdx.x >> 6] = ss;
        s_l[threadIdx.x >> 6] = sl;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        ss = 0.0;
        sl = 0.0;
        for (int k = 0; k < 16; k++) {
            ss += s_s[k];
            sl += s_l[k];
        }
        *loss = (float)((1.0 - (double)lambda) * sl * inv_n + (double)lambda * (1.0 - ss * inv_n));
    }
}

// ---------------------------------------------------------------- regularisers
// Scale and opacity regularisers of the objective over the Gaussians of every
// frame (or the dynamic ones):  L_scale = mean max(0, max_k s_k - s_max)^2,
// L_opacity = mean o (1 - o), s = exp(l_s), o = sigmoid(l_o), in FP64 from
// the FP32 texel values.  Three kernels: block sums of (count, hinge^2,
// o (1 - o)); their total and the two means; the weighted gradients added to
// the texel gradient (l_s through exp on the largest scale's channel, l_o
// through the sigmoid), divided by the count.
constexpr int kRegThreads = 256;

struct RegTerms {
    int kmax;
    double smax, h, o;
};

__device__ __forceinline__ RegTerms reg_terms(const float* P, int64_t stride, double s_max) {
    RegTerms r;
    r.kmax = 0;
    r.smax = exp((double)P[3 * stride]);
    for (int k = 1; k < 3; k++) {
        const double sk = exp((double)P[(3 + k) * stride]);
        if (sk > r.smax) {
            r.smax = sk;
            r.kmax = k;
        }
    }
    r.h = r.smax > s_max ? r.smax - s_max : 0.0;
    r.o = 1.0 / (1.0 + exp(-(double)P[10 * stride]));
    return r;
}

__global__ __launch_bounds__(kRegThreads) void k_reg_sum(const float* __restrict__ params,
                                                         const int64_t* __restrict__ n_dev, int64_t n_cap,
                                                         int32_t F, int32_t C, const uint8_t* __restrict__ dyn,
                                                         double s_max, double* __restrict__ partial) {
    __shared__ double s_w[3][kRegThreads / 64];
    const int64_t n = imin(*n_dev, n_cap);
    double cnt = 0.0, hs = 0.0, os = 0.0;
    for (int64_t g = (int64_t)blockIdx.x * kRegThreads + threadIdx.x; g < (int64_t)F * n;
         g += (int64_t)gridDim.x * kRegThreads) {
        const int32_t f = (int32_t)(g / n);
        const int64_t i = g - (int64_t)f * n;
        if (dyn && !dyn[(int64_t)f * n_cap + i]) continue;
        const RegTerms r = reg_terms(params + (int64_t)f * C * n_cap + i, n_cap, s_max);
        cnt += 1.0;
        hs += r.h * r.h;
        os += r.o * (1.0 - r.o);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        cnt += __shfl_xor(cnt, o, 64);
        hs += __shfl_xor(hs, o, 64);
        os += __shfl_xor(os, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_w[0][threadIdx.x >> 6] = cnt;
        s_w[1][threadIdx.x >> 6] = hs;
        s_w[2][threadIdx.x >> 6] = os;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int w = 0; w < kRegThreads / 64; w++) t += s_w[threadIdx.x][w];
        partial[3 * blockIdx.x + threadIdx.x] = t;
    }
}

// partial[3 PG_REG_BLOCKS] <- the count; loss[0..1] <- the two means
__global__ void k_reg_final(double* __restrict__ partial, float* __restrict__ loss) {
    if (threadIdx.x != 0) return;
    double cnt = 0.0, hs = 0.0, os = 0.0;
    for (int b = 0; b < PG_REG_BLOCKS; b++) {
        cnt += partial[3 * b];
        hs += partial[3 * b + 1];
        os += partial[3 * b + 2];
    }
    partial[3 * PG_REG_BLOCKS] = cnt;
    loss[0] = cnt > 0.0 ? (float)(hs / cnt) : 0.0f;
    loss[1] = cnt > 0.0 ? (float)(os / cnt) : 0.0f;
}

__global__ __launch_bounds__(kRegThreads) void k_reg_grad(const float* __restrict__ params,
                                                          const int64_t* __restrict__ n_dev, int64_t n_cap,
                                                          int32_t F, int32_t C, const uint8_t* __restrict__ dyn,
                                                          const int32_t* __restrict__ gauss_texel, int64_t HW,
                                                          double s_max, double w_scale, double w_opacity,
                                                          const double* __restrict__ partial,
                                                          float* __restrict__ gatlas) {
    const int64_t n = imin(*n_dev, n_cap);
    const double cnt = partial[3 * PG_REG_BLOCKS];
    const int64_t g = (int64_t)blockIdx.x * kRegThreads + threadIdx.x;
    if (g >= (int64_t)F * n || cnt <= 0.0) return;
    const int32_t f = (int32_t)(g / n);
    const int64_t i = g - (int64_t)f * n;
    if (dyn && !dyn[(int64_t)f * n_cap + i]) return;
    const RegTerms r = reg_terms(params + (int64_t)f * C * n_cap + i, n_cap, s_max);
    float* out = gatlas + (int64_t)f * C * HW + gauss_texel[i];
    if (r.h > 0.0) out[(int64_t)(3 + r.kmax) * HW] += (float)(w_scale * (2.0 * r.h * r.smax) / cnt);
    out[10 * HW] += (float)(w_opacity * ((1.0 - 2.0 * r.o) * r.o * (1.0 - r.o)) / cnt);
}

}  // namespace

hipError_t launch_regularisers(const float* params, const int64_t* n_dev, int64_t n_cap, int32_t F, int32_t C,
                               const int32_t* gauss_texel, int64_t HW, const uint8_t* dyn, double s_max,
                               double w_scale, double w_opacity, float* gatlas, float* loss, double* partial,
                               hipStream_t s) {
    k_reg_sum<<<PG_REG_BLOCKS, kRegThreads, 0, s>>>(params, n_dev, n_cap, F, C, dyn, s_max, partial);
    k_reg_final<<<1, 64, 0, s>>>(partial, loss);
    if (n_cap > 0)
        k_reg_grad<<<(unsigned)ceil_div((int64_t)F * n_cap, kRegThreads), kRegThreads, 0, s>>>(
            params, n_dev, n_cap, F, C, dyn, gauss_texel, HW, s_max, w_scale, w_opacity, partial, gatlas);
    return hipGetLastError();
}

// Pairs of partial sums that hold any table's strips or blocks: strips of kStripMin rows are
// at most two for each block of 32 x 32 pixels they touch.
int64_t photo_sums(const pg_views* v) { return (int64_t)(kB / kStripMin) * v->n_ssim_blocks; }

// Rows of a strip, or 0 for the block kernel.  One round of its work-groups takes 27 us,
// while a strip cannot be done before its rows and the 20 it runs beside them.  Above that
// the height for which these fits of the measured times (us) are least: 1.6 to 1.75 ns a
// row when the chip is full (16 views of 1024x768, 32, 64 and 192 rows: 550, 482, 438), and
// at least a wave's way down its rows, 60 + 0.034 a strip for 52 of them (360: 68, 720: 83,
// 1,280: 106).  Heights 16 / 32 / 64 / 192, and blocks: 9 views of 256x256 59 / 67 / 96 / 241,
// 59; 3 of 640x480 74 / 83 / 108 / 242, 75; one of 1920x1080 130 / 103 / 132 / 241, 135; 12 of
// 512x512 190 / 170 / 137 / 276, 198; 130 of 108x832 643 / 498 / 445 / 490, 836; 30 of 1024x768
// 1,249 / 969 / 844 / 827, 1,405.  Narrow views leave most of a strip's columns idle: blocks
// would be faster there (200 views of 64x64 76 against 90), but have a tenth of the digits where
// images are close.
int32_t photo_strip_rows(const pg_camera* cams, int32_t n_views) {
    auto count = [&](int32_t v, int32_t cols, int32_t rows) {
        return ceil_div(cams[v].width, cols) * ceil_div(cams[v].height, rows);
    };
    int64_t blocks = 0;
    for (int32_t v = 0; v < n_views; v++) blocks += count(v, kB, kB);
    if (blocks <= kBlockRound) return 0;
    double best = 0.0;
    int32_t rows = 0;
    for (const auto& c : {std::make_pair(192, 1.72), {64, 1.62}, {32, 1.75}, {kStripMin, 1.75}}) {
        double n = 0.0, work = 0.0;
        int32_t longest = 0;
        for (int32_t v = 0; v < n_views; v++) {
            const int32_t steps = std::min(c.first, cams[v].height) + 4 * kR;
            n += (double)count(v, kStripCols, c.first);
            work += (double)count(v, kStripCols, c.first) * steps;
            longest = std::max(longest, steps);
        }
        const double t = std::max(1e-3 * c.second * work, (60.0 + 0.034 * n) * longest / 52.0);
        if (rows == 0 || t < best) {
            best = t;
            rows = c.first;
        }
    }
    return rows;
}
int64_t photo_groups(int32_t w, int32_t h, int32_t rows) {
    return rows ? ceil_div(w, kStripCols) * ceil_div(h, rows) : ceil_div(w, kB) * ceil_div(h, kB);
}

hipError_t launch_photo(const pg_views* v, const float* image, const float* target, float lambda, float* dimg,
                        float* loss, double* partial, hipStream_t s) {
    const int64_t nb = v->n_photo;
    if (nb == 0 || v->n_pixels == 0) return hipSuccess;
    Win win;
    double g[kK], sum = 0.0;
    for (int k = 0; k < kK; k++) {
        const double d = (double)(k - kR);
        g[k] = exp(-(d * d) / (2.0 * 1.5 * 1.5));
        sum += g[k];
    }
    for (int k = 0; k < kK; k++) win.w[k] = (float)(g[k] / sum);
    const double inv_n = 1.0 / (3.0 * (double)v->n_pixels);
    if (v->photo_rows)
        k_photo<<<(unsigned)nb, kChannels * kLanes, 0, s>>>(v->d_views, v->n_views, v->d_photo_base, v->photo_rows,
                                                            image, target, win, lambda, inv_n, dimg, partial);
    else
        k_photo_blocks<<<(unsigned)nb, kBlockThreads, 0, s>>>(v->d_views, v->n_views, v->d_photo_base, image, target,
                                                              win, lambda, inv_n, dimg, partial);
    k_photo_final<<<1, 1024, 0, s>>>(partial, nb, lambda, inv_n, loss);
    return hipGetLastError();
}

}  // namespace pg
