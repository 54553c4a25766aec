// a2 -- EWA projection of every Gaussian into every view of its frame, and
// (a5, second half) its adjoint back to the texel channels.
//
// Formulas: Sigma = R(q) diag(s)^2 R(q)^T; Sigma_c = W Sigma W^T; J the
// perspective Jacobian at the camera-space mean; Sigma2D = J Sigma_c J^T
// with +0.3 added to the diagonal; det / z validity test; lambda_max and the
// radius ceil(3 sqrt(lambda_max)) ("Covariance-Aware Gaussian Masking",
// Sec. 4.2, and Algorithm 1 steps 1-4); X_c = R X + t and the pixel mean
// (supplementary, viewer section); SH colour of the 3DGS record (Sec. 3).
//
// Every quantity that decides an integer (culls, radius, tile rectangle,
// depth key) is computed in FP64 from the FP32 texels in one fixed order:
// sums of products left to right in ascending index, no contraction (this
// file is compiled with -ffp-contract=off), IEEE division and square root.
// The outputs the compositing kernels read are rounded to FP32 once.
//
// Launch shape: the threads of a Gaussian of a frame read the texel record
// once and loop over the views of that frame, so a batched call reads the
// parameters once instead of once per view.  Work per (Gaussian, view) is ~800
// VALU instructions, most of them FP64, against 80 bytes written: bound by the
// issue and the latency of its FP64 chains (50 views, 14.0 M records: 830 ->
// 608 us with the edges facing the mean only in the tile tests, one barrier less
// per view and the split roles; 1.9 of the 4.8 TB/s a copy reaches).
//
// The adjoint runs as three passes: a streaming sum of each record's
// instance slots, the geometric chain in FP64 (position, scale, rotation,
// opacity), and the SH colour chain in FP32 (its 48 coefficient gradients and
// the view-direction term of the position gradient).  Splitting them keeps
// both under 256 registers without spills.
#include "pg_internal.h"

#pragma clang fp contract(off)

namespace pg {

namespace {

constexpr double kNearZ = 0.2;
constexpr double kLowPass = 0.3;
constexpr double kDetMin = 1e-7;

// Real SH normalisations (Condon-Shortley phase kept).
constexpr double kY0 = 0.28209479177387814;   // 1 / (2 sqrt(pi))
constexpr double kY1 = 0.4886025119029199;    // sqrt(3 / (4 pi))
constexpr double kY2a = 1.0925484305920792;   // sqrt(15 / pi) / 2
constexpr double kY2b = 0.31539156525252005;  // sqrt(5 / pi) / 4
constexpr double kY2c = 0.5462742152960396;   // sqrt(15 / pi) / 4
constexpr double kY3a = 0.5900435899266435;   // sqrt(35 / (2 pi)) / 4
constexpr double kY3b = 2.890611442640554;    // sqrt(105 / pi) / 2
constexpr double kY3c = 0.4570457994644658;   // sqrt(21 / (2 pi)) / 4
constexpr double kY3d = 0.3731763325901154;   // sqrt(7 / pi) / 4
constexpr double kY3e = 1.445305721320277;    // sqrt(105 / pi) / 4

template <int L>
__device__ __forceinline__ void sh_basis(double x, double y, double z, double* Y) {
    Y[0] = kY0;
    if (L >= 1) {
        Y[1] = -kY1 * y;
        Y[2] = kY1 * z;
        Y[3] = -kY1 * x;
    }
    if (L >= 2) {
        Y[4] = kY2a * x * y;
        Y[5] = -kY2a * y * z;
        Y[6] = kY2b * (3.0 * z * z - 1.0);
        Y[7] = -kY2a * x * z;
        Y[8] = kY2c * (x * x - y * y);
    }
    if (L >= 3) {
        Y[9] = -kY3a * y * (3.0 * x * x - y * y);
        Y[10] = kY3b * x * y * z;
        Y[11] = -kY3c * y * (5.0 * z * z - 1.0);
        Y[12] = kY3d * z * (5.0 * z * z - 3.0);
        Y[13] = -kY3c * x * (5.0 * z * z - 1.0);
        Y[14] = kY3e * z * (x * x - y * y);
        Y[15] = -kY3a * x * (x * x - 3.0 * y * y);
    }
}

// World-space part of the chain, shared by every view of a Gaussian.
struct World {
    double mu[3], s[3], qn, qh[4], o;
    double Rq[9], M[9], S[9];
};

__device__ __forceinline__ void world_chain(const float* rec, World& w) {
    w.mu[0] = rec[0]; w.mu[1] = rec[1]; w.mu[2] = rec[2];
    w.s[0] = exp((double)rec[3]); w.s[1] = exp((double)rec[4]); w.s[2] = exp((double)rec[5]);
    const double qw = rec[6], qx = rec[7], qy = rec[8], qz = rec[9];
    w.qn = sqrt(((qw * qw + qx * qx) + qy * qy) + qz * qz);
    w.qh[0] = qw / w.qn; w.qh[1] = qx / w.qn; w.qh[2] = qy / w.qn; w.qh[3] = qz / w.qn;
    w.o = 1.0 / (1.0 + exp(-(double)rec[10]));
    const double a = w.qh[0], x = w.qh[1], y = w.qh[2], z = w.qh[3];
    w.Rq[0] = 1.0 - 2.0 * (y * y + z * z);
    w.Rq[1] = 2.0 * (x * y - a * z);
    w.Rq[2] = 2.0 * (x * z + a * y);
    w.Rq[3] = 2.0 * (x * y + a * z);
    w.Rq[4] = 1.0 - 2.0 * (x * x + z * z);
    w.Rq[5] = 2.0 * (y * z - a * x);
    w.Rq[6] = 2.0 * (x * z - a * y);
    w.Rq[7] = 2.0 * (y * z + a * x);
    w.Rq[8] = 1.0 - 2.0 * (x * x + y * y);
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int k = 0; k < 3; k++) w.M[3 * r + k] = w.Rq[3 * r + k] * w.s[k];
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int k = r; k < 3; k++)
            // symmetric bit for bit: the products commute
            w.S[3 * r + k] = w.S[3 * k + r] =
                (w.M[3 * r] * w.M[3 * k] + w.M[3 * r + 1] * w.M[3 * k + 1]) + w.M[3 * r + 2] * w.M[3 * k + 2];
}

// Camera part of the chain.
struct Cam {
    double xc, yc, zc;
    double Sc[9], J[6];
    double ap, bp, cp, det;
};

__device__ __forceinline__ bool camera_chain(const ViewDev& V, const World& w, Cam& c) {
    const double* R = V.R;
    c.xc = ((R[0] * w.mu[0] + R[1] * w.mu[1]) + R[2] * w.mu[2]) + V.t[0];
    c.yc = ((R[3] * w.mu[0] + R[4] * w.mu[1]) + R[5] * w.mu[2]) + V.t[1];
    c.zc = ((R[6] * w.mu[0] + R[7] * w.mu[1]) + R[8] * w.mu[2]) + V.t[2];
    if (!(c.zc > kNearZ)) return false;
    double A[9];
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int k = 0; k < 3; k++) A[3 * r + k] = (R[3 * r] * w.S[k] + R[3 * r + 1] * w.S[3 + k]) + R[3 * r + 2] * w.S[6 + k];
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int k = 0; k < 3; k++) c.Sc[3 * r + k] = (A[3 * r] * R[3 * k] + A[3 * r + 1] * R[3 * k + 1]) + A[3 * r + 2] * R[3 * k + 2];
    const double z2 = c.zc * c.zc;
    c.J[0] = V.fx / c.zc;
    c.J[1] = 0.0;
    c.J[2] = -(V.fx * c.xc) / z2;
    c.J[3] = 0.0;
    c.J[4] = V.fy / c.zc;
    c.J[5] = -(V.fy * c.yc) / z2;
    double T[6];
#pragma unroll
    for (int r = 0; r < 2; r++)
#pragma unroll
        for (int k = 0; k < 3; k++) T[3 * r + k] = (c.J[3 * r] * c.Sc[k] + c.J[3 * r + 1] * c.Sc[3 + k]) + c.J[3 * r + 2] * c.Sc[6 + k];
    const double s00 = (T[0] * c.J[0] + T[1] * c.J[1]) + T[2] * c.J[2];
    const double s01 = (T[0] * c.J[3] + T[1] * c.J[4]) + T[2] * c.J[5];
    const double s11 = (T[3] * c.J[3] + T[4] * c.J[4]) + T[5] * c.J[5];
    c.ap = s00 + kLowPass;
    c.bp = s01;
    c.cp = s11 + kLowPass;
    c.det = c.ap * c.cp - c.bp * c.bp;
    return true;
}

template <int L>
__device__ __forceinline__ void view_dir(const ViewDev& V, const double mu[3], double d[3], double* dn) {
    d[0] = mu[0] - V.cw[0];
    d[1] = mu[1] - V.cw[1];
    d[2] = mu[2] - V.cw[2];
    *dn = sqrt((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]);
    const double inv = 1.0 / *dn;      // the direction only feeds the colour (no integer decision)
    d[0] *= inv; d[1] *= inv; d[2] *= inv;
}

// ---- FP32 SH basis and its contracted gradient for the colour adjoint

template <int L>
__device__ __forceinline__ void sh_basis_f(float x, float y, float z, float* Y) {
    Y[0] = (float)kY0;
    if (L >= 1) {
        Y[1] = -(float)kY1 * y;
        Y[2] = (float)kY1 * z;
        Y[3] = -(float)kY1 * x;
    }
    if (L >= 2) {
        Y[4] = (float)kY2a * x * y;
        Y[5] = -(float)kY2a * y * z;
        Y[6] = (float)kY2b * (3.0f * z * z - 1.0f);
        Y[7] = -(float)kY2a * x * z;
        Y[8] = (float)kY2c * (x * x - y * y);
    }
    if (L >= 3) {
        Y[9] = -(float)kY3a * y * (3.0f * x * x - y * y);
        Y[10] = (float)kY3b * x * y * z;
        Y[11] = -(float)kY3c * y * (5.0f * z * z - 1.0f);
        Y[12] = (float)kY3d * z * (5.0f * z * z - 3.0f);
        Y[13] = -(float)kY3c * x * (5.0f * z * z - 1.0f);
        Y[14] = (float)kY3e * z * (x * x - y * y);
        Y[15] = -(float)kY3a * x * (x * x - 3.0f * y * y);
    }
}

template <int L>
__device__ __forceinline__ void sh_grad_dot_f(float x, float y, float z, const float* w, float g[3]) {
    float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f;
    if (L >= 1) {
        g0 -= (float)kY1 * w[3];
        g1 -= (float)kY1 * w[1];
        g2 += (float)kY1 * w[2];
    }
    if (L >= 2) {
        g0 += (float)kY2a * y * w[4] - (float)kY2a * z * w[7] + 2.0f * (float)kY2c * x * w[8];
        g1 += (float)kY2a * x * w[4] - (float)kY2a * z * w[5] - 2.0f * (float)kY2c * y * w[8];
        g2 += -(float)kY2a * y * w[5] + 6.0f * (float)kY2b * z * w[6] - (float)kY2a * x * w[7];
    }
    if (L >= 3) {
        const float p3 = 3.0f * x * x - 3.0f * y * y, p5 = 5.0f * z * z - 1.0f;
        g0 += -6.0f * (float)kY3a * x * y * w[9] + (float)kY3b * y * z * w[10] - (float)kY3c * p5 * w[13] + 2.0f * (float)kY3e * x * z * w[14]
              - (float)kY3a * p3 * w[15];
        g1 += -(float)kY3a * p3 * w[9] + (float)kY3b * x * z * w[10] - (float)kY3c * p5 * w[11] - 2.0f * (float)kY3e * y * z * w[14]
              + 6.0f * (float)kY3a * x * y * w[15];
        g2 += (float)kY3b * x * y * w[10] - 10.0f * (float)kY3c * y * z * w[11] + (float)kY3d * (15.0f * z * z - 3.0f) * w[12]
              - 10.0f * (float)kY3c * x * z * w[13] + (float)kY3e * (x * x - y * y) * w[14];
    }
    g[0] = g0;
    g[1] = g1;
    g[2] = g2;
}

// Tile culling by the ellipse.  A tile of the rectangle is kept when the
// smallest q over the rectangle spanned by its pixel centres is at most 9 +
// 1e-3 (the margin covers the compositor's FP32 evaluation of q): zero when
// the mean lies inside, else the least of the four edge minima, each the
// parabola on that edge at its clamped vertex (on x = X the vertex is at
// y = (-B / C) X, on y = Y at x = (-B / A) Y).  Rectangles of more than
// kMaskTiles tiles keep every tile.  This is an optimisation of the method's
// tile lists (every tile of the rectangle): a dropped tile has q > 9 at every
// pixel centre, so no pixel of it would composite the Gaussian, and the image
// and gradients do not change.
constexpr int kMaskTiles = 64;
constexpr double kQCull = 9.001;
constexpr int kProjBlk = 128;
constexpr int64_t kProjFill = 1024;     // work-groups that fill the chip

__device__ __forceinline__ double q_at(double A, double B, double C, double X, double Y) {
    return (A * X * X + 2.0 * B * X * Y) + C * Y * Y;
}

// Least q over the pixel-centre rectangle [X0, X1] x [Y0, Y1] (offsets from the
// mean).  Moving from a point towards the mean lowers q, so the least point lies
// on an edge that faces the mean: x = Xn or y = Yn, the rectangle's nearest
// coordinates (0 when the range holds it: the candidate then lies on the other
// edge, or is the mean itself).  The far edges need no test.
__device__ __forceinline__ double rect_qmin(double A, double B, double C, double ky, double kx, double X0,
                                            double X1, double Y0, double Y1) {
    const double Xn = fmin(fmax(0.0, X0), X1), Yn = fmin(fmax(0.0, Y0), Y1);
    const double ya = fmin(fmax(ky * Xn, Y0), Y1), xb = fmin(fmax(kx * Yn, X0), X1);
    return fmin(q_at(A, B, C, Xn, ya), q_at(A, B, C, xb, Yn));
}

// Colour of a Gaussian seen along the unit direction to it, FP64; it decides no
// integer, so its sums are fused multiply-adds.
template <int L>
__device__ __forceinline__ void sh_color(const ViewDev& V, const double mu[3], const float* sh, float col[3]) {
    constexpr int NB = (L + 1) * (L + 1);
    double d[3], dn;
    view_dir<L>(V, mu, d, &dn);
    double Y[16];
    sh_basis<L>(d[0], d[1], d[2], Y);
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NB; j++)
#pragma unroll
        for (int ch = 0; ch < 3; ch++) acc[ch] = fma(Y[j], (double)sh[3 * j + ch], acc[ch]);
#pragma unroll
    for (int ch = 0; ch < 3; ch++) {
        const double raw = 0.5 + acc[ch];
        col[ch] = (float)(raw > 0.0 ? raw : 0.0);
    }
}

// One work-group per kProjBlk Gaussians of a frame, looping over the frame's
// views (a chunk of them: see launch_project).  Each view's tile tests are
// shared out over the work-group: rectangles range from one tile to dozens, so a
// thread testing only its own would hold its wave for the largest rectangle
// among 64.  Per view every geometry thread stages its record (mean, conic,
// edge-vertex slopes, rectangle) in LDS and appends its tests' (owner, tile)
// words to a list (in no fixed order: the tests only OR bits); then thread t
// takes tests t, t + threads, ... and ORs kept tiles into the owner's LDS mask.
//
// SPLIT: the geometry and the colour run in waves of their own.  Two waves hold
// the world chain of the Gaussians, two their SH coefficients and the FP64 basis,
// and a view's colours cross through LDS; all four share the tile tests.  In one
// thread the two need over 200 registers at degree 3, two waves per SIMD, and the
// kernel waits on the latency of its FP64 chains; apart they fit 128, four waves.
// The waves' prologues (world chain, coefficient loads) run side by side with
// nothing to share, so it takes enough views to pay: degree 3, 293 k Gaussians
// and 50 views 698 us together, 608 split; 410 k and 16 views 305 / 297; 410 k
// and 10 views 202 / 206; 3.1 M and 10 views 1,200 / 1,274.
constexpr int kSplitViews = 12;
template <bool SPLIT>
constexpr int proj_threads() { return SPLIT ? 2 * kProjBlk : kProjBlk; }

template <int L, bool SPLIT>
__global__ __launch_bounds__(proj_threads<SPLIT>()) __attribute__((amdgpu_waves_per_eu(SPLIT ? 4 : 1)))
void k_project(const ViewDev* __restrict__ views, const int32_t* __restrict__ frame_views,
               const int32_t* __restrict__ view_order, int32_t C, int64_t N, int32_t tw, int32_t th,
               const float* __restrict__ params, pg_splat* __restrict__ splats, pg_bin* __restrict__ bins,
               pg_tile_set* __restrict__ tiles, uint8_t* __restrict__ visible) {
    constexpr int NB = (L + 1) * (L + 1);
    constexpr int kThreads = proj_threads<SPLIT>();
    __shared__ double s_geo[7][kProjBlk];       // mean x, y; conic A, B, C; slopes -B/C, -B/A
    __shared__ int32_t s_rect[4][kProjBlk];     // x_lo, y_lo, width, 2^16 / width rounded up
    __shared__ uint16_t s_item[kProjBlk * kMaskTiles];   // test: owner thread << 6 | rectangle bit
    __shared__ unsigned long long s_mask[kProjBlk];
    __shared__ float s_col[2][3][kProjBlk];     // colours of even and odd views of the loop (split roles)
    __shared__ int32_t s_total[2];              // tests of even and odd views of the loop
    const int tid = threadIdx.x, own = tid % kProjBlk;
    // grid (Gaussian chunks, frames, view chunks): the frame, its views and so every
    // view's camera are uniform over the work-group, and the camera is read with scalar loads
    const int32_t f = (int32_t)blockIdx.y;
    const int64_t i0 = (int64_t)blockIdx.x * kProjBlk + own;
    const bool has = i0 < N;
    const int64_t i = has ? i0 : 0;
    const int32_t fv0 = frame_views[f], fv1 = frame_views[f + 1];
    const int32_t per = (fv1 - fv0 + (int32_t)gridDim.z - 1) / (int32_t)gridDim.z;
    const int32_t v0 = fv0 + (int32_t)blockIdx.z * per, v1 = min(fv1, v0 + per);
    if (v0 >= v1) return;     // uniform over the work-group
    const float* P = params + (int64_t)f * C * N + i;
    if (tid < 2) s_total[tid] = 0;
    __syncthreads();
    // the view's tests, by every thread; the kept tiles are in s_mask after the second barrier
    auto tile_tests = [&](int32_t k) __attribute__((always_inline)) {
        __syncthreads();
        const int32_t total = s_total[k & 1];
        if (tid == 0) s_total[(k + 1) & 1] = 0;      // last read before the previous view's second barrier
        for (int32_t q = tid; q < total; q += kThreads) {
            const uint32_t it = s_item[q];
            const int32_t lo = (int32_t)(it >> 6);                 // owner
            const int32_t bit = (int32_t)(it & 63u);               // row-major index in the rectangle
            const int32_t row = (bit * s_rect[3][lo]) >> 16;        // bit / width (bit < 64)
            const int32_t tx = s_rect[0][lo] + (bit - row * s_rect[2][lo]), ty = s_rect[1][lo] + row;
            const double X0 = ((double)tx * tw + 0.5) - s_geo[0][lo], X1 = X0 + (double)(tw - 1);
            const double Y0 = ((double)ty * th + 0.5) - s_geo[1][lo], Y1 = Y0 + (double)(th - 1);
            const double qmin = rect_qmin(s_geo[2][lo], s_geo[3][lo], s_geo[4][lo], s_geo[5][lo], s_geo[6][lo], X0,
                                          X1, Y0, Y1);
            if (qmin <= kQCull) atomicOr(&s_mask[lo], 1ull << bit);
        }
        __syncthreads();
    };
    float sh[3 * NB];
    if (SPLIT && __builtin_amdgcn_readfirstlane(tid) >= kProjBlk) {
        // ---- colour waves
        const double mu[3] = {P[0], P[N], P[2 * N]};
#pragma unroll
        for (int k = 0; k < 3 * NB; k++) sh[k] = P[(int64_t)(11 + k) * N];
        for (int32_t vi = v0; vi < v1; vi++) {
            const int32_t k = vi - v0;
            float col[3];
            sh_color<L>(views[view_order[vi]], mu, sh, col);
#pragma unroll
            for (int ch = 0; ch < 3; ch++) s_col[k & 1][ch][own] = col[ch];
            tile_tests(k);
        }
        return;
    }
    float rec[11];
#pragma unroll
    for (int k = 0; k < 11; k++) rec[k] = has ? P[(int64_t)k * N] : 0.0f;
    if (!SPLIT) {
#pragma unroll
        for (int k = 0; k < 3 * NB; k++) sh[k] = P[(int64_t)(11 + k) * N];
    }
    World w;
    world_chain(rec, w);
    const double itw = 1.0 / (double)tw, ith = 1.0 / (double)th;   // exact: tw, th are 8, 16 or 32
    bool any = false;
    for (int32_t vi = v0; vi < v1; vi++) {
        const int32_t v = view_order[vi], k = vi - v0;
        const ViewDev& V = views[v];
        Cam c;
        float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0, o2 = o0;
        uint4 bo = make_uint4(0u, 0u, 0u, 0u);
        int32_t nrect = 0;      // tiles of the rectangle (0: culled)
        double mx = 0.0, my = 0.0, A = 1.0, B = 0.0, Cq = 1.0;
        int32_t ixl = 0, iyl = 0, ixh = 0, iyh = 0;
        const bool ok = has && camera_chain(V, w, c) && (c.det > kDetMin);
        if (ok) {
            const double tr = c.ap + c.cp;
            const double lam = 0.5 * (tr + sqrt(fmax(0.0, tr * tr - 4.0 * c.det)));
            const double rr = ceil(3.0 * sqrt(lam));
            mx = (V.fx * c.xc) / c.zc + V.cx;
            my = (V.fy * c.yc) / c.zc + V.cy;
            // visibility (the set sparse Adam updates): some pixel of the image lies
            // within r of the mean on both axes; independent of the tile shape and of
            // the tile culling below
            if (mx + rr >= 0.0 && mx - rr < (double)V.W && my + rr >= 0.0 && my - rr < (double)V.H) any = true;
            // the view table only admits tile sides of 8, 16 or 32: dividing by a power of
            // two is exactly multiplying by its reciprocal, so these equal the divisions
            const double xlo = fmax(0.0, floor((mx - rr) * itw));
            const double xhi = fmin((double)(V.TX - 1), floor((mx + rr) * itw));
            const double ylo = fmax(0.0, floor((my - rr) * ith));
            const double yhi = fmin((double)(V.TY - 1), floor((my + rr) * ith));
            const float zf = (float)c.zc;
            if (!SPLIT) {
                float col[3];
                sh_color<L>(V, w.mu, sh, col);
                o2 = make_float4(col[0], col[1], col[2], 0.0f);
            }
            o2.w = zf;
            // the conic decides no integer by itself (the tile test below keeps a
            // margin), so one reciprocal serves its three entries
            const double idet = 1.0 / c.det;
            A = c.cp * idet;
            B = -c.bp * idet;
            Cq = c.ap * idet;
            const uint64_t bx = (uint64_t)__double_as_longlong(mx), by = (uint64_t)__double_as_longlong(my);
            o0 = make_float4(__uint_as_float((uint32_t)bx), __uint_as_float((uint32_t)(bx >> 32)),
                             __uint_as_float((uint32_t)by), __uint_as_float((uint32_t)(by >> 32)));   // the FP64 mean's bits
            o1 = make_float4((float)A, (float)B, (float)Cq, (float)w.o);
            if (xlo <= xhi && ylo <= yhi) {
                ixl = (int32_t)xlo;
                iyl = (int32_t)ylo;
                ixh = (int32_t)xhi;
                iyh = (int32_t)yhi;
                nrect = (ixh - ixl + 1) * (iyh - iyl + 1);
                bo.x = (uint32_t)(ixl & 0xffff) | ((uint32_t)(iyl & 0xffff) << 16);
                bo.y = (uint32_t)(ixh & 0xffff) | ((uint32_t)(iyh & 0xffff) << 16);
                bo.z = __float_as_uint(zf);
            }
        }
        // ---- tile tests, shared out over the work-group
        const int32_t ntest = nrect <= kMaskTiles ? nrect : 0;
        const int32_t wdt = ixh - ixl + 1;
        s_geo[0][own] = mx;
        s_geo[1][own] = my;
        s_geo[2][own] = A;
        s_geo[3][own] = B;
        s_geo[4][own] = Cq;
        const double iac = 1.0 / (A * Cq);         // edge-vertex slopes -B / C and -B / A
        s_geo[5][own] = -B * A * iac;
        s_geo[6][own] = -B * Cq * iac;
        s_rect[0][own] = ixl;
        s_rect[1][own] = iyl;
        s_rect[2][own] = wdt;
        s_rect[3][own] = (65536 + wdt - 1) / wdt;
        s_mask[own] = 0ull;
        int32_t incl = ntest;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t u = __shfl_up(incl, o, 64);
            if ((tid & 63) >= o) incl += u;
        }
        int32_t at = 0;
        if ((tid & 63) == 63) at = atomicAdd(&s_total[k & 1], incl);      // the wave's place in the list
        at = __builtin_amdgcn_readlane(at, 63) + incl - ntest;
        for (int32_t b = 0; b < ntest; b++) s_item[at + b] = (uint16_t)((own << 6) | b);
        tile_tests(k);
        const uint64_t tmask = ntest ? (uint64_t)s_mask[own] : 0ull;
        const int32_t nt = ntest ? (int32_t)__popcll(tmask) : nrect;
        uint4 ts = make_uint4(0u, 0u, 0u, 0u);
        if (nt > 0) {
            bo.w = (uint32_t)nt;
            ts = make_uint4((uint32_t)tmask, (uint32_t)(tmask >> 32), bo.x,
                            (uint32_t)(ixh - ixl + 1) | ((uint32_t)(iyh - iyl + 1) << 16));
        } else {
            bo = make_uint4(0u, 0u, 0u, 0u);
        }
        if (SPLIT && ok) {
            o2.x = s_col[k & 1][0][own];
            o2.y = s_col[k & 1][1][own];
            o2.z = s_col[k & 1][2][own];
        }
        if (has) {
            const int64_t gv = (int64_t)v * N + i;
            float4* sp = reinterpret_cast<float4*>(splats + gv);
            sp[0] = o0;
            sp[1] = o1;
            sp[2] = o2;
            reinterpret_cast<uint4*>(bins)[gv] = bo;
            reinterpret_cast<uint4*>(tiles)[gv] = ts;
        }
    }
    if (any) visible[(int64_t)f * N + i] = 1;
}

// ---------------------------------------------------------------- flow masking
// Covariance-aware flow masking (Sec. 4.2 masking paragraph, Algorithm 1):
// a Gaussian is dynamic when, in some view of its frame, a pixel whose centre
// is within r = ceil(3 sqrt(lambda_max)) of the mean on both axes and inside
// the image has q <= 9 and a non-zero flow mask (the OR across cameras).
//
// k_tile_motion marks the cells of 8 x 4 pixels holding any motion, a byte per
// screen tile.  k_flow_mask then works in two phases per work-group (one view, kFlowRecs Gaussians):
//  1. An FP32 bound per record: a disc around the mean that contains the exact
//     square (the largest scale through the Jacobian's norm, every rounding
//     covered), and whether a motion cell lies under it.  Most records end
//     here after ~80 instructions instead of the FP64 projection's ~450.  A
//     Gaussian that an earlier view has already labelled ends at once; where the
//     groups are many rounds of the chip, most are, and the others are first
//     collected in LDS so that every lane has one.
//  2. The records left are collected in LDS, so that every lane has one: the
//     FP64 projection, culls and radius of k_project, and the cells under the
//     ellipse's box.  Then eight lanes take a record and scan the box's rows
//     from the middle out, eight mask bytes per load, with q <= 9 in FP64 at
//     the centres whose mask is set.  The label is exactly that of a scan of
//     every pixel of the square.  (One lane per record waits for the largest
//     box among 64: 730 us against 482.)  Squares past kFlowSide, if a
//     cell under them holds motion, are scanned by a whole wave, 64 pixels per
//     round, only in tiles that hold motion, which are found eight a load.  They are
//     dealt to the four waves: the collected list's first wave would hold most of
//     them, and the others wait.
// A hit writes 1 to the Gaussian's zeroed label: every writer stores the same
// value, so the OR over views needs no atomics.  A Gaussian's chunk runs on one
// XCD for every view, so its parameters and labels stay in that L2.
// 14.0 M records of 50 views of 1024x768, 3 % of motion: the whole call 1,720 us
// with the FP64 projection of every record and a wave per flagged record; 575
// with the two phases; 430 with cells of 8 x 4 pixels instead of whole tiles;
// 339 with the unlabelled records collected and the next one's parameters read
// ahead; 329 now, of which the motion cells 25 and the fetch 42.  Larger Gaussians, 2.4 M records of 10 views, 3 % of motion: 638 us by the
// projection of every record, 1,098 with large squares walked by the wave that
// collected them, 548.
constexpr int kFlowThreads = 256;
constexpr int kFlowRecs = 2048;        // Gaussians per work-group at most
constexpr int64_t kFlowFill = 2048;    // work-groups that fill the chip
// LDS left unused, so that five groups share a CU: with six (as the registers allow) so
// many views run beside each other that each sees fewer labels of the others (50 views
// of 276 k Gaussians, all motion, four / five / six groups: 423 / 440 / 525 us; 5 %: 322 / 302
// / 291).
constexpr int kFlowSpare = 6144;
constexpr int kFlowSide = 64;          // largest side of a square that eight lanes scan

// Eight mask bytes from p on (zero past the end of the masks).
__device__ __forceinline__ uint64_t mask8(const uint8_t* __restrict__ masks, int64_t p, int64_t n) {
    uint64_t w = 0;
    if (p + 8 <= n) {
        __builtin_memcpy(&w, masks + p, 8);
    } else {
        for (int k = 0; p + k < n; k++) w |= (uint64_t)masks[p + k] << (8 * k);
    }
    return w;
}
__device__ __forceinline__ uint64_t first_bytes(uint64_t w, int32_t n) {
    return n >= 8 ? w : (n > 0 ? w & ((1ull << (8 * n)) - 1) : 0ull);
}

// A tile is 256 pixels, 32 runs of eight: half a wave per tile, one run per lane.
// The tile's byte has a bit per cell of 8 x 4 pixels (row-major) that holds motion.
// The view is looked up once per group and again only for tiles past its end.  On
// many tiles a lane takes TILES of them, so that as many loads are in flight (50 views
// of 1024 x 768, 39 MB of masks: 40 us with a tile and a look-up per lane, 25 with four);
// few tiles spread over more groups instead (4 views of 800 x 600 with four tiles per
// lane: 1.6 us more).
constexpr int kMotionTiles = 4;
constexpr int64_t kMotionMany = 32768;
template <int TILES>
__global__ __launch_bounds__(256) void k_tile_motion(const ViewDev* __restrict__ views, int nv, int64_t n_tiles,
                                                     int64_t n_pixels, int32_t tw,
                                                     const uint8_t* __restrict__ masks, uint8_t* __restrict__ tmot) {
    const int64_t tile0 = (int64_t)blockIdx.x * (8 * TILES);
    const int32_t runs = tw / 8, th = 256 / tw;
    const int32_t v0 = find_view_by_tile(views, nv, tile0);
    const int64_t next = v0 + 1 < nv ? views[v0 + 1].tile_base : n_tiles;
    const int32_t k = (int32_t)(threadIdx.x % 32);
    bool any[TILES];
#pragma unroll
    for (int q = 0; q < TILES; q++) {
        const int64_t tile = tile0 + q * 8 + threadIdx.x / 32;
        any[q] = false;
        if (tile < n_tiles) {
            const ViewDev& V = views[tile < next ? v0 : find_view_by_tile(views, nv, tile)];
            const uint32_t local = (uint32_t)(tile - V.tile_base), ty = local / (uint32_t)V.TX;
            const int32_t x = (int32_t)(local - ty * (uint32_t)V.TX) * tw + (k % runs) * 8;
            const int32_t y = (int32_t)ty * th + k / runs;
            if (x < V.W && y < V.H)
                any[q] = first_bytes(mask8(masks, V.pix_base + (int64_t)y * V.W + x, n_pixels), V.W - x) != 0;
        }
    }
#pragma unroll
    for (int q = 0; q < TILES; q++) {
        const int64_t tile = tile0 + q * 8 + threadIdx.x / 32;
        const uint64_t b = __ballot(any[q]);
        uint32_t h = (uint32_t)(threadIdx.x & 32 ? b >> 32 : b);
        h |= h >> runs;             // four rows of runs into one
        h |= h >> (2 * runs);
        uint32_t cells = 0;
        for (int32_t r = 0; r < th / 4; r++) cells |= ((h >> (4 * r * runs)) & ((1u << runs) - 1u)) << (r * runs);
        if (tile < n_tiles && k == 0) tmot[tile] = (uint8_t)cells;
    }
}

// Whether a cell under the pixels [x0, x1] x [y0, y1] (inside the view) holds motion.
// Squares several tiles wide read eight tiles at a time and end at the first row that
// holds some: without motion a lane walks all of its tiles, one load after the other
// (the same Gaussians without motion: 352 us with an FP64 projection each and a load per
// tile, 549 with the two phases and a load per tile, 169).
constexpr int kMotionWide = 6;
template <bool WIDE>
__device__ __forceinline__ bool motion_under(const ViewDev& V, const uint8_t* __restrict__ tmot, int64_t n_tiles,
                                             int32_t x0, int32_t x1, int32_t y0, int32_t y1, int32_t tw, int32_t th) {
    const int32_t runs = tw / 8, sx = __builtin_ctz(tw), sy = __builtin_ctz(th);
    const uint32_t rep = runs == 1 ? 0xffu : (runs == 2 ? 0x55u : 0x11u);       // a row's columns in every row
    const int32_t tx0 = x0 >> sx, tx1 = x1 >> sx;
    uint32_t any = 0;
    if (WIDE && tx1 - tx0 >= kMotionWide) {
        const uint64_t left = ((2u << (runs - 1)) - (1u << ((x0 - (tx0 << sx)) >> 3))) * rep;
        const uint64_t right = ((2u << ((x1 - (tx1 << sx)) >> 3)) - 1u) * rep;
        for (int32_t ty = y0 >> sy; ty <= y1 >> sy; ty++) {
            const int32_t r0 = max(y0 - (ty << sy), 0) >> 2, r1 = min(y1 - (ty << sy), th - 1) >> 2;
            const uint64_t rows = 0x0101010101010101ull * ((1u << ((r1 + 1) * runs)) - (1u << (r0 * runs)));
            const int64_t row = V.tile_base + (int64_t)ty * V.TX;
            uint64_t hit = 0;
            for (int32_t tx = tx0; tx <= tx1; tx += 8) {
                uint64_t w = first_bytes(mask8(tmot, row + tx, n_tiles), tx1 - tx + 1) & rows;
                if (tx == tx0) w &= left | ~0xffull;
                if (tx1 - tx < 8) w &= ~(0xffull << (8 * (tx1 - tx))) | right << (8 * (tx1 - tx));
                hit |= w;
            }
            if (hit) return true;
        }
        return false;
    }
    for (int32_t ty = y0 >> sy; ty <= y1 >> sy; ty++) {
        const int32_t r0 = max(y0 - (ty << sy), 0) >> 2, r1 = min(y1 - (ty << sy), th - 1) >> 2;
        const uint32_t rows = (1u << ((r1 + 1) * runs)) - (1u << (r0 * runs));
        const uint8_t* row = tmot + V.tile_base + (int64_t)ty * V.TX;
#pragma unroll 2
        for (int32_t tx = tx0; tx <= tx1; tx++) {
            const int32_t c0 = max(x0 - (tx << sx), 0) >> 3, c1 = min(x1 - (tx << sx), tw - 1) >> 3;
            any |= row[tx] & rows & (((2u << c1) - (1u << c0)) * rep);
        }
    }
    return any != 0;
}

__global__ void k_fill_u8(uint8_t* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// False when the record is certainly static in this view: culled by depth, or
// no motion cell under a square that contains the exact one.
// e = 2^-21 bounds eight FP32 roundings; each quantity carries its own bound.
struct Shape {
    float x, y, z, s0, s1, s2;      // position, log scales
};
__device__ __forceinline__ bool flow_may_hit(const ViewDev& V, float rn2, const Shape& g, int32_t tw, int32_t th,
                                             const uint8_t* __restrict__ tmot, int64_t n_tiles) {
    constexpr float e = 4.76837158e-7f;
    const float x = g.x, y = g.y, z = g.z;
    const float ls = fmaxf(fmaxf(g.s0, g.s1), g.s2);
    const float* R = V.Rf;
    const float xc = fmaf(R[0], x, fmaf(R[1], y, fmaf(R[2], z, V.tf[0])));
    const float yc = fmaf(R[3], x, fmaf(R[4], y, fmaf(R[5], z, V.tf[1])));
    const float zc = fmaf(R[6], x, fmaf(R[7], y, fmaf(R[8], z, V.tf[2])));
    const float ax = fabsf(x), ay = fabsf(y), az = fabsf(z);
    auto mag = [&](int r) {
        return fmaf(fabsf(R[3 * r]), ax, fmaf(fabsf(R[3 * r + 1]), ay, fmaf(fabsf(R[3 * r + 2]), az, fabsf(V.tf[r]))));
    };
    const float ex = e * mag(0), ey = e * mag(1), ez = e * mag(2);
    if (zc + ez < 0.19999f) return false;           // z_c <= 0.2: culled
    const float zl = fmaxf(zc - ez, 0.19f);         // every z_c that is kept is at least this
    const float iz = 1.0f / zl;
    const float u = (fabsf(xc) + ex) * iz, v = (fabsf(yc) + ey) * iz;       // |x_c / z_c| at most
    const float fu = V.fxf * iz, fv = V.fyf * iz;
    // largest eigenvalue of J J^T, times the largest eigenvalue of the camera-space covariance
    const float a = fu * fu * (1.0f + u * u), d = fv * fv * (1.0f + v * v), b = fu * fv * u * v;
    const float jj = 0.5f * (a + d + sqrtf((a - d) * (a - d) + 4.0f * b * b));
    const float lam = jj * rn2 * __expf(2.0f * ls) * 1.001f + 0.3001f;
    // the mean's bound: both ends of z_c's interval, and the roundings of f x / z + c
    const float izc = 1.0f / fmaxf(zc, 0.19f);
    const float px = V.fxf * xc * izc + (float)V.cx, py = V.fyf * yc * izc + (float)V.cy;
    const float r = 3.0015f * sqrtf(lam) + 1.01f;
    const float rx = r + 2.0f * (fu * (ex + u * ez) + e * (V.fxf * u + fabsf((float)V.cx)));
    const float ry = r + 2.0f * (fv * (ey + v * ez) + e * (V.fyf * v + fabsf((float)V.cy)));
    const float fx0 = px - rx, fx1 = px + rx, fy0 = py - ry, fy1 = py + ry;
    if (fx1 < 0.0f || fx0 > (float)V.W || fy1 < 0.0f || fy0 > (float)V.H) return false;
    // a square over many tiles, where the bound is wide of the ellipse, or a bound that is not a
    // number goes to the exact test (8 views of 59 k Gaussians of 55 pixels, 5 % of motion, us:
    // half sides of up to 256 tested here 1,801, 128 1,702, 64 1,532)
    if (!(rx < 64.0f && ry < 64.0f && fabsf(px) < 1e8f && fabsf(py) < 1e8f)) return true;
    const int32_t x0 = (int32_t)fmaxf(fx0, 0.0f), y0 = (int32_t)fmaxf(fy0, 0.0f);
    return motion_under<true>(V, tmot, n_tiles, min(x0, V.W - 1), min((int32_t)fx1, V.W - 1), min(y0, V.H - 1), min((int32_t)fy1, V.H - 1),
                        tw, th);
}

// A record's clipped square and quadratic form (x1 < x0: nothing to scan).
struct Square {
    double mx, my, A, B, C;
    int32_t x0, y0, x1, y1;     // y1 negative (of a square that is not empty): ~y1 of a large one
};

__global__ __launch_bounds__(kFlowThreads) void k_flow_mask(const ViewDev* __restrict__ views, int32_t nv, int32_t C,
                                                            int64_t N, int32_t recs, int32_t open, int64_t n_tiles, int64_t n_pixels,
                                                            int32_t tw, int32_t th,
                                                            const float* __restrict__ params,
                                                            const uint8_t* __restrict__ masks,
                                                            const uint8_t* __restrict__ tmot, uint8_t* dyn_gauss,
                                                            unsigned long long* __restrict__ counters) {
    __shared__ uint16_t s_open[kFlowRecs], s_rec[kFlowRecs];
    __shared__ Square s_sq[kFlowThreads];
    __shared__ int32_t s_left, s_count;
    // work-group b runs on XCD b mod 8: chunks of Gaussians are dealt to the XCDs,
    // and an XCD takes its chunks view by view
    const int64_t chunks = ceil_div(N, recs), per = ceil_div(chunks, 8);
    const int64_t j = blockIdx.x / 8, c = (int64_t)(blockIdx.x % 8) + 8 * (j % per);
    const int32_t v = (int32_t)(j / per);
    if (c >= chunks || v >= nv) return;
    const ViewDev& V = views[v];
    const int lane = (int)(threadIdx.x & 63);
    const int64_t i0 = c * recs;
    const float* P0 = params + (int64_t)V.frame * C * N;
    const int64_t out0 = (int64_t)V.frame * N;
    uint64_t tests = 0;
    if (threadIdx.x == 0) s_left = s_count = 0;
    // |R R^T| bounds the squared norm of the camera matrix (1 for a rotation)
    float rn2 = 0.0f;
#pragma unroll
    for (int r = 0; r < 3; r++) {
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; k++)
            sum += fabsf(fmaf(V.Rf[3 * r], V.Rf[3 * k], fmaf(V.Rf[3 * r + 1], V.Rf[3 * k + 1], V.Rf[3 * r + 2] * V.Rf[3 * k + 2])));
        rn2 = fmaxf(rn2, sum);
    }
    __syncthreads();
    // appends the lanes' records to a list (in any order)
    auto append = [&](bool keep, int32_t k, uint16_t* list, int32_t* n) __attribute__((always_inline)) {
        const uint64_t m = __ballot(keep);
        int32_t at = 0;
        if (lane == 0 && m) at = atomicAdd(n, (int32_t)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (keep) list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = (uint16_t)k;
    };
    // an earlier view's label ends a record (a stale 0 only costs the test; with the test
    // counter the labels are not looked at, so the count is the same every time)
    auto labelled = [&](int32_t k) __attribute__((always_inline)) {
        return !counters && __hip_atomic_load(dyn_gauss + out0 + i0 + k, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP) != 0;
    };
    int32_t left = (int32_t)imin(recs, N - i0);
    if (open) {     // the records without a label, collected so that every lane has one
        bool keep[kFlowRecs / kFlowThreads];
#pragma unroll
        for (int q = 0; q < kFlowRecs / kFlowThreads; q++) {
            const int32_t k = (int32_t)threadIdx.x + q * kFlowThreads;
            keep[q] = k < left && !labelled(k);
        }
#pragma unroll
        for (int q = 0; q < kFlowRecs / kFlowThreads; q++)
            append(keep[q], (int32_t)threadIdx.x + q * kFlowThreads, s_open, &s_left);
        __syncthreads();
        left = s_left;
    }
    // ---- phase 1: the next record's parameters are read while one is tested
    auto record = [&](int32_t at) __attribute__((always_inline)) {
        at = min(at, left - 1);
        return open ? (int32_t)s_open[at] : at;
    };
    auto shape = [&](int32_t k) __attribute__((always_inline)) {
        const float* P = P0 + i0 + k;
        return Shape{P[0], P[N], P[2 * N], P[3 * N], P[4 * N], P[5 * N]};
    };
    if (left > 0) {
        int32_t k_next = record((int32_t)threadIdx.x);
        Shape next = shape(k_next);
        for (int32_t base = 0; base < left; base += kFlowThreads) {
            const int32_t at = base + (int32_t)threadIdx.x, k = k_next;
            const Shape g = next;
            const bool done = !open && at < left && labelled(k);
            k_next = record(at + kFlowThreads);
            next = shape(k_next);
            const bool keep = at < left && flow_may_hit(V, rn2, g, tw, th, tmot, n_tiles) && !done;
            append(keep, k, s_rec, &s_count);
        }
    }
    __syncthreads();
    // ---- phase 2
    const int32_t count = s_count;
    for (int32_t base = 0; base < count; base += kFlowThreads) {
        const int32_t at = base + (int32_t)threadIdx.x;
        bool large = false;
        int32_t ix0 = 0, ix1 = -1, iy0 = 0, iy1 = -1;
        double mx = 0.0, my = 0.0, A = 1.0, B = 0.0, Cq = 1.0;
        if (at < count) {
            const int64_t i = i0 + s_rec[at];
            float rec[11];
#pragma unroll
            for (int k = 0; k < 11; k++) rec[k] = P0[(int64_t)k * N + i];
            World w;
            world_chain(rec, w);
            Cam cam;
            if (camera_chain(V, w, cam) && cam.det > kDetMin) {
                const double tr = cam.ap + cam.cp;
                const double lam = 0.5 * (tr + sqrt(fmax(0.0, tr * tr - 4.0 * cam.det)));
                const double rr = ceil(3.0 * sqrt(lam));
                mx = (V.fx * cam.xc) / cam.zc + V.cx;
                my = (V.fy * cam.yc) / cam.zc + V.cy;
                const double x0 = fmax(0.0, ceil(mx - rr - 0.5)), x1 = fmin((double)(V.W - 1), floor(mx + rr - 0.5));
                const double y0 = fmax(0.0, ceil(my - rr - 0.5)), y1 = fmin((double)(V.H - 1), floor(my + rr - 0.5));
                if (x0 <= x1 && y0 <= y1) {
                    ix0 = (int32_t)x0;
                    ix1 = (int32_t)x1;
                    iy0 = (int32_t)y0;
                    iy1 = (int32_t)y1;
                    A = cam.cp / cam.det;
                    B = -cam.bp / cam.det;
                    Cq = cam.ap / cam.det;
                    large = ix1 - ix0 >= kFlowSide || iy1 - iy0 >= kFlowSide;
                    if (!large) {
                        // q <= 9 lies inside the ellipse's box (half-extents 3 sqrt of the
                        // covariance's diagonal, widened past every rounding)
                        const float ex = 3.003f * sqrtf((float)cam.ap) + 0.02f, ey = 3.003f * sqrtf((float)cam.cp) + 0.02f;
                        ix0 = max(ix0, (int32_t)ceilf((float)(mx - 0.5 - (double)ex) - 0.01f));
                        ix1 = min(ix1, (int32_t)floorf((float)(mx - 0.5 + (double)ex) + 0.01f));
                        iy0 = max(iy0, (int32_t)ceilf((float)(my - 0.5 - (double)ey) - 0.01f));
                        iy1 = min(iy1, (int32_t)floorf((float)(my - 0.5 + (double)ey) + 0.01f));
                    }
                    const bool motion = large ? motion_under<true>(V, tmot, n_tiles, ix0, ix1, iy0, iy1, tw, th)
                                              : ix0 <= ix1 && iy0 <= iy1 &&
                                                    motion_under<false>(V, tmot, n_tiles, ix0, ix1, iy0, iy1, tw, th);
                    if (!motion) {
                        large = false;
                        ix1 = ix0 - 1;
                    }
                }
            }
        }
        // eight lanes per record: each takes every eighth row, from the middle out
        __syncthreads();        // the previous step's records are done with
        s_sq[threadIdx.x] = {mx, my, A, B, Cq, ix0, iy0, ix1, large ? ~iy1 : iy1};
        __syncthreads();
        const int32_t sub = lane % 8;
        for (int32_t r = threadIdx.x / 8; r < kFlowThreads && base + r < count; r += kFlowThreads / 8) {
            const Square q = s_sq[r];
            const int32_t n = q.x1 - q.x0 + 1;
            if (n <= 0 || q.y1 < 0) continue;         // culled, no motion, or left to the whole wave
            const int32_t mid = min(max((int32_t)q.my, q.y0), q.y1);      // |mean| is finite: the square is not empty
            const int32_t last = 2 * max(q.y1 - mid, mid - q.y0);         // rows mid, mid + 1, mid - 1, mid + 2, ...
            const int64_t p0 = V.pix_base + q.x0;
            bool hit = false;
            for (int32_t k = sub; k <= last && !hit; k += 8) {
                const int32_t y = mid + ((k & 1) ? (k + 1) / 2 : -(k / 2));
                if (y < q.y0 || y > q.y1) continue;
                const double dy = ((double)y + 0.5) - q.my;
                for (int32_t o = 0; o < n && !hit; o += 16) {
                    const int64_t p = p0 + (int64_t)y * V.W + o;
                    uint64_t m0 = first_bytes(mask8(masks, p, n_pixels), n - o);
                    uint64_t m1 = n - o > 8 ? first_bytes(mask8(masks, p + 8, n_pixels), n - o - 8) : 0ull;
                    while ((m0 | m1) && !hit) {
                        const bool lo = m0 != 0;
                        const int32_t k8 = (int32_t)(__builtin_ctzll(lo ? m0 : m1) >> 3);
                        const uint64_t clear = ~(0xffull << (8 * k8));
                        if (lo) m0 &= clear; else m1 &= clear;
                        tests++;
                        hit = q_at(q.A, q.B, q.C, ((double)(q.x0 + o + (lo ? 0 : 8) + k8) + 0.5) - q.mx, dy) <= 9.0;
                    }
                }
            }
            if (hit) dyn_gauss[out0 + i0 + s_rec[base + r]] = 1;      // every writer stores the same value
        }
        // squares too large for that: all lanes on one record, the records dealt to the waves
        // (the list's first wave alone would hold most of them)
        const int wave = (int)threadIdx.x / 64, mine = 4 * lane + wave;
        uint64_t todo = __ballot(base + mine < count && s_sq[mine].x1 >= s_sq[mine].x0 && s_sq[mine].y1 < 0);
        while (todo) {
            const int32_t r = 4 * __builtin_ctzll(todo) + wave;
            todo &= todo - 1;
            const Square q = s_sq[r];
            const int32_t sx0 = __builtin_amdgcn_readfirstlane(q.x0), sx1 = __builtin_amdgcn_readfirstlane(q.x1);
            const int32_t sy0 = __builtin_amdgcn_readfirstlane(q.y0), sy1 = ~__builtin_amdgcn_readfirstlane(q.y1);
            const uint8_t* M = masks + V.pix_base;
            const int32_t kx = __builtin_ctz(tw), ky = __builtin_ctz(th);
            bool any = false;
            for (int32_t ty = sy0 >> ky; ty <= sy1 >> ky && !any; ty++) {
                for (int32_t t8 = sx0 >> kx; t8 <= sx1 >> kx && !any; t8 += 8) {      // eight tiles a load
                    const uint64_t w = first_bytes(mask8(tmot, V.tile_base + (int64_t)ty * V.TX + t8, n_tiles),
                                                   (sx1 >> kx) - t8 + 1);
                    uint64_t moving = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(w >> 32)) << 32 |
                                      (uint32_t)__builtin_amdgcn_readfirstlane((int)w);
                    while (moving && !any) {
                        const int32_t k = __builtin_ctzll(moving) >> 3, tx = t8 + k;
                        moving &= ~(0xffull << (8 * k));
                        for (int32_t p = lane; p < 256 && !any; p += 64) {       // a tile is 256 pixels
                            const int32_t x = (tx << kx) + (p & (tw - 1)), y = (ty << ky) + (p >> kx);
                            bool hit = false;
                            if (x >= sx0 && x <= sx1 && y >= sy0 && y <= sy1 && M[(int64_t)y * V.W + x]) {
                                tests++;
                                hit = q_at(q.A, q.B, q.C, ((double)x + 0.5) - q.mx, ((double)y + 0.5) - q.my) <= 9.0;
                            }
                            any = __ballot(hit) != 0;
                        }
                    }
                }
            }
            if (any && lane == 0) dyn_gauss[out0 + i0 + s_rec[base + r]] = 1;
        }
    }
    if (counters) {
        unsigned long long t = tests;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if (lane == 0 && t) atomicAdd(counters, t);
    }
}

// Texel form of the labels: 1 where the texel's Gaussian is dynamic in some frame.
__global__ __launch_bounds__(256) void k_dyn_texel(const uint8_t* __restrict__ dyn_gauss,
                                                   const int32_t* __restrict__ texel_gauss, int64_t HW, int32_t F,
                                                   int64_t N, uint8_t* __restrict__ dyn_texel) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= HW) return;
    const int32_t gi = texel_gauss[t];
    uint8_t d = 0;
    if (gi >= 0 && gi < N)
        for (int32_t f = 0; f < F; f++) d |= dyn_gauss[(int64_t)f * N + gi];
    dyn_texel[t] = d;
}

// ---------------------------------------------------------------- adjoint
//
// With Q the conic matrix and Gh = [[da, db/2], [db/2, dc]] (q = a dx^2 +
// 2 b dx dy + c dy^2): dL/dSigma2D = -Q Gh Q; dL/dSigma_c = J^T (.) J;
// dL/dJ = 2 (dL/dSigma2D) J Sigma_c; dL/dSigma = W^T (dL/dSigma_c) W;
// dL/dM = 2 (dL/dSigma) M with M = R(q) diag(s); the mean through J and
// through dJ/dmu_c; SH through the basis and the view direction.  Texel
// chain: l_s via s, the raw quaternion via the normalisation, l_o via o (1 - o).
// Geometric part of the adjoint, FP64: position, log-scale, quaternion and
// logit-opacity gradients through the EWA chain of every view of the
// Gaussian's frame.  FP64 because the gradient of a rotation about an
// elongated Gaussian's long axis (and the quaternion's tangent component in
// general) is a small difference of large terms: in FP32 a few texels of the
// 2048^2 workload missed 1e-3.  No SH coefficients are held here.
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(3))) void k_project_bwd_geo(const ViewDev* __restrict__ views,
                                                         const int32_t* __restrict__ frame_views,
                                                         const int32_t* __restrict__ view_order, int32_t F,
                                                         int32_t C, int64_t N, int64_t n_gv,
                                                         const float* __restrict__ params,
                                                         float* __restrict__ grad2d,
                                                         const int32_t* __restrict__ gauss_texel,
                                                         const uint8_t* __restrict__ dyn, int64_t HW,
                                                         float* __restrict__ gatlas, int32_t accumulate) {
    // grid (Gaussian chunks, frames): the frame and its cameras are uniform over the
    // work-group, so the cameras are read with scalar loads
    const int32_t f = (int32_t)blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int32_t v0 = frame_views[f], v1 = frame_views[f + 1];
    const float* P = params + (int64_t)f * C * N + i;
    float rec[11];
#pragma unroll
    for (int k = 0; k < 11; k++) rec[k] = P[(int64_t)k * N];
    double acc[11];
#pragma unroll
    for (int k = 0; k < 11; k++) acc[k] = 0.0;
    // dL/dSigma (world) and dL/do summed over the views: the scale, rotation and
    // activation chains after them are linear and view-independent, so they run
    // once per Gaussian on the sums instead of once per record
    // (dL/dSigma is symmetric: its upper triangle 00, 01, 02, 11, 12, 22 is summed)
    double GSw_sum[6], go_sum = 0.0;
#pragma unroll
    for (int k = 0; k < 6; k++) GSw_sum[k] = 0.0;
    World w;     // in the view loop only its mean, Sigma and opacity are used
    bool have_world = false;
    // the record's slot sums (0 for culled records): the compositing moments
    // sum dq' (dx, dy, dx^2, dx dy, dy^2) and sum dq', with dq' = alpha dL/dalpha;
    // the next view's are loaded while this view's are used
    float nxt[6];
    auto load6 = [&](int32_t vi) __attribute__((always_inline)) {
        const int64_t gv = (int64_t)view_order[vi] * N + i;
#pragma unroll
        for (int k = 0; k < 6; k++) nxt[k] = grad2d[(int64_t)k * n_gv + gv];
    };
    if (v0 < v1) load6(v0);
    for (int32_t vi = v0; vi < v1; vi++) {
        const int32_t v = view_order[vi];
        const int64_t gv = (int64_t)v * N + i;
        double g6[6];
        bool nz = false;
#pragma unroll
        for (int k = 0; k < 6; k++) {
            g6[k] = (double)nxt[k];
            nz |= (nxt[k] != 0.0f);
        }
        if (vi + 1 < v1) load6(vi + 1);
        if (!nz) continue;
        if (!have_world) {
            world_chain(rec, w);
            have_world = true;
        }
        const ViewDev& V = views[v];
        Cam c;
        if (!camera_chain(V, w, c)) continue;   // never for a record with a gradient: the forward kept it
        // (gradients only from here on: reciprocals instead of divisions)
        const double idet = 1.0 / c.det;
        const double Q00 = c.cp * idet, Q01 = -c.bp * idet, Q11 = c.ap * idet;
        // 2D gradients from the moments (dL/dq = -dq'/2): dL/dm = Q (m0, m1),
        // dL/d(a, b, c) = -(m2 / 2, m3, m4 / 2), and dL/do = sum e dL/dalpha =
        // sum dq' / o (alpha = o e^{-q/2} wherever dq' is not zero); written back
        // as the record's grad2d
        {
            const double m0 = g6[0], m1 = g6[1];
            g6[0] = Q00 * m0 + Q01 * m1;
            g6[1] = Q01 * m0 + Q11 * m1;
            g6[2] = -0.5 * g6[2];
            g6[3] = -g6[3];
            g6[4] = -0.5 * g6[4];
            g6[5] = g6[5] / w.o;
#pragma unroll
            for (int k = 0; k < 6; k++) grad2d[(int64_t)k * n_gv + gv] = (float)g6[k];
        }
        const double G00 = g6[2], G01 = 0.5 * g6[3], G11 = g6[4];
        // QG = Q Gh ; GS = -(QG Q)
        const double QG00 = Q00 * G00 + Q01 * G01, QG01 = Q00 * G01 + Q01 * G11;
        const double QG10 = Q01 * G00 + Q11 * G01, QG11 = Q01 * G01 + Q11 * G11;
        const double GS00 = -(QG00 * Q00 + QG01 * Q01);
        const double GS01 = -(QG00 * Q01 + QG01 * Q11);
        const double GS11 = -(QG10 * Q01 + QG11 * Q11);
        // GJ = GS J (2x3)
        double GJ[6];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            GJ[k] = GS00 * c.J[k] + GS01 * c.J[3 + k];
            GJ[3 + k] = GS01 * c.J[k] + GS11 * c.J[3 + k];
        }
        // dL/dSigma_c = J^T GJ
        double GSc[9];
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int k = 0; k < 3; k++) GSc[3 * r + k] = c.J[r] * GJ[k] + c.J[3 + r] * GJ[3 + k];
        // dL/dJ = 2 GJ Sigma_c
        double GJm[6];
#pragma unroll
        for (int r = 0; r < 2; r++)
#pragma unroll
            for (int k = 0; k < 3; k++)
                GJm[3 * r + k] = 2.0 * (GJ[3 * r] * c.Sc[k] + GJ[3 * r + 1] * c.Sc[3 + k] + GJ[3 * r + 2] * c.Sc[6 + k]);
        // dL/dSigma = R^T GSc R
        const double* R = V.R;
        double tmp[9], GSw[9];
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int k = 0; k < 3; k++) tmp[3 * r + k] = GSc[3 * r] * R[k] + GSc[3 * r + 1] * R[3 + k] + GSc[3 * r + 2] * R[6 + k];
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int k = r; k < 3; k++) GSw[3 * r + k] = R[r] * tmp[k] + R[3 + r] * tmp[3 + k] + R[6 + r] * tmp[6 + k];
        GSw_sum[0] += GSw[0];
        GSw_sum[1] += GSw[1];
        GSw_sum[2] += GSw[2];
        GSw_sum[3] += GSw[4];
        GSw_sum[4] += GSw[5];
        GSw_sum[5] += GSw[8];
        // mean: dm/dmu_c = J, plus the dependence of J on mu_c
        const double iz = 1.0 / c.zc, iz2 = iz * iz, iz3 = iz2 * iz;
        double gmc0 = c.J[0] * g6[0] + c.J[3] * g6[1];
        double gmc1 = c.J[1] * g6[0] + c.J[4] * g6[1];
        double gmc2 = c.J[2] * g6[0] + c.J[5] * g6[1];
        gmc0 += GJm[2] * (-V.fx * iz2);
        gmc1 += GJm[5] * (-V.fy * iz2);
        gmc2 += GJm[0] * (-V.fx * iz2) + GJm[2] * (2.0 * V.fx * c.xc * iz3) + GJm[4] * (-V.fy * iz2)
                + GJm[5] * (2.0 * V.fy * c.yc * iz3);
#pragma unroll
        for (int k = 0; k < 3; k++) acc[k] += R[k] * gmc0 + R[3 + k] * gmc1 + R[6 + k] * gmc2;
        go_sum += g6[5];
    }
    if (have_world) {
        // The world chain again, so that its rotation, scale and M need no registers
        // during the view loop (the opaque step keeps the compiler from reusing w).
#pragma unroll
        for (int k = 0; k < 11; k++) asm volatile("" : "+v"(rec[k]));
        world_chain(rec, w);
        const double Gs[9] = {GSw_sum[0], GSw_sum[1], GSw_sum[2], GSw_sum[1], GSw_sum[3], GSw_sum[4],
                              GSw_sum[2], GSw_sum[4], GSw_sum[5]};
        // dL/dM = 2 GSw M ; dL/ds (log-scale) ; dL/dRq -> the normalised quaternion -> the stored one
        double gs[3] = {0.0, 0.0, 0.0}, GR[9];
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const double gm = 2.0 * (Gs[3 * r] * w.M[k] + Gs[3 * r + 1] * w.M[3 + k] +
                                         Gs[3 * r + 2] * w.M[6 + k]);
                gs[k] += gm * w.Rq[3 * r + k];
                GR[3 * r + k] = gm * w.s[k];
            }
        const double qa = w.qh[0], qx = w.qh[1], qy = w.qh[2], qz = w.qh[3];
        double gq[4];
        gq[0] = 2.0 * (-qz * GR[1] + qy * GR[2] + qz * GR[3] - qx * GR[5] - qy * GR[6] + qx * GR[7]);
        gq[1] = 2.0 * (qy * GR[1] + qz * GR[2] + qy * GR[3] - 2.0 * qx * GR[4] - qa * GR[5] + qz * GR[6] + qa * GR[7]
                       - 2.0 * qx * GR[8]);
        gq[2] = 2.0 * (-2.0 * qy * GR[0] + qx * GR[1] + qa * GR[2] + qx * GR[3] + qz * GR[5] - qa * GR[6] + qz * GR[7]
                       - 2.0 * qy * GR[8]);
        gq[3] = 2.0 * (-2.0 * qz * GR[0] - qa * GR[1] + qx * GR[2] + qa * GR[3] - 2.0 * qz * GR[4] + qy * GR[5]
                       + qx * GR[6] + qy * GR[7]);
        const double qd = gq[0] * qa + gq[1] * qx + gq[2] * qy + gq[3] * qz;
#pragma unroll
        for (int k = 0; k < 3; k++) acc[3 + k] += w.s[k] * gs[k];
#pragma unroll
        for (int k = 0; k < 4; k++) acc[6 + k] += (gq[k] - w.qh[k] * qd) / w.qn;
        acc[10] += go_sum * w.o * (1.0 - w.o);
    }
    const int64_t texel = gauss_texel[i];
    const float m = dyn ? (dyn[texel] ? 1.f : 0.f) : 1.f;
    float* out = gatlas + (int64_t)f * C * HW + texel;
#pragma unroll
    for (int k = 0; k < 11; k++) {
        if (accumulate) out[(int64_t)k * HW] += m * (float)acc[k];
        else out[(int64_t)k * HW] = m * (float)acc[k];
    }
}

// Colour part of the adjoint, FP32: SH coefficient gradients Y_j gc and the
// view-direction term of the position gradient, added to what the geometric
// kernel wrote.  The clamp decision (colour = max(0, 0.5 + sum Y k)) is the
// forward's: the FP32 sum settles it away from 0, and near 0 the forward's
// stored colour (0 exactly where its FP64 sum clamped) is read back.
template <int L>
__global__ __launch_bounds__(128) void k_project_bwd_sh(const ViewDev* __restrict__ views,
                                                        const int32_t* __restrict__ frame_views,
                                                        const int32_t* __restrict__ view_order, int32_t F,
                                                        int32_t C, int64_t N, int64_t n_gv,
                                                        const float* __restrict__ params,
                                                        const pg_splat* __restrict__ splats,
                                                        const float* __restrict__ grad2d,
                                                        const int32_t* __restrict__ gauss_texel,
                                                        const uint8_t* __restrict__ dyn, int64_t HW,
                                                        float* __restrict__ gatlas, int32_t accumulate) {
    constexpr int NB = (L + 1) * (L + 1);
    // grid (Gaussian chunks, frames): the frame and its cameras are uniform over the
    // work-group, so the cameras are read with scalar loads
    const int32_t f = (int32_t)blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int32_t v0 = frame_views[f], v1 = frame_views[f + 1];
    const float* P = params + (int64_t)f * C * N + i;
    const double mu[3] = {P[0], P[N], P[2 * N]};
    float sh[3 * NB];
#pragma unroll
    for (int k = 0; k < 3 * NB; k++) sh[k] = P[(int64_t)(11 + k) * N];
    float acc[3 * NB], gmu[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 3 * NB; k++) acc[k] = 0.0f;
    float nxt[3];     // the next view's colour gradients, loaded while this view's are used
    auto load3 = [&](int32_t vi) __attribute__((always_inline)) {
        const int64_t gv = (int64_t)view_order[vi] * N + i;
#pragma unroll
        for (int ch = 0; ch < 3; ch++) nxt[ch] = grad2d[(int64_t)(6 + ch) * n_gv + gv];
    };
    if (v0 < v1) load3(v0);
    for (int32_t vi = v0; vi < v1; vi++) {
        const int32_t v = view_order[vi];
        const float gcol[3] = {nxt[0], nxt[1], nxt[2]};
        if (vi + 1 < v1) load3(vi + 1);
        if (gcol[0] == 0.0f && gcol[1] == 0.0f && gcol[2] == 0.0f) continue;
        const ViewDev& V = views[v];
        double dd64[3], dn64;
        view_dir<L>(V, mu, dd64, &dn64);
        const float d[3] = {(float)dd64[0], (float)dd64[1], (float)dd64[2]};
        const float dn = (float)dn64;
        float Y[NB];
        sh_basis_f<L>(d[0], d[1], d[2], Y);
        // clamp decision: the FP32 colour sum settles it unless it lies within 1e-3 of the clamp;
        // there the forward's own decision is read back from its colour (max(0, its FP64 sum),
        // stored as float: 0 exactly when it clamped), instead of forming the FP64 sum again
        // (whose sixteen doubles doubled this kernel's registers)
        float gc[3];
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            float raw = 0.5f;
#pragma unroll
            for (int j = 0; j < NB; j++) raw = fmaf(Y[j], sh[3 * j + ch], raw);
            bool clamped = raw < 0.0f;
            if (fabsf(raw) < 1e-3f) clamped = !(splats[(int64_t)v * N + i].color[ch] > 0.0f);
            gc[ch] = clamped ? 0.0f : gcol[ch];   // clamped channel: no gradient
        }
        // SH coefficients: dL/dk[j][ch] = Y_j gc_ch; direction: sum_j (sum_ch k[j][ch] gc_ch) grad Y_j
        float wj[NB];
#pragma unroll
        for (int j = 0; j < NB; j++) {
#pragma unroll
            for (int ch = 0; ch < 3; ch++) acc[3 * j + ch] += Y[j] * gc[ch];
            wj[j] = (sh[3 * j] * gc[0] + sh[3 * j + 1] * gc[1]) + sh[3 * j + 2] * gc[2];
        }
        float gd[3];
        sh_grad_dot_f<L>(d[0], d[1], d[2], wj, gd);
        const float dd = gd[0] * d[0] + gd[1] * d[1] + gd[2] * d[2];
#pragma unroll
        for (int k = 0; k < 3; k++) gmu[k] += (gd[k] - d[k] * dd) / dn;
    }
    const int64_t texel = gauss_texel[i];
    const float m = dyn ? (dyn[texel] ? 1.f : 0.f) : 1.f;
    float* out = gatlas + (int64_t)f * C * HW + texel;
#pragma unroll
    for (int k = 0; k < 3; k++) out[(int64_t)k * HW] += m * gmu[k];   // after the geometric kernel
#pragma unroll
    for (int k = 0; k < 3 * NB; k++) {
        if (accumulate) out[(int64_t)(11 + k) * HW] += m * acc[k];
        else out[(int64_t)(11 + k) * HW] = m * acc[k];
    }
}

// Per-record sums of the instance slots.  Slots are laid out record by
// record in (view, id) order, so one work-group takes 256 consecutive
// records, whose slots form one contiguous range; the group streams it
// through LDS in coalesced chunks (ten independent loads per thread in
// flight) while each thread adds its own record's slots in rectangle
// row-major order, and grad2d is written coalesced.  A slot counts only when
// its tag is this sort's generation (the adjoint wrote it in this step);
// after an overflowed sort there are no slots and every sum is 0.
//
// Two kinds of record would leave the chip waiting for one thread, and are summed
// by lanes side by side instead (lane l adds slots l, l + W, ..., then the W
// partial sums are added in a fixed tree; as deterministic as the serial order):
//  - records of more than kSumSerial tiles (a Gaussian close to a camera covers
//    thousands) by a whole wave, and the stream passes over their slots;
//  - every record, by 16 lanes, when there are too few records to fill the chip
//    with 256 per work-group.  4,096 Gaussians in a 1920x1080 view (21 tiles a
//    record): projection adjoint 243 -> 18 us; from 131,000 records on the stream is faster
//    (three 1024x768 views of 65,536 Gaussians 39 us against 52).
constexpr int kSumRecs = 256;
constexpr int kSumChunk = 256;    // instances per LDS chunk (10 KiB)
constexpr int kSumSerial = 64;    // most tiles a thread adds by itself
constexpr int kSumLanes = 16;     // lanes per record of the few-record kernel
constexpr int kSumWide = 256;     // ... which gives longer records a whole wave
constexpr int64_t kSumFew = 1 << 16;

// The current generation's slots [first, first + nt) summed by W neighbouring
// lanes (sub: this lane's index among them); every lane gets the sums.
template <int W>
__device__ __forceinline__ void sum_slots(const float* __restrict__ inst_grad, int64_t first, int32_t nt, uint32_t gen,
                                          int sub, float s9[9]) {
#pragma unroll
    for (int k = 0; k < 9; k++) s9[k] = 0.0f;
#pragma unroll 2
    for (int32_t u = sub; u < nt; u += W) {
        const float* src = inst_grad + (first + u) * kSlotWords;
        float x[kSlotWords];
#pragma unroll
        for (int k = 0; k < kSlotWords; k++) x[k] = src[k];
        const bool now = __float_as_uint(x[kSlotWords - 1]) == gen;      // written this step
#pragma unroll
        for (int k = 0; k < 9; k++) s9[k] += now ? x[k] : 0.0f;
    }
#pragma unroll
    for (int o = W / 2; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < 9; k++) s9[k] += __shfl_xor(s9[k], o, 64);
}

// A record's slots: the first and their number (0 after an overflowed sort).
// The kept tiles come from the slot offsets (an exclusive scan of them over
// every record), so the 16-byte bins need not be read.
__device__ __forceinline__ int32_t slot_range(const int32_t* __restrict__ inst_first,
                                              const int64_t* __restrict__ n_inst_dev, int64_t cap, int64_t gv,
                                              int64_t n_gv, int64_t& first) {
    first = 0;
    if (gv >= n_gv || *n_inst_dev > cap) return 0;
    first = inst_first[gv];
    return (int32_t)((gv + 1 < n_gv ? (int64_t)inst_first[gv + 1] : *n_inst_dev) - first);
}

__global__ __launch_bounds__(256) void k_slot_sum_few(const int32_t* __restrict__ inst_first,
                                                      const int64_t* __restrict__ n_inst_dev, int64_t cap,
                                                      const float* __restrict__ inst_grad, int64_t n_gv,
                                                      float* __restrict__ grad2d) {
    const int64_t gv = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kSumLanes;
    const int lane = threadIdx.x & 63, sub = lane % kSumLanes;
    const uint32_t gen = (uint32_t)n_inst_dev[1];
    int64_t first;
    const int32_t nt = slot_range(inst_first, n_inst_dev, cap, gv, n_gv, first);
    float s9[9];
    sum_slots<kSumLanes>(inst_grad, first, nt <= kSumWide ? nt : 0, gen, sub, s9);
    uint64_t wide = __ballot(nt > kSumWide && sub == 0);
    while (wide) {
        const int src = __builtin_ctzll(wide);
        wide &= wide - 1;
        float w9[9];
        sum_slots<64>(inst_grad, __shfl(first, src, 64), __shfl(nt, src, 64), gen, lane, w9);
        if (lane / kSumLanes == src / kSumLanes) {
#pragma unroll
            for (int k = 0; k < 9; k++) s9[k] = w9[k];
        }
    }
    if (gv < n_gv && sub < 9) {
        float v = s9[0];
#pragma unroll
        for (int k = 1; k < 9; k++) v = sub == k ? s9[k] : v;
        grad2d[(int64_t)sub * n_gv + gv] = v;
    }
}

__global__ __launch_bounds__(kSumRecs) void k_slot_sum(const int32_t* __restrict__ inst_first,
                                                       const int64_t* __restrict__ n_inst_dev, int64_t cap,
                                                       const float* __restrict__ inst_grad, int64_t n_gv,
                                                       float* __restrict__ grad2d) {
    __shared__ float s_g[kSumChunk * kSlotWords];
    __shared__ int64_t s_range[2];
    __shared__ int32_t s_end[kSumRecs];         // the records' last slots + 1, from the group's first
    __shared__ uint64_t s_skip[kSumRecs / 64];  // which of them are long, or have no slots
    const int64_t g0 = (int64_t)blockIdx.x * kSumRecs;
    const int64_t gv = g0 + threadIdx.x;
    const int64_t glast = imin(g0 + kSumRecs, n_gv) - 1;
    const uint32_t gen = (uint32_t)n_inst_dev[1];
    int64_t first;
    const int32_t nt = slot_range(inst_first, n_inst_dev, cap, gv, n_gv, first);
    const bool is_long = nt > kSumSerial;
    const int lane = threadIdx.x & 63;
    if (gv == g0) s_range[0] = first;
    if (gv == glast) s_range[1] = first + nt;
    const uint64_t wave_skip = __ballot(is_long || nt == 0);
    if (lane == 0) s_skip[threadIdx.x / 64] = wave_skip;
    const bool any_long = __syncthreads_or(is_long);
    const int64_t e0 = s_range[0], e1 = s_range[1];
    s_end[threadIdx.x] = (int32_t)((gv < glast ? first + nt : e1) - e0);
    __syncthreads();
    int32_t end[kSumRecs / 64];
#pragma unroll
    for (int q = 0; q < kSumRecs / 64; q++) end[q] = s_end[q * 64 + lane];
    // the next slot from c on that is not a long record's: where c's record is long, the
    // start of the next one that is not (wave-uniform; each lane knows four records' ends)
    auto next_short = [&](int64_t c) __attribute__((always_inline)) {
        if (!any_long || c >= e1) return c;
        int32_t r = 0;
#pragma unroll
        for (int q = 0; q < kSumRecs / 64; q++) r += __popcll(__ballot(end[q] <= (int32_t)(c - e0)));
        if (!((s_skip[r / 64] >> (r % 64)) & 1)) return c;
        int32_t to = kSumRecs;
#pragma unroll
        for (int q = kSumRecs / 64 - 1; q >= 0; q--) {
            const uint64_t from = r <= q * 64 ? ~0ull : (r < q * 64 + 64 ? ~0ull << (r - q * 64) : 0ull);
            const uint64_t m = ~s_skip[q] & from;
            if (m) to = q * 64 + __builtin_ctzll(m);
        }
        return e0 + s_end[to - 1];      // to > r: a record follows one
    };
    float s9[9];
#pragma unroll
    for (int k = 0; k < 9; k++) s9[k] = 0.0f;
    for (int64_t c0 = next_short(e0); c0 < e1; c0 = next_short(c0 + kSumChunk)) {
        const int64_t c1 = imin(e1, c0 + kSumChunk);
        const int32_t nw = (int32_t)((c1 - c0) * kSlotWords);
        __syncthreads();
        const float* src = inst_grad + c0 * kSlotWords;
        float x[kSlotWords];
#pragma unroll
        for (int r = 0; r < kSlotWords; r++) {
            const int32_t w = r * kSumRecs + threadIdx.x;
            x[r] = w < nw ? src[w] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < kSlotWords; r++) s_g[r * kSumRecs + threadIdx.x] = x[r];
        __syncthreads();
        if (is_long) continue;
        const int32_t a = (int32_t)(imax(first, c0) - c0), b = (int32_t)(imin(first + nt, c1) - c0);
        for (int32_t u = a; u < b; u++) {
            if (__float_as_uint(s_g[u * kSlotWords + kSlotWords - 1]) != gen) continue;   // not written this step
#pragma unroll
            for (int k = 0; k < 9; k++) s9[k] += s_g[u * kSlotWords + k];
        }
    }
    uint64_t todo = __ballot(is_long);
    while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        float w9[9];
        sum_slots<64>(inst_grad, __shfl(first, src, 64), __shfl(nt, src, 64), gen, lane, w9);
        if (lane == src) {
#pragma unroll
            for (int k = 0; k < 9; k++) s9[k] = w9[k];
        }
    }
    if (gv <= glast) {
#pragma unroll
        for (int k = 0; k < 9; k++) grad2d[(int64_t)k * n_gv + gv] = s9[k];
    }
}

}  // namespace

hipError_t launch_flow_mask(const pg_views* v, const float* params, const uint8_t* masks, uint8_t* tile_motion,
                            uint8_t* dyn_gauss, const int32_t* texel_gauss, int64_t HW, uint8_t* dyn_texel,
                            uint64_t* counters, hipStream_t s) {
    const int64_t nfn = (int64_t)v->frames * v->n_gauss;
    if (nfn > 0) k_fill_u8<<<(unsigned)ceil_div(nfn, 256), 256, 0, s>>>(dyn_gauss, nfn);
    if (v->n_tiles > 0) {
        const int tiles = v->n_tiles > kMotionMany ? kMotionTiles : 1;
        auto* kernel = tiles == 1 ? k_tile_motion<1> : k_tile_motion<kMotionTiles>;
        kernel<<<(unsigned)ceil_div(v->n_tiles, 8 * tiles), 256, 0, s>>>(
            v->d_views, v->n_views, v->n_tiles, v->n_pixels, v->tiling.tile_w, masks, tile_motion);
    }
    if (v->n_gv > 0) {
        // Few records: smaller chunks, so that they spread over the chip (2,048 Gaussians per
        // group / this rule: 10 views of 12,800 Gaussians 109 / 49 us, 30 of 90,000 176 / 146)
        const int64_t want = ceil_div(v->n_gv, kFlowFill * kFlowThreads);
        const int32_t recs = kFlowThreads * (int32_t)imin(want, kFlowRecs / kFlowThreads);
        const int64_t per = ceil_div(ceil_div(v->n_gauss, recs), 8);
        // Groups of one or two rounds run beside each other and see no labels yet (collecting
        // there: 30 views of 72 k Gaussians 139 / 142 us, 2 of 432 k 107 / 110).
        const int32_t open = 8 * per * v->n_views > 2 * kFlowFill;
        k_flow_mask<<<(unsigned)(8 * per * v->n_views), kFlowThreads, kFlowSpare, s>>>(
            v->d_views, v->n_views, v->channels, v->n_gauss, recs, open, v->n_tiles, v->n_pixels, v->tiling.tile_w, v->tiling.tile_h,
            params, masks, tile_motion, dyn_gauss, reinterpret_cast<unsigned long long*>(counters));
    }
    if (dyn_texel && HW > 0)
        k_dyn_texel<<<(unsigned)ceil_div(HW, 256), 256, 0, s>>>(dyn_gauss, texel_gauss, HW, v->frames, v->n_gauss,
                                                               dyn_texel);
    return hipGetLastError();
}

hipError_t launch_project(const pg_views* v, const float* params, pg_splat* splats, pg_bin* bins,
                          pg_tile_set* tiles, uint8_t* visible, hipStream_t s) {
    const int64_t n = (int64_t)v->frames * v->n_gauss;
    if (n == 0) return hipSuccess;
    const int64_t groups = ceil_div(v->n_gauss, kProjBlk);
    // View chunks where the Gaussians alone do not fill the chip (4,096 Gaussians in 16 views:
    // 135 -> 14 us; 65,536 in 8 views 59 -> 29 us); with enough work-groups the world chain
    // run once per chunk costs more than the extra ones hide (8 to 25 views per group were
    // no faster than 50 at 2,286 groups).
    const int64_t chunks = imin(ceil_div(kProjFill, groups * v->frames), ceil_div(v->n_views, v->frames));
    const dim3 grid((unsigned)groups, (unsigned)v->frames, (unsigned)imax(chunks, 1));
    const bool split = v->sh_degree >= 2 && ceil_div(v->n_views, v->frames * imax(chunks, 1)) > kSplitViews;
    auto args = [&](auto kern) {
        kern<<<grid, split ? proj_threads<true>() : proj_threads<false>(), 0, s>>>(
            v->d_views, v->d_frame_views, v->d_view_order, v->channels, v->n_gauss, v->tiling.tile_w,
            v->tiling.tile_h, params, splats, bins, tiles, visible);
    };
    switch (v->sh_degree) {
        case 0: args(k_project<0, false>); break;
        case 1: args(k_project<1, false>); break;
        case 2: args(split ? k_project<2, true> : k_project<2, false>); break;
        default: args(split ? k_project<3, true> : k_project<3, false>); break;
    }
    return hipGetLastError();
}

hipError_t launch_slot_sum(const pg_views* v, const int32_t* inst_first,
                           const int64_t* n_inst_dev, int64_t cap, const float* inst_grad, float* grad2d,
                           hipStream_t s) {
    if (v->n_gv == 0) return hipSuccess;
    if (v->n_gv <= kSumFew)
        k_slot_sum_few<<<(unsigned)ceil_div(v->n_gv * kSumLanes, 256), 256, 0, s>>>(inst_first, n_inst_dev, cap,
                                                                                    inst_grad, v->n_gv, grad2d);
    else
        k_slot_sum<<<(unsigned)ceil_div(v->n_gv, kSumRecs), kSumRecs, 0, s>>>(inst_first, n_inst_dev, cap, inst_grad,
                                                                              v->n_gv, grad2d);
    return hipGetLastError();
}

hipError_t launch_project_bwd(const pg_views* v, const float* params, const pg_splat* splats, float* grad2d,
                              const int32_t* gauss_texel, const uint8_t* dyn, int32_t H, int32_t W,
                              float* dL_datlas, int32_t accumulate, hipStream_t s) {
    const int64_t HW = (int64_t)H * W;
    if (!accumulate) {
        hipError_t e = fill_u32(dL_datlas, 0u, (int64_t)v->frames * v->channels * HW, s);
        if (e != hipSuccess) return e;
    }
    const int64_t n = (int64_t)v->frames * v->n_gauss;
    if (n == 0) return hipGetLastError();
    const dim3 grid((unsigned)ceil_div(v->n_gauss, 128), (unsigned)v->frames);
    k_project_bwd_geo<<<grid, 128, 0, s>>>(v->d_views, v->d_frame_views, v->d_view_order, v->frames, v->channels,
                                           v->n_gauss, v->n_gv, params, grad2d, gauss_texel, dyn, HW, dL_datlas,
                                           accumulate);
    auto args = [&](auto kern) {
        kern<<<grid, 128, 0, s>>>(v->d_views, v->d_frame_views, v->d_view_order, v->frames, v->channels, v->n_gauss,
                                  v->n_gv, params, splats, grad2d, gauss_texel, dyn, HW, dL_datlas, accumulate);
    };
    switch (v->sh_degree) {
        case 0: args(k_project_bwd_sh<0>); break;
        case 1: args(k_project_bwd_sh<1>); break;
        case 2: args(k_project_bwd_sh<2>); break;
        default: args(k_project_bwd_sh<3>); break;
    }
    return hipGetLastError();
}

}  // namespace pg
