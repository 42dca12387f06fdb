// Re-triangulation of points with the cameras held fixed: the alternative to
// the back-substitution of Eq. (5) that Sec. 3.1 names (points re-estimated
// from the camera poses), and the third costly step Sec. 6 lists.
//
// Per point, over its track:
//   - optional linear start: each observed pixel is undistorted (the radius
//     r of the normalised image point solves r (1 + k1 r^2 + k2 r^4) =
//     |pixel| / f, Newton from r = |pixel| / f) to (x, y) with R X + t
//     parallel to (x, y, 1); the equations (x R_3 - R_1) X = t_1 - x t_3,
//     (y R_3 - R_2) X = t_2 - y t_3 of all observations are solved in the
//     least-squares sense through their 3x3 normal matrix;
//   - n_gn Gauss-Newton steps on the point's reprojection error:
//     X += (sum J_p^T J_p)^-1 (-sum J_p^T e).
// One wave per chunk of whole tracks, one lane per observation (the layout
// of the point stage): lanes form their terms and sum them together through
// LDS (nine sums shared by the track's lanes: with one lane forming all nine,
// its reads of up to 12 x 9 values an iteration kept LDS busy for half the
// time), and every lane solves the 3x3 system for itself (the wave takes as
// long with one lane at work), so X needs no way back through LDS.
//
// Bound by FP64 arithmetic (24 bytes an observation).  A lane's rotation
// matrix does not change over the steps and is formed once; the undistortion
// stops where Newton's quadratic convergence has reached the last bit (its
// step never fell under 1e-17 of the radius, so it ran to its limit of 60).
// 9.4M observations, linear start and 4 steps: 1,300 us before, 615 now.
#include "ba_common.hpp"

namespace ba {

namespace {

constexpr int BS = 256;
constexpr int WPB = BS / kWave;

// s = (A00 A01 A02 A11 A12 A22, b0 b1 b2): x = A^-1 b by L D L^T (one
// division a pivot, no square root); false unless A is positive definite
__device__ __forceinline__ bool solve3(const double* s, double* x) {
    const double i0 = 1.0 / s[0];
    const double l10 = s[1] * i0, l20 = s[2] * i0;
    const double d1 = s[3] - l10 * s[1];
    const double i1 = 1.0 / d1;
    const double t21 = s[4] - l20 * s[1];
    const double l21 = t21 * i1;
    const double d2 = s[5] - l20 * s[2] - l21 * t21;
    const double y1 = s[7] - l10 * s[6];
    const double y2 = s[8] - l20 * s[6] - l21 * y1;
    x[2] = y2 / d2;
    x[1] = y1 * i1 - l21 * x[2];
    x[0] = s[6] * i0 - l10 * x[1] - l20 * x[2];
    return s[0] > 0.0 && d1 > 0.0 && d2 > 0.0 && isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]);
}

// radius of the normalised image point whose distorted radius is rho (after
// a step of 1e-10 of the radius the next one is below its last bit)
__device__ __forceinline__ double undistort_radius(double rho, double k1, double k2) {
    double r = rho;
    for (int it = 0; it < 60; ++it) {
        const double r2 = r * r;
        const double g = r * (1.0 + k1 * r2 + k2 * r2 * r2) - rho;
        const double dg = 1.0 + 3.0 * k1 * r2 + 5.0 * k2 * r2 * r2;
        const double step = g / dg;
        r -= step;
        if (fabs(step) <= 1e-10 * fabs(r)) break;
    }
    return r;
}

// R(w) = I + a [w]x + b [w]x^2 as diag(s) + D, row-major: s_i = 1 or -1, whichever
// is next to R_ii, which leaves small entries of D that carry no rounding of
// entries near 1: D_ii = -b (|w|^2 - w_i^2), or with 1 + cos|w| = a^2 / b (since
// sin^2 = (1 - cos)(1 + cos)) D_ii = a^2 / b + b w_i^2
struct Rot {
    double D[9];
    int neg;   // bit i: s_i = -1
    __device__ __forceinline__ double s(int i, double v) const { return (neg >> i & 1) ? -v : v; }
};
__device__ __forceinline__ void rotation(const double* w, Rot& R) {
    const double s2[3] = {w[0] * w[0], w[1] * w[1], w[2] * w[2]};
    double a, b, as, bs;
    rot_coeffs(s2[0] + s2[1] + s2[2], a, b, as, bs);
    const double opc = a * a / b;
    const double m[3] = {b * (s2[1] + s2[2]), b * (s2[0] + s2[2]), b * (s2[0] + s2[1])};
    R.neg = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const bool neg = m[i] > 1.0;
        R.neg |= (int)neg << i;
        R.D[i * 4] = neg ? opc + b * s2[i] : -m[i];
    }
    R.D[1] = -a * w[2] + b * w[0] * w[1]; R.D[2] = a * w[1] + b * w[0] * w[2];
    R.D[3] = a * w[2] + b * w[1] * w[0]; R.D[5] = -a * w[0] + b * w[1] * w[2];
    R.D[6] = -a * w[1] + b * w[2] * w[0]; R.D[7] = a * w[0] + b * w[2] * w[1];
}

// The terms of observation (camera c with rotation Q, pixel ou, ov) in the normal equations
// of the linear multi-view solve: A^T A (6 unique) and A^T b of its two rows
// (x R_3 - R_1) X = t_1 - x t_3, (y R_3 - R_2) X = t_2 - y t_3.
__device__ __forceinline__ void tri_linear_terms(const double* c, const Rot& Q, double ou, double ov, double* m) {
    const double* D = Q.D;
    const double R[9] = {Q.s(0, 1.0) + D[0], D[1], D[2], D[3], Q.s(1, 1.0) + D[4], D[5], D[6], D[7], Q.s(2, 1.0) + D[8]};
    const double rho = sqrt(ou * ou + ov * ov) / c[6];
    double x = 0.0, y = 0.0;
    if (rho > 0.0) {
        const double r = undistort_radius(rho, c[7], c[8]);
        x = ou / c[6] * (r / rho);
        y = ov / c[6] * (r / rho);
    }
    const double a1[3] = {x * R[6] - R[0], x * R[7] - R[1], x * R[8] - R[2]};
    const double a2[3] = {y * R[6] - R[3], y * R[7] - R[4], y * R[8] - R[5]};
    const double b1 = c[3] - x * c[5], b2 = c[4] - y * c[5];
    m[0] = a1[0] * a1[0] + a2[0] * a2[0];
    m[1] = a1[0] * a1[1] + a2[0] * a2[1];
    m[2] = a1[0] * a1[2] + a2[0] * a2[2];
    m[3] = a1[1] * a1[1] + a2[1] * a2[1];
    m[4] = a1[1] * a1[2] + a2[1] * a2[2];
    m[5] = a1[2] * a1[2] + a2[2] * a2[2];
    m[6] = a1[0] * b1 + a2[0] * b2;
    m[7] = a1[1] * b1 + a2[1] * b2;
    m[8] = a1[2] * b1 + a2[2] * b2;
}

// The terms of the Gauss-Newton step on the point's reprojection error at X:
// J_p^T J_p (6 unique) and -J_p^T e (the projection and J_p of project_point,
// with the rotation given).  The point is turned by (s X + t) + D X, whose
// first sum is exact or nearly so: R X rounds at the size of X before the
// translation takes most of it away.  Error against 64 bits relative to the
// points' norm, 9.4M observations of strips 900 units long and of a 100 x 100
// block: R X 8.3e-16 and 5.1e-16 (605 us the strips), the projection's
// X + a w x X + b w x (w x X) + t 4.3e-16 and 5.2e-16 (673), (X + t) + (R - I) X
// 3.4e-16 and 5.6e-16 (612), this 3.4e-16 and 4.4e-16 (614).
__device__ __forceinline__ void tri_gn_terms(const double* c, const Rot& Q, const double* X, double ou, double ov,
                                             double* m) {
    const double* D = Q.D;
    const double P0 = (Q.s(0, X[0]) + c[3]) + D[0] * X[0] + D[1] * X[1] + D[2] * X[2];
    const double P1 = (Q.s(1, X[1]) + c[4]) + D[3] * X[0] + D[4] * X[1] + D[5] * X[2];
    const double P2 = (Q.s(2, X[2]) + c[5]) + D[6] * X[0] + D[7] * X[1] + D[8] * X[2];
    const double iz = 1.0 / P2;
    const double x = P0 * iz, y = P1 * iz;
    const double r2 = x * x + y * y;
    const double f = c[6], k1 = c[7], k2 = c[8];
    const double d = 1.0 + r2 * (k1 + k2 * r2);
    const double eu = f * d * x - ou, ev = f * d * y - ov;
    const double dd = k1 + 2.0 * k2 * r2;
    const double A00 = f * (d + 2.0 * x * x * dd), A01 = f * (2.0 * x * y * dd), A11 = f * (d + 2.0 * y * y * dd);
    const double E00 = A00 * iz, E01 = A01 * iz, E02 = -(A00 * x + A01 * y) * iz;
    const double E10 = A01 * iz, E11 = A11 * iz, E12 = -(A01 * x + A11 * y) * iz;
    const double R[9] = {Q.s(0, 1.0) + D[0], D[1], D[2], D[3], Q.s(1, 1.0) + D[4], D[5], D[6], D[7], Q.s(2, 1.0) + D[8]};
    double jp[6];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        jp[j] = E00 * R[j] + E01 * R[3 + j] + E02 * R[6 + j];
        jp[3 + j] = E10 * R[j] + E11 * R[3 + j] + E12 * R[6 + j];
    }
    m[0] = jp[0] * jp[0] + jp[3] * jp[3];
    m[1] = jp[0] * jp[1] + jp[3] * jp[4];
    m[2] = jp[0] * jp[2] + jp[3] * jp[5];
    m[3] = jp[1] * jp[1] + jp[4] * jp[4];
    m[4] = jp[1] * jp[2] + jp[4] * jp[5];
    m[5] = jp[2] * jp[2] + jp[5] * jp[5];
    m[6] = -(jp[0] * eu + jp[3] * ev);
    m[7] = -(jp[1] * eu + jp[4] * ev);
    m[8] = -(jp[2] * eu + jp[5] * ev);
}

// One wave per workgroup: its barriers hold a single wave.  Five waves a SIMD
// asked for: at 100 registers, four without, it took 671 us instead of 621 (two
// spilled) in an earlier form of the terms.
template <bool LINEAR>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(5))) void k_triangulate(int n_chunk, const int32_t* __restrict__ chunk_ptr, int n,
                                                       const int32_t* __restrict__ obs_cam,
                                                       const int32_t* __restrict__ obs_pt,
                                                       const int32_t* __restrict__ obs_row,
                                                       const double* __restrict__ uv, const double* __restrict__ cams,
                                                       const double* __restrict__ dxc, const double* pts,
                                                       double* out, int delta, int n_gn,
                                                       int* __restrict__ n_failed) {
    __shared__ double sA[9][kWave];   // the lanes' terms
    const int lane = threadIdx.x;
    const int chunk = xcd_block();
    const int k0 = chunk_ptr[chunk], k1 = chunk_ptr[chunk + 1];
    const int k = k0 + lane;
    const bool act = k < k1;
    const int p = act ? obs_pt[k] : -1;
    const Track tk = chunk_track(act, p, lane, k1 - k0);
    const int head = tk.head, tl = tk.len;
    double c[9], X[3];
    Rot Q;
    double ou = 0.0, ov = 0.0;
    bool ok = true;   // the same in every lane of a track
    if (act) {
        const double* c0 = cams + (int64_t)obs_cam[k] * 9;
        const int row = obs_row[k];
#pragma unroll
        for (int i = 0; i < 9; ++i) c[i] = c0[i] + ((dxc && row >= 0) ? dxc[(int64_t)row * 9 + i] : 0.0);
        rotation(c, Q);
        ou = uv[k];
        ov = uv[n + k];
        // start: the point as given (out may be pts: the track's lanes all
        // read it before its first lane writes it)
#pragma unroll
        for (int i = 0; i < 3; ++i) X[i] = pts[(int64_t)p * 3 + i] + (delta ? out[(int64_t)p * 3 + i] : 0.0);
    }
    for (int it = LINEAR ? -1 : 0; it < n_gn; ++it) {
        if (act) {
            double m[9];
            if (LINEAR && it < 0) tri_linear_terms(c, Q, ou, ov, m);
            else tri_gn_terms(c, Q, X, ou, ov, m);
#pragma unroll
            for (int j = 0; j < 9; ++j) sA[j][lane] = m[j];
        }
        __syncthreads();
        // the track's lanes share the nine sums: each forms every tl-th one in
        // place of its first term (no other lane reads that row's entries)
        if (act)
            for (int j = lane - head; j < 9; j += tl) {
                double v = 0.0;
                for (int q = 0; q < tl; ++q) v += sA[j][head + q];
                sA[j][head] = v;
            }
        __syncthreads();
        if (act && ok) {
            double sum[9], d[3];
#pragma unroll
            for (int j = 0; j < 9; ++j) sum[j] = sA[j][head];
            ok = solve3(sum, d);
            if (ok)
#pragma unroll
                for (int i = 0; i < 3; ++i) X[i] = LINEAR && it < 0 ? d[i] : X[i] + d[i];
        }
        __syncthreads();
    }
    if (act && head == lane) {
        if (!ok) atomicAdd(n_failed, 1);
#pragma unroll
        for (int i = 0; i < 3; ++i) out[(int64_t)p * 3 + i] = X[i] - (delta ? pts[(int64_t)p * 3 + i] : 0.0);
    }
}

// The same for a track longer than a wave: one workgroup per point, its
// threads striding over the track, sums reduced in a fixed order (strided
// thread sums, the wave's shuffle tree, then the waves in order).
template <bool LINEAR>
__global__ __launch_bounds__(BS) void k_triangulate_long(const int32_t* __restrict__ long_ptr, int n,
                                                         const int32_t* __restrict__ obs_cam,
                                                         const int32_t* __restrict__ obs_pt,
                                                         const int32_t* __restrict__ obs_row,
                                                         const double* __restrict__ uv, const double* __restrict__ cams,
                                                         const double* __restrict__ dxc, const double* __restrict__ pts,
                                                         double* __restrict__ out, int delta, int n_gn,
                                                         int* __restrict__ n_failed) {
    __shared__ double sh[9][WPB];
    __shared__ double sX[3];
    __shared__ int sok;
    const int k0 = long_ptr[blockIdx.x], k1 = long_ptr[blockIdx.x + 1];
    const int p = obs_pt[k0];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (threadIdx.x == 0) {
        for (int i = 0; i < 3; ++i) sX[i] = pts[(int64_t)p * 3 + i] + (delta ? out[(int64_t)p * 3 + i] : 0.0);
        sok = 1;
    }
    __syncthreads();
    auto camera = [&](int k, double* c) {
        const double* c0 = cams + (int64_t)obs_cam[k] * 9;
        const int row = obs_row[k];
#pragma unroll
        for (int i = 0; i < 9; ++i) c[i] = c0[i] + ((dxc && row >= 0) ? dxc[(int64_t)row * 9 + i] : 0.0);
    };
    // sums of the track's terms into sh[m][0] (all threads then read them)
    auto reduce9 = [&](double* v) {
#pragma unroll
        for (int m = 0; m < 9; ++m) {
            const double w = wave_sum(v[m]);
            if (lane == 0) sh[m][wv] = w;
        }
        __syncthreads();
        if (threadIdx.x == 0)
#pragma unroll
            for (int m = 0; m < 9; ++m) {
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < WPB; ++w) t += sh[m][w];
                v[m] = t;
            }
    };
    for (int it = LINEAR ? -1 : 0; it < n_gn; ++it) {
        double v[9];
#pragma unroll
        for (int m = 0; m < 9; ++m) v[m] = 0.0;
        const double X[3] = {sX[0], sX[1], sX[2]};
        for (int k = k0 + threadIdx.x; k < k1; k += BS) {
            double c[9], t[9];
            Rot Q;
            camera(k, c);
            rotation(c, Q);
            if (it < 0) tri_linear_terms(c, Q, uv[k], uv[n + k], t);
            else tri_gn_terms(c, Q, X, uv[k], uv[n + k], t);
#pragma unroll
            for (int m = 0; m < 9; ++m) v[m] += t[m];
        }
        reduce9(v);
        if (threadIdx.x == 0 && sok) {
            double d[3];
            sok = solve3(v, d);
            if (sok)
                for (int i = 0; i < 3; ++i) sX[i] = it < 0 ? d[i] : sX[i] + d[i];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (!sok) atomicAdd(n_failed, 1);
        for (int i = 0; i < 3; ++i) out[(int64_t)p * 3 + i] = sX[i] - (delta ? pts[(int64_t)p * 3 + i] : 0.0);
    }
}

}  // namespace

void launch_triangulate(ba_ctx* c, const double* cams, const double* dxc, const double* pts, double* out, int delta,
                        int linear, int n_gn, int* n_failed) {
    const int nb = c->n_chunk;
    const int n = (int)c->n_obs;
    if (nb > 0) {
        if (linear)
            k_triangulate<true><<<nb, kWave, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, n, c->obs_cam, c->obs_pt,
                                                          c->obs_row, c->obs_uv, cams, dxc, pts, out, delta, n_gn,
                                                          n_failed);
        else
            k_triangulate<false><<<nb, kWave, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, n, c->obs_cam, c->obs_pt,
                                                           c->obs_row, c->obs_uv, cams, dxc, pts, out, delta, n_gn,
                                                           n_failed);
    }
    if (c->n_long > 0) {
        if (linear)
            k_triangulate_long<true><<<c->n_long, BS, 0, c->stream>>>(c->long_ptr, n, c->obs_cam, c->obs_pt,
                                                                      c->obs_row, c->obs_uv, cams, dxc, pts, out,
                                                                      delta, n_gn, n_failed);
        else
            k_triangulate_long<false><<<c->n_long, BS, 0, c->stream>>>(c->long_ptr, n, c->obs_cam, c->obs_pt,
                                                                       c->obs_row, c->obs_uv, cams, dxc, pts, out,
                                                                       delta, n_gn, n_failed);
    }
}

}  // namespace ba
