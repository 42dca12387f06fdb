// Factorised sparse approximate inverse of the RCS (Kolotilina-Yeremin FSAI
// on the lower pattern of Eq. (4)'s camera blocks): M^-1 = G^T G with G
// block-lower-triangular, row i non-zero in the columns J_i (camera i and
// up to kFsaiM - 1 lower neighbours).  Row i is the last block row of the
// inverse Cholesky factor of the local matrix S[J_i, J_i]:
//   S[J_i, J_i] = L L^T  =>  G_i = E_i^T L^-1,
// which satisfies (G_i S)_j = 0 for j in J_i, j != i and G_i S G_i^T = I,
// with G_ii lower triangular with positive diagonal.
//
// The local matrix is factored in FP32 in LDS after block-Jacobi
// normalisation (its diagonal blocks become I):
//   Ahat_jk = L_j^-1 S_jk L_k^-T,  S_jj = L_j L_j^T,
// and the result is mapped back: G_ij = Ghat_ij L_j^-1.  G is written in
// three layouts: the RCS block slots (for copies out), by rows of G and by
// rows of G^T (the two products of the PCG).
#include "ba_common.hpp"

namespace ba {

namespace {

constexpr int BS = 256;

__device__ __forceinline__ int tix(int a, int b) { return a * (a + 1) / 2 + b; }

// An[kb] = L_r^-1 S_rc L_c^-T for the off-diagonal blocks, three blocks per
// workgroup (81 threads each); FP64 arithmetic, FP32 result.
__global__ __launch_bounds__(BS) void k_fsai_norm(int64_t n_blk, const int32_t* __restrict__ brow,
                                                  const int32_t* __restrict__ col_idx, const double* __restrict__ blk,
                                                  const double* __restrict__ Linv, float* __restrict__ An) {
    __shared__ double sS[3][81], sLr[3][81], sLc[3][81], sW[3][81];
    const int lb = threadIdx.x / 81, pq = threadIdx.x % 81;
    const int64_t kb = (int64_t)blockIdx.x * 3 + lb;
    const bool act = lb < 3 && kb < n_blk;
    int r = 0, c = 0;
    if (act) {
        r = brow[kb];
        c = col_idx[kb];
        sS[lb][pq] = blk[kb * 81 + pq];
        sLr[lb][pq] = Linv[(int64_t)r * 81 + pq];
        sLc[lb][pq] = Linv[(int64_t)c * 81 + pq];
    }
    __syncthreads();
    const int p = pq / 9, q = pq % 9;
    if (act && r != c) {
        double w = 0.0;   // W = L_r^-1 S: W[p][q] = sum_{u <= p} Lr[p][u] S[u][q]
        for (int u = 0; u <= p; ++u) w += sLr[lb][p * 9 + u] * sS[lb][u * 9 + q];
        sW[lb][pq] = w;
    }
    __syncthreads();
    if (act && r != c) {
        double a = 0.0;   // W L_c^-T: sum_{v <= q} W[p][v] Lc[q][v]
        for (int v = 0; v <= q; ++v) a += sW[lb][p * 9 + v] * sLc[lb][q * 9 + v];
        An[kb * 81 + pq] = (float)a;
    }
}

__device__ __forceinline__ float lane_value(float v, int l) {   // l: the same for all lanes
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ __forceinline__ float quotient(float v, float root, float inv) {   // v / root, the product corrected once
    const float w = v * inv;
    return fmaf(fmaf(-w, root, v), inv, w);
}

// Cholesky of a 9x9 SPD tile by one wave: lane r < 9 holds row r, a pivot's
// column reaches the other lanes as scalars.  a: row r of L (above the
// diagonal: undefined); root, inv: L's diagonal and its reciprocals.  Returns
// false if a pivot was not positive.
__device__ __forceinline__ bool chol9(const float* T, int lane, float* a, float* root, float* inv) {
    const int r = min(lane, 8);
#pragma unroll
    for (int q = 0; q < 9; ++q) a[q] = T[r * 9 + q];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const float d = lane_value(a[k], k);
        ok = ok && d > 0.f;
        // 1 / sqrt(d) and sqrt(d), each corrected once
        const float d1 = d > 0.f ? d : 1.f;
        float y = __builtin_amdgcn_rsqf(d1), s = d1 * y;
        s = fmaf(0.5f * y, fmaf(-s, s, d1), s);
        y = fmaf(y, fmaf(-s, y, 1.f), y);
        root[k] = s;
        inv[k] = y;
        const float l = quotient(a[k], s, y);   // L[r][k] in the lanes r >= k
        a[k] = l;
#pragma unroll
        for (int c = k + 1; c < 9; ++c) a[c] -= l * lane_value(l, c);
    }
    return ok;
}

// One workgroup per RCS row: up to 28 tiles a side, 406 of 324 bytes in LDS, so
// one workgroup a CU, and the time is a row's chain of m steps (a 2,000-camera
// grid's rows hold about 20 tiles a side).  So a step is kept short:
//   - the waves that have panel rows factor the diagonal tile each for itself,
//     in registers: no barrier between the two, and no division in the panel;
//   - the trailing matrix stays in registers, three rows of a tile per thread
//     (tasks in order of their column, so that whole waves fall idle as the
//     columns are done); a column goes to LDS when its turn comes;
//   - the last block row of the inverse is found from right to left with the
//     sums kept in registers and the stored inverses of the diagonal factors.
// Two barriers a step each way.  Measured against 256 threads with the trailing
// matrix in LDS, the factor by one wave through shuffles and divisions in the
// panel: 300 rows of 28 tiles a side 525 -> 226 us, 2,000 rows 1,387 -> 618.
// (Panel rows as products with the factor's inverse: 230 and 625 us, but an
// error against FP64 1.1 to 3 times as large; this form's is that of before:
// 6.8e-8, 6.2e-8, 7.3e-8 and 1.0e-7 of G's norm on four blocks, 6.8e-8, 6.9e-8,
// 7.2e-8 and 1.0e-7 before.)
constexpr int FT = 1024;
constexpr int kOwn = (kFsaiTiles * 3 + FT - 1) / FT;            // tile thirds of a thread
constexpr int kOwnR = ((kFsaiM - 1) * 81 + FT - 1) / FT;        // sums of the last row of a thread

__global__ __launch_bounds__(FT) void k_fsai(const int32_t* __restrict__ fs_ptr, const int32_t* __restrict__ fs_J,
                                             const int32_t* __restrict__ fs_slot, const int64_t* __restrict__ fs_tptr,
                                             const int32_t* __restrict__ fs_tile, const float* __restrict__ An,
                                             const double* __restrict__ Linv, const int32_t* __restrict__ gu_pos,
                                             float* __restrict__ G, float* __restrict__ Gl, float* __restrict__ Gu,
                                             int* __restrict__ flags) {
    extern __shared__ float sT[];   // tiles (a, b), a >= b
    __shared__ float sP[81];
    __shared__ int s_bad;
    const int row = blockIdx.x;
    const int j0 = fs_ptr[row], m = fs_ptr[row + 1] - j0;
    const int32_t* tiles = fs_tile + fs_tptr[row];
    const int nt = m * (m + 1) / 2, last = m - 1;
    const int tid = threadIdx.x, lane = tid % kWave;
    auto tile = [&](int a, int b) { return sT + tix(a, b) * 81; };
    // tiles (a, b), a >= b: Ahat(J_a, J_b) = An[(J_b, J_a)]^T
    float acc[kOwn][27];
    int ta[kOwn], tc[kOwn], tp[kOwn];   // tile (ta, tc), rows tp .. tp + 2; tc = -1: none
#pragma unroll
    for (int s = 0; s < kOwn; ++s) {
        const int task = tid + s * FT;
        ta[s] = 0; tc[s] = -1; tp[s] = task % 3 * 3;
        if (task >= nt * 3) continue;
        const int rev = nt - 1 - task / 3;   // column by column, from the last one backwards
        int w = (int)((sqrtf(8.f * (float)rev + 1.f) - 1.f) * 0.5f);
        if ((w + 1) * (w + 2) / 2 <= rev) ++w;
        if (w * (w + 1) / 2 > rev) --w;
        tc[s] = last - w;
        ta[s] = last - (rev - w * (w + 1) / 2);
        const int kb = tiles[tix(ta[s], tc[s])];
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int p = tp[s] + r;
                acc[s][r * 9 + q] = kb == -2 ? (p == q ? 1.f : 0.f) : kb < 0 ? 0.f : An[(int64_t)kb * 81 + q * 9 + p];
            }
        if (tc[s] == 0)
#pragma unroll
            for (int v = 0; v < 27; ++v) tile(ta[s], 0)[tp[s] * 9 + v] = acc[s][v];
    }
    if (tid == 0) s_bad = 0;
    for (int b = 0; b < m; ++b) {
        __syncthreads();   // column b is in LDS
        const int np = (last - b) * 9;   // panel rows
        float l[9];
        if (tid - lane < max(np, 1)) {
            float root[9], inv[9];
            const bool ok = chol9(tile(b, b), lane, l, root, inv);
            if (!ok && tid == 0) s_bad = 1;
            // L_ab L_bb^T = T_ab, row p by forward substitution
            float* Tr = tid < np ? tile(b + 1 + tid / 9, b) + tid % 9 * 9 : sP;
            float t[9];
#pragma unroll
            for (int u = 0; u < 9; ++u) t[u] = tid < np ? Tr[u] : 0.f;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                t[q] = quotient(t[q], root[q], inv[q]);
#pragma unroll
                for (int u = q + 1; u < 9; ++u) t[u] -= t[q] * lane_value(l[q], u);
            }
            if (tid < np)
#pragma unroll
                for (int q = 0; q < 9; ++q) Tr[q] = t[q];
        }
        __syncthreads();
        if (tid < 9)
#pragma unroll
            for (int q = 0; q < 9; ++q) tile(b, b)[tid * 9 + q] = l[q];
        // trailing update: T_ac -= L_ab L_cb^T for b < c <= a
#pragma unroll
        for (int s = 0; s < kOwn; ++s) {
            if (tc[s] <= b) continue;
            const float* La = tile(ta[s], b) + tp[s] * 9;
            const float* Lc = tile(tc[s], b);
            float lr[27];
#pragma unroll
            for (int v = 0; v < 27; ++v) lr[v] = La[v];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                float lc[9];
#pragma unroll
                for (int u = 0; u < 9; ++u) lc[u] = Lc[q * 9 + u];
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    float v = 0.f;
#pragma unroll
                    for (int u = 0; u < 9; ++u) v += lr[r * 9 + u] * lc[u];
                    acc[s][r * 9 + q] -= v;
                }
            }
            if (tc[s] == b + 1)
#pragma unroll
                for (int v = 0; v < 27; ++v) tile(ta[s], b + 1)[tp[s] * 9 + v] = acc[s][v];
        }
    }
    __syncthreads();
    // the inverses of the diagonal factors, all at once: a column per thread
    {
        const int c = tid % 9, b = tid / 9;
        float x[9];
        if (b < m) {
            const float* L = tile(b, b);
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                float v = r == c ? 1.f : 0.f;
#pragma unroll
                for (int q = 0; q < r; ++q) v -= L[r * 9 + q] * x[q];
                x[r] = r < c ? 0.f : v / L[r * 9 + r];
            }
        }
        __syncthreads();
        if (b < m)
#pragma unroll
            for (int r = 0; r < 9; ++r) tile(b, b)[r * 9 + c] = x[r];
        __syncthreads();
    }
    // last block row of L^-1: R_last = L_last,last^-1; for b < last
    // R_b = -(sum_{a > b} R_a L_ab) L_bb^-1.  R_b is kept in tile (last, b),
    // whose L_last,b every sum takes in the first step.
    float sum[kOwnR];
#pragma unroll
    for (int s = 0; s < kOwnR; ++s) sum[s] = 0.f;
    for (int a = last; a > 0; --a) {
        const float* Ra = tile(last, a);
#pragma unroll
        for (int s = 0; s < kOwnR; ++s) {
            const int e = tid + s * FT, b = e / 81, pq = e % 81, p = pq / 9, q = pq % 9;
            if (b >= a) continue;
            const float* Lab = tile(a, b);
            float v = 0.f;
#pragma unroll
            for (int u = 0; u < 9; ++u) v += Ra[p * 9 + u] * Lab[u * 9 + q];
            sum[s] += v;
            if (b == a - 1) sP[pq] = -sum[s];
        }
        __syncthreads();
        if (tid < 81) {
            const int p = tid / 9, q = tid % 9;
            const float* Li = tile(a - 1, a - 1);
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < 9; ++u) v += (double)sP[p * 9 + u] * (double)Li[u * 9 + q];
            tile(last, a - 1)[tid] = (float)v;
        }
        __syncthreads();
    }
    // G_{i, J_b} = R_b L_{J_b}^-1 (FP64 accumulation); block-Jacobi row if
    // the local factorisation failed
    const bool bad = s_bad != 0;
    for (int e = tid; e < m * 81; e += FT) {
        const int b = e / 81, pq = e % 81, p = pq / 9, q = pq % 9;
        const int j = fs_J[j0 + b];
        const double* Lj = Linv + (int64_t)j * 81;
        double s = 0.0;
        if (!bad) {
            const float* Rb = tile(last, b);
            for (int u = q; u < 9; ++u) s += (double)Rb[p * 9 + u] * Lj[u * 9 + q];
        } else if (b == last) {
            s = Lj[pq];
        }
        const float g = (float)s;
        G[(int64_t)fs_slot[j0 + b] * 81 + pq] = g;
        Gl[(int64_t)(j0 + b) * 81 + pq] = g;
        Gu[(int64_t)gu_pos[j0 + b] * 81 + q * 9 + p] = g;
    }
    if (bad && tid == 0) atomicAdd(flags + 2, 1);
}

}  // namespace

void launch_fsai(ba_ctx* c) {
    const int64_t nb = c->n_blk;
    if (nb > 0)
        k_fsai_norm<<<(unsigned)((nb + 2) / 3), BS, 0, c->stream>>>(nb, c->fs.brow, c->col_idx, c->blk, c->Linv,
                                                                    c->fs.An);
    const size_t lds = (size_t)c->fs.max_m * (c->fs.max_m + 1) / 2 * 81 * sizeof(float);
    if (c->n_rows > 0)
        k_fsai<<<c->n_rows, FT, lds, c->stream>>>(c->fs.ptr, c->fs.J, c->fs.slot, c->fs.tptr, c->fs.tile, c->fs.An,
                                                c->Linv, c->upper ? c->fs.gl_self : c->fs.gu_pos, c->fs.G, c->fs.Gl,
                                                c->fs.Gu, c->flags);
    c->fs.gu_upper = c->upper;
}

}  // namespace ba
