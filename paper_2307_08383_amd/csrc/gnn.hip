// Learned correction to block-Jacobi preconditioning of the RCS.
//
// A message-passing network over the camera-pair graph (the non-zero blocks
// of the RCS are the camera pairs with common points, Sec. 4) maps each RCS
// instance to per-camera lower-triangular factors Lt_i (diagonal exp(.)),
// giving SPD preconditioner blocks P_i = L_i^-T Lt_i Lt_i^T L_i^-1 with
// S_ii = L_i L_i^T; a zero decoder gives Lt_i = I, i.e. block-Jacobi exactly.
// Training minimises the Hutchinson estimate of ||B A - I||_F^2 / (9 n) in
// the block-Jacobi-normalised space A = L^-1 S L^-T, B = blockdiag(Lt Lt^T).
//
// All dense layers run on bf16 MFMA (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation; weight gradients are split over rows and the partial tiles
// summed in a fixed order, message aggregation is a segmented sum over a
// source-sorted directed edge list and its backward walks each edge's twin,
// so forward, backward and the optimiser are deterministic (no atomics).
#include <algorithm>
#include <stdexcept>
#include <cstring>
#include <vector>

#include "gnn.hpp"
#include "host_par.hpp"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace ba {
namespace gnn {

namespace {

constexpr int BS = 256;
constexpr int KSPLIT_ROWS = 2048;     // rows per weight-gradient partial

inline int nblk(int64_t n, int b = BS) { return (int)((n + b - 1) / b); }

// ---------------------------------------------------------------------------
// GEMM: C[M][N] = sum_k A(m,k) B(k,n) (+ bias[n]) (relu), with
// A(m,k) = A[m*sam + k*sak], B(k,n) = B[k*sbk + n*sbn] in bf16, FP32
// accumulation.  One block computes a 64 x 64 tile over the K range
// [z*kchunk, min(K, (z+1)*kchunk)) and writes it at C + z*zstride.
// Lane layout of v_mfma_f32_16x16x32_bf16: lane l holds A row l%16 and
// B column l%16 for k = 8*(l/16) .. +7; the result lane holds column l%16,
// rows 4*(l/16) .. +3.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_gemm(int M, int N, int K, int kchunk, const __bf16* __restrict__ A,
                                             int64_t sam, int64_t sak, const __bf16* __restrict__ B, int64_t sbk,
                                             int64_t sbn, const float* __restrict__ bias, int relu,
                                             float* __restrict__ C, int64_t ldc, int64_t zstride,
                                             __bf16* __restrict__ Cb, int64_t ldcb) {
    __shared__ __bf16 sA[64][40];
    __shared__ __bf16 sB[32][72];
    const int tid = threadIdx.x, w = tid / kWave, l = tid % kWave;
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int k0 = blockIdx.z * kchunk, k1 = min(K, k0 + kchunk);
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const __bf16 zero = (__bf16)0.0f;
    for (int kb = k0; kb < k1; kb += 32) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int idx = tid + BS * t;
            const int r = idx / 32, c = idx % 32;
            const int m = m0 + r, k = kb + c;
            sA[r][c] = (m < M && k < k1) ? A[(int64_t)m * sam + (int64_t)k * sak] : zero;
            const int rb = idx / 64, cb = idx % 64;
            const int kk = kb + rb, nn = n0 + cb;
            sB[rb][cb] = (kk < k1 && nn < N) ? B[(int64_t)kk * sbk + (int64_t)nn * sbn] : zero;
        }
        __syncthreads();
        bf16x8 a;
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = sA[16 * w + l % 16][8 * (l / 16) + j];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            bf16x8 b;
#pragma unroll
            for (int j = 0; j < 8; ++j) b[j] = sB[8 * (l / 16) + j][16 * nt + l % 16];
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nt], 0, 0, 0);
        }
        __syncthreads();
    }
    float* Cz = C + (int64_t)blockIdx.z * zstride;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + 16 * w + 4 * (l / 16) + i;
            const int n = n0 + 16 * nt + l % 16;
            if (m < M && n < N) {
                float v = acc[nt][i];
                if (bias) v += bias[n];
                if (relu) v = v > 0.f ? v : 0.f;
                Cz[(int64_t)m * ldc + n] = v;
                if (Cb) Cb[(int64_t)m * ldcb + n] = (__bf16)v;
            }
        }
}

// The same product for row-major A [M][K] and B [K][N] (unit column
// strides), K a multiple of 32, N a multiple of 8, rows 16-byte aligned:
// every thread brings one 8-value vector of the A tile and one of the B tile
// per K step; B is stored transposed in LDS so that each MFMA operand is one
// 16-byte LDS read.  Same tiles, lane layout and accumulation order as k_gemm.
// Rows of a message input [h_src, h_dst, g_edge] (3 x H values, bf16) read
// in place: row m is H[src[m]], H[dst[m]], G[eid ? eid[m] : m].
struct GatherRows {
    const int32_t* src;
    const int32_t* dst;
    const int32_t* eid;
    const __bf16* Hn;
    const __bf16* Ge;
};

template <bool GA>
__global__ __launch_bounds__(BS) void k_gemm_v(int M, int N, int K, const __bf16* __restrict__ A, int64_t lda,
                                               GatherRows gr, const __bf16* __restrict__ B, int64_t ldb,
                                               const float* __restrict__ bias, int relu, float* __restrict__ C,
                                               int64_t ldc, __bf16* __restrict__ Cb, int64_t ldcb) {
    __shared__ __align__(16) __bf16 sA[64][40];
    __shared__ __align__(16) __bf16 sBt[64][40];
    const int tid = threadIdx.x, w = tid / kWave, l = tid % kWave;
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int ar = tid / 4, ac = (tid % 4) * 8;   // A tile: row, first k
    const int bk = tid / 8, bn = (tid % 8) * 8;   // B tile: k, first n
    const bool aok = m0 + ar < M, bok = n0 + bn < N;
    const __bf16* Ap = A + (int64_t)(m0 + ar) * lda + ac;
    const __bf16* seg[3] = {nullptr, nullptr, nullptr};   // GA: the row's three H-wide pieces
    if (GA && aok) {
        const int m = m0 + ar;
        seg[0] = gr.Hn + (int64_t)gr.src[m] * H;
        seg[1] = gr.Hn + (int64_t)gr.dst[m] * H;
        seg[2] = gr.Ge + (int64_t)(gr.eid ? gr.eid[m] : m) * H;
    }
    const __bf16* Bp = B + (int64_t)bk * ldb + n0 + bn;
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 zero8;
#pragma unroll
    for (int j = 0; j < 8; ++j) zero8[j] = (__bf16)0.0f;
    for (int kb = 0; kb < K; kb += 32) {
        bf16x8 av = zero8;
        if (aok) {
            if (GA) {
                const int k = kb + ac;   // a vector never straddles two H-wide pieces
                av = *reinterpret_cast<const bf16x8*>(seg[k / H] + k % H);
            } else {
                av = *reinterpret_cast<const bf16x8*>(Ap + kb);
            }
        }
        const bf16x8 bv = bok ? *reinterpret_cast<const bf16x8*>(Bp + (int64_t)kb * ldb) : zero8;
        *reinterpret_cast<bf16x8*>(&sA[ar][ac]) = av;
#pragma unroll
        for (int j = 0; j < 8; ++j) sBt[bn + j][bk] = bv[j];
        __syncthreads();
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&sA[16 * w + l % 16][8 * (l / 16)]);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(&sBt[16 * nt + l % 16][8 * (l / 16)]);
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nt], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + 16 * w + 4 * (l / 16) + i;
            const int n = n0 + 16 * nt + l % 16;
            if (m < M && n < N) {
                float v = acc[nt][i];
                if (bias) v += bias[n];
                if (relu) v = v > 0.f ? v : 0.f;
                C[(int64_t)m * ldc + n] = v;
                if (Cb) Cb[(int64_t)m * ldcb + n] = (__bf16)v;
            }
        }
}

// out[i] = sum_z part[z][i] in order z = 0, 1, ...
__global__ __launch_bounds__(BS) void k_sum_split(int64_t n, int nz, const float* __restrict__ part,
                                                  float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
    for (int z = 0; z < nz; ++z) s += part[(int64_t)z * n + i];
    out[i] = s;
}

// column sums of a row-major [rows][cols] FP32 matrix, first per chunk of
// 1024 rows (partial[chunk][col]), then over chunks in order
__global__ __launch_bounds__(BS) void k_colsum_part(int rows, int cols, const float* __restrict__ src, int64_t ld,
                                                    float* __restrict__ part) {
    const int c = threadIdx.x;
    if (c >= cols) return;
    const int r0 = blockIdx.x * 1024, r1 = min(rows, r0 + 1024);
    float s = 0.f;
    for (int r = r0; r < r1; ++r) s += src[(int64_t)r * ld + c];
    part[(int64_t)blockIdx.x * cols + c] = s;
}

__global__ __launch_bounds__(BS) void k_colsum_fin(int nchunk, int cols, const float* __restrict__ part,
                                                   float* __restrict__ out) {
    const int c = threadIdx.x;
    if (c >= cols) return;
    float s = 0.f;
    for (int z = 0; z < nchunk; ++z) s += part[(int64_t)z * cols + c];
    out[c] = s;
}

__global__ __launch_bounds__(BS) void k_to_bf16(int64_t n, const float* __restrict__ src, __bf16* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i < n) dst[i] = (__bf16)src[i];
}

// ---------------------------------------------------------------------------
// features
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_feat_node(int n, const int32_t* __restrict__ diag_blk,
                                                  const double* __restrict__ blk, double* __restrict__ Linv,
                                                  __bf16* __restrict__ xn, int* __restrict__ flags) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= n) return;
    const double* S = blk + (int64_t)diag_blk[i] * 81;
    double L[81];
    for (int q = 0; q < 81; ++q) L[q] = 0.0;
    bool ok = true;
    for (int j = 0; j < 9; ++j) {
        double s = S[j * 9 + j];
        for (int q = 0; q < j; ++q) s -= L[j * 9 + q] * L[j * 9 + q];
        if (!(s > 0.0)) { ok = false; s = 1.0; }
        L[j * 9 + j] = sqrt(s);
        for (int r = j + 1; r < 9; ++r) {
            double t = S[r * 9 + j];
            for (int q = 0; q < j; ++q) t -= L[r * 9 + q] * L[j * 9 + q];
            L[r * 9 + j] = t / L[j * 9 + j];
        }
    }
    if (!ok) flags[0] = 1;
    // lower-triangular inverse in place
    for (int j = 0; j < 9; ++j) {
        L[j * 9 + j] = 1.0 / L[j * 9 + j];
        for (int r = j + 1; r < 9; ++r) {
            double t = 0.0;
            for (int q = j; q < r; ++q) t -= L[r * 9 + q] * L[q * 9 + j];
            L[r * 9 + j] = t / L[r * 9 + r];
        }
    }
    for (int q = 0; q < 81; ++q) Linv[(int64_t)i * 81 + q] = L[q];
    double d[9], ld[9], mean = 0.0;
    for (int r = 0; r < 9; ++r) {
        d[r] = 1.0 / sqrt(S[r * 9 + r]);
        ld[r] = log(S[r * 9 + r]);
        mean += ld[r];
    }
    mean /= 9.0;
    __bf16* x = xn + (int64_t)i * F_NODE;
    int q = 0;
    for (int r = 0; r < 9; ++r)
        for (int c = r + 1; c < 9; ++c, ++q) x[q] = (__bf16)(S[r * 9 + c] * d[r] * d[c]);
    for (int r = 0; r < 9; ++r) x[36 + r] = (__bf16)(ld[r] - mean);
    for (int r = 45; r < F_NODE; ++r) x[r] = (__bf16)0.0f;
}

// Normalised edge blocks A_e = L_i^-1 S_ij L_j^-T (FP32) and their bf16
// features.  Three edges a pass, one thread per block entry; only the edges
// that apply their stored upper block as is (elow) are computed, and the twin
// (the reverse edge) takes the transpose, A_twin = A_e^T.  The three blocks of
// an edge are staged in LDS with contiguous loads, then the two triangular
// products are formed in two passes (same summation order as a thread-per-edge
// loop).  A workgroup goes through many passes and asks for the next pass's
// blocks before it forms this one's products: with a workgroup per three edges,
// half of them twins that do nothing, 735,000 edges took 613 us, 418 now.
constexpr int kFE = 3;   // edges a pass
__global__ __launch_bounds__(256) void k_feat_edge(int n_low, const int32_t* __restrict__ elow,
                                                   const int32_t* __restrict__ esrc, const int32_t* __restrict__ edst,
                                                   const int32_t* __restrict__ eblk, const int32_t* __restrict__ etwin,
                                                   const double* __restrict__ blk, const double* __restrict__ Linv,
                                                   float* __restrict__ A, __bf16* __restrict__ xe) {
    __shared__ double sS[kFE][81], sLi[kFE][81], sLj[kFE][81], sT[kFE][81];
    const int le = threadIdx.x / 81, pq = threadIdx.x % 81;
    const int r = pq / 9, c = pq % 9;
    double vs = 0.0, vi = 0.0, vj = 0.0;
    int e = -1;
    auto request = [&](int64_t pass) {
        const int64_t at = pass * kFE + le;
        e = le < kFE && at < n_low ? elow[at] : -1;
        if (e < 0) return;
        vs = blk[(int64_t)eblk[e] * 81 + pq];
        vi = Linv[(int64_t)esrc[e] * 81 + pq];
        vj = Linv[(int64_t)edst[e] * 81 + pq];
    };
    const int64_t n_pass = ((int64_t)n_low + kFE - 1) / kFE;
    request(blockIdx.x);
    for (int64_t pass = blockIdx.x; pass < n_pass; pass += gridDim.x) {
        const int cur = e;
        if (cur >= 0) {
            sS[le][pq] = vs;
            sLi[le][pq] = vi;
            sLj[le][pq] = vj;
        }
        __syncthreads();
        request(pass + gridDim.x);
        if (cur >= 0) {   // T = S_ij Lj^T
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if (q <= c) t += sS[le][r * 9 + q] * sLj[le][c * 9 + q];
            sT[le][pq] = t;
        }
        __syncthreads();
        if (cur >= 0) {   // A = Li T
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if (q <= r) t += sLi[le][r * 9 + q] * sT[le][q * 9 + c];
            const int64_t tw = etwin[cur];
            A[(int64_t)cur * 81 + pq] = (float)t;
            A[tw * 81 + c * 9 + r] = (float)t;
            __bf16* x = xe + (int64_t)cur * F_EDGE;
            __bf16* xt = xe + tw * F_EDGE;
            x[pq] = (__bf16)t;
            xt[c * 9 + r] = (__bf16)t;
            if (pq < F_EDGE - 81) {
                x[81 + pq] = (__bf16)0.0f;
                xt[81 + pq] = (__bf16)0.0f;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// message passing pieces
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_gather_msg(int E, const int32_t* __restrict__ esrc, const int32_t* __restrict__ edst,
                                                   const __bf16* __restrict__ Hb, const __bf16* __restrict__ Gb,
                                                   __bf16* __restrict__ Xm) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)E * 3 * H) return;
    const int e = (int)(t / (3 * H)), f = (int)(t % (3 * H));
    __bf16 v;
    if (f < H) v = Hb[(int64_t)esrc[e] * H + f];
    else if (f < 2 * H) v = Hb[(int64_t)edst[e] * H + f - H];
    else v = Gb[(int64_t)e * H + f - 2 * H];
    Xm[t] = v;
}

// Xu[i] = [Hb[i], mean over the edges leaving i of Mm]
__global__ __launch_bounds__(BS) void k_aggregate(int n, const int32_t* __restrict__ eptr, const float* __restrict__ Mm,
                                                  const __bf16* __restrict__ Hb, __bf16* __restrict__ Xu) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)n * H) return;
    const int i = (int)(t / H), f = (int)(t % H);
    float s = 0.f;
    for (int e = eptr[i]; e < eptr[i + 1]; ++e) s += Mm[(int64_t)e * H + f];
    const int deg = eptr[i + 1] - eptr[i];
    if (deg > 0) s /= (float)deg;
    Xu[(int64_t)i * 2 * H + f] = Hb[(int64_t)i * H + f];
    Xu[(int64_t)i * 2 * H + H + f] = (__bf16)s;
}

__global__ __launch_bounds__(BS) void k_residual(int64_t n, float* __restrict__ Hf, const float* __restrict__ T,
                                                 __bf16* __restrict__ Hb) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const float v = Hf[i] + T[i];
    Hf[i] = v;
    Hb[i] = (__bf16)v;
}

// Rademacher probes from a counter-based hash (splitmix64 finaliser)
__global__ __launch_bounds__(BS) void k_probes(int64_t n, unsigned long long seed, float* __restrict__ Z) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    unsigned long long x = seed + 0x9E3779B97F4A7C15ull * (unsigned long long)(i + 1);
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    Z[i] = (x & 1ull) ? 1.f : -1.f;
}

// Y[p][i] = Z[p][i] + sum_{e leaving i} A_e Z[p][dst(e)]
__global__ __launch_bounds__(BS) void k_normprod(int n, int P, const int32_t* __restrict__ eptr,
                                                 const int32_t* __restrict__ edst, const float* __restrict__ A,
                                                 const float* __restrict__ Z, float* __restrict__ Y) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)n * P * 9) return;
    const int c = (int)(t % 9);
    const int i = (int)((t / 9) % n);
    const int p = (int)(t / (9 * (int64_t)n));
    const float* Zp = Z + (int64_t)p * n * 9;
    float s = Zp[(int64_t)i * 9 + c];
    for (int e = eptr[i]; e < eptr[i + 1]; ++e) {
        const float* Ae = A + (int64_t)e * 81 + c * 9;
        const float* zj = Zp + (int64_t)edst[e] * 9;
#pragma unroll
        for (int q = 0; q < 9; ++q) s += Ae[q] * zj[q];
    }
    Y[t] = s;
}

// lower-triangular factor from a decoder row: diagonal exp(o[r]), strict
// lower part row-major from o[9 ..]
__device__ __forceinline__ void factor_from_out(const float* o, float* Lt) {
    int q = 9;
    for (int r = 0; r < 9; ++r)
        for (int c = 0; c < 9; ++c) {
            if (c < r) Lt[r * 9 + c] = o[q++];
            else if (c == r) Lt[r * 9 + c] = expf(o[r]);
            else Lt[r * 9 + c] = 0.f;
        }
}

// per node: loss_i = sum_p |B y - z|^2 (scaled) and d loss / d o
__global__ __launch_bounds__(64) void k_loss(int n, int P, float scale, const float* __restrict__ O,
                                             const float* __restrict__ Y, const float* __restrict__ Z,
                                             float* __restrict__ dO, float* __restrict__ lpart) {
    __shared__ float red[64];
    const int i = blockIdx.x * 64 + threadIdx.x;
    float li = 0.f;
    if (i < n) {
        float Lt[81], B[81], Gs[81];
        factor_from_out(O + (int64_t)i * F_OUT, Lt);
        for (int r = 0; r < 9; ++r)
            for (int c = 0; c < 9; ++c) {
                float s = 0.f;
                for (int q = 0; q <= (r < c ? r : c); ++q) s += Lt[r * 9 + q] * Lt[c * 9 + q];
                B[r * 9 + c] = s;
                Gs[r * 9 + c] = 0.f;
            }
        for (int p = 0; p < P; ++p) {
            const float* y = Y + ((int64_t)p * n + i) * 9;
            const float* z = Z + ((int64_t)p * n + i) * 9;
            float res[9];
            for (int r = 0; r < 9; ++r) {
                float s = -z[r];
                for (int c = 0; c < 9; ++c) s += B[r * 9 + c] * y[c];
                res[r] = s;
                li += s * s;
            }
            for (int r = 0; r < 9; ++r)
                for (int c = 0; c < 9; ++c) Gs[r * 9 + c] += 2.f * scale * res[r] * y[c];
        }
        li *= scale;
        // dLt = (G + G^T) Lt
        float* d = dO + (int64_t)i * F_OUT;
        int q = 9;
        for (int r = 0; r < 9; ++r)
            for (int c = 0; c <= r; ++c) {
                float s = 0.f;
                for (int k = c; k < 9; ++k) s += (Gs[r * 9 + k] + Gs[k * 9 + r]) * Lt[k * 9 + c];
                if (c == r) d[r] = s * Lt[r * 9 + r];
                else d[q++] = s;
            }
        for (int r = 45; r < F_OUT; ++r) d[r] = 0.f;
    }
    red[threadIdx.x] = li;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.f;
        for (int t = 0; t < 64; ++t) s += red[t];
        lpart[blockIdx.x] = s;
    }
}

__global__ void k_loss_fin(int nb, const float* __restrict__ lpart, double* __restrict__ out) {
    if (threadIdx.x != 0) return;
    double s = 0.0;
    for (int b = 0; b < nb; ++b) s += lpart[b];
    out[0] = s;
}

// dX = dY * (Y > 0) in FP32 and bf16
__global__ __launch_bounds__(BS) void k_relu_back(int64_t n, const float* __restrict__ dY, const float* __restrict__ Y,
                                                  int64_t ldy, int cols, int64_t lddy, float* __restrict__ out,
                                                  __bf16* __restrict__ outb) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= n) return;
    const int64_t r = t / cols, c = t % cols;
    const float v = Y[r * ldy + c] > 0.f ? dY[r * lddy + c] : 0.f;
    out[t] = v;
    outb[t] = (__bf16)v;
}

// dMm[e] = dXu[src(e)][64 + f] / deg(src(e)) * (Mm[e] > 0)
__global__ __launch_bounds__(BS) void k_msg_back(int E, const int32_t* __restrict__ esrc, const int32_t* __restrict__ eptr,
                                                 const float* __restrict__ dXu, const float* __restrict__ Mm,
                                                 float* __restrict__ dMm, __bf16* __restrict__ dMmb) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)E * H) return;
    const int e = (int)(t / H), f = (int)(t % H);
    const int s = esrc[e];
    const float v = Mm[t] > 0.f ? dXu[(int64_t)s * 2 * H + H + f] / (float)(eptr[s + 1] - eptr[s]) : 0.f;
    dMm[t] = v;
    dMmb[t] = (__bf16)v;
}

// dH[i] += dXu[i][0:64] + sum_{e leaving i} (dXm[e][0:64] + dXm[twin(e)][64:128]);
// dG[e] += dXm[e][128:192]
__global__ __launch_bounds__(BS) void k_msg_scatter(int n, const int32_t* __restrict__ eptr,
                                                    const int32_t* __restrict__ etwin, const float* __restrict__ dXu,
                                                    const float* __restrict__ dXm, float* __restrict__ dH) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)n * H) return;
    const int i = (int)(t / H), f = (int)(t % H);
    float s = dH[t] + dXu[(int64_t)i * 2 * H + f];
    for (int e = eptr[i]; e < eptr[i + 1]; ++e)
        s += dXm[(int64_t)e * 3 * H + f] + dXm[(int64_t)etwin[e] * 3 * H + H + f];
    dH[t] = s;
}

__global__ __launch_bounds__(BS) void k_edge_grad(int64_t n, const float* __restrict__ dXm, float* __restrict__ dG,
                                                  int first) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= n) return;
    const int64_t e = t / H, f = t % H;
    const float v = dXm[e * 3 * H + 2 * H + f];
    dG[t] = first ? v : dG[t] + v;
}

__global__ __launch_bounds__(BS) void k_adam(int64_t n, float* __restrict__ w, float* __restrict__ m,
                                             float* __restrict__ v, const float* __restrict__ g, float lr, float b1,
                                             float b2, float eps, float bc1, float bc2, __bf16* __restrict__ wb) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    w[i] = wi;
    wb[i] = (__bf16)wi;
}

__global__ __launch_bounds__(BS) void k_accum(int64_t n, const float* __restrict__ g, float* __restrict__ acc, int first,
                                              float scale) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    acc[i] = first ? scale * g[i] : acc[i] + scale * g[i];
}

// P_i = Linv_i^T (Lt Lt^T) Linv_i, written as Minv_i + Linv_i^T (Lt Lt^T - I)
// Linv_i when the block-Jacobi inverse Minv is given, so that a zero
// correction reproduces it exactly
__global__ __launch_bounds__(64) void k_assemble(int n, const float* __restrict__ O, const double* __restrict__ Linv,
                                                 const double* __restrict__ Minv, double* __restrict__ P) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= n) return;
    float Ltf[81];
    factor_from_out(O + (int64_t)i * F_OUT, Ltf);
    const double* Li = Linv + (int64_t)i * 81;
    // D = Lt Lt^T (minus I with a base), T = D Li, P = base + Li^T T
    double D[81];
    for (int r = 0; r < 9; ++r)
        for (int c = 0; c < 9; ++c) {
            double s = 0.0;
            for (int k = 0; k < 9; ++k) s += (double)Ltf[r * 9 + k] * (double)Ltf[c * 9 + k];
            D[r * 9 + c] = (Minv && r == c) ? s - 1.0 : s;
        }
    double Tm[81];
    for (int r = 0; r < 9; ++r)
        for (int c = 0; c < 9; ++c) {
            double s = 0.0;
            for (int k = 0; k < 9; ++k) s += D[r * 9 + k] * Li[k * 9 + c];
            Tm[r * 9 + c] = s;
        }
    for (int r = 0; r < 9; ++r)
        for (int c = 0; c < 9; ++c) {
            double s = 0.0;
            for (int k = 0; k < 9; ++k) s += Li[k * 9 + r] * Tm[k * 9 + c];
            P[(int64_t)i * 81 + r * 9 + c] = Minv ? Minv[(int64_t)i * 81 + r * 9 + c] + s : s;
        }
}

// ---------------------------------------------------------------------------
// factorised head (FSAI pattern): M^-1 = G^T G, G block-lower-triangular on
// the sets J_i; in the block-Jacobi-normalised coordinates Ghat = G L,
// Ghat_ii = Lt_i (node decoder) and, for the members j < i,
// Ghat_ij = reshape(Wo2^T relu(Wo1^T [h_i, h_j, g_ij] + bo1) + bo2)[:81]
//           - ao[:81] * A_ij.
// Training minimises the Kaporin functional
//   f = (1/(9n)) sum_i [tr(Ghat_i Ahat[J_i, J_i] Ghat_i^T) - 2 log det Ghat_ii],
// whose minimiser over the pattern is the exact FSAI factor.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int ftix(int a, int b) { return a * (a + 1) / 2 + b; }

// X_f = [h_i, h_j, g_ij] (bf16) of the FSAI edges
__global__ __launch_bounds__(BS) void k_fgather(int fE, const int32_t* __restrict__ fsrc,
                                                const int32_t* __restrict__ fdst, const int32_t* __restrict__ fe,
                                                const __bf16* __restrict__ Hb, const __bf16* __restrict__ Gb,
                                                __bf16* __restrict__ Xf) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)fE * 3 * H) return;
    const int64_t f = t / (3 * H);
    const int c = (int)(t % (3 * H));
    __bf16 v;
    if (c < H)
        v = Hb[(int64_t)fsrc[f] * H + c];
    else if (c < 2 * H)
        v = Hb[(int64_t)fdst[f] * H + c - H];
    else
        v = Gb[(int64_t)fe[f] * H + c - 2 * H];
    Xf[t] = v;
}

// element pq of Ghat for member b of row i (m members, first FSAI edge f0)
__device__ __forceinline__ float ghat_elem(int i, int b, int m, int f0, int u_edge, int pq, const float* __restrict__ O,
                                           const float* __restrict__ OE, const float* __restrict__ ao,
                                           const float* __restrict__ A) {
    if (b < m - 1) return OE[(int64_t)(f0 + b) * F_OFF + pq] - ao[pq] * A[(int64_t)u_edge * 81 + pq];
    const int p = pq / 9, q = pq % 9;
    const float* o = O + (int64_t)i * F_OUT;
    if (q == p) return expf(o[p]);
    if (q < p) return o[9 + p * (p - 1) / 2 + q];
    return 0.f;
}

// One workgroup per row: the row's term of the Kaporin functional (kpart,
// unscaled) and its gradient with respect to the decoder output (dO, all
// 48 entries), the head output (dOE, 96 entries per FSAI edge) and, per
// FSAI edge, the contributions to d/d ao (aE, 81 entries).
__global__ __launch_bounds__(BS) void k_kaporin(float scale, const int32_t* __restrict__ fptr,
                                                const int32_t* __restrict__ fedge, const int64_t* __restrict__ ftptr,
                                                const int32_t* __restrict__ ftile, const float* __restrict__ A,
                                                const float* __restrict__ O, const float* __restrict__ OE,
                                                const float* __restrict__ ao, float* __restrict__ dO,
                                                float* __restrict__ dOE, float* __restrict__ aE,
                                                double* __restrict__ kpart) {
    __shared__ float T[kFsaiTiles][81];
    __shared__ float Gm[kFsaiM][81];
    __shared__ double red[BS / 64];
    const int i = blockIdx.x;
    const int j0 = fptr[i], m = fptr[i + 1] - j0;
    const int f0 = j0 - i;
    const int32_t* tiles = ftile + ftptr[i];
    const int nt = m * (m + 1) / 2;
    for (int e = threadIdx.x; e < nt * 81; e += BS) {
        const int ti = e / 81, pq = e % 81;
        const int kb = tiles[ti];
        T[ti][pq] = kb == -2 ? ((pq / 9 == pq % 9) ? 1.f : 0.f) : (kb < 0 ? 0.f : A[(int64_t)kb * 81 + pq]);
    }
    for (int e = threadIdx.x; e < m * 81; e += BS) {
        const int b = e / 81;
        Gm[b][e % 81] = ghat_elem(i, b, m, f0, b < m - 1 ? fedge[j0 + b] : 0, e % 81, O, OE, ao, A);
    }
    __syncthreads();
    double fsum = 0.0;
    for (int e = threadIdx.x; e < m * 81; e += BS) {
        const int b = e / 81, pq = e % 81, p = pq / 9, q = pq % 9;
        // Y_b[p][q] = sum_a (Ghat_a Ahat(J_a, J_b))[p][q]
        float y = 0.f;
        for (int a = 0; a < m; ++a) {
            const float* Ga = Gm[a] + p * 9;
            if (a >= b) {
                const float* t = T[ftix(a, b)];
#pragma unroll
                for (int v = 0; v < 9; ++v) y += Ga[v] * t[v * 9 + q];
            } else {
                const float* t = T[ftix(b, a)];
#pragma unroll
                for (int v = 0; v < 9; ++v) y += Ga[v] * t[q * 9 + v];
            }
        }
        const float g = Gm[b][pq];
        fsum += (double)y * (double)g;
        float d = scale * y;
        if (b == m - 1) {
            if (q == p) {
                d -= scale / g;
                dO[(int64_t)i * F_OUT + p] = d * g;   // Ghat_pp = exp(o_p)
            } else if (q < p) {
                dO[(int64_t)i * F_OUT + 9 + p * (p - 1) / 2 + q] = d;
            }
        } else {
            const int64_t f = f0 + b;
            dOE[f * F_OFF + pq] = d;
            aE[f * 81 + pq] = -d * A[(int64_t)fedge[j0 + b] * 81 + pq];
        }
    }
    // padding entries
    if (threadIdx.x < F_OUT - 45) dO[(int64_t)i * F_OUT + 45 + threadIdx.x] = 0.f;
    for (int e = threadIdx.x; e < (m - 1) * (F_OFF - 81); e += BS)
        dOE[(int64_t)(f0 + e / (F_OFF - 81)) * F_OFF + 81 + e % (F_OFF - 81)] = 0.f;
    // row term: trace part plus -2 log det Ghat_ii = -2 sum_k o_k
    double v = fsum;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < BS / 64; ++w) t += red[w];
        for (int k = 0; k < 9; ++k) t -= 2.0 * (double)O[(int64_t)i * F_OUT + k];
        kpart[i] = t;
    }
}

// loss = sum_i kpart_i / N (fixed order, one block)
__global__ void k_kaporin_total(int n, double inv_n9, const double* __restrict__ kpart, double* __restrict__ out) {
    __shared__ double red[BS];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += BS) v += kpart[i];
    red[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < BS; ++k) t += red[k];
        out[0] = t * inv_n9;
    }
}

// dH[j] += sum over FSAI edges with source j of dXf[:, 0:H] and with
// destination j of dXf[:, H:2H] (fixed order)
__global__ __launch_bounds__(BS) void k_fscatter_h(int n, const int32_t* __restrict__ fptr,
                                                   const int32_t* __restrict__ fd_ptr,
                                                   const int32_t* __restrict__ fd_list, const float* __restrict__ dXf,
                                                   float* __restrict__ dH) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)n * H) return;
    const int j = (int)(t / H), c = (int)(t % H);
    float s = 0.f;
    for (int f = fptr[j] - j; f < fptr[j + 1] - (j + 1); ++f) s += dXf[(int64_t)f * 3 * H + c];
    for (int k = fd_ptr[j]; k < fd_ptr[j + 1]; ++k) s += dXf[(int64_t)fd_list[k] * 3 * H + H + c];
    dH[t] += s;
}

// dG[e] += dXf[f, 2H:3H] for the FSAI edge f of directed edge e
__global__ __launch_bounds__(BS) void k_fscatter_g(int E, const int32_t* __restrict__ e2f, const float* __restrict__ dXf,
                                                   float* __restrict__ dG) {
    const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (t >= (int64_t)E * H) return;
    const int e = (int)(t / H), c = (int)(t % H);
    const int f = e2f[e];
    if (f >= 0) dG[t] += dXf[(int64_t)f * 3 * H + 2 * H + c];
}

// One workgroup per row i: G_ij = Ghat_ij L_j^-1 for the row's members
// (Ghat from the decoder for the diagonal member, from the head for the
// others) into the layouts the apply reads: Gl (G by rows), Gu (the
// transposed block at gu_pos), Gs (the block slots); with Gh, instead of
// Gu, the UPPER apply's FP16 copy: each transposed block with its rows
// (the columns of G_ij) divided by Dn of the member's column block, scaled
// by its largest magnitude (hs); elements 0..7 of a row as halves in one
// 16-byte group (Gh, 36 words per member), element 8 in Gh8.  30,625 rows of
// 24 members: 625 us with an FP64 division and the divisions of its place per
// entry and the loads of L_j one after another (610 on the same GPU), 586 now.
__global__ __launch_bounds__(BS) void k_fassemble(const int32_t* __restrict__ fptr, const int32_t* __restrict__ fJ,
                                                  const int32_t* __restrict__ fedge, const int32_t* __restrict__ fslot,
                                                  const float* __restrict__ O, const float* __restrict__ OE,
                                                  const float* __restrict__ ao, const float* __restrict__ A,
                                                  const double* __restrict__ Linv, const int32_t* __restrict__ gu_pos,
                                                  float* __restrict__ Gl, float* __restrict__ Gu, float* __restrict__ Gs,
                                                  const double* __restrict__ Dn, uint32_t* __restrict__ Gh,
                                                  uint16_t* __restrict__ Gh8, float* __restrict__ hs) {
    __shared__ float gh[kFsaiM][81];
    __shared__ float gv[kFsaiM][81];
    __shared__ float smax[kFsaiM];
    __shared__ double rD[kFsaiM][9];   // 1 / Dn of the members' columns
    const int i = blockIdx.x;
    const int j0 = fptr[i], m = fptr[i + 1] - j0, f0 = j0 - i;
    // thread: entry (p, q) of every third member, so that its place is worked
    // out once
    const int b0 = threadIdx.x / 81, pq = threadIdx.x % 81, p = pq / 9, q = pq % 9;
    if (b0 < 3)
        for (int b = b0; b < m; b += 3) {
            gh[b][pq] = ghat_elem(i, b, m, f0, b < m - 1 ? fedge[j0 + b] : 0, pq, O, OE, ao, A);
            if (Gh && pq < 9) rD[b][pq] = 1.0 / Dn[(int64_t)fJ[j0 + b] * 9 + pq];
        }
    __syncthreads();
    if (b0 < 3)
        for (int b = b0; b < m; b += 3) {
            const int64_t u = j0 + b;
            const double* Lj = Linv + (int64_t)fJ[u] * 81;
            double l[9], s = 0.0;
#pragma unroll
            for (int v = 0; v < 9; ++v) l[v] = Lj[v * 9 + q];
#pragma unroll
            for (int v = 0; v < 9; ++v)
                if (v >= q) s += (double)gh[b][p * 9 + v] * l[v];
            const float g = (float)s;
            if (Gl) Gl[u * 81 + pq] = g;
            if (Gs) Gs[(int64_t)fslot[u] * 81 + pq] = g;
            if (Gh) gv[b][q * 9 + p] = (float)((double)g * rD[b][q]);
            else if (Gu) Gu[(int64_t)gu_pos[u] * 81 + q * 9 + p] = g;
        }
    if (!Gh) return;
    __syncthreads();
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
    for (int b = wv; b < m; b += BS / 64) {
        float mx = fabsf(gv[b][lane]);
        if (lane + 64 < 81) mx = fmaxf(mx, fabsf(gv[b][lane + 64]));
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        if (lane == 0) smax[b] = mx > 0.f && mx <= 3.0e38f ? mx : 1.f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < m * 36; e += BS) {
        const int b = e / 36, w = e % 36, c = w / 4, a = 2 * (w % 4);
        const float sc = smax[b];
        const _Float16 lo = (_Float16)(gv[b][c * 9 + a] / sc);
        const _Float16 hi = (_Float16)(gv[b][c * 9 + a + 1] / sc);
        Gh[(int64_t)(j0 + b) * 36 + w] =
            (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    for (int e = threadIdx.x; e < m * 9; e += BS) {
        const int b = e / 9, c = e % 9;
        Gh8[(int64_t)(j0 + b) * 9 + c] = __builtin_bit_cast(uint16_t, (_Float16)(gv[b][c * 9 + 8] / smax[b]));
    }
    for (int b = threadIdx.x; b < m; b += BS) hs[j0 + b] = smax[b];
}

__global__ __launch_bounds__(BS) void k_add(int64_t n, const float* __restrict__ a, float* __restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i < n) b[i] += a[i];
}

template <typename T>
void grow(T** p, size_t n) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    BA_HIP_CHECK(hipMalloc((void**)p, std::max<size_t>(n, 1) * sizeof(T)));
}

void ensure_work(Work& W, int n, int E, int P) {
    if (n <= W.cap_n && E <= W.cap_E && P <= W.cap_p) return;
    n = std::max(n, W.cap_n);
    E = std::max(E, W.cap_E);
    P = std::max(P, std::max(W.cap_p, 4));
    const size_t nh = (size_t)n * H, eh = (size_t)E * H;
    grow(&W.H0, nh); grow(&W.Hf, nh); grow(&W.G, eh); grow(&W.O, (size_t)n * F_OUT);
    grow(&W.Z, (size_t)P * n * 9); grow(&W.Y, (size_t)P * n * 9);
    grow(&W.Hb, 4 * nh); grow(&W.Gb, eh);
    grow(&W.Xm, (size_t)N_LAYERS * 3 * eh); grow(&W.Xu, (size_t)N_LAYERS * 2 * nh);
    grow(&W.Mm, (size_t)N_LAYERS * eh); grow(&W.T, (size_t)N_LAYERS * nh);
    grow(&W.dO, (size_t)n * F_OUT); grow(&W.dH, nh); grow(&W.dT, nh); grow(&W.dXu, 2 * nh);
    grow(&W.dMm, eh); grow(&W.dXm, 3 * eh); grow(&W.dG, eh);
    grow(&W.dOb, (size_t)n * F_OUT); grow(&W.dTb, nh); grow(&W.dMmb, eh);
    const size_t big = std::max(nh, eh);
    grow(&W.dP, big); grow(&W.dPb, big);
    const size_t rows = std::max(n, E);
    const size_t nsplit = (rows + KSPLIT_ROWS - 1) / KSPLIT_ROWS;
    grow(&W.split, nsplit * 3 * H * std::max(std::max(H, F_OFF), HO));
    grow(&W.colpart, ((rows + 1023) / 1024) * 3 * H);
    grow(&W.loss_part, (size_t)n / 64 + 2);
    grow(&W.loss, 2);
    W.cap_n = n; W.cap_E = E; W.cap_p = P;
}

void ensure_fwork(Work& W, const Graph& g) {
    if (g.fE <= W.cap_f && g.n <= W.cap_fn) return;
    const int fE = std::max(std::max(g.fE, W.cap_f), 1), n = std::max(std::max(g.n, W.cap_fn), 1);
    grow(&W.Xf, (size_t)fE * 3 * H); grow(&W.OE, (size_t)fE * F_OFF); grow(&W.dOE, (size_t)fE * F_OFF);
    grow(&W.dOEb, (size_t)fE * F_OFF); grow(&W.dXf, (size_t)fE * 3 * H); grow(&W.aE, (size_t)fE * 81);
    grow(&W.Z1, (size_t)fE * HO); grow(&W.Z1b, (size_t)fE * HO); grow(&W.dZ1, (size_t)fE * HO);
    grow(&W.dZ1p, (size_t)fE * HO); grow(&W.dZ1b, (size_t)fE * HO);
    grow(&W.kpart, (size_t)n);
    W.cap_f = fE; W.cap_fn = n;
}

void gemm(hipStream_t st, int M, int N, int K, const __bf16* A, int64_t sam, int64_t sak, const __bf16* B,
          int64_t sbk, int64_t sbn, const float* bias, bool relu, float* C, int64_t ldc, __bf16* Cb, int64_t ldcb) {
    if (M == 0) return;
    dim3 grid(nblk(M, 64), nblk(N, 64), 1);
    const bool vec = sak == 1 && sbn == 1 && K % 32 == 0 && N % 8 == 0 && sam % 8 == 0 && sbk % 8 == 0 &&
                     reinterpret_cast<uintptr_t>(A) % 16 == 0 && reinterpret_cast<uintptr_t>(B) % 16 == 0;
    if (vec)
        k_gemm_v<false><<<grid, BS, 0, st>>>(M, N, K, A, sam, GatherRows{}, B, sbk, bias, relu ? 1 : 0, C, ldc, Cb,
                                             ldcb);
    else
        k_gemm<<<grid, BS, 0, st>>>(M, N, K, K, A, sam, sak, B, sbk, sbn, bias, relu ? 1 : 0, C, ldc, 0, Cb, ldcb);
}

// C = [H[src], H[dst], G[eid]] B (+ bias) (relu) without forming the input
// rows (K = 3 H; B row-major [3 H][N], N a multiple of 8)
void gemm_gather(hipStream_t st, int M, int N, const GatherRows& gr, const __bf16* B, const float* bias, bool relu,
                 float* C, int64_t ldc, __bf16* Cb, int64_t ldcb) {
    if (M == 0) return;
    if (N % 8 != 0 || reinterpret_cast<uintptr_t>(B) % 16 != 0 || reinterpret_cast<uintptr_t>(gr.Hn) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(gr.Ge) % 16 != 0)
        throw std::runtime_error("gemm_gather: operands must be 16-byte aligned, N a multiple of 8");
    dim3 grid(nblk(M, 64), nblk(N, 64), 1);
    k_gemm_v<true><<<grid, BS, 0, st>>>(M, N, 3 * H, nullptr, 0, gr, B, N, bias, relu ? 1 : 0, C, ldc, Cb, ldcb);
}

// dW[Kin][Nout] = X^T dY over `rows` rows (X: [rows][ldx] bf16, dY: [rows][ldy] bf16)
void wgrad(hipStream_t st, Work& W, int Kin, int Nout, int rows, const __bf16* X, int64_t ldx, const __bf16* dY,
           int64_t ldy, float* dW) {
    const int nz = std::max(1, (rows + KSPLIT_ROWS - 1) / KSPLIT_ROWS);
    dim3 grid(nblk(Kin, 64), nblk(Nout, 64), nz);
    k_gemm<<<grid, BS, 0, st>>>(Kin, Nout, rows, KSPLIT_ROWS, X, 1, ldx, dY, ldy, 1, nullptr, 0, W.split, Nout,
                                (int64_t)Kin * Nout, nullptr, 0);
    const int64_t n = (int64_t)Kin * Nout;
    k_sum_split<<<nblk(n), BS, 0, st>>>(n, nz, W.split, dW);
}

void colsum(hipStream_t st, Work& W, int rows, int cols, const float* src, int64_t ld, float* out) {
    const int nc = std::max(1, (rows + 1023) / 1024);
    k_colsum_part<<<nc, BS, 0, st>>>(rows, cols, src, ld, W.colpart);
    k_colsum_fin<<<1, BS, 0, st>>>(nc, cols, W.colpart, out);
}

// train: also form the message inputs X_m (the backward pass needs them);
// inference reads them in place inside the GEMM
void forward(ba_gnn* net, Graph& g, hipStream_t st, bool train = true) {
    Work& W = net->work;
    const int n = g.n, E = g.E;
    const __bf16* wb = net->wb;
    const float* w = net->w;
    const int64_t nh = (int64_t)n * H, eh = (int64_t)E * H;
    gemm(st, n, H, F_NODE, g.xn, F_NODE, 1, wb + OFF_WN, H, 1, w + OFF_BN, true, W.H0, H, W.Hb, H);
    BA_HIP_CHECK(hipMemcpyAsync(W.Hf, W.H0, nh * sizeof(float), hipMemcpyDeviceToDevice, st));
    if (E > 0) gemm(st, E, H, F_EDGE, g.xe, F_EDGE, 1, wb + OFF_WE, H, 1, w + OFF_BE, true, W.G, H, W.Gb, H);
    for (int l = 0; l < N_LAYERS; ++l) {
        __bf16* Hb = W.Hb + l * nh;
        __bf16* Xm = W.Xm + (int64_t)l * 3 * eh;
        __bf16* Xu = W.Xu + (int64_t)l * 2 * nh;
        float* Mm = W.Mm + (int64_t)l * eh;
        float* T = W.T + (int64_t)l * nh;
        if (E > 0 && train) {
            k_gather_msg<<<nblk(3 * eh), BS, 0, st>>>(E, g.esrc, g.edst, Hb, W.Gb, Xm);
            gemm(st, E, H, 3 * H, Xm, 3 * H, 1, wb + off_M(l), H, 1, w + off_c(l), true, Mm, H, nullptr, 0);
        } else if (E > 0) {
            gemm_gather(st, E, H, GatherRows{g.esrc, g.edst, nullptr, Hb, W.Gb}, wb + off_M(l), w + off_c(l), true,
                        Mm, H, nullptr, 0);
        }
        k_aggregate<<<nblk(nh), BS, 0, st>>>(n, g.eptr, Mm, Hb, Xu);
        gemm(st, n, H, 2 * H, Xu, 2 * H, 1, wb + off_U(l), H, 1, w + off_u(l), true, T, H, nullptr, 0);
        k_residual<<<nblk(nh), BS, 0, st>>>(nh, W.Hf, T, W.Hb + (l + 1) * nh);
    }
    gemm(st, n, F_OUT, H, W.Hb + N_LAYERS * nh, H, 1, wb + OFF_WD, F_OUT, 1, w + OFF_BD, false, W.O, F_OUT, nullptr, 0);
}

// factorised head: X_f, Z1 = relu(Wo1^T X_f + bo1), OE = Wo2^T Z1 + bo2 for
// the FSAI edges
void head_forward(ba_gnn* net, Graph& g, hipStream_t st, bool train = true) {
    Work& W = net->work;
    if (g.fE == 0) return;
    const int64_t nh = (int64_t)g.n * H;
    if (train) {
        k_fgather<<<nblk((int64_t)g.fE * 3 * H), BS, 0, st>>>(g.fE, g.fsrc, g.fdst, g.fe, W.Hb + N_LAYERS * nh,
                                                               W.Gb, W.Xf);
        gemm(st, g.fE, HO, 3 * H, W.Xf, 3 * H, 1, net->wb + OFF_WO1, HO, 1, net->w + OFF_BO1, true, W.Z1, HO, W.Z1b,
             HO);
    } else {
        gemm_gather(st, g.fE, HO, GatherRows{g.fsrc, g.fdst, g.fe, W.Hb + N_LAYERS * nh, W.Gb}, net->wb + OFF_WO1,
                    net->w + OFF_BO1, true, W.Z1, HO, W.Z1b, HO);
    }
    gemm(st, g.fE, F_OFF, HO, W.Z1b, HO, 1, net->wb + OFF_WO2, F_OFF, 1, net->w + OFF_BO2, false, W.OE, F_OFF,
         nullptr, 0);
}

// loss for probes already in W.Z: Y = A Z, loss and dO
void loss(ba_gnn* net, Graph& g, int P, hipStream_t st) {
    Work& W = net->work;
    const int n = g.n;
    k_normprod<<<nblk((int64_t)n * P * 9), BS, 0, st>>>(n, P, g.eptr, g.edst, g.A, W.Z, W.Y);
    const float scale = 1.f / (float)(P * 9 * (int64_t)n);
    const int nb = nblk(n, 64);
    k_loss<<<nb, 64, 0, st>>>(n, P, scale, W.O, W.Y, W.Z, W.dO, W.loss_part);
    k_loss_fin<<<1, 64, 0, st>>>(nb, W.loss_part, W.loss);
}

void backward(ba_gnn* net, Graph& g, float* grad, hipStream_t st, bool head = false) {
    Work& W = net->work;
    const int n = g.n, E = g.E;
    const __bf16* wb = net->wb;
    const int64_t nh = (int64_t)n * H, eh = (int64_t)E * H;
    // decoder
    k_to_bf16<<<nblk((int64_t)n * F_OUT), BS, 0, st>>>((int64_t)n * F_OUT, W.dO, W.dOb);
    wgrad(st, W, H, F_OUT, n, W.Hb + N_LAYERS * nh, H, W.dOb, F_OUT, grad + OFF_WD);
    colsum(st, W, n, F_OUT, W.dO, F_OUT, grad + OFF_BD);
    // dH = dO Wd^T   (B(k=o, n=h) = Wd[h][o])
    gemm(st, n, H, F_OUT, W.dOb, F_OUT, 1, wb + OFF_WD, 1, F_OUT, nullptr, false, W.dH, H, nullptr, 0);
    const bool fhead = head && g.fE > 0;
    if (fhead) {
        const int64_t no = (int64_t)g.fE * F_OFF;
        k_to_bf16<<<nblk(no), BS, 0, st>>>(no, W.dOE, W.dOEb);
        wgrad(st, W, HO, F_OFF, g.fE, W.Z1b, HO, W.dOEb, F_OFF, grad + OFF_WO2);
        colsum(st, W, g.fE, F_OFF, W.dOE, F_OFF, grad + OFF_BO2);
        BA_HIP_CHECK(hipMemsetAsync(grad + OFF_AO, 0, F_OFF * sizeof(float), st));
        colsum(st, W, g.fE, 81, W.aE, 81, grad + OFF_AO);
        // dZ1 = dOE Wo2^T, through the ReLU, then Wo1
        gemm(st, g.fE, HO, F_OFF, W.dOEb, F_OFF, 1, wb + OFF_WO2, 1, F_OFF, nullptr, false, W.dZ1, HO, nullptr, 0);
        const int64_t nz = (int64_t)g.fE * HO;
        k_relu_back<<<nblk(nz), BS, 0, st>>>(nz, W.dZ1, W.Z1, HO, HO, HO, W.dZ1p, W.dZ1b);
        wgrad(st, W, 3 * H, HO, g.fE, W.Xf, 3 * H, W.dZ1b, HO, grad + OFF_WO1);
        colsum(st, W, g.fE, HO, W.dZ1p, HO, grad + OFF_BO1);
        // dX_f = dZ1 Wo1^T  (B(k=o, n=x) = Wo1[x][o])
        gemm(st, g.fE, 3 * H, HO, W.dZ1b, HO, 1, wb + OFF_WO1, 1, HO, nullptr, false, W.dXf, 3 * H, nullptr, 0);
        k_fscatter_h<<<nblk(nh), BS, 0, st>>>(n, g.fptr, g.fd_ptr, g.fd_list, W.dXf, W.dH);
    } else {
        BA_HIP_CHECK(hipMemsetAsync(grad + OFF_HEAD, 0, (N_PARAMS - OFF_HEAD) * sizeof(float), st));
    }
    for (int l = N_LAYERS - 1; l >= 0; --l) {
        const __bf16* Xm = W.Xm + (int64_t)l * 3 * eh;
        const __bf16* Xu = W.Xu + (int64_t)l * 2 * nh;
        const float* Mm = W.Mm + (int64_t)l * eh;
        const float* T = W.T + (int64_t)l * nh;
        k_relu_back<<<nblk(nh), BS, 0, st>>>(nh, W.dH, T, H, H, H, W.dT, W.dTb);
        wgrad(st, W, 2 * H, H, n, Xu, 2 * H, W.dTb, H, grad + off_U(l));
        colsum(st, W, n, H, W.dT, H, grad + off_u(l));
        gemm(st, n, 2 * H, H, W.dTb, H, 1, wb + off_U(l), 1, H, nullptr, false, W.dXu, 2 * H, nullptr, 0);
        if (E > 0) {
            k_msg_back<<<nblk(eh), BS, 0, st>>>(E, g.esrc, g.eptr, W.dXu, Mm, W.dMm, W.dMmb);
            wgrad(st, W, 3 * H, H, E, Xm, 3 * H, W.dMmb, H, grad + off_M(l));
            colsum(st, W, E, H, W.dMm, H, grad + off_c(l));
            gemm(st, E, 3 * H, H, W.dMmb, H, 1, wb + off_M(l), 1, H, nullptr, false, W.dXm, 3 * H, nullptr, 0);
            k_edge_grad<<<nblk(eh), BS, 0, st>>>(eh, W.dXm, W.dG, l == N_LAYERS - 1);
        } else {
            BA_HIP_CHECK(hipMemsetAsync(grad + off_M(l), 0, (3 * H * H + H) * sizeof(float), st));
        }
        k_msg_scatter<<<nblk(nh), BS, 0, st>>>(n, g.eptr, g.etwin, W.dXu, W.dXm, W.dH);
    }
    if (fhead) k_fscatter_g<<<nblk(eh), BS, 0, st>>>(E, g.e2f, W.dXf, W.dG);
    // encoders
    k_relu_back<<<nblk(nh), BS, 0, st>>>(nh, W.dH, W.H0, H, H, H, W.dP, W.dPb);
    wgrad(st, W, F_NODE, H, n, g.xn, F_NODE, W.dPb, H, grad + OFF_WN);
    colsum(st, W, n, H, W.dP, H, grad + OFF_BN);
    if (E > 0) {
        k_relu_back<<<nblk(eh), BS, 0, st>>>(eh, W.dG, W.G, H, H, H, W.dP, W.dPb);
        wgrad(st, W, F_EDGE, H, E, g.xe, F_EDGE, W.dPb, H, grad + OFF_WE);
        colsum(st, W, E, H, W.dP, H, grad + OFF_BE);
    } else {
        BA_HIP_CHECK(hipMemsetAsync(grad + OFF_WE, 0, (F_EDGE * H + H) * sizeof(float), st));
    }
}

}  // namespace

void build_graph(Graph& g, int n, const int64_t* row_ptr, const int32_t* col_idx, const int32_t* blk_pairs,
                 hipStream_t st) {
    Phases ph("build_graph");
    // directed edges by source, destinations ascending: for source r the
    // blocks (s, r), s < r (t = 1: the block transposed), in ascending s,
    // then the row's own upper blocks (r, s) (t = 0); the twin of an edge is
    // the other direction through the same block
    const int64_t nb = row_ptr[n];
    std::vector<int32_t> diag(n), brow(nb);
    for (int r = 0; r < n; ++r) {
        diag[r] = (int32_t)row_ptr[r];
        for (int64_t k = row_ptr[r]; k < row_ptr[r + 1]; ++k) brow[k] = r;
    }
    std::vector<int64_t> lptr;
    std::vector<int32_t> lblk;   // blocks (s, r), s < r, of each column r, ascending s
    counting_sort(nb, n, [&](int64_t k) { return k == row_ptr[brow[k]] ? -1 : col_idx[k]; }, lptr, lblk);
    std::vector<int32_t> eptr(n + 1, 0);
    for (int r = 0; r < n; ++r)
        eptr[r + 1] = eptr[r] + (int32_t)(lptr[r + 1] - lptr[r]) + (int32_t)(row_ptr[r + 1] - row_ptr[r] - 1);
    const int E = eptr[n];
    std::vector<int32_t> src(E), dst(E), eb(E), et(E), twin(E), e_up(nb, -1), e_lo(nb, -1);
    parallel_for(n, 256, [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r) {
            int32_t e = eptr[r];
            for (int64_t i = lptr[r]; i < lptr[r + 1]; ++i, ++e) {
                const int32_t k = lblk[i];
                src[e] = (int32_t)r; dst[e] = brow[k]; eb[e] = k; et[e] = 1;
                e_lo[k] = e;
            }
            for (int64_t k = row_ptr[r] + 1; k < row_ptr[r + 1]; ++k, ++e) {
                src[e] = (int32_t)r; dst[e] = col_idx[k]; eb[e] = (int32_t)k; et[e] = 0;
                e_up[k] = e;
            }
        }
    });
    ph.mark("edges");
    parallel_for(E, 1 << 16, [&](int64_t e0, int64_t e1, int) {
        for (int64_t e = e0; e < e1; ++e) twin[e] = et[e] ? e_up[eb[e]] : e_lo[eb[e]];
    });
    ph.mark("twins");
    g.n = n;
    g.E = E;
    auto up = [&](int32_t** p, const std::vector<int32_t>& h) {
        BA_HIP_CHECK(hipMalloc((void**)p, std::max<size_t>(h.size(), 1) * sizeof(int32_t)));
        if (!h.empty()) BA_HIP_CHECK(hipMemcpyAsync(*p, h.data(), h.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
        g.bytes += h.size() * sizeof(int32_t);
    };
    up(&g.eptr, eptr); up(&g.esrc, src); up(&g.edst, dst); up(&g.etwin, twin); up(&g.eblk, eb);
    std::vector<int32_t> low;
    for (size_t e = 0; e < et.size(); ++e)
        if (et[e] == 0) low.push_back((int32_t)e);
    g.n_low = (int32_t)low.size();
    up(&g.elow, low);
    up(&g.diag_blk, diag);
    BA_HIP_CHECK(hipMalloc((void**)&g.xn, (size_t)std::max(n, 1) * F_NODE * sizeof(__bf16)));
    BA_HIP_CHECK(hipMalloc((void**)&g.xe, (size_t)std::max(E, 1) * F_EDGE * sizeof(__bf16)));
    BA_HIP_CHECK(hipMalloc((void**)&g.A, (size_t)std::max(E, 1) * 81 * sizeof(float)));
    BA_HIP_CHECK(hipMalloc((void**)&g.Linv, (size_t)std::max(n, 1) * 81 * sizeof(double)));
    BA_HIP_CHECK(hipMalloc((void**)&g.flags, 4 * sizeof(int)));
    g.bytes += (size_t)n * (F_NODE * 2 + 81 * 8) + (size_t)E * (F_EDGE * 2 + 81 * 4);
    g.n_blk = (int)row_ptr[n];
    ph.mark("upload+alloc");
    if (blk_pairs) {
        std::vector<int32_t> fptr, fJ, fslot;
        fsai_sets(n, row_ptr, col_idx, blk_pairs, fptr, fJ, fslot);
        auto edge = [&](int32_t a, int32_t b) -> int32_t {   // directed edge a -> b or -1
            const auto first = dst.begin() + eptr[a], last = dst.begin() + eptr[a + 1];
            const auto it = std::lower_bound(first, last, b);
            return (it != last && *it == b) ? (int32_t)(it - dst.begin()) : -1;
        };
        const int fm = (int)fJ.size();
        // per set J_i: its members' edges i -> j (all but i itself) and the
        // local tile of edges (J_a -> J_b), filled rows in parallel at
        // offsets fixed by the set sizes
        std::vector<int64_t> ftptr(n + 1, 0);
        std::vector<int32_t> fsp(n + 1, 0);
        int max_m = 1;
        for (int i = 0; i < n; ++i) {
            const int m = fptr[i + 1] - fptr[i];
            max_m = std::max(max_m, m);
            fsp[i + 1] = fsp[i] + (m - 1);
            ftptr[i + 1] = ftptr[i] + (int64_t)m * (m + 1) / 2;
        }
        const int fE0 = fsp[n];
        std::vector<int32_t> fedge(fm, -1), ftile(ftptr[n]), fsrc(fE0), fdst(fE0), fe(fE0), e2f(E, -1);
        parallel_for(n, 256, [&](int64_t i0, int64_t i1, int) {
            for (int64_t i = i0; i < i1; ++i) {
                const int j0 = fptr[i], m = fptr[i + 1] - j0;
                for (int b = 0; b < m - 1; ++b) {
                    const int32_t f = fsp[i] + b;
                    fedge[j0 + b] = edge((int32_t)i, fJ[j0 + b]);
                    e2f[fedge[j0 + b]] = f;
                    fsrc[f] = (int32_t)i;
                    fdst[f] = fJ[j0 + b];
                    fe[f] = fedge[j0 + b];
                }
                int64_t d = ftptr[i];
                for (int a = 0; a < m; ++a)
                    for (int b = 0; b <= a; ++b, ++d) ftile[d] = a == b ? -2 : edge(fJ[j0 + a], fJ[j0 + b]);
            }
        });
        ph.mark("fsai tiles");
        const int fE = (int)fsrc.size();
        std::vector<int32_t> fd_ptr(n + 1, 0), fd_list(fE);
        for (int f = 0; f < fE; ++f) fd_ptr[fdst[f] + 1]++;
        for (int i = 0; i < n; ++i) fd_ptr[i + 1] += fd_ptr[i];
        {
            std::vector<int32_t> fill(fd_ptr.begin(), fd_ptr.end() - 1);
            for (int f = 0; f < fE; ++f) fd_list[fill[fdst[f]]++] = f;
        }
        up(&g.fptr, fptr); up(&g.fJ, fJ); up(&g.fedge, fedge); up(&g.fslot, fslot); up(&g.ftile, ftile);
        up(&g.fsrc, fsrc); up(&g.fdst, fdst); up(&g.fe, fe); up(&g.fd_ptr, fd_ptr); up(&g.fd_list, fd_list);
        up(&g.e2f, e2f);
        BA_HIP_CHECK(hipMalloc((void**)&g.ftptr, (n + 1) * sizeof(int64_t)));
        BA_HIP_CHECK(hipMemcpyAsync(g.ftptr, ftptr.data(), (n + 1) * sizeof(int64_t), hipMemcpyHostToDevice, st));
        g.fm = fm;
        g.fE = fE;
        g.max_m = max_m;
        g.has_fsai = true;
    }
    BA_HIP_CHECK(hipStreamSynchronize(st));
    ph.mark("fsai upload");
}

void free_graph(Graph& g) {
    void* p[] = {g.eptr, g.esrc, g.edst, g.etwin, g.eblk, g.elow, g.diag_blk, g.xn, g.xe, g.A, g.Linv, g.flags,
                 g.fptr, g.fJ, g.fedge, g.fslot, g.ftile, g.ftptr, g.fsrc, g.fdst, g.fe, g.fd_ptr, g.fd_list, g.e2f};
    for (void* q : p)
        if (q) (void)hipFree(q);
    g = Graph();
}

void compute_features(Graph& g, const double* blk, hipStream_t st) {
    BA_HIP_CHECK(hipMemsetAsync(g.flags, 0, 4 * sizeof(int), st));
    if (g.n > 0) k_feat_node<<<nblk(g.n, 64), 64, 0, st>>>(g.n, g.diag_blk, blk, g.Linv, g.xn, g.flags);
    if (g.E > 0)
        k_feat_edge<<<(unsigned)std::min<int64_t>((g.n_low + kFE - 1) / kFE, 2048), 256, 0, st>>>(
            g.n_low, g.elow, g.esrc, g.edst, g.eblk, g.etwin, blk, g.Linv, g.A, g.xe);
    BA_HIP_CHECK(hipGetLastError());
}

void infer_preconditioner(ba_gnn* net, Graph& g, const double* Minv, double* P, hipStream_t st) {
    ensure_work(net->work, g.n, g.E, 1);
    forward(net, g, st, false);
    k_assemble<<<nblk(g.n, 64), 64, 0, st>>>(g.n, net->work.O, g.Linv, Minv, P);
    BA_HIP_CHECK(hipGetLastError());
}

void infer_factor(ba_gnn* net, Graph& g, const int32_t* gu_pos, float* Gl, float* Gu, float* Gslots, hipStream_t st,
                  const double* Dn, uint32_t* Gh, uint16_t* Gh8, float* hs) {
    ensure_work(net->work, g.n, g.E, 1);
    ensure_fwork(net->work, g);
    forward(net, g, st, false);
    head_forward(net, g, st, false);
    if (g.fm > 0 && g.n > 0)
        k_fassemble<<<g.n, BS, 0, st>>>(g.fptr, g.fJ, g.fedge, g.fslot, net->work.O, net->work.OE, net->w + OFF_AO,
                                        g.A, g.Linv, gu_pos, Gl, Gu, Gslots, Dn, Gh, Gh8, hs);
    BA_HIP_CHECK(hipGetLastError());
}

void fsai_sets(int n, const int64_t* row_ptr, const int32_t* col_idx, const int32_t* blk_pairs,
               std::vector<int32_t>& ptr, std::vector<int32_t>& J, std::vector<int32_t>& slot) {
    // blocks (r, i), r < i, of each column i in ascending r
    const int64_t nb = row_ptr[n];
    std::vector<int32_t> brow(nb);
    parallel_for(n, 256, [&](int64_t r0, int64_t r1, int) {
        for (int64_t r = r0; r < r1; ++r)
            for (int64_t kb = row_ptr[r]; kb < row_ptr[r + 1]; ++kb) brow[kb] = (int32_t)r;
    });
    std::vector<int64_t> lptr;
    std::vector<int32_t> lblk;
    counting_sort(nb, n, [&](int64_t kb) { return kb == row_ptr[brow[kb]] ? -1 : col_idx[kb]; }, lptr, lblk);
    ptr.assign(n + 1, 0);
    for (int i = 0; i < n; ++i)
        ptr[i + 1] = ptr[i] + (int32_t)std::min<int64_t>(lptr[i + 1] - lptr[i], kFsaiM - 1) + 1;
    J.resize(ptr[n]);
    slot.resize(ptr[n]);
    // per row (in parallel): the kFsaiM - 1 lower neighbours with the most
    // common points (ties to the lower row), in ascending order, then i
    parallel_for(n, 256, [&](int64_t i0, int64_t i1, int) {
        std::vector<std::pair<int32_t, int64_t>> L;
        for (int64_t i = i0; i < i1; ++i) {
            L.clear();
            for (int64_t t = lptr[i]; t < lptr[i + 1]; ++t) L.push_back({brow[lblk[t]], lblk[t]});
            std::sort(L.begin(), L.end(), [&](const std::pair<int32_t, int64_t>& x, const std::pair<int32_t, int64_t>& y) {
                const int32_t cx = blk_pairs[x.second], cy = blk_pairs[y.second];
                return cx != cy ? cx > cy : x.first < y.first;
            });
            if ((int)L.size() > kFsaiM - 1) L.resize(kFsaiM - 1);
            std::sort(L.begin(), L.end());
            int32_t d = ptr[i];
            for (auto& e : L) {
                J[d] = e.first;
                slot[d++] = (int32_t)e.second;
            }
            J[d] = (int32_t)i;
            slot[d] = (int32_t)row_ptr[i];
        }
    });
}


void free_work(Work& W) {
    void* p[] = {W.H0, W.Hf, W.G, W.O, W.Z, W.Y, W.Hb, W.Gb, W.Xm, W.Xu, W.Mm, W.T, W.dO, W.dH, W.dT, W.dXu,
                 W.dMm, W.dXm, W.dG, W.dOb, W.dTb, W.dMmb, W.dPb, W.dP, W.split, W.colpart, W.loss_part, W.loss,
                 W.Xf, W.dOEb, W.OE, W.dOE, W.dXf, W.aE, W.kpart, W.Z1, W.Z1b, W.dZ1, W.dZ1p, W.dZ1b};
    for (void* q : p)
        if (q) (void)hipFree(q);
    W = Work();
}

// one graph: probes (host or generated), forward, loss, backward into grad
void loss_grad(ba_gnn* net, Graph& g, int P, const float* probes_host, unsigned long long seed, float* grad,
               hipStream_t st) {
    ensure_work(net->work, g.n, g.E, P);
    Work& W = net->work;
    const int64_t nz = (int64_t)P * g.n * 9;
    if (probes_host)
        BA_HIP_CHECK(hipMemcpyAsync(W.Z, probes_host, nz * sizeof(float), hipMemcpyHostToDevice, st));
    else
        k_probes<<<nblk(nz), BS, 0, st>>>(nz, seed, W.Z);
    forward(net, g, st);
    loss(net, g, P, st);
    if (grad) backward(net, g, grad, st);
    BA_HIP_CHECK(hipGetLastError());
}

// one graph: forward with the factorised head, Kaporin loss, backward
void fsai_loss_grad(ba_gnn* net, Graph& g, float* grad, hipStream_t st) {
    ensure_work(net->work, g.n, g.E, 1);
    ensure_fwork(net->work, g);
    Work& W = net->work;
    forward(net, g, st);
    head_forward(net, g, st);
    const double N = 9.0 * g.n;
    k_kaporin<<<g.n, BS, 0, st>>>((float)(2.0 / N), g.fptr, g.fedge, g.ftptr, g.ftile, g.A, W.O, W.OE,
                                  net->w + OFF_AO, W.dO, W.dOE, W.aE, W.kpart);
    k_kaporin_total<<<1, BS, 0, st>>>(g.n, 1.0 / N, W.kpart, W.loss);
    if (grad) backward(net, g, grad, st, true);
    BA_HIP_CHECK(hipGetLastError());
}

void adam(ba_gnn* net, const float* g, float lr, hipStream_t st) {
    net->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = 1.f - powf(b1, (float)net->step), bc2 = 1.f - powf(b2, (float)net->step);
    k_adam<<<nblk(N_PARAMS), BS, 0, st>>>(N_PARAMS, net->w, net->m, net->v, g, lr, b1, b2, 1e-8f, bc1, bc2, net->wb);
}

void accumulate(const float* g, float* acc, bool first, float scale, hipStream_t st) {
    k_accum<<<nblk(N_PARAMS), BS, 0, st>>>(N_PARAMS, g, acc, first ? 1 : 0, scale);
}

// plain GEMM entry for tests: C[M][N] = A[M][K] B[K][N] (row-major bf16 bits)
void test_gemm(int M, int N, int K, const __bf16* A, const __bf16* B, float* C, hipStream_t st) {
    gemm(st, M, N, K, A, K, 1, B, N, 1, nullptr, false, C, N, nullptr, 0);
}

}  // namespace gnn
}  // namespace ba

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
namespace {
thread_local std::string g_gnn_error;

template <typename F>
ba_status gnn_guard(std::string* err, F&& f) {
    try {
        return f();
    } catch (const ba_hip_error& e) {
        if (err) *err = e.what;
        g_gnn_error = e.what;
        return BA_ERR_DEVICE;
    } catch (const std::bad_alloc&) {
        g_gnn_error = "host allocation failed";
        return BA_ERR_OUT_OF_MEMORY;
    }
}
}  // namespace

extern "C" {

int64_t ba_gnn_param_count(void) { return ba::gnn::N_PARAMS; }

const char* ba_gnn_last_error(void) { return g_gnn_error.c_str(); }

ba_status ba_gnn_create(const float* params, void* stream, ba_gnn** out) {
    if (!out || !params) return BA_ERR_INVALID_ARG;
    *out = nullptr;
    ba_gnn* net = new ba_gnn();
    net->stream = (hipStream_t)stream;
    ba_status s = gnn_guard(&net->err, [&]() {
        const size_t n = ba::gnn::N_PARAMS;
        BA_HIP_CHECK(hipMalloc((void**)&net->w, n * sizeof(float)));
        BA_HIP_CHECK(hipMalloc((void**)&net->m, n * sizeof(float)));
        BA_HIP_CHECK(hipMalloc((void**)&net->v, n * sizeof(float)));
        BA_HIP_CHECK(hipMalloc((void**)&net->grad, n * sizeof(float)));
        BA_HIP_CHECK(hipMalloc((void**)&net->gsum, n * sizeof(float)));
        BA_HIP_CHECK(hipMalloc((void**)&net->wb, n * sizeof(__bf16)));
        return BA_OK;
    });
    if (s == BA_OK) s = ba_gnn_set_params(net, params);
    if (s != BA_OK) {
        ba_gnn_destroy(net);
        return s;
    }
    *out = net;
    return BA_OK;
}

void ba_gnn_destroy(ba_gnn* net) {
    if (!net) return;
    (void)hipStreamSynchronize(net->stream);
    void* p[] = {net->w, net->m, net->v, net->grad, net->gsum, net->wb};
    for (void* q : p)
        if (q) (void)hipFree(q);
    ba::gnn::free_work(net->work);
    delete net;
}

ba_status ba_gnn_set_params(ba_gnn* net, const float* params) {
    if (!net || !params) return BA_ERR_INVALID_ARG;
    return gnn_guard(&net->err, [&]() {
        const size_t n = ba::gnn::N_PARAMS;
        BA_HIP_CHECK(hipMemcpyAsync(net->w, params, n * sizeof(float), hipMemcpyHostToDevice, net->stream));
        BA_HIP_CHECK(hipMemsetAsync(net->m, 0, n * sizeof(float), net->stream));
        BA_HIP_CHECK(hipMemsetAsync(net->v, 0, n * sizeof(float), net->stream));
        ba::gnn::k_to_bf16<<<ba::gnn::nblk(n), ba::gnn::BS, 0, net->stream>>>(n, net->w, net->wb);
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        net->step = 0;
        return BA_OK;
    });
}

ba_status ba_gnn_get_params(ba_gnn* net, float* params) {
    if (!net || !params) return BA_ERR_INVALID_ARG;
    return gnn_guard(&net->err, [&]() {
        BA_HIP_CHECK(hipMemcpyAsync(params, net->w, ba::gnn::N_PARAMS * sizeof(float), hipMemcpyDeviceToHost, net->stream));
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        return BA_OK;
    });
}

ba_status ba_gnn_graph_from_host(int32_t n_rows, const int64_t* row_ptr, const int32_t* col_idx, const double* blk,
                                 const int32_t* blk_pairs, ba_gnn_graph** out) {
    if (!out || n_rows <= 0 || !row_ptr || !col_idx || !blk) return BA_ERR_INVALID_ARG;
    *out = nullptr;
    for (int32_t r = 0; r < n_rows; ++r)
        if (row_ptr[r + 1] <= row_ptr[r] || col_idx[row_ptr[r]] != r) {
            g_gnn_error = "each row needs its diagonal block first";
            return BA_ERR_INVALID_ARG;
        }
    const int64_t n_blk = row_ptr[n_rows];
    for (int64_t k = 0; k < n_blk; ++k)
        if (col_idx[k] < 0 || col_idx[k] >= n_rows) {
            g_gnn_error = "column index out of range";
            return BA_ERR_INVALID_ARG;
        }
    ba_gnn_graph* G = new ba_gnn_graph();
    double* dblk = nullptr;
    ba_status s = gnn_guard(nullptr, [&]() {
        ba::gnn::build_graph(G->g, n_rows, row_ptr, col_idx, blk_pairs, nullptr);
        BA_HIP_CHECK(hipMalloc((void**)&dblk, (size_t)n_blk * 81 * sizeof(double)));
        BA_HIP_CHECK(hipMemcpy(dblk, blk, (size_t)n_blk * 81 * sizeof(double), hipMemcpyHostToDevice));
        ba::gnn::compute_features(G->g, dblk, nullptr);
        int flag = 0;
        BA_HIP_CHECK(hipMemcpy(&flag, G->g.flags, sizeof(int), hipMemcpyDeviceToHost));
        BA_HIP_CHECK(hipFree(dblk));
        dblk = nullptr;
        if (flag) {
            g_gnn_error = "a diagonal block is not positive definite";
            return BA_ERR_NOT_SPD;
        }
        return BA_OK;
    });
    if (dblk) (void)hipFree(dblk);
    if (s != BA_OK) {
        ba::gnn::free_graph(G->g);
        delete G;
        return s;
    }
    *out = G;
    return BA_OK;
}

void ba_gnn_graph_destroy(ba_gnn_graph* G) {
    if (!G) return;
    (void)hipDeviceSynchronize();
    ba::gnn::free_graph(G->g);
    delete G;
}

ba_status ba_gnn_loss_grad(ba_gnn* net, ba_gnn_graph* G, int32_t n_probes, const float* probes, uint64_t seed,
                           double* loss_host, float* grad_host) {
    if (!net || !G || n_probes <= 0) return BA_ERR_INVALID_ARG;
    return gnn_guard(&net->err, [&]() {
        ba::gnn::loss_grad(net, G->g, n_probes, probes, seed, grad_host ? net->grad : nullptr, net->stream);
        if (loss_host)
            BA_HIP_CHECK(hipMemcpyAsync(loss_host, net->work.loss, sizeof(double), hipMemcpyDeviceToHost, net->stream));
        if (grad_host)
            BA_HIP_CHECK(hipMemcpyAsync(grad_host, net->grad, ba::gnn::N_PARAMS * sizeof(float), hipMemcpyDeviceToHost,
                                        net->stream));
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        return BA_OK;
    });
}

ba_status ba_gnn_train_step(ba_gnn* net, ba_gnn_graph* const* graphs, int32_t n_graphs, int32_t n_probes, uint64_t seed,
                            float lr, double* loss_host) {
    if (!net || !graphs || n_graphs <= 0 || n_probes <= 0 || !(lr > 0.f)) return BA_ERR_INVALID_ARG;
    return gnn_guard(&net->err, [&]() {
        double total = 0.0;
        for (int32_t i = 0; i < n_graphs; ++i) {
            ba::gnn::loss_grad(net, graphs[i]->g, n_probes, nullptr, seed + 0x632BE59BD9B4E019ull * (uint64_t)(i + 1),
                               net->grad, net->stream);
            ba::gnn::accumulate(net->grad, net->gsum, i == 0, 1.f / (float)n_graphs, net->stream);
            double l = 0.0;
            BA_HIP_CHECK(hipMemcpyAsync(&l, net->work.loss, sizeof(double), hipMemcpyDeviceToHost, net->stream));
            BA_HIP_CHECK(hipStreamSynchronize(net->stream));
            total += l;
        }
        ba::gnn::adam(net, net->gsum, lr, net->stream);
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        if (loss_host) *loss_host = total / n_graphs;
        return BA_OK;
    });
}

ba_status ba_gnn_fsai_loss_grad(ba_gnn* net, ba_gnn_graph* G, double* loss_host, float* grad_host) {
    if (!net || !G) return BA_ERR_INVALID_ARG;
    if (!G->g.has_fsai) {
        g_gnn_error = "graph built without common-point counts (no FSAI sets)";
        return BA_ERR_STATE;
    }
    return gnn_guard(&net->err, [&]() {
        ba::gnn::fsai_loss_grad(net, G->g, grad_host ? net->grad : nullptr, net->stream);
        if (loss_host)
            BA_HIP_CHECK(hipMemcpyAsync(loss_host, net->work.loss, sizeof(double), hipMemcpyDeviceToHost, net->stream));
        if (grad_host)
            BA_HIP_CHECK(hipMemcpyAsync(grad_host, net->grad, ba::gnn::N_PARAMS * sizeof(float), hipMemcpyDeviceToHost,
                                        net->stream));
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        return BA_OK;
    });
}

ba_status ba_gnn_fsai_train_step(ba_gnn* net, ba_gnn_graph* const* graphs, int32_t n_graphs, float lr,
                                 double* loss_host) {
    if (!net || !graphs || n_graphs <= 0 || !(lr > 0.f)) return BA_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n_graphs; ++i)
        if (!graphs[i] || !graphs[i]->g.has_fsai) {
            g_gnn_error = "graph built without common-point counts (no FSAI sets)";
            return BA_ERR_STATE;
        }
    return gnn_guard(&net->err, [&]() {
        double total = 0.0;
        for (int32_t i = 0; i < n_graphs; ++i) {
            ba::gnn::fsai_loss_grad(net, graphs[i]->g, net->grad, net->stream);
            ba::gnn::accumulate(net->grad, net->gsum, i == 0, 1.f / (float)n_graphs, net->stream);
            double l = 0.0;
            BA_HIP_CHECK(hipMemcpyAsync(&l, net->work.loss, sizeof(double), hipMemcpyDeviceToHost, net->stream));
            BA_HIP_CHECK(hipStreamSynchronize(net->stream));
            total += l;
        }
        ba::gnn::adam(net, net->gsum, lr, net->stream);
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        if (loss_host) *loss_host = total / n_graphs;
        return BA_OK;
    });
}

ba_status ba_gnn_fsai_factor(ba_gnn* net, ba_gnn_graph* G, float* G_host) {
    if (!net || !G || !G_host) return BA_ERR_INVALID_ARG;
    if (!G->g.has_fsai) {
        g_gnn_error = "graph built without common-point counts (no FSAI sets)";
        return BA_ERR_STATE;
    }
    return gnn_guard(&net->err, [&]() {
        const size_t nb = (size_t)G->g.n_blk * 81;
        float* dG = nullptr;
        BA_HIP_CHECK(hipMalloc((void**)&dG, nb * sizeof(float)));
        BA_HIP_CHECK(hipMemsetAsync(dG, 0, nb * sizeof(float), net->stream));
        ba::gnn::infer_factor(net, G->g, nullptr, nullptr, nullptr, dG, net->stream);
        BA_HIP_CHECK(hipMemcpyAsync(G_host, dG, nb * sizeof(float), hipMemcpyDeviceToHost, net->stream));
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        BA_HIP_CHECK(hipFree(dG));
        return BA_OK;
    });
}

ba_status ba_gnn_preconditioner(ba_gnn* net, ba_gnn_graph* G, double* P_host) {
    if (!net || !G || !P_host) return BA_ERR_INVALID_ARG;
    return gnn_guard(&net->err, [&]() {
        double* dP = nullptr;
        BA_HIP_CHECK(hipMalloc((void**)&dP, (size_t)G->g.n * 81 * sizeof(double)));
        ba::gnn::infer_preconditioner(net, G->g, nullptr, dP, net->stream);
        BA_HIP_CHECK(hipMemcpyAsync(P_host, dP, (size_t)G->g.n * 81 * sizeof(double), hipMemcpyDeviceToHost, net->stream));
        BA_HIP_CHECK(hipStreamSynchronize(net->stream));
        BA_HIP_CHECK(hipFree(dP));
        return BA_OK;
    });
}

ba_status ba_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t* A, const uint16_t* B, float* C) {
    if (M <= 0 || N <= 0 || K <= 0 || !A || !B || !C) return BA_ERR_INVALID_ARG;
    return gnn_guard(nullptr, [&]() {
        __bf16 *dA = nullptr, *dB = nullptr;
        float* dC = nullptr;
        BA_HIP_CHECK(hipMalloc((void**)&dA, (size_t)M * K * 2));
        BA_HIP_CHECK(hipMalloc((void**)&dB, (size_t)K * N * 2));
        BA_HIP_CHECK(hipMalloc((void**)&dC, (size_t)M * N * 4));
        BA_HIP_CHECK(hipMemcpy(dA, A, (size_t)M * K * 2, hipMemcpyHostToDevice));
        BA_HIP_CHECK(hipMemcpy(dB, B, (size_t)K * N * 2, hipMemcpyHostToDevice));
        ba::gnn::test_gemm(M, N, K, dA, dB, dC, nullptr);
        BA_HIP_CHECK(hipMemcpy(C, dC, (size_t)M * N * 4, hipMemcpyDeviceToHost));
        BA_HIP_CHECK(hipFree(dA));
        BA_HIP_CHECK(hipFree(dB));
        BA_HIP_CHECK(hipFree(dC));
        return BA_OK;
    });
}

}  // extern "C"
