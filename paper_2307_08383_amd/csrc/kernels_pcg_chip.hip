// PCG (Sec. 3.2, Eq. (6)-(7)) with the whole solve in one kernel, for
// systems whose block rows fit the chip's registers: every workgroup holds
// the rows of S it owns (both triangles) in registers for the whole solve, so
// an iteration reads no block of S and launches nothing.  The recurrence, the
// stop test and the deflation are those of kernels_pcg.hip (its kernels A, B,
// Bf and Cf); the set-up kernels run before it as usual.
//
// What bounds it is latency: per iteration one grid-wide sum (d^T q), whose
// result every workgroup needs before it can go on, and the exchange of the
// vector z (with the factorised preconditioner also r' and t) with the
// workgroups that own neighbouring rows.  The second sum (r^T z, r^T r, the
// deflation's (S W)^T z) is taken after the next product, so it costs no
// wait.  On the 2,000-camera block (198 workgroups) an iteration takes 7.1 us:
// 2.3 for the first sum, 1.9 for the exchange, 1.2 for the product with its
// row sums, 0.6 to collect the second sum, the rest barriers and the row's
// own work.  One kernel per phase instead (each followed by the partial sums
// and the index, block and vector loads that depend on each other) took
// 16.8 us.  Per iteration against those kernels: 16 cameras in one workgroup
// 2.7 us (7.9), 84 rows of shared intrinsics 5.3 (10.8), 300 cameras with a
// dense S and FSAI 23 (37.8), FSAI with deflation on the 2,000-camera block
// 21.7 (26.4: its factors stay in the L2s and it exchanges three vectors).
//
// Exchange: a double travels as two 8-byte words, each half the value and
// the number of the exchange it belongs to.  Words are written and read with
// relaxed device-scope atomics (which bypass the caches that are not shared
// by all workgroups), and a reader polls the data itself until the number is
// the one it waits for: one trip through memory, no flag and no cache
// write-back.  (A device-scope fence, which writes back and invalidates the
// L2s, takes 45 us with 256 workgroups.)  Words of step k + 1 are written
// only after the grid-wide sum of step k, to which every reader of the old
// words has contributed by then; the sums alternate between two buffers, so
// one buffer per vector is enough.  The sums' words are written to kRep
// replicas, each polled by a part of the workgroups (250 workgroups: 3.6 us a
// sum with one copy, 2.7 with 4 or 8).
//
// All workgroups are resident at once (cooperative launch, at most one per
// CU).  Every wait is bounded all the same: a workgroup that waits too long
// reports it in state[4] and returns, so do the others, and the host solves
// with the kernels of kernels_pcg.hip.
#include <algorithm>

#include "ba_common.hpp"

namespace ba {

namespace {

constexpr int BS = 512;
constexpr int NW = BS / kWave;         // 8 waves
constexpr int GRPW = kWave / 9;        // 7 lane groups of 9 per wave
constexpr int kGrp = NW * GRPW;        // 56 lane groups
constexpr int kMaxNB = 11;             // blocks of S held by a lane group (FP64: 198 registers a lane)
constexpr int kCap = kGrp * kMaxNB;    // blocks of S a workgroup can hold
constexpr int kMaxRows = 40;           // rows per workgroup (one thread per component; bounded by LDS)
constexpr int kMaxG = 256;             // workgroups (one per CU)
constexpr int kRep = 4;                // replicas of a sum's words
constexpr int NP = 9;                  // values of a partial (kernels_pcg.hip)
constexpr int kW = 7;
constexpr int kSpin = 1 << 21;         // polls before a wait gives up (over a second)

struct ChipArgs {
    int max_iter, n_part, s32;
    double tol;
    const int32_t *brow, *cptr, *cols;                 // plan (ba::Chip)
    const int32_t *sf_ptr, *sf_col, *sf_src;           // rows of both triangles
    const double *blk, *M;
    const double *x, *r, *z, *pR;                      // set-up results
    const double *W, *SW, *Einv;
    double* out;
    int* state;
    double* scal;
    u64* stamp;
    u64 *zlo, *zhi, *rlo, *rhi, *tlo, *thi, *slots;    // exchanged words
    const int32_t *gl_ptr, *gl_col, *gu_ptr, *gu_col;  // factor by rows and its transpose by rows
    const float *Gl, *Gu;
};

// (a base that is the same for all threads and a 32-bit byte offset, so that
// no 64-bit address per array lives in the registers)
__device__ __forceinline__ void put(u64* lo, u64* hi, unsigned off, double v, unsigned ep) {
    const u64 b = __builtin_bit_cast(u64, v);
    __hip_atomic_store((u64*)((char*)lo + off), (b & 0xffffffffull) | ((u64)ep << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store((u64*)((char*)hi + off), (b >> 32) | ((u64)ep << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 peek(const u64* p, unsigned off) {
    return __hip_atomic_load((const u64*)((const char*)p + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double join(u64 lo, u64 hi) {
    return __builtin_bit_cast(double, (lo & 0xffffffffull) | (hi << 32));
}

struct __attribute__((packed, aligned(4))) Row3f { float a, b, c; };
__device__ __forceinline__ void load_row9(const float* __restrict__ p, float* v) {
    const Row3f* r = reinterpret_cast<const Row3f*>(p);
    const Row3f x = r[0], y = r[1], z = r[2];
    v[0] = x.a; v[1] = x.b; v[2] = x.c; v[3] = y.a; v[4] = y.b; v[5] = y.c; v[6] = z.a; v[7] = z.b; v[8] = z.c;
}

// position of column c in the workgroup's ascending column list
__device__ __forceinline__ int find_col(const int* cols, int n, int c) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (cols[m] < c) lo = m + 1; else hi = m;
    }
    return lo;
}

// A workgroup's rows are r0 .. r0 + R - 1; row lr takes the lane groups
// gs[lr] .. gs[lr + 1] - 1, each with NB consecutive blocks of the row.
// Thread 9 lr + i owns component i of row lr of every vector.
//
// The nine lanes of a group hold a block by rows (lane i forms component i of
// its product, reading the vector's nine values from LDS) or, with 4 to 8
// blocks a group, by columns: a lane then reads one value a block and the
// group sums its nine partial results through LDS once, 18 + NB LDS accesses
// a lane instead of 9 NB, which is what bounds the product (128 bytes a clock).
// With 11 blocks the nine sums would not fit the registers beside them.

template <int NB, bool FACT, bool DEFL>
__global__ __launch_bounds__(BS) void k_pcg_chip(ChipArgs a) {
    constexpr bool kCol = NB >= 4 && NB <= 8;
    constexpr int NV = DEFL ? NP : 2;                    // values of a step's second sum
    constexpr int kBlk = kGrp * NB;                      // blocks of S, and distinct columns, of a workgroup
    __shared__ double zs[kBlk][9];                       // the vector's rows this workgroup reads
    __shared__ double part[kGrp][9];
    __shared__ double pc[kCol ? kGrp : 1][9][9];         // a group's partial results, [component][lane]
    __shared__ double sM[FACT ? 1 : kMaxRows][81];
    __shared__ double sr[FACT && !DEFL ? 1 : kMaxRows][9];
    __shared__ double sW[DEFL ? 2 * kW : 1][DEFL ? kMaxRows * 9 : 1];   // W and S W of the own rows
    __shared__ double sE[DEFL ? kW * kW : 1], smu[DEFL ? kW : 1];
    __shared__ double sz[DEFL ? kMaxRows * 9 : 1];
    __shared__ double sh[NV * NW], shw[NV * 4];
    __shared__ int scol[kBlk];
    __shared__ int16_t slc[kBlk];                        // position in zs of every block's column
    __shared__ int gs[kMaxRows + 1];
    __shared__ int16_t sgl[FACT ? kBlk : 1], sgu[FACT ? kBlk : 1];
    __shared__ int fg[FACT ? 2 : 1][kMaxRows + 2];       // lane groups of the factors' rows; [R + 1]: entries a group
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int G = gridDim.x, wg = blockIdx.x;
    const int r0 = a.brow[wg], R = a.brow[wg + 1] - r0;
    const int c0 = a.cptr[wg], nc = a.cptr[wg + 1] - c0;
    for (int u = tid; u < nc; u += BS) scol[u] = a.cols[c0 + u];
    for (int u = tid; u < kGrp * NB; u += BS) slc[u] = 0;
    if (tid < NV * NW) sh[tid] = 0.0;
    if (tid < NV * 4) shw[tid] = 0.0;
    if (tid == 0) s_bad = 0;
    // lane groups of the rows before row `lane` when a group takes up to q of
    // a row's entries (one wave: R <= 40)
    auto group_starts = [&](const int32_t* ptr, int q, int* out) {
        int n = lane < R ? (ptr[r0 + lane + 1] - ptr[r0 + lane] + q - 1) / q : 0;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_up(n, o, kWave);
            if (lane >= o) n += t;
        }
        if (lane < R) out[lane + 1] = n;
        if (lane == 0) out[0] = 0;
        return __shfl(n, kWave - 1, kWave);   // groups in all
    };
    if (wave == 0) group_starts(a.sf_ptr, NB, gs);
    if (FACT && (wave == 1 || wave == 2)) {
        // the fewest entries a group that fit the lane groups (a factor's rows
        // have at most the entries of S's rows, so kMaxNB always fits)
        const int32_t* ptr = wave == 1 ? a.gl_ptr : a.gu_ptr;
        int q = 1;
        while (group_starts(ptr, q, fg[wave - 1]) > kGrp && q < kMaxNB) ++q;
        if (lane == 0) fg[wave - 1][R + 1] = q;
    }
    __syncthreads();
    // this lane's part of the workgroup's blocks of S
    const int grp = lane < GRPW * 9 ? wave * GRPW + lane / 9 : kGrp;
    const int comp = lane % 9;
    double b[NB][9];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int c = 0; c < 9; ++c) b[j][c] = 0.0;
    if (grp < gs[R]) {
        int lr = 0;
        while (gs[lr + 1] <= grp) ++lr;
        const int e0 = a.sf_ptr[r0 + lr] + (grp - gs[lr]) * NB, e1 = a.sf_ptr[r0 + lr + 1];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int e = e0 + j;
            if (e < e1) {
                const int src = a.sf_src[e];
                const double* B = a.blk + (int64_t)(src >> 1) * 81;
                const bool strided = ((src & 1) != 0) != kCol;   // transposed block by rows, or stored one by columns
                const int base = strided ? comp : comp * 9, step = strided ? 9 : 1;
#pragma unroll
                for (int c = 0; c < 9; ++c) {
                    const double v = B[base + c * step];
                    b[j][c] = a.s32 ? (double)(float)v : v;
                }
                if (comp == 0) slc[grp * NB + j] = (int16_t)find_col(scol, nc, a.sf_col[e]);
            }
        }
    }
    // thread (row, component): its entries of the vectors
    const bool own = tid < R * 9;
    const int lr = tid / 9, ci = tid % 9;
    const int64_t o = (int64_t)(r0 + lr) * 9 + ci;
    double x = 0.0, r = 0.0, z = 0.0, q = 0.0, d = 0.0;
    if (own) { x = a.x[o]; r = a.r[o]; z = a.z[o]; }
    for (int u = tid; u < nc * 9; u += BS) zs[u / 9][u % 9] = a.z[(int64_t)scol[u / 9] * 9 + u % 9];
    if (DEFL) {
        if (own)
            for (int v = 0; v < kW; ++v) {
                sW[v][tid] = a.W[((int64_t)(r0 + lr) * kW + v) * 9 + ci];
                sW[kW + v][tid] = a.SW[((int64_t)(r0 + lr) * kW + v) * 9 + ci];
            }
        if (tid < kW * kW) sE[tid] = a.Einv[tid];
    }
    int fl_e0 = 0, fl_n = 0, fu_e0 = 0, fu_n = 0;   // this lane group's entries of both factors
    if (FACT) {
        const int gl0 = a.gl_ptr[r0], ngl = a.gl_ptr[r0 + R] - gl0;
        const int gu0 = a.gu_ptr[r0], ngu = a.gu_ptr[r0 + R] - gu0;
        for (int u = tid; u < ngl; u += BS) sgl[u] = (int16_t)find_col(scol, nc, a.gl_col[gl0 + u]);
        for (int u = tid; u < ngu; u += BS) sgu[u] = (int16_t)find_col(scol, nc, a.gu_col[gu0 + u]);
        auto mine = [&](const int32_t* ptr, const int* g, int base, int& e0, int& n) {
            if (grp >= g[R]) return;
            int l = 0;
            while (g[l + 1] <= grp) ++l;
            const int per = g[R + 1];
            e0 = ptr[r0 + l] + (grp - g[l]) * per - base;
            n = min(per, ptr[r0 + l + 1] - base - e0);
        };
        mine(a.gl_ptr, fg[0], gl0, fl_e0, fl_n);
        mine(a.gu_ptr, fg[1], gu0, fu_e0, fu_n);
    } else {
        for (int u = tid; u < R * 81; u += BS) sM[u / 81][u % 81] = a.M[(int64_t)r0 * 81 + u];
    }
    // totals of the set-up's partials
#pragma unroll 1
    for (int j = 0; j < NV; ++j) {
        double t = 0.0;
        for (int i = tid; i < a.n_part; i += BS) t += a.pR[(int64_t)i * NP + j];
        t = wave_sum(t);
        if (lane == 0) sh[j * NW + wave] = t;
    }
    __syncthreads();
    auto waves = [&](int j) {   // sum of value j over the waves
        double t[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) t[w] = sh[j * NW + w];
        return ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    };
    double rz = waves(0), rr = waves(1);
    if (DEFL && tid < kW) shw[(2 + tid) * 4] = waves(2 + tid);   // shw: the totals in four parts
    __syncthreads();
    const int own_waves = (R * 9 + kWave - 1) / kWave;
    if (tid < NV * NW && tid % NW >= own_waves) sh[tid] = 0.0;   // those waves add nothing to sums of their own threads
    const double r0sq = rr;
    // Grid-wide sums: publish1() / publish2() leave this workgroup's sums,
    // collect() the totals of n values over all workgroups in shw (four parts
    // each, the same order, so the same values, everywhere), false if a wait
    // was too long.  nsum numbers them.
    unsigned nsum = 0, nvec = 0;
    auto post = [&](int n) {
        ++nsum;
        __syncthreads();
        if (G == 1) {
            if (tid < n) shw[tid * 4] = waves(tid);
        } else if (tid < n * kRep) {
            const int j = tid % n, rep = tid / n;
            put(a.slots, a.slots + kMaxG, (((((nsum & 1) * kRep + rep) * NP + j) * 2) * kMaxG + wg) * 8u, waves(j), nsum);
        }
    };
    auto publish1 = [&](double v) {
        if (wave < own_waves) {
            const double s = wave_sum(own ? v : 0.0);
            if (lane == 0) sh[wave] = s;
        }
        post(1);
    };
    // r^T z, r^T r and, deflated, (S W)^T z: two sums a wave over its own
    // threads, or (nine sums) each wave one or two sums over all own threads
    auto publish2 = [&](double r, double z) {
        if (!DEFL) {
            if (wave < own_waves) {
                const double s0 = wave_sum(own ? r * z : 0.0), s1 = wave_sum(own ? r * r : 0.0);
                if (lane == 0) { sh[wave] = s0; sh[NW + wave] = s1; }
            }
        } else {
            if (own) { sr[DEFL ? lr : 0][ci] = r; sz[DEFL ? tid : 0] = z; }
            __syncthreads();
            for (int j = wave; j < NV; j += NW) {
                double s = 0.0;
                for (int t = lane; t < R * 9; t += kWave) {
                    const double zt = sz[DEFL ? t : 0], rt = (&sr[0][0])[DEFL ? t : 0];
                    s += j == 0 ? rt * zt : j == 1 ? rt * rt : sW[DEFL ? kW + j - 2 : 0][DEFL ? t : 0] * zt;
                }
                s = wave_sum(s);
                if (lane < NW) sh[j * NW + lane] = lane == 0 ? s : 0.0;
            }
        }
        post(NV);
    };
    // waves 0..3 poll the first half of the values, waves 4..7 the second; a
    // thread polls one workgroup's words
    auto collect = [&](int n) {
        constexpr int kAt = DEFL ? 3 : 1;   // values a poll
        const int half = wave / 4, j1 = half ? n : (n + 1) / 2;
        if (G > 1 && (wave % 4) * kWave < G) {   // waves past the last workgroup's words add nothing
            const int t = tid % kMaxG;
            const unsigned p = ((((nsum & 1) * kRep + wg % kRep) * NP * 2) * kMaxG + min(t, G - 1)) * 8u;
#pragma unroll 1
            for (int j0 = half * ((n + 1) / 2); j0 < j1; j0 += kAt) {
                u64 w[kAt][2];
                int spin = 0;
                for (;;) {
                    bool ok = true;
#pragma unroll
                    for (int i = 0; i < kAt; ++i) {
                        const int j = min(j0 + i, j1 - 1);
                        w[i][0] = peek(a.slots, p + (2 * j) * kMaxG * 8u);
                        w[i][1] = peek(a.slots + kMaxG, p + (2 * j) * kMaxG * 8u);
                    }
#pragma unroll
                    for (int i = 0; i < kAt; ++i)
                        ok = ok && (unsigned)(w[i][0] >> 32) == nsum && (unsigned)(w[i][1] >> 32) == nsum;
                    if (ok) break;
                    if (++spin > kSpin) { s_bad = 1; break; }
                }
#pragma unroll
                for (int i = 0; i < kAt; ++i) {
                    const double s = wave_sum(t < G ? join(w[i][0], w[i][1]) : 0.0);
                    if (lane == 0 && j0 + i < j1) shw[(j0 + i) * 4 + wave % 4] = s;
                }
            }
        }
        __syncthreads();
        return s_bad == 0;
    };
    auto total = [&](int j) { return (shw[j * 4] + shw[j * 4 + 1]) + (shw[j * 4 + 2] + shw[j * 4 + 3]); };
    // Own value v of a vector out to the other workgroups, and the rows this
    // workgroup reads into zs.  nvec numbers the iterations' exchanges.
    // Two values a thread at once (more would not fit the registers).
    auto receive = [&](int u0, const u64* lo, const u64* hi) {
        constexpr int kEx = 2;
        const int n = nc * 9;
        unsigned at[kEx];
        u64 w[kEx][2];
#pragma unroll
        for (int i = 0; i < kEx; ++i) {
            const int u = u0 + i * BS < n ? u0 + i * BS : u0;
            at[i] = (unsigned)(scol[u / 9] * 9 + u % 9) * 8u;
        }
        int spin = 0;
        for (;;) {
            bool ok = true;
#pragma unroll
            for (int i = 0; i < kEx; ++i) { w[i][0] = peek(lo, at[i]); w[i][1] = peek(hi, at[i]); }
#pragma unroll
            for (int i = 0; i < kEx; ++i) ok = ok && (unsigned)(w[i][0] >> 32) == nvec && (unsigned)(w[i][1] >> 32) == nvec;
            if (ok) break;
            if (++spin > kSpin) { s_bad = 1; break; }
        }
#pragma unroll
        for (int i = 0; i < kEx; ++i) {
            const int u = u0 + i * BS;
            if (u < n) (&zs[0][0])[u] = join(w[i][0], w[i][1]);
        }
    };
    auto exchange = [&](double v, u64* lo, u64* hi) {
        if (G == 1) {
            if (own) zs[lr][ci] = v;   // the column list is all rows
            __syncthreads();
            return true;
        }
        if (own) put(lo, hi, (unsigned)o * 8u, v, nvec);
#pragma unroll 1
        for (int u = tid; u < nc * 9; u += 2 * BS) receive(u, lo, hi);
        __syncthreads();
        return s_bad == 0;
    };
    // Sum of the partial results of lane groups g0 .. g1 - 1, in order
    auto group_sum = [&](int g0, int g1) {
        double s = 0.0;
        for (int g = g0; g < g1; g += 8) {
            double t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j] = part[min(g + j, g1 - 1)][ci];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += g + j < g1 ? t[j] : 0.0;
        }
        return s;
    };
    // Own value of a factor times the vector in zs (requesting a lane group's
    // entries before the exchange spills at 8 blocks of S a group and costs
    // more than it saves: 24 to 33 us an iteration against 21, FSAI with
    // deflation on the 2,000-camera block)
    auto factor = [&](const float* F, const int* g, int e0, int n, const int16_t* li) {
        constexpr int U = NB >= 6 ? 1 : 2;   // entries in flight
        double y = 0.0;
#pragma unroll 1
        for (int e = 0; e < n; e += U) {
            float f[U][9];
#pragma unroll
            for (int u = 0; u < U; ++u)
                load_row9((const float*)((const char*)F + (unsigned)((e0 + min(e + u, n - 1)) * 81 + comp * 9) * 4u), f[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e + u >= n) break;
                const double* v = zs[li[e0 + e + u]];
#pragma unroll
                for (int c = 0; c < 9; ++c) y += (double)f[u][c] * v[c];
            }
        }
        if (grp < kGrp) part[grp][comp] = y;
        __syncthreads();
        return own ? group_sum(g[lr], g[lr + 1]) : 0.0;
    };
    const int sg = min(grp, kGrp - 1) * NB;
    int k = 0;
    double rz_old = 1.0;
    bool fine = true;
    __syncthreads();
    for (;;) {
        // S z: the product needs no scalar, so it goes before the sums of the
        // previous step are collected
        double y = 0.0;
        if (kCol) {
            double acc[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) acc[i] = 0.0;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const double v = zs[slc[sg + j]][comp];
#pragma unroll
                for (int i = 0; i < 9; ++i) acc[i] += b[j][i] * v;
            }
            // within the wave, whose LDS accesses run in order: no barrier of the
            // workgroup, but the reads must stay after all the writes
            if (grp < kGrp)
#pragma unroll
                for (int i = 0; i < 9; ++i) pc[kCol ? grp : 0][i][comp] = acc[i];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (grp < kGrp)
#pragma unroll
                for (int i = 0; i < 9; ++i) y += pc[kCol ? grp : 0][comp][i];
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const double* v = zs[slc[sg + j]];
#pragma unroll
                for (int c = 0; c < 9; ++c) y += b[j][c] * v[c];
            }
        }
        if (grp < kGrp) part[grp][comp] = y;
        __syncthreads();
        const double s = own ? group_sum(gs[lr], gs[lr + 1]) : 0.0;
        if (k > 0) {
            if (!collect(NV)) { fine = false; break; }
            rz_old = rz;
            rz = total(0);
            rr = total(1);
        }
        const bool conv = (rr == 0.0) || (sqrt(rr) <= a.tol * sqrt(r0sq));
        if (conv || k >= a.max_iter) {
            if (wg == 0 && tid == 0) {
                a.state[0] = 1;
                a.state[2] = conv ? BA_OK : BA_ERR_NOT_CONVERGED;
                a.state[3] = k;
                a.scal[1] = r0sq > 0.0 ? sqrt(rr / r0sq) : 0.0;
            }
            break;
        }
        const double beta = k == 0 ? 0.0 : rz / rz_old;
        double wm = 0.0, swm = 0.0;
        if (DEFL) {
            if (tid < kW) {
                double mu = 0.0;
#pragma unroll 2
                for (int v = 0; v < kW; ++v) mu += sE[DEFL ? tid * kW + v : 0] * total(DEFL ? 2 + v : 0);
                smu[tid] = mu;
            }
            __syncthreads();
            if (own)
#pragma unroll
                for (int u = 0; u < kW; ++u) {
                    const double mu = smu[DEFL ? u : 0];
                    wm += sW[DEFL ? u : 0][DEFL ? tid : 0] * mu;
                    swm += sW[DEFL ? kW + u : 0][DEFL ? tid : 0] * mu;
                }
        }
        q = (k == 0 ? s : s + beta * q) - swm;
        d = (k == 0 ? z : z + beta * d) - wm;
        publish1(d * q);   // has a barrier between the last read of shw and its reuse
        if (!collect(1)) { fine = false; break; }
        const double dq = total(0);
        if (!(dq > 0.0)) {
            if (wg == 0 && tid == 0) { a.state[0] = 1; a.state[2] = BA_ERR_NOT_SPD; a.state[3] = k; }
            break;
        }
        const double alpha = rz / dq;
        x += alpha * d;
        r -= alpha * q;
        ++nvec;
        if (FACT) {
            if (!exchange(own ? r : 0.0, a.rlo, a.rhi)) { fine = false; break; }
            const double t = factor(a.Gl + (int64_t)a.gl_ptr[r0] * 81, fg[0], fl_e0, fl_n, sgl);
            if (!exchange(t, a.tlo, a.thi)) { fine = false; break; }
            z = factor(a.Gu + (int64_t)a.gu_ptr[r0] * 81, fg[FACT ? 1 : 0], fu_e0, fu_n, sgu);
        } else {
            if (own) sr[FACT ? 0 : lr][ci] = r;
            __syncthreads();
            if (own) {
                z = 0.0;
#pragma unroll
                for (int c = 0; c < 9; ++c) z += sM[FACT ? 0 : lr][ci * 9 + c] * sr[FACT ? 0 : lr][c];
            }
        }
        publish2(r, z);
        if (!exchange(z, a.zlo, a.zhi)) { fine = false; break; }
        ++k;
    }
    if (!fine) {
        if (tid == 0) a.state[4] = 1;
        return;
    }
    if (own) a.out[o] = x;
    stamp_now(a.stamp);
}

template <int NB>
const void* chip_kernel(bool fact, bool defl) {
    if (fact) return defl ? (const void*)k_pcg_chip<NB, true, true> : (const void*)k_pcg_chip<NB, true, false>;
    return defl ? (const void*)k_pcg_chip<NB, false, true> : (const void*)k_pcg_chip<NB, false, false>;
}

const void* chip_kernel(int nb, bool fact, bool defl) {
    switch (nb) {
        case 1: return chip_kernel<1>(fact, defl);
        case 2: return chip_kernel<2>(fact, defl);
        case 4: return chip_kernel<4>(fact, defl);
        case 6: return chip_kernel<6>(fact, defl);
        case 8: return chip_kernel<8>(fact, defl);
        default: return chip_kernel<kMaxNB>(fact, defl);
    }
}

}  // namespace

// The plan of the on-chip solve from the rows of both triangles (host):
// contiguous rows per workgroup, as few blocks per lane group as possible
// (NB) with at most one workgroup per CU; a system that fits one workgroup
// takes one (its sums need no exchange).  G = 0: the system does not fit.
void plan_chip(int n_rows, const int32_t* sf_ptr, const int32_t* sf_col, int n_cu, ChipPlan& P) {
    P = ChipPlan();
    const int most = std::min(kMaxG, n_cu);
    auto cut = [&](int nb, std::vector<int32_t>& brow) {
        brow.assign(1, 0);
        int groups = 0;
        for (int r = 0; r < n_rows; ++r) {
            const int n = (sf_ptr[r + 1] - sf_ptr[r] + nb - 1) / nb;
            if (n > kGrp) return false;
            if (groups + n > kGrp || r - brow.back() >= kMaxRows) {
                brow.push_back(r);
                groups = 0;
                if ((int)brow.size() > most) return false;
            }
            groups += n;
        }
        brow.push_back(n_rows);
        return true;
    };
    if (n_rows <= 0 || sf_ptr[n_rows] > (int64_t)kCap * most) return;
    std::vector<int32_t> brow;
    for (int one = 1; one >= 0 && P.NB == 0; --one)
        for (int nb : {1, 2, 4, 6, 8, kMaxNB})
            if (cut(nb, brow) && (!one || brow.size() == 2)) {
                P.NB = nb;
                break;
            }
    if (P.NB == 0) return;
    P.G = (int)brow.size() - 1;
    P.cptr.assign(1, 0);
    std::vector<int32_t> seen(n_rows, -1);   // last workgroup that listed a column
    for (int g = 0; g < P.G; ++g) {
        const size_t c0 = P.cols.size();
        if (P.G == 1) {   // all rows, in order: the exchange writes them in place
            for (int r = 0; r < n_rows; ++r) P.cols.push_back(r);
        } else {
            for (int32_t e = sf_ptr[brow[g]]; e < sf_ptr[brow[g + 1]]; ++e)
                if (seen[sf_col[e]] != g) {
                    seen[sf_col[e]] = g;
                    P.cols.push_back(sf_col[e]);
                }
            std::sort(P.cols.begin() + c0, P.cols.end());
        }
        P.cptr.push_back((int32_t)P.cols.size());
    }
    P.brow = std::move(brow);
}

// The solve after its set-up (k_pcg_init, which cleared the exchanged words,
// and for mode 1 the first z); false if it could not be launched.
bool launch_chip(ba_ctx* c, int mode, const double* M, int defl, int n_part, double tol, int max_iter, double* out) {
    const Chip& H = c->chip;
    const Pcg& P = c->pcg;
    const Fsai& F = c->fs;
    ChipArgs a{};
    a.max_iter = max_iter; a.n_part = n_part; a.s32 = c->s32; a.tol = tol;
    a.brow = H.brow; a.cptr = H.cptr; a.cols = H.cols;
    a.sf_ptr = c->sf_ptr; a.sf_col = c->sf_col; a.sf_src = c->sf_src;
    a.blk = c->blk; a.M = M;
    a.x = P.x; a.r = P.r[0]; a.z = P.z; a.pR = P.pR;
    a.W = P.W; a.SW = P.SW; a.Einv = P.Einv;
    a.out = out; a.state = P.state; a.scal = P.scal; a.stamp = c->h_stamp + kStBack;
    // vectors of the other kernels and the deflation's partials, free here
    a.zlo = (u64*)P.u; a.zhi = (u64*)P.q; a.rlo = (u64*)P.d; a.rhi = (u64*)P.r[1];
    a.tlo = (u64*)P.tb; a.thi = (u64*)F.tg; a.slots = (u64*)P.pE;
    static_assert(2 * kRep * NP * 2 * kMaxG <= 49 * 1024, "the sums' words fit the deflation partials");
    if (mode != 0) {
        a.gl_ptr = F.ptr; a.gl_col = F.J; a.gu_ptr = F.gu_ptr; a.gu_col = F.gu_col;
        a.Gl = F.Gl; a.Gu = F.Gu;
    }
    const void* k = chip_kernel(H.NB, mode != 0, defl);
    void* args[] = {&a};
    const hipError_t e = H.G == 1 ? hipLaunchKernel(k, dim3(1), dim3(BS), args, 0, c->stream)
                                  : hipLaunchCooperativeKernel(k, dim3(H.G), dim3(BS), args, 0, c->stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

// Words that the set-up clears for launch_chip
int64_t chip_slot_words() { return (int64_t)2 * kRep * NP * 2 * kMaxG; }

}  // namespace ba
