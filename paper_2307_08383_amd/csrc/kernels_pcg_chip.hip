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
// wait; its words are asked for before the product, and z goes out before the
// sums are formed, so that the first poll for it finds it.  On the 2,000-camera
// block (198 workgroups) an iteration takes 6.6 us, on 300 cameras (36) 4.7:
// 2.5 (1.2) for the first sum, 1.5 for the exchange, 1.2 for the product with
// its row sums, the rest barriers and the row's own work.  One kernel per phase
// instead (each followed by the partial sums and the index, block and vector
// loads that depend on each other) took 16.8 us.  Per iteration against those
// kernels: 16 cameras in one workgroup 2.7 us (7.9), 84 rows of shared
// intrinsics 4.5 (10.8), 300 cameras with a dense S and FSAI 22 (37.8), FSAI
// with deflation on the 2,000-camera block 21.7 (26.4: its factors stay in the
// L2s and it exchanges three vectors).
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
    constexpr bool kPeek = !FACT && !DEFL && NB <= 8;    // registers for words and places held ahead
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
    // thread polls one workgroup's words.  peek_sums: the first poll's loads,
    // ahead of work that needs no sum
    constexpr int kAt = DEFL ? 3 : 1;      // values a poll
    u64 wp[kPeek ? kAt : 1][2];
    const int half = wave / 4, tw = tid % kMaxG;
    const bool polls = G > 1 && (wave % 4) * kWave < G;   // waves past the last workgroup's words add nothing
    auto peek_sums = [&](int j0, int j1, u64 (*w)[2]) {
        const unsigned p = ((((nsum & 1) * kRep + wg % kRep) * NP * 2) * kMaxG + min(tw, G - 1)) * 8u;
#pragma unroll
        for (int i = 0; i < kAt; ++i) {
            const int j = min(j0 + i, j1 - 1);
            w[i][0] = peek(a.slots, p + (2 * j) * kMaxG * 8u);
            w[i][1] = peek(a.slots + kMaxG, p + (2 * j) * kMaxG * 8u);
        }
    };
    auto collect = [&](int n, bool peeked) {
        const int j1 = half ? n : (n + 1) / 2;
        if (polls) {
            const int t = tw;
#pragma unroll 1
            for (int j0 = half * ((n + 1) / 2); j0 < j1; j0 += kAt) {
                u64 w[kAt][2];
                int spin = 0;
                for (;;) {
                    bool ok = true;
                    if (kPeek && peeked) {
#pragma unroll
                        for (int i = 0; i < kAt; ++i) { w[i][0] = wp[kPeek ? i : 0][0]; w[i][1] = wp[kPeek ? i : 0][1]; }
                    } else {
                        peek_sums(j0, j1, w);
                    }
                    peeked = false;
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
    constexpr int kEx = 2;
    auto places = [&](int u0, unsigned* at) {
#pragma unroll
        for (int i = 0; i < kEx; ++i) {
            const int u = u0 + i * BS < nc * 9 ? u0 + i * BS : min(u0, nc * 9 - 1);
            at[i] = (unsigned)(scol[u / 9] * 9 + u % 9) * 8u;
        }
    };
    unsigned at0[kPeek ? kEx : 1];   // of the first round, which is the only one up to 113 columns
    if constexpr (kPeek) places(tid, at0);
    auto receive = [&](int u0, const unsigned* at, const u64* lo, const u64* hi) {
        const int n = nc * 9;
        u64 w[kEx][2];
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
    auto send = [&](double v, u64* lo, u64* hi) {
        if (G > 1 && own) put(lo, hi, (unsigned)o * 8u, v, nvec);
    };
    auto take = [&](double v, u64* lo, u64* hi) {
        if (G == 1) {
            if (own) zs[lr][ci] = v;   // the column list is all rows
            __syncthreads();
            return true;
        }
        if constexpr (kPeek)
            if (tid < nc * 9) receive(tid, at0, lo, hi);
#pragma unroll 1
        for (int u = tid + (kPeek ? kEx * BS : 0); u < nc * 9; u += kEx * BS) {
            unsigned at[kEx];
            places(u, at);
            receive(u, at, lo, hi);
        }
        __syncthreads();
        return s_bad == 0;
    };
    auto exchange = [&](double v, u64* lo, u64* hi) {
        send(v, lo, hi);
        return take(v, lo, hi);
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
        // previous step are collected, whose words are asked for now
        if (kPeek && k > 0 && polls) peek_sums(half * ((NV + 1) / 2), half ? NV : (NV + 1) / 2, wp);
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
            if (!collect(NV, kPeek)) { fine = false; break; }
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
        if (!collect(1, false)) { fine = false; break; }
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
        // z goes out before the sums are formed, so that it has arrived, or is
        // nearly there, at the first poll (a poll that misses costs another trip)
        send(z, a.zlo, a.zhi);
        publish2(r, z);
        if (!take(z, a.zlo, a.zhi)) { fine = false; break; }
        ++k;
    }
    if (!fine) {
        if (tid == 0) a.state[4] = 1;
        return;
    }
    if (own) a.out[o] = x;
    stamp_now(a.stamp);
}

// The solve in the order of sums of kernels_pcg.hip's kernels A and B (FULL
// product, block-diagonal M, no deflation), bit for bit, for solves whose
// result hangs on that order (run_pcg).  A wave owns a row, as in kernel A:
// lane group g holds the row's entries g, g + 7, ... by rows and lanes 0..8 add
// the seven groups in order, then hold the row's entries of the vectors.  d^T q
// goes out by four rows (a workgroup of kernel A), r^T z and r^T r by 28 rows (one
// of kernel B): the workgroup that owns the first of these takes r and z of all
// 28 from the exchange and adds them.  All sums run over the same trees.
//   Against the kernel above: rows fixed to eight a workgroup, nine LDS reads a
// block, two vectors exchanged and the second sum behind one more trip: 7.8 us
// an iteration against 6.6 on the 2,000-camera block, 6.4 against 4.7 on 300
// cameras, where one kernel per phase takes 16.8 and 11.
constexpr int kOrdRows = NW;   // rows of a workgroup
constexpr int kOrdB = 28;      // rows of a partial of the second sum

template <int NB>
__global__ __launch_bounds__(BS) void k_pcg_ord(int n_rows, ChipArgs a) {
    __shared__ double zs[kGrp * NB][9];
    __shared__ double sM[kOrdRows][81];
    __shared__ double sr[kOrdRows][9];
    __shared__ double part[kOrdRows][GRPW][9];
    __shared__ double sh[2][NW], sq[2 * 4];
    __shared__ int scol[kGrp * NB];
    __shared__ int16_t slc[kGrp * NB];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int G = gridDim.x, wg = blockIdx.x;
    const int row = wg * kOrdRows + wave;
    const int c0 = a.cptr[wg], nc = a.cptr[wg + 1] - c0;
    const int n_a = (n_rows + 3) / 4, n_b = (n_rows + kOrdB - 1) / kOrdB;   // partials of the two sums
    for (int u = tid; u < nc; u += BS) scol[u] = a.cols[c0 + u];
    if (tid == 0) s_bad = 0;
    __syncthreads();
    const int grp = lane / 9, comp = lane % 9;
    const bool live = row < n_rows, own = live && lane < 9;
    const int64_t o = (int64_t)row * 9 + comp;
    double b[NB][9];
    int n_own = 0;   // entries of this lane's group
    const int sg = (wave * GRPW + min(grp, GRPW - 1)) * NB;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int c = 0; c < 9; ++c) b[j][c] = 0.0;
        if (live && grp < GRPW) {
            const int e = a.sf_ptr[row] + grp + j * GRPW;
            if (e < a.sf_ptr[row + 1]) {
                const int src = a.sf_src[e];
                const double* B = a.blk + (int64_t)(src >> 1) * 81;
                const int base = (src & 1) ? comp : comp * 9, step = (src & 1) ? 9 : 1;
#pragma unroll
                for (int c = 0; c < 9; ++c) {
                    const double v = B[base + c * step];
                    b[j][c] = a.s32 ? (double)(float)v : v;
                }
                if (comp == 0) slc[sg + j] = (int16_t)find_col(scol, nc, a.sf_col[e]);
                n_own = j + 1;
            }
        }
    }
    double x = 0.0, r = 0.0, z = 0.0, q = 0.0, d = 0.0;
    if (own) { x = a.x[o]; r = a.r[o]; z = a.z[o]; }
    for (int u = tid; u < nc * 9; u += BS) zs[u / 9][u % 9] = a.z[(int64_t)scol[u / 9] * 9 + u % 9];
    if (live)
        for (int u = lane; u < 81; u += kWave) sM[wave][u] = a.M[(int64_t)row * 81 + u];
    // a sum over partials p(i), i < n: thread i < 256 adds i, i + 256, ..., then
    // the tree of its wave, then the four waves in order (sum_partials)
    auto over_waves = [&](int j) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) t += sq[j * 4 + w];
        return t;
    };
    if (wave < 4)
        for (int j = 0; j < 2; ++j) {
            double s = 0.0;
            for (int i = tid; i < a.n_part; i += 256) s += a.pR[(int64_t)i * NP + j];
            s = wave_sum(s);
            if (lane == 0) sq[j * 4 + wave] = s;
        }
    __syncthreads();
    double rz = over_waves(0), rr = over_waves(1), rz_old = 1.0;
    const double r0sq = rr;
    // words of partial i of sum j (0: d^T q, 1: r^T z, 2: r^T r)
    auto slot = [&](int rep, int j, int i) { return (unsigned)(((rep * 3 + j) * 2 * 2 * kMaxG) + i) * 8u; };
    u64* const hi_slots = a.slots + 2 * kMaxG;
    // the values of two words, polled together
    auto poll = [&](const u64* lo0, const u64* hi0, unsigned at0, const u64* lo1, const u64* hi1, unsigned at1, unsigned ep,
                    double& v0, double& v1) {
        int spin = 0;
        for (;;) {
            const u64 w[4] = {peek(lo0, at0), peek(hi0, at0), peek(lo1, at1), peek(hi1, at1)};
            v0 = join(w[0], w[1]);
            v1 = join(w[2], w[3]);
            if ((unsigned)(w[0] >> 32) == ep && (unsigned)(w[1] >> 32) == ep && (unsigned)(w[2] >> 32) == ep &&
                (unsigned)(w[3] >> 32) == ep)
                return;
            if (++spin > kSpin) { s_bad = 1; return; }
        }
    };
    const int myrep = wg % kRep;
    // places of this thread's first two values of z
    auto place = [&](int u) { return (unsigned)(scol[u / 9] * 9 + u % 9) * 8u; };
    const bool two = tid + BS < nc * 9;
    unsigned p0 = 0, p1 = 0;
    if (tid < nc * 9) {
        p0 = place(tid);
        p1 = two ? place(tid + BS) : p0;
    }
    unsigned step = 0;   // numbers the words of an iteration
    int k = 0;
    bool fine = true;
    __syncthreads();
    for (;;) {
        // S z
        double y = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j < n_own) {
                const double* v = zs[slc[sg + j]];
#pragma unroll
                for (int c = 0; c < 9; ++c) y += b[j][c] * v[c];
            }
        if (grp < GRPW) part[wave][grp][comp] = y;
        wave_lds_sync();
        double s = 0.0;
        if (own) {
            s = part[wave][0][comp];
#pragma unroll
            for (int g = 1; g < GRPW; ++g) s += part[wave][g][comp];
        }
        if (k > 0) {
            if (wave < 4) {   // n_b <= 74
                double t0 = 0.0, t1 = 0.0;
                if (tid < n_b) {
                    double v0, v1;
                    poll(a.slots, hi_slots, slot(myrep, 1, tid), a.slots, hi_slots, slot(myrep, 2, tid), step, v0, v1);
                    t0 += v0;
                    t1 += v1;
                }
                t0 = wave_sum(t0);
                t1 = wave_sum(t1);
                if (lane == 0) { sq[wave] = t0; sq[4 + wave] = t1; }
            }
            __syncthreads();
            if (s_bad) { fine = false; break; }
            rz_old = rz;
            rz = over_waves(0);
            rr = over_waves(1);
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
        q = k == 0 ? s : s + beta * q;
        d = k == 0 ? z : z + beta * d;
        ++step;
        double dqr = 0.0;
        if (own) dqr += d * q;
        dqr = wave_sum(dqr);
        if (lane == 0) sh[0][wave] = dqr;
        __syncthreads();   // also: every wave has read sq
        if (tid < 2 * kRep) {
            const int h = tid % 2, i = wg * 2 + h;
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) t += sh[0][h * 4 + w];
            if (i < n_a) put(a.slots, hi_slots, slot(tid / 2, 0, i), t, step);
        }
        if (wave < 4) {
            double t = 0.0;
            if (tid < n_a) {   // n_a <= 512
                double v0, v1;
                poll(a.slots, hi_slots, slot(myrep, 0, tid), a.slots, hi_slots,
                     slot(myrep, 0, tid + 256 < n_a ? tid + 256 : tid), step, v0, v1);
                t += v0;
                if (tid + 256 < n_a) t += v1;
            }
            t = wave_sum(t);
            if (lane == 0) sq[wave] = t;
        }
        __syncthreads();
        if (s_bad) { fine = false; break; }
        const double dq = over_waves(0);
        if (!(dq > 0.0)) {
            if (wg == 0 && tid == 0) { a.state[0] = 1; a.state[2] = BA_ERR_NOT_SPD; a.state[3] = k; }
            break;
        }
        const double alpha = rz / dq;
        x += alpha * d;
        r -= alpha * q;
        if (own) {
            sr[wave][comp] = r;
            put(a.rlo, a.rhi, (unsigned)o * 8u, r, step);
        }
        wave_lds_sync();
        if (own) {
            double t = 0.0;
#pragma unroll
            for (int c = 0; c < 9; ++c) t += sM[wave][comp * 9 + c] * sr[wave][c];
            z = t;
            put(a.zlo, a.zhi, (unsigned)o * 8u, z, step);
        }
        // the second sum's partials whose first row this workgroup owns (at most one)
        const int pb = (wg * kOrdRows + kOrdB - 1) / kOrdB;
        if (pb < n_b && pb * kOrdB < (wg + 1) * kOrdRows) {
            if (wave < 4) {
                const int at = pb * kOrdB * 9 + tid;
                const bool act = tid < kOrdB * 9 && at < n_rows * 9;
                double s0 = 0.0, s1 = 0.0;
                if (act) {
                    double zt, rt;
                    poll(a.zlo, a.zhi, (unsigned)at * 8u, a.rlo, a.rhi, (unsigned)at * 8u, step, zt, rt);
                    s0 += rt * zt;
                    s1 += rt * rt;
                }
                s0 = wave_sum(s0);
                s1 = wave_sum(s1);
                if (lane == 0) { sh[0][4 + wave] = s0; sh[1][4 + wave] = s1; }
            }
            __syncthreads();
            if (tid < 2 * kRep) {
                const int j = tid % 2;
                double t = 0.0;
#pragma unroll
                for (int w = 0; w < 4; ++w) t += sh[j][4 + w];
                put(a.slots, hi_slots, slot(tid / 2, 1 + j, pb), t, step);
            }
        }
        double v0, v1;
        if (tid < nc * 9) {
            poll(a.zlo, a.zhi, p0, a.zlo, a.zhi, p1, step, v0, v1);
            (&zs[0][0])[tid] = v0;
            if (two) (&zs[0][0])[tid + BS] = v1;
        }
#pragma unroll 1
        for (int u = tid + 2 * BS; u < nc * 9; u += 2 * BS) {   // more than 113 columns
            const int u1 = u + BS < nc * 9 ? u + BS : u;
            poll(a.zlo, a.zhi, place(u), a.zlo, a.zhi, place(u1), step, v0, v1);
            (&zs[0][0])[u] = v0;
            (&zs[0][0])[u1] = v1;
        }
        __syncthreads();
        if (s_bad) { fine = false; break; }
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
// contiguous rows per workgroup, NB blocks per lane group, at most one
// workgroup per CU; a system that fits one workgroup takes one (its sums need
// no exchange).  G = 0: the system does not fit.
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
    // One workgroup where it holds all rows, with the fewest blocks a lane group
    // that do.  Else as few workgroups as the product leaves cheap: a sum's and
    // an exchange's latency grows with the workgroups whose words are polled,
    // the product's time with the blocks a group, steeply from 11 (spills) on.
    // Least blocks a group 1, 2, 4, 6, 8: 100 cameras 5.88, 4.95, 4.80, 4.74,
    // 5.01 us an iteration; 300 cameras 6.13, 6.13, 5.25, 5.06, 5.28; 500
    // cameras of a partition 6.71, 6.71, 6.23, 5.85, 5.94; 700 cameras 6.03,
    // 6.03, 6.02, 5.72, 5.53; 84 rows of shared intrinsics 5.26, 5.26, 5.03,
    // 4.90, 5.15; 300 cameras, FSAI 12.0, 11.9, 11.0, 10.9, 12.8.
    // The largest that fit, 3,510 cameras with 132,800 entries and 11 blocks a
    // group: 9.5 us, FSAI with deflation 29.7, against 27.7 and 44.6 with one
    // kernel per phase: the spills cost less than the launches and reads of S.
    for (int one = 1; one >= 0 && P.NB == 0; --one)
        for (int nb : {1, 2, 4, 6, 8, kMaxNB})
            if ((one || nb >= 6) && cut(nb, brow) && (!one || brow.size() == 2)) {
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

// The plan of the solve in the other kernels' order: eight rows a workgroup,
// their entries dealt to seven lane groups a row.  G = 0: it does not fit.
void plan_chip_ordered(int n_rows, const int32_t* sf_ptr, const int32_t* sf_col, int n_cu, ChipPlan& P) {
    P = ChipPlan();
    int most = 0;
    for (int r = 0; r < n_rows; ++r) most = std::max(most, sf_ptr[r + 1] - sf_ptr[r]);
    const int G = (n_rows + kOrdRows - 1) / kOrdRows;
    if (n_rows <= 0 || G > std::min(kMaxG, n_cu) || most > GRPW * kMaxNB) return;
    P.G = G;
    for (int nb : {kMaxNB, 8, 6, 4})
        if (most <= GRPW * nb) P.NB = nb;
    P.cptr.assign(1, 0);
    std::vector<int32_t> seen(n_rows, -1);
    for (int g = 0; g < G; ++g) {
        const size_t c0 = P.cols.size();
        for (int32_t e = sf_ptr[g * kOrdRows]; e < sf_ptr[std::min(n_rows, (g + 1) * kOrdRows)]; ++e)
            if (seen[sf_col[e]] != g) {
                seen[sf_col[e]] = g;
                P.cols.push_back(sf_col[e]);
            }
        std::sort(P.cols.begin() + c0, P.cols.end());
        P.cptr.push_back((int32_t)P.cols.size());
    }
}

bool launch_chip_ordered(ba_ctx* c, const double* M, int n_part, double tol, int max_iter, double* out) {
    const Chip& H = c->chip_ord;
    const Pcg& P = c->pcg;
    ChipArgs a{};
    a.max_iter = max_iter; a.n_part = n_part; a.s32 = c->s32; a.tol = tol;
    a.cptr = H.cptr; a.cols = H.cols;
    a.sf_ptr = c->sf_ptr; a.sf_col = c->sf_col; a.sf_src = c->sf_src;
    a.blk = c->blk; a.M = M;
    a.x = P.x; a.r = P.r[0]; a.z = P.z; a.pR = P.pR;
    a.out = out; a.state = P.state; a.scal = P.scal; a.stamp = c->h_stamp + kStBack;
    a.zlo = (u64*)P.u; a.zhi = (u64*)P.q; a.rlo = (u64*)P.d; a.rhi = (u64*)P.r[1]; a.slots = (u64*)P.pE;
    const void* k = H.NB == 4   ? (const void*)k_pcg_ord<4>
                    : H.NB == 6 ? (const void*)k_pcg_ord<6>
                    : H.NB == 8 ? (const void*)k_pcg_ord<8>
                                : (const void*)k_pcg_ord<kMaxNB>;
    int n_rows = c->n_rows;
    void* args[] = {&n_rows, &a};
    const hipError_t e = H.G == 1 ? hipLaunchKernel(k, dim3(1), dim3(BS), args, 0, c->stream)
                                  : hipLaunchCooperativeKernel(k, dim3(H.G), dim3(BS), args, 0, c->stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

// Words that the set-up clears for launch_chip
int64_t chip_slot_words() { return (int64_t)2 * kRep * NP * 2 * kMaxG; }
static_assert(kRep * 3 * 4 * kMaxG <= 2 * kRep * NP * 2 * kMaxG, "the ordered solve's words are among them");

}  // namespace ba
