// Reduced-camera-system formation (Eq. (3)-(4), Sec. 5) and point
// back-substitution (Eq. (5)).
//
// With V*_p = L_p L_p^T (3x3 Cholesky) and K_a = J_pa L_p^-T (2x3) for an
// observation a of point p by camera i:
//   W_ip V*_p^-1 W_jp^T = J_ca^T (K_a K_b^T) J_cb          (camera pair i, j)
//   U_i - sum_p W_ip V*_p^-1 W_ip^T = sum_a J_ca^T (I - K_a K_a^T) J_ca
//   b_i = l_c - W V*^-1 l_p = -sum_a J_ca^T (e_a + K_a lhat_p),  lhat_p = L_p^-1 l_p
//   dx_p = L_p^-T (lhat_p - sum_a K_a^T J_ca dx_c)          (Eq. (5))
// so the point stage only adds K (6 values) to each observation's J_c record
// and every later stage reads one 24-value record per observation.  The
// off-diagonal blocks are segmented reductions over the observation couples
// of each camera pair (sorted once, no atomics); the diagonal blocks are
// reductions over each camera's observations.
#include <type_traits>

#include "ba_common.hpp"

namespace ba {

namespace {

constexpr int BS = 256;
constexpr int WPB = BS / kWave;   // waves per block

// Point terms from the track sums s = (V: 00 01 02 11 12 22, l_p): the
// Cholesky factor of V* = V + lambda diag(V), lhat = L^-1 l_p and the
// reciprocals of L's diagonal, r = (L00, L10, L11, L20, L21, L22, lhat,
// 1/L00, 1/L11, 1/L22).  Returns false if V* is not positive definite.
constexpr int kPT = 12;   // point terms shared with a track's lanes
constexpr int kPTRow = kPT + 1;   // a lane's row in LDS: an odd number of values, so that the lanes' rows spread over the banks
__device__ __forceinline__ bool point_terms(const double* s, double lambda, double* r) {
    const double V00 = s[0] * (1.0 + lambda), V11 = s[3] * (1.0 + lambda), V22 = s[5] * (1.0 + lambda);
    const double L00 = sqrt(V00), i00 = 1.0 / L00;
    const double L10 = s[1] * i00, L20 = s[2] * i00;
    const double d1 = V11 - L10 * L10;
    const double L11 = sqrt(d1), i11 = 1.0 / L11;
    const double L21 = (s[4] - L20 * L10) * i11;
    const double d2 = V22 - L20 * L20 - L21 * L21;
    const double L22 = sqrt(d2), i22 = 1.0 / L22;
    const double y0 = s[6] * i00;
    const double y1 = (s[7] - L10 * y0) * i11;
    const double y2 = (s[8] - L20 * y0 - L21 * y1) * i22;
    r[0] = L00; r[1] = L10; r[2] = L11; r[3] = L20; r[4] = L21; r[5] = L22;
    r[6] = y0; r[7] = y1; r[8] = y2; r[9] = i00; r[10] = i11; r[11] = i22;
    return V00 > 0.0 && d1 > 0.0 && d2 > 0.0;
}

// K = J_p L^-T from the point terms r: row r of K solves L y = J_p[r]^T.
__device__ __forceinline__ void point_K(const double* r, const double* jp, double* K) {
    const double L10 = r[1], L20 = r[3], L21 = r[4], i00 = r[9], i11 = r[10], i22 = r[11];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        const double y0 = jp[3 * rr] * i00;
        const double y1 = (jp[3 * rr + 1] - L10 * y0) * i11;
        const double y2 = (jp[3 * rr + 2] - L20 * y0 - L21 * y1) * i22;
        K[3 * rr] = y0; K[3 * rr + 1] = y1; K[3 * rr + 2] = y2;
    }
}

// ebar = e + K lhat, with K as stored (T), at the observation's position in
// its camera's list (rpos < 0: fixed camera, no RCS row).  The diagonal
// stage reads it in that order instead of gathering e and lhat.
template <typename T>
__device__ __forceinline__ void store_ebar(const double* r, const double* K, double eu, double ev, int rpos,
                                           double* __restrict__ ebar) {
    if (rpos < 0) return;
    double Kt[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) Kt[m] = (double)(T)K[m];
    const double v0 = eu + Kt[0] * r[6] + Kt[1] * r[7] + Kt[2] * r[8];
    const double v1 = ev + Kt[3] * r[6] + Kt[4] * r[7] + Kt[5] * r[8];
    reinterpret_cast<double2*>(ebar)[rpos] = make_double2(v0, v1);
}

// ---------------------------------------------------------------------------
// point stage: one wave per chunk of whole tracks (<= 64 observations), one
// lane per observation.  Track sums V_p, l_p are reduced through LDS by the
// lane holding the first observation of the track.  The waves of a workgroup
// share nothing and do not wait for each other.  Bound by memory: K goes to
// the last 48 of each record's 192 bytes, so every line is written in parts
// (25 M observations, FP64: 1.9 GB read and 2.6 GB written in 1,772 us; 1,806
// with each lane writing its K, 1,880 without the XCD-contiguous order).
// ---------------------------------------------------------------------------
// FROM_K: J_p is not stored; it is formed as K L^T from the record and the
// point terms of the previous formation (read before they are replaced),
// rounded to T and stored in Jp, so that later formations of the same
// linearization read it instead of forming it again.
template <typename T, bool FROM_K = false>
__global__ __launch_bounds__(BS) void k_point(int n_chunk, const int32_t* __restrict__ chunk_ptr,
                                              const int32_t* __restrict__ obs_pt, const int32_t* __restrict__ chunk_q,
                                              T* __restrict__ R, T* __restrict__ Jp, const double* __restrict__ e,
                                              double lambda, double* __restrict__ ptL, const int32_t* __restrict__ obs_rpos,
                                              double* __restrict__ ebar, int* __restrict__ flags) {
    __shared__ __align__(16) double sP[WPB][kWave][kPTRow];   // track sums, the head's point terms, then K
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int chunk = xcd_block() * WPB + wv;
    int k0 = 0, k1 = 0;
    if (chunk < n_chunk) { k0 = chunk_ptr[chunk]; k1 = chunk_ptr[chunk + 1]; }
    const int k = k0 + lane;
    const bool act = k < k1;
    double jp[6];
    double2 ek = make_double2(0.0, 0.0);
    int rpos = -1;
    const int p = act ? obs_pt[k] : -1;
    const Track tk = chunk_track(act, p, lane, k1 - k0);
    const int head = tk.head, tl = tk.len;
    const int64_t q = chunk < n_chunk ? (int64_t)chunk_q[chunk] + tk.idx : 0;   // internal point index
    if (act) {
        if (FROM_K) {
            double K[6];
            load6(R + (int64_t)k * kRec + 18, K);
            jp_from_K(K, ptL + q * 9, jp);
#pragma unroll
            for (int m = 0; m < 6; ++m) jp[m] = (double)(T)jp[m];
            store6(Jp + (int64_t)k * 6, jp);
        } else {
            load6(Jp + (int64_t)k * 6, jp);
        }
        ek = reinterpret_cast<const double2*>(e)[k];
        rpos = obs_rpos[k];
        sP[wv][lane][0] = jp[0] * jp[0] + jp[3] * jp[3];
        sP[wv][lane][1] = jp[0] * jp[1] + jp[3] * jp[4];
        sP[wv][lane][2] = jp[0] * jp[2] + jp[3] * jp[5];
        sP[wv][lane][3] = jp[1] * jp[1] + jp[4] * jp[4];
        sP[wv][lane][4] = jp[1] * jp[2] + jp[4] * jp[5];
        sP[wv][lane][5] = jp[2] * jp[2] + jp[5] * jp[5];
        sP[wv][lane][6] = -(jp[0] * ek.x + jp[3] * ek.y);
        sP[wv][lane][7] = -(jp[1] * ek.x + jp[4] * ek.y);
        sP[wv][lane][8] = -(jp[2] * ek.x + jp[5] * ek.y);
    }
    wave_lds_sync();
    if (act && head == lane) {
        double s[9];
#pragma unroll
        for (int m = 0; m < 9; ++m) s[m] = 0.0;
        for (int q = 0; q < tl; ++q)
#pragma unroll
            for (int m = 0; m < 9; ++m) s[m] += sP[wv][lane + q][m];
        double r[kPT];
        if (!point_terms(s, lambda, r)) flags[0] = 1;
        // the head's own row is read by no other lane: it holds the track's terms now
#pragma unroll
        for (int m = 0; m < kPT; ++m) sP[wv][lane][m] = r[m];
#pragma unroll
        for (int m = 0; m < 9; ++m) ptL[q * 9 + m] = r[m];
    }
    wave_lds_sync();
    double K[6];
    if (act) {
        point_K(sP[wv][head], jp, K);
        store_ebar<T>(sP[wv][head], K, ek.x, ek.y, rpos, ebar);
    }
    wave_lds_sync();   // every lane has its point terms
    T* stage = reinterpret_cast<T*>(&sP[wv][0][0]);
    if (act) store6(stage + lane * 6, K);
    wave_lds_sync();
    // K into the records: neighbouring lanes write neighbouring 16 (FP32: 8) bytes
    using V = typename std::conditional<sizeof(T) == 8, uint4, uint2>::type;
    constexpr int kV = (int)(sizeof(V) / sizeof(T));
    for (int i = lane; i < 3 * (k1 - k0); i += kWave)
        *reinterpret_cast<V*>(R + (int64_t)(k0 + i / 3) * kRec + 18 + (i % 3) * kV) =
            reinterpret_cast<const V*>(stage)[i];
}

// ---------------------------------------------------------------------------
// linearization fused with the point stage (the LM step after an accepted
// step): one wave per chunk of whole tracks, one lane per observation.  Each
// lane forms its residual and Jacobian blocks (Eq. (1)); J_c and J_p are
// rounded to T first, so the records, point terms and e + K lhat equal
// those of k_linearize followed by k_point.  J_p itself is not stored: it
// is K L^T wherever it is needed.  The track sums go through LDS as in
// k_point, and the records are written whole through LDS (below).
// ---------------------------------------------------------------------------
// Waves per workgroup of the fused stage: one, so that its barriers hold a
// single wave (on the 60,000-camera partition, FP64, measured against four
// waves on the same GPU: 7.01 against 7.29 ms, and 7.82 against 7.97 ms on
// another; two waves 7.09 ms).  Its chunks go to the XCDs in contiguous
// ranges (7.56 against 7.80 ms): a chunk boundary splits lines of the
// observation arrays, which the neighbouring chunk then finds in L2.
constexpr int kLinNW = 1;

template <typename T, int NW>
__device__ __forceinline__ void linpoint(int n_chunk, const int32_t* __restrict__ chunk_ptr, int n,
                                                 const int32_t* __restrict__ obs_cam,
                                                 const int32_t* __restrict__ obs_pt,
                                                 const int32_t* __restrict__ chunk_q, const double* __restrict__ uv,
                                                 const double* __restrict__ cams, const double* __restrict__ pts,
                                                 double lambda, T* __restrict__ R,
                                                 double* __restrict__ e, double* __restrict__ ptL,
                                                 const int32_t* __restrict__ obs_rpos, double* __restrict__ ebar,
                                                 double* __restrict__ part, int* __restrict__ flags) {
    constexpr int kRecB = kRec * (int)sizeof(T), kPadB = kRecB + 16;   // a staged record's stride: over all banks
    constexpr int kPer = sizeof(T) == 8 ? 32 : kWave;                  // records per round
    // track sums, the head's point terms, then staging
    __shared__ __align__(16) char sS[NW][kPer * kPadB];
    static_assert(kPer * kPadB >= kWave * kPTRow * (int)sizeof(double), "both uses fit");
    __shared__ double sh[NW];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    double (*sP)[kPTRow] = reinterpret_cast<double (*)[kPTRow]>(sS[wv]);
    const int chunk = xcd_block() * NW + wv;   // neighbouring chunks on one XCD
    int k0 = 0, k1 = 0;
    if (chunk < n_chunk) { k0 = chunk_ptr[chunk]; k1 = chunk_ptr[chunk + 1]; }
    const int k = k0 + lane;
    const bool act = k < k1;
    double jc[18], jp[6];
    double cost = 0.0, eu = 0.0, ev = 0.0;
    int rpos = -1;
    const int p = act ? obs_pt[k] : -1;
    const Track tk = chunk_track(act, p, lane, k1 - k0);
    const int head = tk.head, tl = tk.len;
    const int64_t q = chunk < n_chunk ? (int64_t)chunk_q[chunk] + tk.idx : 0;   // internal point index
    if (act) {
        const double* X = pts + (int64_t)p * 3;
        rpos = obs_rpos[k];
        double pu, pv;
        project_point<true>(cams + (int64_t)obs_cam[k] * 9, X[0], X[1], X[2], pu, pv, jc, jp);
        eu = pu - uv[k];
        ev = pv - uv[n + k];
        if (!records_in_range<T>(jc, jp, eu, ev)) flags[2] = 1;
#pragma unroll
        for (int m = 0; m < 18; ++m) jc[m] = (double)(T)jc[m];
#pragma unroll
        for (int m = 0; m < 6; ++m) jp[m] = (double)(T)jp[m];
        reinterpret_cast<double2*>(e)[k] = make_double2(eu, ev);
        cost = 0.5 * (eu * eu + ev * ev);
        sP[lane][0] = jp[0] * jp[0] + jp[3] * jp[3];
        sP[lane][1] = jp[0] * jp[1] + jp[3] * jp[4];
        sP[lane][2] = jp[0] * jp[2] + jp[3] * jp[5];
        sP[lane][3] = jp[1] * jp[1] + jp[4] * jp[4];
        sP[lane][4] = jp[1] * jp[2] + jp[4] * jp[5];
        sP[lane][5] = jp[2] * jp[2] + jp[5] * jp[5];
        sP[lane][6] = -(jp[0] * eu + jp[3] * ev);
        sP[lane][7] = -(jp[1] * eu + jp[4] * ev);
        sP[lane][8] = -(jp[2] * eu + jp[5] * ev);
    }
    const double csum = block_sum<NW * kWave>(cost, sh);   // contains the barrier for sP
    if (threadIdx.x == 0) part[blockIdx.x] = csum;
    if (act && head == lane) {
        double s[9];
#pragma unroll
        for (int m = 0; m < 9; ++m) s[m] = 0.0;
        for (int q = 0; q < tl; ++q)
#pragma unroll
            for (int m = 0; m < 9; ++m) s[m] += sP[lane + q][m];
        double r[kPT];
        if (!point_terms(s, lambda, r)) flags[0] = 1;
        // the head's own row is read by no other lane: it holds the track's terms now
#pragma unroll
        for (int m = 0; m < kPT; ++m) sP[lane][m] = r[m];
#pragma unroll
        for (int m = 0; m < 9; ++m) ptL[q * 9 + m] = r[m];
    }
    __syncthreads();
    double K[6];
    if (act) {
        point_K(sP[head], jp, K);
        store_ebar<T>(sP[head], K, eu, ev, rpos, ebar);
    }
    __syncthreads();   // every lane has its point terms: sP is free for staging
    // The wave's records (J_c, K) are contiguous in memory; they are staged
    // through the wave's part of LDS and written with contiguous 16-byte
    // chunks spread over the lanes, instead of each lane writing its own
    // record at a 192-byte (96-byte) stride.
    char* stage = sS[wv];
    const int nrec = k1 - k0;
#pragma unroll
    for (int r0 = 0; r0 < kWave; r0 += kPer) {
        if (act && lane >= r0 && lane < r0 + kPer) {
            T* d = reinterpret_cast<T*>(stage + (lane - r0) * kPadB);
            store_jc(d, jc);
            store6(d + 18, K);
        }
        __syncthreads();
        wave_records_out<kRecB, kPadB>(reinterpret_cast<char*>(R + (int64_t)(k0 + r0) * kRec), stage,
                                       min(nrec - r0, kPer), lane);
        __syncthreads();
    }
}

// FP32 records: 96 registers allow five waves per SIMD without spilling;
// the FP64 build keeps the default (it would spill).
__global__ __launch_bounds__(kLinNW * kWave) __attribute__((amdgpu_waves_per_eu(5))) void k_linpoint_f(int n_chunk, const int32_t* __restrict__ chunk_ptr, int n,
                                                 const int32_t* __restrict__ obs_cam,
                                                 const int32_t* __restrict__ obs_pt,
                                                 const int32_t* __restrict__ chunk_q, const double* __restrict__ uv,
                                                 const double* __restrict__ cams, const double* __restrict__ pts,
                                                 double lambda, float* __restrict__ R,
                                                 double* __restrict__ e, double* __restrict__ ptL,
                                                 const int32_t* __restrict__ obs_rpos, double* __restrict__ ebar,
                                                 double* __restrict__ part, int* __restrict__ flags) {
    linpoint<float, kLinNW>(n_chunk, chunk_ptr, n, obs_cam, obs_pt, chunk_q, uv, cams, pts, lambda, R, e, ptL, obs_rpos, ebar, part, flags);
}
__global__ __launch_bounds__(kLinNW * kWave) void k_linpoint_d(int n_chunk, const int32_t* __restrict__ chunk_ptr, int n,
                                                 const int32_t* __restrict__ obs_cam,
                                                 const int32_t* __restrict__ obs_pt,
                                                 const int32_t* __restrict__ chunk_q, const double* __restrict__ uv,
                                                 const double* __restrict__ cams, const double* __restrict__ pts,
                                                 double lambda, double* __restrict__ R,
                                                 double* __restrict__ e, double* __restrict__ ptL,
                                                 const int32_t* __restrict__ obs_rpos, double* __restrict__ ebar,
                                                 double* __restrict__ part, int* __restrict__ flags) {
    linpoint<double, kLinNW>(n_chunk, chunk_ptr, n, obs_cam, obs_pt, chunk_q, uv, cams, pts, lambda, R, e, ptL, obs_rpos, ebar, part, flags);
}

// ---------------------------------------------------------------------------
// off-diagonal pair stage.  One wave per workgroup, 16 lanes per camera pair
// = 4 couple slots x 4 column quarters ({0,1,2}, {3,4}, {5,6}, {7,8}); each
// lane accumulates the 9 rows of its columns of
//   S_ij -= J_ca^T (K_a K_b^T) J_cb
// over the couples of its slot, then the 4 slots are reduced by shuffles.
// A lane group works on one unit: a whole segment, or a piece of one whose
// partial block is summed by k_pair_sum.  A step covers the wave's 16
// couples; their two records are copied from global memory straight into LDS
// (16-byte lane copies that bypass the registers, spread over the whole wave,
// so every record is fetched once per step instead of once per lane of its
// couple).
//   What bounds it: the records' way from L2 and HBM, 384 (FP32: 192) bytes a
// couple, behind a latency of two microseconds under load.  So the copies of
// the next kBuf - 1 steps are in flight while a step is computed, from kBuf
// LDS buffers.  The buffers are separate arrays and the loop is unrolled by
// them: reads of one array of buffers made the compiler wait for every copy
// in flight before each step.  The couples' indices are read kBuf steps
// before their copies are issued, so that waiting for an index never waits
// for a younger copy, and the single wave needs no barrier.
//   Four neighbouring lanes copy the four 16-byte chunks of one 64-byte piece
// of a record (one address a cycle otherwise: 2,982 against 3,044 us, 207
// against 221 us below), and a couple's piece lies rotated by its lane group
// (chunk h at slot h ^ group), so that the wave's 16 couples read one value
// from 16 different bank quads.
//   Measured: 15,000 cameras, 57.6 M couples, FP64 3,500 -> 2,660 us with the
// tiles described where the units are built; 18,000 cameras, 42.4 M couples,
// FP32 records 1,707 -> 1,450 us; 2,000 cameras, 3.8 M couples, FP64 229 -> 207.
//   Units are stored by tiles or clusters of cameras (longest first inside
// each); workgroup b runs on XCD b mod 8, which takes the waves of its own
// contiguous range of units (ranges of equal work), keeping the records of
// neighbouring cameras in its L2.
// ---------------------------------------------------------------------------
constexpr int kPairWave = 4;   // units (camera pairs or pieces) per wave

struct XcdRanges { int wv[9]; };

// Buffers: two, which the FP64 instance's 6 KB each allow to 12 waves a CU
// (three a SIMD; asking for four makes the compiler spill).  FP64 with three
// buffers and 8 waves where units are long (kDeepSteps steps on average): 2,644
// against 2,815 us at 25 steps a unit, 218 against 207 at 10, where starting
// and reducing a unit weighs more than the copies' latency.  FP32: two and
// 12 waves (1,420 us) against three (1,454) and four (1,499).
constexpr int kDeepSteps = 16;

template <typename T, int kBuf, bool SUB = false>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(kBuf == 2 ? 3 : 2))) void k_offdiag(
    int n_unit, XcdRanges xr, const int32_t* __restrict__ unit_rng, const int32_t* __restrict__ unit_dst,
    const int32_t* __restrict__ trip, const T* __restrict__ R, double* __restrict__ blk, double* __restrict__ pblk,
    u64* stamp) {
    stamp_now(stamp);
    constexpr int kVal = 16 / sizeof(T);                             // values per 16-byte chunk
    constexpr int kCh = kRec / kVal;                                 // chunks per record (12 or 6)
    constexpr int kCpl = 4 * kPairWave;                              // couples per step
    constexpr int kLoads = kCpl * 2 * kCh / kWave;                   // chunk copies per lane per step
    static_assert(kCpl == 16 && kLoads * kWave == kCpl * 2 * kCh, "staging must tile the wave");
    static_assert(kBuf == 2 || kBuf == 3, "two or three buffers");
    constexpr int kBufV = kLoads * kWave * kVal;
    __shared__ __align__(16) T sC0[kBufV];
    __shared__ __align__(16) T sC1[kBufV];
    __shared__ __align__(16) T sC2[kBuf > 2 ? kBufV : 1];
    const int xcd = blockIdx.x % 8;
    const int wv = xr.wv[xcd] + (int)(blockIdx.x / 8);
    if (wv >= xr.wv[xcd + 1]) return;   // whole workgroup (one wave) leaves
    const int lane = threadIdx.x;
    const int grp = lane / 16, gl = lane % 16;
    const int slot = gl / 4, quarter = gl % 4;
    const int unit = wv * kPairWave + grp;
    const int cpl = grp * 4 + slot;                      // this lane's couple in a step
    const int c0 = quarter == 0 ? 0 : 2 * quarter + 1;   // 0, 3, 5, 7
    const int nc = quarter == 0 ? 3 : 2;
    const bool live = unit < n_unit;
    int t0 = 0, t1 = 0;
    if (live) { const int2 r = reinterpret_cast<const int2*>(unit_rng)[unit]; t0 = r.x; t1 = r.y; }
    int steps = (t1 - t0 + 3) / 4;
    steps = max(steps, __shfl_xor(steps, 16, kWave));
    steps = max(steps, __shfl_xor(steps, 32, kWave));
    steps = __builtin_amdgcn_readfirstlane(steps);
    // this lane's couple of step st (past the unit's end: its last one)
    auto couple = [&](int st) {
        return reinterpret_cast<const int2*>(trip)[max(0, min(t0 + 4 * st + slot, t1 - 1))];
    };
    // copy k of the wave fills its slots k * 64 .. k * 64 + 63: lane L moves
    // chunk 4 k + (L % 4 ^ L / 16) of couple L / 4, its own (chunks past kCh: the b record's)
    const int q4 = quarter ^ grp;
    auto issue = [&](T* dst, int2 ab) {
        const char* pa = reinterpret_cast<const char*>(R) + (int64_t)ab.x * (kRec * (int)sizeof(T));
        const char* pb = reinterpret_cast<const char*>(R) + (int64_t)ab.y * (kRec * (int)sizeof(T));
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int h = 4 * k + q4;
            const char* src = 4 * k + 3 < kCh ? pa + h * 16
                              : 4 * k >= kCh ? pb + (h - kCh) * 16
                                             : (h < kCh ? pa + h * 16 : pb + (h - kCh) * 16);
            __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)(dst + k * kWave * kVal),
                                             16, 0, 0);
        }
    };
    double acc[27];
#pragma unroll
    for (int m = 0; m < 27; ++m) acc[m] = 0.0;
    // One step: its records are in buf once at most the kBuf - 2 younger steps'
    // copies are in flight; those of step st + kBuf - 1 go to nbuf.  With three
    // buffers the copies past the last step (the units' last couples once
    // more) are issued too: leaving them out would leave the number in flight
    // open.
    int2 nx[kBuf];
    auto step = [&](const T* buf, T* nbuf, int2& nxt, int st) {
        __builtin_amdgcn_s_waitcnt(0x0f70 | ((kBuf - 2) * kLoads));   // vmcnt only
        if (kBuf > 2 || st + 1 < steps) {
            issue(nbuf, nxt);
            nxt = couple(st + 2 * kBuf - 1);
        }
        // value v of this lane's couple (v < kRec: record a, else record b)
        const T* me = buf + cpl * 4 * kVal;
        auto at = [&](int v) {
            const int h = v / kVal;
            return (double)me[(h / 4) * (kWave * kVal) + ((h % 4) ^ grp) * kVal + v % kVal];
        };
        const int t = t0 + 4 * st + slot;
        if (t < t1) {
            double ka[6], kb[6], jb0[3], jb1[3];
#pragma unroll
            for (int m = 0; m < 6; ++m) { ka[m] = at(18 + m); kb[m] = at(kRec + 18 + m); }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int c = c0 + (q < nc ? q : 0);
                jb0[q] = at(kRec + c);
                jb1[q] = at(kRec + 9 + c);
            }
            double m00 = ka[0] * kb[0] + ka[1] * kb[1] + ka[2] * kb[2];
            const double m01 = ka[0] * kb[3] + ka[1] * kb[4] + ka[2] * kb[5];
            const double m10 = ka[3] * kb[0] + ka[4] * kb[1] + ka[5] * kb[2];
            double m11 = ka[3] * kb[3] + ka[4] * kb[4] + ka[5] * kb[5];
            if (SUB) {
                const int2 ab = reinterpret_cast<const int2*>(trip)[t];
                if ((ab.x >> 1) == (ab.y >> 1)) { m00 -= 1.0; m11 -= 1.0; }
            }
            double p0[3], p1[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                p0[q] = m00 * jb0[q] + m01 * jb1[q];
                p1[q] = m10 * jb0[q] + m11 * jb1[q];
            }
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                const double a0 = at(r), a1 = at(9 + r);
#pragma unroll
                for (int q = 0; q < 3; ++q) acc[r * 3 + q] += a0 * p0[q] + a1 * p1[q];
            }
        }
    };
    {
        int2 first[kBuf - 1];
#pragma unroll
        for (int k = 0; k < kBuf - 1; ++k) first[k] = couple(k);
#pragma unroll
        for (int k = 0; k < kBuf; ++k) nx[k] = couple(kBuf - 1 + k);
        // these loads end here: left pending, the loop's first wait would be for everything
#pragma unroll
        for (int k = 0; k < kBuf; ++k) asm volatile("" : "+v"(nx[k].x), "+v"(nx[k].y));
        issue(sC0, first[0]);
        if constexpr (kBuf > 2) issue(sC1, first[1]);
    }
    for (int st = 0; st < steps; st += kBuf) {
        if constexpr (kBuf == 2) {
            step(sC0, sC1, nx[0], st);
            if (st + 1 < steps) step(sC1, sC0, nx[1], st + 1);
        } else {
            step(sC0, sC2, nx[0], st);
            step(sC1, sC0, nx[1], st + 1);
            step(sC2, sC1, nx[2], st + 2);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);   // no copy is on its way to LDS when the wave ends
#pragma unroll
    for (int m = 0; m < 27; ++m) {
        acc[m] += __shfl_xor(acc[m], 4, kWave);
        acc[m] += __shfl_xor(acc[m], 8, kWave);
    }
    if (live && slot == 0) {
        const int dst = unit_dst[unit];
        double* out = dst >= 0 ? blk + (int64_t)dst * 81 : pblk + (int64_t)(-dst - 1) * 81;
#pragma unroll
        for (int r = 0; r < 9; ++r)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (q < nc) out[r * 9 + c0 + q] = -acc[r * 3 + q];
    }
}

// Blocks of split segments: the sum of their chunks' partial blocks, in
// chunk order (one thread per block entry).
__global__ __launch_bounds__(BS) void k_pair_sum(int n_lseg, const int32_t* __restrict__ lseg_blk,
                                                 const int32_t* __restrict__ lseg_ptr,
                                                 const double* __restrict__ pblk, double* __restrict__ blk) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= (int64_t)n_lseg * 81) return;
    const int l = (int)(i / 81), e = (int)(i % 81);
    double v = 0.0;
    for (int p = lseg_ptr[l]; p < lseg_ptr[l + 1]; ++p) v += pblk[(int64_t)p * 81 + e];
    blk[(int64_t)lseg_blk[l] * 81 + e] = v;
}

// The same for the segments of many chunks (a physical camera's own block, the
// pairs of a landmark that most images see): a workgroup per segment, 12
// groups of 81 threads each summing a contiguous part of its chunks in order,
// then the groups in order.  With one thread walking all chunks the stage of
// an 80-image block with 4 physical cameras took 303 us in it, 15 now.
constexpr int kSumG = 12;
__global__ __launch_bounds__(1024) void k_pair_sum_long(const int32_t* __restrict__ lseg_blk,
                                                        const int32_t* __restrict__ lseg_ptr,
                                                        const double* __restrict__ pblk, double* __restrict__ blk) {
    __shared__ double sh[kSumG][81];
    const int l = blockIdx.x, g = threadIdx.x / 81, e = threadIdx.x % 81;
    const int p0 = lseg_ptr[l], n = lseg_ptr[l + 1] - p0, per = (n + kSumG - 1) / kSumG;
    if (g < kSumG) {
        const int a = p0 + min(n, g * per), b = p0 + min(n, (g + 1) * per);
        double v = 0.0;
        for (int p = a; p < b; p += 8) {
            double t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = pblk[(int64_t)min(p + i, b - 1) * 81 + e];
#pragma unroll
            for (int i = 0; i < 8; ++i) v += p + i < b ? t[i] : 0.0;
        }
        sh[g][e] = v;
    }
    __syncthreads();
    if (threadIdx.x < 81) {
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < kSumG; ++i) v += sh[i][e];
        blk[(int64_t)lseg_blk[l] * 81 + e] = v;
    }
}

// ---------------------------------------------------------------------------
// diagonal stage: one workgroup per RCS row over the camera's observations;
// S_ii = sum J_c^T (I - K K^T) J_c +
// lambda diag(U), U = sum J_c^T J_c, b_i = -sum J_c^T (e + K lhat), then the
// block-Jacobi inverse S_ii^-1 (Cholesky and triangular inverse).  A lane
// holds 63 FP64 sums, which allows two waves per SIMD: with a wave per row a
// CU works on eight rows at once, and while one lane of a wave factors its
// row's block the other waves keep loading.
// ---------------------------------------------------------------------------
// NW waves (one workgroup) share a row's observations.  One where the rows
// alone fill the chip, with barriers that hold a single wave (on the
// 60,000-camera partition, FP64: 4.37 against 4.51 ms with four rows a
// workgroup); four below kDiagRows rows, which leave most of the chip idle and
// whose time is a row's serial chain of gathers (300 cameras of 840
// observations: 24 against 31 us; 2,000 cameras: 96 against 90).
constexpr int kDiagRows = 1024;

template <typename T, int NW>
__global__ __launch_bounds__(NW * kWave) void k_diag(int n_rows, const int32_t* __restrict__ rowobs_ptr,
                                             const int32_t* __restrict__ rowobs, const int32_t* __restrict__ row_ptr,
                                             const T* __restrict__ R, const double* __restrict__ ebar, double lambda, double* __restrict__ blk, double* __restrict__ rhs,
                                             double* __restrict__ Minv, double* __restrict__ Linv,
                                             int* __restrict__ flags, u64* stamp) {
    stamp_now(stamp);
    __shared__ double sred[NW][64];
    __shared__ double S[81], sL[81], L[81];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int row = blockIdx.x;
    double A[64];   // the 45 unique values of the block, diag(U) (9), the right-hand side (9)
#pragma unroll
    for (int m = 0; m < 64; ++m) A[m] = 0.0;
    const int i0 = rowobs_ptr[row], i1 = rowobs_ptr[row + 1];
    for (int idx = i0 + threadIdx.x; idx < i1; idx += NW * kWave) {
        const int k = rowobs[idx];
        double jc[18], K[6];
        const T* rk = R + (int64_t)k * kRec;
        load_jc(rk, jc);
        load6(rk + 18, K);
        const double2 v = reinterpret_cast<const double2*>(ebar)[idx];   // e + K lhat
        const double n00 = 1.0 - (K[0] * K[0] + K[1] * K[1] + K[2] * K[2]);
        const double n01 = -(K[0] * K[3] + K[1] * K[4] + K[2] * K[5]);
        const double n11 = 1.0 - (K[3] * K[3] + K[4] * K[4] + K[5] * K[5]);
        const double v0 = v.x, v1 = v.y;
        double q0[9], q1[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) {
            q0[c] = n00 * jc[c] + n01 * jc[9 + c];
            q1[c] = n01 * jc[c] + n11 * jc[9 + c];
        }
        int m = 0;
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            A[45 + r] += jc[r] * jc[r] + jc[9 + r] * jc[9 + r];
            A[54 + r] -= jc[r] * v0 + jc[9 + r] * v1;
#pragma unroll
            for (int c = r; c < 9; ++c, ++m) A[m] += jc[r] * q0[c] + jc[9 + r] * q1[c];
        }
    }
    sred[wv][wave_sums64_at(lane)] = wave_sums64(A);   // the wave's 63 sums
    __syncthreads();
    auto total = [&](int m) {   // value m over the waves, in order
        double t = sred[0][m];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += sred[w][m];
        return t;
    };
    for (int e = threadIdx.x; e < 81; e += NW * kWave) {
        const int i = e / 9, j = e % 9;
        const int a = i < j ? i : j, b = i < j ? j : i;
        const int m = a * 9 - a * (a - 1) / 2 + (b - a);   // packed upper-triangle index
        double v = total(m);
        if (i == j) v += lambda * total(45 + i);
        S[e] = v;
        blk[(int64_t)row_ptr[row] * 81 + e] = v;
    }
    if (threadIdx.x < 9) rhs[(int64_t)row * 9 + threadIdx.x] = total(54 + threadIdx.x);
    __syncthreads();
    if (wv == 0 && !wave_factor9(S, sL, L, lane) && lane == 0) flags[1] = 1;
    __syncthreads();
    // S^-1 = L^-T L^-1: entry (i, j) = sum_{q >= max(i,j)} Li[q][i] Li[q][j]
    for (int e = threadIdx.x; e < 81; e += NW * kWave) {
        const int i = e / 9, j = e % 9;
        double t = 0.0;
        for (int q = (i > j ? i : j); q < 9; ++q) t += L[q * 9 + i] * L[q * 9 + j];
        Minv[(int64_t)row * 81 + e] = t;
        Linv[(int64_t)row * 81 + e] = L[e];
    }
}

// ---------------------------------------------------------------------------
// back-substitution (Eq. (5)): dx_p = L^-T (lhat - sum_a K_a^T J_ca dxc_a),
// and with it the model terms of the gain ratio, |J dx|^2 and dx^T l with
// l = -J^T e: the solve's right-hand side is w = L^T dx_p, so an
// observation's J dx = J_c dxc + K w with no J_p (J_p = K L^T).  One wave per
// chunk of whole tracks, one lane per observation; per-block partials of the
// two model terms.  Bound by reading the records; everything that needs only
// the chunk's place is asked for at once (25 M observations, FP64: 1,611 ->
// 1,590 us, 4.1 TB/s; 2.4 M: 94.7 -> 92.0).
// ---------------------------------------------------------------------------
// four waves per workgroup (on the 60,000-camera partition, FP64: 6.40 ms
// against 6.46 with two and 6.50 with one), blocks in XCD-contiguous order
// (6.31 against 6.39 ms)
constexpr int kBackNW = 4;

template <typename T>
__global__ __launch_bounds__(kBackNW * kWave) void k_backsub(int n_chunk, const int32_t* __restrict__ chunk_ptr,
                                                const int32_t* __restrict__ obs_pt, const int32_t* __restrict__ obs_row,
                                                const int32_t* __restrict__ chunk_q, const T* __restrict__ R,
                                                const double* __restrict__ ptL, const double* __restrict__ dxc,
                                                const double* __restrict__ e, double* __restrict__ dxp,
                                                double* __restrict__ part, int nb) {
    __shared__ double sP[kBackNW][kWave][3];
    __shared__ double sh[kBackNW];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int chunk = xcd_block() * kBackNW + wv;
    int k0 = 0, k1 = 0;
    if (chunk < n_chunk) { k0 = chunk_ptr[chunk]; k1 = chunk_ptr[chunk + 1]; }
    const int k = k0 + lane;
    const bool act = k < k1;
    const int p = act ? obs_pt[k] : -1;
    const Track tk = chunk_track(act, p, lane, k1 - k0);
    const int head = tk.head, tl = tk.len;
    const int64_t q = chunk < n_chunk ? (int64_t)chunk_q[chunk] + tk.idx : 0;   // internal point index
    double K[6], L[9], g0 = 0.0, g1 = 0.0;
    double2 ek;
    if (act && head == lane) {
#pragma unroll
        for (int m = 0; m < 9; ++m) L[m] = ptL[q * 9 + m];
    }
    if (act) {
        ek = reinterpret_cast<const double2*>(e)[k];
        const int row = obs_row[k];
        const T* rk = R + (int64_t)k * kRec;
        load6(rk + 18, K);
        if (row >= 0) {
            double jc[18];
            load_jc(rk, jc);
            const double* dc = dxc + (int64_t)row * 9;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const double c = dc[i];
                g0 += jc[i] * c;
                g1 += jc[9 + i] * c;
            }
        }
        sP[wv][lane][0] = K[0] * g0 + K[3] * g1;
        sP[wv][lane][1] = K[1] * g0 + K[4] * g1;
        sP[wv][lane][2] = K[2] * g0 + K[5] * g1;
    }
    wave_lds_sync();
    if (act && head == lane) {
        double u0 = 0.0, u1 = 0.0, u2 = 0.0;
        for (int q = 0; q < tl; ++q) { u0 += sP[wv][lane + q][0]; u1 += sP[wv][lane + q][1]; u2 += sP[wv][lane + q][2]; }
        u0 = L[6] - u0; u1 = L[7] - u1; u2 = L[8] - u2;
        // L^T x = u with L = [[L00,0,0],[L10,L11,0],[L20,L21,L22]]
        const double x2 = u2 / L[5];
        const double x1 = (u1 - L[4] * x2) / L[2];
        const double x0 = (u0 - L[1] * x1 - L[3] * x2) / L[0];
        dxp[(int64_t)p * 3 + 0] = x0;
        dxp[(int64_t)p * 3 + 1] = x1;
        dxp[(int64_t)p * 3 + 2] = x2;
        // the head's own row is read by no other lane now: w for the track
        sP[wv][lane][0] = u0; sP[wv][lane][1] = u1; sP[wv][lane][2] = u2;
    }
    wave_lds_sync();
    double jdx2 = 0.0, dxl = 0.0;
    if (act) {
        const double* w = sP[wv][head];
        const double a0 = g0 + K[0] * w[0] + K[1] * w[1] + K[2] * w[2];
        const double a1 = g1 + K[3] * w[0] + K[4] * w[1] + K[5] * w[2];
        jdx2 = a0 * a0 + a1 * a1;
        dxl = -(a0 * ek.x + a1 * ek.y);
    }
    const double s0 = block_sum<kBackNW * kWave>(jdx2, sh);
    const double s1 = block_sum<kBackNW * kWave>(dxl, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = s0;
        part[nb + blockIdx.x] = s1;
    }
}

// The model terms |J dx|^2 and dx^T l for a dx_p given from outside (after
// re-triangulation): J_p dx_p = K (L^T dx_p) with L from the point terms;
// same layout and partials as k_backsub
template <typename T>
__global__ __launch_bounds__(BS) void k_model_terms(int n_chunk, const int32_t* __restrict__ chunk_ptr,
                                                    const int32_t* __restrict__ obs_pt,
                                                    const int32_t* __restrict__ obs_row,
                                                    const int32_t* __restrict__ chunk_q, const T* __restrict__ R,
                                                    const double* __restrict__ ptL, const double* __restrict__ dxc,
                                                    const double* __restrict__ dxp, const double* __restrict__ e,
                                                    double* __restrict__ part, int nb) {
    __shared__ double sh[WPB];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int chunk = blockIdx.x * WPB + wv;
    int k0 = 0, k1 = 0;
    if (chunk < n_chunk) { k0 = chunk_ptr[chunk]; k1 = chunk_ptr[chunk + 1]; }
    const int k = k0 + lane;
    const bool act = k < k1;
    const int p = act ? obs_pt[k] : -1;
    const Track tk = chunk_track(act, p, lane, k1 - k0);
    const int64_t q = chunk < n_chunk ? (int64_t)chunk_q[chunk] + tk.idx : 0;
    double jdx2 = 0.0, dxl = 0.0;
    if (act) {
        const int row = obs_row[k];
        const T* rk = R + (int64_t)k * kRec;
        double K[6], g0 = 0.0, g1 = 0.0;
        load6(rk + 18, K);
        if (row >= 0) {
            double jc[18];
            load_jc(rk, jc);
            const double* dc = dxc + (int64_t)row * 9;
#pragma unroll
            for (int i = 0; i < 9; ++i) { g0 += jc[i] * dc[i]; g1 += jc[9 + i] * dc[i]; }
        }
        const double* L = ptL + q * 9;   // L00, L10, L11, L20, L21, L22
        const double* d = dxp + (int64_t)p * 3;
        const double w0 = L[0] * d[0] + L[1] * d[1] + L[3] * d[2];
        const double w1 = L[2] * d[1] + L[4] * d[2];
        const double w2 = L[5] * d[2];
        const double a0 = g0 + K[0] * w0 + K[1] * w1 + K[2] * w2;
        const double a1 = g1 + K[3] * w0 + K[4] * w1 + K[5] * w2;
        const double2 ek = reinterpret_cast<const double2*>(e)[k];
        jdx2 = a0 * a0 + a1 * a1;
        dxl = -(a0 * ek.x + a1 * ek.y);
    }
    const double s0 = block_sum<BS>(jdx2, sh);
    const double s1 = block_sum<BS>(dxl, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = s0;
        part[nb + blockIdx.x] = s1;
    }
}

// ---------------------------------------------------------------------------
// Tracks longer than a wave (more than 64 observations): one workgroup per
// point, its threads striding over the track; the track sums are reduced in
// a fixed order (each thread's strided sum, the wave's shuffle tree, then the
// four waves in order).  The arithmetic per observation is that of the wave
// kernels above.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void add_point_sums(const double* jp, double eu, double ev, double* v) {
    v[0] += jp[0] * jp[0] + jp[3] * jp[3];
    v[1] += jp[0] * jp[1] + jp[3] * jp[4];
    v[2] += jp[0] * jp[2] + jp[3] * jp[5];
    v[3] += jp[1] * jp[1] + jp[4] * jp[4];
    v[4] += jp[1] * jp[2] + jp[4] * jp[5];
    v[5] += jp[2] * jp[2] + jp[5] * jp[5];
    v[6] -= jp[0] * eu + jp[3] * ev;
    v[7] -= jp[1] * eu + jp[4] * ev;
    v[8] -= jp[2] * eu + jp[5] * ev;
}

// linearization fused with the point stage for point q0 + blockIdx.x (as
// linpoint: J_p is not stored, the second pass projects again for it);
// part[blockIdx.x] = the track's cost
template <typename T>
__global__ __launch_bounds__(BS) void k_linpoint_long(int q0, const int32_t* __restrict__ long_ptr, int n,
                                                      const int32_t* __restrict__ obs_cam,
                                                      const int32_t* __restrict__ obs_pt, const double* __restrict__ uv,
                                                      const double* __restrict__ cams, const double* __restrict__ pts,
                                                      double lambda, T* __restrict__ R, double* __restrict__ e,
                                                      double* __restrict__ ptL, const int32_t* __restrict__ obs_rpos,
                                                      double* __restrict__ ebar, double* __restrict__ part,
                                                      int* __restrict__ flags) {
    __shared__ double sh[10][WPB];
    __shared__ double sr[kPT];
    const int k0 = long_ptr[blockIdx.x], k1 = long_ptr[blockIdx.x + 1];
    const int64_t q = (int64_t)q0 + blockIdx.x;
    const int p = obs_pt[k0];
    const double X0 = pts[(int64_t)p * 3], X1 = pts[(int64_t)p * 3 + 1], X2 = pts[(int64_t)p * 3 + 2];
    double v[10];
#pragma unroll
    for (int m = 0; m < 10; ++m) v[m] = 0.0;
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        double jc[18], jp[6], pu, pv;
        project_point<true>(cams + (int64_t)obs_cam[k] * 9, X0, X1, X2, pu, pv, jc, jp);
        const double eu = pu - uv[k], ev = pv - uv[n + k];
        if (!records_in_range<T>(jc, jp, eu, ev)) flags[2] = 1;
#pragma unroll
        for (int m = 0; m < 18; ++m) jc[m] = (double)(T)jc[m];
#pragma unroll
        for (int m = 0; m < 6; ++m) jp[m] = (double)(T)jp[m];
        reinterpret_cast<double2*>(e)[k] = make_double2(eu, ev);
        store_jc(R + (int64_t)k * kRec, jc);
        add_point_sums(jp, eu, ev, v);
        v[9] += 0.5 * (eu * eu + ev * ev);
    }
    block_reduce<10>(v, sh);
    if (threadIdx.x == 0) {
        double r[kPT];
        if (!point_terms(v, lambda, r)) flags[0] = 1;
#pragma unroll
        for (int m = 0; m < kPT; ++m) sr[m] = r[m];
#pragma unroll
        for (int m = 0; m < 9; ++m) ptL[q * 9 + m] = r[m];
        part[blockIdx.x] = v[9];
    }
    __syncthreads();
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        double jp[6], pu, pv, K[6];
        project_point<true, false>(cams + (int64_t)obs_cam[k] * 9, X0, X1, X2, pu, pv, nullptr, jp);
#pragma unroll
        for (int m = 0; m < 6; ++m) jp[m] = (double)(T)jp[m];
        point_K(sr, jp, K);
        store6(R + (int64_t)k * kRec + 18, K);
        store_ebar<T>(sr, K, pu - uv[k], pv - uv[n + k], obs_rpos[k], ebar);
    }
}

// point stage (a new damping) for point q0 + blockIdx.x, as k_point
template <typename T, bool FROM_K>
__global__ __launch_bounds__(BS) void k_point_long(int q0, const int32_t* __restrict__ long_ptr, T* __restrict__ R,
                                                   T* __restrict__ Jp, const double* __restrict__ e, double lambda,
                                                   double* __restrict__ ptL, const int32_t* __restrict__ obs_rpos,
                                                   double* __restrict__ ebar, int* __restrict__ flags) {
    __shared__ double sh[9][WPB];
    __shared__ double sr[kPT];
    __shared__ double sL[6];   // the previous formation's factor (FROM_K)
    const int k0 = long_ptr[blockIdx.x], k1 = long_ptr[blockIdx.x + 1];
    const int64_t q = (int64_t)q0 + blockIdx.x;
    if (FROM_K && threadIdx.x < 6) sL[threadIdx.x] = ptL[q * 9 + threadIdx.x];
    __syncthreads();
    auto jp_of = [&](int k, double* jp) {
        if (FROM_K) {
            double K[6];
            load6(R + (int64_t)k * kRec + 18, K);
            jp_from_K(K, sL, jp);
#pragma unroll
            for (int m = 0; m < 6; ++m) jp[m] = (double)(T)jp[m];
        } else {
            load6(Jp + (int64_t)k * 6, jp);
        }
    };
    double v[9];
#pragma unroll
    for (int m = 0; m < 9; ++m) v[m] = 0.0;
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        double jp[6];
        jp_of(k, jp);
        if (FROM_K) store6(Jp + (int64_t)k * 6, jp);
        const double2 ek = reinterpret_cast<const double2*>(e)[k];
        add_point_sums(jp, ek.x, ek.y, v);
    }
    block_reduce<9>(v, sh);
    if (threadIdx.x == 0) {
        double r[kPT];
        if (!point_terms(v, lambda, r)) flags[0] = 1;
#pragma unroll
        for (int m = 0; m < kPT; ++m) sr[m] = r[m];
#pragma unroll
        for (int m = 0; m < 9; ++m) ptL[q * 9 + m] = r[m];
    }
    __syncthreads();
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        double jp[6], K[6];
        jp_of(k, jp);   // FROM_K: from the previous K, which this thread replaces only now
        const double2 ek = reinterpret_cast<const double2*>(e)[k];
        point_K(sr, jp, K);
        store6(R + (int64_t)k * kRec + 18, K);
        store_ebar<T>(sr, K, ek.x, ek.y, obs_rpos[k], ebar);
    }
}

// J_c dxc of observation k (0 for a fixed camera)
template <typename T>
__device__ __forceinline__ void jc_dxc(const T* __restrict__ rk, int row, const double* __restrict__ dxc, double& g0,
                                       double& g1) {
    g0 = 0.0; g1 = 0.0;
    if (row < 0) return;
    double jc[18];
    load_jc(rk, jc);
    const double* dc = dxc + (int64_t)row * 9;
#pragma unroll
    for (int i = 0; i < 9; ++i) { g0 += jc[i] * dc[i]; g1 += jc[9 + i] * dc[i]; }
}

// back-substitution and the model terms for point q0 + blockIdx.x, as
// k_backsub; part[blockIdx.x], part[stride + blockIdx.x]
template <typename T>
__global__ __launch_bounds__(BS) void k_backsub_long(int q0, const int32_t* __restrict__ long_ptr,
                                                     const int32_t* __restrict__ obs_pt,
                                                     const int32_t* __restrict__ obs_row, const T* __restrict__ R,
                                                     const double* __restrict__ ptL, const double* __restrict__ dxc,
                                                     const double* __restrict__ e, double* __restrict__ dxp,
                                                     double* __restrict__ part, int stride) {
    __shared__ double sh[3][WPB];
    __shared__ double su[3];
    const int k0 = long_ptr[blockIdx.x], k1 = long_ptr[blockIdx.x + 1];
    const int64_t q = (int64_t)q0 + blockIdx.x;
    const int p = obs_pt[k0];
    double v[3] = {0.0, 0.0, 0.0};
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        const T* rk = R + (int64_t)k * kRec;
        double K[6], g0, g1;
        load6(rk + 18, K);
        jc_dxc(rk, obs_row[k], dxc, g0, g1);
        v[0] += K[0] * g0 + K[3] * g1;
        v[1] += K[1] * g0 + K[4] * g1;
        v[2] += K[2] * g0 + K[5] * g1;
    }
    block_reduce<3>(v, sh);
    if (threadIdx.x == 0) {
        const double* L = ptL + q * 9;
        const double u0 = L[6] - v[0], u1 = L[7] - v[1], u2 = L[8] - v[2];
        const double x2 = u2 / L[5];
        const double x1 = (u1 - L[4] * x2) / L[2];
        const double x0 = (u0 - L[1] * x1 - L[3] * x2) / L[0];
        dxp[(int64_t)p * 3 + 0] = x0;
        dxp[(int64_t)p * 3 + 1] = x1;
        dxp[(int64_t)p * 3 + 2] = x2;
        su[0] = u0; su[1] = u1; su[2] = u2;
    }
    __syncthreads();
    double t[2] = {0.0, 0.0};
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        const T* rk = R + (int64_t)k * kRec;
        double K[6], g0, g1;
        load6(rk + 18, K);
        jc_dxc(rk, obs_row[k], dxc, g0, g1);
        const double a0 = g0 + K[0] * su[0] + K[1] * su[1] + K[2] * su[2];
        const double a1 = g1 + K[3] * su[0] + K[4] * su[1] + K[5] * su[2];
        const double2 ek = reinterpret_cast<const double2*>(e)[k];
        t[0] += a0 * a0 + a1 * a1;
        t[1] -= a0 * ek.x + a1 * ek.y;
    }
    block_reduce<2>(t, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = t[0];
        part[stride + blockIdx.x] = t[1];
    }
}

// the model terms for a given dx_p (after re-triangulation), as k_model_terms
template <typename T>
__global__ __launch_bounds__(BS) void k_model_terms_long(int q0, const int32_t* __restrict__ long_ptr,
                                                         const int32_t* __restrict__ obs_pt,
                                                         const int32_t* __restrict__ obs_row, const T* __restrict__ R,
                                                         const double* __restrict__ ptL, const double* __restrict__ dxc,
                                                         const double* __restrict__ dxp, const double* __restrict__ e,
                                                         double* __restrict__ part, int stride) {
    __shared__ double sh[2][WPB];
    const int k0 = long_ptr[blockIdx.x], k1 = long_ptr[blockIdx.x + 1];
    const int64_t q = (int64_t)q0 + blockIdx.x;
    const int p = obs_pt[k0];
    const double* L = ptL + q * 9;   // L00, L10, L11, L20, L21, L22
    const double* d = dxp + (int64_t)p * 3;
    const double w0 = L[0] * d[0] + L[1] * d[1] + L[3] * d[2];
    const double w1 = L[2] * d[1] + L[4] * d[2];
    const double w2 = L[5] * d[2];
    double t[2] = {0.0, 0.0};
    for (int k = k0 + threadIdx.x; k < k1; k += BS) {
        const T* rk = R + (int64_t)k * kRec;
        double K[6], g0, g1;
        load6(rk + 18, K);
        jc_dxc(rk, obs_row[k], dxc, g0, g1);
        const double a0 = g0 + K[0] * w0 + K[1] * w1 + K[2] * w2;
        const double a1 = g1 + K[3] * w0 + K[4] * w1 + K[5] * w2;
        const double2 ek = reinterpret_cast<const double2*>(e)[k];
        t[0] += a0 * a0 + a1 * a1;
        t[1] -= a0 * ek.x + a1 * ek.y;
    }
    block_reduce<2>(t, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = t[0];
        part[stride + blockIdx.x] = t[1];
    }
}

}  // namespace

template <typename T>
void launch_point_t(ba_ctx* c, double lambda) {
    const int nb = (c->n_chunk + WPB - 1) / WPB;
    T* R = (T*)c->R;
    T* Jp = (T*)c->Jp;
    if (nb > 0) {
        if (c->jp_valid)
            k_point<T><<<nb, BS, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, c->obs_pt, c->chunk_q, R, Jp, c->e, lambda,
                                                 c->ptL, c->obs_rpos, c->ebar, c->flags);
        else
            k_point<T, true><<<nb, BS, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, c->obs_pt, c->chunk_q, R, Jp, c->e,
                                                       lambda, c->ptL, c->obs_rpos, c->ebar, c->flags);
    }
    if (c->n_long > 0) {
        if (c->jp_valid)
            k_point_long<T, false><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, R, Jp, c->e, lambda,
                                                                    c->ptL, c->obs_rpos, c->ebar, c->flags);
        else
            k_point_long<T, true><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, R, Jp, c->e, lambda,
                                                                   c->ptL, c->obs_rpos, c->ebar, c->flags);
    }
}

void launch_point(ba_ctx* c, double lambda) {
    if (c->precision == BA_MIXED)
        launch_point_t<float>(c, lambda);
    else
        launch_point_t<double>(c, lambda);
    c->jp_valid = true;
}

void launch_linearize_point(ba_ctx* c, const double* cams, const double* pts, double lambda, u64* stamp) {
    const int nb = (c->n_chunk + kLinNW - 1) / kLinNW;
    const int n = (int)c->n_obs;
    if (nb + (int64_t)c->n_long > c->n_part)
        throw ba_hip_error(hipErrorInvalidValue, "cost partials exceed their buffer", __FILE__, __LINE__);
    if (nb > 0) {
        if (c->precision == BA_MIXED)
            k_linpoint_f<<<nb, kLinNW * kWave, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, n, c->obs_cam, c->obs_pt, c->chunk_q,
                                                   c->obs_uv, cams, pts, lambda, (float*)c->R, c->e, c->ptL,
                                                   c->obs_rpos, c->ebar, c->part, c->flags);
        else
            k_linpoint_d<<<nb, kLinNW * kWave, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, n, c->obs_cam, c->obs_pt, c->chunk_q,
                                                   c->obs_uv, cams, pts, lambda, (double*)c->R, c->e, c->ptL,
                                                   c->obs_rpos, c->ebar, c->part, c->flags);
    }
    if (c->n_long > 0) {
        if (c->precision == BA_MIXED)
            k_linpoint_long<float><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, n, c->obs_cam,
                                                                    c->obs_pt, c->obs_uv, cams, pts, lambda,
                                                                    (float*)c->R, c->e, c->ptL, c->obs_rpos,
                                                                    c->ebar, c->part + nb, c->flags);
        else
            k_linpoint_long<double><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, n, c->obs_cam,
                                                                     c->obs_pt, c->obs_uv, cams, pts, lambda,
                                                                     (double*)c->R, c->e, c->ptL, c->obs_rpos,
                                                                     c->ebar, c->part + nb, c->flags);
    }
    launch_reduce(c, c->part, nb + c->n_long, 1, c->scal + 0, stamp);
    c->jp_valid = false;   // J_p = K L^T where it is needed
}

void launch_offdiag(ba_ctx* c, u64* stamp) {
    if (c->n_unit == 0) {
        if (stamp) launch_stamp(c, (int)(stamp - c->h_stamp));
        return;
    }
    XcdRanges xr;
    int most = 0;
    for (int x = 0; x < 9; ++x) xr.wv[x] = c->xcd_wv[x];
    for (int x = 0; x < 8; ++x) most = std::max(most, xr.wv[x + 1] - xr.wv[x]);
    const int grid = 8 * most;
    if (c->shared)
        k_offdiag<double, 2, true><<<grid, kWave, 0, c->stream>>>(c->n_unit, xr, c->unit_rng, c->unit_dst, c->trip,
                                                                  (const double*)c->R, c->blk, c->pblk, stamp);
    else if (c->precision == BA_MIXED)
        k_offdiag<float, 2><<<grid, kWave, 0, c->stream>>>(c->n_unit, xr, c->unit_rng, c->unit_dst, c->trip,
                                                           (const float*)c->R, c->blk, c->pblk, stamp);
    else if (c->unit_steps >= (int64_t)kDeepSteps * c->n_unit)
        k_offdiag<double, 3><<<grid, kWave, 0, c->stream>>>(c->n_unit, xr, c->unit_rng, c->unit_dst, c->trip,
                                                            (const double*)c->R, c->blk, c->pblk, stamp);
    else
        k_offdiag<double, 2><<<grid, kWave, 0, c->stream>>>(c->n_unit, xr, c->unit_rng, c->unit_dst, c->trip,
                                                            (const double*)c->R, c->blk, c->pblk, stamp);
    if (c->n_lseg > 0) {
        const int nl = c->n_lseg_long, ns = c->n_lseg - nl;
        const int64_t n = (int64_t)ns * 81;
        if (nl > 0) k_pair_sum_long<<<nl, 1024, 0, c->stream>>>(c->lseg_blk, c->lseg_ptr, c->pblk, c->blk);
        if (ns > 0)
            k_pair_sum<<<(unsigned)((n + BS - 1) / BS), BS, 0, c->stream>>>(ns, c->lseg_blk + nl, c->lseg_ptr + nl,
                                                                            c->pblk, c->blk);
    }
}

template <typename T>
void launch_diag_t(ba_ctx* c, double lambda, u64* stamp) {
    const T* R = (const T*)c->R;
    if (c->n_rows < kDiagRows)
        k_diag<T, 4><<<c->n_rows, 4 * kWave, 0, c->stream>>>(c->n_rows, c->rowobs_ptr, c->rowobs, c->row_ptr, R, c->ebar,
                                                             lambda, c->blk, c->rhs, c->Minv, c->Linv, c->flags, stamp);
    else
        k_diag<T, 1><<<c->n_rows, kWave, 0, c->stream>>>(c->n_rows, c->rowobs_ptr, c->rowobs, c->row_ptr, R, c->ebar,
                                                         lambda, c->blk, c->rhs, c->Minv, c->Linv, c->flags, stamp);
}

void launch_diag(ba_ctx* c, double lambda, u64* stamp) {
    if (c->n_rows == 0) {
        if (stamp) launch_stamp(c, (int)(stamp - c->h_stamp));
        return;
    }
    if (c->precision == BA_MIXED)
        launch_diag_t<float>(c, lambda, stamp);
    else
        launch_diag_t<double>(c, lambda, stamp);
}

// back-substitution; the model terms go to scal[2] (|J dx|^2) and scal[3]
// (dx^T l): per-block partials of the chunks, then one per long track
template <typename T>
void launch_back_substitute_t(ba_ctx* c, const double* dxc, double* dxp, int nb, int stride) {
    const T* R = (const T*)c->R;
    if (nb > 0)
        k_backsub<T><<<nb, kBackNW * kWave, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, c->obs_pt, c->obs_row, c->chunk_q, R, c->ptL,
                                               dxc, c->e, dxp, c->part, stride);
    if (c->n_long > 0)
        k_backsub_long<T><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, c->obs_pt, c->obs_row, R, c->ptL,
                                                           dxc, c->e, dxp, c->part + nb, stride);
}

void launch_back_substitute(ba_ctx* c, const double* dxc, double* dxp, u64* stamp) {
    const int nb = (c->n_chunk + kBackNW - 1) / kBackNW;
    const int stride = nb + c->n_long;
    if (stride == 0) {
        if (stamp) launch_stamp(c, (int)(stamp - c->h_stamp));
        return;
    }
    if (2 * (int64_t)stride > c->n_part)
        throw ba_hip_error(hipErrorInvalidValue, "model-term partials exceed their buffer", __FILE__, __LINE__);
    if (c->precision == BA_MIXED)
        launch_back_substitute_t<float>(c, dxc, dxp, nb, stride);
    else
        launch_back_substitute_t<double>(c, dxc, dxp, nb, stride);
    launch_reduce(c, c->part, stride, 2, c->scal + 2, stamp);
}

// the model terms for dx_p replaced after back-substitution
template <typename T>
void launch_model_terms_t(ba_ctx* c, const double* dxc, const double* dxp, int nb, int stride) {
    const T* R = (const T*)c->R;
    if (nb > 0)
        k_model_terms<T><<<nb, BS, 0, c->stream>>>(c->n_chunk, c->chunk_ptr, c->obs_pt, c->obs_row, c->chunk_q, R,
                                                   c->ptL, dxc, dxp, c->e, c->part, stride);
    if (c->n_long > 0)
        k_model_terms_long<T><<<c->n_long, BS, 0, c->stream>>>(c->q_long0, c->long_ptr, c->obs_pt, c->obs_row, R,
                                                               c->ptL, dxc, dxp, c->e, c->part + nb, stride);
}

void launch_model_terms(ba_ctx* c, const double* dxc, const double* dxp, u64* stamp) {
    const int nb = (c->n_chunk + WPB - 1) / WPB;
    const int stride = nb + c->n_long;
    if (stride == 0) {
        if (stamp) launch_stamp(c, (int)(stamp - c->h_stamp));
        return;
    }
    if (2 * (int64_t)stride > c->n_part)
        throw ba_hip_error(hipErrorInvalidValue, "model-term partials exceed their buffer", __FILE__, __LINE__);
    if (c->precision == BA_MIXED)
        launch_model_terms_t<float>(c, dxc, dxp, nb, stride);
    else
        launch_model_terms_t<double>(c, dxc, dxp, nb, stride);
    launch_reduce(c, c->part, stride, 2, c->scal + 2, stamp);
}

}  // namespace ba
