// rmpc_device.h -- device-side building blocks shared by the library's HIP kernels:
// map addressing and occupancy, compensated float32 sums, wave/block reductions and the
// float64 3x3 resolve.  gfx950 only (64-wide wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rmpcast.h"
#include "rmpc_kernels.h"

namespace rmpc {

constexpr int kWave = 64;
constexpr int kBlock = 256;                 // threads per block of the ray kernels
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxBlocks = kMaxPartialSlots;

// Per-ray debug flags (same bit values as the public RMPC_RAY_*).
constexpr uint32_t kRayTie = RMPC_RAY_TIE;
constexpr uint32_t kRayRangeTie = RMPC_RAY_RANGE_TIE;
constexpr uint32_t kRayStartFace = RMPC_RAY_START_FACE;
constexpr uint32_t kRayInCollision = RMPC_RAY_IN_COLLISION;

// Occupancy of a stored value: TSDF <= 0 (NaN is free), occupancy byte != 0.
template <int DT> struct Voxel;
template <> struct Voxel<RMPC_TSDF_F32> {
    using T = float;
    static __device__ __forceinline__ bool occ(float v) { return v <= 0.0f; }
};
template <> struct Voxel<RMPC_TSDF_F16> {
    using T = uint16_t;
    // binary16 <= 0 as one half-precision comparison (NaN compares false: free)
    static __device__ __forceinline__ bool occ(uint16_t b)
    {
        return __builtin_bit_cast(_Float16, b) <= (_Float16)0.0f;
    }
};
template <> struct Voxel<RMPC_OCC_U8> {
    using T = uint8_t;
    static __device__ __forceinline__ bool occ(uint8_t v) { return v != 0; }
};

// Blocks are dispatched round-robin over the 8 XCDs (block b runs on XCD b % 8).  Give each
// XCD a contiguous run of tiles so that its L2 sees one compact cone of ray directions (or run of
// bricks).
__device__ __forceinline__ int xcd_tile(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

// ------------------------------------------------------------------------------------
// compensated float32 sums (error-free TwoSum; the compensations are kept to the end)
// ------------------------------------------------------------------------------------

__device__ __forceinline__ void csum_add(float &s, float &c, float x)
{
#pragma clang fp contract(off)
    float t = s + x;
    float bp = t - s;
    float err = (s - (t - bp)) + (x - bp);
    s = t;
    c += err;
}

__device__ __forceinline__ void csum_merge(float &s, float &c, float s2, float c2)
{
#pragma clang fp contract(off)
    float t = s + s2;
    float bp = t - s;
    float err = (s - (t - bp)) + (s2 - bp);
    s = t;
    c = (c + c2) + err;
}

// The quantities one query reduces: the 6 unique entries of sum A_i, the 3 of sum b_i
// (each as a compensated pair) and four integer counters.
struct Acc {
    float s[9], c[9];
    int32_t n_hit, n_contrib, n_tie, visits;

    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int k = 0; k < 9; ++k) { s[k] = 0.0f; c[k] = 0.0f; }
        n_hit = n_contrib = n_tie = visits = 0;
    }
};

// ------------------------------------------------------------------------------------
// block and grid reductions of Acc
//
// A block writes one row per thread to LDS.  Nine groups of 16 lanes (threads 0..143) merge
// one compensated pair each and four groups in the last wave (threads 192..255) add one
// integer counter each, so no wave mixes the two kinds.  Lane q of a group merges rows q,
// q+16, ... in row order (all 16 loaded first), and the 16 lanes combine with a butterfly
// that always puts the lower lane first.  (A pairwise tree over the 16 rows was no faster.)  Every step has a fixed order, so results do not
// depend on timing.
// ------------------------------------------------------------------------------------

constexpr int kSumWords = 22;                 // 9 sums, 9 compensations, 4 counters
constexpr int kRowWords = 23;                 // odd row stride: conflict-free column reads
constexpr int kColLanes = 16;
constexpr int kPairLanes = 9 * kColLanes;     // threads merging the compensated pairs
constexpr int kIntLane0 = kBlock - 4 * kColLanes;   // first thread adding the counters
constexpr int kReduceLdsWords = kBlock * kRowWords;
static_assert(kPairLanes <= kIntLane0 && kIntLane0 % kWave == 0, "pair and counter lanes share a wave");

__device__ __forceinline__ void row_store(float *row, const Acc &a)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) { row[k] = a.s[k]; row[9 + k] = a.c[k]; }
    int32_t *q = reinterpret_cast<int32_t *>(row + 18);
    q[0] = a.n_hit; q[1] = a.n_contrib; q[2] = a.n_tie; q[3] = a.visits;
}

// The value of the lane across the given step of a butterfly over 16 lanes, in one instruction: lane
// ^ 1, ^ 2, and, where 4 (8) lanes hold the same value already, any of the other 4 (8), which
// mirroring the 8 (16) lanes reaches.  (Through LDS, __shfl_xor, the four steps waited some 400
// cycles.)
template <int OFF>
__device__ __forceinline__ int32_t across(int32_t v)
{
    constexpr int ctrl = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : OFF == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, true);
}

template <int OFF>
__device__ __forceinline__ void pair_step(int t, float &s, float &c)
{
    const float s2 = __int_as_float(across<OFF>(__float_as_int(s)));
    const float c2 = __int_as_float(across<OFF>(__float_as_int(c)));
    const bool upper = (t & OFF) != 0;
    float ls = upper ? s2 : s, lc = upper ? c2 : c;
    csum_merge(ls, lc, upper ? s : s2, upper ? c : c2);
    s = ls;
    c = lc;
}

// Butterfly over the 16 lanes of a pair group; the lower lane's value is always the left
// operand of the merge.
__device__ __forceinline__ void pair_butterfly(int t, float &s, float &c)
{
    pair_step<1>(t, s, c);
    pair_step<2>(t, s, c);
    pair_step<4>(t, s, c);
    pair_step<8>(t, s, c);
}

__device__ __forceinline__ int32_t int_butterfly(int32_t v)
{
    v += across<1>(v);
    v += across<2>(v);
    v += across<4>(v);
    return v + across<8>(v);
}

// The thread index through an empty asm statement.  The reductions' LDS addresses and lane
// masks depend on it alone, and in a kernel that loops over tiles the compiler would otherwise
// compute them once before the loop and keep them in registers through every walk.
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

constexpr int kColRows = kBlock / kColLanes;       // rows a lane merges

// A lane's share of a column: the pair sums of its kColRows rows and, in the counter lanes, their
// sum of one counter.
struct Column {
    float s[kColRows], c[kColRows];
    int32_t n;
};

// Take the kBlock rows in LDS: as they are (first) or merged after the rows taken before.
__device__ __forceinline__ void column_rows(Column &o, const float *lds, int t, bool first)
{
    const int q = t % kColLanes;
    if (t < kPairLanes) {
        const int col = t / kColLanes;
        float s[kColRows], c[kColRows];
#pragma unroll
        for (int u = 0; u < kColRows; ++u) {
            s[u] = lds[(q + u * kColLanes) * kRowWords + col];
            c[u] = lds[(q + u * kColLanes) * kRowWords + 9 + col];
        }
#pragma unroll
        for (int u = 0; u < kColRows; ++u) {
            if (first) { o.s[u] = s[u]; o.c[u] = c[u]; }
            else csum_merge(o.s[u], o.c[u], s[u], c[u]);
        }
    } else if (t >= kIntLane0) {
        const int col = (t - kIntLane0) / kColLanes;
        const int32_t *rows = reinterpret_cast<const int32_t *>(lds);
        int32_t v = first ? 0 : o.n;
#pragma unroll
        for (int u = 0; u < kColRows; ++u) v += rows[(q + u * kColLanes) * kRowWords + 18 + col];
        o.n = v;
    }
}

// The columns' totals, written to out[] in partial layout (9 sums, 9 compensations, 4 counters).
__device__ __forceinline__ void column_store(const Column &o, int t, float *out)
{
    const int q = t % kColLanes;
    if (t < kPairLanes) {
        const int col = t / kColLanes;
        float s = o.s[0], c = o.c[0];
#pragma unroll
        for (int u = 1; u < kColRows; ++u) csum_merge(s, c, o.s[u], o.c[u]);
        pair_butterfly(t, s, c);
        if (q == 0) { out[col] = s; out[9 + col] = c; }
    } else if (t >= kIntLane0) {
        const int32_t v = int_butterfly(o.n);
        if (q == 0) reinterpret_cast<int32_t *>(out)[18 + (t - kIntLane0) / kColLanes] = v;
    }
}

// The block total, written to out[].
__device__ __forceinline__ void block_reduce_store(const Acc &a, float *lds, float *out)
{
    const int t = opaque_tid();
    row_store(lds + t * kRowWords, a);
    __syncthreads();
    Column o;
    column_rows(o, lds, t, true);
    column_store(o, t, out);
}

// ------------------------------------------------------------------------------------
// float64 resolve: f = S^+ b  (Eq. 1 with the pseudo-inverse cut rank_tol * lambda_max)
// ------------------------------------------------------------------------------------

// Reciprocal and reciprocal square root from the hardware estimates plus two Newton steps
// (relative error near 1 ulp; a Jacobi rotation only needs c^2 + s^2 = 1 to that level).
__device__ __forceinline__ double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double rsqrt64(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    r = r * fma(-0.5 * x * r, r, 1.5);
    return r * fma(-0.5 * x * r, r, 1.5);
}

// One Jacobi rotation in the (P, Q) plane that annihilates S[P][Q]; V accumulates the
// eigenvectors as columns.  Compile-time indices keep everything in registers.
template <int P, int Q>
__device__ __forceinline__ void jacobi_rotate(double (&S)[3][3], double (&V)[3][3])
{
    const double spq = S[P][Q];
    if (spq == 0.0) return;
    const double theta = (S[Q][Q] - S[P][P]) * (0.5 * rcp64(spq));
    const double at = fabs(theta);
    // t = sign(theta) / (|theta| + sqrt(theta^2 + 1)), the smaller root of t^2 + 2 t theta = 1
    double t;
    if (at > 1e100) {
        t = 0.5 * rcp64(theta);
    } else {
        const double y = fma(at, at, 1.0);
        t = rcp64(at + y * rsqrt64(y));
        t = theta < 0.0 ? -t : t;
    }
    const double c = rsqrt64(fma(t, t, 1.0));
    const double s = t * c;
    constexpr int R = 3 - P - Q;                 // the untouched index
    const double spp = S[P][P], sqq = S[Q][Q], srp = S[R][P], srq = S[R][Q];
    S[P][P] = spp - t * spq;
    S[Q][Q] = sqq + t * spq;
    S[P][Q] = S[Q][P] = 0.0;
    S[R][P] = S[P][R] = c * srp - s * srq;
    S[R][Q] = S[Q][R] = s * srp + c * srq;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double vkp = V[k][P], vkq = V[k][Q];
        V[k][P] = c * vkp - s * vkq;
        V[k][Q] = s * vkp + c * vkq;
    }
}

// Eigenvalues of a symmetric 3x3 matrix, ascending, from the trigonometric solution of its
// characteristic cubic: with q = tr S / 3, p^2 = |S - q I|_F^2 / 6 and B = (S - q I) / p, the
// eigenvalues are q + 2 p cos(phi + 2 pi k / 3), phi = acos(det B / 2) / 3.  Each is within a
// few units of rounding of |S| of the exact value.  False for a diagonal matrix.
__device__ inline bool sym3_eigvals(const double (&S)[3][3], double (&lam)[3])
{
    const double p1 = S[0][1] * S[0][1] + S[0][2] * S[0][2] + S[1][2] * S[1][2];
    if (p1 == 0.0) return false;
    const double q = (S[0][0] + S[1][1] + S[2][2]) * (1.0 / 3.0);
    const double d0 = S[0][0] - q, d1 = S[1][1] - q, d2 = S[2][2] - q;
    const double p = sqrt((d0 * d0 + d1 * d1 + d2 * d2 + 2.0 * p1) * (1.0 / 6.0));
    const double ip = 1.0 / p;
    const double b00 = d0 * ip, b11 = d1 * ip, b22 = d2 * ip;
    const double b01 = S[0][1] * ip, b02 = S[0][2] * ip, b12 = S[1][2] * ip;
    const double det = b00 * (b11 * b22 - b12 * b12) - b01 * (b01 * b22 - b12 * b02) + b02 * (b01 * b12 - b11 * b02);
    const double r = fmin(1.0, fmax(-1.0, 0.5 * det));
    const double phi = acos(r) * (1.0 / 3.0);
    lam[2] = q + 2.0 * p * cos(phi);
    lam[0] = q + 2.0 * p * cos(phi + 2.0943951023931957);          // + 2 pi / 3
    lam[1] = 3.0 * q - lam[0] - lam[2];
    return true;
}

// Resolve a symmetric PSD 3x3 metric sum: eigenvalues (ascending), rank, ILL flag and f.
// A sum whose smallest eigenvalue lies clearly above the ILL band and whose condition number
// lies clearly below the ILL limit (both by a relative margin of 1e-9, far above the closed
// form's error) has full rank and no ILL flag: there f = S^-1 b by the adjugate, which is the
// pseudo-inverse; every other sum takes the cyclic Jacobi path below.
__device__ inline void resolve3(const double (&Sin)[3][3], const double (&b)[3], double rank_tol,
                                double (&f)[3], double (&lam)[3], int32_t &rank, uint32_t &flags)
{
    {
        double l[3];
        if (sym3_eigvals(Sin, l) && l[2] > 0.0 && l[0] > 10.0 * (rank_tol * l[2]) * (1.0 + 1e-9) &&
            l[2] < 1e3 * (1.0 - 1e-9) * l[0]) {
            const double(&A)[3][3] = Sin;
            // cofactors (symmetric for a symmetric matrix, so the adjugate is the same matrix)
            const double c00 = A[1][1] * A[2][2] - A[1][2] * A[2][1];
            const double c01 = A[1][2] * A[2][0] - A[1][0] * A[2][2];
            const double c02 = A[1][0] * A[2][1] - A[1][1] * A[2][0];
            const double c11 = A[0][0] * A[2][2] - A[0][2] * A[2][0];
            const double c12 = A[0][1] * A[2][0] - A[0][0] * A[2][1];
            const double c22 = A[0][0] * A[1][1] - A[0][1] * A[1][0];
            const double id = 1.0 / (A[0][0] * c00 + A[0][1] * c01 + A[0][2] * c02);
            f[0] = (c00 * b[0] + c01 * b[1] + c02 * b[2]) * id;
            f[1] = (c01 * b[0] + c11 * b[1] + c12 * b[2]) * id;
            f[2] = (c02 * b[0] + c12 * b[1] + c22 * b[2]) * id;
            lam[0] = l[0]; lam[1] = l[1]; lam[2] = l[2];
            rank = 3;
            return;
        }
    }
    double S[3][3], V[3][3];
    double frob2 = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            S[i][j] = Sin[i][j];
            V[i][j] = i == j ? 1.0 : 0.0;
            frob2 += S[i][j] * S[i][j];
        }
    for (int sweep = 0; sweep < 32; ++sweep) {
        const double off2 = S[0][1] * S[0][1] + S[0][2] * S[0][2] + S[1][2] * S[1][2];
        if (off2 <= 1e-30 * frob2) break;
        jacobi_rotate<0, 1>(S, V);
        jacobi_rotate<0, 2>(S, V);
        jacobi_rotate<1, 2>(S, V);
    }
    // sort eigenpairs ascending (a 3-element network on indices)
    int i0 = 0, i1 = 1, i2 = 2;
    double d0 = S[0][0], d1 = S[1][1], d2 = S[2][2];
    if (d1 < d0) { double t = d0; d0 = d1; d1 = t; int u = i0; i0 = i1; i1 = u; }
    if (d2 < d1) { double t = d1; d1 = d2; d2 = t; int u = i1; i1 = i2; i2 = u; }
    if (d1 < d0) { double t = d0; d0 = d1; d1 = t; int u = i0; i0 = i1; i1 = u; }
    lam[0] = d0; lam[1] = d1; lam[2] = d2;
    const int idx[3] = {i0, i1, i2};
    f[0] = f[1] = f[2] = 0.0;
    rank = 0;
    if (!(d2 > 0.0)) return;
    const double tau = rank_tol * d2;
    double lmin_kept = d2;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double l = lam[j];
        if (l >= 0.1 * tau && l <= 10.0 * tau) flags |= RMPC_Q_ILL;
        if (!(l > tau)) continue;
        ++rank;
        lmin_kept = fmin(lmin_kept, l);
        const int col = idx[j];
        double q0, q1, q2;
        // column `col` of V without dynamic register indexing
        q0 = col == 0 ? V[0][0] : (col == 1 ? V[0][1] : V[0][2]);
        q1 = col == 0 ? V[1][0] : (col == 1 ? V[1][1] : V[1][2]);
        q2 = col == 0 ? V[2][0] : (col == 1 ? V[2][1] : V[2][2]);
        const double qb = (q0 * b[0] + q1 * b[1] + q2 * b[2]) / l;
        f[0] += q0 * qb; f[1] += q1 * qb; f[2] += q2 * qb;
    }
    if (d2 / lmin_kept > 1e3) flags |= RMPC_Q_ILL;
}

// A store that the host can see as soon as it is acknowledged (wait_stores).
template <typename T>
__device__ __forceinline__ void store_system(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Turn a reduced accumulator into the public result (run by one thread).
__device__ inline void finalize_result(const Acc &a, double rank_tol, int32_t n_rays,
                                       uint32_t extra_flags, rmpc_result *out)
{
    double sv[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) sv[k] = (double)a.s[k] + (double)a.c[k];
    // unique entries: 0 xx, 1 xy, 2 xz, 3 yy, 4 yz, 5 zz, then b x, y, z
    const double S[3][3] = {{sv[0], sv[1], sv[2]}, {sv[1], sv[3], sv[4]}, {sv[2], sv[4], sv[5]}};
    const double b[3] = {sv[6], sv[7], sv[8]};
    double f[3], lam[3];
    int32_t rank = 0;
    uint32_t flags = extra_flags;
    resolve3(S, b, rank_tol, f, lam, rank, flags);
    if (a.n_tie > 0) flags |= RMPC_Q_TIE;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        out->f[i] = f[i];
        out->b[i] = b[i];
        out->lambda[i] = lam[i];
#pragma unroll
        for (int j = 0; j < 3; ++j) out->A[3 * i + j] = S[i][j];
    }
    out->rank = rank;
    out->n_hit = a.n_hit;
    out->n_contrib = a.n_contrib;
    out->n_tie = a.n_tie;
    out->flags = flags;
    out->n_rays = n_rays;
    out->visits = (int64_t)a.visits;
}

// The wave's first lane has filled `from` (LDS): the wave stores it to host memory, 8 bytes a lane, in
// one instruction.  (Stored word by word by one lane the 176 bytes crossed the bus as 25 writes: 80
// queries of 16 rays took 127 us, 512 took 218.)
static_assert(sizeof(rmpc_result) % 8 == 0 && sizeof(rmpc_result) / 8 <= kWave, "a word per lane");
__device__ __forceinline__ void store_result(const rmpc_result *from, rmpc_result *out)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int lane = threadIdx.x & (kWave - 1);
    if (lane < (int)(sizeof(rmpc_result) / 8))
        store_system(reinterpret_cast<uint64_t *>(out) + lane, reinterpret_cast<const uint64_t *>(from)[lane]);
}

// A row in partial layout, in LDS.
__device__ __forceinline__ void acc_from_words(const float *w, Acc &a)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) { a.s[k] = w[k]; a.c[k] = w[9 + k]; }
    a.n_hit = __float_as_int(w[18]); a.n_contrib = __float_as_int(w[19]);
    a.n_tie = __float_as_int(w[20]); a.visits = __float_as_int(w[21]);
}

// Waits until this wave's earlier stores have been acknowledged.  Stores and atomics of agent
// (system) scope are acknowledged by the memory that all XCDs (and the host) share, so an atomic
// issued after the wait is seen by nobody before them, without the write-back of the whole L2
// that a release operation makes here.
__device__ __forceinline__ void wait_stores()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The total of n rows that other blocks have written to device memory, past this XCD's L2, written
// to out[].  256 rows at a time: 16 lanes load a row (11 of them 8 bytes each) and put it into LDS
// as a thread's row.  (A row per thread, 88 bytes at a stride of 128, made every load instruction
// 64 requests: 512 rows took 4.9 us to arrive and be merged against 3.2, a
// 65,536-ray query 33.6 us against 31.2.)
__device__ __forceinline__ void rows_reduce_store(const float *rows, int n, float *lds, float *out)
{
    const int t = opaque_tid(), q = t & (kColLanes - 1), row = t / kColLanes;
    const uint64_t *words = reinterpret_cast<const uint64_t *>(rows) + min(q, kSumWords / 2 - 1);
    float *to = lds + row * kRowWords + 2 * q;
    Column o;
    for (int r0 = 0; r0 < n; r0 += kBlock) {
        uint64_t w[kColRows];
#pragma unroll
        for (int k = 0; k < kColRows; ++k) {
            const uint32_t r = (uint32_t)min(r0 + row + k * kColLanes, n - 1);
            w[k] = __hip_atomic_load(words + r * (kPartialWords / 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (r0) __syncthreads();             // the rows before have been taken
        if (q < kSumWords / 2)
#pragma unroll
            for (int k = 0; k < kColRows; ++k) {
                const uint64_t v = r0 + row + k * kColLanes < n ? w[k] : 0ull;
                to[k * kColLanes * kRowWords] = __uint_as_float((uint32_t)v);
                to[k * kColLanes * kRowWords + 1] = __uint_as_float((uint32_t)(v >> 32));
            }
        __syncthreads();
        column_rows(o, lds, t, r0 == 0);
    }
    column_store(o, t, out);
}

// Where one reduction keeps its state: tile rows (one per tile), a ticket, the result slot,
// and the completion publication.  A batch shares `finished` (queries done so far) among its
// queries and publishes once, when the last one is done.
struct FinishSlots {
    float *tile_rows;
    uint32_t *tickets;
    rmpc_result *out;
    uint32_t *finished;          // null for a single query
    int32_t n_queries;
    uint64_t *done;              // null: nothing is published
    uint64_t seq;
};

// Grid reduction: every block stores its total in its row and takes a ticket; the last block
// merges all rows -- rows r, r + 256, ... in that order, then the block tree merges those 256
// -- so the result depends on the rows and their count only, never on the
// order in which blocks finish.  It resolves, writes the result and publishes.
//
// Rows, tickets and results go past the L2 with agent- and system-scope accesses, ordered by
// waiting for the stores before the ticket is taken.  With a release on every ticket and an
// acquire in the last block, each block wrote its XCD's whole L2 back (and the last block
// invalidated it) under the blocks still walking: a batch of 512 map queries (45,000 tiles) took
// 2.88 ms instead of 2.23, a 65,536-point scan 12.3 us instead of 10.8.
__device__ inline void grid_finish(const Acc &a, int b, int nb, const FinishSlots &F,
                                   double rank_tol, int32_t n_rays, uint32_t extra_flags, float *lds)
{
    __shared__ int last;
    __shared__ __align__(16) float tot[kPartialWords];
    block_reduce_store(a, lds, tot);
    __syncthreads();
    if (threadIdx.x < kWave) {
        // the first wave stores the block's row (one word per lane) and takes the ticket
        const int t = opaque_tid();
        if (t < kSumWords)
            __hip_atomic_store(F.tile_rows + (size_t)b * kPartialWords + t, tot[t], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        wait_stores();
        if (t == 0) {
            const uint32_t prev = __hip_atomic_fetch_add(F.tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = prev == (uint32_t)(nb - 1);
        }
    }
    __syncthreads();
    if (!last) return;
    rows_reduce_store(F.tile_rows, nb, lds, tot);
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    rmpc_result *res = reinterpret_cast<rmpc_result *>(lds);
    if (threadIdx.x == 0) {
        Acc total;
        acc_from_words(tot, total);
        __hip_atomic_store(F.tickets, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        finalize_result(total, rank_tol, n_rays, extra_flags, res);
    }
    store_result(res, F.out);
    wait_stores();
    if (threadIdx.x == 0) {
        bool publish = true;
        if (F.finished) {
            // every query's result has reached the host before the publication
            const uint32_t prev = __hip_atomic_fetch_add(F.finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            publish = prev == (uint32_t)(F.n_queries - 1);
            if (publish) {
                __hip_atomic_store(F.finished, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                wait_stores();
            }
        }
        // publish: the results are visible to the host before the sequence number (no word to
        // publish to: the result stays in device memory, ordered by the stream)
        if (publish && F.done) __hip_atomic_store(F.done, F.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace rmpc
