// edt.hip -- exact Euclidean distance transform of a resident map's occupancy, the distance
// field behind the single-lookup ESDF policy of Sec. III-D: for every voxel the squared
// centre-to-centre distance, in voxels, to the nearest occupied voxel.  The squared distance
// separates over the axes: the squared distance to the nearest occupied voxel of each x row,
// then min over j of g_j + (i - j)^2 along y and along z.  Integer arithmetic.
//
// The rows' occupancy goes to bit words first (from the map's box entries: 2 bytes per 8 voxels),
// from which the y pass works out the row distances itself, so the field is written by the y pass
// and read and written by the z pass and nothing else.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rmpc_device.h"
#include "rmpc_kernels.h"

namespace rmpc {

namespace {

constexpr int32_t kFar = 1 << 30;   // larger than any squared distance of an allowed grid

// 32 voxels of an x row: which are occupied, the last occupied voxel of the row before them
// (kNoneBefore: none) and the first after them (kNoneAfter: none).
struct alignas(8) RowWord {
    uint32_t mask;
    int16_t before, after;
};
constexpr int32_t kNoneBefore = -0x8000, kNoneAfter = 0x7fff;
constexpr int32_t kNoRow = 0x4000;      // above every distance within a row, below one to an end that has none
constexpr int32_t kMost = 0x7fffffff;   // above every candidate (kFar + 4,095^2)

// Distance from voxel i of the row (bit i & 31 of its word) to the nearest occupied one, kNoRow or
// more when the row has none: the nearest at or left of it is the highest set bit up to it, else
// the one before the word, at or right of it the lowest set bit from it on, else the one after.
__device__ __forceinline__ int32_t row_distance(const RowWord &r, int32_t i)
{
    const uint32_t upto = r.mask << (31 - (i & 31)), from = r.mask >> (i & 31);
    const int32_t left = upto ? __builtin_clz(upto) : i - r.before;
    const int32_t right = from ? __builtin_ctz(from) : r.after - i;
    return min(left, right);
}

// The occupancy of 64 voxels of a row and the occupied voxels nearest to them, in one lane.
struct RowChunk {
    uint64_t mask;
    int32_t before, after;
};

__device__ __forceinline__ RowWord half_word(const RowChunk &c, int chunk, bool high)
{
    const uint32_t lo = (uint32_t)c.mask, hi = (uint32_t)(c.mask >> 32);
    RowWord r;
    r.mask = high ? hi : lo;
    r.before = (int16_t)(high && lo ? chunk * 64 + 31 - __clz(lo) : c.before);
    r.after = (int16_t)(!high && hi ? chunk * 64 + 32 + __ffs(hi) - 1 : c.after);
    return r;
}

// Two bits per brick of two bricks' entries (a word): the occupancy of the x pair of voxels at bit
// `sub` of the occupied ones, joined to four bits.
__device__ __forceinline__ uint32_t pair_bits(uint32_t w, uint32_t sub)
{
    const uint32_t occ = (w >> 15) & 0x00010001u, t = (w >> sub) & 0x00030003u & (occ | (occ << 1));
    return (t | (t >> 14)) & 15u;
}

// The occupancy of voxels 64 chunk .. 64 chunk + 63 of an x row, from 32 entries (64 consecutive
// bytes); voxels without entries (a partial map) from the grid.
template <int DT>
__device__ __forceinline__ uint64_t chunk_mask(const MapView &m, int64_t row, int chunk)
{
    const uint32_t z = (uint32_t)row / (uint32_t)m.ny, y = (uint32_t)row - z * (uint32_t)m.ny;
    const uint32_t sub = 2u * (y & 1u) + 4u * (z & 1u);
    const int first = chunk * 32, n = (int)(y >> 1) < m.nby && (int)(z >> 1) < m.nbz ? min(32, m.nbx - first) : 0;
    const uint16_t *box = m.box + (size_t)m.nbx * ((y >> 1) + (size_t)m.nby * (z >> 1)) + first;
    uint64_t mask = 0;
    if (n == 32) {
        typedef uint32_t __attribute__((aligned(2))) word_at2;
        const word_at2 *w = reinterpret_cast<const word_at2 *>(box);
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            lo |= pair_bits(w[k], sub) << (4 * k);
            hi |= pair_bits(w[k + 8], sub) << (4 * k);
        }
        mask = (uint64_t)lo | ((uint64_t)hi << 32);
    } else {
        for (int k = 0; k < n; ++k) mask |= (uint64_t)(pair_bits(box[k], sub) & 3u) << (2 * k);
    }
    if constexpr (DT != RMPC_OCC_U8) {
        if (m.partial) {
            const auto *data = static_cast<const typename Voxel<DT>::T *>(m.data);
            const int end = min(64, m.nx - 64 * chunk);
            for (int k = 2 * max(n, 0); k < end; ++k)
                if (Voxel<DT>::occ(data[row * m.nx + 64 * chunk + k])) mask |= 1ull << k;
        }
    }
    const int left = m.nx - 64 * chunk;                   // (a brick may reach past the row: free there)
    return left >= 64 ? mask : mask & ((1ull << left) - 1ull);
}

// The x pass: a lane per 64 voxels, a power of two of lanes (group) per row.  Scans over a row's
// lanes give each the last occupied voxel before its own and the first after them.  It writes the
// rows' words, or (words null: no memory for them) the squared distances themselves.
template <int DT>
__global__ void __launch_bounds__(256) edt_rows_kernel(MapView m, int group_log2, RowWord *words, int32_t *g, uint32_t *flag)
{
    if (flag && blockIdx.x == 0 && threadIdx.x < 3) flag[threadIdx.x] = 0u;
    const uint32_t id = blockIdx.x * 256u + threadIdx.x;  // (at most 64 x 4,096^2)
    const int64_t row = id >> group_log2;
    const int group = 1 << group_log2, chunk = (int)(id & (group - 1));
    const int nch = (m.nx + 63) >> 6;
    const bool in = row < (int64_t)m.ny * m.nz && chunk < nch;
    RowChunk r{in ? chunk_mask<DT>(m, row, chunk) : 0ull, 0, 0};
    // inclusive prefix max of the chunks' last occupied index, suffix min of their first
    int32_t before = r.mask ? (chunk << 6) + 63 - __clzll(r.mask) : kNoneBefore;
    int32_t after = r.mask ? (chunk << 6) + __ffsll((unsigned long long)r.mask) - 1 : kNoneAfter;
    for (int o = 1; o < group; o <<= 1) {
        const int32_t b = __shfl_up(before, o, 64), a = __shfl_down(after, o, 64);
        if (chunk >= o) before = max(before, b);
        if (chunk + o < group) after = min(after, a);
    }
    // exclusive: chunks strictly before / after this one
    r.before = __shfl_up(before, 1, 64);
    r.after = __shfl_down(after, 1, 64);
    if (chunk == 0) r.before = kNoneBefore;
    if (chunk == group - 1) r.after = kNoneAfter;
    if (!in) return;
    if (words) {
        words[(row * nch + chunk) * 2] = half_word(r, chunk, false);
        words[(row * nch + chunk) * 2 + 1] = half_word(r, chunk, true);
        return;
    }
    for (int32_t i = chunk << 6; i < min((chunk + 1) << 6, m.nx); ++i) {
        const int32_t d = row_distance(half_word(r, chunk, (i & 32) != 0), i);
        g[row * m.nx + i] = d < kNoRow ? d * d : kFar;
    }
}

// ------------------------------------------------------------------------------------------
// The y and z passes while squared distances stay below kCap: 16-bit candidates, two elements per
// instruction.  A block takes a strip of 32 (16, 8, 4) neighbouring lines whole into LDS (row j: the
// lines' consecutive 16-bit values), and every thread searches outward from its row i for four
// lines at once: the candidates i - d and i + d of all of them are two 8-byte LDS reads, and three
// packed instructions per two lines, min(a, b) + d^2 (saturating) and the running minimum.  The
// search goes on while d^2 is below the largest of the four values found.  Lanes of a wave hold
// neighbouring lines and rows, whose distances are alike, and read contiguous LDS.  Six packed
// instructions and two reads per distance serve 256 elements.
//
// Figures (400^3 paper-shaped map): y pass 223 us, z pass 179 us (it moves 512 MB, 100 us at the
// rate of a copy), rows 22 us; the three passes with 32-bit candidates, element by element, took
// 1,330 us in all.  One 1-in-1,000 random map 1,016 -> 385 us, one occupied corner (narrow passes
// given up, then wide ones) 5.8 -> 1.4 ms, 96^3 66 -> 50 us.
//
// A value of kCap stands for "kCap or more", also in the field between the passes: a result below
// it needs none of those.  A result that reaches it (no occupied voxel within 255 voxels) raises
// flag[0], and the wide passes below do the transform again; a last strip without a value below kCap
// gets -1, which is its result if all strips are such (flag[1]: one was, flag[2]: one was not).
// Where the grid is too small for any of that, flag is null.
// ------------------------------------------------------------------------------------------
constexpr int32_t kCap = 65535;
constexpr int kPad = 3;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int32_t Int4 __attribute__((ext_vector_type(4)));
typedef Int4 Int4At4 __attribute__((aligned(4)));
struct alignas(8) Quad {
    u16x2 a, b;
};

__device__ __forceinline__ uint32_t load_flag(const uint32_t *flag)
{
    return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool WORDS, int CLOG>
__device__ __forceinline__ bool load_strip(Quad *lds, const int32_t *g, const RowWord *words, int32_t len, int64_t stride,
                                           int32_t nx, int32_t x0, int64_t base, int64_t q)
{
    constexpr int kLanes = 1 << (CLOG - 2);               // threads per row, four lines each
    constexpr int kUnroll = 4;
    const int c = 4 * (threadIdx.x & (kLanes - 1)), nw32 = 2 * ((nx + 63) >> 6);
    uint32_t seen = kCap;
    for (int j0 = threadIdx.x / kLanes; j0 < len; j0 += kUnroll * (256 / kLanes)) {
        alignas(16) int32_t v[kUnroll][4];
        RowWord r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int j = min(j0 + u * (256 / kLanes), len - 1);
            if constexpr (WORDS) {
                r[u] = words[(q * len + j) * nw32 + min((x0 + c) >> 5, nw32 - 1)];
            } else {
                const int32_t *p = g + base + j * stride;
                if (c + 4 <= nx - x0) {
                    *reinterpret_cast<Int4 *>(v[u]) = *reinterpret_cast<const Int4At4 *>(p + c);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[u][k] = p[min(c + k, nx - 1 - x0)];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int j = j0 + u * (256 / kLanes);
            if constexpr (WORDS)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int32_t d = row_distance(r[u], x0 + c + k);
                    v[u][k] = (int32_t)__umul24(d, d);
                }
            if (j < len) {
                Quad o;
                o.a = u16x2{(uint16_t)min(v[u][0], kCap), (uint16_t)min(v[u][1], kCap)};
                o.b = u16x2{(uint16_t)min(v[u][2], kCap), (uint16_t)min(v[u][3], kCap)};
                lds[j * kLanes + (threadIdx.x & (kLanes - 1))] = o;
                seen = min(seen, (uint32_t)min(min(v[u][0], v[u][1]), min(v[u][2], v[u][3])));
            }
        }
    }
    return seen < kCap;
}

template <bool WORDS, int CLOG>
__global__ void __launch_bounds__(256) edt_strip_kernel(int32_t *g, const RowWord *words, int32_t len, int64_t stride,
                                                        int32_t nx, int32_t strips, int64_t outer, int last_pass,
                                                        uint32_t *flag, uint32_t *flag_host)
{
    extern __shared__ Quad strip_mem[];                   // [len + 2 kPad][lines / 4]
    Quad *strip = strip_mem;
    constexpr int kLanes = 1 << (CLOG - 2), kRows = 256 / kLanes;
    // the last pass of a transform that another block has given up does nothing (one load decides for
    // the block: other blocks raise the flag at any time, and threads that read it one by one could
    // part before the barriers below)
    if (flag) {
        __shared__ uint32_t given_up;
        if (threadIdx.x == 0) given_up = load_flag(flag);
        __syncthreads();
        if (given_up != 0u) return;
    }
    const int64_t q = blockIdx.x / strips;                // z (y pass) or y (z pass)
    const int32_t x0 = (int32_t)(blockIdx.x % strips) << CLOG;
    const int64_t base = x0 + outer * q;
    // kPad rows of kCap on both sides, so that a clamped group of rows reads nothing beyond them
    strip += kPad * kLanes;
    if (threadIdx.x < 2 * kPad * kLanes) {
        const int r = threadIdx.x / kLanes;
        const u16x2 cap = {(uint16_t)kCap, (uint16_t)kCap};
        strip[(r < kPad ? r - kPad : len + r - kPad) * kLanes + (threadIdx.x & (kLanes - 1))] = Quad{cap, cap};
    }
    // (a strip without a value below kCap has none to find)
    const int any = __syncthreads_or(load_strip<WORDS, CLOG>(strip, g, words, len, stride, nx, x0, base, q));
    const int lane = threadIdx.x & (kLanes - 1), c = 4 * lane, left = nx - x0 - c;
    const Quad *col = strip + lane;
    bool over = false;
    if (flag && threadIdx.x == 0) {
        // the store is at the L2 before the load: of two blocks of different kinds one sees the other
        if (load_flag(flag + (any ? 2 : 1)) == 0u) {
            __hip_atomic_store(flag + (any ? 2 : 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_stores();
        }
        over = load_flag(flag + (any ? 1 : 2)) != 0u;
    }
    for (int i = threadIdx.x / kLanes; i < len; i += kRows) {
        Quad best = col[i * kLanes];
        for (int d = 1; d < (any ? 256 : 0); d += 4) {
            const u16x2 m2 = __builtin_elementwise_max(best.a, best.b);
            if ((uint32_t)__mul24(d, d) >= (uint32_t)max(m2.x, m2.y)) break;
            // rows i - d - 3 .. i - d and i + d .. i + d + 3; past an end all four move towards it, to
            // where the row within is nearer than its distance taken here
            const Quad *lo = col + max(i - d, 0) * kLanes, *hi = col + min(i + d, len - 1) * kLanes;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint16_t dd = (uint16_t)min((d + u) * (d + u), kCap);
                const u16x2 d2 = {dd, dd};
                const Quad p = lo[-u * kLanes], n = hi[u * kLanes];
                best.a = __builtin_elementwise_min(
                    best.a, __builtin_elementwise_add_sat(__builtin_elementwise_min(p.a, n.a), d2));
                best.b = __builtin_elementwise_min(
                    best.b, __builtin_elementwise_add_sat(__builtin_elementwise_min(p.b, n.b), d2));
            }
        }
        int32_t v[4] = {best.a.x, best.a.y, best.b.x, best.b.y};
        if (last_pass && !any) v[0] = v[1] = v[2] = v[3] = -1;
        int32_t *p = g + base + c + i * stride;
        if (left >= 4) {
            *reinterpret_cast<Int4At4 *>(p) = Int4{v[0], v[1], v[2], v[3]};
            over = over || max(max(v[0], v[1]), max(v[2], v[3])) == kCap;
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < left) {
                    p[k] = v[k];
                    over = over || v[k] == kCap;
                }
        }
    }
    if (flag && over) {
        __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(flag_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ------------------------------------------------------------------------------------------
// The wide passes: any distance, 32-bit candidates.
// ------------------------------------------------------------------------------------------

// A block takes a strip of W = 2^WLOG neighbouring lines (consecutive x) whole into LDS, element by
// element (row j of the strip: W consecutive words, so that lanes on neighbouring lines never meet
// in a bank, whatever rows they read), and writes every element's min over j of line_j + (i - j)^2
// straight to its place.
//
// The j that attains the minimum never decreases along a line: for j < j' the difference of the two
// candidates only grows with i.  A thread takes kChunk elements of one line: it finds the best j of
// the first by an outward search (as far as (i - j)^2 stays below the best value found) and gets the
// one past its last from its neighbour; halving between known ones, each element's search is
// bounded by the two around it, and the elements between every fourth one share one sweep of their
// bounds.  That bounds the work of a line with far neighbours: a map with one occupied voxel takes
// 1.1 ms at 400^3, an outward search from every element 5.8.  (Where distances are short the narrow
// passes' search costs less: more candidates, at a tenth of the instructions.)
constexpr int kChunkLog2 = 6;
constexpr int kChunk = 1 << kChunkLog2;

template <int WLOG>
struct Line {
    const int32_t *at;                                    // element 0 in LDS
    int32_t last;
    __device__ __forceinline__ int32_t operator[](int32_t j) const { return at[j << WLOG]; }
};

// (24-bit products: full-rate instructions)
template <int WLOG>
__device__ __forceinline__ void candidate(const Line<WLOG> &l, int32_t i, int32_t j, int32_t &best, int32_t &arg)
{
    const int32_t d = i - j, v = __mul24(d, d) + l[j];
    arg = v < best ? j : arg;
    best = min(best, v);
}

// Best j of element i among all: outward from i, four distances per pass, indices clamped at the
// line's ends (a clamped candidate is one of the line's at its true distance).
template <int WLOG>
__device__ __forceinline__ void search_all(const Line<WLOG> &l, int32_t i, int32_t &best, int32_t &arg)
{
    best = l[i];
    arg = i;
    for (int32_t d = 1; d <= l.last && __mul24(d, d) < best; d += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            candidate(l, i, max(i - d - u, 0), best, arg);
            candidate(l, i, min(i + d + u, l.last), best, arg);
        }
    }
}

// Best j of element i within [lo, hi], N at a time.
template <int N, int WLOG>
__device__ __forceinline__ void search_in(const Line<WLOG> &l, int32_t i, int32_t lo, int32_t hi, int32_t &best,
                                          int32_t &arg)
{
    best = kMost;
    arg = lo;
    for (int32_t j = lo; j <= hi; j += N) {
#pragma unroll
        for (int u = 0; u < N; ++u) candidate(l, i, min(j + u, hi), best, arg);
    }
}

template <int WLOG>
__global__ void __launch_bounds__(256) edt_lines_kernel(int32_t *g, int32_t len, int64_t stride,
                                                        int32_t nx, int32_t strips, int64_t outer, int last_pass)
{
    extern __shared__ int32_t lds[];                      // line[len][W], arg[chunks + 1][W], found[W]
    constexpr int wlog = WLOG, W = 1 << WLOG;
    const int chunks = (len + kChunk - 1) >> kChunkLog2;
    int32_t *arg_of = lds + (len << wlog);
    int32_t *found = arg_of + ((chunks + 1) << wlog);
    const int64_t q = blockIdx.x / strips;                // z (y pass) or y (z pass)
    const int32_t x0 = (int32_t)(blockIdx.x % strips) << wlog;
    const int64_t base = x0 + outer * q;
    const int nw = min(W, nx - x0);                       // lines of this strip inside the grid
    const int n = len << wlog;
    if ((int)threadIdx.x < W) found[threadIdx.x] = 0;
    __syncthreads();
    constexpr int kUnroll = 8;
    for (int i0 = threadIdx.x; i0 < n; i0 += kUnroll * 256) {
        int32_t v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int idx = i0 + u * 256, w = idx & (W - 1);
            v[u] = idx < n && w < nw ? g[base + w + (int64_t)(idx >> wlog) * stride] : kFar;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int idx = i0 + u * 256;
            if (idx < n) {
                lds[idx] = v[u];
                if (v[u] < kFar) found[idx & (W - 1)] = 1;    // every writer stores the same value
            }
        }
    }
    __syncthreads();
    // the best j of every chunk's first element, and of the line's last
    for (int k = threadIdx.x; k < (chunks + 1) << wlog; k += 256) {
        const int w = k & (W - 1);
        const Line<WLOG> l{lds + w, len - 1};
        int32_t best, arg = 0;
        if (w < nw && found[w]) search_all(l, min((k >> wlog) << kChunkLog2, len - 1), best, arg);
        arg_of[k] = arg;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < chunks << wlog; k += 256) {
        const int w = k & (W - 1);
        if (w >= nw) continue;
        const int32_t i0 = (k >> wlog) << kChunkLog2;
        const Line<WLOG> l{lds + w, len - 1};
        int32_t *out = g + base + w;
        auto store = [&](int32_t i, int32_t v) {
            if (i < len) out[i * stride] = last_pass && v >= kFar ? -1 : v;
        };
        if (!found[w]) {
            // nothing finite on the line
            for (int32_t i = i0; i < min(i0 + kChunk, len); ++i) store(i, kFar);
            continue;
        }
        // every fourth element's best j, halving
        int32_t arg[kChunk / 4 + 1];
        arg[0] = arg_of[k];
        arg[kChunk / 4] = arg_of[k + W];
        {
            const int32_t d = i0 - arg[0];
            store(i0, l[arg[0]] + __mul24(d, d));
        }
#pragma unroll
        for (int half = kChunk / 8; half >= 1; half >>= 1)
#pragma unroll
            for (int m = half; m < kChunk / 4; m += 2 * half) {
                const int32_t i = i0 + 4 * m;
                int32_t best;
                // (an element past the line's end takes no part: the next known one stands for it)
                if (i < len) {
                    if (half >= 2) search_in<4>(l, i, arg[m - half], arg[m + half], best, arg[m]);
                    else search_in<2>(l, i, arg[m - half], arg[m + half], best, arg[m]);
                    store(i, best);
                } else {
                    arg[m] = arg[m + half];
                }
            }
        // the three elements between each two
#pragma unroll
        for (int m = 0; m < kChunk / 4; ++m) {
            const int32_t i = i0 + 4 * m;
            if (i + 1 >= len) break;
            const int32_t hi = arg[m + 1];
            int32_t b1 = kMost, b2 = b1, b3 = b1;
            for (int32_t j = arg[m]; j <= hi; j += 2) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int32_t jj = min(j + u, hi), v = l[jj], d = i + 1 - jj;
                    b1 = min(b1, __mul24(d, d) + v);
                    b2 = min(b2, __mul24(d + 1, d + 1) + v);
                    b3 = min(b3, __mul24(d + 2, d + 2) + v);
                }
            }
            store(i + 1, b1);
            store(i + 2, b2);
            store(i + 3, b3);
        }
    }
}

// LDS a strip of 2^wlog lines of len elements takes.  At most 54 KiB, so that three blocks share a
// CU (strips of 32 lines, rows of 128 bytes, up to 420 elements; of two lines at 4,096 elements).
constexpr size_t kStripLds = 54 * 1024;

size_t strip_lds(int32_t len, int wlog)
{
    const size_t chunks = ((size_t)len + kChunk - 1) / kChunk;
    return (((size_t)len + chunks + 2) << wlog) * sizeof(int32_t);
}

int strip_wlog(int32_t len)
{
    int wlog = 5;
    while (wlog > 1 && strip_lds(len, wlog) > kStripLds) --wlog;
    return wlog;
}

hipError_t launch_lines(int32_t *g, int32_t len, int64_t stride, int32_t nx, int64_t others, int64_t outer,
                        int last_pass, hipStream_t s)
{
    const int wlog = strip_wlog(len);
    const int32_t strips = (nx + (1 << wlog) - 1) >> wlog;
    const auto kernel = wlog == 5 ? edt_lines_kernel<5> : wlog == 4 ? edt_lines_kernel<4>
                      : wlog == 3 ? edt_lines_kernel<3> : wlog == 2 ? edt_lines_kernel<2> : edt_lines_kernel<1>;
    kernel<<<(unsigned)(others * strips), 256, strip_lds(len, wlog), s>>>(g, len, stride, nx, strips, outer, last_pass);
    return hipGetLastError();
}

// log2 of a strip's lines.  Wider strips read and write longer rows of memory, above all in the z pass;
// narrower ones take less LDS (2 bytes per line and element: 13 KiB at 208 elements, 26 at 832, 63 at
// 4,000, where two blocks share a CU), which leaves a CU more waves for a search that waits for LDS.
// Transforms of 150 lines of planes with y (z) lines of n elements, one voxel in 1,000 occupied, by strips
// of 8, 16 and 32 lines, us:
//   400    154 (207)  153 (162)  176 (153)      2,000  174 (212), 16 lines 232 (211)
//   832    143 (187)  155 (152)  202 (163)      3,500  251 (290),  4 lines 224 (367)
//   1,300  188 (246)  221 (202)  221 (204; 32 lines do not fit)
// so 16 lines up to 832, 8 beyond (to 1,300 about as good for both axes together), and 4 where 8 do not
// fit 64 KiB; up to 208 elements 32 lines were as good or better than 16 (96^3, one in ten occupied:
// 34 us against 37).
inline int strip_clog(int len) { return len <= 208 ? 5 : len <= 832 ? 4 : len <= 4000 ? 3 : 2; }

template <bool WORDS>
hipError_t launch_strips(int32_t *g, const RowWord *words, int32_t len, int64_t stride, int32_t nx, int64_t others,
                         int64_t outer, int last_pass, uint32_t *flag, uint32_t *flag_host, hipStream_t s)
{
    const int clog = strip_clog(len);
    const int32_t strips = (nx + (1 << clog) - 1) >> clog;
    const auto kernel = clog == 5 ? edt_strip_kernel<WORDS, 5>
                      : clog == 4 ? edt_strip_kernel<WORDS, 4> : clog == 3 ? edt_strip_kernel<WORDS, 3> : edt_strip_kernel<WORDS, 2>;
    kernel<<<(unsigned)(others * strips), 256, (size_t)(len + 2 * kPad) * 2 << clog, s>>>(g, words, len, stride, nx, strips, outer,
                                                                            last_pass, flag, flag_host);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_rows_dt(const MapView &m, RowWord *words, int32_t *out, uint32_t *flag, hipStream_t s)
{
    int group_log2 = 0;
    while (1 << group_log2 < (m.nx + 63) >> 6) ++group_log2;
    const int64_t n = ((int64_t)m.ny * m.nz) << group_log2;
    edt_rows_kernel<DT><<<(unsigned)((n + 255) / 256), 256, 0, s>>>(m, group_log2, words, out, flag);
    return hipGetLastError();
}

hipError_t launch_rows(const MapView &m, RowWord *words, int32_t *out, uint32_t *flag, hipStream_t s)
{
    switch (m.dtype) {
    case RMPC_TSDF_F32: return launch_rows_dt<RMPC_TSDF_F32>(m, words, out, flag, s);
    case RMPC_TSDF_F16: return launch_rows_dt<RMPC_TSDF_F16>(m, words, out, flag, s);
    default: return launch_rows_dt<RMPC_OCC_U8>(m, words, out, flag, s);
    }
}

constexpr size_t kFlagBytes = kEdtFlagBytes;

// Distance in metres at voxel (i, j, k), indices clamped into the grid; -1 when the grid has
// no occupied voxel.
__device__ double esdf_at(const EsdfArgs &A, int i, int j, int k)
{
    i = i < 0 ? 0 : (i >= A.nx ? A.nx - 1 : i);
    j = j < 0 ? 0 : (j >= A.ny ? A.ny - 1 : j);
    k = k < 0 ? 0 : (k >= A.nz ? A.nz - 1 : k);
    const int32_t q = A.sq[(int64_t)i + (int64_t)A.nx * ((int64_t)j + (int64_t)A.ny * k)];
    return q < 0 ? -1.0 : A.h * sqrt((double)q);
}

// Single-lookup ESDF policy (Sec. III-D): the distance of the position's voxel, its gradient by
// central differences over the six neighbours (divided by 2h), the obstacle direction
// r = -grad / |grad|, one obstacle policy (Eqs. 4-9) for (r, d) in float64, resolved.  Nothing
// occupied or a zero gradient: all sums zero.  One wave: lane k reads voxel k of the seven, every
// lane computes the rest, lane 0 writes.  Bound by the launch and the way back: the result goes
// straight to host memory with its sequence number after it (with a copy and a wait for the stream
// the call took 32 us, now 19).
__global__ void esdf_policy_kernel(EsdfArgs A)
{
#pragma clang fp contract(off)
    const int lane = threadIdx.x;
    const int c0 = A.v0[0], c1 = A.v0[1], c2 = A.v0[2];
    // lanes 1, 2: +-x; 3, 4: +-y; 5, 6: +-z; the others: the voxel itself
    const int axis = lane >= 1 && lane <= 6 ? (lane - 1) >> 1 : 3, step = lane & 1 ? 1 : -1;
    const double mine = esdf_at(A, c0 + (axis == 0 ? step : 0), c1 + (axis == 1 ? step : 0), c2 + (axis == 2 ? step : 0));
    const double d = __shfl(mine, 0, 64);
    double S[3][3] = {}, b[3] = {}, f[3] = {}, lam[3] = {};
    int32_t rank = 0, n_hit = 0, n_contrib = 0;
    uint32_t flags = d == 0.0 ? RMPC_Q_IN_COLLISION : 0u;
    double grad[3] = {0.0, 0.0, 0.0};
    if (d >= 0.0) {
        for (int a = 0; a < 3; ++a) grad[a] = (__shfl(mine, 1 + 2 * a, 64) - __shfl(mine, 2 + 2 * a, 64)) / (2.0 * A.h);
    }
    const double gn = sqrt(grad[0] * grad[0] + grad[1] * grad[1] + grad[2] * grad[2]);
    if (d >= 0.0 && gn > 0.0) {
        const double rh[3] = {-grad[0] / gn, -grad[1] / gn, -grad[2] / gn};
        const double n[3] = {-rh[0], -rh[1], -rh[2]};            // away from the obstacle
        const double erep = A.eta_rep * exp(-d / A.nu_rep);
        const double vn = -(A.vel[0] * n[0] + A.vel[1] * n[1] + A.vel[2] * n[2]);
        const double mx = vn > 0.0 ? vn : 0.0;
        const double kd = A.eta_damp / (d / A.nu_damp + A.eps);
        double fd[3], fo[3];
        for (int a = 0; a < 3; ++a) {
            fd[a] = kd * (mx * mx * n[a]);
            fo[a] = erep * n[a] + fd[a];
        }
        const double nf = sqrt(fd[0] * fd[0] + fd[1] * fd[1] + fd[2] * fd[2]);
        const double den = nf + A.c * log1p(exp(-2.0 * A.c * nf));
        const double w = d > A.radius ? 0.0 : d * d / (A.radius * A.radius) - 2.0 * d / A.radius + 1.0;
        double sv[3];
        for (int a = 0; a < 3; ++a) sv[a] = fd[a] / den;
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) S[i][j] = w * sv[i] * sv[j];
        for (int i = 0; i < 3; ++i) b[i] = S[i][0] * fo[0] + S[i][1] * fo[1] + S[i][2] * fo[2];
        n_hit = 1;
        n_contrib = d < A.radius && (A.vel[0] * rh[0] + A.vel[1] * rh[1] + A.vel[2] * rh[2]) > 0.0;
        resolve3(S, b, A.rank_tol, f, lam, rank, flags);
    }
    __shared__ rmpc_result res;
    if (lane == 0) {
        for (int i = 0; i < 3; ++i) {
            res.f[i] = f[i];
            res.b[i] = b[i];
            res.lambda[i] = lam[i];
            for (int j = 0; j < 3; ++j) res.A[3 * i + j] = S[i][j];
        }
        res.rank = rank;
        res.n_hit = n_hit;
        res.n_contrib = n_contrib;
        res.n_tie = 0;
        res.flags = flags;
        res.n_rays = 1;
        res.visits = 0;
    }
    store_result(&res, A.out);
    wait_stores();
    if (lane == 0) store_system(A.done, A.seq);
}

}  // namespace

hipError_t launch_esdf(const EsdfArgs &a, hipStream_t s)
{
    esdf_policy_kernel<<<1, 64, 0, s>>>(a);
    return hipGetLastError();
}

size_t edt_scratch_bytes(const MapView &m)
{
    return kFlagBytes + 2 * sizeof(RowWord) * (size_t)((m.nx + 63) >> 6) * m.ny * m.nz;
}

hipError_t launch_edt(const MapView &m, int32_t *out, void *scratch, size_t scratch_bytes, uint32_t *flag_host,
                      hipStream_t s)
{
    if (!scratch || scratch_bytes < kFlagBytes) return hipErrorInvalidValue;
    uint32_t *flag = static_cast<uint32_t *>(scratch);
    RowWord *words = scratch_bytes < edt_scratch_bytes(m)
                         ? nullptr
                         : reinterpret_cast<RowWord *>(static_cast<uint8_t *>(scratch) + kFlagBytes);
    const int64_t plane = (int64_t)m.nx * m.ny;
    if (hipError_t e = launch_rows(m, words, out, flag, s)) return e;
    // y: lines (x, z), elements nx apart; z: lines (x, y), elements nx ny apart
    const hipError_t e = words ? launch_strips<true>(out, words, m.ny, m.nx, m.nx, m.nz, plane, 0, nullptr, nullptr, s)
                               : launch_strips<false>(out, nullptr, m.ny, m.nx, m.nx, m.nz, plane, 0, nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    // no distance in a grid of this diagonal reaches kCap, and one occupied voxel leaves a value below it
    // in every strip of the last pass: no need to watch for either (16^3 25.9 -> 25.6 us, 25.4
    // with the passes before; 96^3 46.5 -> 39.7)
    const int64_t dx = m.nx - 1, dy = m.ny - 1, dz = m.nz - 1;
    const bool near = dx * dx + dy * dy + dz * dz < kCap;
    return launch_strips<false>(out, nullptr, m.nz, plane, m.nx, m.ny, m.nx, 1, near ? nullptr : flag, flag_host, s);
}

hipError_t launch_edt_wide(const MapView &m, int32_t *out, hipStream_t s)
{
    const int64_t plane = (int64_t)m.nx * m.ny;
    if (hipError_t e = launch_rows(m, nullptr, out, nullptr, s)) return e;
    if (hipError_t e = launch_lines(out, m.ny, m.nx, m.nx, m.nz, plane, 0, s)) return e;
    return launch_lines(out, m.nz, plane, m.nx, m.ny, m.nx, 1, s);
}

}  // namespace rmpc
