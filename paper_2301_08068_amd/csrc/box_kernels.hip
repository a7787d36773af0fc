// box_kernels.hip -- the box entries of an uploaded map (rmpc_dense.h): per brick of 2 x 2 x 2
// voxels a box of free bricks around it, or its occupancy and its widest free voxel layer.
//
// The extents come from Chebyshev distances between bricks, taken on bit sets (one bit per brick,
// rows along x in 64-bit words), where a dilation step costs a few instructions per 64 bricks:
//   layers  the square dilations by 1 .. 6 bricks, within the layers of bricks perpendicular to
//           each axis, of the bricks' six voxel layers.  Counting the steps that do not reach a
//           brick (in bit-sliced counters) gives its free layers' extents (1 .. 7); the union of
//           an axis' two sides gives the extents of a slab one brick thick
//   cube    the cubic dilations by 1 .. 6: the half extent d of the free cube around a brick
//   slab    close to a surface (d <= 3) the slab of half thickness d, perpendicular to the
//           axis that allows the widest one, takes the cube's place, so that rays that graze floors
//           and walls cross long runs of free space too
//   far     where the cubes of the 27 bricks 3 (6) away are free as well, half extent 10 (13)
// (modelled on the paper-shaped map, the slowest of 64 neighbouring rays takes 24 boxes next to the
// floor with cubes of up to 255 bricks alone, 10 with these; elsewhere 17-22 and 11-16).
//
// Bound by the copy: the grid is read once and written once (float32 and float16 maps).  A 400^3
// float32 grid: 85 us for the copy (6.0 TB/s) with the occupancy, 13 us for the layer sets, 22 and 19
// for the dilations, 20 for the choice, 22 to write the entries; a copy and one thread per 8^3 cell
// and per 2^3 brick took 91 + 147 + 65 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rmpc_device.h"
#include "rmpc_kernels.h"

namespace rmpc {

namespace {

constexpr int kSteps = 6;                         // dilation steps; extents 1 .. kSteps + 1 come from them
constexpr uint32_t kUnitBox = box_extents(1, 1, 1);

// Scratch: the occupancy of every brick's voxels (a byte), then bit sets of `words` 64-bit words each.
// A set's words lie along one of the grid's axes (`axis`), its rows along the next, its planes along
// the third: x, y, z, or with x and y, or x and z, changed over (`axis` 1, 2).  A grid a few bricks
// wide in x has most of a word's 64 bits past its end: with words along x always, one of 2 x 2,048 x
// 2,048 float32 voxels took 436 MB of scratch and 1,037 us to upload (now 7.9 MB, 68 us), one of
// 1 x 4,096 x 4,096 bytes 1.8 GB and 5.4 ms (31 MB, 87 us).
struct Scratch {
    BoxMask mask;                                 // 0: free
    uint64_t *layer;                              // 6: voxel layers axis 0 low, high, axis 1 low, ...
    uint64_t *cz, *cy, *cx;                       // kSteps each: dilated slabs, perpendicular to axis 2, 1, 0
    uint64_t *yx;                                 // 2 kSteps: the layers of axis 0 dilated along axis 1
    uint64_t *best;                               // 6: extent (3 bits), side and axis (2 bits) of the best layer
    uint64_t *best_y;                             // 6: of the best perpendicular to axis 1 alone
    uint64_t *cube;                               // 3: bits of d
    uint64_t *full;                               // 1: d = kSteps + 1
    int64_t words;
    int32_t axis;
    int32_t n0, n1, n2, w;                        // bricks along the axes in this order; words of a row
    bool wall0, wall1, wall2;                     // an odd last voxel layer without entries
};
constexpr int kSets = 6 + 3 * kSteps + 2 * kSteps + 6 + 3 + 1 + 6;

inline int64_t set_words(const MapView &m, int axis)
{
    const int64_t n[3] = {m.nbx, m.nby, m.nbz};
    return (n[axis] + 63) / 64 * (n[0] * n[1] * n[2] / std::max<int64_t>(n[axis], 1));
}

// The axis that words lie along: x, whose neighbours are neighbours in memory, unless another takes
// less than three quarters of its words (48 x 400 x 400, along y half of them: 66 -> 63 us; 70 x 300 x
// 300, 0.7 of them: 65 and 66 us).
inline int word_axis(const MapView &m)
{
    const int other = set_words(m, 2) < set_words(m, 1) ? 2 : 1;
    return 4 * set_words(m, other) < 3 * set_words(m, 0) ? other : 0;
}

Scratch scratch_at(const MapView &m, uint8_t *p)
{
    Scratch s;
    s.axis = word_axis(m);
    const int32_t n[3] = {m.nbx, m.nby, m.nbz};
    const bool wall[3] = {2 * m.nbx < m.nx, 2 * m.nby < m.ny, 2 * m.nbz < m.nz};
    const int a1 = s.axis == 1 ? 0 : 1, a2 = s.axis == 2 ? 0 : 2;
    s.n0 = n[s.axis]; s.n1 = n[a1]; s.n2 = n[a2];
    s.wall0 = wall[s.axis]; s.wall1 = wall[a1]; s.wall2 = wall[a2];
    s.w = (s.n0 + 63) >> 6;
    s.words = set_words(m, s.axis);
    s.mask = box_mask(m, p);
    s.layer = reinterpret_cast<uint64_t *>(p + s.mask.bytes);
    s.cz = s.layer + 6 * s.words;
    s.cy = s.cz + kSteps * s.words;
    s.cx = s.cy + kSteps * s.words;
    s.yx = s.cx + kSteps * s.words;
    s.best = s.yx + 2 * kSteps * s.words;
    s.cube = s.best + 6 * s.words;
    s.full = s.cube + 3 * s.words;
    s.best_y = s.full + s.words;
    return s;
}

// (what the extents below reach, and twice it fits five bits)
static_assert(13 <= kBoxMax && 2 * kBoxMax < 32, "half extents of box entries");

__device__ __forceinline__ uint16_t unit_entry(uint32_t mask)
{
    return (uint16_t)(mask ? kBoxOccupied | kBoxNoLayer | mask : kUnitBox);
}

// Occupancy of every brick, copying the voxels to dst (null: no copy; every voxel of the grid is
// copied, those outside the bricks of a partial map by copy_rest_kernel).  A thread takes W
// consecutive bricks of a row: with W = 2 each of its four voxel rows is one load of four
// elements (rows of a multiple of four elements, aligned), with W = 1 any grid.
// UNIT: write entries of single-brick boxes instead of the masks.
template <int DT, int W, bool UNIT>
__global__ void __launch_bounds__(256) brick_kernel(MapView m, const typename Voxel<DT>::T *src,
                                                    typename Voxel<DT>::T *dst, BoxMask mask, uint16_t *box)
{
    using T = typename Voxel<DT>::T;
    const uint32_t nw = ((uint32_t)m.nbx + W - 1) / W;
    const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= (uint64_t)nw * m.nby * m.nbz) return;
    const uint32_t row = (uint32_t)(id / nw), bx = (uint32_t)(id - (uint64_t)row * nw) * W;
    const uint32_t bz = row / (uint32_t)m.nby, by = row - bz * (uint32_t)m.nby;
    uint32_t occ[W] = {};
    if constexpr (W == 2) {
        struct alignas(4 * sizeof(T)) Quad { T v[4]; };
        Quad q[4];
        bool in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t y = 2 * by + (k & 1), z = 2 * bz + (k >> 1);
            in[k] = y < (uint32_t)m.ny && z < (uint32_t)m.nz;
            const uint64_t at = 2 * bx + (uint64_t)m.nx * (in[k] ? y + (uint64_t)m.ny * z : 0u);
            q[k] = *reinterpret_cast<const Quad *>(src + at);
            if (dst && in[k]) *reinterpret_cast<Quad *>(dst + at) = q[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (in[k] && Voxel<DT>::occ(q[k].v[i])) occ[i >> 1] |= 1u << ((i & 1) + 2 * k);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t x = 2 * bx + (k & 1), y = 2 * by + ((k >> 1) & 1), z = 2 * bz + (k >> 2);
            if (x >= (uint32_t)m.nx || y >= (uint32_t)m.ny || z >= (uint32_t)m.nz) continue;
            const uint64_t at = x + (uint64_t)m.nx * (y + (uint64_t)m.ny * z);
            const T v = src[at];
            if (dst) dst[at] = v;
            if (Voxel<DT>::occ(v)) occ[0] |= 1u << k;
        }
    }
#pragma unroll
    for (int i = 0; i < W; ++i) {
        if (bx + i >= (uint32_t)m.nbx) break;
        if constexpr (UNIT) box[(uint64_t)row * m.nbx + bx + i] = unit_entry(occ[i]);
        else mask.at[(bx + i) * mask.sx + by * mask.sy + bz * mask.sz] = (uint8_t)occ[i];
    }
}

// The voxels of a partial map that lie outside its bricks: at the end of every row (the first
// row_blocks blocks, a thread per row), and the rows of an odd last layer along y or z, a block each.
// (A block per row of the grid, most of them for one voxel, took 18 us on a 255^3 float16 map against
// 5.)
template <int DT>
__global__ void __launch_bounds__(256) copy_rest_kernel(MapView m, const typename Voxel<DT>::T *src,
                                                        typename Voxel<DT>::T *dst, uint32_t row_blocks, uint32_t y_rows)
{
    if (blockIdx.x < row_blocks) {
        const uint64_t row = (uint64_t)blockIdx.x * 256 + threadIdx.x;
        if (row >= (uint64_t)m.ny * m.nz) return;
        for (int x = 2 * m.nbx; x < m.nx; ++x) dst[x + (uint64_t)m.nx * row] = src[x + (uint64_t)m.nx * row];
        return;
    }
    // row y of z = k (the last y), or of z = nz - 1
    const uint32_t k = blockIdx.x - row_blocks;
    const uint64_t row = k < y_rows ? (uint64_t)m.ny - 1 + (uint64_t)m.ny * k : (uint64_t)(k - y_rows) + (uint64_t)m.ny * (m.nz - 1);
    for (uint32_t x = threadIdx.x; x < (uint32_t)m.nx; x += 256) dst[x + (uint64_t)m.nx * row] = src[x + (uint64_t)m.nx * row];
}

// The layer sets from the masks: a lane takes four bricks of a row, eight lanes join their bits to
// 32-bit words.  Bricks past the row's end are free, or occupied on a partial axis (bricks there
// have no entries, so a box must not cover them).  id: the four bricks, neighbouring lanes' one after
// the other.
__device__ __forceinline__ void layer_bits(const Scratch &s, int64_t id)
{
    const int64_t row = id / (16 * s.w);
    const int x = (int)(id - row * 16 * s.w) * 4;
    const bool in = row < (int64_t)s.n1 * s.n2;
    uint32_t v = s.wall0 ? ~0u : 0u;
    if (in && x < s.n0) {
        const uint32_t last = s.n0 - x;                                // bricks of the row from here
        const uint32_t past = last < 4 ? ~0u << (8 * last) : 0u;
        v = (*reinterpret_cast<const uint32_t *>(s.mask.at + row * (int64_t)s.mask.pitch + x) & ~past) | (v & past);
    }
    // the voxels of a layer, by the layer's axis in the sets' order
    const uint32_t selx = 0x55u, sely = 0x33u, selz = 0x0fu;
    const uint32_t sel0 = s.axis == 0 ? selx : (s.axis == 1 ? sely : selz), sel1 = s.axis == 1 ? selx : sely,
                   sel2 = s.axis == 2 ? selx : selz;
    const uint32_t sel[6] = {sel0, ~sel0 & 0xffu, sel1, ~sel1 & 0xffu, sel2, ~sel2 & 0xffu};
    const int lane = (int)(id & 7), shift = 4 * lane;
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const uint32_t t = v & (sel[k] * 0x01010101u);
        // the top bit of every non-zero byte, gathered into four bits
        const uint32_t top = (((t & 0x7f7f7f7fu) + 0x7f7f7f7fu) | t) & 0x80808080u;
        uint32_t b = ((((top >> 7) * 0x01020408u) >> 24) & 15u) << shift;
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) b |= __shfl_xor(b, o, 8);
        mine = lane == k ? b : mine;
    }
    if (in && lane < 6) reinterpret_cast<uint32_t *>(s.layer + lane * s.words)[id >> 3] = mine;
}

__global__ void __launch_bounds__(256) layer_bits_kernel(Scratch s)
{
    layer_bits(s, (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
}

// One word of a set, its row and its place: rows are w words apart, planes w n1 (x, y and z below
// stand for the sets' axes in their order).
struct Place {
    int64_t at, sy, sz;
    int wi, w, y, ny, z, nz;
    bool wall_x, wall_y, wall_z, ok;
};

__device__ __forceinline__ Place place_of(const Scratch &s, int64_t id)
{
    Place p;
    p.ok = id < s.words;
    p.at = p.ok ? id : 0;
    p.w = s.w;
    const int64_t row = p.at / s.w;
    p.wi = (int)(p.at - row * s.w);
    p.z = (int)(row / s.n1);
    p.y = (int)(row - (int64_t)p.z * s.n1);
    p.ny = s.n1;
    p.nz = s.n2;
    p.sy = s.w;
    p.sz = (int64_t)s.w * s.n1;
    p.wall_x = s.wall0;
    p.wall_y = s.wall1;
    p.wall_z = s.wall2;
    return p;
}

__device__ __forceinline__ uint64_t word_at(const uint64_t *set, int64_t at, int i, int n, bool wall)
{
    return (unsigned)i < (unsigned)n ? set[at] : (i >= n && wall ? ~0ull : 0ull);
}

// The word j rows away along y or z (out of the grid: free, or occupied past a partial axis).
__device__ __forceinline__ uint64_t word_y(const uint64_t *set, const Place &p, int j)
{
    return word_at(set, p.at + j * p.sy, p.y + j, p.ny, p.wall_y);
}
__device__ __forceinline__ uint64_t word_z(const uint64_t *set, const Place &p, int j)
{
    return word_at(set, p.at + j * p.sz, p.z + j, p.nz, p.wall_z);
}

// A word with the 32 bits before and after it in its row, lowest first.
struct Window {
    uint32_t w[4];
};

__device__ __forceinline__ Window window_at(const uint64_t *set, const Place &p, int64_t at, bool in, bool ones)
{
    if (!in) {
        const uint32_t v = ones ? ~0u : 0u;
        return Window{{v, v, v, v}};
    }
    const uint64_t c = set[at];
    const uint32_t before = p.wi > 0 ? (uint32_t)(set[at - 1] >> 32) : 0u;
    const uint32_t after = p.wi + 1 < p.w ? (uint32_t)set[at + 1] : (p.wall_x ? ~0u : 0u);
    return Window{{before, (uint32_t)c, (uint32_t)(c >> 32), after}};
}

__device__ __forceinline__ Window window_row(const uint64_t *set, const Place &p, bool along_z, int j)
{
    const int i = (along_z ? p.z : p.y) + j, n = along_z ? p.nz : p.ny;
    return window_at(set, p, p.at + j * (along_z ? p.sz : p.sy), (unsigned)i < (unsigned)n,
                     i >= n && (along_z ? p.wall_z : p.wall_y));
}

__device__ __forceinline__ void join(Window &a, const Window &b)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) a.w[i] |= b.w[i];
}

// The window's word dilated by K along x: bits joined with those up to K above and below, by
// shifts that double the reach.
template <int K>
__device__ __forceinline__ uint64_t smear(const Window &v)
{
    uint32_t r1 = v.w[1], r2 = v.w[2], r3 = v.w[3], l0 = v.w[0], l1 = v.w[1], l2 = v.w[2];
    auto step = [&](int n) {
        r1 |= __builtin_amdgcn_alignbit(r2, r1, n);
        r2 |= __builtin_amdgcn_alignbit(r3, r2, n);
        r3 |= r3 >> n;
        l2 |= __builtin_amdgcn_alignbit(l2, l1, 32 - n);
        l1 |= __builtin_amdgcn_alignbit(l1, l0, 32 - n);
        l0 |= l0 << n;
    };
    step(1);
    if constexpr (K == 2) step(1);
    if constexpr (K >= 3) step(2);
    if constexpr (K > 3) step(K - 3);
    return (uint64_t)(r1 | l1) | ((uint64_t)(r2 | l2) << 32);
}

// 64 counters of three bits.
struct Count {
    uint64_t b0, b1, b2;
    __device__ __forceinline__ void add(uint64_t x)
    {
        const uint64_t c = b0 & x, d = b1 & c;
        b0 ^= x;
        b1 ^= c;
        b2 ^= d;
    }
};

__device__ __forceinline__ uint64_t above(const Count &a, const Count &b)
{
    const uint64_t e2 = ~(a.b2 ^ b.b2), e1 = ~(a.b1 ^ b.b1);
    return (a.b2 & ~b.b2) | (e2 & ((a.b1 & ~b.b1) | (e1 & a.b0 & ~b.b0)));
}
__device__ __forceinline__ uint64_t pick(uint64_t m, uint64_t a, uint64_t b) { return (m & a) | (~m & b); }
__device__ __forceinline__ Count pick(uint64_t m, const Count &a, const Count &b)
{
    return Count{pick(m, a.b0, b.b0), pick(m, a.b1, b.b1), pick(m, a.b2, b.b2)};
}

// The widest free layer so far: its extent, its side and its axis (x 0, y 1, z 2; 3 with side 1:
// none).
struct Best {
    Count q;
    uint64_t side, a0, a1;
    __device__ __forceinline__ void offer(const Count &c, bool high, int axis)
    {
        const uint64_t m = above(c, q);
        q = pick(m, c, q);
        side = pick(m, high ? ~0ull : 0ull, side);
        a0 = pick(m, axis & 1 ? ~0ull : 0ull, a0);
        a1 = pick(m, axis & 2 ? ~0ull : 0ull, a1);
    }
    __device__ __forceinline__ void offer(const Best &o)
    {
        const uint64_t m = above(o.q, q);
        q = pick(m, o.q, q);
        side = pick(m, o.side, side);
        a0 = pick(m, o.a0, a0);
        a1 = pick(m, o.a1, a1);
    }
    __device__ __forceinline__ void load(const uint64_t *set, int64_t words, int64_t at)
    {
        const uint64_t *o = set + at;
        q = Count{o[0], o[words], o[2 * words]};
        side = o[3 * words];
        a0 = o[4 * words];
        a1 = o[5 * words];
    }
    __device__ __forceinline__ void store(uint64_t *set, int64_t words, int64_t at) const
    {
        uint64_t *o = set + at;
        o[0] = q.b0; o[words] = q.b1; o[2 * words] = q.b2;
        o[3 * words] = side; o[4 * words] = a0; o[5 * words] = a1;
    }
};

// One step of the dilations of an axis' two voxel layers within the planes along x and the rows
// (y or z): ta, tb hold the layers' rows up to K away.
template <int K>
__device__ __forceinline__ void plane_step(const uint64_t *a, const uint64_t *b, const Place &p, bool along_z, Window &ta,
                                           Window &tb, Count &qa, Count &qb, uint64_t *out)
{
    join(ta, window_row(a, p, along_z, -K));
    join(ta, window_row(a, p, along_z, K));
    join(tb, window_row(b, p, along_z, -K));
    join(tb, window_row(b, p, along_z, K));
    const uint64_t ca = smear<K>(ta), cb = smear<K>(tb);
    qa.add(~ca);
    qb.add(~cb);
    out[p.at] = ca | cb;
}

__device__ __forceinline__ void plane(const Scratch &s, const Place &p, int axis, uint64_t *out, Best &best)
{
    const bool along_z = axis == 1;
    const uint64_t *a = s.layer + 2 * axis * s.words, *b = a + s.words;
    Window ta = window_row(a, p, along_z, 0), tb = window_row(b, p, along_z, 0);
    Count qa{~a[p.at], 0, 0}, qb{~b[p.at], 0, 0};
    plane_step<1>(a, b, p, along_z, ta, tb, qa, qb, out);
    plane_step<2>(a, b, p, along_z, ta, tb, qa, qb, out + s.words);
    plane_step<3>(a, b, p, along_z, ta, tb, qa, qb, out + 2 * s.words);
    plane_step<4>(a, b, p, along_z, ta, tb, qa, qb, out + 3 * s.words);
    plane_step<5>(a, b, p, along_z, ta, tb, qa, qb, out + 4 * s.words);
    plane_step<6>(a, b, p, along_z, ta, tb, qa, qb, out + 5 * s.words);
    best.offer(qa, false, axis);
    best.offer(qb, true, axis);
}

// Layers perpendicular to z (kind, blockIdx.y, 0) and y (1), and the first half (along y) of those
// perpendicular to x (2).  A thread per word leaves a SIMD two waves on a 400^3 map, waiting for
// loads: three kinds of blocks instead of one thread doing all of it, and two in the next kernel,
// 26 + 30 us -> 22 + 19 (with the blocks of
// neighbouring words on one XCD; 22 + 26 without).
__device__ __forceinline__ void planes(const Scratch &s, const Place &p, int kind)
{
    if (kind < 2) {
        Best best{Count{0, 0, 0}, ~0ull, ~0ull, ~0ull};
        if (kind == 0) {
            plane(s, p, 2, s.cz, best);
            best.store(s.best, s.words, p.at);
        } else {
            plane(s, p, 1, s.cy, best);
            best.store(s.best_y, s.words, p.at);
        }
        return;
    }
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const uint64_t *set = s.layer + side * s.words;
        uint64_t t = set[p.at];
#pragma unroll
        for (int k = 1; k <= kSteps; ++k) {
            t |= word_y(set, p, -k) | word_y(set, p, k);
            s.yx[(side * kSteps + k - 1) * s.words + p.at] = t;
        }
    }
}

__global__ void __launch_bounds__(256) planes_kernel(Scratch s)
{
    const Place p = place_of(s, (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
    if (p.ok) planes(s, p, blockIdx.y);
}

// Layers perpendicular to x (the second half, along z; kind 0), and the cubes (1).
__device__ __forceinline__ void cubes(const Scratch &s, const Place &p, int kind)
{
    if (kind == 1) {
        Count d{~0ull, 0, 0};
#pragma unroll
        for (int k = 1; k <= kSteps; ++k) {
            const uint64_t *set = s.cz + (k - 1) * s.words;
            uint64_t t = set[p.at];
#pragma unroll
            for (int j = 1; j <= k; ++j) t |= word_z(set, p, -j) | word_z(set, p, j);
            d.add(~t);
        }
        uint64_t *c = s.cube + p.at;
        c[0] = d.b0; c[s.words] = d.b1; c[2 * s.words] = d.b2;
        s.full[p.at] = d.b0 & d.b1 & d.b2;
        return;
    }
    Best best, best_y;
    best.load(s.best, s.words, p.at);
    best_y.load(s.best_y, s.words, p.at);
    best.offer(best_y);
    Count q[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) q[side] = Count{~s.layer[side * s.words + p.at], 0, 0};
#pragma unroll
    for (int k = 1; k <= kSteps; ++k) {
        uint64_t all = 0;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const uint64_t *set = s.yx + (side * kSteps + k - 1) * s.words;
            uint64_t t = set[p.at];
#pragma unroll
            for (int j = 1; j <= k; ++j) t |= word_z(set, p, -j) | word_z(set, p, j);
            q[side].add(~t);
            all |= t;
        }
        s.cx[(k - 1) * s.words + p.at] = all;
    }
    best.offer(q[0], false, 0);
    best.offer(q[1], true, 0);
    best.store(s.best, s.words, p.at);
}

__global__ void __launch_bounds__(256) cubes_kernel(Scratch s)
{
    const Place p = place_of(s, (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
    if (p.ok) cubes(s, p, blockIdx.y);
}

// Extents (bit-sliced) of the slab of half thickness d (1 .. 3: masks t1, t2, t3) perpendicular to
// an axis: the dilated slabs one and two bricks along it join in.
struct Near5 {
    uint64_t c, n1, n2;                               // the word itself, its neighbours 1 and 2 away
};

__device__ __forceinline__ Near5 near_rows(const uint64_t *set, const Place &p, bool along_z)
{
    // (no wall: a slab is at most as thick as the cube, which ends at it)
    Near5 r;
    r.c = set[p.at];
    const int i = along_z ? p.z : p.y, n = along_z ? p.nz : p.ny;
    const int64_t st = along_z ? p.sz : p.sy;
    r.n1 = word_at(set, p.at - st, i - 1, n, false) | word_at(set, p.at + st, i + 1, n, false);
    r.n2 = word_at(set, p.at - 2 * st, i - 2, n, false) | word_at(set, p.at + 2 * st, i + 2, n, false);
    return r;
}

__device__ __forceinline__ Near5 near_bits(const uint64_t *set, const Place &p)
{
    const uint64_t c = set[p.at];
    const uint64_t before = p.wi > 0 ? set[p.at - 1] : 0ull, after = p.wi + 1 < p.w ? set[p.at + 1] : 0ull;
    Near5 r;
    r.c = c;
    r.n1 = (c << 1) | (before >> 63) | (c >> 1) | (after << 63);
    r.n2 = (c << 2) | (before >> 62) | (c >> 2) | (after << 62);
    return r;
}

__device__ __forceinline__ void slab_add(Count &q, const Near5 &v, uint64_t t1, uint64_t t2, uint64_t t3)
{
    const uint64_t s2 = v.c | v.n1, s3 = s2 | v.n2;
    q.add(~((t1 & v.c) | (t2 & s2) | (t3 & s3)));
}

// The bricks whose 27 neighbours by steps of n bricks (themselves included) have full cubes.  The
// grid's last row or brick stands for those past it (they are free, and of a cube there only the
// part that reaches into the grid matters).
template <int N>
__device__ __forceinline__ uint64_t far_bits(const Scratch &s, const Place &p)
{
    uint64_t c = ~0ull, before = ~0ull, after = ~0ull;
    const int db = p.wi > 0 ? -1 : 0, da = p.wi + 1 < p.w ? 1 : 0;
#pragma unroll
    for (int k = -N; k <= N; k += N)
#pragma unroll
        for (int j = -N; j <= N; j += N) {
            const int y = min(max(p.y + j, 0), p.ny - 1), z = min(max(p.z + k, 0), p.nz - 1);
            const uint64_t *v = s.full + p.wi + p.w * ((int64_t)y + (int64_t)p.ny * z);
            c &= v[0];
            before &= v[db];
            after &= v[da];
        }
    if (db == 0) before = (c & 1ull) ? ~0ull : 0ull;
    if (da == 0) after = (c >> 63) ? ~0ull : 0ull;
    return c & ((c >> N) | (after << (64 - N))) & ((c << N) | (before >> (64 - N)));
}

// The entries' bit planes, one word of 64 bricks per thread, written over sets that only the same
// thread still reads (the layers, then the best layers and the cubes).
constexpr int kEntryPlanes = 14;

__device__ __forceinline__ uint64_t *entry_plane(const Scratch &s, int k)
{
    return k < 6 ? s.layer + k * s.words : s.best + (k - 6) * s.words;
}

__device__ __forceinline__ void select(const Scratch &s, const Place &p)
{
    const uint64_t *c = s.cube + p.at;
    const Count d{c[0], c[s.words], c[2 * s.words]};
    const uint64_t t1 = d.b0 & ~d.b1 & ~d.b2, t2 = ~d.b0 & d.b1 & ~d.b2, t3 = d.b0 & d.b1 & ~d.b2;
    Count qx{~0ull, 0, 0}, qy = qx, qz = qx;
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
        slab_add(qx, near_bits(s.cx + k * s.words, p), t1, t2, t3);
        slab_add(qy, near_rows(s.cy + k * s.words, p, false), t1, t2, t3);
        slab_add(qz, near_rows(s.cz + k * s.words, p, true), t1, t2, t3);
    }
    // the widest slab, where it is wider than the cube
    const uint64_t yz = above(qz, qy);
    Count q = pick(yz, qz, qy);
    const uint64_t px = ~above(q, qx);
    q = pick(px, qx, q);
    const uint64_t use = (t1 | t2 | t3) & above(q, d);
    const uint64_t ax = use & px, ay = use & ~px & ~yz, az = use & ~px & yz;
    Count ex = pick(use & ~ax, q, d), ey = pick(use & ~ay, q, d), ez = pick(use & ~az, q, d);
    const uint64_t occ = s.layer[4 * s.words + p.at] | s.layer[5 * s.words + p.at];
    const uint64_t *h = s.best + p.at;
    const uint64_t h0 = h[0], h1 = h[s.words], h2 = h[2 * s.words], side = h[3 * s.words];
    uint64_t a0 = h[4 * s.words], a1 = h[5 * s.words];
    // from the sets' axes back to the grid's
    if (s.axis == 1) {
        const Count e = ex;
        ex = ey;
        ey = e;
        a0 ^= ~a1;                                    // 0 <-> 1
    } else if (s.axis == 2) {
        const Count e = ex;
        ex = ez;
        ez = e;
        a1 ^= ~a0;                                    // 0 <-> 2
    }
    const uint64_t far3 = far_bits<3>(s, p), far6 = far_bits<6>(s, p);
    // bits 1-3, 6-8, 11-13 of a free brick's entry; bits 8, 9, 10, 11-13 of an occupied one's; bit 15;
    // half extent 10, 13
    const uint64_t o[kEntryPlanes] = {ex.b0 & ~occ, ex.b1 & ~occ, ex.b2 & ~occ, ey.b0 & ~occ, ey.b1 & ~occ,
                                      pick(occ, side, ey.b2), occ & a0, occ & a1, pick(occ, h0, ez.b0),
                                      pick(occ, h1, ez.b1), pick(occ, h2, ez.b2), occ, far3, far6};
#pragma unroll
    for (int k = 0; k < kEntryPlanes; ++k) entry_plane(s, k)[p.at] = o[k];
}

__global__ void __launch_bounds__(256) select_kernel(Scratch s)
{
    const Place p = place_of(s, (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
    if (p.ok) select(s, p);
}

// The entries: a wave writes those of kExpandWords consecutive words (64 each), each lane picking its
// bit of every plane.  The planes' words come by scalar loads of several words at once: a word at a
// time, 14 loads of 8 bytes for 128 bytes of entries left the kernel waiting for them (43 us
// on a 400^3 map against 22;
// four words spill scalar registers: 33).
constexpr int kExpandWords = 2;

// Where the entry of the sets' brick (0, 0, 0) lies, and those one on along each axis.
struct BoxOut {
    uint16_t *box;
    uint32_t s0, s1, s2;
};

__global__ void __launch_bounds__(256) expand_kernel(Scratch s, BoxOut out)
{
    const uint32_t word0 = __builtin_amdgcn_readfirstlane((xcd_tile(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)) * kExpandWords);
    if (word0 >= (uint32_t)s.words) return;
    const uint32_t bits[kEntryPlanes] = {1u << 1, 1u << 2, 1u << 3, 1u << 6, 1u << 7, 1u << 8, 1u << 9, 1u << 10,
                                         1u << 11, 1u << 12, 1u << 13, kBoxOccupied, 0u, 0u};
    // (reads past the last word stay within the scratch: sets follow the planes)
    typedef const __attribute__((address_space(4))) uint64_t *ConstPtr;
    uint64_t v[kEntryPlanes][kExpandWords];
#pragma unroll
    for (int k = 0; k < kEntryPlanes; ++k) {
        const ConstPtr plane = (ConstPtr)(uintptr_t)(entry_plane(s, k) + word0);
#pragma unroll
        for (int i = 0; i < kExpandWords; ++i) v[k][i] = plane[i];
    }
    uint32_t row = word0 / (uint32_t)s.w, wi = word0 - row * (uint32_t)s.w;
#pragma unroll
    for (int i = 0; i < kExpandWords; ++i) {
        if (word0 + i >= (uint32_t)s.words) return;
        uint32_t e = 0;
#pragma unroll
        for (int k = 0; k < 12; ++k) e |= __builtin_amdgcn_inverse_ballot_w64(v[k][i]) ? bits[k] : 0u;
        e = __builtin_amdgcn_inverse_ballot_w64(v[12][i]) ? box_extents(10, 10, 10) : e;
        e = __builtin_amdgcn_inverse_ballot_w64(v[13][i]) ? box_extents(13, 13, 13) : e;
        const int x = (int)wi * 64 + (int)(threadIdx.x & 63);
        if (x < s.n0) {
            // (words along x: the planes' rows follow one another)
            const uint32_t z = s.axis ? row / (uint32_t)s.n1 : 0u, y = row - z * (uint32_t)s.n1;
            const uint32_t mask = s.mask.at[row * s.mask.pitch + x];              // 0 for a free brick
            out.box[x * out.s0 + y * out.s1 + z * out.s2] = (uint16_t)(e | mask);
        }
        if (++wi == (uint32_t)s.w) {
            wi = 0;
            ++row;
        }
    }
}

// Without scratch, after the single-brick entries: free cubes, in place and doubling.  The first step
// gives half extent 2 to the free bricks whose 26 neighbours are free; a later one gives half
// extent `to` to those whose eight neighbours `step` bricks away along every axis have at least
// `from` (their cubes cover the wider one).  An entry only grows, and stays free or occupied, so it does
// not matter whether a neighbour is read before or after it has grown in the same step.
// (65,536 rays from the middle of 400^3 voxels, 1 in 10,000 occupied: 64 us by single-brick boxes, 29
// with these, 27 with the extents.  The upload without scratch takes 576 us, of which 115 are not
// these; 208 with scratch.)
struct Widen {
    int32_t from, step, to;
};
constexpr Widen kWiden[] = {{1, 1, 2}, {2, 1, 3}, {3, 2, 5}, {5, 4, 9}};

__global__ void __launch_bounds__(256) widen_kernel(MapView m, uint16_t *box, Widen g)
{
    const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= (uint64_t)m.nbx * m.nby * m.nbz) return;
    auto entry = [&](uint64_t at) { return (uint32_t)__hip_atomic_load(box + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    const uint32_t own = entry(id);
    // (all three extents of an entry are the same here)
    if (own >= kBoxOccupied || (own & 31u) < 2u * (uint32_t)g.from) return;
    const uint32_t row = (uint32_t)(id / (uint32_t)m.nbx);
    const int x = (int)(id - (uint64_t)row * m.nbx), z = (int)(row / (uint32_t)m.nby), y = (int)(row - (uint32_t)z * m.nby);
    // past a partial axis lie voxels without entries; past the others, where everything is free, the
    // last brick stands for those beyond it (of a cube there only the part in the grid matters)
    if ((2 * m.nbx < m.nx && x + g.step >= m.nbx) || (2 * m.nby < m.ny && y + g.step >= m.nby) ||
        (2 * m.nbz < m.nz && z + g.step >= m.nbz))
        return;
    const int by = g.from == 1 ? 1 : 2;                       // the first step looks at the bricks between too
    for (int c = -1; c <= 1; c += by)
        for (int b = -1; b <= 1; b += by)
            for (int a = -1; a <= 1; a += by) {
                const int i = min(max(x + a * g.step, 0), m.nbx - 1), j = min(max(y + b * g.step, 0), m.nby - 1),
                          k = min(max(z + c * g.step, 0), m.nbz - 1);
                const uint32_t e = entry((uint64_t)i + (uint64_t)m.nbx * ((uint64_t)j + (uint64_t)m.nby * k));
                if (e >= kBoxOccupied || (e & 31u) < 2u * (uint32_t)g.from) return;
            }
    const uint32_t to = (uint32_t)g.to;
    __hip_atomic_store(box + id, (uint16_t)box_extents(to, to, to), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

template <int DT, int W, bool UNIT>
void launch_bricks(const BoxArgs &a, const BoxMask &mask, hipStream_t s)
{
    using T = typename Voxel<DT>::T;
    const MapView &m = a.map;
    T *dst = DT == RMPC_OCC_U8 || a.src == m.data ? nullptr : static_cast<T *>(const_cast<void *>(m.data));
    const int64_t n = (int64_t)((m.nbx + W - 1) / W) * m.nby * m.nbz;
    if (n > 0)
        brick_kernel<DT, W, UNIT><<<blocks_for(n), 256, 0, s>>>(m, static_cast<const T *>(a.src), dst, mask,
                                                               const_cast<uint16_t *>(m.box));
    if (dst && m.partial) {
        const uint32_t row_blocks = 2 * m.nbx < m.nx ? blocks_for((int64_t)m.ny * m.nz) : 0u;
        const uint32_t y_rows = 2 * m.nby < m.ny ? (uint32_t)m.nz : 0u, z_rows = 2 * m.nbz < m.nz ? (uint32_t)m.ny : 0u;
        if (row_blocks + y_rows + z_rows)
            copy_rest_kernel<DT><<<row_blocks + y_rows + z_rows, 256, 0, s>>>(m, static_cast<const T *>(a.src), dst, row_blocks,
                                                                             y_rows);
    }
}

void launch_extents(const MapView &m, const Scratch &p, hipStream_t s)
{
    if (p.words == 0) return;
    // every launch's blocks in eight equal runs of words, one per XCD: a kernel's reads of the set
    // before and of rows above and below find most of them in their own L2
    auto blocks = [](int64_t n) { return blocks_for((n + 2047) / 2048 * 2048); };
    const uint32_t st[3] = {1u, (uint32_t)m.nbx, (uint32_t)m.nbx * (uint32_t)m.nby};
    const BoxOut out{const_cast<uint16_t *>(m.box), st[p.axis], st[p.axis == 1 ? 0 : 1], st[p.axis == 2 ? 0 : 2]};
    layer_bits_kernel<<<blocks(16 * p.words), 256, 0, s>>>(p);
    planes_kernel<<<dim3(blocks(p.words), 3), 256, 0, s>>>(p);
    cubes_kernel<<<dim3(blocks(p.words), 2), 256, 0, s>>>(p);
    select_kernel<<<blocks(p.words), 256, 0, s>>>(p);
    expand_kernel<<<blocks((p.words + kExpandWords - 1) / kExpandWords * 64), 256, 0, s>>>(p, out);
}

void launch_widen(const MapView &m, hipStream_t s)
{
    const int64_t n = (int64_t)m.nbx * m.nby * m.nbz;
    if (n == 0) return;
    for (const Widen &g : kWiden) widen_kernel<<<blocks_for(n), 256, 0, s>>>(m, const_cast<uint16_t *>(m.box), g);
}

template <int DT>
void launch_boxes_dt(const BoxArgs &a, hipStream_t s)
{
    using T = typename Voxel<DT>::T;
    const MapView &m = a.map;
    const bool wide = m.nx % 4 == 0 && reinterpret_cast<uintptr_t>(a.src) % (4 * sizeof(T)) == 0;
    if (!a.scratch) {
        if (wide) launch_bricks<DT, 2, true>(a, BoxMask{}, s);
        else launch_bricks<DT, 1, true>(a, BoxMask{}, s);
        launch_widen(m, s);
        return;
    }
    const Scratch p = scratch_at(m, a.scratch);
    if (wide) launch_bricks<DT, 2, false>(a, p.mask, s);
    else launch_bricks<DT, 1, false>(a, p.mask, s);
    launch_extents(m, p, s);
}

}  // namespace

BoxMask box_mask(const MapView &m, uint8_t *scratch)
{
    const int axis = word_axis(m);
    const uint32_t n[3] = {(uint32_t)m.nbx, (uint32_t)m.nby, (uint32_t)m.nbz}, pitch = (n[axis] + 3u) & ~3u;
    const int a1 = axis == 1 ? 0 : 1, a2 = axis == 2 ? 0 : 2;
    uint32_t st[3];
    st[axis] = 1;
    st[a1] = pitch;
    st[a2] = pitch * n[a1];
    return BoxMask{scratch, st[0], st[1], st[2], pitch, ((size_t)st[a2] * n[a2] + 255) / 256 * 256};
}

size_t box_scratch_bytes(const MapView &m)
{
    const int64_t words = set_words(m, word_axis(m));
    return words == 0 ? 0 : box_mask(m, nullptr).bytes + (size_t)(8 * kSets * words);
}

void launch_cell_boxes(const MapView &m, uint8_t *scratch, hipStream_t s) { launch_extents(m, scratch_at(m, scratch), s); }

hipError_t launch_unit_boxes(const MapView &m, hipStream_t s)
{
    launch_widen(m, s);
    return hipGetLastError();
}

hipError_t launch_map_boxes(const BoxArgs &a, hipStream_t s)
{
    switch (a.map.dtype) {
    case RMPC_TSDF_F32: launch_boxes_dt<RMPC_TSDF_F32>(a, s); break;
    case RMPC_TSDF_F16: launch_boxes_dt<RMPC_TSDF_F16>(a, s); break;
    default: launch_boxes_dt<RMPC_OCC_U8>(a, s); break;
    }
    return hipGetLastError();
}

}  // namespace rmpc
