// sparse.hip -- the raycast-and-policy query on a sparse block map: the single-query and debug
// kernels over the walk of rmpc_sparse.h, and the kernels that build a sparse map's occupancy
// masks, table flags, index and brick entries at upload.

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rmpc_device.h"
#include "rmpc_kernels.h"
#include "rmpc_sparse.h"
#include "rmpc_walk.h"

namespace rmpc {

namespace {

template <int K, int SV>
__global__ void __launch_bounds__(kBlock, 2) sparse_rmp_kernel(RayArgs A)
{
    __shared__ __align__(16) float lds[kReduceLdsWords];
    sparse_tile<K, SV>(A, xcd_tile(blockIdx.x, gridDim.x), gridDim.x,
                   single_slots(A.partials, A.ticket, A.result, A.done, A.seq), lds);
}

// Per-ray outputs: the hit as slot * 512 + (x + 8 y + 64 z within the block), -1 on a miss.
template <int K, int SV>
__global__ void __launch_bounds__(kBlock, 2) sparse_trace_kernel(RayArgs A)
{
    int slot0;
    bool occ0;
    uint64_t m0[kLayers];
    const bool in_coll = start_block(A, slot0, occ0, m0);
    const int S = A.segments;
    const int p = blockIdx.x * kBlock + threadIdx.x;
    const int j = p < A.n_list * S ? p / S : 0;
    const int seg = p & (S - 1);
    const float4 rr = load_ray(A.rays, j);
    const int i = __float_as_int(rr.w);
    const bool valid = p < A.n_list * S && i < A.n_rays;
    if (in_coll) {
        if (valid && seg == 0) {
            A.dbg_hit[i] = slot0 * kBlockVoxels + (A.v0[0] & 7) + 8 * (A.v0[1] & 7) + 64 * (A.v0[2] & 7);
            A.dbg_dist[i] = 0.0;
            A.dbg_flags[i] = (uint8_t)(A.start_flags | kRayInCollision);
            if (A.dbg_visits) A.dbg_visits[i] = 1;
        }
        return;
    }
    const SOut o = sparse_trace<K>(A, valid, seg, S, rr.x, rr.y, rr.z, slot0, occ0, m0);
    // the ray's visit count is the sum over its group
    int v = o.visits_lane;
    for (int off = 1; off < S; off <<= 1) v += __shfl_xor(v, off, kWave);
    if (o.report) {
        A.dbg_hit[i] = o.hit ? o.hit_slot * kBlockVoxels + o.hit_local : -1;
        A.dbg_dist[i] = o.hit ? sparse_distance<SV>(A, rr.x, rr.y, rr.z, o.d) : o.d;
        A.dbg_flags[i] = (uint8_t)o.flags;
        if (A.dbg_visits) A.dbg_visits[i] = v;
    }
}

// What an upload writes of a map's index, all null and zero for a map without one.
struct IndexBuild {
    uint32_t *index;                                      // cells entries
    int64_t cells;
    uint16_t *bricks;                                     // 64 per slot
    BoxMask mask;                                         // the cells' occupancy
    uint16_t *box;                                        // the cells' boxes
    uint64_t *bits;                                       // per slot a bit per brick
};

// Occupancy words of every slot (thread: one slot's layer) from its stored values.  The same launch
// clears the index and its cells' occupancy: an upload of few blocks is as long as its launches (with
// 13 of them, two fills of memory among them, one of 16 blocks took 87 us, with 8 76).
template <int DT>
__global__ void __launch_bounds__(256) sparse_mask_kernel(SparseView v, uint64_t *occ, IndexBuild b)
{
    using T = typename Voxel<DT>::T;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int64_t i = t; i < b.cells; i += step) b.index[i] = 0u;
    for (int64_t i = t; i < (int64_t)(b.mask.bytes / 8); i += step) reinterpret_cast<uint64_t *>(b.mask.at)[i] = 0ull;
    if (t >= (int64_t)v.n_slots * kLayers) return;
    const T *vals = static_cast<const T *>(v.values) + (size_t)t * 64;   // layer z of slot t / 8
    uint64_t w = 0;
    for (int k = 0; k < 64; ++k) w |= Voxel<DT>::occ(vals[k]) ? 1ull << k : 0ull;
    occ[t] = w;
}

// Table entry i: whether its slot's occupancy has any bit set; in the index an occupied block's slot,
// and 255 in the cells' occupancy.
__device__ __forceinline__ void table_entry(const SparseView &v, HashEntry *table, const IndexBuild &b, uint32_t i)
{
    if (i > v.table_mask) return;
    HashEntry &e = table[i];
    if (e.key == kEmptyKey || e.slot < 0 || e.slot >= v.n_slots) return;
    uint64_t any = 0;
    for (int k = 0; k < kLayers; ++k) any |= v.occ[(size_t)e.slot * kLayers + k];
    e.occupied = any != 0 ? 1u : 0u;
    if (any == 0 || !b.index) return;
    const uint32_t bits = (1u << kBlockCoordBits) - 1u;
    const int x = (int)((uint32_t)e.key & bits) - kBlockCoordBias - v.lo[0];
    const int y = (int)((uint32_t)(e.key >> 21) & bits) - kBlockCoordBias - v.lo[1];
    const int z = (int)((uint32_t)(e.key >> 42) & bits) - kBlockCoordBias - v.lo[2];
    b.index[x + v.nb[0] * (y + (int64_t)v.nb[1] * z)] = kBlockOccupied | (uint32_t)e.slot;
    b.mask.at[x * b.mask.sx + y * b.mask.sy + z * b.mask.sz] = 255u;
}

// A slot's 64 bricks (a wave): their voxels' occupancy, and one bit each in bits[slot].
__device__ __forceinline__ void brick_masks(const SparseView &v, const IndexBuild &b, int slot, int brick)
{
    if (slot >= v.n_slots) return;
    const uint64_t *w = v.occ + (size_t)slot * kLayers + 2 * (brick >> 4);
    const int at = 2 * (brick & 3) + 16 * ((brick >> 2) & 3);
    uint32_t mask = 0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
        mask |= (uint32_t)(((w[dz] >> at) & 3u) | (((w[dz] >> (at + 8)) & 3u) << 2)) << (4 * dz);
    const uint64_t any = __ballot(mask != 0u);
    b.bricks[(size_t)slot * 64 + brick] = (uint16_t)mask;
    if (brick == 0) b.bits[slot] = any;
}

// The table's entries (the first table_blocks blocks, a thread each), and the slots' bricks.
__global__ void __launch_bounds__(256) sparse_table_kernel(SparseView v, HashEntry *table, IndexBuild b, uint32_t table_blocks)
{
    if (blockIdx.x < table_blocks) table_entry(v, table, b, blockIdx.x * 256 + threadIdx.x);
    else brick_masks(v, b, (int)(blockIdx.x - table_blocks) * 4 + (int)(threadIdx.x >> 6), threadIdx.x & 63);
}

// A free block's box in the index, and the brick entries of an occupied one (a wave for each of the
// index's blocks; one that reads a neighbour's entry asks only whether it is occupied, and its slot,
// which stay): an occupied brick's voxels, without a free layer; around a free one the free cube, half extent 1 .. 5 (what the 27 blocks around tell),
// or where it is narrow (below 3) the widest slab one brick thick.
__global__ void __launch_bounds__(256) brick_boxes_kernel(SparseView v, IndexBuild build)
{
    __shared__ uint32_t rows[4][144];                     // 12 bricks along x, for y and z from 4 before the block on
    const int64_t n = (int64_t)v.nb[0] * v.nb[1] * v.nb[2];
    const int64_t at = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const uint32_t e = at < n ? build.index[at] : 0u;
    const bool mine = (e & kBlockOccupied) != 0u;
    if (!mine && at < n && lane == 0) build.index[at] = build.box[at];
    uint32_t *row = rows[threadIdx.x >> 6];
    if (mine) {
        const int64_t yz = at / v.nb[0];
        const int x = (int)(at - yz * v.nb[0]), z = (int)(yz / v.nb[1]), y = (int)(yz - (int64_t)z * v.nb[1]);
        // lanes 0 .. 26: a neighbouring block's bricks
        uint64_t near = 0;
        if (lane < 27) {
            const int px = x + lane % 3 - 1, py = y + lane / 3 % 3 - 1, pz = z + lane / 9 - 1;
            if ((unsigned)px < (unsigned)v.nb[0] && (unsigned)py < (unsigned)v.nb[1] && (unsigned)pz < (unsigned)v.nb[2]) {
                const uint32_t q = build.index[px + v.nb[0] * (py + (int64_t)v.nb[1] * pz)];
                if (q & kBlockOccupied) near = build.bits[q & ~kBlockOccupied];
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int r = lane + 64 * k, ry = r % 12, rz = min(r / 12, 11), from = 3 * (ry >> 2) + 9 * (rz >> 2);
            const int s = 4 * (ry & 3) + 16 * (rz & 3);
            uint32_t w = 0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const uint64_t m = __shfl((unsigned long long)near, from + i, 64);
                w |= (uint32_t)((m >> s) & 15u) << (4 * i);
            }
            if (r < 144) row[r] = w;
        }
    }
    __syncthreads();
    if (!mine) return;
    uint16_t *out = build.bricks + ((size_t)(e & ~kBlockOccupied) * 64 + lane);
    const uint32_t mask = *out;
    if (mask) {
        *out = (uint16_t)(kBoxOccupied | kBoxNoLayer | mask);
        return;
    }
    // nearest occupied brick, in bricks, at most 5: at all, and within the layer of bricks
    // perpendicular to each axis
    const int i = 4 + (lane & 3), j = 4 + ((lane >> 2) & 3), k = 4 + (lane >> 4);
    int d = 5, dx = 5, dy = 5, dz = 5;
    for (int c = -4; c <= 4; ++c)
        for (int b = -4; b <= 4; ++b) {
            const uint32_t w = row[(j + b) + 12 * (k + c)];
            const uint32_t right = w >> i, left = w << (31 - i);
            const int ring = max(abs(b), abs(c));
            const int r = max(ring, min(right ? __builtin_ctz(right) : 5, left ? __builtin_clz(left) : 5));
            d = min(d, r);
            dz = c == 0 ? min(dz, r) : dz;
            dy = b == 0 ? min(dy, r) : dy;
            dx = right & 1u ? min(dx, ring) : dx;
        }
    uint32_t o = box_extents(d, d, d);
    if (d < 3 && max(dx, max(dy, dz)) > d)
        o = dz >= dx && dz >= dy ? box_extents(dz, dz, 1) : (dy >= dx ? box_extents(dy, 1, dy) : box_extents(1, dx, dx));
    *out = (uint16_t)o;
}

MapView index_cells(const SparseView &v)
{
    MapView m{};
    m.nbx = v.nb[0]; m.nby = v.nb[1]; m.nbz = v.nb[2];
    m.nx = 2 * m.nbx; m.ny = 2 * m.nby; m.nz = 2 * m.nbz;
    return m;
}

size_t round256(size_t n) { return (n + 255) / 256 * 256; }

template <int K, int SV>
hipError_t launch_sparse_k(const RayArgs &A, hipStream_t s, bool debug, hipEvent_t e0, hipEvent_t e1)
{
    const dim3 g((A.n_list * A.segments + kBlock - 1) / kBlock), blk(kBlock);
    if (debug) {
        sparse_trace_kernel<K, SV><<<g, blk, 0, s>>>(A);
    } else if (e0) {
        hipExtLaunchKernelGGL(sparse_rmp_kernel<K, SV>, g, blk, 0, s, e0, e1, 0, A);
    } else {
        sparse_rmp_kernel<K, SV><<<g, blk, 0, s>>>(A);
    }
    return hipGetLastError();
}

template <int K>
hipError_t launch_sparse_sv(const RayArgs &A, hipStream_t s, bool debug, hipEvent_t e0, hipEvent_t e1)
{
    if (!A.subvoxel) return launch_sparse_k<K, kSvNone>(A, s, debug, e0, e1);
    if (A.sp.dtype == RMPC_TSDF_F32) return launch_sparse_k<K, kSvF32>(A, s, debug, e0, e1);
    return launch_sparse_k<K, kSvF16>(A, s, debug, e0, e1);
}

}  // namespace

hipError_t launch_sparse(const RayArgs &A, hipStream_t s, bool debug, hipEvent_t e0, hipEvent_t e1)
{
    if (A.sparse == 2) return launch_raycast(A, s, debug, e0, e1);
    switch (A.lookahead) {
    case 4: return launch_sparse_sv<4>(A, s, debug, e0, e1);
    case 16: return launch_sparse_sv<16>(A, s, debug, e0, e1);
    default: return launch_sparse_sv<8>(A, s, debug, e0, e1);
    }
}

// Scratch: the occupancy and bit sets of the index's boxes, their entries, the bricks' bits.
size_t sparse_index_scratch_bytes(const SparseView &v)
{
    const size_t cells = (size_t)v.nb[0] * v.nb[1] * v.nb[2];
    return round256(box_scratch_bytes(index_cells(v))) + round256(sizeof(uint16_t) * cells) + sizeof(uint64_t) * (size_t)v.n_slots;
}

hipError_t launch_sparse_build(const SparseView &v, HashEntry *table, uint8_t *scratch, hipStream_t s)
{
    uint64_t *occ = const_cast<uint64_t *>(v.occ);
    MapView m{};
    IndexBuild b{};
    if (v.index) {
        m = index_cells(v);
        b.index = const_cast<uint32_t *>(v.index);
        b.cells = (int64_t)v.nb[0] * v.nb[1] * v.nb[2];
        b.bricks = const_cast<uint16_t *>(v.bricks);
        b.mask = box_mask(m, scratch);
        b.box = reinterpret_cast<uint16_t *>(scratch + round256(box_scratch_bytes(m)));
        b.bits = reinterpret_cast<uint64_t *>(reinterpret_cast<uint8_t *>(b.box) + round256(sizeof(uint16_t) * (size_t)b.cells));
        m.box = b.box;
    }
    const unsigned n = (unsigned)((v.n_slots * kLayers + 255) / 256);
    switch (v.dtype) {
    case RMPC_TSDF_F32: sparse_mask_kernel<RMPC_TSDF_F32><<<n, 256, 0, s>>>(v, occ, b); break;
    case RMPC_TSDF_F16: sparse_mask_kernel<RMPC_TSDF_F16><<<n, 256, 0, s>>>(v, occ, b); break;
    default: sparse_mask_kernel<RMPC_OCC_U8><<<n, 256, 0, s>>>(v, occ, b); break;
    }
    const uint32_t table_blocks = v.table_mask / 256 + 1, slot_blocks = v.index ? ((uint32_t)v.n_slots + 3) / 4 : 0u;
    sparse_table_kernel<<<table_blocks + slot_blocks, 256, 0, s>>>(v, table, b, table_blocks);
    if (v.index) {
        launch_cell_boxes(m, scratch, s);
        brick_boxes_kernel<<<(unsigned)((b.cells + 3) / 4), 256, 0, s>>>(v, b);
    }
    return hipGetLastError();
}

}  // namespace rmpc
