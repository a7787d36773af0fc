// raycast.hip -- the fused raycast-and-policy kernel (Sec. III-E, III-F), its debug twin, the
// batch kernel and the LiDAR scan kernel (Sec. III-G).
//
// Each ray's parameter range [0, max_range / h] is split into S segments that S adjacent
// lanes walk at the same time (S = 1, 2, 4, 8 or 16): the first hit along a ray is the hit of
// the lowest segment that finds one, so a query's critical path is one segment long instead of
// one ray.  Inside a segment a lane walks from free box to free box (rmpc_dense.h) and stops at
// the first occupied voxel, at its segment's end, at max_range or at the grid's surface.  A wave
// ballot after every step stops lanes whose ray already has a hit in a lower segment.  The lane
// holding the ray's hit evaluates the obstacle policy of Sec. III-C in registers and adds it to
// compensated float32 sums; the last block to finish resolves in float64.

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rmpc_dense.h"
#include "rmpc_device.h"
#include "rmpc_kernels.h"
#include "rmpc_sparse.h"
#include "rmpc_walk.h"

namespace rmpc {

namespace {

// Slot of the block of voxel (vx, vy, vz) if it has an occupied voxel, else -1.
__device__ __forceinline__ int indexed_slot(const SparseView &S, int vx, int vy, int vz)
{
    const uint32_t ix = (uint32_t)((vx >> kBlockLog2) - S.lo[0]), iy = (uint32_t)((vy >> kBlockLog2) - S.lo[1]),
                   iz = (uint32_t)((vz >> kBlockLog2) - S.lo[2]);
    if (ix >= (uint32_t)S.nb[0] || iy >= (uint32_t)S.nb[1] || iz >= (uint32_t)S.nb[2]) return -1;
    const uint32_t e = S.index[ix + (uint32_t)S.nb[0] * (iy + __umul24(iz, (uint32_t)S.nb[1]))];
    return e & kBlockOccupied ? (int)(e & ~kBlockOccupied) : -1;
}

// What a trace reports for an occupied voxel: its index in the grid, on a sparse map its slot and
// its place in the block.
template <int DT>
__device__ __forceinline__ int hit_index(const RayArgs &A, int vx, int vy, int vz)
{
    if constexpr (is_indexed(DT))
        return indexed_slot(A.sp, vx, vy, vz) * kBlockVoxels + (vx & 7) + 8 * (vy & 7) + 64 * (vz & 7);
    return vx + A.map.nx * (vy + A.map.ny * vz);
}

// The start voxel is occupied: every ray hits at distance 0 (same address for all lanes).
template <int DT>
__device__ __forceinline__ bool start_occupied(const RayArgs &A)
{
    if constexpr (is_indexed(DT)) {
        const SparseView &S = A.sp;
        const int slot = indexed_slot(S, A.v0[0], A.v0[1], A.v0[2]);
        return slot >= 0 && ((S.occ[(size_t)slot * kLayers + (A.v0[2] & 7)] >> ((A.v0[0] & 7) + 8 * (A.v0[1] & 7))) & 1ull) != 0;
    }
    const MapView &m = A.map;
    const int bx = A.v0[0] >> kBrickLog2, by = A.v0[1] >> kBrickLog2, bz = A.v0[2] >> kBrickLog2;
    if constexpr (DT != RMPC_OCC_U8 && !is_indexed(DT)) {
        if (bx >= m.nbx || by >= m.nby || bz >= m.nbz)
            return Voxel<DT>::occ(static_cast<const typename Voxel<DT>::T *>(m.data)[(uint32_t)A.lin0]);
    }
    const uint32_t e = m.box[(uint32_t)bx + (uint32_t)m.nbx * ((uint32_t)by + (uint32_t)m.nby * (uint32_t)bz)];
    const int at = (A.v0[0] & 1) | ((A.v0[1] & 1) << 1) | ((A.v0[2] & 1) << 2);
    return (e & kBoxOccupied) != 0u && ((e >> at) & 1u) != 0u;
}

// Per-ray outcome, valid in the lane that reports the ray (its hit segment, else segment 0).
struct RayOut {
    bool report;
    bool hit;
    double d;
    uint32_t flags;
    int visits_lane;                  // the ray's visit count in one lane of its group, else 0
    int fx, fy, fz;                   // the hit voxel (debug)
};

// Walk one ray with the S lanes of its group; every lane of the wave must call this.
template <int DT, bool PART>
__device__ __forceinline__ RayOut trace_group(const RayArgs &A, bool valid, int seg, int S,
                                              float rx, float ry, float rz)
{
    const BoxRay R = box_ray<DT>(A, rx, ry, rz);
    BoxWalk w;
    bool last;
    float t_lo, t_hi, t_first;
    const bool ran = box_segment(A, R, seg, S, w, last, t_lo, t_hi, t_first) && valid;
    const float t_end = fminf(R.t_exit, last ? t_lo : t_hi);

    const int lane = threadIdx.x & (kWave - 1);
    const int base = lane & ~(S - 1);
    const uint64_t seg_bits = (1ull << S) - 1ull;        // S <= 16
    const uint64_t lower = ((1ull << seg) - 1ull) << base;
    // kSteps steps between looks at the other lanes; a lane leaves them as soon as it stops
    constexpr int kSteps = 4;
    w.left = ran ? 0 : kWalkEnded;
    for (;;) {
        if (__ballot(w.left == kWalkHit) & lower) w.left = kWalkEnded;   // a lower segment already hit
        if (!__any(w.left >= 0)) break;
        if (w.left >= 0) w.left = kSteps;
        while (w.left > 0) box_step<DT, PART>(A, R, w, t_end, t_lo, t_hi, t_first);
    }
    const bool hit = w.left == kWalkHit;
    const BoxResult e = box_finish(A, R, w, last, t_lo, t_hi);
    // combine the group: the lowest segment with a hit owns the ray; the lowest segment whose
    // walk ended holds the ray's last voxel
    const uint64_t gh = (__ballot(hit) >> base) & seg_bits;
    const int h = gh ? __ffsll((unsigned long long)gh) - 1 : S;
    const uint64_t ge = (__ballot(ran && e.ended) >> base) & seg_bits;
    const int t = ge ? __ffsll((unsigned long long)ge) - 1 : S;
    const bool keep = ran && seg <= h;
    RayOut o;
    // voxels entered, start voxel included: every step changes one coordinate by one toward
    // the ray's direction, so the count follows from the first and the last voxel
    o.visits_lane = valid && seg == t ? 1 + abs(e.fx - A.v0[0]) + abs(e.fy - A.v0[1]) + abs(e.fz - A.v0[2]) : 0;
    const uint64_t tm = (__ballot(keep && w.tie) >> base) & seg_bits;
    const uint64_t rm = (__ballot(keep && e.rtie) >> base) & seg_bits;
    o.report = valid && seg == (h < S ? h : 0);
    o.hit = hit && seg == h;
    o.fx = e.fx; o.fy = e.fy; o.fz = e.fz;
    o.d = o.hit ? e.d : __builtin_huge_val();
    o.flags = A.start_flags | (tm ? kRayTie : 0u) | (rm ? kRayRangeTie : 0u);
    return o;
}

// The stored value of voxel (i, j, k) of a dense map, the indices clamped into the grid, as
// float64 (exact for float32 and binary16): the field reader of sub-voxel distances.
template <int DT>
struct DenseField {
    const typename Voxel<DT>::T *data;
    int nx, ny, nz;
    __device__ __forceinline__ double operator()(int i, int j, int k) const
    {
        i = i < 0 ? 0 : (i >= nx ? nx - 1 : i);
        j = j < 0 ? 0 : (j >= ny ? ny - 1 : j);
        k = k < 0 ? 0 : (k >= nz ? nz - 1 : k);
        const typename Voxel<DT>::T v = data[(uint32_t)i + (uint32_t)nx * ((uint32_t)j + (uint32_t)ny * (uint32_t)k)];
        if constexpr (DT == RMPC_TSDF_F32) return (double)v;
        else return (double)__builtin_bit_cast(_Float16, v);
    }
};

template <int DT>
__device__ __forceinline__ double subvoxel_distance(const RayArgs &A, float rx, float ry, float rz, double d)
{
    if constexpr (DT == kIndexedF32) return sparse_distance<kSvF32>(A, rx, ry, rz, d);
    else if constexpr (DT == kIndexedF16) return sparse_distance<kSvF16>(A, rx, ry, rz, d);
    else {
        const DenseField<DT> f{static_cast<const typename Voxel<DT>::T *>(A.map.data), A.map.nx, A.map.ny, A.map.nz};
        return subvoxel_at(A, f, rx, ry, rz, d);
    }
}

// One 256-lane tile of a map query: lane -> (ray position, segment).  Waves stay whole (the
// traversal uses wave-wide ballots); lanes past the end, or whose list entry is >= n_rays,
// take part as idle members.  A lane traces first and only then holds accumulators.
template <int DT, bool PART>
__device__ __forceinline__ void ray_tile(const RayArgs &A, int tile, int n_tiles, const FinishSlots &F,
                                         float *lds)
{
    const bool in_coll = start_occupied<DT>(A);
    const int S = A.segments;
    const int p = tile * kBlock + threadIdx.x;
    const int j = p < A.n_list * S ? p / S : 0;
    const int seg = p & (S - 1);
    const float4 rr = load_ray(A.rays, j);
    const bool valid = p < A.n_list * S && __float_as_int(rr.w) < A.n_rays;
    const float rx = rr.x, ry = rr.y, rz = rr.z;
    Acc acc;
    acc.zero();
    if (in_coll) {
        if (valid && seg == 0) {
            acc.visits = 1;
            acc.n_hit = 1;
            acc.n_contrib = contributes(A, rx, ry, rz, 0.0);
            policy_set(A.pol, rx, ry, rz, 0.0f, acc);
        }
    } else {
        const RayOut o = trace_group<DT, PART>(A, valid, seg, S, rx, ry, rz);
        acc.visits = o.visits_lane;
        if (o.report) {
            acc.n_tie = (o.flags & kRayTie) != 0;
            if (o.hit) {
                double d = o.d;
                if constexpr (DT != RMPC_OCC_U8 && DT != kIndexed)
                    if (A.subvoxel) d = subvoxel_distance<DT>(A, rx, ry, rz, d);
                acc.n_hit = 1;
                acc.n_contrib = contributes(A, rx, ry, rz, d);
                policy_set(A.pol, rx, ry, rz, (float)d, acc);
            }
        }
    }
    grid_finish(acc, tile, n_tiles, F, A.rank_tol, A.n_rays, in_coll ? RMPC_Q_IN_COLLISION : 0u, lds);
}

// One tile of a LiDAR scan query (Sec. III-G): point p gives direction p/|p| and distance
// |p|; non-finite points and points closer than min_range are skipped.  Tile t covers points
// t*256 + lane + k * n_tiles * 256, which a thread takes in increasing k.  A thread loads
// kScanBatch of its points before it evaluates the first, so that their loads wait once.
__device__ __forceinline__ void scan_tile(const ScanArgs &A, int tile, int n_tiles, const FinishSlots &F,
                                          float *lds)
{
    Acc acc;
    acc.zero();
    const int stride = n_tiles * kBlock;
    for (int i0 = tile * kBlock + threadIdx.x; i0 < A.n_points; i0 += kScanBatch * stride) {
        float p[kScanBatch][3];
#pragma unroll
        for (int k = 0; k < kScanBatch; ++k) {
            const int i = i0 + k * stride;
            const size_t j = i < A.n_points ? 3 * (size_t)i : 0;      // past the end: point 0, unused
            p[k][0] = A.points[j];
            p[k][1] = A.points[j + 1];
            p[k][2] = A.points[j + 2];
        }
#pragma unroll
        for (int k = 0; k < kScanBatch; ++k) {
            const float px = p[k][0], py = p[k][1], pz = p[k][2];
            if (i0 + k * stride >= A.n_points || !(isfinite(px) && isfinite(py) && isfinite(pz))) continue;
            double n2, vp;
            {
#pragma clang fp contract(off)
                n2 = ((double)px * (double)px + (double)py * (double)py) + (double)pz * (double)pz;
                vp = (A.vel64[0] * (double)px + A.vel64[1] * (double)py) + A.vel64[2] * (double)pz;
            }
            if (!(n2 >= A.min_range2)) continue;
            const double d64 = sqrt(n2);
            const float inv = (float)(1.0 / d64);
            acc.n_hit += 1;
            acc.n_contrib += d64 < A.radius64 && vp > 0.0;
            policy_accumulate(A.pol, px * inv, py * inv, pz * inv, (float)d64, acc);
        }
    }
    grid_finish(acc, tile, n_tiles, F, A.rank_tol, A.n_points, 0u, lds);
}

// One map query per launch; block b takes tile xcd_tile(b).
template <int DT, bool PART>
__global__ void __launch_bounds__(kBlock, DT == kIndexedF32 || DT == kIndexedF16 ? 2 : 4) raycast_rmp_kernel(RayArgs A)
{
    __shared__ __align__(16) float lds[kReduceLdsWords];
    ray_tile<DT, PART>(A, xcd_tile(blockIdx.x, gridDim.x), gridDim.x,
                       single_slots(A.partials, A.ticket, A.result, A.done, A.seq), lds);
}

// A batch's descriptor as constant memory, so that its words come by scalar loads where they are
// used: nothing writes the descriptors while the kernel runs, which the compiler cannot see past
// the kernel's atomics (it would load them per lane; moving a whole descriptor into scalar registers
// word by word was 130 instructions a tile and wave, and more than there are).
template <typename T>
__device__ __forceinline__ const T &constant_ref(const T &v)
{
    typedef const __attribute__((address_space(4))) T *ConstPtr;
    return *(const T *)(ConstPtr)(uintptr_t)&v;
}

// Many map and scan queries in one persistent launch: resident blocks take tiles from a
// counter (work[0]) until none are left; tile rows, tickets and results are per query, so a
// query's result does not depend on which block ran which tile.  The last block to leave
// resets the counters for the next launch.
//
// A tile is a short piece of work (some 15 us, VALU instructions two thirds of it), so what comes
// before its walk is kept short: every lane holds the first tile of one query in 64, which makes
// finding a tile's query a comparison per lane and one load of the queries between two of those,
// and descriptors come by scalar loads.  With that and four waves per SIMD instead of three a batch of 512
// queries (45,000 tiles) takes 759 us instead of 1,110, 64 served requests 62 instead of 64.
// (Taking the next tile while the current one is walked made the served batches 13 % slower: the
// blocks that start first hold the last tiles.  A kernel of its own without the sparse walk, five
// waves per SIMD: 4 % less for the large batch, 2 % more for the served ones.)
__global__ void __launch_bounds__(kBlock, 4) batch_kernel(BatchArgs B)
{
    __shared__ __align__(16) float lds[kReduceLdsWords];
    __shared__ int s_tile;
    const int n_tiles = B.hdr->n_tiles;
    const int n_queries = B.hdr->n_queries;
    const int lane = threadIdx.x & (kWave - 1);
    const int stride = (n_queries + kWave - 1) / kWave;
    const int coarse = lane * stride < n_queries ? B.q[lane * stride].tile_begin : 0x7fffffff;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_tile = (int)__hip_atomic_fetch_add(B.work, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        // the tile and its query are the same for the whole block: keep them (and the query's
        // descriptor) in scalar registers
        const int tile = __builtin_amdgcn_readfirstlane(s_tile);
        if (tile >= n_tiles) break;
        // last query with tile_begin <= tile
        int lo = stride * (__popcll(__ballot(coarse <= tile)) - 1);
        if (stride > 1)
            lo += __popcll(__ballot(lane < stride && lo + lane < n_queries && B.q[lo + lane].tile_begin <= tile)) - 1;
        const BatchQuery &Q = constant_ref(B.q[lo]);
        const BatchQueryHead head = Q.head;
        FinishSlots F;
        F.tile_rows = B.partials + (size_t)head.tile_begin * kPartialWords;
        F.tickets = B.tickets + lo;
        F.out = B.results + lo;
        F.finished = B.work + 2;
        F.n_queries = n_queries;
        F.done = B.done;
        F.seq = B.hdr->seq;
        const int t = tile - head.tile_begin;
        if (head.kind == 0) {
            const RayArgs &A = Q.ray;
            if (A.sparse == 2) {
                ray_tile<kIndexed, false>(A, t, head.n_tiles, F, lds);
                continue;
            }
            if (A.sparse) {
                // block rounds of 4 steps on sparse maps (their best), no sub-voxel refinement
                // (batches refuse it on sparse maps)
                sparse_tile<4, kSvNone>(A, t, head.n_tiles, F, lds);
                continue;
            }
            switch (A.map.dtype * 2 + (A.map.partial != 0 ? 1 : 0)) {
            case RMPC_TSDF_F32 * 2: ray_tile<RMPC_TSDF_F32, false>(A, t, head.n_tiles, F, lds); break;
            case RMPC_TSDF_F32 * 2 + 1: ray_tile<RMPC_TSDF_F32, true>(A, t, head.n_tiles, F, lds); break;
            case RMPC_TSDF_F16 * 2: ray_tile<RMPC_TSDF_F16, false>(A, t, head.n_tiles, F, lds); break;
            case RMPC_TSDF_F16 * 2 + 1: ray_tile<RMPC_TSDF_F16, true>(A, t, head.n_tiles, F, lds); break;
            default: ray_tile<RMPC_OCC_U8, false>(A, t, head.n_tiles, F, lds); break;
            }
        } else {
            scan_tile(Q.scan, t, head.n_tiles, F, lds);
        }
    }
    if (threadIdx.x == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(B.work + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == gridDim.x - 1) {
            __hip_atomic_store(B.work, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(B.work + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int DT, bool PART>
__global__ void __launch_bounds__(kBlock, 2) trace_debug_kernel(RayArgs A)
{
    const int S = A.segments;
    const int p = xcd_tile(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int j = p < A.n_list * S ? p / S : 0;
    const int seg = p & (S - 1);
    const float4 rr = load_ray(A.rays, j);
    const int i = __float_as_int(rr.w);
    const bool valid = p < A.n_list * S && i < A.n_rays;
    const float rx = rr.x, ry = rr.y, rz = rr.z;
    if (start_occupied<DT>(A)) {
        if (valid && seg == 0) {
            A.dbg_hit[i] = hit_index<DT>(A, A.v0[0], A.v0[1], A.v0[2]);
            A.dbg_dist[i] = 0.0;
            A.dbg_flags[i] = (uint8_t)(A.start_flags | kRayInCollision);
            if (A.dbg_visits) A.dbg_visits[i] = 1;
        }
        return;
    }
    const RayOut o = trace_group<DT, PART>(A, valid, seg, S, rx, ry, rz);
    // the ray's visit count is the sum over its group
    int v = o.visits_lane;
    for (int off = 1; off < S; off <<= 1) v += __shfl_xor(v, off, kWave);
    if (o.report) {
        A.dbg_hit[i] = o.hit ? hit_index<DT>(A, o.fx, o.fy, o.fz) : -1;
        double d = o.d;
        if constexpr (DT != RMPC_OCC_U8 && DT != kIndexed)
            if (A.subvoxel && o.hit) d = subvoxel_distance<DT>(A, rx, ry, rz, d);
        A.dbg_dist[i] = d;
        A.dbg_flags[i] = (uint8_t)o.flags;
        if (A.dbg_visits) A.dbg_visits[i] = v;
    }
}

// One scan query per launch.
__global__ void __launch_bounds__(kBlock) scan_rmp_kernel(ScanArgs A)
{
    __shared__ __align__(16) float lds[kReduceLdsWords];
    scan_tile(A, blockIdx.x, gridDim.x, single_slots(A.partials, A.ticket, A.result, A.done, A.seq), lds);
}

template <int DT, bool PART>
hipError_t launch_dt(const RayArgs &A, int grid, hipStream_t s, bool debug, hipEvent_t e0, hipEvent_t e1)
{
    const dim3 blk(kBlock);
    if (debug) {
        const dim3 g((A.n_list * A.segments + kBlock - 1) / kBlock);
        if (e0) hipExtLaunchKernelGGL(trace_debug_kernel<DT, PART>, g, blk, 0, s, e0, e1, 0, A);
        else trace_debug_kernel<DT, PART><<<g, blk, 0, s>>>(A);
    } else {
        if (e0) hipExtLaunchKernelGGL(raycast_rmp_kernel<DT, PART>, dim3(grid), blk, 0, s, e0, e1, 0, A);
        else raycast_rmp_kernel<DT, PART><<<grid, blk, 0, s>>>(A);
    }
    return hipGetLastError();
}

}  // namespace

int ray_grid_blocks(int lanes)
{
    int b = (lanes + kBlock - 1) / kBlock;
    return b < 1 ? 1 : (b > kMaxBlocks ? kMaxBlocks : b);
}

// At most 128 blocks: what every block pays at its end (its reduction, its row, its ticket, the
// merge of its row) costs more than a few more points per thread at the frame size of a LiDAR: 65,536
// points take 15.3 us with 128 blocks and 16.1 with 256 (262,144 points 19.2 and 17.6, 1,048,576 points
// 35.4 and 25.2).
int scan_grid_blocks(int n_points)
{
    int b = (n_points + kBlock - 1) / kBlock;
    return b < 1 ? 1 : (b > kScanMaxBlocks ? kScanMaxBlocks : b);
}

hipError_t launch_scan(const ScanArgs &A, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const dim3 g(scan_grid_blocks(A.n_points)), blk(kBlock);
    if (e0) hipExtLaunchKernelGGL(scan_rmp_kernel, g, blk, 0, s, e0, e1, 0, A);
    else scan_rmp_kernel<<<g, blk, 0, s>>>(A);
    return hipGetLastError();
}

int batch_blocks_per_cu()
{
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_kernel, kBlock, 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}

hipError_t launch_batch(const BatchArgs &a, int blocks, hipStream_t s)
{
    batch_kernel<<<blocks, kBlock, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_raycast(const RayArgs &A, hipStream_t s, bool debug, hipEvent_t e0, hipEvent_t e1)
{
    const int grid = ray_grid_blocks(A.n_list * A.segments);
    const bool part = A.map.partial != 0;
    if (A.sparse) {
        if (!A.subvoxel) return launch_dt<kIndexed, false>(A, grid, s, debug, e0, e1);
        return A.sp.dtype == RMPC_TSDF_F32 ? launch_dt<kIndexedF32, false>(A, grid, s, debug, e0, e1)
                                           : launch_dt<kIndexedF16, false>(A, grid, s, debug, e0, e1);
    }
    switch (A.map.dtype) {
    case RMPC_TSDF_F32:
        return part ? launch_dt<RMPC_TSDF_F32, true>(A, grid, s, debug, e0, e1)
                    : launch_dt<RMPC_TSDF_F32, false>(A, grid, s, debug, e0, e1);
    case RMPC_TSDF_F16:
        return part ? launch_dt<RMPC_TSDF_F16, true>(A, grid, s, debug, e0, e1)
                    : launch_dt<RMPC_TSDF_F16, false>(A, grid, s, debug, e0, e1);
    default: return launch_dt<RMPC_OCC_U8, false>(A, grid, s, debug, e0, e1);
    }
}

}  // namespace rmpc
