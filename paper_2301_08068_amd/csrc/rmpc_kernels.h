// rmpc_kernels.h -- plain-data launch arguments shared by the C-ABI layer and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rmpcast.h"

namespace rmpc {

// The dense configurations' lookahead as reported by default (their walks do not plan ahead).
constexpr int kLookahead = 8;

// Threads per block of the query kernels (one tile = this many lanes).
constexpr int kBlockThreads = 256;

// Block-partial slots of one reduction (one per block of a launch).
constexpr int kMaxPartialSlots = 4096;

// Words of one block partial in device memory: 18 floats + 4 integers, padded.
constexpr int kPartialWords = 32;

// Blocks of one scan query (at the end each costs more than a loop over a few more points).
constexpr int kScanMaxBlocks = 128;
constexpr int kScanBatch = 8;                // scan points a thread loads before it evaluates them

// log2 of the edge, in voxels, of a brick, and of the cells that the arena layout counts.
constexpr int kCellLog2 = 3;
constexpr int kBrickLog2 = 1;

// Box entry of a brick (16 bits).
//   Free brick: three 5-bit fields from bit 0 that hold twice the half extents (2 ex, 2 ey, 2 ez;
//   1 <= e <= kBoxMax bricks): every brick within ex - 1, ey - 1 and ez - 1 of it along x, y and z
//   is free (or outside the grid).
//   Occupied brick: kBoxOccupied, the occupancy of its voxels in the low byte (bit (x & 1) + 2 (y
//   & 1) + 4 (z & 1)), and one of its six voxel layers that is free: bit 8 the side, bits 9-10 the
//   axis a (3: none, with side 1), bits 11-14 its half extent e: the voxel layer on that side of
//   axis a is free in every brick within e - 1 of it along the other two axes.
constexpr uint32_t kBoxOccupied = 0x8000u;
constexpr uint32_t kBoxNoLayer = (1u << 8) | (3u << 9);
constexpr int kBoxMax = 15;
constexpr uint32_t box_extents(uint32_t ex, uint32_t ey, uint32_t ez) { return 2u * (ex | (ey << 5) | (ez << 10)); }

// A resident map: float32 and float16 maps keep the voxel grid x-fastest (element offset x + nx
// (y + ny z)); uint8 maps keep only the box entries, which hold every voxel's occupancy.
struct MapView {
    const void *data;            // the grid (uint8 maps: null)
    const uint16_t *box;         // one entry per brick, x-fastest
    int32_t nx, ny, nz, dtype;
    int32_t nbx, nby, nbz;       // bricks with an entry along each axis
    int32_t partial;             // non-zero: an odd last layer of voxels has no entries
    int32_t lo;                  // first voxel along every axis (0; a sparse map's box walk: -kFarVoxel)
    int32_t span;                // bound of a walk's coordinates (for the float32 error)
};
constexpr int32_t kFarVoxel = 1 << 24;

// A sparse map: 8 x 8 x 8-voxel blocks stored where the world has content (every other voxel
// is free), found through an open-addressed hash table from block coordinates to slots.
constexpr int kBlockLog2 = 3;
constexpr int kBlockEdge = 1 << kBlockLog2;
constexpr int kBlockVoxels = 512;
// Block coordinates are signed 21-bit integers (|voxel coordinate| < 2^23 voxels).
constexpr int kBlockCoordBits = 21;
constexpr int32_t kBlockCoordBias = 1 << (kBlockCoordBits - 1);
constexpr uint64_t kEmptyKey = ~0ull;

// One table entry (16 bytes, one load): the packed block coordinates, the block's slot and
// whether any of its voxels is occupied.
struct alignas(16) HashEntry {
    uint64_t key;
    int32_t slot;
    uint32_t occupied;
};

// Key of block (bx, by, bz): the three biased 21-bit coordinates, x lowest.  Valid keys have
// bit 63 clear, so they never equal kEmptyKey.
__host__ __device__ inline uint64_t block_key(int32_t bx, int32_t by, int32_t bz)
{
    return (uint64_t)(uint32_t)(bx + kBlockCoordBias) | ((uint64_t)(uint32_t)(by + kBlockCoordBias) << 21) |
           ((uint64_t)(uint32_t)(bz + kBlockCoordBias) << 42);
}

// First table index of a key: the 64-bit finaliser of MurmurHash3 (fmix64), masked.
__host__ __device__ inline uint32_t block_hash(uint64_t k, uint32_t mask)
{
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return (uint32_t)k & mask;
}

constexpr uint32_t kBlockOccupied = 1u << 31;
// A map's index is built where no coordinate exceeds this, and a query walks by it where none of the
// walk's does (in float32 terms: 1/60 of a voxel).
constexpr int32_t kIndexSpan = 1 << 16;
struct SparseView {
    const HashEntry *table;      // table_mask + 1 entries (a power of two, at least twice the blocks)
    uint32_t table_mask;
    int32_t n_slots;
    const uint64_t *occ;         // per slot 8 words: word z holds bit x + 8 y of the block's layer z
    const void *values;          // per slot 512 elements, x fastest within the block
    int32_t dtype;
    int32_t pad;
    double free_value;           // TSDF maps: the field's value outside the stored blocks
    // the box walk's index (null: the map has none), over the blocks of a box that holds all stored
    // ones: block lo + (x, y, z) at x + nb[0] (y + nb[1] z)
    const uint32_t *index;       // kBlockOccupied | slot, or a free block's box of free blocks: the bits of box_extents
    const uint16_t *bricks;      // 64 brick entries per slot (as a dense map's; bricks of other slots count as well)
    int32_t lo[3], nb[3];
};

// Policy constants in float32 (reciprocals precomputed on the host).
struct PolicyF {
    float vx, vy, vz;            // robot velocity
    float c, eta_rep, inv_nu_rep, eta_damp, inv_nu_damp, radius, inv_radius, eps;
    // non-zero: none of them makes a ray's terms NaN whose damping is zero or that hits beyond the
    // radius (quotients 0 / 0, products 0 inf of a parameter that is zero, huge or infinite in float32)
    int32_t tame;
};

// One entry of an ordered ray list: the float32 direction of Halton ray i and i itself, so
// that a lane gets its ray with one 16-byte load.
struct alignas(16) RayRec {
    float x, y, z;
    int32_t i;
};

// Everything one map query needs.
struct RayArgs {
    MapView map;                 // dense maps
    SparseView sp;               // sparse maps
    int32_t sparse;              // 0: a dense map, 1: a sparse one by its table, 2: by its index
    const RayRec *rays;          // ordered ray list; entries with i >= n_rays are skipped
    int32_t n_list;              // length of `rays` (>= n_rays)
    int32_t n_rays;
    float g[3];                  // start in grid units, float32((x - origin) / h)
    int32_t v0[3];               // start voxel floor(g)
    int32_t base[3];             // sparse maps walked by their index far from the origin: the voxel that g, v0 and
                                 //   sp.lo count from, else 0
    int32_t lin0;                // its logical index
    uint32_t start_flags;        // RMPC_RAY_START_FACE when g is within 1e-5 of a face
    float tmax_lo, tmax_hi;      // float32 guard band around max_range / h
    double tmax_v;               // parameter span split into segments: min(max_range / h, grid diagonal)
    int32_t segments;            // segments per ray (1, 2, 4, 8 or 16): a tile holds kBlock / segments rays
    int32_t lookahead;           // sparse maps: block steps planned per round (4, 8 or 16)
    double max_range, h;
    int32_t subvoxel;            // non-zero: refine hit distances on the interpolated TSDF
    double vel64[3];             // velocity, float64 (for the exact contribution count)
    double radius64;
    PolicyF pol;
    double rank_tol;
    float *partials;             // per-block partial sums
    uint32_t *ticket;            // arrival counter, zero between launches
    rmpc_result *result;         // written by the last block
    uint64_t *done;              // host-visible completion word, set to seq after the result
    uint64_t seq;
    // debug outputs (trace kernel only)
    int32_t *dbg_hit;
    double *dbg_dist;
    uint8_t *dbg_flags;
    int32_t *dbg_visits;
};

// LiDAR scan query.
struct ScanArgs {
    const float *points;         // n x 3 float32
    int32_t n_points;
    double min_range2;           // squared minimum range, float64
    double vel64[3];
    double radius64;
    PolicyF pol;
    double rank_tol;
    float *partials;
    uint32_t *ticket;
    rmpc_result *result;         // host (pinned) or device memory
    uint64_t *done;              // host-visible completion word, or null (result left on the stream)
    uint64_t seq;
};

// One query of a batched launch, and what every tile of it needs first.
struct BatchQueryHead {
    int32_t kind;                // 0: map query (ray), 1: scan query (scan)
    int32_t tile_begin;          // first tile of this query in the batch
    int32_t n_tiles;             // 256-lane tiles of this query
    int32_t pad;
};
struct BatchQuery {
    union {
        BatchQueryHead head;
        struct { int32_t kind, tile_begin, n_tiles, pad; };
    };
    union {
        RayArgs ray;
        ScanArgs scan;
    };
};

// Per-launch header of a batch, in device memory (so a captured launch can be replayed).
struct BatchHeader {
    int32_t n_queries;
    int32_t n_tiles;
    uint64_t seq;
};

// Launch arguments of the persistent batch kernel (pointers only).
struct BatchArgs {
    const BatchHeader *hdr;
    const BatchQuery *__restrict__ q;
    uint32_t *work;              // [0] next tile, [1] blocks exited, [2] queries finished
    uint32_t *tickets;           // one per query
    float *partials;             // tile rows of all queries
    rmpc_result *results;        // one per query (pinned host memory)
    uint64_t *done;              // completion word, set to hdr->seq when all queries are done
};

constexpr int kBatchMaxQueries = 4096;
constexpr int kBatchMaxTiles = 262144;

struct DirsArgs {
    float *out;                  // structure of arrays with stride n
    int32_t n;
};

// Keep, in order, the entries of `order` (a permutation of 0..n_all-1) that are < n.
struct CompactArgs {
    const int32_t *order;
    int32_t n_all;
    int32_t n;
    int32_t *counts;             // n_all / 1024 per-chunk counts (scratch)
    int32_t *out;                // n entries
};

// out[k] = {dirs[idx[k]] (x, y, z from a structure of arrays with stride `stride`), idx[k]}.
struct GatherArgs {
    const int32_t *idx;
    int32_t n;
    const float *dirs;
    int32_t stride;
    RayRec *out;
};

// Build a map's box entries (and its grid) from the voxels at src.
struct BoxArgs {
    MapView map;                 // data and box already point into the arena
    const void *src;             // device memory: the voxels, x-fastest (map.data: in place)
    uint8_t *scratch;            // box_scratch_bytes, or null: narrower boxes
};

int ray_grid_blocks(int n_rays);
int scan_grid_blocks(int n_points);
// When ev0/ev1 are non-null the kernel is launched with hipExtLaunchKernelGGL so the two
// events carry the dispatch's own start and end timestamps.
hipError_t launch_raycast(const RayArgs &a, hipStream_t s, bool debug, hipEvent_t ev0 = nullptr,
                          hipEvent_t ev1 = nullptr);
hipError_t launch_scan(const ScanArgs &a, hipStream_t s, hipEvent_t ev0 = nullptr,
                       hipEvent_t ev1 = nullptr);
hipError_t launch_directions(const DirsArgs &a, hipStream_t s);
hipError_t launch_map_boxes(const BoxArgs &a, hipStream_t s);
// What launch_map_boxes without scratch does to entries of single-brick boxes (m.box).
hipError_t launch_unit_boxes(const MapView &m, hipStream_t s);
// Scratch bytes of launch_map_boxes.
size_t box_scratch_bytes(const MapView &m);
hipError_t launch_compact(const CompactArgs &a, hipStream_t s);
hipError_t launch_gather(const GatherArgs &a, hipStream_t s);
// Exact squared Euclidean distance transform of the map's occupancy into out (x fastest) where
// every distance stays below 256 voxels; otherwise *flag_host (pinned, cleared by the caller) is
// set and out is undefined.  scratch: edt_scratch_bytes, or at least kEdtFlagBytes (the row
// distances then go through out), 256-byte aligned.
constexpr size_t kEdtFlagBytes = 256;
hipError_t launch_edt(const MapView &m, int32_t *out, void *scratch, size_t scratch_bytes, uint32_t *flag_host,
                      hipStream_t s);
// The same for any distance, without scratch.
hipError_t launch_edt_wide(const MapView &m, int32_t *out, hipStream_t s);
size_t edt_scratch_bytes(const MapView &m);

// The single-lookup ESDF policy at one position.
struct EsdfArgs {
    const int32_t *sq;           // squared distance transform, x fastest
    int32_t nx, ny, nz;
    int32_t v0[3];               // the position's voxel
    double h;
    double vel[3];
    double c, eta_rep, nu_rep, eta_damp, nu_damp, radius, eps, rank_tol;
    rmpc_result *out;            // pinned host memory
    uint64_t *done;              // host-visible completion word, set to seq after the result
    uint64_t seq;
};
hipError_t launch_esdf(const EsdfArgs &a, hipStream_t s);
// One map query on a sparse map (debug: per-ray outputs instead of the policy).
hipError_t launch_sparse(const RayArgs &a, hipStream_t s, bool debug, hipEvent_t ev0 = nullptr,
                         hipEvent_t ev1 = nullptr);
// Occupancy masks of a sparse map's blocks from their values, the table's occupied flags, and (v.index
// not null) its index and brick entries, with scratch: sparse_index_scratch_bytes, 256-byte aligned.
size_t sparse_index_scratch_bytes(const SparseView &v);
hipError_t launch_sparse_build(const SparseView &v, HashEntry *table, uint8_t *scratch, hipStream_t s);
// Where launch_cell_boxes reads a cell's occupancy in its scratch: one byte (0 or 255) each, cell
// (x, y, z) at x sx + y sy + z sz (at most 2^28 cells); rows of `pitch` bytes, in all `bytes`.
struct BoxMask {
    uint8_t *at;
    uint32_t sx, sy, sz, pitch;
    size_t bytes;
};
BoxMask box_mask(const MapView &m, uint8_t *scratch);
// The boxes of a grid of nbx x nby x nbz cells from their occupancy at the start of scratch
// (box_scratch_bytes; the occupancy zeroed and set by the caller), written to box.
void launch_cell_boxes(const MapView &m, uint8_t *scratch, hipStream_t s);
// Persistent fused batch: `blocks` resident blocks pull tiles from a counter.
hipError_t launch_batch(const BatchArgs &a, int blocks, hipStream_t s);
// Resident blocks per CU of the batch kernel.
int batch_blocks_per_cu();

}  // namespace rmpc
