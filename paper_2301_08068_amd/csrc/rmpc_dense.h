// rmpc_dense.h -- the exact ray walk over a dense map, or a sparse one by its index (Sec. III-E/F):
// a 3-D DDA that crosses free space box by box.
//
// A resident map has one 16-bit entry per brick of 2 x 2 x 2 voxels (box_kernels.hip): a box of
// bricks around it that holds no occupied voxel, or, for a brick with an occupied voxel, which of
// its eight voxels are occupied and how far one of its voxel layers is free.  A walk reads the entry
// of the voxel it is in, takes the first crossing of a face of that box (layer, voxel) and continues
// in the voxel entered there.  Box faces are voxel faces, so the crossing taken is one that the
// voxel walk takes too, and every voxel skipped is free.
//
// Exactness: crossings are compared in float32 as T = (F - g) / r with F the integer face
// coordinate (never accumulated; within 1.8e-7 T of its value).  The voxel entered is the floor
// of g + T r along the other two axes.  When that point lies near a voxel face along more than
// the crossed axis, or the crossing lies near max_range, the crossing and the voxel are decided
// in float64 from the definition's formula, lowest axis first on exact ties.  All coordinates
// are direction-signed (s * coordinate, s the sign of r along the axis), so a walk only moves
// toward larger values.
//
// What bounds a query is the longest chain of steps: a step is a dependent 2-byte load and 38 VALU
// instructions (25 more in an occupied brick), 550 cycles for a wave that has its SIMD nearly to
// itself, and the slowest of 64 neighbouring rays of a 65,536-ray query takes 9-15 of them (one
// segment per ray), the slowest of all 30-45.  Planning voxel, brick and 8^3-cell steps eight at a
// time instead (33 VALU instructions a step, 240 a round) took 15-18 rounds of 2.2 us in the
// slowest waves: that query's kernel 42-44 us against 24, a batch of 512 queries 2.23 ms against
// 1.13 (20 us and 0.76 ms with the reductions and the batch kernel as they are now).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rmpc_kernels.h"
#include "rmpc_walk.h"

namespace rmpc {

// A segment starts this far (voxel units) before the end of the one before it, so that every
// crossing within the float32 error of a boundary is walked by the segment before (and twice
// that error, where it is larger).
constexpr float kSegOverlap = 0.01f;

// What the walk reads, besides the three storage types of dense maps: the index of a sparse map
// (whose hit distances are refined on no, a float32 or a float16 field).
constexpr int kIndexed = 3, kIndexedF32 = 4, kIndexedF16 = 5;
constexpr bool is_indexed(int dt) { return dt >= kIndexed; }

struct BoxRay {
    float rx, ry, rz;                 // direction
    float gsx, gsy, gsz;              // start, signed
    float arx, ary, arz;              // |1 / r|, finite
    float hsx, hsy, hsz;              // gs + tol
    float tol;                        // bound of the float32 error of a coordinate g + T r up to the ray's end
    int kx, ky, kz, k0;               // byte offset of a brick's entry: k0 + x kx + y ky + z kz with x, y, z the signed
                                      //   coordinates of its first voxel (even numbers); sparse maps: the signs of
                                      //   the axes (0 or -1) in kx, ky, kz
    uint32_t flip;                    // voxel-in-brick index bits of the axes walked downward
    float t_exit;                     // float32 parameter of the first face of the grid's surface ahead
};

struct BoxWalk {
    int ux, uy, uz;                   // current voxel, signed
    float t;                          // float32 parameter at which it was entered, -1: the segment's start
    int left;                         // steps to take before the next look at the other lanes, or:
    uint32_t tie;                     // non-zero: a near-tie at a decision taken
};
constexpr int kWalkEnded = -1;        // the walk has ended without a hit in its segment
constexpr int kWalkHit = -2;          // the current voxel is the first occupied one

// Signed voxel index of voxel v, and back (the map is its own inverse).
__device__ __forceinline__ int signed_voxel(float r, int v) { return r >= 0.0f ? v : -v - 1; }

// Signed coordinate of the surface of a grid of n voxels that a ray leaves through.
__device__ __forceinline__ int signed_edge(const MapView &m, float r, int n) { return r >= 0.0f ? n : -m.lo; }

// Float64 parameter of signed face F along an axis (+inf for r = 0).
__device__ __forceinline__ double signed_face64(int F, float g, float r)
{
    return r != 0.0f ? face64(r > 0.0f ? F : -F, g, r) : __builtin_huge_val();
}

__device__ __forceinline__ float box_crossing(int F, float gs, float ar) { return ((float)F - gs) * ar; }

// Bound of the float32 error of a coordinate g + T r (voxel units), with a margin of about two: T
// carries three roundings (1.8e-7 T), the coordinate two (6e-8 each of at most the span).
__device__ __forceinline__ float box_tol(const MapView &m, float t)
{
    return fmaf(4e-7f, t, fmaf(2.5e-7f, (float)m.span, 1e-6f));
}

template <int DT>
__device__ __forceinline__ BoxRay box_ray(const RayArgs &A, float rx, float ry, float rz)
{
    const MapView &m = A.map;
    BoxRay R;
    R.rx = rx; R.ry = ry; R.rz = rz;
    const bool px = rx >= 0.0f, py = ry >= 0.0f, pz = rz >= 0.0f;
    R.gsx = px ? A.g[0] : -A.g[0];
    R.gsy = py ? A.g[1] : -A.g[1];
    R.gsz = pz ? A.g[2] : -A.g[2];
    // finite, so that a start on a face (F - g = 0) along a vanishing component gives no NaN; an
    // axis with r = 0 counts as walked upward, where the face ahead lies strictly past g
    R.arx = fminf(fabsf(1.0f / rx), 3e38f);
    R.ary = fminf(fabsf(1.0f / ry), 3e38f);
    R.arz = fminf(fabsf(1.0f / rz), 3e38f);
    // (24-bit multiplications: at most 2^12 voxels per axis, 2^22 bricks per layer; two bytes per
    // brick and two voxels per brick cancel)
    const int sx = 1, sy = m.nbx, sz = m.nbx * m.nby;
    R.kx = px ? sx : -sx;
    R.ky = py ? sy : -sy;
    R.kz = pz ? sz : -sz;
    if constexpr (is_indexed(DT)) {
        R.kx = px ? 0 : -1;
        R.ky = py ? 0 : -1;
        R.kz = pz ? 0 : -1;
    }
    in_vgpr(R.kx);                    // (a multiplication by a stride, not by a choice of two constants)
    R.k0 = -2 * ((px ? 0 : sx) + (py ? 0 : sy) + (pz ? 0 : sz));
    R.flip = (px ? 0u : 1u) | (py ? 0u : 2u) | (pz ? 0u : 4u);
    R.t_exit = fminf(box_crossing(signed_edge(m, rx, m.nx), R.gsx, R.arx),
                     fminf(box_crossing(signed_edge(m, ry, m.ny), R.gsy, R.ary),
                           box_crossing(signed_edge(m, rz, m.nz), R.gsz, R.arz)));
    R.tol = box_tol(m, fminf(R.t_exit, A.tmax_hi));
    R.hsx = R.gsx + R.tol;
    R.hsy = R.gsy + R.tol;
    R.hsz = R.gsz + R.tol;
    return R;
}

// floor(x) as an integer in one instruction.
__device__ __forceinline__ int floor_int(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    int i;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
    return i;
#else
    return (int)floorf(x);
#endif
}

// The entry of the current voxel's brick, whose first voxel is (ex, ey, ez).  Grids whose entries
// cover whole bricks only (PART) treat a voxel outside them as a brick with just that voxel's
// occupancy.
template <int DT, bool PART>
__device__ __forceinline__ uint32_t box_entry(const MapView &m, const BoxRay &R, const BoxWalk &w, int ex, int ey,
                                              int ez)
{
    const uint32_t off = (uint32_t)(__mul24(ez, R.kz) + (__mul24(ey, R.ky) + (__mul24(ex, R.kx) + R.k0)));
    if constexpr (PART) {
        const int vx = signed_voxel(R.rx, w.ux), vy = signed_voxel(R.ry, w.uy), vz = signed_voxel(R.rz, w.uz);
        if ((vx >> kBrickLog2) >= m.nbx || (vy >> kBrickLog2) >= m.nby || (vz >> kBrickLog2) >= m.nbz) {
            const auto *vox = static_cast<const typename Voxel<DT>::T *>(m.data);
            const bool o = Voxel<DT>::occ(vox[(uint32_t)vx + (uint32_t)m.nx * ((uint32_t)vy + (uint32_t)m.ny * (uint32_t)vz)]);
            return kBoxOccupied | kBoxNoLayer | (o ? 0xffu : 0u);
        }
    }
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(m.box) + off);
}

// A sparse map's counterpart of box_entry.  An index entry per 8^3 block of the box around the stored
// blocks holds a box of free blocks, or the slot of a block with an occupied voxel, whose bricks'
// entries are one more load.  Planning block steps four at a time with a hash probe each, and voxel
// steps on the block's occupancy, took 115 us for 65,536 rays in an outdoor map 96 m wide (0.05 m
// voxels, 10 m range) against 43, batches of such queries in proportion.
// Gives the faces ahead of the box around the current voxel, and returns its brick's entry if its
// block has an occupied voxel (else 0).  Outside the index the box reaches to the
// index along one axis that the ray has not reached it on (everything nearer is free), or past
// every range when it lies behind.
__device__ __forceinline__ uint32_t indexed_entry(const SparseView &S, const BoxRay &R, const BoxWalk &w, int &Fx, int &Fy,
                                                  int &Fz)
{
    const int vx = w.ux ^ R.kx, vy = w.uy ^ R.ky, vz = w.uz ^ R.kz;
    const uint32_t ix = (uint32_t)((vx >> kBlockLog2) - S.lo[0]), iy = (uint32_t)((vy >> kBlockLog2) - S.lo[1]),
                   iz = (uint32_t)((vz >> kBlockLog2) - S.lo[2]);
    if (ix < (uint32_t)S.nb[0] && iy < (uint32_t)S.nb[1] && iz < (uint32_t)S.nb[2]) {
        uint32_t e = S.index[ix + (uint32_t)S.nb[0] * (iy + __umul24(iz, (uint32_t)S.nb[1]))];
        if ((e & kBlockOccupied) == 0u) {
            Fx = (w.ux & ~7) + 4 * (int)(e & 31u);
            Fy = (w.uy & ~7) + 4 * (int)((e >> 5) & 31u);
            Fz = (w.uz & ~7) + 4 * (int)((e >> 10) & 31u);
            return 0u;
        }
        e = S.bricks[(e << 6) | (((uint32_t)vx >> 1) & 3u) | (((uint32_t)vy << 1) & 12u) | (((uint32_t)vz << 3) & 48u)];
        Fx = (w.ux & ~1) + (int)(e & 31u);
        Fy = (w.uy & ~1) + (int)((e >> 5) & 31u);
        Fz = (w.uz & ~1) + (int)((e >> 10) & 31u);
        return e;
    }
    // signed first voxel of the index and the one past its last
    const int ax = 8 * (R.kx ? -S.lo[0] - S.nb[0] : S.lo[0]), bx = ax + 8 * S.nb[0];
    const int ay = 8 * (R.ky ? -S.lo[1] - S.nb[1] : S.lo[1]), by = ay + 8 * S.nb[1];
    const int az = 8 * (R.kz ? -S.lo[2] - S.nb[2] : S.lo[2]), bz = az + 8 * S.nb[2];
    Fx = Fy = Fz = kFarVoxel;
    if (w.ux < bx && w.uy < by && w.uz < bz) {
        if (w.ux < ax) Fx = ax;
        else if (w.uy < ay) Fy = ay;
        else Fz = az;
    }
    return 0u;
}

// Signed coordinate along axis b of the voxel the walk is in right after the crossing of axis a
// at float64 parameter t64 (float32 ta), known to lie in [lo, hi].
__device__ __forceinline__ int box_coord64(const MapView &m, float gs, float g, float r, int b, int a, float ta,
                                           double t64, int lo, int hi, bool &tie)
{
    const float y = fmaf(ta, fabsf(r), gs);
    const float fl = floorf(y), fr = y - fl, tol = box_tol(m, ta);
    int c = (int)fl;
    if (fr > tol && fr < 1.0f - tol && c >= lo && c <= hi) return c;
    c = min(max(c, lo), hi);
    if (c > lo) {                     // was the face into c crossed before?
        const double f = signed_face64(c, g, r);
        tie = tie || fabs(f - t64) < 1e-5;
        if (!(f < t64 || (f == t64 && b < a))) return c - 1;
    }
    if (c < hi) {                     // or the face out of c?
        const double f = signed_face64(c + 1, g, r);
        tie = tie || fabs(f - t64) < 1e-5;
        if (f < t64 || (f == t64 && b < a)) return c + 1;
    }
    return c;
}

// The crossing out of a box with faces (Fx, Fy, Fz) ahead, decided in float64.  Returns false
// when the walk ends inside the box (segment end, max_range or the grid's surface).
__device__ __forceinline__ bool box_step64(const RayArgs &A, const BoxRay &R, BoxWalk &w, int Fx, int Fy, int Fz,
                                           float t_lo, float t_hi)
{
    const MapView &m = A.map;
    const int ex = signed_edge(m, R.rx, m.nx), ey = signed_edge(m, R.ry, m.ny), ez = signed_edge(m, R.rz, m.nz);
    Fx = min(Fx, ex); Fy = min(Fy, ey); Fz = min(Fz, ez);
    const double X = signed_face64(Fx, A.g[0], R.rx), Y = signed_face64(Fy, A.g[1], R.ry), Z = signed_face64(Fz, A.g[2], R.rz);
    int a = 0;
    double t64 = X;
    if (Y < t64) { a = 1; t64 = Y; }
    if (Z < t64) { a = 2; t64 = Z; }
    bool tie = (a != 0 && X - t64 < 1e-5) || (a != 1 && Y - t64 < 1e-5) || (a != 2 && Z - t64 < 1e-5);
    // (a choice between values: one between R's fields would keep R in private memory)
    const float Tx = box_crossing(Fx, R.gsx, R.arx), Ty = box_crossing(Fy, R.gsy, R.ary), Tz = box_crossing(Fz, R.gsz, R.arz);
    const float ta = a == 0 ? Tx : (a == 1 ? Ty : Tz);
    if (ta > t_hi) return false;
    if (ta >= t_lo && t64 * A.h > A.max_range) return false;           // closed interval
    if (a == 0 ? Fx == ex : (a == 1 ? Fy == ey : Fz == ez)) return false;
    const int nx = a == 0 ? Fx : box_coord64(m, R.gsx, A.g[0], R.rx, 0, a, ta, t64, w.ux, Fx - 1, tie);
    const int ny = a == 1 ? Fy : box_coord64(m, R.gsy, A.g[1], R.ry, 1, a, ta, t64, w.uy, Fy - 1, tie);
    const int nz = a == 2 ? Fz : box_coord64(m, R.gsz, A.g[2], R.rz, 2, a, ta, t64, w.uz, Fz - 1, tie);
    w.ux = nx; w.uy = ny; w.uz = nz;
    w.t = ta;
    w.tie |= tie ? 1u : 0u;
    return true;
}

// Distance of y from the middle between two integers: 1/2 on an integer.
__device__ __forceinline__ float off_middle(float y) { return fabsf(y - floorf(y) - 0.5f); }

__device__ __forceinline__ float fraction(float y)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_fractf(y);
#else
    return y - floorf(y);
#endif
}

// One step: read the current voxel's entry; on an occupied voxel the walk has hit, else it
// moves to the voxel entered where it leaves the entry's box.  t_end: the smallest parameter at
// which the walk may end (the segment's end, the grid's surface, the range band from t_lo on);
// t_first: voxels entered before this belong to the segment before, which tests them.
//
// A point shifted by tol along each axis has the entered voxel as its floor: along the crossed axis
// it lies just past the face (within 2 tol), along the others it does unless a face is within tol,
// and then two axes (the middle of the three fractions) are within 2 tol above a face.
template <int DT, bool PART>
__device__ __forceinline__ void box_step(const RayArgs &A, const BoxRay &R, BoxWalk &w, float t_end, float t_lo,
                                         float t_hi, float t_first)
{
    const int ex = w.ux & ~1, ey = w.uy & ~1, ez = w.uz & ~1;
    uint32_t e;
    int Fx, Fy, Fz;                   // faces ahead of the box
    if constexpr (is_indexed(DT)) {
        e = indexed_entry(A.sp, R, w, Fx, Fy, Fz);
    } else {
        e = box_entry<DT, PART>(A.map, R, w, ex, ey, ez);
        Fx = ex + (int)(e & 31u);
        Fy = ey + (int)((e >> 5) & 31u);
        Fz = ez + (int)((e >> 10) & 31u);
    }
    if (e >= kBoxOccupied) {
        const uint32_t at = (((uint32_t)w.ux & 1u) | (((uint32_t)w.uy & 1u) << 1) | (((uint32_t)w.uz & 1u) << 2)) ^ R.flip;
        if (((e >> at) & 1u) != 0u && w.t >= t_first) {
            w.left = kWalkHit;
            return;
        }
        // the voxel's own faces, or those of the free voxel layer that it lies in
        const uint32_t axis = (e >> 9) & 3u;
        const bool in = (((at >> axis) ^ (e >> 8)) & 1u) == 0u;
        const int reach = (int)((e >> 10) & 30u);
        Fx = (in & (axis != 0u)) ? ex + reach : w.ux + 1;
        Fy = (in & (axis != 1u)) ? ey + reach : w.uy + 1;
        Fz = (in & (axis != 2u)) ? ez + reach : w.uz + 1;
    }
    const float Tx = box_crossing(Fx, R.gsx, R.arx), Ty = box_crossing(Fy, R.gsy, R.ary), Tz = box_crossing(Fz, R.gsz, R.arz);
    const float t1 = __builtin_amdgcn_fmed3f(Tx, fminf(Ty, Tz), -kInf);
    const float yx = fmaf(t1, fabsf(R.rx), R.hsx), yy = fmaf(t1, fabsf(R.ry), R.hsy), yz = fmaf(t1, fabsf(R.rz), R.hsz);
    const float near = __builtin_amdgcn_fmed3f(fraction(yx), fraction(yy), fraction(yz));
    if ((near < 2.0f * R.tol) | (t1 >= t_end)) {
        // the segment's end, or (away from near-ties) the grid's surface; else decide in float64
        if (t1 > t_hi || (near >= 2.0f * R.tol && t1 < t_lo) || !box_step64(A, R, w, Fx, Fy, Fz, t_lo, t_hi)) {
            w.left = kWalkEnded;
            return;
        }
    } else {
        w.ux = floor_int(yx);
        w.uy = floor_int(yy);
        w.uz = floor_int(yz);
        w.t = t1;
    }
    --w.left;
}

// How a segment's walk ended without a hit: whether the ray's walk ended in it, and then the
// last voxel entered.
struct BoxEnd {
    bool ended;
    bool range;                       // at max_range (else at the grid's surface)
    double t64;                       // grid's surface: parameter and axis of the crossing, when it
    int a;                            //   lies near max_range
    int ux, uy, uz;
};

__device__ __forceinline__ BoxEnd box_end(const RayArgs &A, const BoxRay &R, const BoxWalk &w, bool last, float t_lo,
                                          float t_hi)
{
    const MapView &m = A.map;
    const int ex = signed_edge(m, R.rx, m.nx), ey = signed_edge(m, R.ry, m.ny), ez = signed_edge(m, R.rz, m.nz);
    BoxEnd o;
    o.t64 = __builtin_huge_val();
    o.a = 2;
    bool leaves = R.t_exit < (last ? t_lo : t_hi);
    // the grid's surface in float64: its axis (lowest on ties) and parameter
    double s64 = __builtin_huge_val();
    int sa = 0;
    const float t_range = 0.5f * (A.tmax_lo + A.tmax_hi);             // max_range / h
    float t = leaves ? R.t_exit : t_range;
    const float tol = box_tol(m, t);
    const float ox = off_middle(fmaf(t, fabsf(R.rx), R.gsx)), oy = off_middle(fmaf(t, fabsf(R.ry), R.gsy));
    const float oz = off_middle(fmaf(t, fabsf(R.rz), R.gsz));
    const float near_one = fmaxf(ox, fmaxf(oy, oz)), near_two = __builtin_amdgcn_fmed3f(ox, oy, oz);
    const bool band = last && !leaves && R.t_exit <= t_hi;
    const bool exact = band || (leaves ? near_two : near_one) >= 0.5f - tol;
    if (exact) {
        s64 = signed_face64(ex, A.g[0], R.rx);
        const double Y = signed_face64(ey, A.g[1], R.ry), Z = signed_face64(ez, A.g[2], R.rz);
        if (Y < s64) { sa = 1; s64 = Y; }
        if (Z < s64) { sa = 2; s64 = Z; }
        if (band && s64 * A.h <= A.max_range) {
            leaves = true;
            t = R.t_exit;
            o.t64 = s64;
            o.a = sa;
        }
    }
    o.range = last && !leaves;
    o.ended = leaves || o.range;
    int u[3];
    const int lo[3] = {w.ux, w.uy, w.uz}, edge[3] = {ex, ey, ez};
    const float gs[3] = {R.gsx, R.gsy, R.gsz}, r[3] = {R.rx, R.ry, R.rz};
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const float y = fmaf(t, fabsf(r[b]), gs[b]);
        int c = (int)floorf(y);
        if (exact && off_middle(y) >= 0.5f - tol) {
            // is the nearest face crossed?
            c = (int)floorf(y + 0.5f);
            const double f = signed_face64(c, A.g[b], r[b]);
            const bool crossed = leaves ? f < s64 || (f == s64 && b < sa) : f * A.h <= A.max_range;
            c = crossed ? c : c - 1;
        }
        u[b] = max(lo[b], min(c, edge[b] - 1));
    }
    o.ux = u[0]; o.uy = u[1]; o.uz = u[2];
    return o;
}

// Whether a crossing of the walk up to parameter t64 along axis a (+inf: all) lies within 1e-5
// voxel of max_range.
__device__ __forceinline__ bool box_range_tie(const RayArgs &A, const BoxRay &R, double t64, int a)
{
    const MapView &m = A.map;
    const float t = 0.5f * (A.tmax_lo + A.tmax_hi);
    // a crossing that far from max_range leaves its face up to 1e-5 from the ray's point there
    const float tol = box_tol(m, t) + 1.1e-5f;
    const int n[3] = {m.nx, m.ny, m.nz};
    const float gs[3] = {R.gsx, R.gsy, R.gsz}, r[3] = {R.rx, R.ry, R.rz};
    bool tie = false;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const float y = fmaf(t, fabsf(r[b]), gs[b]);
        if (off_middle(y) < 0.5f - tol) continue;
        const int c = (int)floorf(y + 0.5f);
        if (c <= signed_voxel(r[b], A.v0[b]) || c > signed_edge(m, r[b], n[b])) continue;
        const double f = signed_face64(c, A.g[b], r[b]);
        if (fabs(f * A.h - A.max_range) < 1e-5 * A.h && (f < t64 || (f == t64 && b <= a))) tie = true;
    }
    return tie;
}

// Put the walk into a voxel a little before parameter t_first.  Where a face may lie on either side
// of the float32 position the voxel is the one behind it, which the ray need not pass: the walk
// leaves it at a crossing before t_first, and from there on is the ray's own.  (The voxel ahead of a
// face that is still to be crossed would leave out the voxels until then: an error of 0.004 voxel
// across a face is 0.1 along a ray that crosses it at 0.04.)  Returns false past the grid.
__device__ __forceinline__ bool box_start(const RayArgs &A, const BoxRay &R, float t_first, BoxWalk &w)
{
    const MapView &m = A.map;
    const float t = t_first - fmaxf(kSegOverlap, 2.0f * R.tol);
    w.ux = max(w.ux, min((int)floorf(fmaf(t, fabsf(R.rx), R.gsx) - R.tol), signed_edge(m, R.rx, m.nx) - 1));
    w.uy = max(w.uy, min((int)floorf(fmaf(t, fabsf(R.ry), R.gsy) - R.tol), signed_edge(m, R.ry, m.ny) - 1));
    w.uz = max(w.uz, min((int)floorf(fmaf(t, fabsf(R.rz), R.gsz) - R.tol), signed_edge(m, R.rz, m.nz) - 1));
    return t < R.t_exit;
}

// Start walking segment seg of S of a ray: its start voxel and its end.  Returns false for a
// segment that starts past the grid.
__device__ __forceinline__ bool box_segment(const RayArgs &A, const BoxRay &R, int seg, int S, BoxWalk &w, bool &last,
                                            float &t_lo, float &t_hi, float &t_first)
{
    const float len = (float)A.tmax_v / (float)S;
    w.ux = signed_voxel(R.rx, A.v0[0]);
    w.uy = signed_voxel(R.ry, A.v0[1]);
    w.uz = signed_voxel(R.rz, A.v0[2]);
    w.t = -1.0f;
    w.left = kWalkEnded;
    w.tie = 0u;
    last = seg == S - 1;
    t_lo = last ? A.tmax_lo : kInf;
    t_hi = last ? A.tmax_hi : len * (float)(seg + 1);
    t_first = len * (float)seg;       // (segment 0 starts in a free voxel)
    if (seg == 0) return true;
    return box_start(A, R, t_first, w);
}

// A segment's result once its walk has stopped.
struct BoxResult {
    bool ended;                       // the ray's walk ends in this segment
    double d;                         // hit distance, metres (+inf without a hit)
    bool rtie;
    int fx, fy, fz;                   // last voxel entered when ended
};

__device__ __forceinline__ BoxResult box_finish(const RayArgs &A, const BoxRay &R, const BoxWalk &w, bool last,
                                                float t_lo, float t_hi)
{
    BoxResult o;
    o.d = __builtin_huge_val();
    o.rtie = false;
    int ux = w.ux, uy = w.uy, uz = w.uz;
    if (w.left == kWalkHit) {
        o.ended = true;
        // the hit voxel was entered across the last crossed of its three faces behind (a face
        // behind the start has a parameter <= 0); its axis matters only beside max_range, where
        // the highest axis of equal crossings is the last one
        const float Tx = R.rx != 0.0f ? box_crossing(ux, R.gsx, R.arx) : -kInf;
        const float Ty = R.ry != 0.0f ? box_crossing(uy, R.gsy, R.ary) : -kInf;
        const float Tz = R.rz != 0.0f ? box_crossing(uz, R.gsz, R.arz) : -kInf;
        const float t1 = fmaxf(Tx, fmaxf(Ty, Tz)), t2 = __builtin_amdgcn_fmed3f(Tx, Ty, Tz);
        int a = Tx == t1 ? 0 : (Ty == t1 ? 1 : 2);
        // (one division for the lanes of all axes)
        const float gx = A.g[0], gy = A.g[1], gz = A.g[2];
        const float ra = a == 0 ? R.rx : (a == 1 ? R.ry : R.rz), ga = a == 0 ? gx : (a == 1 ? gy : gz);
        const int ua = a == 0 ? ux : (a == 1 ? uy : uz);
        double t64 = face64(ra > 0.0f ? ua : -ua, ga, ra);
        if (t1 - t2 <= 1e-5f + 1e-6f * t1) {
            const double huge = __builtin_huge_val();
            const double X = R.rx != 0.0f ? signed_face64(ux, A.g[0], R.rx) : -huge;
            const double Y = R.ry != 0.0f ? signed_face64(uy, A.g[1], R.ry) : -huge;
            const double Z = R.rz != 0.0f ? signed_face64(uz, A.g[2], R.rz) : -huge;
            a = 0;
            t64 = X;
            if (Y >= t64) { a = 1; t64 = Y; }
            if (Z >= t64) { a = 2; t64 = Z; }
        }
        o.d = t64 * A.h;
        if (w.t >= t_lo) o.rtie = box_range_tie(A, R, t64, a);
    } else {
        const BoxEnd e = box_end(A, R, w, last, t_lo, t_hi);
        o.ended = e.ended;
        ux = e.ux; uy = e.uy; uz = e.uz;
        if (e.range || (e.ended && e.t64 < __builtin_huge_val())) o.rtie = box_range_tie(A, R, e.t64, e.a);
    }
    o.fx = signed_voxel(R.rx, ux);
    o.fy = signed_voxel(R.ry, uy);
    o.fz = signed_voxel(R.rz, uz);
    return o;
}

}  // namespace rmpc
