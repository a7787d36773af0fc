// walk_host.hip -- the dense walk of csrc/rmpc_dense.h compiled for the host, ray by ray and segment by
// segment, combined as the kernels combine a ray's lanes (tests/test_walk_host.py).  The header is the
// library's own; the device builtins it uses have host stand-ins here.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <cstring>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))

static __device__ inline float host_med3(float a, float b, float c)
{
    const float lo = a < b ? a : b, hi = a < b ? b : a;
    return c < lo ? lo : (c > hi ? hi : c);
}
#define __builtin_amdgcn_fmed3f host_med3
#define __float_as_int(x) __builtin_bit_cast(int, (float)(x))
#define __int_as_float(x) __builtin_bit_cast(float, (int)(x))
#define __mul24(a, b) ((a) * (b))
#define __umul24(a, b) ((a) * (b))

#include "rmpc_dense.h"

using namespace rmpc;

namespace {

constexpr int kMostSteps = 100000;      // above the steps of any walk of the tests

template <bool PART>
bool one_ray(const RayArgs &A, const float *dir, int S, int32_t *hit, double *d, uint8_t *flags, int32_t *visits)
{
    const BoxRay R = box_ray<RMPC_TSDF_F32>(A, dir[0], dir[1], dir[2]);
    *hit = -1;
    *d = HUGE_VAL;
    *flags = (uint8_t)A.start_flags;
    bool found = false, ended = false;
    for (int seg = 0; seg < S && !found; ++seg) {
        BoxWalk w;
        bool last;
        float t_lo, t_hi, t_first;
        const bool ran = box_segment(A, R, seg, S, w, last, t_lo, t_hi, t_first);
        const float t_end = fminf(R.t_exit, last ? t_lo : t_hi);
        w.left = ran ? 0 : kWalkEnded;
        for (int n = 0; w.left >= 0; ++n) {
            if (n == kMostSteps) return false;
            w.left = 1;
            box_step<RMPC_TSDF_F32, PART>(A, R, w, t_end, t_lo, t_hi, t_first);
        }
        found = w.left == kWalkHit;
        const BoxResult e = box_finish(A, R, w, last, t_lo, t_hi);
        if (!ran) continue;
        *flags |= (w.tie ? RMPC_RAY_TIE : 0u) | (e.rtie ? RMPC_RAY_RANGE_TIE : 0u);
        if (e.ended && !ended) {
            // (the lowest segment whose walk ended holds the last voxel)
            ended = true;
            *visits = 1 + abs(e.fx - A.v0[0]) + abs(e.fy - A.v0[1]) + abs(e.fz - A.v0[2]);
        }
        if (found) {
            *hit = e.fx + A.map.nx * (e.fy + A.map.ny * e.fz);
            *d = e.d;
        }
    }
    return ended;
}

}  // namespace

// Walk n rays of S segments from grid position g in a float32 grid with box entries; false when a walk
// does not end.
extern "C" int walk_rays(const float *grid, const uint16_t *box, const int32_t *dims, const int32_t *bricks, const float *g,
                         double h, double max_range, const float *dirs, int n, int S, int32_t *hit, double *d,
                         uint8_t *flags, int32_t *visits)
{
    RayArgs A;
    memset(&A, 0, sizeof A);
    A.map.data = grid;
    A.map.box = box;
    A.map.nx = dims[0]; A.map.ny = dims[1]; A.map.nz = dims[2];
    A.map.nbx = bricks[0]; A.map.nby = bricks[1]; A.map.nbz = bricks[2];
    A.map.partial = 2 * bricks[0] < dims[0] || 2 * bricks[1] < dims[1] || 2 * bricks[2] < dims[2];
    A.map.span = dims[0] > dims[1] ? (dims[0] > dims[2] ? dims[0] : dims[2]) : (dims[1] > dims[2] ? dims[1] : dims[2]);
    for (int a = 0; a < 3; ++a) {
        A.g[a] = g[a];
        A.v0[a] = (int32_t)floor(g[a]);
        const double fr = (double)g[a] - floor((double)g[a]);
        if (fr < 1e-5 || 1.0 - fr < 1e-5) A.start_flags |= RMPC_RAY_START_FACE;
    }
    const double tmax = max_range / h;
    A.tmax_lo = (float)(tmax * (1.0 - 1e-6) - 2e-5);
    A.tmax_hi = (float)(tmax * (1.0 + 1e-6) + 2e-5);
    A.tmax_v = fmin(tmax, sqrt((double)dims[0] * dims[0] + (double)dims[1] * dims[1] + (double)dims[2] * dims[2]) + 2.0);
    A.max_range = max_range;
    A.h = h;
    for (int i = 0; i < n; ++i) {
        const bool ok = A.map.partial ? one_ray<true>(A, dirs + 3 * i, S, hit + i, d + i, flags + i, visits + i)
                                      : one_ray<false>(A, dirs + 3 * i, S, hit + i, d + i, flags + i, visits + i);
        if (!ok) return 0;
    }
    return 1;
}
