// Slabs of planes of the two-kernel 3D executor: how many planes a slab holds,
// and which planes a launch of it covers.  Host arithmetic only.
#pragma once

#include <stdint.h>

namespace fdtdp {

constexpr int kSlabSteps = 16;     // steps taken on a slab before the next
// Fewer steps than this go over the whole grid: the cache serves a slab's second
// step only (step(1): 384^3 FP32 1375 us in slabs, 1295 over the whole grid; step(2),
// a step: 1278 in slabs, 1292).
constexpr int kSlabLeast = 2;
constexpr int64_t kSlabAbove = 192LL << 20, kSlabBytes = 100LL << 20, kSlabMin = 24;

// Planes of an x slab of a walled grid of nx planes of plane_bytes (E and H),
// in whole runs of the ni planes a thread walks; 0: the whole grid at once.
// A grid that does not fit the 256 MB memory-side cache is stepped in slabs
// that do, kSlabSteps steps on each before the next.  Around 100 MB of fields a
// slab: 256^3 FP64 849 -> 774 us a step, 384^3 FP32 1297 -> 1185, where 200 MB
// gain 1% and 50 MB cost as much in launches.  A slab has at least kSlabSteps
// planes, so that the first one, which ends a plane lower every step
// (slab_range), still holds one at the last of them.
inline int64_t slab_planes(int64_t nx, int64_t plane_bytes, int64_t ni)
{
    if (nx * plane_bytes <= kSlabAbove) return 0;
    const int64_t most = kSlabBytes / plane_bytes > kSlabMin ? kSlabBytes / plane_bytes : kSlabMin;
    const int64_t n = (nx + most - 1) / most;
    int64_t L = (nx + n - 1) / n;
    if (L < kSlabSteps) L = kSlabSteps;
    L = (L + ni - 1) / ni * ni;
    return L < nx ? L : 0;
}

// The planes [ia, ib) that step t (from 0) of the slab at plane s covers: the t
// below the slab's, so that every H finds the E of the plane above it one step
// behind and every E the H of the plane below already advanced.
struct SlabRange {
    int64_t ia, ib;
};
inline SlabRange slab_range(int64_t nx, int64_t L, int64_t s, int t)
{
    return {s > t ? s - t : 0, s + L < nx ? s + L - t : nx};
}

}  // namespace fdtdp
