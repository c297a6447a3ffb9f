// How the eight waves of a workgroup share the groups of its split of K (w4_slices.hip, bf16_rows.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace dmr {

constexpr int kSharingWaves = 8;

struct WaveShare {
    int g0, n;      // groups [g0, g0 + n)
};
inline __host__ __device__ WaveShare wave_share(int groups, int gps, int split, int wave) {
    const int gA = split * gps, ng = groups - gA < gps ? groups - gA : gps;
    const int per = ng / kSharingWaves, rest = ng % kSharingWaves;
    return {gA + wave * per + (wave < rest ? wave : rest), per + (wave < rest ? 1 : 0)};
}

// The group that a request for a wave's i-th one names.  Past the wave's last the request goes to a resource of no bytes, so that the
// number of loads in flight never changes; it names a group of the layer all the same, so that nothing rests on whether the bounds
// check of a buffer load counts the scalar offset.
inline __host__ __device__ int requested_group(const WaveShare &s, int i, int groups) {
    return s.g0 + i < groups ? s.g0 + i : groups - 1;
}

}  // namespace dmr
