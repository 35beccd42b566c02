// The start vector of Alg. 1 (device code shared by the single and the batched driver).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hub {

// SplitMix64 (Steele, Lea & Flood 2014): output k of the stream started at
// `seed` is the published finaliser applied to seed + k * 0x9E3779B97F4A7C15.
__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + k * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Element J of the random start vector: 2u - 1 with u = top 53 bits / 2^53.
__device__ inline double start_value(uint64_t seed, int64_t J)
{
    const double u = (double)(splitmix64_at(seed, (uint64_t)J + 1) >> 11) * 0x1.0p-53;
    return 2.0 * u - 1.0;
}

__device__ inline double start_or_given(const double *__restrict__ given, uint64_t seed, int64_t J)
{
    return given ? given[J] : start_value(seed, J);
}

}  // namespace hub
