// Values that cross workgroups inside one launch: the workgroups that share a vocabulary row leave one 8-byte word each
// (or a few) and take those of the others.
//
// Words travel as relaxed agent-scope atomic stores and loads (write-through / read-through to the level all compute units
// share; each XCD has its own L2), a value and "it is there" in the same 8 bytes, so nothing has to be acknowledged first
// and no cache is written back or invalidated.  MI355X, publish to all seen: 0.6-1.0 us with up to 512 workgroups exchanging
// at once, 1.7 us with 1024, 3 us with 2048, all of which poll the same few lines; and 2048 workgroups take 4.8 us to start,
// 512 take 1.2.  So rows are shared by FEW workgroups of 1024 threads.
//
// Nobody depends on being met: a workgroup looks for the words of the others kPatience times at most and then computes
// what is missing itself, with the same instructions on the same inputs and so with the same result.  Whether all parts of
// a row are resident at once, and in which order they run, decides how long a launch takes and nothing else.
#pragma once
#include "device_utils.h"

namespace adaspec {

// Looks at the others' words, about 0.7 us each.  Parts of a row are neighbours in the grid, so that they start within a few
// microseconds of each other; the limit matters only where something else holds the compute units.
#ifndef ADASPEC_PATIENCE
#define ADASPEC_PATIENCE 64
#endif
constexpr int kPatience = ADASPEC_PATIENCE;

constexpr unsigned long long kNoWord = ~0ull;         // what an earlier kernel of the call leaves in every word

__device__ __forceinline__ void publish_u64(void *p, unsigned long long v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long fetch_u64(const void *p)
{
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a sum as a word (any NaN becomes the one that is not kNoWord)
__device__ __forceinline__ unsigned long long word_of(double x)
{
    return x != x ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(x);
}
__device__ __forceinline__ double double_of(unsigned long long w) { return __longlong_as_double((long long)w); }

// One wavefront: lane t with `wanted` takes the word at `p`; up to `looks` times, until all are there.  Returns the
// lane's word (kNoWord: not there, or not wanted).
__device__ __forceinline__ unsigned long long take_words(const unsigned long long *p, bool wanted, int looks)
{
    unsigned long long w = kNoWord;
    for (int n = 0; n < looks; ++n) {
        if (wanted && w == kNoWord) w = fetch_u64(p);
        if (__ballot(wanted && w == kNoWord) == 0ull) break;
    }
    return w;
}

}  // namespace adaspec
