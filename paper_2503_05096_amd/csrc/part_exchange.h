// Values that cross workgroups inside one launch: the workgroups that share a vocabulary row leave one 8-byte word each
// (or a few) and take those of the others.
//
// Words travel as relaxed agent-scope atomic stores and loads (write-through / read-through to the level all compute units
// share; each XCD has its own L2), a value and "it is there" in the same 8 bytes, so nothing has to be acknowledged first
// and no cache is written back or invalidated.  MI355X, publish to all seen: 0.6-1.0 us with up to 512 workgroups exchanging
// at once, 1.7 us with 1024, 3 us with 2048, all of which poll the same few lines; and 2048 workgroups take 4.8 us to start,
// 512 take 1.2.  So rows are shared by FEW workgroups, of 512 or 1024 threads.
//
// Nobody depends on being met: a workgroup looks for a word of another one ADASPEC_PATIENCE times at most and then computes
// what is missing itself, with the same instructions on the same inputs and so with the same result.  Whether all parts of
// a row are resident at once, and in which order they run, decides how long a launch takes and nothing else.  What that costs: 13 us
// per exchange for 64 looks in vain, and the parts that are missing (if nobody ever meets, patience 0, captured calls: draft
// sampling of 128 rows of V = 128256 19 -> 40 us, of 8 of V = 524288 in fp32 14 -> 253; acceptance of 64 fp32 rows 35 -> 102; walks of 64 trees
// 32 -> 63).  A workgroup that starts when the others have left finds their words where a kernel of the call clears them, and taken back
// where marks are used.
#pragma once
#include "device_utils.h"

namespace adaspec {

// Looks at the others' words, 0.2 us each while nobody writes and up to 0.7 while the others publish.  Parts of a row are neighbours in the grid, so that they start within a few
// microseconds of each other; the limit matters only where something else holds the compute units.
// (Tests build the library with other numbers, also with one that differs from word to word.)
#ifndef ADASPEC_PATIENCE
#define ADASPEC_PATIENCE(word) 64
#endif

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

// One wavefront: lane t with `wanted` takes the word at `p`, once all are there or patience has run out.  Returns the
// lane's word (kNoWord: not there, or not wanted).
__device__ __forceinline__ unsigned long long take_words(const unsigned long long *p, bool wanted)
{
    unsigned long long w = kNoWord;
    const int looks = ADASPEC_PATIENCE(p);
    for (int n = 0; n < looks; ++n) {
        if (wanted && w == kNoWord) w = fetch_u64(p);
        if (__ballot(wanted && w == kNoWord) == 0ull) break;
    }
    return w;
}

// Words that no earlier kernel of the call has cleared: the value, and the value with the launch's mark folded in.  A pair is
// there if its halves differ by exactly the mark; marks are spread over all 64 bits and never given twice, so that leftovers
// of whatever kind, or one half of an old pair beside one of a new one, do not look like it.  A captured launch keeps its
// mark: what one replay leaves must be taken back before the next could read it (see the kernels).
struct MarkedWord { unsigned long long value, check; };
__device__ __forceinline__ void publish_marked(MarkedWord *p, unsigned long long v, unsigned long long mark)
{
    publish_u64(&p->value, v);
    publish_u64(&p->check, v ^ mark);
}
__device__ __forceinline__ void take_back(MarkedWord *p)
{
    publish_u64(&p->value, 0ull);
    publish_u64(&p->check, 0ull);
}
// One wavefront, like take_words; returns whether the lane has its value.
__device__ __forceinline__ bool take_marked(const MarkedWord *p, bool wanted, unsigned long long mark, unsigned long long &v)
{
    bool there = false;
    const int looks = ADASPEC_PATIENCE(p);
    for (int n = 0; n < looks; ++n) {
        if (wanted && !there) {
            const unsigned long long a = fetch_u64(&p->value), b = fetch_u64(&p->check);
            there = (a ^ b) == mark;
            v = a;
        }
        if (__ballot(wanted && !there) == 0ull) break;
    }
    return there;
}

// One wavefront: where a point of a cumulative mass falls.  Lane t brings the mass of the t-th piece, `before` is the running
// total in front of all of them.  Returns the first piece with mass whose running total exceeds tau, else (rounding left
// none) the last with mass, else -1; `ahead` = running total in front of it.
__device__ __forceinline__ int find_piece(double mass, double before, double tau, int lane, double &ahead)
{
    const double upto = before + wave_scan_incl(mass, lane);
    const unsigned long long cross = __ballot(mass > 0.0 && upto > tau), filled = __ballot(mass > 0.0);
    const int at = cross ? (int)__builtin_ctzll(cross) : (filled ? 63 - (int)__builtin_clzll(filled) : -1);
    ahead = __shfl(upto - mass, at < 0 ? 0 : at, kWave);
    return at;
}

}  // namespace adaspec
