// Vocabulary rows cut into PARTS that small workgroups (256 threads) sweep, or that larger ones (512, 1024) hold in registers: the
// pieces shared by the acceptance
// (accept_parts.hip, accept_shared.hip), draft sampling (draft_parts.hip) and trees (tree_fast.hip).  A row is a sequence
// of CHUNKS of 16 bytes of logits (8 elements of 16 bits, 4 of fp32) with as many probabilities beside them; a STEP is
// one chunk per thread.
#pragma once
#include "adaspec_internal.h"
#include "device_utils.h"
#include "row_registers.h"

namespace adaspec {

constexpr int kQT = 256;                    // threads per workgroup
constexpr int kQW = kQT / kWave;            // 4 wavefronts
constexpr int kStatSteps = 8;               // statistics pass: steps in flight, and the shortest part (32 KB of logits)
constexpr int kStatWgsPerCu = 6;            // ... workgroups that fit a compute unit (80 registers each)
constexpr int kStatTargetWgsPerCu = 3;      // ... and how many the launch aims for: few long streams read faster than many short ones
constexpr int kStatParts = 8;               // ... parts per row at most, of up to 64 steps: V <= 8 * 64 * 256 * 4 = 524288
constexpr int kSumSteps = 4;                // mass pass: steps per part
constexpr int kSumChunks = kSumSteps * kQT; // ... chunks per part (16 KB of logits)
constexpr int kSumParts = 128;              // ... parts per row at most
constexpr int kPartsMaxVocab = 524288;
static_assert(kSumSteps == kQW, "one wavefront per step in the final search");
static_assert(kSumParts * kQW == 2 * kQT, "two (part, wavefront) pairs per thread in the final search");
static_assert(kPartsMaxVocab <= kSumParts * kSumChunks * 4 && kPartsMaxVocab <= kStatParts * 64 * kQT * 4, "fp32 rows fit");

// 16 bytes per lane through a buffer descriptor (past the end of the buffer: zeros); AUX = cache policy bits
// of the instruction (0 = default, 2 = non-temporal: data that is read once)
constexpr int kAuxDefault = 0, kAuxStream = 2;
template <int AUX>
__device__ __forceinline__ uint4 part_load16(__amdgpu_buffer_rsrc_t rs, uint32_t lane_offset, int step_offset)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)lane_offset, step_offset, AUX);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// ---- chunks of logits -------------------------------------------------------------------------------
template <class LT> struct Chunk {                    // 16-bit types
    using P = Pair16<LT>;
    static constexpr int kN = 8;
    static __device__ __forceinline__ void unpack(const uint4 &v, float (&x)[kN])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[2 * e] = P::lo(w[e]); x[2 * e + 1] = P::hi(w[e]); }
    }
    // chunks past the end of the row arrive as zeros (range check of the buffer) and become -inf in place
    static __device__ __forceinline__ void blank(uint4 &v, bool past)
    {
        const uint32_t ninf = past ? P::kNegInf2 : 0u;
        v.x |= ninf; v.y |= ninf; v.z |= ninf; v.w |= ninf;
    }
};
template <> struct Chunk<F32> {
    static constexpr int kN = 4;
    static __device__ __forceinline__ void unpack(const uint4 &v, float (&x)[kN])
    {
        x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y); x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ void blank(uint4 &v, bool past)
    {
        constexpr uint32_t kNegInf = 0xff800000u;
        v.x = past ? kNegInf : v.x; v.y = past ? kNegInf : v.y; v.z = past ? kNegInf : v.z; v.w = past ? kNegInf : v.w;
    }
};

// ---- the draft probabilities beside a chunk of N logits: 8, 16 or 32 bytes ----------------------------
template <int N, class PT> struct ProbChunk {
    static constexpr int kBytes = N * (int)sizeof(typename PT::storage);
    uint32_t w[kBytes / 4];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int k = 0; k < kBytes / 4; ++k) w[k] = 0u;
    }
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t lane_offset, int step_offset)
    {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        if constexpr (kBytes == 8) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)lane_offset, step_offset, kAuxDefault);
            w[0] = v.x; w[1] = v.y;
        } else {
#pragma unroll
            for (int k = 0; k < kBytes / 16; ++k) {
                const uint4 v = part_load16<kAuxDefault>(rs, lane_offset + 16 * k, step_offset);
                w[4 * k] = v.x; w[4 * k + 1] = v.y; w[4 * k + 2] = v.z; w[4 * k + 3] = v.w;
            }
        }
    }
    __device__ __forceinline__ void unpack(float (&x)[N]) const
    {
        if constexpr (sizeof(typename PT::storage) == 4) {
#pragma unroll
            for (int e = 0; e < N; ++e) x[e] = __uint_as_float(w[e]);
        } else {
#pragma unroll
            for (int e = 0; e < N / 2; ++e) { x[2 * e] = Pair16<PT>::lo(w[e]); x[2 * e + 1] = Pair16<PT>::hi(w[e]); }
        }
    }
    __device__ __forceinline__ void keep()            // opaque to the optimiser (see keep_packed)
    {
#pragma unroll
        for (int k = 0; k < kBytes / 4; ++k) asm volatile("" : "+v"(w[k]));
    }
};

// 2^((l - m) c).  16-bit logits: one fused operation, relative to mc = scaled_ref(m, c).  fp32
// logits: the difference first, as the portable kernel does it.
template <class LT>
__device__ __forceinline__ float exp_weight(float l, float m, float c, float mc)
{
    if constexpr (sizeof(typename LT::storage) == 4) return __builtin_amdgcn_exp2f((l - m) * c);
    else return __builtin_amdgcn_exp2f(fmaf(l, c, -mc));
}

// exponent that moves a sum of such weights from the reference a to the reference b
template <class LT>
__device__ __forceinline__ float ref_gap(float a, float b, float c)
{
    if constexpr (sizeof(typename LT::storage) == 4) return (a - b) * c;
    else return scaled_ref(a, c) - scaled_ref(b, c);
}

// exact maximum of the values of a chunk
template <class LT>
__device__ __forceinline__ float chunk_max(const uint4 &v, float m)
{
    float x[Chunk<LT>::kN];
    Chunk<LT>::unpack(v, x);
#pragma unroll
    for (int e = 0; e < Chunk<LT>::kN; ++e) m = fmaxf(m, x[e]);
    return m;
}

// Exact maximum of a thread's STEPS chunks.  16-bit types: on the bit patterns.  Both are sign-magnitude:
// among non-negative values the order of the patterns as SIGNED 16-bit integers is the order of the
// values, and every negative value is a negative integer, so a packed signed maximum (one instruction per
// two elements) is exact as soon as one value is >= +0.  A thread that holds nothing but negative values
// (masked vocabularies) wants the smallest magnitude instead: the packed UNSIGNED minimum.
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
template <class LT, int STEPS>
__device__ __forceinline__ float thread_max(const uint4 (&lg)[STEPS])
{
    if constexpr (sizeof(typename LT::storage) == 4) {
        float m = -INFINITY;
#pragma unroll
        for (int it = 0; it < STEPS; ++it) m = chunk_max<LT>(lg[it], m);
        return m;
    } else {
        short2v pm = {(short)0x8000, (short)0x8000};
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {
            const uint32_t w[4] = {lg[it].x, lg[it].y, lg[it].z, lg[it].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) pm = __builtin_elementwise_max(pm, __builtin_bit_cast(short2v, w[e]));
        }
        int top = max((int)pm.x, (int)pm.y);
        if (top < 0) {
            ushort2v pn = {(unsigned short)0xffff, (unsigned short)0xffff};
#pragma unroll
            for (int it = 0; it < STEPS; ++it) {
                const uint32_t w[4] = {lg[it].x, lg[it].y, lg[it].z, lg[it].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) pn = __builtin_elementwise_min(pn, __builtin_bit_cast(ushort2v, w[e]));
            }
            top = min((int)pn.x, (int)pn.y);
        }
        return Pair16<LT>::lo((uint32_t)top & 0xffffu);
    }
}

// The same, with NaNs passed over as chunk_max does it (the packed maximum of a thread that holds one is that NaN): for
// parts that another workgroup may have to compute chunk by chunk, from the same maxima.
template <class LT, int STEPS>
__device__ __forceinline__ float thread_max_of_numbers(const uint4 (&lg)[STEPS])
{
    float m = thread_max<LT, STEPS>(lg);
    if (sizeof(typename LT::storage) == 2 && m != m) {
        m = -INFINITY;
#pragma unroll
        for (int it = 0; it < STEPS; ++it) m = chunk_max<LT>(lg[it], m);
    }
    return m;
}

// ---- one part of a row, streamed once ------------------------------------------------------------------------------
// Part h takes the steps h, h + n_parts, h + 2 n_parts, ... of the row, so that the workgroups of a row sweep it together
// (neighbouring addresses are in flight at the same time), and reads them past the caches when the row is read only here.
// kStatSteps steps are in flight, each consumed as it lands: a compute unit needs about as long for the exponentials of
// a row as the memory system needs to deliver it, and only a stream whose arithmetic runs under its own loads gets both
// done in the time of one.  `issued` runs once the first loads are under way.
//   !kArgMax maximum and normaliser on line, against the thread's running maximum m_run.  Both 16-bit formats are
//            sign-magnitude: among non-negative values the order of the bit patterns as SIGNED 16-bit integers is the
//            order of the values and every negative value is a negative integer, so a running packed signed maximum (one
//            instruction per two elements) is the exact maximum as soon as the thread has seen one value >= +0; until
//            then (masked vocabularies) the chunk's float maximum is taken the slow way.  fp32 chunks (half as many
//            elements per byte) take the float maximum throughout.
//   kArgMax  arg-max, lowest index on ties (a thread meets its elements in index order)
struct PartStream { float m_run, zt; ArgMax best; };
template <class LT, bool kArgMax, int AUX, class F>
__device__ __forceinline__ PartStream stream_part(__amdgpu_buffer_rsrc_t rl, int row_chunks, int n_parts, int h, int V, float c,
                                                  int tid, F issued)
{
    constexpr int kN = Chunk<LT>::kN;
    const int steps = (ceil_div(row_chunks, kQT) - h + n_parts - 1) / n_parts;
    const uint32_t tid16 = (uint32_t)tid * 16u;
    PartStream out;
    const float lowest = lowest_ref<LT>(c);              // (m_run until something above it comes)
    out.m_run = lowest; out.zt = 0.f; out.best = ArgMax{-INFINITY, V};
    short2v pm = {(short)0x8000, (short)0x8000};
    uint4 lg[kStatSteps];
#pragma unroll
    for (int u = 0; u < kStatSteps; ++u) lg[u] = part_load16<AUX>(rl, tid16, (u * n_parts + h) * (kQT * 16));
    issued();
    for (int s0 = 0; s0 < steps; s0 += kStatSteps) {
#pragma unroll
        for (int u = 0; u < kStatSteps; ++u) {
            const int chunk = ((s0 + u) * n_parts + h) * kQT + tid;
            uint4 v = lg[u];
            Chunk<LT>::blank(v, chunk >= row_chunks);
            float x[kN];
            float mn;                                        // maximum so far
            if constexpr (kArgMax) {
                mn = chunk_max<LT>(v, out.best.v);
                if (mn > out.best.v) {                       // (rarely: the search stays off the common path)
                    Chunk<LT>::unpack(v, x);
                    int at = 0;
#pragma unroll
                    for (int e = kN - 1; e >= 0; --e) at = x[e] == mn ? e : at;
                    out.best = ArgMax{mn, chunk * kN + at};
                }
            } else {
                if constexpr (kN == 4) {
                    mn = chunk_max<LT>(v, out.m_run);
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) pm = __builtin_elementwise_max(pm, __builtin_bit_cast(short2v, w[e]));
                    const int top = max((int)pm.x, (int)pm.y);
                    mn = top >= 0 ? Pair16<LT>::lo((uint32_t)top & 0xffffu) : chunk_max<LT>(v, out.m_run);
                }
                if (mn > out.m_run) {
                    out.zt *= __builtin_amdgcn_exp2f(ref_gap<LT>(out.m_run, mn, c));      // (-inf - finite) -> 0
                    out.m_run = mn;
                }
                if (out.m_run > lowest) {
                    const float mnc = scaled_ref(out.m_run, c);
                    Chunk<LT>::unpack(v, x);
#pragma unroll
                    for (int e = 0; e < kN; ++e) out.zt += exp_weight<LT>(x[e], out.m_run, c, mnc);
                }
            }
            // the request for the step that takes this one's place (past the row: zeros, no traffic)
            lg[u] = part_load16<AUX>(rl, tid16, ((s0 + u + kStatSteps) * n_parts + h) * (kQT * 16));
            __builtin_amdgcn_sched_barrier(0);       // one step at a time: nothing unpacked ahead of its turn
        }
    }
    if (!(out.m_run > lowest)) out.m_run = -INFINITY;
    return out;
}

// over the workgroup: (maximum, normaliser) of the threads' streams; the result is thread 0's
template <class LT>
__device__ __forceinline__ HalfStat reduce_norm(const PartStream &st, float c, float *s_m, double *s_z, int lane, int wv)
{
    const float mw = wave_max(st.m_run);
    const double zw = wave_sum(st.m_run > -INFINITY ? (double)(st.zt * __builtin_amdgcn_exp2f(ref_gap<LT>(st.m_run, mw, c))) : 0.0);
    if (lane == 0) { s_m[wv] = mw; s_z[wv] = zw; }
    lds_barrier();
    HalfStat out;
    out.m = s_m[0]; out.arg = 0; out.Z = 0.0;
#pragma unroll
    for (int w = 1; w < kQW; ++w) out.m = fmaxf(out.m, s_m[w]);
#pragma unroll
    for (int w = 0; w < kQW; ++w)
        out.Z += s_m[w] > -INFINITY ? s_z[w] * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(s_m[w], out.m, c)) : 0.0;
    return out;
}
// over the workgroup: arg-max (index >= V if nothing is above -inf)
__device__ __forceinline__ ArgMax reduce_argmax(ArgMax best, float *s_m, int *s_i, int lane, int wv)
{
    best = wave_argmax(best);
    if (lane == 0) { s_m[wv] = best.v; s_i[wv] = best.i; }
    lds_barrier();
    ArgMax b{s_m[0], s_i[0]};
#pragma unroll
    for (int w = 1; w < kQW; ++w) b = argmax_merge(b, ArgMax{s_m[w], s_i[w]});
    return b;
}

// ---- the (part, wavefront) pair of a row that holds a point of its cumulative mass ------------------------------------
// Thread t of a 256-thread workgroup brings the masses of the pairs 2t and 2t + 1 (0 past the end).  The first barrier of
// pair_totals also makes room in the scratch.
struct PairScratch { double wave[kQW]; double before; int pick[kQW], last[kQW]; };
// running total after this thread's two pairs; R = total of all
__device__ __forceinline__ double pair_totals(PairScratch &s, double both, int tid, int lane, int wv, double &R)
{
    const double incl = wave_scan_incl(both, lane);
    __syncthreads();
    if (lane == 63) s.wave[wv] = incl;
    __syncthreads();
    double before = 0.0;
    R = 0.0;
#pragma unroll
    for (int w = 0; w < kQW; ++w) {
        if (w < wv) before += s.wave[w];
        R += s.wave[w];
    }
    return before + incl;
}
// the first pair with mass whose running total exceeds tau (rounding may leave none: then the last one with mass), or -1;
// s.before = running total in front of it.  (Ballots and one LDS word per wavefront: LDS atomics on one word, which half
// of the threads would hit, took 2 us of a 10 us kernel.)
__device__ __forceinline__ int pick_pair(PairScratch &s, double w0, double w1, double at1, double tau, int tid, int lane, int wv)
{
    const double at0 = at1 - w1;
    const bool hit0 = w0 > 0.0 && at0 > tau, hit1 = w1 > 0.0 && at1 > tau;
    const unsigned long long claims = __ballot(hit0 || hit1), first_of_two = __ballot(hit0);
    const unsigned long long any = __ballot(w0 > 0.0 || w1 > 0.0), second_of_two = __ballot(w1 > 0.0);
    if (lane == 0) {
        const int c = claims ? (int)__builtin_ctzll(claims) : 0, l = any ? 63 - (int)__builtin_clzll(any) : 0;
        s.pick[wv] = claims ? 2 * (kWave * wv + c) + ((first_of_two >> c) & 1 ? 0 : 1) : -1;
        s.last[wv] = any ? 2 * (kWave * wv + l) + ((second_of_two >> l) & 1 ? 1 : 0) : -1;
    }
    __syncthreads();
    int pick = -1, last = -1;
#pragma unroll
    for (int w = 0; w < kQW; ++w) {
        if (pick < 0) pick = s.pick[w];
        last = max(last, s.last[w]);
    }
    if (pick < 0) pick = last;
    if (pick >= 0 && (pick >> 1) == tid) s.before = (pick & 1) ? at0 : at0 - w0;
    __syncthreads();
    return pick;
}
// Inside the pair: wavefront w holds its step w, `mine` = the mass of the lane's chunk.  Returns whether this lane owns
// the point; li = running total after the lane.
__device__ __forceinline__ bool own_point(PairScratch &s, double mine, double tau, int lane, int wv, double &li, bool &none)
{
    const double incl = wave_scan_incl(mine, lane);
    if (lane == 63) s.wave[wv] = incl;                        // (last read behind the barriers of pick_pair)
    __syncthreads();
    // the step: first whose running total exceeds tau, else the last with mass
    double at = s.before, base = 0.0;
    int step = -1;
    bool found = false;
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) {
        const double tot = s.wave[it];
        if (!found && tot > 0.0) {
            step = it; base = at;
            found = at + tot > tau;
        }
        at += tot;
    }
    none = step < 0;
    li = base + incl;
    if (step != wv) return false;
    const unsigned long long lhit = __ballot(mine > 0.0 && li > tau);
    const unsigned long long lpos = __ballot(mine > 0.0);
    const int owner = lhit ? (int)__builtin_ctzll(lhit) : 63 - (int)__builtin_clzll(lpos);   // lpos != 0: the step has mass
    return lane == owner;
}
// the element of the owner's chunk: first with weight whose running total exceeds tau, else the last with weight
template <int N>
__device__ __forceinline__ int pick_element(const float (&w)[N], double cum, double scale, double tau)
{
    int pick = -1, last = -1;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        cum += (double)w[e] * scale;
        if (w[e] > 0.f) last = e;
        if (pick < 0 && w[e] > 0.f && cum > tau) pick = e;
    }
    return pick >= 0 ? pick : max(last, 0);
}

// ---- host side: how rows are cut --------------------------------------------------------------------------------------
inline int parts_chunk_elems(int logits_dtype) { return logits_dtype == ADASPEC_F32 ? 4 : 8; }
inline int parts_sum_parts(int vocab, int logits_dtype) { return ceil_div(vocab / parts_chunk_elems(logits_dtype), kSumChunks); }
// Statistics pass: a part is a stream of 8, 16, 32 or 64 steps.  Short streams spread a row over more compute units; long
// ones read faster (measured on MI355X, acceptance of 382 rows of V = 128256: 8 steps 48 us for the whole call, 16 steps
// 44 us, 32 steps 42 us).  Aim: about three workgroups per compute unit, all resident at once; and a row has kStatParts
// parts at most.
inline int parts_stat_parts(int rows, int vocab, int logits_dtype, int compute_units)
{
    const int row_steps = ceil_div(vocab / parts_chunk_elems(logits_dtype), kQT);
    int steps = kStatSteps;
    while (steps < 64 && (row_steps > kStatParts * steps ||
                          (int64_t)rows * ceil_div(row_steps, steps) > (int64_t)kStatTargetWgsPerCu * compute_units))
        steps *= 2;
    return ceil_div(row_steps, steps);
}

}  // namespace adaspec
