// Pieces shared by the matrix-core attention kernels (attn_mfma.hip, attn_ring.hip, attn_rows.hip, attn_d64.hip, attn_f32.hip): MFMA
// wrappers, loads into LDS, the V^T tile layout, the work-unit record.
#pragma once
#include "adaspec_internal.h"
#include "device_utils.h"

namespace adaspec {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;                 // head_dim
constexpr int kBlk = 32;                // tokens per block (two pages)
constexpr int kWaves = 4;
constexpr int kORowStride = 132;        // floats per row of the merge buffer (padded: conflict-free b128)
constexpr float kNegBig = -1.0e30f;     // "no token seen yet": finite, so differences never give NaN
constexpr float kLazyLog2 = 8.0f;       // a row's softmax reference trails its running maximum by at most this (log2 units)

// ---- scores of any size (attn_d64.hip, attn_f32.hip) ------------------------------------------------------------------
// 2^(p scale - m + shift) of N scores, in place.  One multiply-add per score as long as that is no further
// off than the difference of the rounded products; where the reference m is so large that its own rounding would be a
// visible factor (and from 2^31 on one that overflows), the products are rounded as m was and subtracted.
constexpr float kLowestRef = -3.4028235e38f;    // "no token seen yet": below every finite score, and finite itself
constexpr float kLargeRef = 1048576.f;
template <int N, class P>
__device__ __forceinline__ void softmax_weights(P &p, float scale_log2, float m, float shift)
{
    const bool large = fabsf(m) > kLargeRef && m > kLowestRef;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(large) != 0, 0)) {
#pragma clang fp contract(off)
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const float t = p[e] * scale_log2;
            p[e] = __builtin_amdgcn_exp2f((t - m) + shift);
        }
    } else {
        const float m_ref = m - shift;
#pragma unroll
        for (int e = 0; e < N; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(p[e], scale_log2, -m_ref));
    }
}

template <class T> struct Mma;
template <> struct Mma<BF16> {
    // bf16 keeps 8 significant bits: a softmax weight rounded to it is off by up to 2^-9 relative,
    // which with a handful of dominant tokens reaches the 2e-3 output tolerance.  The weights are
    // therefore fed to the matrix core as hi + lo (two bf16 values, 16 significant bits).
    static constexpr bool kSplitP = true;
    static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t pack2(float lo, float hi)
    {
        f32x2 x = {lo, hi};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));   // v_cvt_pk_bf16_f32, RNE
    }
};
template <> struct Mma<F16> {
    static constexpr bool kSplitP = false;       // fp16 keeps 11 bits: 2^-12 relative is enough
    static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t pack2(float lo, float hi)
    {
        f32x2 x = {lo, hi};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, f16x2));    // v_cvt_pk_f16_f32, RNE
    }
};

__device__ __forceinline__ uint4 ld16(const char *p) { return *reinterpret_cast<const uint4 *>(p); }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// K and V are read exactly once per work unit: stream them past the caches.
__device__ __forceinline__ uint4 ld16_stream(const char *p)
{
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

// ---- memory straight into LDS ------------------------------------------------------------------------------------------
// Buffer loads with an LDS destination: lane i lands at lds + 16 i (M0 carries the LDS address; the data never passes through
// registers).  Written in assembly on purpose: the compiler, not knowing which LDS bytes such a load will write, would make
// every later LDS read wait until ALL loads in flight have landed.  The kernels wait for the one they need themselves
// (wait_loads with the number of younger loads): the vector-memory counter retires in order, and whatever the compiler
// puts in front or between only makes such a wait longer.
typedef int v4i32 __attribute__((ext_vector_type(4)));

// raw buffer: offsets in bytes, reads past the end give 0
__device__ __forceinline__ v4i32 buffer_rsrc(const char *p, uint32_t bytes)
{
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    v4i32 r;
    r.x = (int)(uint32_t)a;
    r.y = (int)(uint32_t)(a >> 32);
    r.z = (int)bytes;
    r.w = 0x00020000;
    return r;
}
// one (page, kv head) block of 4 KB
__device__ __forceinline__ v4i32 page_rsrc(const char *p) { return buffer_rsrc(p, 16 * kD * 2); }

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
}
// a page: instruction j moves 1024 bytes; the offset field moves the memory AND the LDS address by 1024 j
__device__ __forceinline__ void load_page_to_lds(const v4i32 &rsrc, uint32_t off0, uint32_t off1, uint32_t off2, uint32_t off3, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %5, 0 offen nt lds\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 nt lds\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 nt lds\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 nt lds"
                 :: "s"(lds), "v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ void load16_to_lds(const v4i32 &rsrc, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds), "v"(off), "s"(rsrc) : "memory", "m0");
}
// 4 bytes per lane, lane i at lds + 4 i
__device__ __forceinline__ void load4_to_lds(const v4i32 &rsrc, uint32_t off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds), "v"(off), "s"(rsrc) : "memory", "m0");
}
// until at most N of this wavefront's vector-memory operations are outstanding / until its LDS reads have returned
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// 16 bytes of a split's state, written through to the level that all compute units share
__device__ __forceinline__ void store_state(float *p, f32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}

// 64-bit transposing LDS read: inside each group of 16 lanes, lane i gives the address of four 16-bit elements, row i / 4 and
// columns 4 (i % 4) .. + 3 of a 4 x 16 tile, and gets column i (rows 0 .. 3).
__device__ __forceinline__ uint2 read_transposed(uint32_t lds)
{
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)lds));
}

// Maximum over the four lanes n, n + 16, n + 32, n + 48 (the lanes that hold the same query row in the
// accumulator layout), left in all four.  gfx950's row-swap instructions do it in the vector ALU: swapping
// a value with itself puts row pairs (then wavefront halves) side by side in the two results, and their
// maximum is the exchange-and-reduce step; a shuffle through LDS costs a round trip of ~100 cycles each.
typedef unsigned int u32x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float max_over_row_groups(float v)
{
    u32x2v r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}

// V^T tile in LDS, in units of 16 bytes (= the 8 k-slots of one channel for one lane group):
//   unit(d = 8c + dd, grp) = 66 dd + 16 grp + c
// The writer lane (grp = tq, c) stores channel 8c + dd at its base + 66*16*dd bytes; the reader
// lane (grp, m = 8h + dd') loads channel 16 dt + m = 8 (2dt + h) + dd' from its base + 32 dt bytes.
// Within a 16-lane group both patterns hit 16 distinct 16-byte bank groups: conflict free.
constexpr int kVtUnits = 66 * 7 + 64;
constexpr int kVtBytes = ((kVtUnits * 16 + 255) / 256) * 256;

// Everything a workgroup needs to know about one work unit; all wave-uniform.
struct Unit {
    int item, gkv, i, ns, L, n, rows, r0, t0, t1, nblk;
    int64_t qrow0, bt_off;      // first query row; offset of the request's row in block_table
};

// ---- direct calls ---------------------------------------------------------------------------------------------------
// The metadata kernel and the schedule table balance a large ragged batch; a small one only waits for them (4.7 us, and
// two more dependent loads at the head of every workgroup). A direct call launches one workgroup per (request, possible
// split, kv head, row group): the numbering follows from the host-side bounds, and the workgroup reads its request's
// lengths (and adds up the rows before them) itself.  The splits are the ones the metadata kernel would have cut.
// false: the request is shorter than this split, or has fewer rows than this group.
// About where the wavefront's first page ids stand follows from the numbering alone: that place is looked at together with
// the lengths, so that the loads which need them mostly find them in the scalar cache instead of one more memory round
// trip away.
__device__ __forceinline__ bool direct_unit(Unit &u, const DirectArgs &a, const int32_t *__restrict__ block_table, int G, int Hkv,
                                            int n_row_groups, int rows_per_group, int block_tokens, int max_pages_per_req, int wv,
                                            int lane)
{
    const int idx = blockIdx.x;
    const int rg = idx % n_row_groups;
    u.gkv = (idx / n_row_groups) % Hkv;
    u.item = idx / (n_row_groups * Hkv);
    u.i = u.item / a.per_req;
    const int s = u.item - u.i * a.per_req;
    u.bt_off = (int64_t)u.i * max_pages_per_req;
    const int first_page = (s * a.split_tokens + wv * block_tokens) >> 4;
    const int warm = block_table[u.bt_off + min(first_page, max_pages_per_req - 1)];
    int part = 0;
    for (int j = lane; j < u.i; j += kWave) part += min(max(a.spec_lens[j], 0), a.max_spec_len) + 1;
    u.L = max(a.ctx_lens[u.i], 1);
    u.n = min(max(a.spec_lens[u.i], 0), a.max_spec_len) + 1;
    u.qrow0 = __builtin_amdgcn_readlane(wave_scan_incl_dpp(part), 63);
    u.ns = min((u.L + a.split_tokens - 1) / a.split_tokens, a.per_req);
    u.rows = u.n * G;
    u.r0 = rg * rows_per_group;
    const int slen = split_len_of(u.L, u.ns, block_tokens);
    u.t0 = s * slen;
    u.t1 = min(u.L, u.t0 + slen);
    u.nblk = (u.t1 - u.t0 + block_tokens - 1) / block_tokens;
    asm volatile("" :: "s"(warm), "s"(u.L));
    return s < u.ns && u.r0 < u.rows && u.qrow0 + u.n <= a.total_q;
}

// ---- direct calls: the splits of a request merged by whoever finishes last --------------------------------------------------
// A combine kernel behind a small call costs a launch on both sides and a kernel boundary, more than its work.  Instead every
// split leaves its states at the level all compute units share (store_state, store_ml), waits until they are there, puts the
// launch's mark into its flag, waits again, and looks at the flags of the request's other splits (for its kv head).  Nobody waits for anybody: of the splits that set their flags, the last one to have done so sees all marks, unless
// one that saw them before has begun to take them back, so at least one merges (two may, with the same result).  A merge
// leaves zeros, so that a captured launch, whose mark is frozen, can be replayed; marks of other launches and whatever else
// stood there are not equal to it.  Flags and decisions are per wavefront: the rows whose states wavefront w of a split has
// stored are the ones that wavefront w of another merges.
__device__ __forceinline__ void store_ml(float *p, float m, float l)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p),
                       (unsigned long long)__float_as_uint(m) | ((unsigned long long)__float_as_uint(l) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
template <class T, int D, int kRows>
__device__ __forceinline__ void merge_splits(const DirectArgs &a, const Unit &u, const float *part_ml, const float *part_o, void *out,
                                             int out_dtype, int Hq, int Hkv, int G, int max_rows, int tid)
{
    // A thread's share: one or two pieces of four channels, of rows 256 / kCols apart, in the one row group there is.  What can be
    // computed ahead is, before the waits: at one wavefront per SIMD every instruction behind them counts.
    constexpr int kCols = D / 4, kPieces = kRows * kCols / 256;
    static_assert(kPieces == 1 || kPieces == 2, "a thread has all its states in registers");
    const int lane = tid & 63, wv = tid >> 6;
    const int64_t first = ((int64_t)u.i * a.per_req * Hkv + u.gkv) * max_rows;             // row 0 in split 0
    const int rows = u.rows, next = Hkv * max_rows;                                        // from one split's row to the next's
    const int states = (u.ns - 1) * next + rows;                                           // up to the last row of the last split
    const auto rs_ml = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(part_ml + first * 2), 0, states * 8, 0x00020000);
    const auto rs_o = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(part_o + first * D), 0, states * D * 4, 0x00020000);
    constexpr int kAgent = 16;                                      // sc1: from the level all compute units share
    const int rl0 = tid / kCols, c = 4 * (tid % kCols);
    int to[kPieces];                                                // output row
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int row = rl0 + k * (256 / kCols);
        to[k] = (row / G) * Hq + u.gkv * G + row % G;
        asm volatile("" : "+v"(to[k]));
    }
    const int split = u.item - u.i * a.per_req;
    unsigned long long *flags = a.flags + ((int64_t)blockIdx.x - (int64_t)split * Hkv) * kWaves + wv;      // of split 0
    const int64_t step = (int64_t)Hkv * kWaves;

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // this wavefront's states are in place
    // (no wavefront needs the others here, but the four together are faster: without the barrier captured calls take 1.5 % longer
    // in the mean of 189 shapes)
    lds_barrier();
    if (lane == 0) __hip_atomic_store(flags + split * step, a.mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned long long seen = a.mark;
    if (lane < u.ns) seen = __hip_atomic_load(flags + lane * step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__ballot(seen != a.mark) != 0) return;
    // (the flags have arrived, or the branch could not have been decided; no load of a state may be moved up across it)
    asm volatile("" ::: "memory");

    // All states are requested before any is looked at.  Splits the request does not have lie past the buffers' ends (zeros, no
    // traffic) and get a maximum of -inf: selects instead of branches.  (At most 512 units come here, of 32
    // rows: the buffers end long before kPast.)
    constexpr uint32_t kPast = 0x40000000u;
    u32x2v ml[kPieces][kMergeMaxSplits];
    u32x4 o[kPieces][kMergeMaxSplits];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int rl = k * (256 / kCols);
        if (rl >= rows) break;
#pragma unroll
        for (int s = 0; s < kMergeMaxSplits; ++s) {
            const uint32_t at = (uint32_t)(rl0 + rl + s * next);    // (behind row rows - 1: not stored)
            ml[k][s] = __builtin_amdgcn_raw_buffer_load_b64(rs_ml, s < u.ns ? at * 8 : kPast, 0, kAgent);
            o[k][s] = __builtin_amdgcn_raw_buffer_load_b128(rs_o, s < u.ns ? at * (D * 4) + c * 4 : kPast, 0, kAgent);
        }
    }
    if (lane < u.ns) __hip_atomic_store(flags + lane * step, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const int rl = k * (256 / kCols);
        if (rl >= rows) break;
        float ms[kMergeMaxSplits], m = -INFINITY, den = 0.f;
#pragma unroll
        for (int s = 0; s < kMergeMaxSplits; ++s) {
            ms[s] = s < u.ns ? __uint_as_float(ml[k][s].x) : -INFINITY;
            m = fmaxf(m, ms[s]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kMergeMaxSplits; ++s) {
            const float w = __builtin_amdgcn_exp2f(ms[s] - m);
            den += w * __uint_as_float(ml[k][s].y);
            acc += w * __builtin_bit_cast(f32x4, o[k][s]);
        }
        if (rl0 + rl >= rows) continue;
        const f32x4 val = acc * (1.0f / den);
        const int64_t obase = (u.qrow0 * Hq + to[k]) * (int64_t)D + c;
        if (sizeof(typename T::storage) == 4 || out_dtype == ADASPEC_F32) {
            *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(out) + obase) = val;
        } else if constexpr (sizeof(typename T::storage) == 2) {
            *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + obase) =
                make_uint2(Mma<T>::pack2(val[0], val[1]), Mma<T>::pack2(val[2], val[3]));
        }
    }
}

}  // namespace adaspec
