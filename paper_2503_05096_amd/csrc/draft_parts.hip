// Draft-side sampling with every row cut into parts: logits and probabilities of any storage types, V % 8 == 0,
// V <= 524288, 16-byte aligned rows.  What the step computes is stated in draft_sample.hip.
//
// One row of V = 128 K elements keeps a compute unit busy for about 30 us (two sweeps of exponentials and the store of the
// probability row), and a draft step has one row per request: with fewer rows than compute units the single-workgroup
// kernels leave most of the chip idle for that long.  Here small workgroups (256 threads) share a row, at the price of
// three kernels:
//   draft_stats_kernel   (row, part): maximum and normaliser of the part, streamed (row_parts.h); greedy rows: arg-max too
//   draft_probs_kernel   (row, part of 1024 chunks): the row's (m, Z) from its parts, q_v = 2^((l_v - m) c) / Z rounded once
//                        and stored, the rounded mass of each wavefront's 256 chunks
//   draft_pick_kernel    one workgroup per row: the (part, wavefront) pair that holds tau = u * sum(q), then its step, lane
//                        and element from the stored row; greedy rows: the arg-max of the parts
// The second kernel re-reads the logits (16-bit rows of a step fit the memory-side cache).  Bound: HBM for large steps, the
// three launches and their dependent accesses for small ones.  MI355X, whole call, one
// workgroup per row before: 64 rows of V = 128256 in fp32 43.6 -> 22.4 us, of V = 262144 in bf16 71 -> 25.3 us; 128 rows of
// V = 128256 in bf16 23.4-24.1 us (26.1 in four parts of 1024 threads).
#include <type_traits>

#include "adaspec_internal.h"
#include "device_utils.h"
#include "row_parts.h"

namespace adaspec {

// a float pair rounded to two values of a 16-bit type (nearest even), packed; and back
template <class PT> struct Round16;
template <> struct Round16<BF16> {
    typedef __bf16 v2 __attribute__((ext_vector_type(2)));
};
template <> struct Round16<F16> {
    typedef _Float16 v2 __attribute__((ext_vector_type(2)));
};
template <class PT>
__device__ __forceinline__ uint32_t round_pair(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 x = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, typename Round16<PT>::v2));
}

template <class LT>
__device__ __forceinline__ float draft_exponent_scale(float T)     // T == 0 stands for T = 1
{
    return T == 0.0f ? 1.4426950408889634f : exponent_scale<LT>(T);
}

// (m, Z, arg-max or -1) of a row from its parts
template <class LT>
__device__ __forceinline__ HalfStat merge_stats(const HalfStat *__restrict__ st, int n_parts, float c)
{
    HalfStat s[kStatParts], out;
    out.m = -INFINITY; out.arg = -1; out.Z = 0.0;
#pragma unroll
    for (int p = 0; p < kStatParts; ++p) {
        s[p].m = -INFINITY; s[p].arg = -1; s[p].Z = 0.0;
        if (p < n_parts) s[p] = st[p];                       // uniform: scalar loads
    }
#pragma unroll
    for (int p = 0; p < kStatParts; ++p) {
        out.m = fmaxf(out.m, s[p].m);
    }
#pragma unroll
    for (int p = 0; p < kStatParts; ++p) {
        if (s[p].m == out.m && s[p].arg >= 0 && (out.arg < 0 || s[p].arg < out.arg)) out.arg = s[p].arg;
        out.Z += s[p].m > -INFINITY ? s[p].Z * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(s[p].m, out.m, c)) : 0.0;
    }
    return out;
}

template <class LT>
__global__ __launch_bounds__(kQT, kStatWgsPerCu) void draft_stats_kernel(
    const char *__restrict__ logits, const float *__restrict__ temperature, int V, int n_parts, int64_t lstride_bytes,
    HalfStat *__restrict__ stats)
{
    __shared__ float s_m[kQW];
    __shared__ double s_z[kQW];
    __shared__ int s_i[kQW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = blockIdx.x / n_parts, h = blockIdx.x % n_parts;
    const float T = temperature[r], c = draft_exponent_scale<LT>(T);
    const int row_chunks = V / Chunk<LT>::kN;
    const __amdgpu_buffer_rsrc_t rl =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(logits) + (int64_t)r * lstride_bytes, 0, row_chunks * 16, 0x00020000);
    HalfStat out;
    if (T == 0.0f) {
        const PartStream st = stream_part<LT, true, true, kAuxDefault>(rl, row_chunks, n_parts, h, V, c, tid, [] {});
        out = reduce_norm<LT>(st, c, s_m, s_z, lane, wv);
        lds_barrier();                                       // s_m is used again
        const ArgMax b = reduce_argmax(st.best, s_m, s_i, lane, wv);
        out.arg = b.i < V ? b.i : -1;
    } else {
        const PartStream st = stream_part<LT, true, false, kAuxDefault>(rl, row_chunks, n_parts, h, V, c, tid, [] {});
        out = reduce_norm<LT>(st, c, s_m, s_z, lane, wv);
    }
    if (tid == 0) stats[(int64_t)r * kStatParts + h] = out;
}

template <class LT, class PT>
__global__ __launch_bounds__(kQT, 8) void draft_probs_kernel(
    const char *__restrict__ logits, const float *__restrict__ temperature, const int32_t *__restrict__ out_rows,
    char *__restrict__ probs, int V, int n_stat_parts, int n_parts, int64_t lstride_bytes, int64_t pstride_bytes,
    const HalfStat *__restrict__ stats, double *__restrict__ mass)
{
    constexpr int kN = Chunk<LT>::kN, kBytes = ProbChunk<kN, PT>::kBytes;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = blockIdx.x / n_parts, h = blockIdx.x % n_parts;
    const int row_chunks = V / kN, chunk0 = h * kSumChunks, nchunks = min(row_chunks - chunk0, kSumChunks);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(logits) + (int64_t)r * lstride_bytes + (int64_t)chunk0 * 16, 0, nchunks * 16, 0x00020000);
    // wavefront w owns the part's chunks 256 w .. 256 w + 255, lane l of its step it the chunk 64 it + l of those
    const int my_chunk = wv * (kSumSteps * kWave) + lane;
    uint4 lg[kSumSteps];
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) lg[it] = part_load16<kAuxDefault>(rl, (uint32_t)my_chunk * 16u, it * (kWave * 16));
    const float T = temperature[r], c = draft_exponent_scale<LT>(T);
    const HalfStat row = merge_stats<LT>(stats + (int64_t)r * kStatParts, n_stat_parts, c);
    const float mc = scaled_ref(row.m, c), invZ = (float)(1.0 / row.Z);   // (a row without any finite logit: q = NaN, as in the other kernels)
    char *prow = probs + (int64_t)(out_rows ? out_rows[r] : r) * pstride_bytes + (int64_t)chunk0 * kBytes;
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(prow, 0, nchunks * kBytes, 0x00020000);
    double total = 0.0;
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) {
        keep_packed(lg[it]);
        Chunk<LT>::blank(lg[it], my_chunk + it * kWave >= nchunks);
        float q[kN];
        Chunk<LT>::unpack(lg[it], q);
#pragma unroll
        for (int e = 0; e < kN; ++e) q[e] = exp_weight<LT>(q[e], row.m, c, mc) * invZ;
        // (the step's offset in the lane offset, scalar offset 0: see the store in draft_fast.hip)
        const int at = (my_chunk + it * kWave) * kBytes;
        if constexpr (std::is_same<PT, F32>::value) {
#pragma unroll
            for (int k = 0; k < kN / 4; ++k)
                __builtin_amdgcn_raw_buffer_store_b128(
                    u32x4{__float_as_uint(q[4 * k]), __float_as_uint(q[4 * k + 1]), __float_as_uint(q[4 * k + 2]), __float_as_uint(q[4 * k + 3])},
                    rp, at + 16 * k, 0, 0);
        } else {
            uint32_t w[kN / 2];
#pragma unroll
            for (int e = 0; e < kN / 2; ++e) {
                w[e] = round_pair<PT>(q[2 * e], q[2 * e + 1]);
                q[2 * e] = Pair16<PT>::lo(w[e]);
                q[2 * e + 1] = Pair16<PT>::hi(w[e]);
            }
            if constexpr (kN == 8) {
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[0], w[1], w[2], w[3]}, rp, at, 0, 0);
            } else {
                typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, rp, at, 0, 0);
            }
        }
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < kN; ++e) acc += q[e];
        total += (double)acc;
    }
    total = wave_sum(total);
    if (lane == 0) mass[((int64_t)r * n_parts + h) * kQW + wv] = total;
}

template <class PT>
__global__ __launch_bounds__(kQT) void draft_pick_kernel(
    const char *__restrict__ probs, const float *__restrict__ temperature, const float *__restrict__ uniforms,
    const int32_t *__restrict__ out_rows, int32_t *__restrict__ tokens, float *__restrict__ confidence, int V, int chunk_elems,
    int n_stat_parts, int n_parts, int64_t pstride_bytes, const HalfStat *__restrict__ stats, const double *__restrict__ mass)
{
    __shared__ PairScratch s_pair;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = blockIdx.x;
    const float T = temperature[r], u = uniforms[r];
    const char *prow = probs + (int64_t)(out_rows ? out_rows[r] : r) * pstride_bytes;
    const int n_pairs = n_parts * kQW;
    double w0 = 0.0, w1 = 0.0;
    if (T != 0.0f && 2 * tid < n_pairs) {
        const double2 w = *reinterpret_cast<const double2 *>(mass + (int64_t)r * n_pairs + 2 * tid);
        w0 = w.x; w1 = w.y;
    }
    if (T == 0.0f) {
        if (tid == 0) {
            const int arg = merge_stats<PT>(stats + (int64_t)r * kStatParts, n_stat_parts, 1.4426950408889634f).arg;
            tokens[r] = arg >= 0 ? arg : 0;
            confidence[r] = arg >= 0 ? load_as_float<PT>(prow, arg) : 0.f;
        }
        return;
    }
    double Q;
    const double at1 = pair_totals(s_pair, w0 + w1, tid, lane, wv, Q);
    const double tau = (double)u * Q;
    const int pair = pick_pair(s_pair, w0, w1, at1, tau, tid, lane, wv);
    if (pair < 0) {                           // no mass (non-finite input): stay defined
        if (tid == 0) { tokens[r] = 0; confidence[r] = 0.f; }
        return;
    }
    // this lane's chunk of the stored row: step wv of the pair
    const int first = (pair / kQW * kSumChunks + ((pair % kQW) * kSumSteps + wv) * kWave + lane) * chunk_elems;
    auto finish = [&](auto n_tag) {
        constexpr int N = decltype(n_tag)::value;
        ProbChunk<N, PT> qc;
        qc.zero();
        if (first < V)
            __builtin_memcpy(qc.w, __builtin_assume_aligned(prow + (int64_t)first * (int)sizeof(typename PT::storage), qc.kBytes < 16 ? 8 : 16), qc.kBytes);
        float q[N], acc = 0.f;
        qc.unpack(q);
#pragma unroll
        for (int e = 0; e < N; ++e) acc += q[e];
        double li;
        bool none;
        const bool owner = own_point(s_pair, (double)acc, tau, lane, wv, li, none);
        if (none && tid == 0) { tokens[r] = 0; confidence[r] = 0.f; }
        if (owner) {
            const int pick = pick_element<N>(q, li - (double)acc, 1.0, tau);
            tokens[r] = first + pick;
            float conf = q[0];
#pragma unroll
            for (int e = 1; e < N; ++e) conf = e == pick ? q[e] : conf;
            confidence[r] = conf;
        }
    };
    if (chunk_elems == 8) finish(std::integral_constant<int, 8>{});
    else finish(std::integral_constant<int, 4>{});
}

bool draft_parts_supported(const adaspec_draft_dims &d) { return d.vocab % 8 == 0 && d.vocab <= kPartsMaxVocab; }

// workspace: HalfStat[R][kStatParts], then double[R][parts][kQW]
static size_t stats_bytes(int rows) { return align_up((size_t)rows * kStatParts * sizeof(HalfStat), 256); }
size_t draft_parts_workspace_bytes(const adaspec_draft_dims &d)
{
    return stats_bytes(d.rows) + (size_t)d.rows * parts_sum_parts(d.vocab, d.logits_dtype) * kQW * sizeof(double);
}

hipError_t launch_draft_parts(const void *logits, const float *temperature, const float *uniforms,
                              const int32_t *out_rows, void *probs, int32_t *tokens, float *confidence,
                              const adaspec_draft_dims &d, char *ws, int compute_units, hipStream_t stream)
{
    if (d.rows == 0) return hipSuccess;
    const int64_t lstride = d.logits_row_stride * (d.logits_dtype == ADASPEC_F32 ? 4 : 2);
    const int64_t pstride = d.probs_row_stride * (d.probs_dtype == ADASPEC_F32 ? 4 : 2);
    const int n_stat_parts = parts_stat_parts(d.rows, d.vocab, d.logits_dtype, compute_units);
    const int n_parts = parts_sum_parts(d.vocab, d.logits_dtype);
    HalfStat *stats = reinterpret_cast<HalfStat *>(ws);
    double *mass = reinterpret_cast<double *>(ws + stats_bytes(d.rows));
    auto launch = [&](auto lt, auto pt) {
        using LT = decltype(lt);
        using PT = decltype(pt);
        hipLaunchKernelGGL((draft_stats_kernel<LT>), dim3(d.rows * n_stat_parts), dim3(kQT), 0, stream, (const char *)logits,
                           temperature, d.vocab, n_stat_parts, lstride, stats);
        hipLaunchKernelGGL((draft_probs_kernel<LT, PT>), dim3(d.rows * n_parts), dim3(kQT), 0, stream, (const char *)logits,
                           temperature, out_rows, (char *)probs, d.vocab, n_stat_parts, n_parts, lstride, pstride, stats, mass);
        hipLaunchKernelGGL((draft_pick_kernel<PT>), dim3(d.rows), dim3(kQT), 0, stream, (const char *)probs, temperature, uniforms,
                           out_rows, tokens, confidence, d.vocab, Chunk<LT>::kN, n_stat_parts, n_parts, pstride, stats, mass);
    };
    auto with_p = [&](auto lt) {
        if (d.probs_dtype == ADASPEC_F32) launch(lt, F32{});
        else if (d.probs_dtype == ADASPEC_F16) launch(lt, F16{});
        else launch(lt, BF16{});
    };
    if (d.logits_dtype == ADASPEC_F32) with_p(F32{});
    else if (d.logits_dtype == ADASPEC_F16) with_p(F16{});
    else with_p(BF16{});
    return hipGetLastError();
}

}  // namespace adaspec
