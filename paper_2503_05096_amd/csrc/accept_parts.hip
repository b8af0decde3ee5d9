// Two-pass acceptance in row PARTS for gfx950: logits and draft probabilities of any storage types, V % 8 == 0,
// V <= 524288, 16-byte aligned rows, up to 1024 requests.
//
// The sequential rule (accept drafts in order, recover one token at the first rejection, else take the
// bonus token) needs two things: the accept test on draft rows, for which the row's softmax statistics
// (m, Z) suffice, and the residual distribution with a draw from it on ONE row per request.  Both are
// sweeps over vocabulary rows of 256 KB and more that a single compute unit takes 7-12 us for; handing whole rows
// to workgroups leaves the chip unevenly loaded (382 rows on 256 compute units) and every row a serial
// chain.  Here every row is cut into parts, one small workgroup (256 threads) each, a few per compute
// unit, all resident at once.
//
// A row is a sequence of CHUNKS of 16 bytes of logits (8 elements of 16 bits, 4 of fp32) with as many draft
// probabilities beside them.
//
//   accept_rowparts_kernel   workgroup = (draft row, part).  Finds the row's request from spec_lens itself
//       (block scan, up to 1024 requests), streams its part of the logits row once (part h = steps h,
//       h + n_parts, ... of 4 KB; 8 steps in flight, maximum and normaliser on line) and leaves the part's
//       (maximum, normaliser) or, for a greedy request, (maximum, arg-max); part 0 also leaves what the
//       accept test needs besides: the draft token, its logit, its draft probability and the uniform.
//       Records are stored per SLOT (request, draft position), so the second pass reads them without
//       knowing where the request's rows start.  Workgroup 0 also writes cu_q and clears the tickets of
//       the second pass; the whole grid clears the words of the other one.
//   accept_decide_kernel     (16-bit rows above V = 12288, large batches, some fp32 rows; the others: accept_shared.hip)  workgroup = (request, part of
//       <= 1024 chunks).  Merges the part
//       statistics of the request's draft rows, applies the accept test to each (one lane per draft), finds
//       the first rejection -> the deciding row; part 0 writes the accepted drafts, the padding and the
//       length.  A greedy rejection is decided by the merged arg-max.  Otherwise the workgroup loads its
//       part of the deciding row (and of its draft-probability row; each wavefront 256 contiguous chunks) and
//       publishes the residual and probability mass of each of its wavefronts; the workgroup that finishes LAST
//       for its request (an integer ticket per request, one atomic add at the exit, no waiting) puts the parts
//       on one scale, finds the (part, wavefront) that holds tau = u1 * R, recomputes that wavefront's
//       256 chunks with the same expressions and picks the element.
// Per-element arithmetic is fp32, sums across lanes and workgroups fp64, in a fixed order: outputs do
// not depend on which workgroup arrives last.
//
// What the time goes to (MI355X, 510 rows of V = 128256, time stamps): a dependent memory access costs
// 1.2-1.7 us and the chain has six of them (first pass: lengths -> row; second pass: slot records -> row,
// then stores acknowledged -> ticket -> partial sums -> the chunks of the draw), the two launches add
// 1.7 us each, and the rows themselves stream at 5.0-5.5 TB/s.  Whole calls: 510 rows of V = 128256 bf16 38.9 us, 192 rows of V = 262144 bf16 32.3 us.  Masses are published per wavefront (16 bytes per 256 chunks) and
// not per step and 16-lane row, so that a row of any length fits the final search of one workgroup with two pairs per
// thread; the four steps of the winning pair are recomputed by one wavefront each.
#include "accept_head.h"
#include "part_exchange.h"

namespace adaspec {

constexpr int kPartsMaxBatch = 1024;        // requests the in-kernel scan covers (4 per thread)
constexpr int kPartsMaxSlots = 32768;       // batch * max_spec_len slots the workspace is laid out for

// Phase time stamps for tuning builds (-DADASPEC_STAMPS): thread 0 of every workgroup leaves the 100 MHz
// wall clock at up to 8 points of each kernel; adaspec_debug_read_stamps copies them out.  Product builds
// compile none of it.
#ifdef ADASPEC_STAMPS
constexpr int kStampGroups = 8192;
static __device__ long long g_stamps[2][kStampGroups][8];
#define ADASPEC_STAMP(which, k)                                                                        \
    do {                                                                                               \
        if (threadIdx.x == 0 && blockIdx.x < kStampGroups) g_stamps[which][blockIdx.x][k] = wall_clock64(); \
    } while (0)
#else
#define ADASPEC_STAMP(which, k) do { } while (0)
#endif

// ---- memory that crosses workgroups inside one launch ---------------------------------------------
// The partial sums of the second pass are written by one workgroup and read by another one of the same
// launch, possibly on another XCD (each XCD has its own L2).  They travel as relaxed agent-scope atomic
// stores and loads (write-through / read-through to the level all XCDs share); the writer waits until its
// stores have been acknowledged before it takes its ticket, and the reader's loads depend on the ticket's
// return value.  No cache-wide write-back or invalidate is needed, and nobody waits for anybody.
__device__ __forceinline__ void publish_stat(HalfStat *p, float m, int arg, double Z)
{
    publish_u64(p, (unsigned long long)__float_as_uint(m) | ((unsigned long long)(uint32_t)arg << 32));
    publish_u64(reinterpret_cast<char *>(p) + 8, (unsigned long long)__double_as_longlong(Z));
}
__device__ __forceinline__ HalfStat fetch_stat(const HalfStat *p)
{
    const unsigned long long a = fetch_u64(p), b = fetch_u64(reinterpret_cast<const char *>(p) + 8);
    HalfStat s;
    s.m = __uint_as_float((uint32_t)a);
    s.arg = (int)(uint32_t)(a >> 32);
    s.Z = __longlong_as_double((long long)b);
    return s;
}

// mass of one wavefront's 256 chunks of a part: [B][n_parts][kQW]
struct WaveMass { double residual, prob; };

// One chunk: residual r_v = max(0, e_v / Z - q_v) and p_v = e_v / Z with e_v = 2^((l_v - m) c).
// The sums and the final search both call this, so they see the same numbers.
template <class LT, class PT>
__device__ __forceinline__ void part_chunk_masses(const uint4 &lv, const ProbChunk<Chunk<LT>::kN, PT> &qv, float m, float c,
                                                  float mc, float invZ, float (&rv)[Chunk<LT>::kN], float (&pv)[Chunk<LT>::kN])
{
    constexpr int N = Chunk<LT>::kN;
    float x[N], q[N];
    Chunk<LT>::unpack(lv, x);
    qv.unpack(q);
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float w = exp_weight<LT>(x[e], m, c, mc);
        rv[e] = fmaxf(0.f, fmaf(w, invZ, -q[e]));
        pv[e] = w * invZ;
    }
}

// (maximum, normaliser) of STEPS chunks per thread over the whole workgroup, relative to the workgroup's
// maximum: every thread sums against its own maximum (no barrier between the two sweeps), the pairs are
// merged over the wavefront and, through LDS, over the workgroup.  Returns false if no finite value exists.
template <class LT, int STEPS>
__device__ __forceinline__ bool part_max_and_norm(uint4 (&lg)[STEPS], float c, float *s_m, double *s_z,
                                                  int lane, int wv, float &m_out, double &z_out)
{
    float mt = thread_max<LT, STEPS>(lg);
    if (mt <= lowest_ref<LT>(c)) mt = -INFINITY;
    float zt = 0.f;
    if (mt > -INFINITY) {
        const float mtc = scaled_ref(mt, c);
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {
            keep_packed(lg[it]);
            float x[Chunk<LT>::kN];
            Chunk<LT>::unpack(lg[it], x);
#pragma unroll
            for (int e = 0; e < Chunk<LT>::kN; ++e) zt += exp_weight<LT>(x[e], mt, c, mtc);
        }
    }
    const float mw = wave_max(mt);
    const double zw = wave_sum(mt > -INFINITY ? (double)(zt * __builtin_amdgcn_exp2f(ref_gap<LT>(mt, mw, c))) : 0.0);
    if (lane == 0) { s_m[wv] = mw; s_z[wv] = zw; }
    lds_barrier();
    float m = s_m[0];
#pragma unroll
    for (int w = 1; w < kQW; ++w) m = fmaxf(m, s_m[w]);
    double z = 0.0;
#pragma unroll
    for (int w = 0; w < kQW; ++w)
        z += s_m[w] > -INFINITY ? s_z[w] * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(s_m[w], m, c)) : 0.0;
    m_out = m; z_out = z;
    return m > -INFINITY;
}

// arg-max (lowest index on ties) of STEPS chunks per thread over the workgroup; chunk0 = first chunk of this lane
template <class LT, int STEPS>
__device__ __forceinline__ ArgMax part_argmax(uint4 (&lg)[STEPS], int chunk0, int V, float *s_m, int *s_i,
                                              int lane, int wv)
{
    constexpr int N = Chunk<LT>::kN;
    ArgMax best{-INFINITY, V};
#pragma unroll
    for (int it = 0; it < STEPS; ++it) {
        keep_packed(lg[it]);
        float x[N];
        Chunk<LT>::unpack(lg[it], x);
        const int base = (chunk0 + it * kWave) * N;
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (x[e] > best.v) best = ArgMax{x[e], base + e};
    }
    return reduce_argmax(best, s_m, s_i, lane, wv);
}

// ---------------------------------------------------------------------------------------------------
// First pass: statistics of every draft row, in parts.
template <class LT>
__global__ __launch_bounds__(kQT, kStatWgsPerCu) void accept_rowparts_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs,
    const int32_t *__restrict__ draft_tokens, const float *__restrict__ uniforms,
    const int32_t *__restrict__ spec_lens, const float *__restrict__ temperature, int B, int V, int total_q,
    int total_draft, int max_spec_len, int n_parts, int64_t lstride, int64_t pstride, int probs_dtype,
    int32_t *__restrict__ cu_q, int32_t *__restrict__ req_ticket, unsigned long long *__restrict__ words, int n_words,
    SlotRec *__restrict__ slot_rec, HalfStat *__restrict__ part_stat)
{
    constexpr int kN = Chunk<LT>::kN, kSize = (int)sizeof(typename LT::storage);
    __shared__ int s_tot[kQW];
    __shared__ int s_row[5];                 // request, position, k, temperature bits, logits row
    __shared__ float s_m[kQW];
    __shared__ double s_z[kQW];
    __shared__ int s_i[kQW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int dr = blockIdx.x / n_parts, h = blockIdx.x % n_parts;      // draft row, part
    ADASPEC_STAMP(0, 0);
    // the words in which the shared second pass's workgroups tell each other their sums, cleared by the whole grid
    for (int w = blockIdx.x * kQT + tid; w < n_words; w += gridDim.x * kQT) words[w] = kNoWord;

    // ---- which request owns draft row dr: scan of n_i = k_i + 1, four requests per thread --------------
    int kk[4];
    float tt[4];
    int n_thread = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = tid * 4 + u;
        kk[u] = -1;
        tt[u] = 0.f;
        if (i < B) {
            kk[u] = min(max(spec_lens[i], 0), max_spec_len);
            tt[u] = temperature[i];
            n_thread += kk[u] + 1;
        }
    }
    const int inc = wave_scan_incl_dpp(n_thread);
    if (lane == 63) s_tot[wv] = inc;
    if (tid == 0) s_row[0] = -1;
    lds_barrier();
    int first = inc - n_thread;              // cu_q of this thread's first request
#pragma unroll
    for (int w = 0; w < kQW; ++w) first += w < wv ? s_tot[w] : 0;
    {
        int q0 = first;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = tid * 4 + u;
            if (kk[u] >= 0) {
                const int d0 = q0 - i;       // first draft row of request i
                if (dr >= d0 && dr < d0 + kk[u]) {
                    s_row[0] = i; s_row[1] = dr - d0; s_row[2] = kk[u];
                    s_row[3] = __float_as_int(tt[u]); s_row[4] = q0 + (dr - d0);
                }
                if (blockIdx.x == 0) {       // one workgroup leaves cu_q and clears the second pass's tickets
                    cu_q[i] = q0;
                    req_ticket[i] = 0;
                    if (i == B - 1) cu_q[B] = q0 + kk[u] + 1;
                }
                q0 += kk[u] + 1;
            }
        }
    }
    lds_barrier();
    const int ri = __builtin_amdgcn_readfirstlane(s_row[0]);
    if (ri < 0 || dr >= total_draft) return;             // no such draft row (also: inconsistent lengths)
    const int j = __builtin_amdgcn_readfirstlane(s_row[1]);
    const float T = __int_as_float(__builtin_amdgcn_readfirstlane(s_row[3]));
    const int r = __builtin_amdgcn_readfirstlane(s_row[4]);
    if (r >= total_q) return;
    ADASPEC_STAMP(0, 1);

    // ---- the part of the row, streamed once (a draft row is read only here: past the caches) -----------
    const int row_chunks = V / kN;
    const char *lrow = logits + (int64_t)r * lstride * kSize;
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(lrow), 0, row_chunks * 16, 0x00020000);
    const int64_t slot = (int64_t)ri * max_spec_len + j;
    HalfStat *my_stat = part_stat + slot * kStatParts + h;
    auto leave_slot = [&]() {
        if (h != 0 || tid != 0) return;
        // what the accept test needs besides (m, Z): these loads travel with the row
        const int x = draft_tokens[dr];
        const int xa = min(max(x, 0), V - 1);            // (address only: an out-of-range token must not fault)
        const int64_t px = (int64_t)dr * pstride + xa;
        SlotRec rec;
        rec.x = x;
        rec.lx_bits = __float_as_uint(load_as_float<LT>(lrow, xa));
        rec.qx_bits = __float_as_uint(probs_dtype == ADASPEC_F32 ? load_as_float<F32>(probs, px)
                                      : probs_dtype == ADASPEC_F16 ? load_as_float<F16>(probs, px) : load_as_float<BF16>(probs, px));
        rec.u0_bits = __float_as_uint(uniforms[2 * (int64_t)r]);
        slot_rec[slot] = rec;
    };
    ADASPEC_STAMP(0, 2);
    if (T == 0.0f) {
        const PartStream st = stream_part<LT, true, kAuxStream>(rl, row_chunks, n_parts, h, V, 0.f, tid, leave_slot);
        const ArgMax b = reduce_argmax(st.best, s_m, s_i, lane, wv);
        if (tid == 0) {
            HalfStat out; out.m = b.v; out.arg = b.i < V ? b.i : -1; out.Z = 0.0; *my_stat = out;
        }
        return;
    }
    const float c = exponent_scale<LT>(T);
    const PartStream st = stream_part<LT, false, kAuxStream>(rl, row_chunks, n_parts, h, V, c, tid, leave_slot);
    const HalfStat out = reduce_norm<LT>(st, c, s_m, s_z, lane, wv);
    if (tid == 0) *my_stat = out;
    ADASPEC_STAMP(0, 3);
}

// ---------------------------------------------------------------------------------------------------
// Second pass: the deciding row of every request, in parts, and the draw.
template <class LT, class PT>
__global__ __launch_bounds__(kQT, sizeof(typename PT::storage) > sizeof(typename LT::storage) ? 6 : 8) void accept_decide_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs,
    const int32_t *__restrict__ draft_tokens, const float *__restrict__ uniforms,
    const int32_t *__restrict__ spec_lens, const float *__restrict__ temperature, int V, int total_q,
    int total_draft, int max_spec_len, int n_stat_parts, int n_parts, int64_t lstride, int64_t pstride,
    const int32_t *__restrict__ cu_q, int32_t *__restrict__ req_ticket, const SlotRec *__restrict__ slot_rec,
    const HalfStat *__restrict__ part_stat, int out_stride, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ out_accept_len, WaveMass *__restrict__ sums, HalfStat *__restrict__ sum_stat)
{
    constexpr int kN = Chunk<LT>::kN, kLSize = (int)sizeof(typename LT::storage), kPSize = (int)sizeof(typename PT::storage);
    using Probs = ProbChunk<kN, PT>;
    __shared__ float s_m[kSumParts];
    __shared__ double s_z[kSumParts];
    __shared__ int s_i[kQW];
    __shared__ int s_last;
    __shared__ PairScratch s_pair;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = blockIdx.x / n_parts, h = blockIdx.x % n_parts;
    ADASPEC_STAMP(1, 0);

    __shared__ DecidingScratch s_dec;
    const DecidingRow d = deciding_row<LT>(s_dec, i, cu_q, spec_lens, temperature, slot_rec, part_stat, max_spec_len, n_stat_parts, lane, wv);
    const int start = d.start, k = d.k, a = d.a;
    const bool sampled = d.sampled;
    const float c = d.c;
    const RowMerge row = d.row;
    const int r = start + a;
    const bool bonus = a >= k;
    int32_t *o = out_tokens + (int64_t)i * out_stride;
    if (h == 0 && wv == 0) {                  // everything but the sampled token
        for (int jj = lane; jj < out_stride; jj += kWave)
            if (jj != a) o[jj] = (jj < a && start - i + jj < total_draft) ? draft_tokens[start - i + jj] : -1;
        if (lane == 0) out_accept_len[i] = a;
    }
    if (r >= total_q) {                       // inconsistent lengths: stay inside the tensors
        if (h == 0 && tid == 0) o[a] = 0;
        return;
    }
    if (!sampled && !bonus) {                 // greedy and rejected: the row's arg-max, already merged
        if (h == 0 && tid == 0) o[a] = row.arg;
        return;
    }

    ADASPEC_STAMP(1, 1);
    // ---- this workgroup's part of the deciding row (and of its draft probabilities) -------------------
    // wavefront w owns the part's chunks 256 w .. 256 w + 255, lane l of its step it the chunk 64 it + l of those
    const int row_chunks = V / kN;
    const int chunk0 = h * kSumChunks;
    const int nchunks = min(row_chunks - chunk0, kSumChunks);        // >= 1 by the choice of n_parts
    const char *lrow = logits + (int64_t)r * lstride * kLSize;
    const char *prow = probs + (int64_t)(r - i) * pstride * kPSize;
    const bool has_q = sampled && !bonus;
    const __amdgpu_buffer_rsrc_t rl =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(lrow) + (int64_t)chunk0 * 16, 0, nchunks * 16, 0x00020000);
    // (a bonus row has no draft probabilities: descriptor of size zero, the loads return zeros)
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(prow) + (int64_t)chunk0 * Probs::kBytes, 0, has_q ? nchunks * Probs::kBytes : 0, 0x00020000);
    const int my_chunk = wv * (kSumSteps * kWave) + lane;            // of step 0, inside the part
    uint4 lg[kSumSteps];
    Probs qg[kSumSteps];
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) lg[it] = part_load16<kAuxDefault>(rl, (uint32_t)my_chunk * 16u, it * (kWave * 16));
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) qg[it].load(rq, (uint32_t)(my_chunk * Probs::kBytes), it * (kWave * Probs::kBytes));
    const float u_draw = uniforms[2 * (int64_t)r + 1];
#pragma unroll
    for (int it = 0; it < kSumSteps; ++it) Chunk<LT>::blank(lg[it], my_chunk + it * kWave >= nchunks);
    HalfStat *my_stat = sum_stat + (int64_t)i * n_parts + h;
    WaveMass *my_sum = sums + ((int64_t)i * n_parts + h) * kQW + wv;
    ADASPEC_STAMP(1, 2);
    if (!sampled) {
        // greedy bonus row: arg-max of the part; the last workgroup merges the parts
        const ArgMax b = part_argmax<LT, kSumSteps>(lg, chunk0 + my_chunk, V, s_m, s_i, lane, wv);
        if (tid == 0) publish_stat(my_stat, b.v, b.i < V ? b.i : -1, 0.0);
    } else {
        float m = row.m;
        double Zd = row.Z;
        bool any = true;
        // a bonus row was not seen by the first pass: maximum and normaliser of this part alone (the last
        // workgroup puts the parts on one scale)
        if (bonus) any = part_max_and_norm<LT, kSumSteps>(lg, c, s_m, s_z, lane, wv, m, Zd);
        double res = 0.0, prob = 0.0;
        if (any) {
            const float mc = scaled_ref(m, c), invZ = (float)(1.0 / Zd);
#pragma unroll
            for (int it = 0; it < kSumSteps; ++it) {
                float rv[kN], pv[kN], acc_r = 0.f, acc_p = 0.f;
                keep_packed(lg[it]);
                qg[it].keep();
                part_chunk_masses<LT, PT>(lg[it], qg[it], m, c, mc, invZ, rv, pv);
#pragma unroll
                for (int e = 0; e < kN; ++e) { acc_r += rv[e]; acc_p += pv[e]; }
                res += (double)acc_r;
                prob += (double)acc_p;
            }
            res = wave_sum(res);
            prob = wave_sum(prob);
        }
        if (lane == 0) {
            publish_u64(&my_sum->residual, (unsigned long long)__double_as_longlong(res));
            publish_u64(&my_sum->prob, (unsigned long long)__double_as_longlong(prob));
        }
        if (tid == 0) publish_stat(my_stat, any ? m : -INFINITY, any ? 0 : -1, any ? Zd : 1.0);
    }

    // ---- ticket: the workgroup that finishes last for this request does the draw ----------------------
    ADASPEC_STAMP(1, 3);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wavefront's stores have been acknowledged
    __syncthreads();
    ADASPEC_STAMP(1, 4);
    if (tid == 0) s_last = __hip_atomic_fetch_add(req_ticket + i, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_parts - 1;
    __syncthreads();
    ADASPEC_STAMP(1, 5);
    if (!s_last) return;

    if (!sampled) {
        if (wv == 0) {
            ArgMax b{-INFINITY, V};
            for (int p = lane; p < n_parts; p += kWave) {
                const HalfStat st = fetch_stat(sum_stat + (int64_t)i * n_parts + p);
                if (st.arg >= 0) b = argmax_merge(b, ArgMax{st.m, st.arg});
            }
            b = wave_argmax(b);
            if (lane == 0) o[a] = b.i < V ? b.i : 0;
        }
        return;
    }
    // thread t: the (part, wavefront) pairs 2t and 2t + 1 (of one part), all parts on one scale
    const int n_pairs = n_parts * kQW;
    HalfStat st;
    st.m = -INFINITY; st.arg = -1; st.Z = 1.0;
    double res[2] = {0.0, 0.0}, pm[2] = {0.0, 0.0};
    if (2 * tid < n_pairs) {
        const WaveMass *src = sums + (int64_t)i * n_pairs + 2 * tid;
        st = fetch_stat(sum_stat + (int64_t)i * n_parts + (tid >> 1));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            res[u] = __longlong_as_double((long long)fetch_u64(&src[u].residual));
            pm[u] = __longlong_as_double((long long)fetch_u64(&src[u].prob));
        }
    }
    if ((tid & 1) == 0) { s_m[tid >> 1] = st.m; s_z[tid >> 1] = st.Z; }
    float M = wave_max(st.m);
    if (lane == 0) s_pair.wave[wv] = (double)M;
    __syncthreads();
    M = (float)s_pair.wave[0];
#pragma unroll
    for (int w = 1; w < kQW; ++w) M = fmaxf(M, (float)s_pair.wave[w]);
    // p_v of part h was computed as 2^((l_v - m_h) c) / Z_h: times Z_h 2^((m_h - M) c) it is relative to M in
    // every part (a rejected draft row has the same (m, Z) in all parts: a common factor, which tau absorbs)
    const double my_sc = st.m > -INFINITY ? st.Z * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(st.m, M, c)) : 0.0;
#pragma unroll
    for (int u = 0; u < 2; ++u) { res[u] *= my_sc; pm[u] *= my_sc; }
    bool use_p = bonus;                                       // (for a bonus row the two sums are the same numbers)
    double R, at1 = pair_totals(s_pair, use_p ? pm[0] + pm[1] : res[0] + res[1], tid, lane, wv, R);
    if (!(R > 0.0) && !use_p) {                               // p == q everywhere (R == 0): draw from p instead
        use_p = true;
        at1 = pair_totals(s_pair, pm[0] + pm[1], tid, lane, wv, R);
    }
    const double tau = (double)u_draw * R;
    const int pair = pick_pair(s_pair, use_p ? pm[0] : res[0], use_p ? pm[1] : res[1], at1, tau, tid, lane, wv);
    ADASPEC_STAMP(1, 6);

    // ---- inside the pair: the step (one wavefront each), then the lane, then the element ------------------
    if (pair < 0 || pair >= n_pairs) {        // no mass anywhere (non-finite input): stay defined
        if (tid == 0) o[a] = 0;
        return;
    }
    const int hh = pair / kQW;
    HalfStat sth;
    sth.m = s_m[hh]; sth.Z = s_z[hh];
    const double sch = sth.m > -INFINITY ? sth.Z * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(sth.m, M, c)) : 0.0;
    const int chunk = hh * kSumChunks + ((pair % kQW) * kSumSteps + wv) * kWave + lane;   // this lane's chunk of the row
    const bool with_q = has_q && !use_p;
    uint4 lv = make_uint4(0, 0, 0, 0);
    Probs qv;
    qv.zero();
    if (chunk < row_chunks) {
        lv = *reinterpret_cast<const uint4 *>(lrow + (int64_t)chunk * 16);
        if (with_q) __builtin_memcpy(qv.w, __builtin_assume_aligned(prow + (int64_t)chunk * Probs::kBytes, Probs::kBytes < 16 ? 8 : 16), Probs::kBytes);
    }
    Chunk<LT>::blank(lv, chunk >= row_chunks);
    float rv[kN], pv[kN], mine32 = 0.f;
    part_chunk_masses<LT, PT>(lv, qv, sth.m, c, scaled_ref(sth.m, c), (float)(1.0 / sth.Z), rv, pv);   // same expressions as the sums
#pragma unroll
    for (int e = 0; e < kN; ++e) {
        if (use_p) rv[e] = pv[e];
        mine32 += rv[e];
    }
    const double mine = (double)mine32 * sch;
    double li;
    bool none;
    const bool owner = own_point(s_pair, mine, tau, lane, wv, li, none);
    if (none && tid == 0) o[a] = 0;           // the sums said there was mass here, the recomputation finds none
    if (owner) o[a] = chunk * kN + pick_element<kN>(rv, li - mine, sch, tau);
    ADASPEC_STAMP(1, 7);
}

static int sum_parts(const adaspec_accept_dims &d) { return parts_sum_parts(d.vocab, d.logits_dtype); }

bool accept_parts_dims_fit(const adaspec_accept_dims &d)
{
    return d.batch <= kPartsMaxBatch && (int64_t)d.batch * d.max_spec_len <= kPartsMaxSlots && d.vocab <= kPartsMaxVocab &&
           d.vocab % 8 == 0 && d.logits_row_stride % 8 == 0 && d.probs_row_stride % 8 == 0;
}

size_t accept_parts_slot_bytes(const adaspec_accept_dims &d)
{
    return (size_t)d.batch * (d.max_spec_len > 0 ? d.max_spec_len : 1) * sizeof(SlotRec);
}
size_t accept_parts_stat_bytes(const adaspec_accept_dims &d)
{
    return (size_t)d.batch * (d.max_spec_len > 0 ? d.max_spec_len : 1) * kStatParts * sizeof(HalfStat);
}
size_t accept_parts_sum_bytes(const adaspec_accept_dims &d)
{
    return (size_t)(d.batch > 0 ? d.batch : 1) * sum_parts(d) * kQW * sizeof(WaveMass);
}
size_t accept_parts_sum_stat_bytes(const adaspec_accept_dims &d)
{
    return (size_t)(d.batch > 0 ? d.batch : 1) * sum_parts(d) * sizeof(HalfStat);
}

hipError_t launch_accept_parts(const AcceptArgs &a, int compute_units)
{
    const adaspec_accept_dims &d = a.dims;
    if (d.batch == 0) return hipSuccess;
    const int n_stat_parts = parts_stat_parts(d.total_draft, d.vocab, d.logits_dtype, compute_units);
    const int n_sum_parts = sum_parts(d);
    int32_t *cu_q = (int32_t *)(a.ws + a.plan.off_cu_q);
    int32_t *ticket = (int32_t *)(a.ws + a.plan.off_req_ticket);
    const SharedParts shared = accept_shared_parts(d, compute_units);
    SlotRec *slot_rec = (SlotRec *)(a.ws + a.plan.off_slot_rec);
    HalfStat *part_stat = (HalfStat *)(a.ws + a.plan.off_part_stat);
    auto first = [&](auto lt) {
        // (the first pass always runs, at least with one workgroup: it also clears the tickets and words)
        const int grid = d.total_draft > 0 ? d.total_draft * n_stat_parts : 1;
        hipLaunchKernelGGL((accept_rowparts_kernel<decltype(lt)>), dim3(grid), dim3(kQT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.draft_tokens, a.uniforms, a.spec_lens,
                           a.temperature, d.batch, d.vocab, d.total_q, d.total_draft, d.max_spec_len, n_stat_parts,
                           d.logits_row_stride, d.probs_row_stride, d.probs_dtype, cu_q, ticket,
                           (unsigned long long *)(a.ws + a.plan.off_part), d.batch * shared.n_words, slot_rec, part_stat);
    };
    auto second = [&](auto lt, auto pt) {
        hipLaunchKernelGGL((accept_decide_kernel<decltype(lt), decltype(pt)>), dim3(d.batch * n_sum_parts), dim3(kQT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.draft_tokens, a.uniforms, a.spec_lens,
                           a.temperature, d.vocab, d.total_q, d.total_draft, d.max_spec_len, n_stat_parts, n_sum_parts,
                           d.logits_row_stride, d.probs_row_stride, cu_q, ticket, slot_rec, part_stat, d.out_stride,
                           a.out_tokens, a.out_accept_len, (WaveMass *)(a.ws + a.plan.off_part),
                           (HalfStat *)(a.ws + a.plan.off_half_stat));
    };
    auto with_logits = [&](auto lt) {
        first(lt);
        if (shared.n_parts > 0) {
            launch_accept_shared(a, shared, n_stat_parts);
            return;
        }
        if (d.probs_dtype == ADASPEC_F32) second(lt, F32{});
        else if (d.probs_dtype == ADASPEC_F16) second(lt, F16{});
        else second(lt, BF16{});
    };
    if (d.logits_dtype == ADASPEC_F32) with_logits(F32{});
    else if (d.logits_dtype == ADASPEC_F16) with_logits(F16{});
    else with_logits(BF16{});
    return hipGetLastError();
}

}  // namespace adaspec

#ifdef ADASPEC_STAMPS
extern "C" int adaspec_debug_read_stamps(int which, long long *host, size_t groups)
{
    if (which < 0 || which > 1 || groups > (size_t)adaspec::kStampGroups) return -2;
    return hipMemcpyFromSymbol(host, HIP_SYMBOL(adaspec::g_stamps), groups * 8 * sizeof(long long),
                               (size_t)which * adaspec::kStampGroups * 8 * sizeof(long long), hipMemcpyDeviceToHost) == hipSuccess ? 0 : -7;
}
#endif
