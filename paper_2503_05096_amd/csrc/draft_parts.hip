// Draft-side sampling with every row cut into parts: logits and probabilities of any storage types, V % 8 == 0,
// V <= 524288, 16-byte aligned rows.  What the step computes is stated in draft_sample.hip.
//
// One row of V = 128 K elements keeps a compute unit busy for about 30 us, and a draft step has one row per request, fewer
// than compute units: rows are shared.  The step is three dependent phases over a row (maximum and normaliser;
// probabilities out and their mass; the draw).  Workgroup (row, part) of 512 or 1024 threads: reads its part once, into registers, and
// never again; the parts of a row tell each other their (maximum, normaliser), then the mass of their rounded
// probabilities (part_exchange.h); the part that holds tau = u * sum(q) finds the element in its registers.  Everything in
// one launch: what a part needs from the others takes about 1 us where a kernel boundary takes 3 and the row has to be
// read again.  The probabilities are stored when the mass is out, so that the stores travel during the second exchange.
//
// Bound: HBM for large steps (33 MB in, 33 out for 128 rows of V = 128256 bf16), latency for small ones.  MI355X, whole call,
// three kernels of row parts before: 128 rows of V = 128256 bf16 24.4 -> 18.4 us (3.6 TB/s), in fp32 37.3 -> 24.0, 64 rows in fp32 22.5 -> 17.1,
// of V = 262144 bf16 24.9 -> 18.7, 300 of V = 128256 47.8 -> 38.5, 8 of V = 524288 17.7 -> 11.0; one row of V = 128256, captured, 9.9 -> 8.8.
#include <type_traits>

#include "adaspec_internal.h"
#include "device_utils.h"
#include "part_exchange.h"
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
    // (T = inf would make it 0: the chunks past the end of a row are -inf, and 0 times that NaN)
    return T == 0.0f ? 1.4426950408889634f : exponent_scale<LT>(T > 1e38f ? 1e38f : T);
}

constexpr int kDraftSteps = 8;                       // chunks per thread at most
constexpr int kDraftMaxParts = 32;                   // two lanes each in the first exchange
constexpr int kDraftT = 512, kDraftWideT = 1024;     // threads, and elements per thread up to which a row stays whole: see
constexpr int kDraftWholeElems = 32;                 // launch_draft_parts
static_assert(kPartsMaxVocab <= kDraftMaxParts * kDraftSteps * kDraftT * 4, "fp32 rows fit");
// What a part tells the others: (maximum, first element with it) and normaliser, then its mass.  A launch leaves the first two taken back:
// whoever has all the masses knows that the others have read them.  The mass is taken back where the next launch starts: nobody
// looks for it before having seen that launch's maximum, which is published after the taking back is in place.
struct DraftWords { MarkedWord top, Z, mass; };

// kInPlace: rows may go where their logits are (what that takes costs the others 0.16 of 18.1 us, so it is left out where it cannot be)
template <class LT, class PT, int NT, bool kInPlace>
__global__ __launch_bounds__(NT, 4) void draft_row_kernel(
    const char *__restrict__ logits, const float *__restrict__ temperature, const float *__restrict__ uniforms,
    const int32_t *__restrict__ out_rows, char *__restrict__ probs, int32_t *__restrict__ tokens, float *__restrict__ confidence,
    int V, int n_parts, int part_steps, int64_t lstride_bytes, int64_t pstride_bytes, DraftWords *__restrict__ all_words,
    unsigned long long mark)
{
    // (a part gives the same bits whether its own workgroup computes it or another one: no product is fused into a sum in one
    // place and not in the other)
#pragma clang fp contract(off)
    constexpr int kN = Chunk<LT>::kN, NW = NT / kWave;
    constexpr bool kKeepsWeights = kN == 8;              // 16-bit logits: the weights; fp32: the logits themselves
    constexpr int kBytes = ProbChunk<kN, PT>::kBytes;    // probabilities of a chunk
    __shared__ float s_m[NW];
    __shared__ double s_z[NW];
    __shared__ int s_i[NW];
    __shared__ float s_part_m[kDraftMaxParts];
    __shared__ int s_part_i[kDraftMaxParts];
    __shared__ double s_part_z[kDraftMaxParts];          // normalisers, then masses
    __shared__ float s_row_m, s_row_inv;
    __shared__ int s_row_arg, s_star, s_wave;            // (s_row_arg: first element with the maximum, or -1)
    __shared__ double s_tau, s_before;
    __shared__ double s_mass[NW];                   // of the own part's wavefronts
    __shared__ unsigned int s_missing;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = blockIdx.x / n_parts, h = blockIdx.x % n_parts;
    DraftWords *words = all_words + (int64_t)r * n_parts;
    if (n_parts > 1 && tid == 0) take_back(&words[h].mass);

    // wavefront w holds 64 * part_steps chunks of a part in a row, lane l of its step it the chunk 64 it + l of those
    const int row_chunks = V / kN, part_chunks = part_steps * NT;
    const int my_chunk = wv * (part_steps * kWave) + lane;
    const float T = temperature[r], u = uniforms[r], c = draft_exponent_scale<LT>(T);
    const bool sampled = T != 0.0f;
    const char *lrow = logits + (int64_t)r * lstride_bytes;
    char *prow = probs + (int64_t)(out_rows ? out_rows[r] : r) * pstride_bytes;
    auto part_size = [&](int part) -> int { return max(0, min(row_chunks - part * part_chunks, part_chunks)); };
    auto part_row = [&](int part) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(lrow) + (int64_t)part * part_chunks * 16, 0, part_size(part) * 16, 0x00020000);
    };
    auto part_probs = [&](int part) {
        return __builtin_amdgcn_make_buffer_rsrc(prow + (int64_t)part * part_chunks * kBytes, 0, part_size(part) * kBytes, 0x00020000);
    };
    auto chunk_index = [&](int part, int it) -> int { return part * part_chunks + my_chunk + it * kWave; };     // in the row

    // What is done with a part is written twice below: for the own one, in registers, and chunk by chunk for parts whose
    // words do not come (and for all parts of a row that goes where its logits are).
    // A thread's weights are relative to its own maximum (0 if it has nothing finite): exponents of the largest are then next to
    // 0, where they are rounded least.  (References known earlier, those of first chunks, were no faster, 19.2 against 19.3 us, and
    // the largest probabilities off by 2e-7 instead of 5e-8.)
    // A NaN makes its whole row NaN: sums are taken over everybody, also over threads, wavefronts and parts without a finite
    // logit (theirs are 0 unless they hold one).
    struct Ref { float m, at; };
    const float lowest = lowest_ref<LT>(c);
    auto ref_of = [&](float m) -> Ref { return Ref{m, m > lowest ? scaled_ref(m, c) : 0.f}; };
    // exponent that moves a thread's weights to the reference of the maximum m
    auto thread_gap = [&](Ref t, float m) -> float { return kKeepsWeights ? t.at - scaled_ref(m, c) : (t.m - m) * c; };
    // a chunk's weights, added up behind z
    auto add_weights = [&](const uint4 &lv, Ref t, float z, float (&w)[kN]) -> float {
        float x[kN];
        Chunk<LT>::unpack(lv, x);
#pragma unroll
        for (int e = 0; e < kN; ++e) {
            const float v = exp_weight<LT>(x[e], t.m > lowest ? t.m : 0.f, c, t.at);
            z += v;
            w[e] = kKeepsWeights ? v : x[e];
        }
        return z;
    };
    // lowest element of a chunk that is its maximum
    auto first_with = [&](const uint4 &lv, float m, int chunk) -> int {
        float x[kN];
        Chunk<LT>::unpack(lv, x);
        int at = 0;
#pragma unroll
        for (int e = kN - 1; e >= 0; --e) at = x[e] == m ? e : at;
        return chunk * kN + at;
    };
    // a chunk's probabilities, rounded, in place; returns their sum.  f moves weights from the thread's reference to the row's
    // and divides by the normaliser.
    auto round_probs = [&](float (&w)[kN], float f, float m, float mc, float inv) -> float {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < kN; e += 2) {
            float q[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) q[k] = kKeepsWeights ? w[e + k] * f : exp_weight<LT>(w[e + k], m, c, mc) * inv;
            if constexpr (!std::is_same<PT, F32>::value) {
                const uint32_t pair = round_pair<PT>(q[0], q[1]);
                q[0] = Pair16<PT>::lo(pair); q[1] = Pair16<PT>::hi(pair);
            }
            w[e] = q[0]; w[e + 1] = q[1];
            acc += q[0];
            acc += q[1];
        }
        return acc;
    };
    // over the workgroup: a part's statistics from its threads' (first half of the way: to LDS)
    auto leave_stats = [&](Ref t, float z_t, int top) {
        const float mw = wave_max(t.m);
        const double zw = wave_sum((double)(z_t * __builtin_amdgcn_exp2f(t.m > lowest ? thread_gap(t, mw) : 0.f)));
        if (lane == 0) { s_m[wv] = mw; s_z[wv] = zw; }
        if (!sampled) {
            const ArgMax b = wave_argmax(ArgMax{t.m, top});
            if (lane == 0) s_i[wv] = b.i;
        }
    };
    auto take_stats = [&](int part, float &m, double &Z, int &arg) {     // (wavefront 0)
        const float mw = lane < NW ? s_m[lane] : -INFINITY;
        m = wave_max(mw);
        Z = wave_sum(lane < NW ? s_z[lane & (NW - 1)] * (double)__builtin_amdgcn_exp2f(mw > lowest ? ref_gap<LT>(mw, m, c) : 0.f) : 0.0);
        arg = sampled ? V : wave_argmax(ArgMax{mw, lane < NW ? s_i[lane] : V}).i;
        if (lane == 0) { s_part_m[part] = m; s_part_i[part] = arg; s_part_z[part] = Z; }
    };
    auto row_stats = [&]() {                                             // (wavefront 0, all parts known)
        const float mp = lane < n_parts ? s_part_m[lane] : -INFINITY, M = wave_max(mp);
        const double sum = wave_sum(lane < n_parts ? s_part_z[lane & 31] * (double)__builtin_amdgcn_exp2f(mp > lowest ? ref_gap<LT>(mp, M, c) : 0.f) : 0.0);
        const int at = s_part_i[lane & 31];
        const ArgMax b = wave_argmax(lane < n_parts && at < V ? ArgMax{mp, at} : ArgMax{-INFINITY, 0x7fffffff});
        // (a row without any finite logit: q = NaN, as in the other kernels)
        if (lane == 0) { s_row_m = M; s_row_inv = (float)(1.0 / sum); s_row_arg = b.i == 0x7fffffff ? -1 : b.i; }
    };
    auto thread_factor = [&](Ref t) -> float {
        return __builtin_amdgcn_exp2f(t.m > lowest ? thread_gap(t, s_row_m) : 0.f) * s_row_inv;
    };

    // a chunk's (rounded) probabilities to memory
    auto store_chunk = [&](__amdgpu_buffer_rsrc_t rp, int it, const float (&q)[kN]) {
        // (the step's offset in the lane offset, scalar offset 0: see the store in draft_fast.hip)
        const int at = (my_chunk + it * kWave) * kBytes;
        uint32_t d[kBytes / 4];
        if constexpr (std::is_same<PT, F32>::value) {
#pragma unroll
            for (int e = 0; e < kN; ++e) d[e] = __float_as_uint(q[e]);
        } else {
#pragma unroll
            for (int e = 0; e < kN / 2; ++e) d[e] = round_pair<PT>(q[2 * e], q[2 * e + 1]);     // (exact)
        }
        if constexpr (kBytes == 8) {
            typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{d[0], d[1]}, rp, at, 0, 0);
        } else {
#pragma unroll
            for (int k = 0; k < kBytes / 16; ++k)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{d[4 * k], d[4 * k + 1], d[4 * k + 2], d[4 * k + 3]}, rp, at + 16 * k, 0, 0);
        }
    };

    // ---- a part chunk by chunk, by the whole workgroup: what its own workgroup's words would have said, left in LDS ------
    auto chunk_at = [&](int part, int it) -> uint4 {
        uint4 v = part_load16<kAuxDefault>(part_row(part), (uint32_t)my_chunk * 16u, it * (kWave * 16));
        Chunk<LT>::blank(v, my_chunk + it * kWave >= part_size(part));
        return v;
    };
    auto compute_stats = [&](int part) {
        float m = -INFINITY, z = 0.f;
        int first = V;
        for (int it = 0; it < part_steps; ++it) {
            const uint4 v = chunk_at(part, it);
            const float mn = chunk_max<LT>(v, m);
            if (mn > m) first = first_with(v, mn, chunk_index(part, it));
            m = mn;
        }
        const Ref t = ref_of(m);
        for (int it = 0; it < part_steps; ++it) {
            float x[kN];
            z = add_weights(chunk_at(part, it), t, z, x);
        }
        lds_barrier();
        leave_stats(t, z, first);
        lds_barrier();
        if (wv == 0) {
            double Z;
            int arg;
            take_stats(part, m, Z, arg);
        }
    };
    auto compute_mass = [&](int part, bool store) {                      // (the row's statistics known)
        const float row_m = s_row_m, row_inv = s_row_inv, mc = scaled_ref(row_m, c);
        const __amdgpu_buffer_rsrc_t rp = part_probs(part);
        float m = -INFINITY;
        for (int it = 0; it < part_steps; ++it) m = chunk_max<LT>(chunk_at(part, it), m);
        const Ref t = ref_of(m);
        const float f = thread_factor(t);
        double total = 0.0;
        for (int it = 0; it < part_steps; ++it) {
            float x[kN];
            add_weights(chunk_at(part, it), t, 0.f, x);
            total += (double)round_probs(x, f, row_m, mc, row_inv);
            if (store) store_chunk(rp, it, x);
        }
        total = wave_sum(total);
        lds_barrier();
        if (lane == 0) s_z[wv] = total;
        lds_barrier();
        if (wv == 0) {
            const double mass = wave_sum(lane < NW ? s_z[lane] : 0.0);
            if (lane == 0) s_part_z[part] = mass;
        }
    };

    // ---- probabilities that go where the logits are --------------------------------------------------------------------
    // What a part has overwritten nobody else could compute again if its words did not come in time: one workgroup takes such a
    // row alone, part by part (a thread stores a chunk it has just read), and draws from what it has stored.
    if constexpr (kInPlace) {
        if (n_parts > 1 && prow == lrow) {
            if (h > 0) return;
            for (int part = 0; part < n_parts; ++part) compute_stats(part);
            if (wv == 0) row_stats();
            lds_barrier();
            for (int part = 0; part < n_parts; ++part) compute_mass(part, true);
            if (wv == 0) {
                double before = 0.0, tau = 0.0;
                int star = s_row_arg < 0 ? -1 : s_row_arg / kN / part_chunks;
                if (sampled) {
                    const double at = lane < n_parts ? s_part_z[lane & 31] : 0.0;
                    tau = (double)u * wave_sum(at);
                    star = find_piece(at, 0.0, tau, lane, before);
                }
                if (lane == 0) { s_star = star; s_before = before; s_tau = tau; }
            }
            __syncthreads();                                 // (the stores are done, too)
            const int star = s_star;
            if (star < 0) {                                  // no mass (non-finite input): stay defined
                if (tid == 0) { tokens[r] = 0; confidence[r] = 0.f; }
                return;
            }
            const __amdgpu_buffer_rsrc_t rp = part_probs(star);
            auto stored = [&](int it, float (&q)[kN]) -> float {
                Chunk<PT>::unpack(part_load16<kAuxDefault>(rp, (uint32_t)my_chunk * 16u, it * (kWave * 16)), q);
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < kN; ++e) acc += q[e];
                return acc;
            };
            float q[kN];
            if (!sampled) {
                for (int it = 0; it < part_steps; ++it) {
                    if (chunk_index(star, it) != s_row_arg / kN) continue;
                    stored(it, q);
                    float conf = q[0];
#pragma unroll
                    for (int e = 1; e < kN; ++e) conf = e == s_row_arg % kN ? q[e] : conf;
                    tokens[r] = s_row_arg; confidence[r] = conf;
                }
                return;
            }
            double total = 0.0, before = 0.0, cum = 0.0;
            for (int it = 0; it < part_steps; ++it) total += (double)stored(it, q);
            total = wave_sum(total);
            if (lane == 0) s_mass[wv] = total;
            lds_barrier();
            const double tau = s_tau;
            if (find_piece(lane < NW ? s_mass[lane & (NW - 1)] : 0.0, s_before, tau, lane, before) != wv) return;
            int step = -1, owner = 0;
            for (int it = 0; it < part_steps; ++it) {
                const double mine = (double)stored(it, q), upto = before + wave_scan_incl(mine, lane);
                const unsigned long long cross = __ballot(mine > 0.0 && upto > tau), filled = __ballot(mine > 0.0);
                if (filled) {
                    step = it;
                    owner = cross ? (int)__builtin_ctzll(cross) : 63 - (int)__builtin_clzll(filled);
                    cum = upto - mine;
                }
                if (cross) break;
                before = last_lane(upto);
            }
            stored(max(step, 0), q);                         // (the piece has mass: some step has)
            const int pick = pick_element<kN>(q, cum, 1.0, tau);
            float conf = q[0];
#pragma unroll
            for (int e = 1; e < kN; ++e) conf = e == pick ? q[e] : conf;
            if (lane == owner) { tokens[r] = chunk_index(star, max(step, 0)) * kN + pick; confidence[r] = conf; }
            return;
        }
    }

    // ---- the own part: weights and their sum ----------------------------------------------------------------------
    float w[kDraftSteps][kN], z_t = 0.f;
    Ref ref;
    int top = V;                                             // (greedy rows) first element with the thread's maximum
    {
        const __amdgpu_buffer_rsrc_t rl = part_row(h);
        const int n = part_size(h);
        uint4 lg[kDraftSteps];
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) {           // (steps a part does not have: no traffic, -inf)
            lg[it] = make_uint4(0, 0, 0, 0);
            if (it < part_steps) lg[it] = part_load16<kAuxDefault>(rl, (uint32_t)my_chunk * 16u, it * (kWave * 16));
        }
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) Chunk<LT>::blank(lg[it], it >= part_steps || my_chunk + it * kWave >= n);
        ref = ref_of(thread_max_of_numbers<LT, kDraftSteps>(lg));
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) {
            keep_packed(lg[it]);
            if (!sampled && top == V && ref.m > -INFINITY && chunk_max<LT>(lg[it], -INFINITY) == ref.m)
                top = first_with(lg[it], ref.m, chunk_index(h, it));
            z_t = add_weights(lg[it], ref, z_t, w[it]);
            __builtin_amdgcn_sched_barrier(0);               // (one step at a time: registers)
        }
    }
    leave_stats(ref, z_t, top);
    lds_barrier();
    const unsigned int others = (unsigned int)((1ull << n_parts) - 1ull) & ~(1u << h);
    if (wv == 0) {
        float m;
        double Z;
        int arg;
        take_stats(h, m, Z, arg);
        unsigned int missing = 0u;
        if (n_parts > 1) {
            if (lane == 0) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (the mass of an earlier launch is taken back)
                publish_marked(&words[h].top, (unsigned long long)__float_as_uint(m) | ((unsigned long long)(uint32_t)arg << 32), mark);
                publish_marked(&words[h].Z, word_of(Z), mark);
            }
            const int p = lane & 31;                                 // lanes 0..31 the maxima, 32..63 the normalisers
            const bool other = (others >> p) & 1u;
            unsigned long long v = 0ull;
            const unsigned long long got = __ballot(take_marked(lane < 32 ? &words[p].top : &words[p].Z, other, mark, v));
            const unsigned int both = (unsigned int)got & (unsigned int)(got >> 32);
            if (other && ((both >> p) & 1u)) {
                if (lane < 32) { s_part_m[p] = __uint_as_float((uint32_t)v); s_part_i[p] = (int)(v >> 32); }
                else s_part_z[p] = double_of(v);
            }
            missing = others & ~both;
        }
        if (missing == 0u) row_stats();
        if (lane == 0) s_missing = missing;
    }
    lds_barrier();
    // (of a part whose statistics did not come in time the mass may be an earlier replay's: not looked at below)
    const unsigned int late = __builtin_amdgcn_readfirstlane(s_missing);
    if (late != 0u) {
        for (unsigned int left = late; left != 0u; left &= left - 1u) compute_stats((int)__builtin_ctz(left));
        if (wv == 0) row_stats();
        lds_barrier();
    }

    const bool counted = sampled || n_parts > 1;             // (the mass of a whole greedy row tells nobody anything)

    // ---- the probabilities, rounded, and their mass -----------------------------------------------------------
    const float row_m = s_row_m, row_inv = s_row_inv, mc = scaled_ref(row_m, c);
    {
        const float f = thread_factor(ref);
        double total = 0.0;
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) {
            if (it >= part_steps) break;
            total += (double)round_probs(w[it], f, row_m, mc, row_inv);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (counted) {
            total = wave_sum(total);
            if (lane == 0) s_z[wv] = total;
        }
    }
    if (counted) lds_barrier();
    if (wv == 0 && counted) {
        const double mass = wave_sum(lane < NW ? s_z[lane] : 0.0);
        if (lane == 0) {
            if (n_parts > 1) publish_marked(&words[h].mass, word_of(mass), mark);
            s_part_z[h] = mass;
        }
    }
    // (the mass is out: the probabilities may follow)
    {
        const __amdgpu_buffer_rsrc_t rp = part_probs(h);
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) {
            if (it >= part_steps) break;
            store_chunk(rp, it, w[it]);
        }
    }
    // the draw (wavefront 0, all masses known): the part, then the wavefront of it, that holds the point
    auto draw = [&]() {
        if (n_parts > 1 && lane == 0) { take_back(&words[h].top); take_back(&words[h].Z); }
        int star = -1, wave = -1;
        double before = 0.0, tau = 0.0;
        if (sampled) {
            const double at = lane < n_parts ? s_part_z[lane & 31] : 0.0;
            tau = (double)u * wave_sum(at);
            star = find_piece(at, 0.0, tau, lane, before);
            if (star == h) {
                double ahead;
                wave = find_piece(lane < NW ? s_mass[lane] : 0.0, before, tau, lane, ahead);
                before = ahead;
            }
        } else if (s_row_arg >= 0) {
            star = s_row_arg / kN / part_chunks;
            wave = s_row_arg / kN % part_chunks / (part_steps * kWave);
        }
        if (star < 0 && h == 0 && lane == 0) { tokens[r] = 0; confidence[r] = 0.f; }      // no mass (non-finite input): stay defined
        if (lane == 0) { s_star = star; s_wave = wave; s_before = before; s_tau = tau; }
    };
    if (wv == 0) {
        if (lane < NW) s_mass[lane] = s_z[lane];
        unsigned int missing = 0u;
        if (n_parts > 1) {
            const bool other = (others >> (lane & 31)) & (unsigned int)(lane < 32);
            unsigned long long v = 0ull;
            const bool got = take_marked(&words[lane & 31].mass, other && !((late >> (lane & 31)) & 1u), mark, v);
            if (got) s_part_z[lane & 31] = double_of(v);
            missing = (unsigned int)__ballot(other && !got);
        }
        if (missing == 0u) draw();
        if (lane == 0) s_missing = missing;
    }
    lds_barrier();
    const unsigned int gone = __builtin_amdgcn_readfirstlane(s_missing);
    if (gone != 0u) {
        for (unsigned int left = gone; left != 0u; left &= left - 1u) compute_mass((int)__builtin_ctz(left), false);
        if (wv == 0) draw();
        lds_barrier();
    }
    if (s_star != h || s_wave != wv) return;

    // ---- one wavefront of one part: the step, the lane, the element -----------------------------------------
    const double tau = s_tau;
    double before = s_before, cum = 0.0;
    int step = -1, owner = 0, pick = 0;
    if (sampled) {
#pragma unroll
        for (int it = 0; it < kDraftSteps; ++it) {
            if (it >= part_steps) break;
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < kN; ++e) acc += w[it][e];
            const double mine = (double)acc, upto = before + wave_scan_incl(mine, lane);
            const unsigned long long cross = __ballot(mine > 0.0 && upto > tau), filled = __ballot(mine > 0.0);
            if (filled) {
                step = it;
                owner = cross ? (int)__builtin_ctzll(cross) : 63 - (int)__builtin_clzll(filled);
                cum = upto - mine;
            }
            if (cross) break;
            before = last_lane(upto);
        }
        if (step < 0) {
            if (lane == 0) { tokens[r] = 0; confidence[r] = 0.f; }
            return;
        }
    } else {
        const int at = s_row_arg / kN % part_chunks - wv * (part_steps * kWave);
        step = at / kWave; owner = at % kWave; pick = s_row_arg % kN;
    }
#pragma unroll
    for (int it = 0; it < kDraftSteps; ++it) {
        if (it != step) continue;
        if (sampled) pick = pick_element<kN>(w[it], cum, 1.0, tau);
        float conf = w[it][0];
#pragma unroll
        for (int e = 1; e < kN; ++e) conf = e == pick ? w[it][e] : conf;
        if (lane == owner) { tokens[r] = (h * part_chunks + my_chunk + it * kWave) * kN + pick; confidence[r] = conf; }
    }
}

bool draft_parts_supported(const adaspec_draft_dims &d) { return d.vocab % 8 == 0 && d.vocab <= kPartsMaxVocab; }

// DraftWords[R][parts].  A row's share is what it was when rows were swept by three kernels: statistics of eight parts and
// 32 bytes per 1024 chunks.
static size_t row_bytes(const adaspec_draft_dims &d) { return kStatParts * sizeof(HalfStat) + (size_t)parts_sum_parts(d.vocab, d.logits_dtype) * kQW * sizeof(double); }
size_t draft_parts_workspace_bytes(const adaspec_draft_dims &d)
{
    return align_up((size_t)d.rows * kStatParts * sizeof(HalfStat), 256) + (size_t)d.rows * parts_sum_parts(d.vocab, d.logits_dtype) * kQW * sizeof(double);
}

hipError_t launch_draft_parts(const void *logits, const float *temperature, const float *uniforms,
                              const int32_t *out_rows, void *probs, int32_t *tokens, float *confidence,
                              const adaspec_draft_dims &d, char *ws, int compute_units, hipStream_t stream)
{
    if (d.rows == 0) return hipSuccess;
    const int64_t lstride = d.logits_row_stride * (d.logits_dtype == ADASPEC_F32 ? 4 : 2);
    const int64_t pstride = d.probs_row_stride * (d.probs_dtype == ADASPEC_F32 ? 4 : 2);
    // Short rows are not shared: the exchanges take longer than what is saved (captured calls, V = 16384 bf16, 1 / 64 / 128 rows in
    // parts 8.2 / 9.1 / 9.3 us, whole 7.3 / 8.0 / 8.3; V = 24576 whole 8.7 / 9.5 / 10.4, in parts 8.1 / 9.2 / 9.8).
    // Else as many parts as there are compute units for: where a compute unit has two of them the second starts 2-3 us later, and
    // everybody waits for it (V = 16384, 128 rows in 512 parts 11.7, in 256 9.3).  Where 512 threads hold too little for that and
    // 1024 do not, 1024 (128 rows of V = 128256 19.8 / 18.9, 192 of 65536 18.6 / 15.6; where both could, 512: 1 row 8.8 / 10.8).
    const int chunks = d.vocab / parts_chunk_elems(d.logits_dtype);
    auto least_parts = [&](int threads) { return ceil_div(chunks, threads * kDraftSteps); };
    const bool wide = (int64_t)d.rows * least_parts(kDraftT) > compute_units && (int64_t)d.rows * least_parts(kDraftWideT) <= compute_units;
    const int threads = wide ? kDraftWideT : kDraftT, steps = ceil_div(chunks, threads), least = least_parts(threads);
    const int room = (int)(row_bytes(d) / sizeof(DraftWords)), most = room < kDraftMaxParts ? room : kDraftMaxParts;
    int n_parts = steps * parts_chunk_elems(d.logits_dtype) <= kDraftWholeElems ? 1 : compute_units / d.rows;
    n_parts = n_parts < least ? least : n_parts > most ? most : n_parts;
    const int part_steps = ceil_div(steps, n_parts);
    n_parts = ceil_div(steps, part_steps);
    // Whether some row may go where its logits are (out_rows is on the device): the rows lie where destinations may be and, with equal
    // strides, whole rows apart.
    const int64_t apart = (int64_t)(reinterpret_cast<intptr_t>(logits) - reinterpret_cast<intptr_t>(probs));
    const bool in_place = apart + (d.rows - 1) * lstride >= 0 && (out_rows || apart <= (d.rows - 1) * pstride) &&
                          (lstride != pstride || apart % pstride == 0);
    auto launch = [&](auto lt, auto pt) {
        using LT = decltype(lt);
        using PT = decltype(pt);
        auto kernel = wide ? draft_row_kernel<LT, PT, kDraftWideT, false> : draft_row_kernel<LT, PT, kDraftT, false>;
        if constexpr (sizeof(typename LT::storage) == sizeof(typename PT::storage)) {
            if (in_place) kernel = wide ? draft_row_kernel<LT, PT, kDraftWideT, true> : draft_row_kernel<LT, PT, kDraftT, true>;
        }
        hipLaunchKernelGGL(kernel, dim3(d.rows * n_parts), dim3(threads), 0, stream, (const char *)logits,
                           temperature, uniforms, out_rows, (char *)probs, tokens, confidence, d.vocab, n_parts, part_steps,
                           lstride, pstride, reinterpret_cast<DraftWords *>(ws), (unsigned long long)next_spread_mark());
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
