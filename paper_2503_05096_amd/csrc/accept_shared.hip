// Two-pass acceptance in row parts, the second pass for fp32 logits and short rows: one or a few workgroups per request, which share its
// deciding row, each with its part in registers (the first pass, and the second one of longer 16-bit rows: accept_parts.hip).
//
// Workgroup (request, part) of 512 threads: the request's deciding row from the first pass's records (accept_head.h), its part of
// that row and of its draft probabilities into registers, the part's mass to the others and theirs from them
// (part_exchange.h); the part that holds the point tau = u1 * R finds the token in its registers.
// What a part tells the others (PartWords): a draft row, whose (m, Z) all of them know, its residual mass; a bonus row its mass relative
// to its own maximum, and that; a greedy bonus row (maximum, arg-max).
//
// Bound: HBM (64 rejected rows of V = 128256: 66 MB) behind a chain of dependent accesses: records, row, the others' words.
// accept_decide_kernel takes 16 KB parts, for fp32 rows twice as many as for 16-bit ones (2048 workgroups of 64 requests take 4.8 us to
// start), sums residual and probability, draws a ticket and reads the winner's chunks again.  MI355X, second pass of 64 requests of
// V = 128256 in fp32, accept_decide_kernel / this one: 22.6 / 16.1 us, all bonus rows 21.9 / 14.4; whole calls 40.1 / 33.1, 25.0 / 16.4, all
// greedy 25.1 / 25.5; 32 of 152064 35.8 / 28.2, 50 of 262144 48.0 / 30.5, 8 of 128256 15.3 / 13.5.  16 bits, V = 4000, captured: 1 request 11.6 / 10.7,
// 64 13.8 / 11.9, 300 15.6 / 13.7; V = 12000 64 13.7 / 13.1, 300 17.6 / 16.7.
#include "accept_head.h"
#include "part_exchange.h"

namespace adaspec {

constexpr int kDecideT = 512;
// chunks per thread at most (probabilities wider than the logits take twice the registers)
constexpr int decide_steps(int logits_size, int probs_size) { return probs_size > logits_size ? 4 : 8; }
constexpr int kDecideMaxParts = 32;                       // two lanes each in the exchange
static_assert(kPartsMaxVocab <= kDecideMaxParts * kDecideT * 8 * 4, "fp32 rows fit");
struct PartWords { unsigned long long mass, top; };

// One chunk: r_v = max(0, e_v / Z - q_v), or p_v = e_v / Z itself, with e_v = 2^((l_v - m) c).
// The sums and the final search both call this, so they see the same numbers.
template <class LT, class PT>
__device__ __forceinline__ float chunk_masses(const uint4 &lv, const ProbChunk<Chunk<LT>::kN, PT> &qv, float m, float c,
                                              float mc, float invZ, bool use_p, float (&rv)[Chunk<LT>::kN])
{
    constexpr int N = Chunk<LT>::kN;
    float x[N], q[N], acc = 0.f;
    Chunk<LT>::unpack(lv, x);
    qv.unpack(q);
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float w = exp_weight<LT>(x[e], m, c, mc);
        rv[e] = use_p ? w * invZ : fmaxf(0.f, fmaf(w, invZ, -q[e]));
        acc += rv[e];
    }
    return acc;
}

template <class LT, class PT>
__global__ __launch_bounds__(kDecideT, 4) void accept_decide_shared_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs,
    const int32_t *__restrict__ draft_tokens, const float *__restrict__ uniforms,
    const int32_t *__restrict__ spec_lens, const float *__restrict__ temperature, int V, int total_q,
    int total_draft, int max_spec_len, int n_stat_parts, int n_parts, int part_steps, int64_t lstride, int64_t pstride,
    const int32_t *__restrict__ cu_q, const SlotRec *__restrict__ slot_rec,
    const HalfStat *__restrict__ part_stat, int out_stride, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ out_accept_len, PartWords *__restrict__ all_words)
{
    // (a part gives the same bits whether its own workgroup computes it or another one)
#pragma clang fp contract(off)
    constexpr int kN = Chunk<LT>::kN, kLSize = (int)sizeof(typename LT::storage), kPSize = (int)sizeof(typename PT::storage);
    constexpr int kSteps = decide_steps(kLSize, kPSize), NW = kDecideT / kWave;
    __shared__ float s_m[NW];
    __shared__ int s_i[NW];
    __shared__ double s_mass[NW], s_own[NW];      // masses of a part's wavefronts; of the own part's
    __shared__ double s_part_mass[kDecideMaxParts];
    __shared__ unsigned long long s_part_top[kDecideMaxParts];
    __shared__ unsigned int s_missing;
    __shared__ int s_star, s_wave, s_again;
    __shared__ double s_before, s_tau, s_scale;
    using Probs = ProbChunk<kN, PT>;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = blockIdx.x / n_parts, h = blockIdx.x % n_parts;

    __shared__ DecidingScratch s_dec;
    const DecidingRow d = deciding_row<LT>(s_dec, i, cu_q, spec_lens, temperature, slot_rec, part_stat, max_spec_len, n_stat_parts, lane, wv);
    const int start = d.start, k = d.k, a = d.a;
    const bool sampled = d.sampled;
    const float c = d.c;
    const int r = start + a;
    const bool bonus = a >= k;
    int32_t *o = out_tokens + (int64_t)i * out_stride;
    if (h == 0 && wv == 1) {                  // everything but the sampled token
        for (int jj = lane; jj < out_stride; jj += kWave)
            if (jj != a) o[jj] = (jj < a && start - i + jj < total_draft) ? draft_tokens[start - i + jj] : -1;
        if (lane == 0) out_accept_len[i] = a;
    }
    if (r >= total_q) {                       // inconsistent lengths: stay inside the tensors
        if (h == 0 && tid == 0) o[a] = 0;
        return;
    }
    if (!sampled && !bonus) {                 // greedy and rejected: the row's arg-max, already merged
        if (h == 0 && tid == 0) o[a] = d.row.arg;
        return;
    }

    // ---- a part of the deciding row (and of its draft probabilities), in registers ---------------------
    // wavefront w holds 64 * part_steps chunks of it in a row, lane l of its step it the chunk 64 it + l of those
    const int row_chunks = V / kN, part_chunks = part_steps * kDecideT;
    const int my_chunk = wv * (part_steps * kWave) + lane;           // of step 0, inside a part
    const char *lrow = logits + (int64_t)r * lstride * kLSize;
    const char *prow = probs + (int64_t)(r - i) * pstride * kPSize;
    const bool has_q = sampled && !bonus;
    const float u_draw = uniforms[2 * (int64_t)r + 1];
    auto part_size = [&](int part) -> int { return max(0, min(row_chunks - part * part_chunks, part_chunks)); };
    auto part_logits = [&](int part) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(lrow) + (int64_t)part * part_chunks * 16, 0, part_size(part) * 16, 0x00020000);
    };
    // (a bonus row has no draft probabilities: descriptor of size zero, the loads return zeros)
    auto part_probs = [&](int part) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(prow) + (int64_t)part * part_chunks * Probs::kBytes, 0,
                                                 has_q ? part_size(part) * Probs::kBytes : 0, 0x00020000);
    };
    uint4 lg[kSteps];
    Probs qg[kSteps];
    {
        const __amdgpu_buffer_rsrc_t rl = part_logits(h), rq = part_probs(h);
#pragma unroll
        for (int it = 0; it < kSteps; ++it) {                // (steps a part does not have: no traffic, -inf)
            lg[it] = make_uint4(0, 0, 0, 0);
            qg[it].zero();
            if (it < part_steps) lg[it] = part_load16<kAuxDefault>(rl, (uint32_t)my_chunk * 16u, it * (kWave * 16));
        }
#pragma unroll
        for (int it = 0; it < kSteps; ++it)
            if (it < part_steps) qg[it].load(rq, (uint32_t)(my_chunk * Probs::kBytes), it * (kWave * Probs::kBytes));
        const int n = part_size(h);
#pragma unroll
        for (int it = 0; it < kSteps; ++it) Chunk<LT>::blank(lg[it], it >= part_steps || my_chunk + it * kWave >= n);
    }

    // ---- what a part amounts to: the steps of the way that its own workgroup and, where its words do not come, others
    // share.  A bonus row was not seen by the first pass: its parts are relative to their own maxima.
    auto leave_max = [&](float m_t) { m_t = wave_max(m_t <= lowest_ref<LT>(c) ? -INFINITY : m_t); if (lane == 0) s_m[wv] = m_t; };
    auto take_max = [&]() -> float {
        float m = s_m[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, s_m[w]);
        return m;
    };
    struct Scale { float m, mc, invZ; };
    const float row_m = d.row.m;
    const Scale draft_scale{row_m, scaled_ref(row_m, c), (float)(1.0 / d.row.Z)};
    // (a part without a finite logit: weights of 0)
    auto bonus_scale = [&](float m) -> Scale { return m > -INFINITY ? Scale{m, scaled_ref(m, c), 1.f} : Scale{0.f, 0.f, 1.f}; };
    auto leave_mass = [&](double mass) { mass = wave_sum(mass); if (lane == 0) s_mass[wv] = mass; };
    auto leave_argmax = [&](ArgMax best) {
        best = wave_argmax(best);
        if (lane == 0) { s_m[wv] = best.v; s_i[wv] = best.i; }
    };
    // (wavefront 0) the part as a whole, in LDS
    auto take_part = [&](int part, float m) {
        double mass = 0.0;
        unsigned long long top = __float_as_uint(m);
        if (sampled) {
            mass = wave_sum(lane < NW ? s_mass[lane] : 0.0);
        } else {
            const ArgMax b = wave_argmax(lane < NW ? ArgMax{s_m[lane], s_i[lane]} : ArgMax{-INFINITY, V});
            top = (unsigned long long)__float_as_uint(b.v) | ((unsigned long long)(uint32_t)b.i << 32);
        }
        if (lane == 0) { s_part_mass[part] = mass; s_part_top[part] = top; }
    };
    auto chunk_argmax = [&](const uint4 &lv, int chunk, ArgMax best) -> ArgMax {
        float x[kN];
        Chunk<LT>::unpack(lv, x);
#pragma unroll
        for (int e = 0; e < kN; ++e)
            if (x[e] > best.v) best = ArgMax{x[e], chunk * kN + e};
        return best;
    };
    // (wavefront 0, all parts known) the part, then the wavefront of it, that holds the point
    auto decide = [&](bool use_p) {
        int star = -1, wave = -1, again = 0;
        double before = 0.0, tau = 0.0, scale = 1.0;
        if (!sampled) {
            ArgMax b{-INFINITY, V};
            if (lane < n_parts) b = ArgMax{__uint_as_float((uint32_t)s_part_top[lane]), (int)(s_part_top[lane] >> 32)};
            b = wave_argmax(b);
            if (lane == 0 && h == 0) o[a] = b.i < V ? b.i : 0;
            star = n_parts;                                   // (nothing left to do)
        } else {
            double at = lane < n_parts ? s_part_mass[lane & (kDecideMaxParts - 1)] : 0.0, sc = 1.0;
            if (bonus) {                                      // all parts on one scale
                const float mp = lane < n_parts ? __uint_as_float((uint32_t)s_part_top[lane & (kDecideMaxParts - 1)]) : -INFINITY;
                const float M = wave_max(mp);
                sc = mp > -INFINITY ? (double)__builtin_amdgcn_exp2f(ref_gap<LT>(mp, M, c)) : 0.0;
                at = mp > -INFINITY ? at * sc : 0.0;
            }
            const double R = wave_sum(at);
            if (!(R > 0.0) && !use_p) {
                again = 1;
            } else {
                tau = (double)u_draw * R;
                star = find_piece(at, 0.0, tau, lane, before);
                if (star < 0 && h == 0 && lane == 0) o[a] = 0;           // no mass anywhere (non-finite input): stay defined
                scale = __shfl(sc, h, kWave);
                if (star == h) {
                    double ahead;
                    wave = find_piece(lane < NW ? s_own[lane] * scale : 0.0, before, tau, lane, ahead);
                    before = ahead;
                }
            }
        }
        if (lane == 0) { s_star = star; s_wave = wave; s_again = again; s_before = before; s_tau = tau; s_scale = scale; }
    };

    // ---- the own part, and the words of the others ----------------------------------------------------------
    Scale own = draft_scale;
    float own_m = row_m;
    if (bonus && sampled) {
        leave_max(thread_max_of_numbers<LT, kSteps>(lg));
        lds_barrier();
        own_m = take_max();
        own = bonus_scale(own_m);
    }
    if (sampled) {
        double mass = 0.0;
#pragma unroll
        for (int it = 0; it < kSteps; ++it) {
            if (it >= part_steps) break;
            float rv[kN];
            keep_packed(lg[it]);
            qg[it].keep();
            mass += (double)chunk_masses<LT, PT>(lg[it], qg[it], own.m, c, own.mc, own.invZ, bonus, rv);
            __builtin_amdgcn_sched_barrier(0);               // (one step at a time: registers)
        }
        leave_mass(mass);
    } else {
        ArgMax best{-INFINITY, V};
#pragma unroll
        for (int it = 0; it < kSteps; ++it) {
            if (it >= part_steps) break;
            best = chunk_argmax(lg[it], h * part_chunks + my_chunk + it * kWave, best);
            __builtin_amdgcn_sched_barrier(0);
        }
        leave_argmax(best);
    }
    lds_barrier();
    PartWords *words = all_words + (int64_t)i * n_parts;
    if (wv == 0) {
        take_part(h, own_m);
        if (lane < NW) s_own[lane] = s_mass[lane];
        unsigned int missing = 0u;
        if (n_parts > 1) {
            if (lane == 0 && sampled) publish_u64(&words[h].mass, word_of(s_part_mass[h]));
            if (lane == 0 && bonus) publish_u64(&words[h].top, s_part_top[h]);
            // lanes 0..31 the masses, 32..63 the maxima, as far as there are any
            const int p = lane & (kDecideMaxParts - 1);
            const bool other = p < n_parts && p != h;
            const unsigned long long v = take_words(lane < kDecideMaxParts ? &words[p].mass : &words[p].top,
                                                    other && (lane < kDecideMaxParts ? sampled : bonus));
            const bool there = v != kNoWord || !(lane < kDecideMaxParts ? sampled : bonus);
            const unsigned long long got = __ballot(other && there);
            const unsigned int both = (unsigned int)got & (unsigned int)(got >> 32);
            if (other && ((both >> p) & 1u)) {
                if (lane < kDecideMaxParts) s_part_mass[p] = sampled ? double_of(v) : 0.0;
                else s_part_top[p] = v;
            }
            missing = (unsigned int)(__ballot(other) & 0xffffffffull) & ~both;
        }
        if (missing == 0u) decide(bonus);
        if (lane == 0) s_missing = missing;
    }
    lds_barrier();
    bool use_p = bonus;
    unsigned int left = __builtin_amdgcn_readfirstlane(s_missing);
    if (left != 0u || s_again) {
        // Parts whose words did not come, chunk by chunk; then, if no part has residual mass (p == q everywhere), all of them with p
        for (;;) {
            if (left == 0u) {
                use_p = true;
                left = (unsigned int)((1ull << n_parts) - 1ull);
            }
            for (; left != 0u; left &= left - 1u) {
                const int part = (int)__builtin_ctz(left);
                const __amdgpu_buffer_rsrc_t rl = part_logits(part), rq = part_probs(part);
                const int n = part_size(part);
                auto chunk_at = [&](int it) -> uint4 {
                    uint4 v = part_load16<kAuxDefault>(rl, (uint32_t)my_chunk * 16u, it * (kWave * 16));
                    Chunk<LT>::blank(v, my_chunk + it * kWave >= n);
                    return v;
                };
                lds_barrier();                               // (what the turn before left has been read)
                float m = row_m;
                if (!sampled) {
                    ArgMax best{-INFINITY, V};
                    for (int it = 0; it < part_steps; ++it) best = chunk_argmax(chunk_at(it), part * part_chunks + my_chunk + it * kWave, best);
                    leave_argmax(best);
                } else {
                    Scale sc = draft_scale;
                    if (bonus) {
                        m = -INFINITY;
                        for (int it = 0; it < part_steps; ++it) m = chunk_max<LT>(chunk_at(it), m);
                        leave_max(m);
                        lds_barrier();
                        m = take_max();
                        sc = bonus_scale(m);
                    }
                    double mass = 0.0;
                    for (int it = 0; it < part_steps; ++it) {
                        float rv[kN];
                        Probs q;
                        q.load(rq, (uint32_t)(my_chunk * Probs::kBytes), it * (kWave * Probs::kBytes));
                        mass += (double)chunk_masses<LT, PT>(chunk_at(it), q, sc.m, c, sc.mc, sc.invZ, use_p, rv);
                    }
                    leave_mass(mass);
                }
                lds_barrier();
                if (wv == 0) {
                    take_part(part, m);
                    if (part == h && lane < NW) s_own[lane] = s_mass[lane];
                }
            }
            if (wv == 0) decide(use_p);
            lds_barrier();
            if (!s_again || use_p) break;
        }
    }
    if (s_star != h || s_wave != wv) return;

    // ---- one wavefront of one part: the step, then the lane, then the element ------------------------------
    const double tau = s_tau, scale = s_scale;
    double before = s_before, cum = 0.0;
    int step = -1, owner = 0;
#pragma unroll
    for (int it = 0; it < kSteps; ++it) {
        if (it >= part_steps) break;
        float rv[kN];
        keep_packed(lg[it]);
        qg[it].keep();
        const double mine = (double)chunk_masses<LT, PT>(lg[it], qg[it], own.m, c, own.mc, own.invZ, use_p, rv) * scale;
        const double upto = before + wave_scan_incl(mine, lane);
        const unsigned long long cross = __ballot(mine > 0.0 && upto > tau), filled = __ballot(mine > 0.0);
        if (filled) {
            step = it;
            owner = cross ? (int)__builtin_ctzll(cross) : 63 - (int)__builtin_clzll(filled);
            cum = upto - mine;
        }
        if (cross) break;
        before = last_lane(upto);
    }
    if (step < 0) {                           // the sums said there was mass here, the recomputation finds none
        if (lane == 0) o[a] = 0;
        return;
    }
#pragma unroll
    for (int it = 0; it < kSteps; ++it) {
        if (it != step) continue;
        float rv[kN];
        chunk_masses<LT, PT>(lg[it], qg[it], own.m, c, own.mc, own.invZ, use_p, rv);
        if (lane == owner) o[a] = (h * part_chunks + my_chunk + it * kWave) * kN + pick_element<kN>(rv, cum, scale, tau);
    }
}

// Parts of the deciding rows (0: the call is not for this kernel).  As many as make the fullest compute unit's work the least: turns
// times (chunks per thread, and two for what a turn costs besides), and one for an exchange.  fp32, 64 requests of V = 128256: 8
// parts; 150 of V = 32000: three 25.1 us, two 26.5.
// A compute unit holds two of these workgroups, and the many small ones of accept_decide_kernel fill the chip better than a second
// turn does (us per captured call, accept_decide_kernel / here, 0-4 drafts, sampled | a third greedy | all greedy: 160 requests of V =
// 50272 32.8 / 34.7 | 29.7 / 32.2 | 21.4 / 22.8, 200 of 40000 31.3 / 35.6 | 28.9 / 31.7 | 20.7 / 23.3, 300 of 16384 23.5 / 26.5 |
// 22.0 / 24.0 | 15.3 / 17.3; within one turn 128 of 50272 28.9 / 27.0 | 25.9 / 25.7 | 17.7 / 18.8, 64 of 32000 16.0 / 14.9 | 15.0 /
// 14.2 | 10.7 / 11.2), except with rows of eight full parts and more (V = 128256, 100: 48.9 / 42.5 | 42.4 / 39.9 | 29.9 / 30.7, 128: 57.3 /
// 51.4 | 48.7 / 46.3 | 35.1 / 35.3; 100000, 128: 46.8 / 45.8 | 40.7 / 42.6 | 29.2 / 31.7), where a second one still pays.
// 16-bit probabilities beside fp32 logits leave less to read: very short and long rows only (V = 4096, 64: 11.9 / 11.3 | 11.9 / 11.1 |
// 9.7 / 9.3; 32000, 100: 18.9 / 20.3 | 17.4 / 19.6 | 12.6 / 13.6; 50272, 64: 21.0 / 20.1 | 18.9 / 19.4 | 13.0 / 13.8; 80000, 64:
// 26.2 / 22.6 | 22.8 / 21.7 | 15.9 / 16.5).
// 16-bit rows have twice the arithmetic per byte, which here follows
// the loads where many small workgroups overlap it, so only short ones come (accept_decide_kernel / here: V = 16000, 300 requests
// 18.4 / 19.0 us; 128256, 128 39.9 / 40.8; 32000, 150 21.3 / 24.8; 262144, 64 33.2 / 33.2; V = 8000, 1000 29.5 / 34.8).
constexpr int kSharedShortRow = 12288, kSharedManyParts = 8;
constexpr int kSharedFewSteps = 2, kSharedManySteps = 32;    // rows beside narrower probabilities: at most, more than
SharedParts accept_shared_parts(const adaspec_accept_dims &d, int compute_units)
{
    SharedParts p{0, 0, 0};
    const bool f32 = d.logits_dtype == ADASPEC_F32;
    if (!f32 && d.vocab > kSharedShortRow) return p;
    const int most = decide_steps(f32 ? 4 : 2, d.probs_dtype == ADASPEC_F32 ? 4 : 2);
    const int steps = ceil_div(d.vocab / parts_chunk_elems(d.logits_dtype), kDecideT), least = ceil_div(steps, most);
    if (f32 && d.probs_dtype != ADASPEC_F32 && steps > kSharedFewSteps && steps <= kSharedManySteps) return p;
    const int64_t workgroups = (int64_t)compute_units * (least >= kSharedManyParts ? 4 : 2);
    // (words of a request lie where the plan has its masses)
    const int room = (int)(accept_parts_sum_bytes(d) / (d.batch > 0 ? d.batch : 1) / sizeof(PartWords));
    int64_t best = INT64_MAX;
    for (int n = least; n <= kDecideMaxParts && n <= steps && n <= room && n * (int64_t)d.batch <= workgroups; ++n) {
        const int each = ceil_div(steps, n);
        const int64_t cost = ((int64_t)d.batch * n + compute_units - 1) / compute_units * (each + 2) + (n > 1 ? 1 : 0);
        if (ceil_div(steps, each) == n && cost < best) {
            best = cost;
            p.n_parts = n;
            p.part_steps = each;
        }
    }
    p.n_words = p.n_parts * (int)(sizeof(PartWords) / sizeof(unsigned long long));
    return p;
}

void launch_accept_shared(const AcceptArgs &a, const SharedParts &p, int n_stat_parts)
{
    const adaspec_accept_dims &d = a.dims;
    auto launch = [&](auto lt, auto pt) {
        hipLaunchKernelGGL((accept_decide_shared_kernel<decltype(lt), decltype(pt)>), dim3(d.batch * p.n_parts), dim3(kDecideT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.draft_tokens, a.uniforms, a.spec_lens, a.temperature,
                           d.vocab, d.total_q, d.total_draft, d.max_spec_len, n_stat_parts, p.n_parts, p.part_steps,
                           d.logits_row_stride, d.probs_row_stride, (const int32_t *)(a.ws + a.plan.off_cu_q),
                           (const SlotRec *)(a.ws + a.plan.off_slot_rec), (const HalfStat *)(a.ws + a.plan.off_part_stat),
                           d.out_stride, a.out_tokens, a.out_accept_len, (PartWords *)(a.ws + a.plan.off_part));
    };
    auto with_p = [&](auto lt) {
        if (d.probs_dtype == ADASPEC_F32) launch(lt, F32{});
        else if (d.probs_dtype == ADASPEC_F16) launch(lt, F16{});
        else launch(lt, BF16{});
    };
    if (d.logits_dtype == ADASPEC_F32) with_p(F32{});
    else if (d.logits_dtype == ADASPEC_F16) with_p(F16{});
    else with_p(BF16{});
}

}  // namespace adaspec
