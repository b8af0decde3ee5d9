// Tree acceptance for 16-bit logits and draft probabilities of one type, V % 8 == 0,
// V <= 524288 (the shapes of the streaming chain kernel), in two kernels:
//
//   1. node statistics: every node's logits row read once, in steps of 8192 elements shared out to small
//      workgroups: per step the maximum and, for a sampled request, the normaliser relative to it (greedy:
//      the arg-max); and per draft node what its accept test needs (its token, the token's logit and draft
//      probability at the parent, the uniform) beside its parent;
//   2. the walk, one workgroup per request: from the root, at every node it reaches it tests
//      the children in turn and, after each rejection, sweeps the node's logits and
//      draft-probability rows once for the next residual mass; where the walk stops it draws
//      the token.  It writes the request's outputs itself.
// Nodes the walk does not reach cost their statistics only, and a node where the first child
// is accepted never reads its draft-probability row.
//
// Same procedure as the portable node kernel (tree.hip):
//   stage 0: P = softmax(logits / T); after each rejected child r = max(0, P - q), P = r / sum(r),
// evaluated in its closed form (see kernel 2).
// The row is walked by 1024 threads with 16-byte loads: element (s * 1024 + t) * 8 + e belongs
// to step s, thread t.  A "sweep" leaves, per step, the total mass S[s] (fp32 sums over the 128
// elements of 16 neighbouring lanes, fp64 above that); R = sum of the S[s].  The draw needs no
// sweep of its own: the step where the prefix crosses comes from S[]; the threads then load
// their 8 elements of that one step again, a scan over the threads finds the one where the
// prefix crosses, and it picks the element.  A test is arithmetic on values already on chip.
//
// Bound: HBM for the statistics; vector arithmetic of one compute unit per sweep in the walk (about 9.6 us at
// V = 128256), whose longest chain of sweeps sets its time.  MI355X, 64 requests, 288 nodes, trees of width 3:
// statistics 16.0 us (one 1024-thread workgroup per node: 23.7), walk 47.2 us with three dependent loads more at every
// node and the test values fetched there, 42.9 without, 39.5 with searches by ballots, 33.5 with unnormalised sweeps,
// 35.2 since every exponent is a difference again (one more operation per element; the accept test's p is off by 7e-8 on
// average instead of 3.2e-7, and a drawn token differed from the walk in 64 bits in 7 of 38400 requests instead of 13).
#include "adaspec_internal.h"
#include "device_utils.h"
#include "row_parts.h"
#include "row_stream.h"

namespace adaspec {

__device__ __forceinline__ int sane_parent_f(int p, int j) { return j == 0 ? -1 : min(max(p, 0), j - 1); }

// What kernel 1 leaves per node: a record for the accept test (nodes j >= 1), then per step of 8192 elements the
// (maximum, arg-max, normaliser) of its elements.
struct TreeNodeRec { int parent, x; float l, q, u0; int pad[3]; };
constexpr int kStatsWgsPerCu = 6;                   // statistics: workgroups per compute unit the launch aims for (all resident)
constexpr int kStepChunks = kNT;                    // 16-byte chunks per step
static_assert(kStepChunks == kSumSteps * kQT, "a step is four chunks per thread of the statistics kernel");
// (528 bytes is what a node took when the workspace rules were laid down: smaller ones keep that size)
size_t tree_node_stat_bytes(int vocab)
{
    const size_t need = sizeof(TreeNodeRec) + (size_t)ceil_div(vocab / 8, kStepChunks) * sizeof(HalfStat);
    return need > kTreeNodeStatMin ? need : kTreeNodeStatMin;
}

// ---- kernel 1: statistics of every node ---------------------------------------------------------
// workgroup = (node, group of steps); the loads of the next step are under way while one is summed.
template <class DT>
__global__ __launch_bounds__(kQT, 6) void tree_node_stats_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs, const int32_t *__restrict__ draft_tokens,
    const int32_t *__restrict__ parents, const float *__restrict__ uniforms, const int32_t *__restrict__ spec_lens,
    const float *__restrict__ temperature, int B, int V, int total_draft, int max_spec_len, int n_groups, int group_steps,
    int64_t lstride, int64_t pstride, char *__restrict__ stats, int stat_bytes)
{
    constexpr int kN = 8;
    __shared__ float s_m[kNSteps][kQW];
    __shared__ double s_z[kNSteps][kQW];
    __shared__ int s_i[kQW], s_tot[kQW], s_own[3];
    __shared__ float s_T;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = blockIdx.x / n_groups, h = blockIdx.x % n_groups;
    const int row_chunks = V / kN, nsteps = ceil_div(row_chunks, kStepChunks);
    const int first = h * group_steps, last = min(nsteps, first + group_steps);
    const __amdgpu_buffer_rsrc_t rl =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(logits) + (int64_t)r * lstride * 2, 0, row_chunks * 16, 0x00020000);
    auto load_step = [&](int s, uint4 (&lg)[kSumSteps]) {            // (past the row: zeros)
#pragma unroll
        for (int it = 0; it < kSumSteps; ++it)
            lg[it] = part_load16<kAuxDefault>(rl, (uint32_t)tid * 16u, (s * kStepChunks + it * kQT) * 16);
    };
    // Which request owns row r is found by a block scan of n_i = k_i + 1, 1024 requests at a time; the lengths of
    // the first ones are requested in front of the row's first step, which travels meanwhile.
    int nn[4];
    float tt[4];
    auto lengths = [&](int base) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + tid * 4 + u;
            nn[u] = i < B ? min(max(spec_lens[i], 0), max_spec_len) + 1 : 0;
            tt[u] = i < B ? temperature[i] : 0.f;
        }
    };
    lengths(0);
    uint4 lg[kSumSteps];
    load_step(first, lg);
    if (tid == 0) s_own[0] = -1;
    int carry = 0;
    for (int base = 0; base < B; base += 4 * kQT) {
        if (base > 0) lengths(base);
        const int n = (nn[0] + nn[1]) + (nn[2] + nn[3]);
        const int inc = wave_scan_incl_dpp(n);
        lds_barrier();                                      // (later trips: s_tot of the trip before has been read)
        if (lane == 63) s_tot[wv] = inc;
        lds_barrier();                                      // LDS only: the row's loads stay in flight
        int pre = carry, tot = carry;
#pragma unroll
        for (int w = 0; w < kQW; ++w) {
            if (w < wv) pre += s_tot[w];
            tot += s_tot[w];
        }
        int start = pre + inc - n;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (r >= start && r < start + nn[u]) { s_own[0] = base + tid * 4 + u; s_own[1] = start; s_T = tt[u]; }
            start += nn[u];
        }
        carry = tot;
        if (r < carry) break;                               // uniform: found
    }
    lds_barrier();
    const int i = s_own[0];
    if (i < 0) return;                                      // no request owns this row (inconsistent metadata)
    const int r0 = s_own[1], j = r - r0;
    const float T = s_T;
    char *node = stats + (int64_t)r * stat_bytes;
    HalfStat *entry = reinterpret_cast<HalfStat *>(node + sizeof(TreeNodeRec));
    if (h == 0 && tid == 0 && j >= 1) {
        TreeNodeRec rec = {};
        rec.parent = sane_parent_f(parents[r], j);
        const int d0 = r0 - i;                              // first draft row of the request
        if (d0 + j - 1 < total_draft) {
            rec.x = draft_tokens[d0 + j - 1];
            const int xa = min(max(rec.x, 0), V - 1);
            rec.l = load_as_float<DT>(logits, (int64_t)(r0 + rec.parent) * lstride + xa);
            rec.q = load_as_float<DT>(probs, (int64_t)(d0 + rec.parent) * pstride + xa);
            rec.u0 = uniforms[2 * (int64_t)(r - 1)];
        }
        *reinterpret_cast<TreeNodeRec *>(node) = rec;
    }
    if (T == 0.0f) {
        // greedy: the arg-max of the group's steps (lowest index on ties), left in its first step
        ArgMax best{-INFINITY, V};
        for (int s = first; s < last; ++s) {
            uint4 nx[kSumSteps];
            load_step(s + 1 < last ? s + 1 : nsteps, nx);            // (another group's step: nothing)
#pragma unroll
            for (int it = 0; it < kSumSteps; ++it) {
                const int chunk = s * kStepChunks + it * kQT + tid;
                Chunk<DT>::blank(lg[it], chunk >= row_chunks);
                float x[kN];
                Chunk<DT>::unpack(lg[it], x);
#pragma unroll
                for (int e = 0; e < kN; ++e)
                    if (x[e] > best.v) best = ArgMax{x[e], chunk * kN + e};
                lg[it] = nx[it];
            }
        }
        best = reduce_argmax(best, s_m[0], s_i, lane, wv);
        if (tid < last - first) {
            HalfStat st;
            st.m = tid == 0 ? best.v : -INFINITY;
            st.arg = tid == 0 && best.i < V ? best.i : -1;
            st.Z = 0.0;
            entry[first + tid] = st;
        }
        return;
    }
    const float c = exponent_scale<DT>(T);
    for (int s = first; s < last; ++s) {
        uint4 nx[kSumSteps];
        load_step(s + 1 < last ? s + 1 : nsteps, nx);            // (another group's step: nothing)
#pragma unroll
        for (int it = 0; it < kSumSteps; ++it) Chunk<DT>::blank(lg[it], s * kStepChunks + it * kQT + tid >= row_chunks);
        // every thread sums against its own maximum; the pairs are merged over the wavefront here, over the
        // wavefronts at the end
        const float mt = thread_max<DT, kSumSteps>(lg);
        float zt = 0.f;
        if (mt > -INFINITY) {
            const float mtc = mt * c;
#pragma unroll
            for (int it = 0; it < kSumSteps; ++it) {
                keep_packed(lg[it]);
                float x[kN];
                Chunk<DT>::unpack(lg[it], x);
#pragma unroll
                for (int e = 0; e < kN; ++e) zt += exp_weight<DT>(x[e], mt, c, mtc);
            }
        }
        const float mw = wave_max(mt);
        // (mt c was rounded in the exponents above, which at low temperatures is visible in the sum: the difference is
        // taken out again here)
        const double zw = wave_sum(mt > -INFINITY ? (double)(zt * __builtin_amdgcn_exp2f((mt - mw) * c - fmaf(mt, c, -(mt * c)))) : 0.0);
        if (lane == 0) { s_m[s - first][wv] = mw; s_z[s - first][wv] = zw; }
#pragma unroll
        for (int it = 0; it < kSumSteps; ++it) lg[it] = nx[it];
    }
    lds_barrier();
    if (tid < last - first) {
        HalfStat st;
        st.m = s_m[tid][0]; st.arg = -1; st.Z = 0.0;
#pragma unroll
        for (int w = 1; w < kQW; ++w) st.m = fmaxf(st.m, s_m[tid][w]);
#pragma unroll
        for (int w = 0; w < kQW; ++w)
            st.Z += s_m[tid][w] > -INFINITY ? s_z[tid][w] * (double)__builtin_amdgcn_exp2f((s_m[tid][w] - st.m) * c) : 0.0;
        entry[first + tid] = st;
    }
}

// ---- kernel 2: the walk of every request ---------------------------------------------------------
// After s rejected children the distribution at a node is
//     P_s = max(0, p - c_s q) / G_s,   G_s = sum_v max(0, p_v - c_s q_v),   c_0 = 0, c_{s+1} = c_s + G_s
// (substitute P_s into r = max(0, P_s - q) and pull the positive factor 1 / G_s out of the maximum).
// So the walk keeps two numbers per node, (c, G), and every sweep costs the same few operations per
// element whatever the stage.  A stage whose residual has no mass leaves (c, G) as they are, and so does
// every later stage at that node.
// A sweep is bound by these operations (one workgroup has a row of 128 K elements to itself, 9 us and more), so p stays
// unnormalised in it: c and G carry the factor Z, p_v is w_v = 2^((l_v - m) / T * log2(e)).  w_v and with it w_v - c q_v is at
// most 1, so that the cut at 0 is the clamp bit of the multiply-add.  The difference l_v - m comes first: folded into one
// multiply-add with a rounded product of m, that rounding would be a common factor of all w_v that the node's normaliser
// does not have (walk of the step below 33.5 instead of 35.2 us, p off by 3e-7 instead of 7e-8 at T = 1, by 2e-6 instead
// of 2e-7 with logits around 60).
struct WalkScratch {
    float  part[kNSteps][kWave];        // per step: fp32 sums of the 64 groups of 16 lanes (wave * 4 + lane / 16)
    double S[kNSteps];
    double wsum[kNW];
    float  ch_l[64], ch_q[64], ch_u[64];   // per draft node: logit and draft probability (at its parent) of its token, its uniform
    int    ch_x[64];                    // its token
    unsigned long long kids;            // of the node the walk stands on: its children, maximum, arg-max, total of S[]
    float  m;
    int    arg;
    double R;
    int fallback, hit, last_thread;
    int fallback_tot[kNW];              // (start-up only) per-wavefront row counts of the requests before this one
};

template <class DT>
__global__ __launch_bounds__(kNT, 4) void accept_tree_walk_fast_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs,
    const float *__restrict__ uniforms, const int32_t *__restrict__ spec_lens,
    const float *__restrict__ temperature, const int32_t *__restrict__ cu_q,
    const char *__restrict__ stats, int stat_bytes, int V, int total_q, int max_spec_len, int64_t lstride,
    int64_t pstride, int out_stride, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ out_accept_len, int32_t *__restrict__ out_path)
{
    __shared__ WalkScratch sm;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = blockIdx.x;
    const int k = min(max(spec_lens[i], 0), max_spec_len);
    const float T = temperature[i];
    // first row of the request: from the metadata kernel if the caller ran it (large batches), else the rows
    // of the requests before it, added up by the workgroup
    int r0;
    if (cu_q != nullptr) {
        r0 = cu_q[i];
    } else {
        int part = 0;
        for (int j = tid; j < i; j += kNT) part += min(max(spec_lens[j], 0), max_spec_len) + 1;
        part = wave_sum(part);
        if (lane == 0) sm.fallback_tot[wv] = part;
        __syncthreads();
        r0 = 0;
#pragma unroll
        for (int w = 0; w < kNW; ++w) r0 += sm.fallback_tot[w];
    }
    if (r0 < 0 || r0 + k + 1 > total_q) return;                 // inconsistent metadata: leave the request alone
    const float cexp = T == 0.0f ? 0.f : exponent_scale<DT>(T);
    const int nsteps = ceil_div(V / 8, kNT);
    int32_t *o = out_tokens + (int64_t)i * out_stride;
    int32_t *pth = out_path + (int64_t)i * out_stride;

    // lane c of the first wavefront keeps node c's parent and leaves the rest of its record in LDS
    int my_parent = -1;
    if (tid >= 1 && tid <= k) {
        const TreeNodeRec rec = *reinterpret_cast<const TreeNodeRec *>(stats + (int64_t)(r0 + tid) * stat_bytes);
        my_parent = rec.parent;
        sm.ch_x[tid] = rec.x; sm.ch_l[tid] = rec.l; sm.ch_q[tid] = rec.q; sm.ch_u[tid] = rec.u0;
    }

    // state of the node the walk stands on
    const char *lrow = logits, *prow = probs;
    float m = 0.f;

    // max(0, w - c q) at one entry from its logit and draft probability (c = 0: w itself)
    auto residual = [&](float l, float q, float c) -> float {
        return __builtin_amdgcn_fmed3f(fmaf(-c, q, __builtin_amdgcn_exp2f((l - m) * cexp)), 0.f, 1.f);
    };
    // this thread's 8 masses of one step: before any sweep w, afterwards max(0, w - c q)
    auto mass8 = [&](bool in_range, const uint4 &lw, const uint4 &qw, bool swept, float c, float (&rv)[8]) -> float {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) rv[e] = 0.f;
        if (in_range) {
            float x[8];
            unpack8<DT>(lw, x);
            if (!swept) {
#pragma unroll
                for (int e = 0; e < 8; ++e) rv[e] = __builtin_amdgcn_exp2f((x[e] - m) * cexp);
            } else {
                float q[8];
                unpack8<DT>(qw, q);
#pragma unroll
                for (int e = 0; e < 8; ++e) rv[e] = residual(x[e], q[e], c);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += rv[e];
        }
        return acc;
    };
    // one sweep over both rows: S[] and the total of max(0, p - c q)
    auto sweep = [&](float c) -> double {
        for_each_step<true>(lrow, prow, nsteps, V, tid, [&](int s, bool in_range, const uint4 &lw, const uint4 &qw) {
            float acc = 0.f;
            if (in_range) {
                float x[8], q[8];
                unpack8<DT>(lw, x);
                unpack8<DT>(qw, q);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc += residual(x[e], q[e], c);
            }
            acc = row16_sum(acc);
            if ((lane & 15) == 0) sm.part[s][wv * 4 + (lane >> 4)] = acc;
        });
        return finish_sweep(sm.part, sm.S, nsteps, wv, lane);
    };

    int u = 0, depth = 0;
    for (;;) {
        const int r = r0 + u;
        lrow = logits + (int64_t)r * lstride * 2;
        prow = probs + (int64_t)(r - i) * pstride * 2;          // read only if the node has children
        __syncthreads();                                        // everything of the previous node has been read
        // the first wavefront: the children of u (lane c looks at node c), and the node's statistics on one scale
        if (tid < kWave) {
            HalfStat st;
            st.m = -INFINITY; st.arg = -1; st.Z = 0.0;
            if (lane < nsteps) st = reinterpret_cast<const HalfStat *>(stats + (int64_t)r * stat_bytes + sizeof(TreeNodeRec))[lane];
            const unsigned long long kmask = __builtin_amdgcn_ballot_w64(lane > u && lane <= k && my_parent == u);
            const float mx = fmaxf(wave_max(st.m), -3.0e38f);   // (stays finite when no logit is: differences stay defined)
            const double part = st.m > -INFINITY ? st.Z * (double)__builtin_amdgcn_exp2f((st.m - mx) * cexp) : 0.0;
            const double total = wave_sum(part);
            const ArgMax best = wave_argmax(st.arg >= 0 ? ArgMax{st.m, st.arg} : ArgMax{-INFINITY, 0x7fffffff});
            if (lane < kNSteps) sm.S[lane] = part;
            if (lane == 0) {
                sm.kids = kmask; sm.hit = -1; sm.last_thread = -1; sm.fallback = -1;
                sm.m = mx; sm.arg = best.i == 0x7fffffff ? 0 : best.i; sm.R = total;
            }
        }
        __syncthreads();
        m = sm.m;
        const int arg = sm.arg;
        double R = sm.R;                                        // total of S[]
        unsigned long long kids = sm.kids;

        int next = -1, cand = arg;
        if (T == 0.0f) {
            // greedy: the first child that carries the target's arg-max, else stop with the arg-max
            while (kids != 0ull && next < 0) {
                const int c = __builtin_ctzll(kids);
                kids &= kids - 1;
                if (sm.ch_x[c] == arg) next = c;
            }
        } else {
            double cd = 0.0, Gd = R;                            // (c, G) of the current distribution
            float cf = 0.f, invG = (float)(1.0 / R);
            bool swept = false, frozen = false;
            while (kids != 0ull) {
                const int c = __builtin_ctzll(kids);
                kids &= kids - 1;
                {   // every thread evaluates the test from the values fetched on arrival: no exchange needed
                    const float qx = sm.ch_q[c];
                    const float px = residual(sm.ch_l[c], qx, cf) * invG;
                    const bool accepted = (qx > 0.f) ? (sm.ch_u[c] < px / qx) : true;
                    if (accepted) { next = c; break; }
                }
                if (frozen) continue;                           // the residual had no mass before: it has none now
                const double ct = cd + Gd;
                const double Gt = sweep((float)ct);
                if (Gt > 0.0) {
                    cd = ct; Gd = Gt;
                    cf = (float)ct; invG = (float)(1.0 / Gt);
                    R = Gt;
                } else {                                        // P == q everywhere: the state stays; S[] again
                    frozen = true;
                    R = sweep(cf);
                }
                swept = true;
            }
            if (next < 0) {
                // ---- the draw from (S, R): of the last sweep, or of the node's statistics ----------------
                const double tau = (double)uniforms[2 * (int64_t)r + 1] * R;
                // lane s of every wavefront looks at step s: the first whose running total exceeds tau, else
                // (rounding left no crossing) the last with mass
                const double Ss = lane < nsteps ? sm.S[lane] : 0.0, upto = wave_scan_incl(Ss, lane);
                const unsigned long long cross = __ballot(Ss > 0.0 && upto > tau), filled = __ballot(Ss > 0.0);
                const int sstar = cross ? (int)__builtin_ctzll(cross) : (filled ? 63 - (int)__builtin_clzll(filled) : 0);
                const double before = __shfl(upto - Ss, sstar, kWave);
                float rv[8];
                float mine;
                {
                    const int v0 = (sstar * kNT + tid) * 8;
                    uint4 lw = make_uint4(0, 0, 0, 0), qw = make_uint4(0, 0, 0, 0);
                    if (v0 < V) {
                        lw = *reinterpret_cast<const uint4 *>(lrow + (int64_t)v0 * 2);
                        if (swept) qw = *reinterpret_cast<const uint4 *>(prow + (int64_t)v0 * 2);
                    }
                    mine = mass8(v0 < V, lw, qw, swept, cf, rv);
                }
                // scan over the threads of that step
                const double wi = wave_scan_incl((double)mine, lane);
                double we = __shfl_up(wi, 1, kWave);
                if (lane == 0) we = 0.0;
                if (lane == 63) sm.wsum[wv] = wi;
                note_last(&sm.last_thread, mine > 0.f, tid);
                __syncthreads();
                double wp = 0.0;
#pragma unroll
                for (int w = 0; w < kNW; ++w) wp += (w < wv) ? sm.wsum[w] : 0.0;
                const double excl = before + wp + we, incl = before + wp + wi;
                const bool crossing = incl > tau && !(excl > tau);
                const int last_thread = sm.last_thread;
                // the crossing thread, and (in case rounding leaves none) the last thread with mass
                if (crossing || tid == last_thread) {
                    const int v0 = (sstar * kNT + tid) * 8;
                    double cum = excl;
                    int pick = -1, lastpos = -1;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        cum += (double)rv[e];
                        if (rv[e] > 0.f) lastpos = v0 + e;
                        if (pick < 0 && cum > tau && rv[e] > 0.f) pick = v0 + e;
                    }
                    if (crossing) sm.hit = pick >= 0 ? pick : lastpos;
                    else sm.fallback = lastpos;
                }
                __syncthreads();
                cand = sm.hit;
                if (cand < 0) cand = sm.fallback;
                if (cand < 0) cand = arg;
            }
        }
        if (next < 0) {                                         // the walk stops here
            if (tid == 0) {
                o[depth] = cand;
                pth[depth] = -1;
                out_accept_len[i] = depth;
            }
            for (int j = depth + 1 + tid; j < out_stride; j += kNT) { o[j] = -1; pth[j] = -1; }
            return;
        }
        if (tid == 0) { o[depth] = sm.ch_x[next]; pth[depth] = next; }
        ++depth;
        u = next;
    }
}

// Every walk workgroup adds up the rows of the requests before its own: fine for a few thousand requests,
// quadratic beyond; larger batches take the row offsets from the metadata kernel.
bool tree_fast_needs_plan(const adaspec_accept_dims &d) { return d.batch > 2048; }

hipError_t launch_accept_tree_fast(const AcceptArgs &a, const int32_t *parents, int compute_units, int32_t *out_path)
{
    const adaspec_accept_dims &d = a.dims;
    if (d.total_q == 0) return hipSuccess;
    char *stats = a.ws + a.plan.off_tree_stat;
    const int stat_bytes = (int)tree_node_stat_bytes(d.vocab), nsteps = ceil_div(d.vocab / 8, kStepChunks);
    // steps per workgroup: the fewest with which the launch has about kStatsWgsPerCu workgroups per compute unit
    int group = 1;
    while (group < nsteps && (int64_t)d.total_q * ceil_div(nsteps, group) > (int64_t)kStatsWgsPerCu * compute_units) group *= 2;
    const int n_groups = ceil_div(nsteps, group);
    auto launch = [&](auto tag) {
        using DT = decltype(tag);
        hipLaunchKernelGGL((tree_node_stats_kernel<DT>), dim3(d.total_q * n_groups), dim3(kQT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.draft_tokens, parents, a.uniforms, a.spec_lens,
                           a.temperature, d.batch, d.vocab, d.total_draft, d.max_spec_len, n_groups, group,
                           d.logits_row_stride, d.probs_row_stride, stats, stat_bytes);
        hipLaunchKernelGGL((accept_tree_walk_fast_kernel<DT>), dim3(d.batch), dim3(kNT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.uniforms, a.spec_lens, a.temperature,
                           tree_fast_needs_plan(d) ? (const int32_t *)(a.ws + a.plan.off_cu_q) : nullptr, stats, stat_bytes,
                           d.vocab, d.total_q, d.max_spec_len, d.logits_row_stride, d.probs_row_stride, d.out_stride,
                           a.out_tokens, a.out_accept_len, out_path);
    };
    if (d.logits_dtype == ADASPEC_F16) launch(F16{});
    else launch(BF16{});
    return hipGetLastError();
}

}  // namespace adaspec
