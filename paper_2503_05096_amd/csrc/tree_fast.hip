// Tree acceptance for 16-bit logits and draft probabilities of one type, V % 8 == 0,
// V <= 524288 (the shapes of the streaming chain kernel), in two kernels:
//
//   1. node statistics: every node's logits row read once, in steps of 8192 elements shared out to small
//      workgroups: per step the maximum and, for a sampled request, the normaliser relative to it (greedy:
//      the arg-max); and per draft node what its accept test needs (its token, the token's logit and draft
//      probability at the parent, the uniform) beside its parent;
//   2. the walk, a few workgroups per request, which share its rows: from the root, at every node it reaches it tests
//      the children in turn and, after each rejection, sums the next residual mass over the node's logits and
//      draft-probability rows; where the walk stops it draws the token.  It writes the request's outputs itself.
// Nodes the walk does not reach cost their statistics only, and a node where the first child
// is accepted never reads its draft-probability row.
//
// Same procedure as the portable node kernel (tree.hip):
//   stage 0: P = softmax(logits / T); after each rejected child r = max(0, P - q), P = r / sum(r),
// evaluated in its closed form (see kernel 2).
// Element (s * 1024 + t) * 8 + e of a row belongs to step s, thread t.  The draw needs no sweep of its own: the part, the
// step and the wavefront where the prefix crosses come from the sums; a scan over that wavefront finds the lane, which
// picks the element.  A test is arithmetic on values already on chip.
//
// Bound: HBM for the statistics; the walk is a chain of sweeps, each the first read of a node's two rows or, on the rows
// in registers, an exchange between the workgroups (part_exchange.h).  With one workgroup per request a sweep was vector
// arithmetic of one compute unit (9.6 us at V = 128256) and three quarters of the chip idle.  MI355X, 64 requests, 288 nodes,
// trees of width 3: statistics 16.5 us (one 1024-thread workgroup per node: 23.7), walk
// 37.0 -> 15.4 us, whole call 56.1 -> 33.2; 8 requests 33.3 -> 17.0, 16 of V = 262144 74.7 -> 24.7, 8 of V = 524288 106 -> 23.  Many
// requests keep one workgroup each (launch_accept_tree_fast has the line).
#include "adaspec_internal.h"
#include "device_utils.h"
#include "part_exchange.h"
#include "row_parts.h"
#include "row_stream.h"

namespace adaspec {

__device__ __forceinline__ int sane_parent_f(int p, int j) { return j == 0 ? -1 : min(max(p, 0), j - 1); }

// What kernel 1 leaves per node: a record for the accept test (nodes j >= 1); per step of 8192 elements the normaliser (or
// the arg-max, greedy requests) and the maximum of its elements; then the words in which the workgroups of the walk exchange
// their parts of a sweep's mass, cleared: sweep s of a request uses those of its node s (every sweep follows the rejection of
// another child, so there are never more of them).
struct TreeNodeRec { int parent, x; float l, q, u0; int pad[3]; };
constexpr int kStatsWgsPerCu = 6;                   // statistics: workgroups per compute unit the launch aims for (all resident)
constexpr int kStepChunks = kNT;                    // 16-byte chunks per step
static_assert(kStepChunks == kSumSteps * kQT, "a step is four chunks per thread of the statistics kernel");
union StepNorm { double Z; long long arg; };
__host__ __device__ __forceinline__ int node_max_at(int nsteps) { return (int)sizeof(TreeNodeRec) + nsteps * 8; }
__host__ __device__ __forceinline__ int node_words_at(int nsteps) { return node_max_at(nsteps) + (nsteps + 1) / 2 * 8; }
// (528 bytes is what a node took when the workspace rules were laid down, and 16 per step what larger ones did: both kept)
size_t tree_node_stat_bytes(int vocab)
{
    const size_t need = sizeof(TreeNodeRec) + (size_t)ceil_div(vocab / 8, kStepChunks) * 16;
    return need > kTreeNodeStatMin ? need : kTreeNodeStatMin;
}

// ---- kernel 1: statistics of every node ---------------------------------------------------------
// workgroup = (node, group of steps); the loads of the next step are under way while one is summed.
template <class DT>
__global__ __launch_bounds__(kQT, 6) void tree_node_stats_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs, const int32_t *__restrict__ draft_tokens,
    const int32_t *__restrict__ parents, const float *__restrict__ uniforms, const int32_t *__restrict__ spec_lens,
    const float *__restrict__ temperature, int B, int V, int total_draft, int max_spec_len, int n_groups, int group_steps,
    int64_t lstride, int64_t pstride, char *__restrict__ stats, int stat_bytes, int n_words)
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
    StepNorm *norm = reinterpret_cast<StepNorm *>(node + sizeof(TreeNodeRec));
    float *top = reinterpret_cast<float *>(node + node_max_at(nsteps));
    if (h == 0 && tid < n_words) reinterpret_cast<unsigned long long *>(node + node_words_at(nsteps))[tid] = kNoWord;
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
            top[first + tid] = tid == 0 ? best.v : -INFINITY;
            norm[first + tid].arg = tid == 0 && best.i < V ? best.i : -1;
        }
        return;
    }
    const float c = exponent_scale<DT>(T);
    // (the same for the workgroup: a scalar register, the vector ones are full)
    const float lowest = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(lowest_ref<DT>(c))));
    for (int s = first; s < last; ++s) {
        uint4 nx[kSumSteps];
        load_step(s + 1 < last ? s + 1 : nsteps, nx);            // (another group's step: nothing)
#pragma unroll
        for (int it = 0; it < kSumSteps; ++it) Chunk<DT>::blank(lg[it], s * kStepChunks + it * kQT + tid >= row_chunks);
        // every thread sums against its own maximum; the pairs are merged over the wavefront here, over the
        // wavefronts at the end
        const float mt = thread_max<DT, kSumSteps>(lg);
        float zt = 0.f;
        if (mt > lowest) {
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
        const double zw = wave_sum(mt > lowest ? (double)(zt * __builtin_amdgcn_exp2f((mt - mw) * c - fmaf(mt, c, -(mt * c)))) : 0.0);
        if (lane == 0) { s_m[s - first][wv] = mw; s_z[s - first][wv] = zw; }
#pragma unroll
        for (int it = 0; it < kSumSteps; ++it) lg[it] = nx[it];
    }
    lds_barrier();
    if (tid < last - first) {
        float m = s_m[tid][0];
        double Z = 0.0;
#pragma unroll
        for (int w = 1; w < kQW; ++w) m = fmaxf(m, s_m[tid][w]);
#pragma unroll
        for (int w = 0; w < kQW; ++w)
            Z += s_m[tid][w] > -INFINITY ? s_z[tid][w] * (double)__builtin_amdgcn_exp2f((s_m[tid][w] - m) * c) : 0.0;
        top[first + tid] = m;
        norm[first + tid].Z = Z;
    }
}

// ---- kernel 2: the walk of every request ---------------------------------------------------------
// After s rejected children the distribution at a node is
//     P_s = max(0, p - c_s q) / G_s,   G_s = sum_v max(0, p_v - c_s q_v),   c_0 = 0, c_{s+1} = c_s + G_s
// (substitute P_s into r = max(0, P_s - q) and pull the positive factor 1 / G_s out of the maximum).
// So the walk keeps two numbers per node, (c, G), and every sweep costs the same few operations per
// element whatever the stage.  A stage whose residual has no mass leaves (c, G) as they are, and so does
// every later stage at that node.
// p stays unnormalised: c and G carry the factor Z, p_v is w_v = 2^((l_v - m) / T * log2(e)).  w_v and with it w_v - c q_v is at
// most 1, so that the cut at 0 is the clamp bit of the multiply-add.  The difference l_v - m comes first: folded into one
// multiply-add with a rounded product of m, that rounding would be a common factor of all w_v that the node's normaliser
// does not have (p off by 3e-7 instead of 7e-8 at T = 1, by 2e-6 instead of 2e-7 with logits around 60).
//
// Workgroup (request, part): all parts walk the same way, as every decision is made from the same numbers; part h owns
// the steps h * part_steps, ... of every row (up to kWalkSteps).  Its w and q of the node the walk stands on are in registers
// from the node's first rejection on: what a sweep takes then is a few operations per element and the exchange of
// the parts' sums.  The part that holds the drawn token writes it (part 0 if there was no sweep), part 0 everything else.
constexpr int kWalkSteps = 4;                          // steps of a part at most
static_assert(kWalkSteps * kNW == kWave, "a lane per (step, wavefront) pair of a part");
struct WalkScratch {
    double S[64][kNSteps];                 // per node and step: mass before any sweep
    double R[64];                          // per node: total of S[node], its inverse, maximum, arg-max, the uniform of a draw there
    float  inv[64], m[64], u1[64];
    int    arg[64];
    float  ch_l[64], ch_q[64], ch_u[64];   // per draft node: logit and draft probability (at its parent) of its token, its uniform
    int    ch_x[64], parent[64];           // its token, its parent
    float4 quad[kWave];                    // this part per (step, wavefront): sums of the four rows of 16 lanes
    double pair[2][kWave];                 // their totals, and per part the mass: of the node's last sweep with mass, and of the
    double part[2][kWave];                 // ... one under way
    double G;                              // total of a sweep, its inverse, parts whose mass nobody has yet
    float  invG;
    unsigned long long missing;
    int star, pair_at;                     // the draw: part (or step) and pair it falls on, running totals in front of them
    double before[2];
    int rows[kNW];                         // (start-up) per wavefront: rows of the requests before this one
};

template <class DT, int STEPS>
__global__ __launch_bounds__(kNT, STEPS == 1 ? 8 : 4) void accept_tree_walk_shared_kernel(
    const char *__restrict__ logits, const char *__restrict__ probs,
    const float *__restrict__ uniforms, const int32_t *__restrict__ spec_lens,
    const float *__restrict__ temperature, const int32_t *__restrict__ cu_q,
    char *__restrict__ stats, int stat_bytes, int n_parts, int part_steps, int V, int total_q, int max_spec_len,
    int64_t lstride, int64_t pstride, int out_stride, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ out_accept_len, int32_t *__restrict__ out_path)
{
    __shared__ WalkScratch sm;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = blockIdx.x / n_parts, h = blockIdx.x % n_parts;
    const int k = min(max(spec_lens[i], 0), max_spec_len);
    const float T = temperature[i];
    if (h > 0 && (T == 0.0f || k == 0)) return;                 // no sweeps, nothing to share
    // first row of the request: from the metadata kernel if the caller ran it (large batches), else the rows
    // of the requests before it, added up by the workgroup
    int r0;
    if (cu_q != nullptr) {
        r0 = cu_q[i];
    } else {
        int part = 0;
        for (int j = tid; j < i; j += kNT) part += min(max(spec_lens[j], 0), max_spec_len) + 1;
        part = wave_sum(part);
        if (lane == 0) sm.rows[wv] = part;
        lds_barrier();
        r0 = 0;
#pragma unroll
        for (int w = 0; w < kNW; ++w) r0 += sm.rows[w];
        r0 = __builtin_amdgcn_readfirstlane(r0);
    }
    if (r0 < 0 || r0 + k + 1 > total_q) return;                 // inconsistent metadata: leave the request alone
    const float cexp = T == 0.0f ? 0.f : exponent_scale<DT>(T);
    const int row_chunks = V / 8, nsteps = ceil_div(row_chunks, kNT);
    char *nodes = stats + (int64_t)r0 * stat_bytes;             // of this request
    int32_t *o = out_tokens + (int64_t)i * out_stride;
    int32_t *pth = out_path + (int64_t)i * out_stride;

    // What decisions are made from is computed by one wavefront and left in LDS: a value that sixteen wavefronts work out for
    // themselves takes sixteen times the instructions.  Here: the nodes' records, and every node's statistics on one
    // scale (a node per wavefront).
    if (wv == 0) {
        if (lane <= k) sm.u1[lane] = uniforms[2 * (int64_t)(r0 + lane) + 1];
        int up = -1;
        if (lane >= 1 && lane <= k) {
            const TreeNodeRec rec = *reinterpret_cast<const TreeNodeRec *>(nodes + (int64_t)lane * stat_bytes);
            up = rec.parent;
            sm.ch_x[lane] = rec.x; sm.ch_l[lane] = rec.l; sm.ch_q[lane] = rec.q; sm.ch_u[lane] = rec.u0;
        }
        sm.parent[lane] = up;
    }
    for (int n = wv; n <= k; n += kNW) {
        const char *node = nodes + (int64_t)n * stat_bytes;
        float top = -INFINITY;
        StepNorm norm;
        norm.Z = 0.0;
        if (lane < nsteps) {
            top = reinterpret_cast<const float *>(node + node_max_at(nsteps))[lane];
            norm = reinterpret_cast<const StepNorm *>(node + sizeof(TreeNodeRec))[lane];
        }
        const float mx = fmaxf(wave_max(top), -3.0e38f);        // (stays finite when no logit is: differences stay defined)
        if (T == 0.0f) {
            const ArgMax best = wave_argmax(lane < nsteps && norm.arg >= 0 ? ArgMax{top, (int)norm.arg} : ArgMax{-INFINITY, 0x7fffffff});
            if (lane == 0) sm.arg[n] = best.i == 0x7fffffff ? 0 : best.i;
        } else {
            const double mass = top > -INFINITY ? norm.Z * (double)__builtin_amdgcn_exp2f((top - mx) * cexp) : 0.0;
            const double total = wave_sum(mass);
            sm.S[n][lane] = mass;
            if (lane == 0) { sm.m[n] = mx; sm.arg[n] = 0; sm.R[n] = total; sm.inv[n] = (float)(1.0 / total); }
        }
    }
    lds_barrier();
    const int my_parent = sm.parent[lane];

    int sweeps = 0, tot = 0;                                    // sweeps so far; sm.part[tot] is the last one with mass
    unsigned long long late = 0ull;                             // parts that were not there in time once
    int u = 0, depth = 0;
    for (;;) {
        const int r = r0 + u, arg = sm.arg[u];
        const float m = sm.m[u];

        // ---- this workgroup's part of the rows of the node the walk stands on --------------------------------------
        float w[STEPS][8];                                     // unnormalised p
        uint4 qw[STEPS];                                       // q, packed
        int held = -1;                                              // part whose values those are
        // (initialised: nothing of the node before is carried along in registers)
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {
            qw[it] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 8; ++e) w[it][e] = 0.f;
        }
        // (c = 0: w itself)
        auto residual = [&](float p, float q, float c) -> float { return __builtin_amdgcn_fmed3f(fmaf(-c, q, p), 0.f, 1.f); };
        auto load_part = [&](int part) {
            const int first = part * part_steps * kNT;              // chunk
            const int bytes = max(0, min(row_chunks - first, part_steps * kNT)) * 16;
            const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(logits) + (int64_t)r * lstride * 2 + (int64_t)first * 16, 0, bytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(probs) + (int64_t)(r - i) * pstride * 2 + (int64_t)first * 16, 0, bytes, 0x00020000);
            uint4 lw[STEPS];
#pragma unroll
            for (int it = 0; it < STEPS; ++it) {               // (past the row: zeros, no traffic)
                if (STEPS > 1 && it >= part_steps) break;
                lw[it] = part_load16<kAuxDefault>(rl, (uint32_t)tid * 16u, it * (kNT * 16));
                qw[it] = part_load16<kAuxDefault>(rq, (uint32_t)tid * 16u, it * (kNT * 16));
            }
#pragma unroll
            for (int it = 0; it < STEPS; ++it) {
                if (STEPS > 1 && it >= part_steps) break;
                Chunk<DT>::blank(lw[it], (it * kNT + tid) * 16 >= bytes);
                unpack8<DT>(lw[it], w[it]);
#pragma unroll
                for (int e = 0; e < 8; ++e) w[it][e] = __builtin_amdgcn_exp2f((w[it][e] - m) * cexp);
                __builtin_amdgcn_sched_barrier(0);                  // (one step at a time: registers)
            }
            held = part;
        };
        auto step_mass = [&](int it, float c) -> float {            // this thread's mass of a step
            float q[8], acc = 0.f;
            keep_packed(qw[it]);                                    // (unpacked for good they would not fit the registers)
            unpack8<DT>(qw[it], q);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += residual(w[it][e], q[e], c);
            return acc;
        };

        // One sweep with the factor c: every part's mass in sm.part[tot ^ 1], the total returned.  Own part first; then,
        // if the others' masses do not come, theirs as well, and the own one again, so that registers and sm.pair end up with it.
        auto sweep = [&](float c) -> double {
            unsigned long long *words = reinterpret_cast<unsigned long long *>(nodes + (int64_t)(++sweeps) * stat_bytes + node_words_at(nsteps));
            double *part = sm.part[tot ^ 1];
            const unsigned long long all = n_parts < kWave ? (1ull << n_parts) - 1ull : ~0ull;
            unsigned long long known = 0ull;
            int target = h;
            for (;;) {
                if (held != target) load_part(target);
#pragma unroll
                for (int it = 0; it < STEPS; ++it) {
                    const float t = STEPS == 1 || it < part_steps ? row16_sum(step_mass(it, c)) : 0.f;
                    if ((lane & 15) == 0) reinterpret_cast<float *>(&sm.quad[it * kNW + wv])[lane >> 4] = t;
                    __builtin_amdgcn_sched_barrier(0);
                }
                lds_barrier();
                if (wv == 0) {
                    double mine = 0.0;
                    if (lane < STEPS * kNW) {
                        const float4 f = sm.quad[lane];
                        mine = ((double)f.x + (double)f.y) + ((double)f.z + (double)f.w);
                    }
                    sm.pair[tot ^ 1][lane] = mine;
                    const double mass = wave_sum(mine);
                    unsigned long long missing = 0ull;
                    if (lane == 0) part[target] = mass;
                    if (known == 0ull && n_parts > 1) {         // the own part: the others may be there, or come
                        if (lane == 0) publish_u64(words + h, word_of(mass));
                        const bool other = lane < n_parts && lane != h, waited = other && !((late >> lane) & 1ull);
                        unsigned long long got = take_words(words + lane, waited);
                        if (other && !waited) got = fetch_u64(words + lane);
                        if (other && got != kNoWord) part[lane] = double_of(got);
                        missing = __ballot(other && got == kNoWord);
                    }
                    const double G = wave_sum(lane < n_parts ? part[lane] : 0.0);
                    if (lane == 0) { sm.missing = missing; sm.G = G; sm.invG = (float)(1.0 / G); }
                }
                lds_barrier();
                if (known == 0ull) {
                    const unsigned long long missing = sm.missing;
                    if (missing == 0ull) break;
                    late |= missing;
                    known = all & ~missing;                     // (the own part among them)
                } else if (target == h) {
                    break;
                } else {
                    known |= 1ull << target;
                }
                target = all & ~known ? (int)__builtin_ctzll(all & ~known) : h;
                lds_barrier();                                  // (what wavefront 0 left has been read)
            }
            return sm.G;
        };

        // the children of u (lane c looks at node c)
        unsigned long long kids = __builtin_amdgcn_ballot_w64(lane > u && lane <= k && my_parent == u);
        int next = -1;
        double cd = 0.0, Gd = 0.0;                              // (c, G) of the current distribution
        float cf = 0.f;
        bool swept = false;
        if (T == 0.0f) {
            // greedy: the first child that carries the target's arg-max, else stop with the arg-max
            while (kids != 0ull && next < 0) {
                const int c = __builtin_ctzll(kids);
                kids &= kids - 1;
                if (sm.ch_x[c] == arg) next = c;
            }
        } else {
            Gd = sm.R[u];
            float invG = sm.inv[u];
            bool frozen = false;
            while (kids != 0ull) {
                const int c = __builtin_ctzll(kids);
                kids &= kids - 1;
                {   // every thread evaluates the test from the values fetched on arrival: no exchange needed
                    const float qx = sm.ch_q[c];
                    const float px = residual(__builtin_amdgcn_exp2f((sm.ch_l[c] - m) * cexp), qx, cf) * invG;
                    const bool accepted = (qx > 0.f) ? (sm.ch_u[c] < px / qx) : true;
                    if (__builtin_amdgcn_readfirstlane((int)accepted)) { next = c; break; }
                }
                if (frozen) continue;                           // the residual had no mass before: it has none now
                const double ct = cd + Gd;
                const double Gt = sweep((float)ct);
                if (Gt > 0.0) {
                    cd = ct; Gd = Gt;
                    cf = (float)ct; invG = sm.invG;
                    tot ^= 1;
                    swept = true;
                } else {                                        // P == q everywhere: the state stays, with its masses
                    frozen = true;
                }
            }
        }
        if (next >= 0) {
            if (h == 0 && tid == 0) { o[depth] = sm.ch_x[next]; pth[depth] = next; }
            ++depth;
            u = next;
            continue;
        }
        // ---- the walk stops here ------------------------------------------------------------------------------
        if (h == 0) {
            if (tid == 0) {
                if (T == 0.0f) o[depth] = arg;
                pth[depth] = -1;
                out_accept_len[i] = depth;
            }
            for (int j = depth + 1 + tid; j < out_stride; j += kNT) { o[j] = -1; pth[j] = -1; }
        }
        if (T == 0.0f) return;
        // ---- the draw: of the last sweep's masses, or of the node's statistics ---------------------------------
        // Lane p of wavefront 0 looks at part p (no sweep: at step p): the first whose running total exceeds tau, else
        // (rounding left no crossing) the last with mass; then likewise at the (step, wavefront) pairs of the part
        const double tau = (double)sm.u1[u] * Gd;
        if (wv == 0) {
            int at = -1;
            double ahead, ahead2 = 0.0;
            const int star = max(find_piece(swept ? (lane < n_parts ? sm.part[tot][lane] : 0.0) : sm.S[u][lane], 0.0, tau, lane, ahead), 0);
            if (swept && star == h) at = find_piece(sm.pair[tot][lane], ahead, tau, lane, ahead2);
            if (lane == 0) { sm.star = star; sm.pair_at = at; sm.before[0] = ahead; sm.before[1] = ahead2; }
        }
        lds_barrier();
        const int star = sm.star;
        if ((swept ? star : 0) != h) return;                    // another part holds the token, or part 0 draws it
        int step = star;                                        // no sweep: the step is known, its elements are loaded
        float rv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (!swept) {
            const int v0 = (star * kNT + tid) * 8;
            if (v0 < V) {
                const uint4 lw = *reinterpret_cast<const uint4 *>(logits + ((int64_t)r * lstride + v0) * 2);
                unpack8<DT>(lw, rv);
#pragma unroll
                for (int e = 0; e < 8; ++e) rv[e] = __builtin_amdgcn_exp2f((rv[e] - m) * cexp);
            }
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += rv[e];
            const double t = wave_sum((double)acc);
            if (lane == 0) sm.pair[tot][wv] = t;
            lds_barrier();
            if (wv == 0) {
                double ahead2;
                const int at = find_piece(lane < kNW ? sm.pair[tot][lane] : 0.0, sm.before[0], tau, lane, ahead2);
                if (lane == 0) { sm.pair_at = at; sm.before[1] = ahead2; }
            }
            lds_barrier();
        }
        const int pair = sm.pair_at;
        if (pair < 0) {                                         // no mass (non-finite input): stay defined
            if (tid == 0) o[depth] = arg;
            return;
        }
        if (pair % kNW != wv) return;
        if (swept) {
            step = h * part_steps + pair / kNW;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (s != pair / kNW) continue;
                float q[8];
                unpack8<DT>(qw[s], q);
#pragma unroll
                for (int e = 0; e < 8; ++e) rv[e] = residual(w[s][e], q[e], cf);
            }
        }
        // the lane, then its element
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += rv[e];
        const double mine = (double)acc, lup = sm.before[1] + wave_scan_incl(mine, lane);
        const unsigned long long lcross = __ballot(mine > 0.0 && lup > tau), lfilled = __ballot(mine > 0.0);
        const int owner = lcross ? (int)__builtin_ctzll(lcross) : 63 - (int)__builtin_clzll(lfilled);   // (the pair has mass)
        if (lane == owner) o[depth] = (step * kNT + tid) * 8 + pick_element<8>(rv, lup - mine, 1.0, tau);
        return;
    }
}

// ---- kernel 2 for many requests: a workgroup per request ---------------------------------------------
// The rows of a node are swept step by step, from memory every time, and p is worked out anew: nothing is kept in registers, so
// that a compute unit is done with its request in one go where it would have several parts in turn.
struct WholeScratch {
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
    __shared__ WholeScratch sm;
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
            const char *node = stats + (int64_t)r * stat_bytes;
            float top = -INFINITY;
            StepNorm norm;
            norm.Z = 0.0;
            if (lane < nsteps) {
                top = reinterpret_cast<const float *>(node + node_max_at(nsteps))[lane];
                norm = reinterpret_cast<const StepNorm *>(node + sizeof(TreeNodeRec))[lane];
            }
            const unsigned long long kmask = __builtin_amdgcn_ballot_w64(lane > u && lane <= k && my_parent == u);
            const float mx = fmaxf(wave_max(top), -3.0e38f);   // (stays finite when no logit is: differences stay defined)
            const double part = T != 0.0f && top > -INFINITY ? norm.Z * (double)__builtin_amdgcn_exp2f((top - mx) * cexp) : 0.0;
            const double total = wave_sum(part);
            const ArgMax best = wave_argmax(T == 0.0f && lane < nsteps && norm.arg >= 0 ? ArgMax{top, (int)norm.arg} : ArgMax{-INFINITY, 0x7fffffff});
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
    // Walk, shared: parts as short as leave every part a compute unit of its own (and its words room behind the node's
    // statistics).  A compute unit holds one part at a time; where several take turns on it, every turn costs about 13 us (the
    // dependent accesses from the lengths to the first sweep, and the draw), and what the shared form saves is 0.6 us per step
    // and sweep, of which the longest chain has up to three.  One workgroup per request / shared, whole call, trees of width 3,
    // V = 128256: 64 of 1-6 drafts 56.1 / 33.2 us, 128 74.0 / 58.9, 155 of 0-2 46.4 / 41.2, 192 of 1-6 90.2 / 82.6, 256 105 / 107,
    // 180 of 0-1 35.4 / 39.8, 233 40.0 / 48.9; V = 50272, 256 of 0-1 24.5 / 29.8, of 0-3 37.5 / 38.2; V = 262144, 64 of 0-3 74.8 / 39.1;
    // V = 8000, 256 of 1-6 21.4 / 19.6, 1024 of 0-3 48 / 51.  Where all requests are greedy nothing is shared, and the further parts only
    // start and leave: 64 of V = 128256 21.2 / 20.8, of 262144, whose parts wait, 38.6 / 41.9 (sampled 100 / 60), one request 7.4 / 7.9; a third
    // greedy, 200 of 1-6 (near the line) 74.3 / 77.6 (all sampled 91.7 / 86.3).
    // Beside another stream's matrix products, which leave no room for a 1024-thread workgroup with its registers full, every part waits for
    // a compute unit: 64 of 1-6 drafts 140 / 222 us while 4096^3 products run.
    const int room = (stat_bytes - node_words_at(nsteps)) / 8;
    int part_steps = 1;
    while (part_steps < kWalkSteps && ((int64_t)d.batch * ceil_div(nsteps, part_steps) > compute_units || ceil_div(nsteps, part_steps) > room))
        part_steps *= 2;
    const int n_parts = ceil_div(nsteps, part_steps);
    const int64_t waiting = (int64_t)d.batch * n_parts - compute_units;
    const bool shared = waiting <= 0 || 22 * waiting <= (int64_t)nsteps * (d.max_spec_len < 3 ? d.max_spec_len : 3) * compute_units;
    auto launch = [&](auto tag) {
        using DT = decltype(tag);
        hipLaunchKernelGGL((tree_node_stats_kernel<DT>), dim3(d.total_q * n_groups), dim3(kQT), 0, a.stream,
                           (const char *)a.logits, (const char *)a.probs, a.draft_tokens, parents, a.uniforms, a.spec_lens,
                           a.temperature, d.batch, d.vocab, d.total_draft, d.max_spec_len, n_groups, group,
                           d.logits_row_stride, d.probs_row_stride, stats, stat_bytes, n_parts);
        const int32_t *cu_q = tree_fast_needs_plan(d) ? (const int32_t *)(a.ws + a.plan.off_cu_q) : nullptr;
        if (shared) {
            auto walk = part_steps == 1 ? accept_tree_walk_shared_kernel<DT, 1> : accept_tree_walk_shared_kernel<DT, kWalkSteps>;
            hipLaunchKernelGGL(walk, dim3(d.batch * n_parts), dim3(kNT), 0, a.stream, (const char *)a.logits,
                               (const char *)a.probs, a.uniforms, a.spec_lens, a.temperature, cu_q, stats, stat_bytes, n_parts,
                               part_steps, d.vocab, d.total_q, d.max_spec_len, d.logits_row_stride, d.probs_row_stride,
                               d.out_stride, a.out_tokens, a.out_accept_len, out_path);
        } else {
            hipLaunchKernelGGL((accept_tree_walk_fast_kernel<DT>), dim3(d.batch), dim3(kNT), 0, a.stream,
                               (const char *)a.logits, (const char *)a.probs, a.uniforms, a.spec_lens, a.temperature, cu_q, stats,
                               stat_bytes, d.vocab, d.total_q, d.max_spec_len, d.logits_row_stride, d.probs_row_stride,
                               d.out_stride, a.out_tokens, a.out_accept_len, out_path);
        }
    };
    if (d.logits_dtype == ADASPEC_F16) launch(F16{});
    else launch(BF16{});
    return hipGetLastError();
}

}  // namespace adaspec
