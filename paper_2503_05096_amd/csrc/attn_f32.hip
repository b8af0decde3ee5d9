// Matrix-core verification attention for fp32 K/V/Q, head_dim 64 or 128 (v_mfma_f32_16x16x4: fp32 products and sums).
//
// The unit, the schedule and the merge are those of attn_mfma.hip: a workgroup of 4 wavefronts takes (request x KV
// split, kv head, row group); wavefront w streams the 16-token pages w, w + 4, ... and holds the online-softmax state of
// all rows.  With 4-byte elements no operand needs LDS or a transposition:
//   S^T[token][row] = K Q^T      lane (g, m) loads 16 bytes = 4 channels of token m at channel 16 j + 4 g; element e of it
//                                is the A operand of step (j, e), whose four k-slots are the channels 16 j + 4 g + e;
//   O^T[d][row]    += V^T P^T    the accumulator lane (g, n) holds S^T[4g + r][n]: step r takes it as B operand with k-slot
//                                g = token 4 g + r; lane (g, m) loads 16 bytes of V of that token at channel 64 h + 4 m, and
//                                element e is the A operand of output tile (h, e) = channels 64 h + 4 m + e.
// Every load instruction reads whole 64-byte (K) or 256-byte (V) pieces of rows.
//
// Bound: HBM at up to two row tiles per unit (512 matrix cycles per tile against 1800 that 16 KB take to arrive), the
// matrix cores at four; latency for small batches.  Measured on MI355X, 4 requests of 128-512 tokens, 8 heads of 64
// (5.3 MB, a direct call): 5.6 us + 4.2 us for the split-KV combine; the vector kernel with its metadata took 102 + 4.7 +
// 4.6 us.  Error of the output against 64 bits 1.3e-7 to 2.6e-7 (vector kernel: 1.7e-7 to 4.7e-7) over contexts 5-655.
#include "adaspec_internal.h"
#include "attn_mfma_common.h"
#include "device_utils.h"

namespace adaspec {

constexpr int kPage = 16;                   // tokens per block of the stream

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 ldf4(const char *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ f32x4 ldf4_stream(const char *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
}

template <int D, int RT, bool kTree, bool kDirect>
__global__ __launch_bounds__(256, (RT <= 2 ? 2 : 1)) void attn_f32_kernel(
    const char *__restrict__ q, const char *__restrict__ k_pages, const char *__restrict__ v_pages,
    const int32_t *__restrict__ block_table, float *__restrict__ out, const int32_t *__restrict__ header,
    const int32_t *__restrict__ unit_meta, const int32_t *__restrict__ sched,
    const unsigned long long *__restrict__ anc, float *__restrict__ part_ml, float *__restrict__ part_o,
    int Hq, int Hkv, int max_pages_per_req, int max_rows, int n_row_groups, float scale_log2, int cus, DirectArgs direct)
{
    constexpr int kRows = 16 * RT, kJ = D / 16, kH = D / 64, kORow = D + 4;
    constexpr int kQLoads = RT * kJ * 64 / 256;
    constexpr int kState = kRows * kORow;                                  // floats of one wavefront's state
    // merge buffer: one state per wavefront, or (four tiles of 128 channels: too large) one that they add into in turn
    constexpr bool kSlabs = kState * kWaves * 4 <= 96 * 1024;
    __shared__ __attribute__((aligned(16))) float obuf[kSlabs ? kWaves * kState : kState];
    __shared__ __attribute__((aligned(16))) f32x4 q_lds[RT * kJ * 64];     // Q^T operands, MFMA lane order
    __shared__ float s_m[kWaves][kRows], s_l[kWaves][kRows];
    __shared__ unsigned long long s_anc[kTree ? kRows : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n16 = lane & 15;
    const int G = Hq / Hkv;
    constexpr int64_t head_bytes = (int64_t)kPage * D * 4;
    const uint32_t k_lane_off = n16 * (D * 4) + 16 * g, v_lane_off = 4 * g * (D * 4) + 16 * n16;
    f32x4 kreg[kJ], vreg[4][kH];

    const int W = gridDim.x, wg = blockIdx.x;
    const int total_units = kDirect ? 0 : header[0] * Hkv * n_row_groups;
    const int n_rounds = kDirect ? 0 : header[2];
    int round = 0;
    int idx_ahead = kDirect ? 0 : sched_position(0, wg, W, cus, header[1]);     // round 0 needs no table
    auto next_unit = [&](Unit &u) -> bool {
        for (; round < n_rounds; ++round) {
            const int idx = idx_ahead;
            idx_ahead = round + 1 < n_rounds ? sched[(int64_t)(round + 1) * W + wg] : -1;
            if (idx < 0 || idx >= total_units) continue;
            const int rg = idx % n_row_groups;
            u.gkv = (idx / n_row_groups) % Hkv;
            const int32_t *mt = unit_meta + 8 * (int64_t)(idx / (n_row_groups * Hkv));
            u.i = mt[0];
            const int sp = mt[1];
            u.ns = mt[2]; u.L = mt[3]; u.n = mt[4]; u.qrow0 = mt[5]; u.item = mt[6];
            u.rows = u.n * G; u.r0 = rg * kRows;
            if (u.r0 >= u.rows) continue;
            const int slen = split_len_of(u.L, u.ns, kPage);
            u.t0 = sp * slen; u.t1 = min(u.L, u.t0 + slen);
            u.nblk = (u.t1 - u.t0 + kPage - 1) / kPage;
            u.bt_off = (int64_t)u.i * max_pages_per_req;
            ++round;
            return true;
        }
        return false;
    };

    auto page_base = [&](const Unit &u, int bi) -> int64_t {
        const int64_t p = block_table[u.bt_off + (u.t0 >> 4) + bi];
        return (p * Hkv + u.gkv) * head_bytes;
    };
    auto load_k = [&](int64_t b) {
#pragma unroll
        for (int j = 0; j < kJ; ++j) kreg[j] = ldf4_stream(k_pages + b + k_lane_off + 64 * j);
    };
    auto load_v = [&](int64_t b) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < kH; ++h) vreg[r][h] = ldf4_stream(v_pages + b + v_lane_off + r * (D * 4) + 256 * h);
    };
    auto first_loads = [&](const Unit &u) {
        if (wv < u.nblk) {
            const int64_t b = page_base(u, wv);
            load_k(b);
            load_v(b);
        }
    };
    auto load_q = [&](const Unit &u, f32x4 (&qv)[kQLoads]) {
#pragma unroll
        for (int k = 0; k < kQLoads; ++k) {
            const int e = tid + 256 * k;                            // entry (row tile, j, lane)
            const int row = u.r0 + 16 * (e / (kJ * 64)) + n16;
            qv[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row < u.rows)
                qv[k] = ldf4(q + (((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * D) * 4 + 64 * ((e >> 6) % kJ) + 16 * g);
        }
    };
    auto load_anc = [&](const Unit &u) -> unsigned long long {
        const int row = u.r0 + tid;
        return (tid < kRows && row < u.rows) ? anc[u.qrow0 + row / G] : 0ull;
    };

    Unit cur, nxt;
    bool have;
    f32x4 qv[kQLoads];
    unsigned long long av = 0ull;
    if constexpr (kDirect) have = direct_unit(cur, direct, block_table, G, Hkv, n_row_groups, kRows, kPage, max_pages_per_req, wv, lane);
    else have = next_unit(cur);
    if (have) {
        first_loads(cur);
        load_q(cur, qv);
        if constexpr (kTree) av = load_anc(cur);
    }

    while (have) {
        const Unit u = cur;
        const bool have_next = kDirect ? false : next_unit(nxt);
        const int first_masked = u.L - u.n + 1;                    // tokens >= this are hidden from some row
#pragma unroll
        for (int k = 0; k < kQLoads; ++k) q_lds[tid + 256 * k] = qv[k];
        if constexpr (kTree) { if (tid < kRows) s_anc[tid] = av; }
        int pos[RT];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            const int row = u.r0 + 16 * nt + n16;
            pos[nt] = row < u.rows ? (u.L - u.n + row / G) : -1;
        }
        lds_barrier();

        float m[RT], lsum[RT];
        f32x4 o[RT][kH][4];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            m[nt] = kLowestRef; lsum[nt] = 0.f;
#pragma unroll
            for (int h = 0; h < kH; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[nt][h][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

        auto block = [&](int bi, auto next_tag) {
            constexpr bool kNext = decltype(next_tag)::value;
            const int tb = u.t0 + bi * kPage;
            int64_t nb = 0;
            if constexpr (kNext) nb = page_base(u, bi + kWaves);

            // ---- S^T = K Q^T: two chains, so that one product's latency hides under the other's ----------
            f32x4 p[RT];
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll
                for (int j = 0; j < kJ; j += 2) {
                    const f32x4 q0 = q_lds[(nt * kJ + j) * 64 + lane], q1 = q_lds[(nt * kJ + j + 1) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc0 = mfma_f32(kreg[j][e], q0[e], acc0);
                        acc1 = mfma_f32(kreg[j + 1][e], q1[e], acc1);
                    }
                }
                p[nt] = acc0 + acc1;
            }
            if constexpr (kNext) load_k(nb);

            // ---- online softmax (per lane: row n16 of each row tile, 4 of the 16 tokens) ----
            const bool need_mask = (tb + kPage > first_masked) || (tb + kPage > u.t1);
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                if (need_mask) {
                    if constexpr (kTree) {
                        const unsigned long long am = s_anc[16 * nt + n16];
                        const int base = u.L - u.n;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int t = tb + 4 * g + e;
                            const int rel = t - base;
                            const bool vis = t < u.t1 && (rel < 0 ? pos[nt] >= 0 : ((am >> (rel & 63)) & 1ull) != 0);
                            p[nt][e] = vis ? p[nt][e] : -INFINITY;
                        }
                    } else {
                        const int lim = min(pos[nt], u.t1 - 1);
#pragma unroll
                        for (int e = 0; e < 4; ++e) p[nt][e] = (tb + 4 * g + e <= lim) ? p[nt][e] : -INFINITY;
                    }
                }
                const float mx = max_over_row_groups(fmaxf(fmaxf(p[nt][0], p[nt][1]), fmaxf(p[nt][2], p[nt][3])));
                // lazy reference: moves only when the block's maximum exceeds it by more than kLazyLog2
                const float mxs = mx * scale_log2;
                const bool grow = mxs > m[nt] + kLazyLog2;
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(grow) != 0, 0)) {
                    const float m_new = grow ? mxs : m[nt];
                    const float alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
                    m[nt] = m_new;
                    lsum[nt] *= alpha;
#pragma unroll
                    for (int h = 0; h < kH; ++h)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[nt][h][e] *= alpha;
                }
                softmax_weights<4>(p[nt], scale_log2, m[nt], 0.f);
                lsum[nt] += (p[nt][0] + p[nt][1]) + (p[nt][2] + p[nt][3]);
            }

            // ---- O^T += V^T P^T -------------------------------------------------------------
            if (tb + kPage > u.L) {                    // the request's last, partial page
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (tb + 4 * g + r >= u.L) {
#pragma unroll
                        for (int h = 0; h < kH; ++h) vreg[r][h] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int h = 0; h < kH; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int nt = 0; nt < RT; ++nt) o[nt][h][e] = mfma_f32(vreg[r][h][e], p[nt][r], o[nt][h][e]);
            if constexpr (kNext) load_v(nb);
        };

        if (wv < u.nblk) {
            int bi = wv;
            for (; bi + kWaves < u.nblk; bi += kWaves) block(bi, std::true_type{});
            block(bi, std::false_type{});
        }

        // ---- next unit: its first page and Q rows travel while this unit's states are merged
        if (have_next) {
            first_loads(nxt);
            load_q(nxt, qv);
            if constexpr (kTree) av = load_anc(nxt);
        }
        // ---- merge the four wavefronts' states through LDS (as in attn_mfma.hip) ----------
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            lsum[nt] += __shfl_xor(lsum[nt], 16, kWave);
            lsum[nt] += __shfl_xor(lsum[nt], 32, kWave);
            if (g == 0) { s_m[wv][16 * nt + n16] = m[nt]; s_l[wv][16 * nt + n16] = lsum[nt]; }
        }
        auto leave_state = [&](float *buf, float (&sc)[RT], bool add) {
#pragma unroll
            for (int nt = 0; nt < RT; ++nt)
#pragma unroll
                for (int h = 0; h < kH; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // lane (g, n16), register r of tile (h, e): channel 64 h + 16 g + 4 r + e
                        f32x4 *dst = reinterpret_cast<f32x4 *>(buf + (16 * nt + n16) * kORow + 64 * h + 16 * g + 4 * r);
                        f32x4 v = f32x4{o[nt][h][0][r], o[nt][h][1][r], o[nt][h][2][r], o[nt][h][3][r]};
                        if constexpr (!kSlabs) {
                            v *= sc[nt];
                            if (add) v += *dst;
                        }
                        *dst = v;
                    }
        };
        float fsc[RT] = {};
        if constexpr (kSlabs) {
            leave_state(obuf + wv * kState, fsc, false);
            lds_barrier();
        } else {
            lds_barrier();          // s_m complete
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                const int rl = 16 * nt + n16;
                float ms = s_m[0][rl];
#pragma unroll
                for (int w = 1; w < kWaves; ++w) ms = fmaxf(ms, s_m[w][rl]);
                fsc[nt] = __builtin_amdgcn_exp2f(m[nt] - ms);
            }
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                if (wv == w) leave_state(obuf, fsc, w > 0);
                lds_barrier();
            }
        }
        // 256 threads: 16*RT rows x D/4 float4 columns
#pragma unroll
        for (int it = 0; it < kRows * (D / 4) / 256; ++it) {
            const int idx = tid + 256 * it;
            const int rl = idx / (D / 4), c4 = idx % (D / 4);
            const int row = u.r0 + rl;
            if (row >= u.rows) continue;
            float ms = s_m[0][rl], ltot = 0.f;
#pragma unroll
            for (int w = 1; w < kWaves; ++w) ms = fmaxf(ms, s_m[w][rl]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float sc = __builtin_amdgcn_exp2f(s_m[w][rl] - ms);
                ltot += sc * s_l[w][rl];
                if constexpr (kSlabs) acc += sc * *reinterpret_cast<const f32x4 *>(obuf + w * kState + rl * kORow + 4 * c4);
            }
            if constexpr (!kSlabs) acc = *reinterpret_cast<const f32x4 *>(obuf + rl * kORow + 4 * c4);
            if (u.ns == 1) {
                const int64_t obase = ((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * (int64_t)D + 4 * c4;
                *reinterpret_cast<f32x4 *>(out + obase) = acc * (1.0f / ltot);
            } else {
                const int64_t idx_row = ((int64_t)u.item * Hkv + u.gkv) * max_rows + row;
                if (kDirect && attn_merge_fits(D, RT) && direct.flags) {
                    store_state(part_o + idx_row * D + 4 * c4, acc);
                    if (c4 == 0) store_ml(part_ml + idx_row * 2, ms, ltot);
                } else {
                    *reinterpret_cast<f32x4 *>(part_o + idx_row * D + 4 * c4) = acc;
                    if (c4 == 0) {
                        part_ml[idx_row * 2] = ms;
                        part_ml[idx_row * 2 + 1] = ltot;
                    }
                }
            }
        }
        if constexpr (kDirect) {
            if constexpr (attn_merge_fits(D, RT)) {
                if (u.ns > 1 && direct.flags)
                    merge_splits<F32, D, kRows>(direct, u, part_ml, part_o, out, ADASPEC_F32, Hq, Hkv, G, max_rows, tid);
            }
            break;
        }
        lds_barrier();              // the next unit overwrites q_lds, s_m and obuf
        cur = nxt;
        have = have_next;
    }
}

// ---- host side -----------------------------------------------------------------------------------------------
template <typename F>
static void with_f32_instance(const AttnArgs &a, F &&f)
{
    const int rt = attn_row_tiles(a.plan.max_rows);
    auto with_mode = [&](auto d_tag, auto rt_tag) {
        if (a.direct) f(d_tag, rt_tag, std::false_type{}, std::true_type{});
        else if (a.parents) f(d_tag, rt_tag, std::true_type{}, std::false_type{});
        else f(d_tag, rt_tag, std::false_type{}, std::false_type{});
    };
    auto with_rt = [&](auto d_tag) {
        if (rt == 1) with_mode(d_tag, std::integral_constant<int, 1>{});
        else if (rt == 2) with_mode(d_tag, std::integral_constant<int, 2>{});
        else with_mode(d_tag, std::integral_constant<int, 4>{});
    };
    if (a.dims.head_dim == 64) with_rt(std::integral_constant<int, 64>{});
    else with_rt(std::integral_constant<int, 128>{});
}

template <int D, int RT, bool kTree, bool kDirect>
static int attn_f32_slots(int cus)
{
    static int slots = 0;
    if (slots == 0) {
        int per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_f32_kernel<D, RT, kTree, kDirect>, 256, 0) != hipSuccess)
            per_cu = 1;
        const int n = cus * (per_cu > 0 ? per_cu : 1);
        slots = n < kMaxSchedW ? n : kMaxSchedW;
    }
    return slots;
}

int attn_f32_grid_slots(const AttnArgs &a, int cus)
{
    int slots = 1;
    with_f32_instance(a, [&](auto d, auto rt, auto tree, auto direct) {
        slots = attn_f32_slots<decltype(d)::value, decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>(cus);
    });
    return slots;
}

hipError_t launch_attn_f32(const AttnArgs &a)
{
    const AttnPlan &p = a.plan;
    const adaspec_attn_dims &d = a.dims;
    if (a.sched_w <= 0) return hipSuccess;                          // no work item can exist
    with_f32_instance(a, [&](auto dd, auto rt, auto tree, auto direct) {
        hipLaunchKernelGGL((attn_f32_kernel<decltype(dd)::value, decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>),
                           dim3(a.sched_w), dim3(256), 0, a.stream, (const char *)a.q, (const char *)a.k_pages,
                           (const char *)a.v_pages, a.block_table, (float *)a.out, (const int32_t *)(a.ws + p.off_header),
                           (const int32_t *)(a.ws + p.off_unit_meta), (const int32_t *)(a.ws + p.off_sched),
                           (const unsigned long long *)(a.ws + p.off_anc), (float *)(a.ws + p.off_part_ml),
                           (float *)(a.ws + p.off_part_o), d.n_q_heads, d.n_kv_heads, d.max_pages_per_req, p.max_rows,
                           a.n_row_groups, a.scale_log2, a.sched_cus, direct_args(a));
    });
    return hipGetLastError();
}

}  // namespace adaspec
