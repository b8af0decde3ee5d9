// Matrix-core verification attention for head_dim 64: 16-bit K/V/Q, any number of query rows per kv head.
//
// Same scheme as attn_mfma.hip (a workgroup of 4 wavefronts takes one unit = (request x KV split, kv head, row
// group); wavefront w streams token blocks w, w + 4, ...; S^T = K Q^T and O^T += V^T P^T in accumulator layouts that
// need no shuffle; the four states are merged through LDS), re-cut for 64-wide heads:
//
//   * a block is 64 tokens (four pages), so that a wavefront keeps the same 16 KB of K and V in flight as with
//     32 tokens of 128 channels; the V^T tile has the same 512 units (two 32-token halves x 64 channels);
//   * the output state is 16 registers per row tile (32 at head_dim 128), so up to FOUR tiles fit one wavefront and
//     no row-split form is needed;
//   * softmax weights reach the matrix core unrounded for all practical purposes: three bf16 pieces (24 bits), or two
//     f16 pieces (22 bits) of weights scaled by 2^7 (at most 2^15, and the pieces stay clear of f16's subnormals).
//     These shapes ran with fp32 weights on the vector kernel before; the matrix core has the room (about a tenth of
//     its time per row tile).
//
// Bound: HBM. Measured on MI355X, 64 requests, 32/8 heads, contexts 256-4096, bf16 (287 MB): main kernel 52 us = 5.5 TB/s,
// whole call 65 us with the metadata (7 us) and the split-KV combine (5 us); the vector kernel took 1024 us. Error of the
// fp32 accumulator against 64 bits 1.2e-7 to 2.7e-7 (vector kernel: 1.4e-7 to 4.1e-7) over contexts 5-5656.
#include "adaspec_internal.h"
#include "attn_mfma_common.h"
#include "device_utils.h"

namespace adaspec {

constexpr int kD64 = 64;
constexpr int kBlk64 = kAttnD64Block;       // tokens per block (four pages)
constexpr int kORow64 = kD64 + 4;           // floats per row of the merge buffer (padded: conflict-free b128)

// softmax weights as a sum of 16-bit matrix operands; kShiftLog2: the weights are kept 2^kShiftLog2 larger
template <class T> struct WeightSplit;
template <> struct WeightSplit<BF16> {
    static constexpr int kPieces = 3;
    static constexpr float kShiftLog2 = 0.f;
    static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
    static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
};
template <> struct WeightSplit<F16> {
    static constexpr int kPieces = 2;
    static constexpr float kShiftLog2 = 7.f;
    static __device__ __forceinline__ float lo(uint32_t w) { return f16_bits_to_float((uint16_t)w); }
    static __device__ __forceinline__ float hi(uint32_t w) { return f16_bits_to_float((uint16_t)(w >> 16)); }
};

template <class T>
__device__ __forceinline__ void split_weights(const float *p, uint4 (&w)[WeightSplit<T>::kPieces])
{
    using S = WeightSplit<T>;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = p[2 * j], b = p[2 * j + 1];
#pragma unroll
        for (int k = 0; k < S::kPieces; ++k) {
            const uint32_t packed = Mma<T>::pack2(a, b);
            (&w[k].x)[j] = packed;
            a -= S::lo(packed);             // exact: the piece is a rounded to fewer bits
            b -= S::hi(packed);
        }
    }
}

template <class T, int RT, bool kTree, bool kDirect>
__global__ __launch_bounds__(256, (RT <= 2 ? 2 : 1)) void attn_d64_kernel(
    const char *__restrict__ q, const char *__restrict__ k_pages, const char *__restrict__ v_pages,
    const int32_t *__restrict__ block_table, void *__restrict__ out, const int32_t *__restrict__ header,
    const int32_t *__restrict__ unit_meta, const int32_t *__restrict__ sched,
    const unsigned long long *__restrict__ anc, float *__restrict__ part_ml, float *__restrict__ part_o,
    int Hq, int Hkv, int max_pages_per_req, int max_rows, int n_row_groups, float scale_log2, int out_dtype, int cus, DirectArgs direct)
{
    constexpr int kRows = 16 * RT;
    // per wavefront: its V^T tile, later its [rows][d] fp32 state for the merge
    constexpr int kSlab = kRows * kORow64 * 4 > kVtBytes ? kRows * kORow64 * 4 : kVtBytes;
    constexpr int kQLoads = (RT * 2 * 64 + 255) / 256;              // Q^T operand entries per thread
    __shared__ __attribute__((aligned(16))) char smem[kWaves * kSlab];
    __shared__ __attribute__((aligned(16))) uint4 q_lds[RT * 2 * 64];   // Q^T operands, MFMA lane order
    __shared__ float s_m[kWaves][kRows], s_l[kWaves][kRows];
    __shared__ unsigned long long s_anc[kTree ? kRows : 1];         // ancestor mask of each row of the unit

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n16 = lane & 15;
    const int v_half = (lane >> 3) & 1, v_c = lane & 7;             // V loads: half-block and 8-channel chunk of the lane
    const int G = Hq / Hkv;
    const int total_units = kDirect ? 0 : header[0] * Hkv * n_row_groups;
    const int64_t head_bytes = (int64_t)16 * kD64 * 2;              // one (page, head) block
    char *my_lds = smem + wv * kSlab;
    // V^T tile unit of (half, channel 8c + dd, group): 66 dd + 16 grp + 8 half + c
    char *vt_wr = my_lds + 16 * lane;
    const char *vt_rd = my_lds + 16 * (66 * (n16 & 7) + 16 * g + (n16 >> 3));
    float *my_state = reinterpret_cast<float *>(my_lds);

    // K operand: lane (g, m) <- token 16 mt + m, channels 32 s + 8 g .. +7
    // V raw:     lane (tq = g, half, c) <- token 32 half + 16 pg + 4 tq + i, channels 8 c .. 8 c + 7
    uint4 kreg[4][2], vreg[2][4];
    const uint32_t k_lane_off = n16 * (kD64 * 2) + 16 * g;
    const uint32_t v_lane_off = (4 * g) * (kD64 * 2) + 16 * v_c;

    const int W = gridDim.x, wg = blockIdx.x;
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
            const int slen = split_len_of(u.L, u.ns, kBlk64);
            u.t0 = sp * slen; u.t1 = min(u.L, u.t0 + slen);
            u.nblk = (u.t1 - u.t0 + kBlk64 - 1) / kBlk64;
            u.bt_off = (int64_t)u.i * max_pages_per_req;
            ++round;
            return true;
        }
        return false;
    };

    // Page ids by scalar loads; pages past the split's end are replaced by the block's first (masks and the tail code
    // keep what they hold out of the result), so that every block issues the same loads.
    auto page_bases = [&](const Unit &u, int bi, int64_t (&b)[4]) {
        const int tb = u.t0 + bi * kBlk64;
        const int64_t at = u.bt_off + (tb >> 4);
        const int64_t p0 = block_table[at];
        b[0] = (p0 * Hkv + u.gkv) * head_bytes;
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            const int64_t p = (tb + 16 * j < u.t1) ? block_table[at + j] : p0;
            b[j] = (p * Hkv + u.gkv) * head_bytes;
        }
    };
    auto load_k = [&](const int64_t (&b)[4]) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int s = 0; s < 2; ++s) kreg[mt][s] = ld16_stream(k_pages + b[mt] + k_lane_off + 64 * s);
    };
    auto load_v = [&](const int64_t (&b)[4]) {
        const char *vp0 = v_pages + (v_half ? b[2] : b[0]) + v_lane_off, *vp1 = v_pages + (v_half ? b[3] : b[1]) + v_lane_off;
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) vreg[0][ii] = ld16_stream(vp0 + ii * (kD64 * 2));
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) vreg[1][ii] = ld16_stream(vp1 + ii * (kD64 * 2));
    };
    auto first_loads = [&](const Unit &u) {
        if (wv < u.nblk) {
            int64_t b[4];
            page_bases(u, wv, b);
            load_k(b);
            load_v(b);
        }
    };
    // this thread's share of the unit's Q^T operands: entry (row tile, s, lane)
    auto load_q = [&](const Unit &u, uint4 (&qv)[kQLoads]) {
#pragma unroll
        for (int k = 0; k < kQLoads; ++k) {
            const int e = tid + 256 * k;
            const int row = u.r0 + 16 * (e >> 7) + n16;
            qv[k] = make_uint4(0, 0, 0, 0);
            if (e < RT * 128 && row < u.rows)
                qv[k] = ld16(q + (((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * kD64) * 2 + 64 * ((e >> 6) & 1) + 16 * g);
        }
    };
    auto load_anc = [&](const Unit &u) -> unsigned long long {
        const int row = u.r0 + tid;
        return (tid < kRows && row < u.rows) ? anc[u.qrow0 + row / G] : 0ull;
    };

    Unit cur, nxt;
    bool have;
    uint4 qv[kQLoads];
    unsigned long long av = 0ull;
    if constexpr (kDirect) have = direct_unit(cur, direct, block_table, G, Hkv, n_row_groups, kRows, kBlk64, max_pages_per_req, wv, lane);
    else have = next_unit(cur);
    if (have) {
        load_q(cur, qv);
        if constexpr (kTree) av = load_anc(cur);
        first_loads(cur);
    }

    while (have) {
        const Unit u = cur;
        const bool have_next = kDirect ? false : next_unit(nxt);
        const int first_masked = u.L - u.n + 1;                    // tokens >= this are hidden from some row
#pragma unroll
        for (int k = 0; k < kQLoads; ++k)
            if (tid + 256 * k < RT * 128) q_lds[tid + 256 * k] = qv[k];
        if constexpr (kTree) { if (tid < kRows) s_anc[tid] = av; }
        int pos[RT];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            const int row = u.r0 + 16 * nt + n16;
            pos[nt] = row < u.rows ? (u.L - u.n + row / G) : -1;
        }
        lds_barrier();

        float m[RT], lsum[RT];
        f32x4 o[RT][4];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            m[nt] = kLowestRef; lsum[nt] = 0.f;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) o[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

        // One 64-token block; kNext: the following block's K and V are requested while this one is being processed.
        auto block = [&](int bi, auto next_tag) {
            constexpr bool kNext = decltype(next_tag)::value;
            const int tb = u.t0 + bi * kBlk64;
            int64_t nb[4] = {0, 0, 0, 0};
            if constexpr (kNext) page_bases(u, bi + kWaves, nb);

            // ---- S^T = K Q^T ------------------------------------------------------------
            float p[RT][16];
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                uint4 qop[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) qop[s] = q_lds[(nt * 2 + s) * 64 + lane];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < 2; ++s) acc = Mma<T>::run(kreg[mt][s], qop[s], acc);
#pragma unroll
                    for (int r = 0; r < 4; ++r) p[nt][4 * mt + r] = acc[r];
                }
            }
            if constexpr (kNext) load_k(nb);

            // ---- online softmax (per lane: row n16 of each row tile, 16 of the 64 tokens) ----
            const bool need_mask = (tb + kBlk64 > first_masked) || (tb + kBlk64 > u.t1);
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                if (need_mask) {
                    if constexpr (kTree) {
                        const unsigned long long am = s_anc[16 * nt + n16];
                        const int base = u.L - u.n;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int t = tb + 16 * (e >> 2) + 4 * g + (e & 3);
                            const int rel = t - base;
                            const bool vis = t < u.t1 && (rel < 0 ? pos[nt] >= 0 : ((am >> (rel & 63)) & 1ull) != 0);
                            p[nt][e] = vis ? p[nt][e] : -INFINITY;
                        }
                    } else {
                        const int lim = min(pos[nt], u.t1 - 1);
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int t = tb + 16 * (e >> 2) + 4 * g + (e & 3);
                            p[nt][e] = (t <= lim) ? p[nt][e] : -INFINITY;
                        }
                    }
                }
                float mx = p[nt][0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx = fmaxf(mx, p[nt][e]);
                mx = max_over_row_groups(mx);
                // lazy reference: moves only when the block's maximum exceeds it by more than kLazyLog2
                const float mxs = mx * scale_log2;
                const bool grow = mxs > m[nt] + kLazyLog2;
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(grow) != 0, 0)) {
                    const float m_new = grow ? mxs : m[nt];
                    const float alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
                    m[nt] = m_new;
                    lsum[nt] *= alpha;
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) o[nt][dt] *= alpha;
                }
                softmax_weights<16>(p[nt], scale_log2, m[nt], WeightSplit<T>::kShiftLog2);
                float psum = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) psum += p[nt][e];
                lsum[nt] += psum;
            }

            // ---- V^T tile: blank the tail, transpose 4x8 in registers, write to LDS --------
            if (tb + kBlk64 > u.L) {                   // the request's last, partial block
#pragma unroll
                for (int pg = 0; pg < 2; ++pg)
#pragma unroll
                    for (int ii = 0; ii < 4; ++ii)
                        if (tb + 32 * v_half + 16 * pg + 4 * g + ii >= u.L) vreg[pg][ii] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t a0 = (&vreg[0][0].x)[w], a1 = (&vreg[0][1].x)[w];
                const uint32_t a2 = (&vreg[0][2].x)[w], a3 = (&vreg[0][3].x)[w];
                const uint32_t b0 = (&vreg[1][0].x)[w], b1 = (&vreg[1][1].x)[w];
                const uint32_t b2 = (&vreg[1][2].x)[w], b3 = (&vreg[1][3].x)[w];
                uint4 even = make_uint4(__builtin_amdgcn_perm(a1, a0, 0x05040100u),
                                        __builtin_amdgcn_perm(a3, a2, 0x05040100u),
                                        __builtin_amdgcn_perm(b1, b0, 0x05040100u),
                                        __builtin_amdgcn_perm(b3, b2, 0x05040100u));
                uint4 odd = make_uint4(__builtin_amdgcn_perm(a1, a0, 0x07060302u),
                                       __builtin_amdgcn_perm(a3, a2, 0x07060302u),
                                       __builtin_amdgcn_perm(b1, b0, 0x07060302u),
                                       __builtin_amdgcn_perm(b3, b2, 0x07060302u));
                *reinterpret_cast<uint4 *>(vt_wr + 66 * 16 * (2 * w)) = even;
                *reinterpret_cast<uint4 *>(vt_wr + 66 * 16 * (2 * w + 1)) = odd;
            }
            if constexpr (kNext) load_v(nb);

            // ---- O^T += V^T P^T, one 32-token half after the other ------------------------------
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                uint4 pop[RT][WeightSplit<T>::kPieces];
#pragma unroll
                for (int nt = 0; nt < RT; ++nt) split_weights<T>(&p[nt][8 * half], pop[nt]);
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) {
                    const uint4 vt = *reinterpret_cast<const uint4 *>(vt_rd + 32 * (4 * half + dt));
#pragma unroll
                    for (int nt = 0; nt < RT; ++nt)
#pragma unroll
                        for (int k = 0; k < WeightSplit<T>::kPieces; ++k) o[nt][dt] = Mma<T>::run(vt, pop[nt][k], o[nt][dt]);
                }
            }
        };

        if (wv < u.nblk) {
            int bi = wv;
            for (; bi + kWaves < u.nblk; bi += kWaves) block(bi, std::true_type{});
            block(bi, std::false_type{});
        }

        // ---- next unit: its first K/V block and Q rows travel while this unit's states are merged
        if (have_next) {
            load_q(nxt, qv);
            if constexpr (kTree) av = load_anc(nxt);
            first_loads(nxt);
        }
        // ---- merge the four wavefronts' states through LDS (as in attn_mfma.hip) ----------
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            lsum[nt] += __shfl_xor(lsum[nt], 16, kWave);
            lsum[nt] += __shfl_xor(lsum[nt], 32, kWave);
            if (g == 0) { s_m[wv][16 * nt + n16] = m[nt]; s_l[wv][16 * nt + n16] = lsum[nt]; }
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                *reinterpret_cast<f32x4 *>(my_state + (16 * nt + n16) * kORow64 + 16 * dt + 4 * g) = o[nt][dt];
        }
        lds_barrier();
        // 256 threads: 16*RT rows x 16 float4 columns
#pragma unroll
        for (int it = 0; it < RT; ++it) {
            const int idx = tid + 256 * it;
            const int rl = idx >> 4, c4 = idx & 15;
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
                acc += sc * *reinterpret_cast<const f32x4 *>(smem + w * kSlab + 4 * (rl * kORow64 + 4 * c4));
            }
            if (u.ns == 1) {
                const float inv = 1.0f / ltot;
                const int64_t obase = ((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * (int64_t)kD64 + 4 * c4;
                if (out_dtype == ADASPEC_F32) {
                    *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(out) + obase) = acc * inv;
                } else {
                    uint2 pk = make_uint2(Mma<T>::pack2(acc[0] * inv, acc[1] * inv),
                                          Mma<T>::pack2(acc[2] * inv, acc[3] * inv));
                    *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + obase) = pk;
                }
            } else {
                const int64_t idx_row = ((int64_t)u.item * Hkv + u.gkv) * max_rows + row;
                if (kDirect && attn_merge_fits(kD64, RT) && direct.flags) {
                    store_state(part_o + idx_row * kD64 + 4 * c4, acc);
                    if (c4 == 0) store_ml(part_ml + idx_row * 2, ms, ltot);
                } else {
                    *reinterpret_cast<f32x4 *>(part_o + idx_row * kD64 + 4 * c4) = acc;
                    if (c4 == 0) {
                        part_ml[idx_row * 2] = ms;
                        part_ml[idx_row * 2 + 1] = ltot;
                    }
                }
            }
        }
        if constexpr (kDirect) {
            if constexpr (attn_merge_fits(kD64, RT)) {
                if (u.ns > 1 && direct.flags)
                    merge_splits<T, kD64, kRows>(direct, u, part_ml, part_o, out, out_dtype, Hq, Hkv, G, max_rows, tid);
            }
            break;
        }
        // the next loop iteration overwrites q_lds, the V^T tiles and s_m: everyone must be done reading the states
        lds_barrier();
        cur = nxt;
        have = have_next;
    }
}

// ---- host side -----------------------------------------------------------------------------------------------
template <typename F>
static void with_d64_instance(const AttnArgs &a, F &&f)
{
    const int rt = attn_row_tiles(a.plan.max_rows);
    auto with_mode = [&](auto tag, auto rt_tag) {
        if (a.direct) f(tag, rt_tag, std::false_type{}, std::true_type{});
        else if (a.parents) f(tag, rt_tag, std::true_type{}, std::false_type{});
        else f(tag, rt_tag, std::false_type{}, std::false_type{});
    };
    auto with_rt = [&](auto tag) {
        if (rt == 1) with_mode(tag, std::integral_constant<int, 1>{});
        else if (rt == 2) with_mode(tag, std::integral_constant<int, 2>{});
        else with_mode(tag, std::integral_constant<int, 4>{});
    };
    if (a.dims.dtype == ADASPEC_F16) with_rt(F16{});
    else with_rt(BF16{});
}

template <typename T, int RT, bool kTree, bool kDirect>
static int attn_d64_slots(int cus)
{
    static int slots = 0;
    if (slots == 0) {
        int per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_d64_kernel<T, RT, kTree, kDirect>, 256, 0) != hipSuccess)
            per_cu = 1;
        const int n = cus * (per_cu > 0 ? per_cu : 1);
        slots = n < kMaxSchedW ? n : kMaxSchedW;
    }
    return slots;
}

int attn_d64_grid_slots(const AttnArgs &a, int cus)
{
    int slots = 1;
    with_d64_instance(a, [&](auto tag, auto rt, auto tree, auto direct) {
        slots = attn_d64_slots<decltype(tag), decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>(cus);
    });
    return slots;
}

hipError_t launch_attn_d64(const AttnArgs &a)
{
    const AttnPlan &p = a.plan;
    const adaspec_attn_dims &d = a.dims;
    if (a.sched_w <= 0) return hipSuccess;                          // no work item can exist
    with_d64_instance(a, [&](auto tag, auto rt, auto tree, auto direct) {
        hipLaunchKernelGGL((attn_d64_kernel<decltype(tag), decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>),
                           dim3(a.sched_w), dim3(256), 0, a.stream, (const char *)a.q, (const char *)a.k_pages,
                           (const char *)a.v_pages, a.block_table, a.out, (const int32_t *)(a.ws + p.off_header),
                           (const int32_t *)(a.ws + p.off_unit_meta), (const int32_t *)(a.ws + p.off_sched),
                           (const unsigned long long *)(a.ws + p.off_anc), (float *)(a.ws + p.off_part_ml),
                           (float *)(a.ws + p.off_part_o), d.n_q_heads, d.n_kv_heads, d.max_pages_per_req, p.max_rows,
                           a.n_row_groups, a.scale_log2, d.out_dtype, a.sched_cus, direct_args(a));
    });
    return hipGetLastError();
}

}  // namespace adaspec
