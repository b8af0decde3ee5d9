// Matrix-core verification attention for units with MANY query rows (more than 32 rows share a kv head: long drafts times a
// wide GQA group): gfx950, 16-bit K/V/Q, head_dim 128, three or four row tiles of 16 rows.
//
// As in attn_mfma.hip, a workgroup of 4 wavefronts takes one unit (request x KV split, kv head, group of up to 16 RT rows),
// wavefront w streams the 32-token blocks w, w + 4, ... of the split and keeps the online-softmax state of ALL rows of the
// unit, S^T = K Q^T and O^T += V^T P^T in accumulator layouts that need no shuffle; the four states are merged through LDS.
// There K and V travel through registers, and beside three row tiles (32 accumulator registers each) those no longer fit.
// Here they travel from memory straight into LDS: every wavefront has a K slot and a V slot of one block each, filled by
// loads with an LDS destination, and nobody else touches them, so the block loop has no barrier.  A slot is requested again
// as soon as its operands are out of it, K's ahead of the arithmetic, V's behind it.  K operands are ordinary 16-byte reads;
// V^T operands come out of the row-major slot through gfx950's transposing reads.
//
// Bound: HBM.  The row split (attn_rows.hip, which keeps the short contexts) shares every block among the four wavefronts, one
// row tile each, behind a barrier per block: a unit of 8 rows keeps one wavefront busy and three waiting, and the operands of a
// block are read four times.  Whole calls on MI355X (bf16, 64/8 heads, up to 48 rows), row split / ring: 64 requests of 2048-8192 tokens
// 258 / 245 us, 48 of 1024-4096 120 / 106, 40 of 4000 160 / 138, 60 of 500 and 4 of 16000 104 / 83, 64 of 300-1000 44.5 / 37.3;
// 28/4 heads, 80 of 1000-6000 137 / 126.  A probe that only loads reaches 6.3 TB/s on this pattern through registers or one
// shared ring and 6.8 TB/s with a ring per wavefront; without the states of the splits the kernel runs at 6.5 TB/s, but
// every byte of them written costs about as much as five read (52 MB beside 2.1 GB: 327 -> 365 us).
#include "adaspec_internal.h"
#include "attn_mfma_common.h"
#include "device_utils.h"

namespace adaspec {

constexpr int kHalfBytes = kBlk * kD * 2;       // K, or V, of a block: two pages of 4 KB
constexpr int kRingBytes = kWaves * 2 * kHalfBytes;

// LDS of a workgroup: per wavefront a K slot and a V slot of one block each; Q^T operands in MFMA lane order; (m, l) of every
// wavefront's rows; tree: the ancestor mask of each row.  Two workgroups per compute unit have 80 KB each, which four row
// tiles fill with ring and Q alone: (m, l) then take the place of Q, and masks are read from memory.
template <int RT, bool kTree> struct RingLds {
    static constexpr int kRows = 16 * RT;
    static constexpr bool kFull = RT == 4;
    static constexpr int kQ = kRingBytes, kQBytes = RT * 4 * 1024;
    static constexpr int kMl = kFull ? kQ : kQ + kQBytes, kMlBytes = kWaves * kRows * 2 * 4;
    static constexpr bool kAncInLds = kTree && !kFull;
    static constexpr int kAnc = kQ + kQBytes + kMlBytes;
    static constexpr int kTouch = kAnc + (kAncInLds ? kRows * 8 : 0);      // where touched Q lines are dropped
    static constexpr int kBytes = kFull ? kQ + kQBytes : kTouch + kWaves * 256;
    static_assert(kBytes <= 81920, "two workgroups per compute unit");
};

template <class T, int RT, bool kTree, bool kDirect>
__global__ __launch_bounds__(256, 2) void attn_ring_kernel(
    const char *__restrict__ q, const char *__restrict__ k_pages, const char *__restrict__ v_pages,
    const int32_t *__restrict__ block_table, void *__restrict__ out, const int32_t *__restrict__ header,
    const int32_t *__restrict__ unit_meta, const int32_t *__restrict__ sched,
    const unsigned long long *__restrict__ anc, float *__restrict__ part_ml, float *__restrict__ part_o,
    int Hq, int Hkv, int max_pages_per_req, int max_rows, int n_row_groups, float scale_log2,
    int out_dtype, int cus, DirectArgs direct)
{
    using Lds = RingLds<RT, kTree>;
    constexpr int kRows = 16 * RT;
    static_assert(kRows + 1 <= kRingQRows, "what the plan allows for");
    __shared__ __attribute__((aligned(1024))) char smem[Lds::kBytes];
    const uint32_t lds_base = lds_address(smem);
    float *s_m = reinterpret_cast<float *>(smem + Lds::kMl), *s_l = s_m + kWaves * kRows;    // [wavefront][row]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);        // wave-uniform by construction
    const int g = lane >> 4, n16 = lane & 15;
    const int G = Hq / Hkv;
    const int total_units = kDirect ? 0 : header[0] * Hkv * n_row_groups;
    const int64_t head_bytes = (int64_t)16 * kD * 2;                // one (page, head) block

    // ---- this wavefront's two slots ------------------------------------------------------------------------
    // A slot holds 32 token rows of 256 bytes.  In K's the 16-byte chunk c of token t stands at place c ^ (t % 16) of its
    // row (operand reads take one chunk of 16 consecutive tokens), in V's the 32-byte chunk cc at place cc ^ (t % 8) (the
    // transposing reads take one 32-byte chunk of 16 consecutive tokens): both without bank conflicts, while the loader
    // fetches whole rows.  A load instruction fills four rows; instruction j of a page has its 1024 j bytes in the offset
    // field, which moves both addresses.
    char *k_slot = smem + wv * 2 * kHalfBytes;
    char *v_slot = k_slot + kHalfBytes;
    const uint32_t k_lds = lds_base + wv * 2 * kHalfBytes, v_lds = k_lds + kHalfBytes;
    uint32_t k_voff[4], v_voff[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) k_voff[j] = g * 256 + 16 * (n16 ^ g ^ (4 * j));
#pragma unroll
    for (int j = 0; j < 2; ++j) v_voff[j] = g * 256 + 16 * (n16 ^ (2 * g) ^ (8 * j));
    // K as A operand of (mt, s): lane (g, m) <- token 16 mt + m, chunk 4 s + g
    uint32_t k_rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) k_rd[s] = n16 * 256 + 16 * ((4 * s + g) ^ n16);
    // V^T as A operand of channel tile dt: lane (g, m) gives the place of token 4 g + m / 4, channels 16 dt + 4 (m % 4) .. + 3,
    // and gets channel 16 dt + m of tokens 4 g .. 4 g + 3
    const uint32_t v_rd = v_lds + (4 * g + (n16 >> 2)) * 256 + 32 * ((4 * g + (n16 >> 2)) & 7) + 8 * (n16 & 3);

    auto read_vt = [&](int dt) -> uint4 {
        const uint2 lo = read_transposed(v_rd ^ (32 * dt)), hi = read_transposed((v_rd ^ (32 * dt)) + 4096);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };

    // ---- work-unit bookkeeping ----------------------------------------------------------------
    // Units are listed longest first and handed out in rounds of W (one unit per workgroup and
    // round).  Which unit a workgroup takes in a round is a table the plan kernel wrote.  No atomic is
    // needed and the next unit is known ahead of time, so its data can be requested early.
    const int W = gridDim.x, wg = blockIdx.x;
    const int n_rounds = kDirect ? 0 : header[2];
    int round = 0;
    int idx_ahead = kDirect ? 0 : sched_position(0, wg, W, cus, header[1]);     // round 0 needs no table
    auto next_unit = [&](Unit &u) -> bool {
        for (; round < n_rounds; ++round) {
            const int idx = idx_ahead;
            // the entry of the following round is requested together with this unit's record, one
            // unit before it is needed
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
            const int slen = split_len_of(u.L, u.ns, kBlk);
            u.t0 = sp * slen; u.t1 = min(u.L, u.t0 + slen);
            u.nblk = (u.t1 - u.t0 + kBlk - 1) / kBlk;
            u.bt_off = (int64_t)u.i * max_pages_per_req;
            ++round;
            return true;
        }
        return false;
    };

    // Page ids are wave-uniform (scalar loads: they never wait on the vector-memory counter).
    // Loads are issued unconditionally so that the counter waits stay exact: a block's second
    // page may lie past the split's end, then the first page is fetched again and masks and the
    // tail code below blank what must not be used.
    auto page_bases = [&](const Unit &u, int bi, int64_t &b0, int64_t &b1) {
        const int tb = u.t0 + bi * kBlk;
        const int64_t p0 = block_table[u.bt_off + (tb >> 4)];
        const int64_t p1 = (tb + 16 < u.t1) ? block_table[u.bt_off + (tb >> 4) + 1] : p0;
        b0 = (p0 * Hkv + u.gkv) * head_bytes;
        b1 = (p1 * Hkv + u.gkv) * head_bytes;
    };
    auto issue_k = [&](int64_t b0, int64_t b1) {
        load_page_to_lds(page_rsrc(k_pages + b0), k_voff[0], k_voff[1], k_voff[2], k_voff[3], k_lds);
        load_page_to_lds(page_rsrc(k_pages + b1), k_voff[0], k_voff[1], k_voff[2], k_voff[3], k_lds + 4096);
    };
    auto issue_v = [&](int64_t b0, int64_t b1) {
        load_page_to_lds(page_rsrc(v_pages + b0), v_voff[0], v_voff[1], v_voff[0], v_voff[1], v_lds);
        load_page_to_lds(page_rsrc(v_pages + b1), v_voff[0], v_voff[1], v_voff[0], v_voff[1], v_lds + 4096);
    };
    // The unit's Q^T operands, a quarter per wavefront: entry (nt, s = wv, lane) of q_lds.  Rows past the last one repeat it
    // (their results are never stored).  Tree: 32 ancestor masks per wavefront beside them, two lanes each.
    auto issue_q = [&](const Unit &u) {
        int lane_q = lane;                                          // (computed from here on every call)
        asm volatile("" : "+v"(lane_q));
        const int n0 = u.r0 / G;                                    // first query row of this group
        const v4i32 rs = buffer_rsrc(q + (u.qrow0 + n0) * Hq * (int64_t)(kD * 2), (uint32_t)(min(u.n - n0, kRows + 1) * Hq) * (kD * 2));
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            const int row = min(u.r0 + 16 * nt + (lane_q & 15), u.rows - 1);
            const uint32_t off = (uint32_t)(((row / G - n0) * Hq + u.gkv * G + row % G) * (kD * 2) + 64 * wv + 16 * (lane_q >> 4));
            load16_to_lds(rs, off, lds_base + Lds::kQ + (nt * 4 + wv) * 1024);
        }
        if constexpr (Lds::kAncInLds) {
            if (32 * wv < kRows) {
                const int row = min(u.r0 + min(32 * wv + (lane_q >> 1), kRows - 1), u.rows - 1);
                if (32 * wv + (lane_q >> 1) < kRows)                // (inactive lanes write nothing)
                    load4_to_lds(buffer_rsrc(reinterpret_cast<const char *>(anc + u.qrow0), (uint32_t)u.n * 8),
                                 (uint32_t)(row / G) * 8 + 4 * (lane_q & 1), lds_base + Lds::kAnc + wv * 256);
            }
        }
    };

    // One 4-byte load per (row, 64-byte share of this wavefront): brings the unit's Q into the L2 ahead of issue_q, which can
    // only start when every wavefront is done with the Q in LDS.
    auto touch_q = [&](const Unit &u) {
        int lane_q = lane;
        asm volatile("" : "+v"(lane_q));
        const int n0 = u.r0 / G, row = min(u.r0 + min(lane_q, kRows - 1), u.rows - 1);
        const v4i32 rs = buffer_rsrc(q + (u.qrow0 + n0) * Hq * (int64_t)(kD * 2), (uint32_t)(min(u.n - n0, kRows + 1) * Hq) * (kD * 2));
        load4_to_lds(rs, (uint32_t)(((row / G - n0) * Hq + u.gkv * G + row % G) * (kD * 2) + 64 * wv), lds_base + Lds::kTouch + wv * 256);
    };

    Unit cur, nxt;
    bool have;
    int64_t b0 = 0, b1 = 0;                     // pages of the block that comes next in this wavefront's stream
    if constexpr (kDirect) have = direct_unit(cur, direct, block_table, G, Hkv, n_row_groups, kRows, kBlk, max_pages_per_req, wv, lane);
    else have = next_unit(cur);
    if (have) {
        if (wv < cur.nblk) {
            page_bases(cur, wv, b0, b1);
            issue_k(b0, b1);
        }
        issue_q(cur);
        // everything but the first block's V (8 loads) has landed; behind the barrier, the other wavefronts' share of Q too
        if (wv < cur.nblk) {
            issue_v(b0, b1);
            wait_loads<8>();
        } else {
            wait_loads<0>();
        }
        lds_barrier();
    }

    while (have) {
        const Unit u = cur;
        bool have_next = false, next_block = false;                 // a next unit; one with a block for this wavefront
        int looked_up = kDirect;
        auto look_up_next = [&]() {
            have_next = next_unit(nxt);
            next_block = have_next && wv < nxt.nblk;
            looked_up = 1;
        };
        const int first_masked = u.L - u.n + 1;                    // tokens >= this are hidden from some row
        int pos[RT];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            const int row = u.r0 + 16 * nt + n16;
            pos[nt] = row < u.rows ? (u.L - u.n + row / G) : -1;
        }
        float m[RT], lsum[RT];
        f32x4 o[RT][8];
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            m[nt] = kNegBig; lsum[nt] = 0.f;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) o[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

#pragma unroll 1
        for (int bi = wv; bi < u.nblk; bi += kWaves) {
            const int tb = u.t0 + bi * kBlk;
            // the block after this one: of this unit, or the first of the next (its record is read one block earlier, in
            // front of a wait for memory, like the page ids: a chain of scalar loads takes some microseconds under load)
            if (!looked_up && bi + 2 * kWaves >= u.nblk) look_up_next();
            const bool more = bi + kWaves < u.nblk, ahead = more || next_block;
            if (more) page_bases(u, bi + kWaves, b0, b1);
            else if (next_block) page_bases(nxt, wv, b0, b1);
            if (bi != wv) wait_loads<8>();                          // K of this block (its V is 8 loads younger)

            // ---- K operands out of the slot, the next block's K into it ----------------------------------------
            uint4 ka[2][4];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int s = 0; s < 4; ++s) ka[mt][s] = *reinterpret_cast<const uint4 *>(k_slot + mt * 4096 + k_rd[s]);
            const bool touch = !Lds::kFull && !more && have_next;
            if (touch) touch_q(nxt);
            if (ahead) {
                wait_lds();
                issue_k(b0, b1);
            }

            // ---- S^T = K Q^T, online softmax (per lane: row n16 of each row tile, 8 of the 32 tokens) -----------
            const bool need_mask = (tb + kBlk > first_masked) || (tb + kBlk > u.t1);
            uint4 pop[RT], pop_lo[RT];
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                uint4 qop[4];
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    qop[s] = *reinterpret_cast<const uint4 *>(smem + Lds::kQ + (nt * 4 + s) * 1024 + lane * 16);
                float sv[8];
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < 4; ++s) acc = Mma<T>::run(ka[mt][s], qop[s], acc);
#pragma unroll
                    for (int r = 0; r < 4; ++r) sv[4 * mt + r] = acc[r];
                }
                if (need_mask) {
                    if constexpr (kTree) {
                        // committed tokens are visible to every real row; new position base + a only if bit a of the
                        // row's mask is set.  As one bit per token of the block: no branches.
                        unsigned long long am;
                        if constexpr (Lds::kAncInLds) {
                            am = *reinterpret_cast<const unsigned long long *>(smem + Lds::kAnc + (16 * nt + n16) * 8);
                        } else {
                            am = anc[u.qrow0 + min(u.r0 + 16 * nt + n16, u.rows - 1) / G];
                        }
                        const int old = u.L - u.n - tb, left = u.t1 - tb;      // committed tokens, tokens of this block
                        uint32_t vis;
                        if (old >= kBlk) vis = ~0u;
                        else if (old >= 0) vis = (uint32_t)(am << old) | ((1u << old) - 1u);
                        else vis = (uint32_t)(am >> (-old & 63));
                        if (left < kBlk) vis &= (1u << left) - 1u;
                        vis = pos[nt] < 0 ? 0u : vis >> (4 * g);               // (padding rows: nothing)
#pragma unroll
                        for (int e = 0; e < 8; ++e) sv[e] = (vis & (1u << (16 * (e >> 2) + (e & 3)))) ? sv[e] : -INFINITY;
                    } else {
                        const int lim = min(pos[nt], u.t1 - 1);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int t = tb + 16 * (e >> 2) + 4 * g + (e & 3);
                            sv[e] = (t <= lim) ? sv[e] : -INFINITY;
                        }
                    }
                }
                float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])),
                                 fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
                mx = max_over_row_groups(mx);
                // Lazy reference: the running reference m of a row moves only when the block's maximum exceeds it
                // by more than kLazyLog2 (weights then stay below 2^kLazyLog2, harmless in fp32 and in the
                // 16-bit operand formats), so the accumulators are rescaled in a handful of blocks per unit
                // instead of in almost every one, and the rescaling sits on a cold path.
                const float mxs = mx * scale_log2;
                const bool grow = mxs > m[nt] + kLazyLog2;
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(grow) != 0, 0)) {
                    const float m_new = grow ? mxs : m[nt];
                    const float alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
                    m[nt] = m_new;
                    lsum[nt] *= alpha;
#pragma unroll
                    for (int dt = 0; dt < 8; ++dt) o[nt][dt] *= alpha;
                }
                const float m_ref = m[nt];
                float p[8], psum = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(fmaf(sv[e], scale_log2, -m_ref));
                    psum += p[e];
                }
                lsum[nt] += psum;
                pop[nt] = make_uint4(Mma<T>::pack2(p[0], p[1]), Mma<T>::pack2(p[2], p[3]),
                                     Mma<T>::pack2(p[4], p[5]), Mma<T>::pack2(p[6], p[7]));
                if constexpr (Mma<T>::kSplitP) {
                    const uint32_t *hi = &pop[nt].x;
                    uint32_t lo[4];
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        lo[w] = Mma<T>::pack2(p[2 * w] - __uint_as_float(hi[w] << 16),
                                              p[2 * w + 1] - __uint_as_float(hi[w] & 0xffff0000u));
                    pop_lo[nt] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                }
            }

            // ---- V of this block: blank the rows past the request's end -----------------------------------------
            if (ahead && touch) wait_loads<9>();
            else if (ahead) wait_loads<8>();
            else wait_loads<0>();
            if (tb + kBlk > u.L) {
                for (int t = u.L - tb + g; t < kBlk; t += 4)
                    *reinterpret_cast<uint4 *>(v_slot + t * 256 + n16 * 16) = make_uint4(0, 0, 0, 0);
            }
            // ---- O^T += V^T P^T, then the next block's V into the slot --------------------------------------------
            uint4 vt = read_vt(0);
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
                uint4 vt_next = vt;
                if (dt < 7) vt_next = read_vt(dt + 1);
#pragma unroll
                for (int nt = 0; nt < RT; ++nt) {
                    o[nt][dt] = Mma<T>::run(vt, pop[nt], o[nt][dt]);
                    if constexpr (Mma<T>::kSplitP) o[nt][dt] = Mma<T>::run(vt, pop_lo[nt], o[nt][dt]);
                }
                vt = vt_next;
            }
            if (more) {
                wait_lds();
                issue_v(b0, b1);
            }
        }
        if (wv >= u.nblk) {                                         // (this unit had no block for this wavefront)
            if (!looked_up) look_up_next();
            if (next_block) {
                page_bases(nxt, wv, b0, b1);
                issue_k(b0, b1);
            }
        }

        // ---- a context of one block (beside longer ones: calls of short contexts only take attn_rows.hip) has one state: straight
        // out of the registers (88 requests of 9-30 tokens, 40 rows, 64/8 heads: 13.3 us, 14.9 through the merge).  Lane (g, n16) holds O^T[16 dt + 4 g .. + 3][row n16 of the tile].
        if (kDirect && u.ns == 1 && u.nblk == 1) {
            if (wv > 0) break;
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                lsum[nt] += __shfl_xor(lsum[nt], 16, kWave);
                lsum[nt] += __shfl_xor(lsum[nt], 32, kWave);
                const int row = u.r0 + 16 * nt + n16;
                if (row >= u.rows) continue;
                const float inv = 1.0f / lsum[nt];
                const int64_t obase = ((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * (int64_t)kD + 4 * g;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    const f32x4 val = o[nt][dt] * inv;
                    if (out_dtype == ADASPEC_F32)
                        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(out) + obase + 16 * dt) = val;
                    else
                        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + obase + 16 * dt) =
                            make_uint2(Mma<T>::pack2(val[0], val[1]), Mma<T>::pack2(val[2], val[3]));
                }
            }
            break;
        }

        // ---- merge the four wavefronts' states through LDS, one row tile at a time: each wavefront leaves its own over its V
        // slot (which holds exactly one tile; the next unit's K travels into the K slot meanwhile), then every output
        // element is put together from the four,
        //   O = sum_w 2^(m_w - m*) O_w, m* = max over wavefronts.
        // The 16-byte pieces of a row are exchanged by the row's number so that neither side meets bank conflicts.
        // (Opaque copies of the thread's numbers: everything below is computed from them here, not kept in registers across
        // the block loop.)
        int tid_m = tid, lane_m = lane;
        asm volatile("" : "+v"(tid_m), "+v"(lane_m));
        const int g_m = lane_m >> 4, n_m = lane_m & 15;
        if constexpr (Lds::kFull) lds_barrier();                    // (m, l) go where Q stands: all are done with it
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            lsum[nt] += __shfl_xor(lsum[nt], 16, kWave);
            lsum[nt] += __shfl_xor(lsum[nt], 32, kWave);
            if (g_m == 0) { s_m[wv * kRows + 16 * nt + n_m] = m[nt]; s_l[wv * kRows + 16 * nt + n_m] = lsum[nt]; }
        }
        // A thread's share of a tile: row tid / 16, two pieces of four channels: side by side where 16-bit results are stored
        // (16 bytes per thread), 64 channels apart where fp32 values are (256 bytes in a row per 16 threads and store).
        // The results leave only when the next unit's first loads are requested and its Q is there: the memory counter
        // retires in order, and in front of those loads the stores would hold up its start (not with four row tiles, whose
        // registers are full).  Split states go past the L2 (nobody reads them before the combine kernel): written back
        // from there while the streams evict them, they cost the reads more (512 units of 48 rows in 4 splits, 52 MB of
        // states: 384 -> 365 us).  And every store instruction costs its turn in a full memory pipeline, however few bytes it
        // moves: (m, l) of all rows leave in one.
        const bool packed = u.ns == 1 && out_dtype != ADASPEC_F32;
        auto piece = [&](int p) { return packed ? 2 * (tid_m & 15) + p : (tid_m & 15) + 16 * p; };
        auto store_result = [&](int nt, const f32x4 (&acc)[2], float inv) {
            const int row = u.r0 + 16 * nt + (tid_m >> 4);
            if (row >= u.rows) return;
            const int64_t obase = ((u.qrow0 + row / G) * Hq + u.gkv * G + row % G) * (int64_t)kD;
            if (packed) {
                *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(out) + obase + 4 * piece(0)) =
                    make_uint4(Mma<T>::pack2(acc[0][0] * inv, acc[0][1] * inv), Mma<T>::pack2(acc[0][2] * inv, acc[0][3] * inv),
                               Mma<T>::pack2(acc[1][0] * inv, acc[1][1] * inv), Mma<T>::pack2(acc[1][2] * inv, acc[1][3] * inv));
            } else if (u.ns == 1) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(out) + obase + 4 * piece(p)) = acc[p] * inv;
            } else {
                const int64_t idx_row = ((int64_t)u.item * Hkv + u.gkv) * max_rows + row;
#pragma unroll
                for (int p = 0; p < 2; ++p) store_state(part_o + idx_row * kD + 4 * piece(p), acc[p]);
            }
        };
        // (m, l) of row rl over the four wavefronts
        auto merged_ml = [&](int rl) {
            float2 v = make_float2(s_m[rl], 0.f);
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v.x = fmaxf(v.x, s_m[w * kRows + rl]);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v.y += __builtin_amdgcn_exp2f(s_m[w * kRows + rl] - v.x) * s_l[w * kRows + rl];
            return v;
        };
        const int tiles = min((u.rows - u.r0 + 15) / 16, RT);       // row tiles that hold rows
        f32x4 res[RT][2];
        float inv[RT];
        float2 row_ml = make_float2(0.f, 0.f);
#pragma unroll
        for (int nt = 0; nt < RT; ++nt) {
            if (nt >= tiles) break;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt)
                *reinterpret_cast<f32x4 *>(v_slot + n_m * 512 + 16 * ((4 * dt + g_m) ^ n_m)) = o[nt][dt];
            lds_barrier();
            if (!Lds::kFull && nt == 0 && have_next) issue_q(nxt);
            const int rt = tid_m >> 4, rl = 16 * nt + rt;
            const float2 ml = merged_ml(rl);
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float sc = __builtin_amdgcn_exp2f(s_m[w * kRows + rl] - ml.x);
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    acc[p] += sc * *reinterpret_cast<const f32x4 *>(smem + (2 * w + 1) * kHalfBytes + rt * 512 + 16 * (piece(p) ^ rt));
            }
            if (nt == 0 && u.ns > 1 && tid_m < kRows) row_ml = merged_ml(tid_m);
            if constexpr (Lds::kFull) {
                store_result(nt, acc, 1.0f / ml.y);
            } else {
                res[nt][0] = acc[0]; res[nt][1] = acc[1];
                inv[nt] = 1.0f / ml.y;
            }
            // the next tile, or the next unit's V, overwrites the slots: everyone must be done reading the states
            if (nt + 1 < RT || have_next) lds_barrier();
        }
        if (have_next) {
            if constexpr (Lds::kFull) issue_q(nxt);
            if (next_block) {
                issue_v(b0, b1);
                wait_loads<8>();
            } else {
                wait_loads<0>();
            }
            lds_barrier();                                          // the next unit's Q (and masks) are in place
        }
        asm volatile("" : "+v"(tid_m));
        if constexpr (!Lds::kFull) {
#pragma unroll
            for (int nt = 0; nt < RT; ++nt) {
                if (nt >= tiles) break;
                store_result(nt, res[nt], inv[nt]);
            }
        }
        if (u.ns > 1 && tid_m < kRows && u.r0 + tid_m < u.rows)
            *reinterpret_cast<float2 *>(part_ml + (((int64_t)u.item * Hkv + u.gkv) * max_rows + u.r0 + tid_m) * 2) = row_ml;
        if constexpr (kDirect) break;
        cur = nxt;
        have = have_next;
    }
}

template <typename T, int RT, bool kTree, bool kDirect>
static int attn_ring_slots(int cus)
{
    static int slots = 0;
    if (slots == 0) {
        int per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_ring_kernel<T, RT, kTree, kDirect>, 256, 0) != hipSuccess)
            per_cu = 1;
        const int n = cus * (per_cu > 0 ? per_cu : 1);
        slots = n < kMaxSchedW ? n : kMaxSchedW;
    }
    return slots;
}

template <typename F>
static void with_ring_instance(const AttnArgs &a, F &&f)
{
    auto with_mode = [&](auto tag, auto rt_tag) {
        if (a.direct) f(tag, rt_tag, std::false_type{}, std::true_type{});
        else if (a.parents) f(tag, rt_tag, std::true_type{}, std::false_type{});
        else f(tag, rt_tag, std::false_type{}, std::false_type{});
    };
    auto with_rt = [&](auto tag) {
        if (attn_row_tiles(a.plan.max_rows) == 3) with_mode(tag, std::integral_constant<int, 3>{});
        else with_mode(tag, std::integral_constant<int, 4>{});
    };
    if (a.dims.dtype == ADASPEC_F16) with_rt(F16{});
    else with_rt(BF16{});
}

int attn_ring_grid_slots(const AttnArgs &a, int cus)
{
    int slots = 0;
    with_ring_instance(a, [&](auto tag, auto rt, auto tree, auto direct) {
        slots = attn_ring_slots<decltype(tag), decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>(cus);
    });
    return slots;
}

hipError_t launch_attn_ring(const AttnArgs &a)
{
    const AttnPlan &p = a.plan;
    const adaspec_attn_dims &d = a.dims;
    if (a.sched_w <= 0) return hipSuccess;                          // no work item can exist
    with_ring_instance(a, [&](auto tag, auto rt, auto tree, auto direct) {
        hipLaunchKernelGGL((attn_ring_kernel<decltype(tag), decltype(rt)::value, decltype(tree)::value, decltype(direct)::value>),
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
