// What the first pass of the acceptance in row parts (accept_parts.hip) leaves, and how a second pass finds a request's deciding row
// from it.
#pragma once
#include "adaspec_internal.h"
#include "device_utils.h"
#include "row_parts.h"

namespace adaspec {

// what part 0 of a draft row leaves for the accept test
struct SlotRec { int x; uint32_t lx_bits, qx_bits, u0_bits; };

// (m, Z) of a whole row from its parts' records, or for a greedy request (maximum, arg-max)
struct RowMerge { float m; double Z; int arg; };
__device__ __forceinline__ void load_row_parts(const HalfStat *__restrict__ st, int n_parts, HalfStat (&s)[kStatParts])
{
#pragma unroll
    for (int p = 0; p < kStatParts; ++p) {
        s[p].m = -INFINITY; s[p].arg = -1; s[p].Z = 0.0;
        if (p < n_parts) s[p] = st[p];
    }
}
template <class LT>
__device__ __forceinline__ RowMerge merge_row_parts(const HalfStat (&s)[kStatParts], float c, bool greedy)
{
    RowMerge out;
    out.Z = 0.0; out.arg = 0;
    if (greedy) {
        ArgMax b{-INFINITY, 0x7fffffff};
#pragma unroll
        for (int p = 0; p < kStatParts; ++p)
            if (s[p].arg >= 0) b = argmax_merge(b, ArgMax{s[p].m, s[p].arg});
        out.m = b.v;
        out.arg = b.i == 0x7fffffff ? 0 : b.i;
        return out;
    }
    float m = s[0].m;
#pragma unroll
    for (int p = 1; p < kStatParts; ++p) m = fmaxf(m, s[p].m);
#pragma unroll
    for (int p = 0; p < kStatParts; ++p)
        out.Z += s[p].m > -INFINITY ? s[p].Z * (double)__builtin_amdgcn_exp2f(ref_gap<LT>(s[p].m, m, c)) : 0.0;
    out.m = m;
    return out;
}

// Second pass for fp32 logits and short rows (accept_shared.hip): parts of the deciding rows, chunks per thread in each, words per request that the
// first pass clears where the plan has off_part.
struct SharedParts { int n_parts, part_steps, n_words; };
SharedParts accept_shared_parts(const adaspec_accept_dims &d, int compute_units);
void launch_accept_shared(const AcceptArgs &a, const SharedParts &p, int n_stat_parts);

// A request's deciding row: its first rejected draft, or the bonus row (a == k).  Every thread of the workgroup calls it; the
// decision is wavefront 0's.
struct DecidingScratch { int a; float m; int arg; double Z; };
struct DecidingRow {
    int start, k;           // first logits row, drafts
    bool sampled;
    float c;                // log2(e) / T
    int a;                  // position of the deciding row
    RowMerge row;           // its statistics, if it is a draft's
};
template <class LT>
__device__ __forceinline__ DecidingRow deciding_row(DecidingScratch &s, int i, const int32_t *__restrict__ cu_q,
                                                    const int32_t *__restrict__ spec_lens, const float *__restrict__ temperature,
                                                    const SlotRec *__restrict__ slot_rec, const HalfStat *__restrict__ part_stat,
                                                    int max_spec_len, int n_stat_parts, int lane, int wv)
{
    DecidingRow out;
    // ---- the request's first rejected draft: wavefront 0 decides, one lane per draft --------------------
    // The records of the request's first 64 slots are requested before anything else: they need neither
    // the draft count nor the row offset (slots beyond the count hold leftovers, which are not looked at).
    // Requested this early they are back before the first workgroups of the launch start streaming rows;
    // later they would queue behind that traffic.
    SlotRec rec;
    HalfStat parts[kStatParts];
    rec.x = 0; rec.lx_bits = rec.qx_bits = rec.u0_bits = 0;
    if (wv == 0 && lane < max_spec_len) {
        const int64_t slot = (int64_t)i * max_spec_len + lane;
        rec = slot_rec[slot];
        load_row_parts(part_stat + slot * kStatParts, n_stat_parts, parts);
    }
    out.start = cu_q[i];
    const int k = out.k = min(max(spec_lens[i], 0), max_spec_len);          // uniform: scalar loads
    const float T = temperature[i];
    const bool sampled = out.sampled = T != 0.0f;
    const float c = out.c = sampled ? exponent_scale<LT>(T) : 0.f;
    if (wv == 0) {
        int a0 = k;
        RowMerge row0;                                               // statistics of the deciding row, if a draft
        row0.m = 0.f; row0.Z = 1.0; row0.arg = 0;
        for (int j0 = 0; j0 < k; j0 += kWave) {
            const int jj = j0 + lane;
            int flag = 1;
            RowMerge mine;
            mine.m = 0.f; mine.Z = 1.0; mine.arg = 0;
            if (jj < k) {
                if (j0 > 0) {                                        // more drafts than lanes: the next 64 slots
                    const int64_t slot = (int64_t)i * max_spec_len + jj;
                    rec = slot_rec[slot];
                    load_row_parts(part_stat + slot * kStatParts, n_stat_parts, parts);
                }
                mine = merge_row_parts<LT>(parts, c, !sampled);
                if (sampled) {
                    const float lx = __uint_as_float(rec.lx_bits), qx = __uint_as_float(rec.qx_bits);
                    const float px = exp_weight<LT>(lx, mine.m, c, scaled_ref(mine.m, c)) * (float)(1.0 / mine.Z);
                    flag = (qx > 0.f) ? (__uint_as_float(rec.u0_bits) < px / qx) : 1;
                } else {
                    flag = rec.x == mine.arg;
                }
            }
            const unsigned long long rej = __ballot(flag == 0);
            if (rej) {
                const int src = (int)__builtin_ctzll(rej);
                a0 = j0 + src;
                row0.m = __shfl(mine.m, src, kWave);
                row0.Z = __shfl(mine.Z, src, kWave);
                row0.arg = __shfl(mine.arg, src, kWave);
                break;
            }
        }
        if (lane == 0) { s.a = a0; s.m = row0.m; s.arg = row0.arg; s.Z = row0.Z; }
    }
    lds_barrier();
    out.row.m = s.m; out.row.arg = s.arg; out.row.Z = s.Z;
    out.a = __builtin_amdgcn_readfirstlane(s.a);
    return out;
}

}  // namespace adaspec
