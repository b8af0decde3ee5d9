// Internal declarations shared by the translation units of libadaspec.so:
// workspace layouts and the launchers each kernel file exports.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/adaspec.h"

namespace adaspec {

// ---- attention workspace -------------------------------------------------
// A "work item" is one (request, KV split); splits of a request have equal
// length (a multiple of the kernel's token block).  Items are stored densely
// in request order; the plan kernel builds the list on the device because the
// context lengths live there.
struct AttnPlan {
    int   split_tokens;     // S: maximum tokens per split
    int   block_tokens;     // split lengths are rounded up to a multiple of this
    int   max_items;        // host-side bound on the number of work items
    int   max_rows;         // (max_spec_len + 1) * G
    // byte offsets into the workspace
    size_t off_header;      // int32[16]: [0] n_items, [1] order of the static schedule, [2] its rounds
    size_t off_cu_q;        // int32[B + 1]
    size_t off_split_base;  // int32[B + 1]: first item of each request
    size_t off_item_req;    // int32[max_items]
    size_t off_item_order;  // int32[max_items]: items sorted by decreasing length (schedule order)
    size_t off_unit_meta;   // int32[max_items][8] in schedule order: request, split, n_splits, L, n, cu_q, item, 0
    size_t off_row_rec;     // int32[TQ][4] per query row: request, n_splits, first split, row base (j * G)
    size_t off_sched;       // int32[rounds][W]: unit taken by workgroup w in each round, or -1 (matrix-core kernels; row 0 is not
                            // read, and only the general plan kernel writes it)
    size_t off_anc;         // uint64[TQ]: tree verification only, ancestor-or-self mask of each query row's node
    size_t off_part_ml;     // float[max_items][Hkv][max_rows][2]  (m in log2 units, l)
    size_t off_part_o;      // float[max_items][Hkv][max_rows][d]
    size_t off_flags;       // uint64[units][4]: direct calls that merge their splits in the kernel (attn_mfma_common.h)
    size_t total_bytes;
    bool direct;            // small chain calls: one workgroup per possible unit, no metadata kernel (attn_mfma_common.h)
    int per_req;            // possible splits per request: ceil(max_pages_per_req * page_size / split_tokens)
    bool row_split;         // more than 32 rows per kv head: attn_rows.hip instead of attn_ring.hip (api.hip)
    bool merged;            // direct, and whoever finishes a request's last split merges them: no combine kernel
};

// Direct calls whose requests can have up to so many splits merge them in the kernel (attn_mfma_common.h), units of so many
// channels and row tiles: see make_attn_plan.
constexpr int kMergeMaxSplits = 4;
constexpr bool attn_merge_fits(int head_dim, int row_tiles) { return row_tiles * head_dim <= 128; }

// What a kernel of a direct call needs to find its unit by itself.
struct DirectArgs {
    const int32_t *ctx_lens, *spec_lens;
    int batch, max_spec_len, total_q, per_req, split_tokens;
    unsigned long long *flags, mark;    // splits merged in the kernel, else null: a word per unit and wavefront; what this launch leaves there
};

// Length of every split of a request with L cached tokens cut into ns splits.
__host__ __device__ inline int split_len_of(int L, int ns, int block_tokens)
{
    const int per = (L + ns - 1) / ns;
    return (per + block_tokens - 1) / block_tokens * block_tokens;
}

// Matrix-core kernels: 16-row query tiles one unit holds and units per (item, kv head).  Up to 32 rows per
// kv head: 1 or 2 tiles (head_dim 128: attn_mfma.hip); up to 48: 3; more: groups of 4 tiles (attn_ring.hip, attn_rows.hip).  The head_dim 64
// and fp32 kernels use 4 tiles for 3.
inline int attn_row_tiles(int max_rows)
{
    return max_rows <= 16 ? 1 : max_rows <= 32 ? 2 : max_rows <= 48 ? 3 : 4;
}
inline int attn_row_groups(int max_rows)
{
    const int r = 16 * attn_row_tiles(max_rows);
    return max_rows > r ? (max_rows + r - 1) / r : 1;
}

// Schedule of the matrix-core kernels: which unit (in the order of decreasing length) workgroup w of W takes in a round that
// is not balanced by accumulated work.  What has to be even is the work per COMPUTE UNIT: workgroups w, w + cus, w + 2 cus,
// ... land on the same one (the dispatcher fills the compute units in order, one workgroup each, then starts over), share
// its load pipeline, and are done when their total is done.  Orders (sched_order chooses, the header carries):
//
// kSchedEven, up to four rounds (two for the row split): a round is cut into sub-rounds of `cus` workgroups, each of which runs through its units
// forwards or backwards.  Directions by the parity of the bits of the sub-round's number (backwards, forwards, forwards,
// backwards, ...): four sub-rounds then even out a convex distribution of lengths as well as a linear one, which strict
// alternation does not; the first runs backwards, so that where the second is not full its long units land beside the shortest
// ones of the first.  Fullest compute unit over the mean, whole rounds in turn / this way: 64 requests of 1024-2048 tokens, 8
// kv heads (512 units for 512 workgroups) 1.15 / 1.00, main kernel 69.6 / 65.4 us; 64 log-normal ones of 128-4096 1.23 / 1.13,
// 64.3 / 60.8 us.
//
// n > 0: two sub-rounds, and n compute units take a third unit in a second round.  On top of even totals that would be streamed
// by those few alone at the end: they take the shortest units for their first two, the others pairs of the longest.  Captured
// calls, whole rounds in turn / even / this way: 270 requests of 500-1500 tokens, 2 kv heads (540 units) 57.6 / 60.5 / 55.4 us, 300
// (600) 60.8 / 64.4 / 60.5, 67 of 1000-1900, 8 kv heads (536) 81.3 / 84.4 / 75.1.  Skewed lengths stay even: pairs of the longest
// would be the longest by far (175 log-normal ones of 128-2000, 4 kv heads 64.3 / 59.0 / 70.9).
//
// kSchedRounds, more rounds: whole rounds in turn, forwards and backwards (300 requests of 100-500, 8 kv heads of 64, five
// rounds: main kernel 41.1 us, even 41.8; three and four rounds gain 3 % from even ones where lengths are skewed, but not in the
// row split, 300 trees of 512-1024, 56 rows: 106 us, even 109).  Also instead of
// thirds where units have several row groups and are not listed by their work (300 trees of 48-96, 128 rows: 12.4 us, thirds 13.0).
constexpr int kSchedEven = 0, kSchedRounds = -1;
constexpr int kEvenRounds = 4, kEvenRoundsRowSplit = 2;
// (in workgroup c of sub-round `sub`; n_sub = sub-rounds per round)
__host__ __device__ inline int sched_position_in(int round, int sub, int c, int n_sub, int W, int cus, int order)
{
    const int base = sub * cus, w = base + c;
    if (order == kSchedRounds) return round * W + ((round & 1) ? W - 1 - w : w);
    if (order > 0 && round == 0) {
        const int two = cus - order;                                // compute units with two units
        if (c < order) return sub == 0 ? W - 1 - c : 2 * two + c;   // (the third goes to workgroup c: behind the shorter one)
        return sub == 0 ? c - order : 2 * two - 1 - (c - order);
    }
    const int width = W - base < cus ? W - base : cus;
    return round * W + base + ((__builtin_popcount(round * n_sub + sub) & 1) ? c : width - 1 - c);
}
__host__ __device__ inline int sched_position(int round, int w, int W, int cus, int order)
{
    const int sub = w / cus;
    return sched_position_in(round, sub, w - sub * cus, (W + cus - 1) / cus, W, cus, order);
}
// Order of a schedule of `total` units.  Whether some third units go on even pairs or on the shortest units follows from which
// leaves the fullest compute unit less: size[k] is the work of unit sched_sample(k) in the order of decreasing length (even
// pairs (k, W - 1 - k) looked at in both ends and in the middle, as most distributions make their sums monotonic between).
__host__ __device__ inline bool sched_asks_sizes(int total, int W, int cus) { return W == 2 * cus && total > W && total <= W + cus; }
constexpr int kSchedSamples = 9;
__host__ __device__ inline int sched_sample(int k, int total, int W, int cus)
{
    const int two = cus - (total - W);
    const int at = k == 0 ? 0 : k == 1 ? W - 1 : k == 2 ? cus / 2 : k == 3 ? W - 1 - cus / 2 : k == 4 ? cus - 1 : k == 5 ? cus
                   : k == 6 ? W : k == 7 ? 2 * two - 1 : 2 * two;
    return at < 0 ? 0 : at;
}
__host__ __device__ inline int sched_order(int total, int W, int cus, int even_rounds, const int (&size)[kSchedSamples])
{
    if (!sched_asks_sizes(total, W, cus)) return total > even_rounds * W ? kSchedRounds : kSchedEven;
    const int ends = size[0] + size[1], quarter = size[2] + size[3], middle = size[4] + size[5];
    const int most = ends > quarter ? (ends > middle ? ends : middle) : (quarter > middle ? quarter : middle);
    const int least = ends < quarter ? (ends < middle ? ends : middle) : (quarter < middle ? quarter : middle);
    const int even = most > least + size[6] ? most : least + size[6];
    const int pair = total < W + cus ? size[0] + size[7] : 0, three = size[8] + size[1] + size[6];
    return even > (pair > three ? pair : three) ? total - W : kSchedEven;
}

// Which kernel family a call takes.  ADASPEC_PATH_FAST names the head_dim 128 form; AUTO also reaches the others.
enum class AttnKind { kVector, kMfma128, kMfma64, kMfmaF32 };
constexpr int kAttnD64Block = 64;   // tokens per block of the head_dim 64 form (attn_d64.hip)
AttnKind attn_kind(const adaspec_attn_dims &d);
AttnPlan make_attn_plan(const adaspec_attn_dims &d, AttnKind kind, bool tree);
bool attn_fast_path_supported(const adaspec_attn_dims &d);

struct AttnArgs {
    const void *q, *k_pages, *v_pages;
    const int32_t *block_table, *ctx_lens, *spec_lens;
    const int32_t *parents = nullptr;   // tree verification: parent node of every query row, else NULL
    void *out;
    adaspec_attn_dims dims;
    float scale_log2;       // scale * log2(e)
    AttnPlan plan;
    char *ws;
    hipStream_t stream;
    // launch shape of the matrix-core kernel (attn_mfma_shape); sched_w = 0 on the vector path
    int sched_w = 0;          // W: workgroups of the launch = columns of the schedule table
    int sched_cus = 1;        // compute units of the device
    int n_row_groups = 1;     // units per (item, kv head)
    int rows_per_group = 16;  // query rows (times G) one unit covers
    bool direct = false;      // plan.direct
};

DirectArgs direct_args(const AttnArgs &a);      // (api.hip; every call gives another mark)
uint64_t next_spread_mark();                    // the same, spread over the 64 bits; never 0

// Upper bound on W for which the workspace holds a schedule table.
constexpr int kMaxSchedW = 1024;
constexpr int64_t kMaxAttnItems = (int64_t)1 << 24;   // (request, split) work items of one attention call

// Fills sched_w / n_row_groups / rows_per_group for the matrix-core kernel's launch of a.dims.
void attn_mfma_shape(AttnArgs &a, AttnKind kind);

hipError_t launch_attn_plan(const AttnArgs &a);
// tree verification: ancestor masks of all query rows (after the plan kernel: it reads cu_q)
hipError_t launch_tree_masks(const AttnArgs &a);
hipError_t launch_attn_vector(const AttnArgs &a);
hipError_t launch_attn_mfma(const AttnArgs &a);
// units of more than 32 rows (attn_ring.hip, or attn_rows.hip where plan.row_split); launch_attn_mfma forwards to them
constexpr int kRingQRows = 65;          // query rows that the (query row, head) rows of one of its units span at most
hipError_t launch_attn_ring(const AttnArgs &a);
int attn_ring_grid_slots(const AttnArgs &a, int cus);   // resident workgroups = columns of the schedule table
hipError_t launch_attn_rows(const AttnArgs &a);
int attn_rows_grid_slots(const AttnArgs &a, int cus);
// head_dim 64 (attn_d64.hip)
hipError_t launch_attn_d64(const AttnArgs &a);
int attn_d64_grid_slots(const AttnArgs &a, int cus);
// fp32, head_dim 64 or 128 (attn_f32.hip)
hipError_t launch_attn_f32(const AttnArgs &a);
int attn_f32_grid_slots(const AttnArgs &a, int cus);
hipError_t launch_attn_combine(const AttnArgs &a);
int attn_combine_waves(const AttnPlan &p, const adaspec_attn_dims &d);   // wavefronts per (row, head) of the combine kernel

// ---- accept workspace ------------------------------------------------------
struct AcceptPlan {
    size_t off_cu_q;        // int32[B + 1]
    size_t off_row_req;     // int32[TQ]
    size_t off_row_flag;    // int32[TQ]  1 = accepted (or bonus row)
    size_t off_row_cand;    // int32[TQ]  token to emit if the request stops at this row
    size_t off_row_meta;    // int32[TQ][8]: request, position j, k, draft token, temperature bits, draft row
    // two-pass form
    size_t off_row_stat;    // RowStat[TQ]: (m, Z) of the sampled draft rows, from the first pass (one workgroup per row)
    size_t off_req_ticket;  // int32[B]: workgroups of the second pass that have finished, per request
    size_t off_slot_rec;    // int32[B * max_spec_len][4] per (request, draft position): token, its logit, its draft
                            // probability, the accept uniform (form in parts)
    size_t off_part_stat;   // HalfStat[B * max_spec_len][8]: (maximum, normaliser | arg-max) of each part of a draft row
    size_t off_half_stat;   // HalfStat[B][parts]: per part of the deciding row
    size_t off_part;        // WaveMass[B][parts][4]: masses of the deciding rows, per wavefront of a part; or, where a few workgroups share
                            // the row (accept_shared.hip), PartWords[B][their parts]
    bool parts;             // the workspace holds what the form in parts needs
    size_t off_tree_stat;   // tree acceptance, last: per-node statistics (tree_node_stat_bytes() each)
    size_t total_bytes;
    size_t noalloc_bytes;   // what adaspec_accept_noalloc's limit is compared with
};
// p_v = 2^((l_v - m) c) / Z of a row (first pass of the two-pass form -> second pass)
struct RowStat { float m; float pad; double Z; };
// per part of a row: (m, Z) the part's sums are relative to; for a greedy row (maximum, arg-max or -1)
struct HalfStat { float m; int arg; double Z; };
AcceptPlan make_accept_plan(const adaspec_accept_dims &d);
bool accept_fast_path_supported(const adaspec_accept_dims &d, const void *logits, const void *probs);

struct AcceptArgs {
    const void *logits, *probs;
    const int32_t *draft_tokens;
    const float *uniforms;
    const int32_t *spec_lens;
    const float *temperature;
    int32_t *out_tokens, *out_accept_len;
    adaspec_accept_dims dims;
    AcceptPlan plan;
    char *ws;
    hipStream_t stream;
};

hipError_t launch_accept_plan(const AcceptArgs &a);
hipError_t launch_accept_vector(const AcceptArgs &a);
hipError_t launch_accept_fast(const AcceptArgs &a);
hipError_t launch_accept_emit(const AcceptArgs &a);
bool accept_stream_path_supported(const adaspec_accept_dims &d, const void *logits, const void *probs);
hipError_t launch_accept_stream(const AcceptArgs &a);
// two-pass form: flags of the draft rows, then one workgroup per request (sampling + outputs)
hipError_t launch_accept_test(const AcceptArgs &a);
hipError_t launch_accept_resolve(const AcceptArgs &a);
// two-pass form with every row cut into parts (accept_parts.hip): up to 1024 requests.  Whether a call can take it is
// decided by its dims alone (plan.parts) and the alignment of its rows.
bool accept_parts_dims_fit(const adaspec_accept_dims &d);
size_t accept_parts_slot_bytes(const adaspec_accept_dims &d);
size_t accept_parts_stat_bytes(const adaspec_accept_dims &d);
size_t accept_parts_sum_bytes(const adaspec_accept_dims &d);
size_t accept_parts_sum_stat_bytes(const adaspec_accept_dims &d);
hipError_t launch_accept_parts(const AcceptArgs &a, int compute_units);

// tree verification (tree.hip, tree_fast.hip): every node's acceptance, then the walk; needs the accept plan's cu_q / row_req
// portable form (any types and sizes): a per-node kernel writes (next node or -1, token if the walk stops here)
// into row_flag / row_cand, a small kernel walks them
hipError_t launch_accept_tree_nodes(const AcceptArgs &a, const int32_t *parents);
// 16-bit rows (shapes of the streaming chain kernel): node statistics, then one workgroup per request, or a few that share
// its rows, walks its tree and writes the outputs (no separate walk kernel)
size_t tree_node_stat_bytes(int vocab);
constexpr size_t kTreeNodeStatMin = 528;
bool tree_fast_needs_plan(const adaspec_accept_dims &d);   // large batches: row offsets from launch_accept_plan
hipError_t launch_accept_tree_fast(const AcceptArgs &a, const int32_t *parents, int compute_units, int32_t *out_path);
hipError_t launch_accept_tree_walk(const AcceptArgs &a, int32_t *out_path);
hipError_t launch_kv_compact_path(void *k_pages, void *v_pages, const int32_t *block_table,
                                  const int32_t *ctx_lens, const int32_t *spec_lens,
                                  const int32_t *out_path, const int32_t *out_accept_len,
                                  const adaspec_attn_dims &d, int path_stride, hipStream_t stream);

hipError_t launch_check_accept_inputs(const int32_t *draft_tokens, const int32_t *spec_lens, const float *temperature,
                                      const adaspec_accept_dims &d, int32_t *err_flags, hipStream_t stream);
hipError_t launch_check_tree_parents(const int32_t *parents, const int32_t *spec_lens, int B, int total_q,
                                     int max_spec_len, int32_t *err_flags, hipStream_t stream);
hipError_t launch_check_ragged(const int32_t *block_table, const int32_t *ctx_lens,
                               const int32_t *spec_lens, const adaspec_attn_dims &d,
                               int32_t *err_flags, hipStream_t stream);

bool draft_sample_supported(const adaspec_draft_dims &d, const void *logits, const void *probs);
hipError_t launch_draft_sample(const void *logits, const float *temperature, const float *uniforms,
                               const int32_t *out_rows, void *probs, int32_t *tokens, float *confidence,
                               const adaspec_draft_dims &d, hipStream_t stream);
bool draft_fast_supported(const adaspec_draft_dims &d);
// rows shared by workgroups, one kernel (draft_parts.hip)
bool draft_parts_supported(const adaspec_draft_dims &d);
size_t draft_parts_workspace_bytes(const adaspec_draft_dims &d);
hipError_t launch_draft_parts(const void *logits, const float *temperature, const float *uniforms,
                              const int32_t *out_rows, void *probs, int32_t *tokens, float *confidence,
                              const adaspec_draft_dims &d, char *ws, int compute_units, hipStream_t stream);
hipError_t launch_draft_fast(const void *logits, const float *temperature, const float *uniforms,
                             const int32_t *out_rows, void *probs, int32_t *tokens, float *confidence,
                             const adaspec_draft_dims &d, hipStream_t stream);
hipError_t launch_kv_append(const void *k_new, const void *v_new, void *k_pages, void *v_pages,
                            const int32_t *block_table, const int32_t *ctx_lens,
                            const int32_t *spec_lens, const adaspec_attn_dims &d, hipStream_t stream);
hipError_t launch_commit(const int32_t *out_tokens, const int32_t *out_accept_len,
                         const int32_t *spec_lens, const int32_t *ctx_lens,
                         const int32_t *next_spec_lens, int32_t *committed_lens,
                         int32_t *next_ctx_lens, int32_t *last_token, int32_t *seq_tokens,
                         int32_t *seq_lens, const adaspec_commit_dims &d, hipStream_t stream);

}  // namespace adaspec
