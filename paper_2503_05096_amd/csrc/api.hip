// C ABI entry points of libadaspec.so: host-side validation, workspace layout
// and the launch sequence of each call.  The entry points that enqueue work make
// no HIP call before their arguments have been validated, so their error paths
// work on a machine with no GPU (adaspec_accept_resolved_path asks the device for
// its compute-unit count; without a device it assumes 256).
#include <math.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <random>

#include "adaspec_internal.h"
#include "device_utils.h"

namespace adaspec {

// the optional event pair of a dims struct: recorded only if both are given
static bool record_event(void *start, void *stop, bool first, hipStream_t stream)
{
    if (!start || !stop) return true;
    return hipEventRecord(static_cast<hipEvent_t>(first ? start : stop), stream) == hipSuccess;
}

// ---- scratch memory of adaspec_accept_noalloc ------------------------------------------------------
// A file-scope device array stands in for the workspace argument: every GPU the library runs on holds
// its own copy, at its own address, until the process ends.  In host code the NAME of the array is
// only a handle for hipGetSymbolAddress; the device address it yields (looked up once per device,
// with that device current) is what kernels, and anything else that touches the memory, are given.
constexpr size_t kNoallocScratchBytes = ADASPEC_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mutex;

// device address of `scratch` on the current device (ADASPEC_OK), or a negative status
static int noalloc_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return ADASPEC_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return ADASPEC_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ADASPEC_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ADASPEC_OK;
}

// compute units of the current device (asked once; 256 if the runtime cannot tell)
static int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus = n;
        else
            cus = 256;
    }
    return cus;
}

static bool dtype_ok(int dt) { return dt == ADASPEC_F32 || dt == ADASPEC_F16 || dt == ADASPEC_BF16; }
static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static int validate_attn_dims(const adaspec_attn_dims *d)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->batch < 0 || d->total_q < d->batch || d->max_spec_len < 0) return ADASPEC_ERR_DIM;
    if ((int64_t)d->total_q > (int64_t)d->batch * (d->max_spec_len + 1)) return ADASPEC_ERR_DIM;
    if (d->n_q_heads <= 0 || d->n_kv_heads <= 0 || d->n_q_heads % d->n_kv_heads) return ADASPEC_ERR_DIM;
    if (d->num_pages <= 0 || d->max_pages_per_req <= 0) return ADASPEC_ERR_DIM;
    if (d->head_dim <= 0) return ADASPEC_ERR_DIM;
    if (!dtype_ok(d->dtype) || !dtype_ok(d->out_dtype)) return ADASPEC_ERR_DTYPE;
    if (d->out_dtype != d->dtype && d->out_dtype != ADASPEC_F32) return ADASPEC_ERR_DTYPE;
    if (d->page_size != 16) return ADASPEC_ERR_UNSUPPORTED;
    if (d->head_dim % 8 || d->head_dim > 256) return ADASPEC_ERR_UNSUPPORTED;
    if (d->path < ADASPEC_PATH_AUTO || d->path > ADASPEC_PATH_FAST) return ADASPEC_ERR_DIM;
    if (!(d->scale >= 0.0f) || isinf(d->scale)) return ADASPEC_ERR_DIM;
    if (d->path == ADASPEC_PATH_FAST && !attn_fast_path_supported(*d)) return ADASPEC_ERR_UNSUPPORTED;
    if (d->plan_mode < ADASPEC_PLAN_BUILD_AND_RUN || d->plan_mode > ADASPEC_PLAN_REUSE) return ADASPEC_ERR_DIM;
    {   // the kernels count work items and units in 32 bits: bound them at the shortest split (256 tokens)
        const int64_t per_req = ((int64_t)d->max_pages_per_req * d->page_size + 255) / 256;
        const int64_t items = (int64_t)d->batch * per_req;
        const int64_t rows = (int64_t)(d->max_spec_len + 1) * (d->n_q_heads / d->n_kv_heads);
        if (rows > (1 << 20) || items > kMaxAttnItems ||
            items * d->n_kv_heads * attn_row_groups((int)rows) >= (int64_t)1 << 31)
            return ADASPEC_ERR_UNSUPPORTED;
    }
    return ADASPEC_OK;
}

// Direct calls (no metadata kernel): at most this many requests (the combine kernel finds a row's request with one scan
// of four per lane) and possible units.  Up to one unit per compute unit there is nothing to balance; with 512 units of
// many requests the schedule, which pairs long and short units on a compute unit, is worth its kernel (64 requests of
// 1024-2048 tokens, 8 kv heads: 79.5 us per layer with it, 82.9 us direct), with 512 of a few requests it is not.
constexpr int kDirectMaxBatch = 256;
constexpr int kDirectMaxUnits = 256, kDirectFewPairs = 128, kDirectMaxUnitsFew = 512;
constexpr int kDirectShortCtx = 512, kDirectLongestShort = 1024, kDirectShortBatch = 1024;
constexpr int kDirectF32Tokens = 262144, kDirectRowsTokens = 262144, kDirectRingTokens = 1048576;   // possible tokens of all units
constexpr int kWavesPerUnit = 4;

AttnKind attn_kind(const adaspec_attn_dims &d)
{
    if (d.path == ADASPEC_PATH_VECTOR) return AttnKind::kVector;
    if (attn_fast_path_supported(d)) return AttnKind::kMfma128;
    // head_dim 64 in 16 bits: the vector kernel is never ahead (MI355X, whole call, bf16, 32/8 heads: 64 requests of
    // 256-4096 tokens 1024 us against 65 us) and its fp32 accumulator is further from 64 bits (3.4e-7 against 2.4e-7)
    if (d.dtype != ADASPEC_F32 && d.head_dim == 64) return AttnKind::kMfma64;
    // fp32 at these head dims: likewise (4 requests of 128-512 tokens, 8 heads of 64: 109 us against 10 us;
    // error against 64 bits 3.7e-7 against 2.1e-7)
    if (d.dtype == ADASPEC_F32 && (d.head_dim == 64 || d.head_dim == 128)) return AttnKind::kMfmaF32;
    return AttnKind::kVector;
}

// More than 32 rows per kv head (16 bits, head_dim 128): the kernel whose wavefronts split the rows (attn_rows.hip) or the
// one whose wavefronts split the tokens (attn_ring.hip).  A unit of a few blocks gives the ring's wavefronts a block each, or
// none, all row tiles of it one after the other, and a merge behind; a unit of many blocks gives the row split a barrier per
// block.  `tokens`: a split of the longest possible request.  The line moves with the number of row tiles and groups (four
// tiles: a longer chain in the ring), with units > 256, where two workgroups share a compute unit, and for trees, whose masks the
// ring with four tiles reads from memory.  MI355X, captured calls, bf16, row split / ring:
//   3 tiles, 64/8 heads, 8 requests of 16-32 tokens 6.0 / 7.2 us, 32-64 6.9 / 7.8, 48-96 7.8 / 8.1, 64-128 8.7 / 8.3, 128-256
//   11.9 / 10.0; 64 of 96-192 14.2 / 15.3, 128-256 16.3 / 16.6; trees, 64 of 128-256 19.8 / 21.5, 256-512 28.0 / 28.3
//   4 tiles, 64/8 heads, 8 requests of 16-32 6.3 / 8.4, 64-128 9.0 / 9.3, 96-192 10.2 / 11.4, 128-256 12.2 / 11.7; 64 of 128-256
//   17.2 / 19.0, 256-512 26.3 / 27.3, 300-600 32.2 / 30.5; trees, 64 of 300-600 32.4 / 34.4, 500-1000 45.3 / 45.8, 128 of 500-1000
//   82.4 / 84.4, 1000-2000 145.7 / 144.7
//   two groups of 4 (72 rows), 64/8 heads, 32 of 128-256 16.3 / 18.0, 256-512 24.4 / 24.5; 250 of 128-256 84.3 / 99.1
// Requests of several splits have units of any length up to the whole split, so only one or two of them are safe to judge by
// the longest: 1 of 288 tokens, 56 rows 12.8 / 14.6, 2 of 375 and 525 13.9 / 15.0, 4 of up to 288 15.6 / 14.9.
static bool rows_split_wins(int tiles, int groups, bool tree, int batch, int64_t units, int64_t per_req, int64_t tokens)
{
    const bool four = tiles > 3, single = groups == 1;
    if (per_req > 1) {
        if (!single && !tree && units > 256 && units <= 512) return tokens <= 256;      // (8 of 300-600, 72 rows: 18.7 / 20.0)
        return four ? batch <= 2 && tokens <= 224 : batch == 1 && tokens <= 160;
    }
    // beyond this many tokens chains in one group are direct calls with the ring only (below), which is ahead of the row split
    // with its schedule (250 of 96-192, 8 kv heads, 3 tiles 51.6 / 46.5; in two groups, whose second is mostly empty, 73.9 / 92.1)
    if (!tree && single && units * tokens > kDirectRowsTokens) return false;
    if (units <= 256) return tokens <= (four ? (tree ? 320 : 192) : (tree ? 128 : 96));
    if (units <= 512) return tokens <= (!four ? (tree ? 416 : 192) : single ? (tree ? 768 : 512) : (tree ? 512 : 416));
    return tokens <= (!four ? (tree ? 128 : 96) : single ? (tree ? 1024 : 192) : (tree ? 512 : 320));
}

AttnPlan make_attn_plan(const adaspec_attn_dims &d, AttnKind kind, bool tree)
{
    AttnPlan p;
    const int G = d.n_q_heads / d.n_kv_heads;
    const bool scheduled = kind != AttnKind::kVector;      // units handed out by the schedule table
    // The matrix-core kernel runs 4 wavefronts per work item, each over up to 256
    // tokens, and merges them on chip; the vector kernel runs one wavefront per
    // item.  With few (request, kv head) pairs the splits are shortened so that
    // the chip still sees enough independent items.
    const int64_t pairs = (int64_t)d.batch * d.n_kv_heads;
    p.max_rows = (d.max_spec_len + 1) * G;
    const bool many_rows = kind == AttnKind::kMfma128 && attn_row_tiles(p.max_rows) > 2;
    if (scheduled) {
        p.block_tokens = kind == AttnKind::kMfma64 ? kAttnD64Block : (kind == AttnKind::kMfmaF32 ? 16 : 32);
        p.split_tokens = pairs >= 256 ? 2048 : (pairs >= 128 ? 1024 : (pairs >= 32 ? 512 : 256));
    } else {
        p.block_tokens = 64;
        p.split_tokens = 256;
    }
    const int64_t max_ctx = (int64_t)d.max_pages_per_req * d.page_size;
    p.direct = false;
    const int n_groups = attn_row_groups(p.max_rows);
    auto row_split = [&]() -> bool {                        // (with the splits of now)
        const int64_t per_req = (max_ctx + p.split_tokens - 1) / p.split_tokens, even = (max_ctx + per_req - 1) / per_req;
        // the ring finds a unit's Q by 32-bit offsets from its first row, the row split by addresses
        const int64_t q_rows = d.max_spec_len + 1 < kRingQRows ? d.max_spec_len + 1 : kRingQRows;
        if (many_rows && q_rows * d.n_q_heads * d.head_dim * 2 > UINT32_MAX) return true;
        return many_rows && rows_split_wins(attn_row_tiles(p.max_rows), n_groups, tree, d.batch, pairs * n_groups * per_req, per_req,
                                            (even + p.block_tokens - 1) / p.block_tokens * p.block_tokens);
    };
    if (scheduled && !tree && d.batch <= kDirectMaxBatch) {
        // Small batches: the shortest split (two blocks per wavefront or more: with one, the workspace and the work of the
        // combine double and the call gets no faster) with which every possible unit has a compute unit of its own, or half
        // of one where there are few (request, kv head) pairs.  Such a call needs no metadata kernel.  What is possible
        // follows from the width of the block table, which a server makes as wide as its longest request: it must not
        // decide how coarsely contexts are cut, so the split is never longer than the one above (or those two blocks); longer
        // ones also sum longer in fp32 (one request of 64000 tokens in f16: error of the output 1.79e-4, 2.05e-4 in splits of
        // 2048).
        // MI355X, one request of 1500 tokens, 6 rows, 32/8 heads of 128, tables of 1.5K / 16K / 32K / 64K tokens: 11.2 /
        // 11.1 / 15.4 / 15.4 us (metadata first: 17.2; splits of up to 2048 to stay direct: 11.2 / 13.2 / 15.1 / 20.5);
        // 16000 tokens under 16K: 22.6 (35.1 with metadata).  With 1024 possible units for few pairs full tables lose
        // (4 requests of 8000 under 8K: 30.2 -> 39.3).
        const int shortest = 2 * kWavesPerUnit * p.block_tokens, longest = p.split_tokens > shortest ? p.split_tokens : shortest;
        // (two units side by side on a compute unit: not with four row tiles in one wavefront's registers; 48 requests of 850
        // tokens, 49 rows, 14/2 heads of 64, under 1800: 29.9 us with 384 possible units, 21.8 with the schedule)
        const bool one_per_cu = kind != AttnKind::kMfma128 && attn_row_tiles(p.max_rows) > 2;
        const int most = pairs < kDirectFewPairs && !one_per_cu ? kDirectMaxUnitsFew : kDirectMaxUnits;
        for (int s = shortest; s <= longest && !p.direct; s *= 2)
            if (d.batch * ((max_ctx + s - 1) / s) * d.n_kv_heads * n_groups <= most) {
                p.direct = true;
                p.split_tokens = s;
            }
    }
    if (scheduled && !tree && !p.direct && max_ctx <= p.split_tokens && max_ctx <= kDirectLongestShort && d.batch <= kDirectShortBatch) {
        // Short contexts: every request is one unit per kv head (no combine), all of them about equally short.  Measured
        // with and without (MI355X, 32/8 heads of 128, bf16): 256 requests of 100-500 tokens 62.6 / 65.5 us, 126 of 119-185
        // 14.0 / 18.5, 64 of 512-1000 39.5 / 42.3, 128 of 256-1000 64.6 / 63.4 (left to the schedule).  The
        // kernels of more than 32 rows and the fp32 kernel lose more by not loading across unit boundaries, and gain as much where
        // units are few: up to 4096 possible tokens per compute unit (ring), 1024 (the others; row split, 72 rows, 200 of 100-400
        // 104 / 87; ring, 64/8 heads, direct / scheduled: 100 of 50-300 tokens, 48 rows
        // 25.5 / 30.8, 64 of 300-1000 37.4 / 39.6, of 400-1000, 40 rows 38.2 / 41.5, 200 of 20-120 30.6 / 37.2).
        const int64_t units = pairs * n_groups;
        const int64_t deep = kind == AttnKind::kMfmaF32 ? kDirectF32Tokens : !many_rows ? 0 : row_split() ? kDirectRowsTokens : kDirectRingTokens;
        p.direct = deep ? units * max_ctx <= deep : units <= (max_ctx <= kDirectShortCtx ? 8192 : 512);
    }
    const int64_t per_req = (max_ctx + p.split_tokens - 1) / p.split_tokens;
    p.per_req = (int)per_req;
    p.row_split = row_split();
    // Splits merged in the kernel, not by a second one: up to 4 possible splits, of one row tile of 128 channels or two of 64.
    // What is saved is most of a launch; from a captured graph, where a launch costs less, no more than the last workgroup of a
    // request takes to read and add up the states, and the line lies where that breaks even.  MI355X, with the combine
    // kernel / merged, calls back to back; captured: 16 bits, 32/8 heads of 128, 1 request of 600 tokens, 16 rows 12.7 / 9.8; 9.4 / 9.5 us,
    // 3 of 500-1000, 8 rows 12.6 / 11.3; 11.0 / 10.9, 8 of 300-1000, 16 rows 13.1 / 12.0; 11.8 / 11.6; 8 of 500-2000, 14/2 heads of 64, 28
    // rows 13.7 / 11.7; 12.4 / 11.6, 1 of 2000, 32/8, 24 rows 13.3 / 11.8; 11.6 / 11.7; fp32, 4 of 128-512, 8/8 heads of 64 11.7 / 8.8; 8.9 /
    // 8.2, 1 of 500, 32/8 of 128, 16 rows 12.4 / 10.9; 10.4 / 10.6.  Not: two tiles of 128 channels, 1 of 600, 24 rows 12.9 / 11.8; 11.1 /
    // 11.6, 1 of 700, 32 rows 13.0 / 12.5; 11.6 / 12.3, 3 of 400-700 12.7 / 12.8; 11.8 / 12.5, fp32, 1 of 480, 32 rows 15.8 / 15.7; 14.9 / 15.5;
    // with 8 splits 1 of 2000 11.0-11.5 / 10.8-11.4; 10.6 / 11.2.
    p.merged = p.direct && per_req > 1 && per_req <= kMergeMaxSplits && attn_merge_fits(d.head_dim, attn_row_tiles(p.max_rows));
    p.max_items = (int)((int64_t)d.batch * per_req);
    size_t off = 0;
    p.off_header = off;     off = align_up(off + 16 * sizeof(int32_t), 256);
    p.off_cu_q = off;       off = align_up(off + (size_t)(d.batch + 1) * 4, 256);
    p.off_split_base = off; off = align_up(off + (size_t)(d.batch + 1) * 4, 256);
    p.off_item_req = off;   off = align_up(off + (size_t)(p.max_items > 0 ? p.max_items : 1) * 4, 256);
    p.off_item_order = off; off = align_up(off + (size_t)(p.max_items > 0 ? p.max_items : 1) * 4, 256);
    p.off_unit_meta = off;  off = align_up(off + (size_t)(p.max_items > 0 ? p.max_items : 1) * 32, 256);
    p.off_row_rec = off;    off = align_up(off + (size_t)(d.total_q > 0 ? d.total_q : 1) * 16, 256);
    {   // schedule table: every unit appears once, every round is W <= kMaxSchedW wide
        const size_t units = (size_t)p.max_items * d.n_kv_heads * attn_row_groups(p.max_rows);
        p.off_sched = off;  off = align_up(off + (scheduled ? units + kMaxSchedW : 1) * 4, 256);
    }
    p.off_anc = off;        off = align_up(off + (size_t)(d.total_q > 0 ? d.total_q : 1) * 8, 256);
    p.off_part_ml = off;
    off = align_up(off + (size_t)p.max_items * d.n_kv_heads * p.max_rows * 2 * sizeof(float), 256);
    p.off_part_o = off;
    off = align_up(off + (size_t)p.max_items * d.n_kv_heads * p.max_rows * d.head_dim * sizeof(float), 256);
    p.off_flags = off;
    if (p.merged) off = align_up(off + (size_t)p.max_items * d.n_kv_heads * n_groups * kWavesPerUnit * sizeof(uint64_t), 256);
    p.total_bytes = off;
    return p;
}

// Marks are never given twice, and start at an arbitrary place: leftovers in a workspace, of whatever kind, do not look
// like one.
static uint64_t next_mark()
{
    static std::atomic<uint64_t> mark{[]() -> uint64_t {
        try {
            std::random_device rd;
            return (uint64_t)rd() << 32 | rd();
        } catch (...) {                         // (no source of entropy: the clock, spread over the word)
            return (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull;
        }
    }()};
    uint64_t m = mark.fetch_add(1, std::memory_order_relaxed);
    return m != 0 ? m : mark.fetch_add(1, std::memory_order_relaxed);      // (0 is what a merge leaves)
}

// (times an odd constant: as many different ones, and 0 only from 0)
uint64_t next_spread_mark() { return next_mark() * 0x9e3779b97f4a7c15ull; }

DirectArgs direct_args(const AttnArgs &a)
{
    DirectArgs d{a.ctx_lens, a.spec_lens, a.dims.batch, a.dims.max_spec_len, a.dims.total_q, a.plan.per_req, a.plan.split_tokens, nullptr, 0};
    if (a.plan.merged) {
        d.flags = reinterpret_cast<unsigned long long *>(a.ws + a.plan.off_flags);
        d.mark = next_mark();
    }
    return d;
}

// chain and tree calls of the same dims ask for the same workspace
static size_t attn_workspace_bytes(const adaspec_attn_dims &d, AttnKind kind)
{
    const size_t chain = make_attn_plan(d, kind, false).total_bytes, tree = make_attn_plan(d, kind, true).total_bytes;
    return chain > tree ? chain : tree;
}

static int validate_accept_dims(const adaspec_accept_dims *d)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->batch < 0 || d->total_q < d->batch || d->max_spec_len < 0) return ADASPEC_ERR_DIM;
    if (d->total_draft != d->total_q - d->batch) return ADASPEC_ERR_DIM;
    if ((int64_t)d->total_q > (int64_t)d->batch * (d->max_spec_len + 1)) return ADASPEC_ERR_DIM;
    if (d->vocab <= 0) return ADASPEC_ERR_DIM;
    if (!dtype_ok(d->logits_dtype) || !dtype_ok(d->probs_dtype)) return ADASPEC_ERR_DTYPE;
    if (d->logits_row_stride < d->vocab || d->probs_row_stride < d->vocab) return ADASPEC_ERR_DIM;
    if (d->out_stride < d->max_spec_len + 1) return ADASPEC_ERR_DIM;
    if (d->path < ADASPEC_PATH_AUTO || d->path > ADASPEC_PATH_TWO_PASS) return ADASPEC_ERR_DIM;
    return ADASPEC_OK;
}

AcceptPlan make_accept_plan(const adaspec_accept_dims &d)
{
    AcceptPlan p;
    size_t off = 0;
    const size_t tq = (size_t)(d.total_q > 0 ? d.total_q : 1);
    p.off_cu_q = off;     off = align_up(off + (size_t)(d.batch + 1) * 4, 256);
    p.off_row_req = off;  off = align_up(off + tq * 4, 256);
    p.off_row_flag = off; off = align_up(off + tq * 4, 256);
    p.off_row_cand = off; off = align_up(off + tq * 4, 256);
    p.off_row_meta = off; off = align_up(off + tq * 32, 256);
    const size_t nb = (size_t)(d.batch > 0 ? d.batch : 1);
    p.off_row_stat = off;   off = align_up(off + tq * sizeof(RowStat), 256);
    p.off_req_ticket = off; off = align_up(off + nb * 4, 256);
    // What the form in parts needs.  16-bit rows of one type up to V = 131072 always have it; for the others
    // it is laid out only where the whole workspace still fits adaspec_accept_noalloc's built-in scratch, so that no
    // call outgrows that array because of it.
    const size_t tree_min = align_up(tq * kTreeNodeStatMin, 256);
    p.parts = accept_parts_dims_fit(d);
    p.off_slot_rec = p.off_part_stat = p.off_half_stat = p.off_part = off;
    if (p.parts) {
        size_t end = off;
        p.off_slot_rec = end;   end = align_up(end + accept_parts_slot_bytes(d), 256);
        p.off_part_stat = end;  end = align_up(end + accept_parts_stat_bytes(d), 256);
        p.off_half_stat = end;  end = align_up(end + accept_parts_sum_stat_bytes(d), 256);
        p.off_part = end;       end = align_up(end + accept_parts_sum_bytes(d), 256);
        const bool narrow = d.logits_dtype != ADASPEC_F32 && d.logits_dtype == d.probs_dtype && d.vocab <= 131072;
        p.parts = narrow || end + tree_min <= kNoallocScratchBytes;
        if (p.parts) off = end;
    }
    p.noalloc_bytes = off + tree_min;
    // tree calls only, and therefore last: the chain call without a workspace does not need all of it
    p.off_tree_stat = off; off = align_up(off + tq * tree_node_stat_bytes(d.vocab), 256);
    p.total_bytes = off;
    return p;
}

}  // namespace adaspec

using namespace adaspec;

extern "C" {

size_t adaspec_verify_attn_workspace_bytes(const adaspec_attn_dims *dims)
{
    if (validate_attn_dims(dims) != ADASPEC_OK) return 0;
    return attn_workspace_bytes(*dims, attn_kind(*dims));
}

// chain (parents == NULL, tree == false) and tree verification share everything but the mask
static int verify_attn_impl(const void *q, const void *k_pages, const void *v_pages,
                            const int32_t *block_table, const int32_t *ctx_lens,
                            const int32_t *spec_lens, const int32_t *parents, bool tree, void *out,
                            const adaspec_attn_dims *dims,
                            void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = validate_attn_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    if (tree && dims->max_spec_len > 63) return ADASPEC_ERR_UNSUPPORTED;
    if (dims->batch == 0) return ADASPEC_OK;
    if (tree && !parents) return ADASPEC_ERR_NULL;
    const bool plan_only = dims->plan_mode == ADASPEC_PLAN_BUILD_ONLY;
    if (!block_table || !ctx_lens || !spec_lens || !workspace) return ADASPEC_ERR_NULL;
    if (!plan_only && (!q || !k_pages || !v_pages || !out)) return ADASPEC_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return ADASPEC_ERR_ALIGN;
    if (!plan_only && (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(out)))
        return ADASPEC_ERR_ALIGN;
    AttnArgs a;
    const AttnKind kind = attn_kind(*dims);
    a.plan = make_attn_plan(*dims, kind, tree);
    if (workspace_bytes < attn_workspace_bytes(*dims, kind)) return ADASPEC_ERR_WORKSPACE;
    a.q = q; a.k_pages = k_pages; a.v_pages = v_pages;
    a.block_table = block_table; a.ctx_lens = ctx_lens; a.spec_lens = spec_lens;
    a.parents = tree ? parents : nullptr;
    a.out = out; a.dims = *dims; a.ws = static_cast<char *>(workspace);
    a.stream = static_cast<hipStream_t>(stream);
    const float scale = dims->scale > 0.0f ? dims->scale : 1.0f / sqrtf((float)dims->head_dim);
    a.scale_log2 = scale * 1.4426950408889634f;

    a.direct = a.plan.direct;
    if (kind != AttnKind::kVector) attn_mfma_shape(a, kind);
    if (dims->plan_mode != ADASPEC_PLAN_REUSE && !a.direct) {
        if (launch_attn_plan(a) != hipSuccess) return ADASPEC_ERR_HIP;
        if (tree && launch_tree_masks(a) != hipSuccess) return ADASPEC_ERR_HIP;
    }
    if (plan_only) return ADASPEC_OK;
    if (!record_event(dims->timing_start, dims->timing_stop, true, a.stream)) return ADASPEC_ERR_HIP;
    hipError_t e = kind == AttnKind::kVector ? launch_attn_vector(a)
                   : kind == AttnKind::kMfma64 ? launch_attn_d64(a)
                   : kind == AttnKind::kMfmaF32 ? launch_attn_f32(a) : launch_attn_mfma(a);
    if (e != hipSuccess) return ADASPEC_ERR_HIP;
    if (!record_event(dims->timing_start, dims->timing_stop, false, a.stream)) return ADASPEC_ERR_HIP;
    if (!a.plan.merged && launch_attn_combine(a) != hipSuccess) return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_verify_attn(const void *q, const void *k_pages, const void *v_pages,
                        const int32_t *block_table, const int32_t *ctx_lens,
                        const int32_t *spec_lens, void *out, const adaspec_attn_dims *dims,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    return verify_attn_impl(q, k_pages, v_pages, block_table, ctx_lens, spec_lens, nullptr, false, out, dims,
                            workspace, workspace_bytes, stream);
}

int adaspec_verify_attn_tree(const void *q, const void *k_pages, const void *v_pages,
                             const int32_t *block_table, const int32_t *ctx_lens,
                             const int32_t *spec_lens, const int32_t *parents, void *out,
                             const adaspec_attn_dims *dims,
                             void *workspace, size_t workspace_bytes, void *stream)
{
    return verify_attn_impl(q, k_pages, v_pages, block_table, ctx_lens, spec_lens, parents, true, out, dims,
                            workspace, workspace_bytes, stream);
}

size_t adaspec_accept_workspace_bytes(const adaspec_accept_dims *dims)
{
    if (validate_accept_dims(dims) != ADASPEC_OK) return 0;
    return make_accept_plan(*dims).total_bytes;
}

// The kernel path a call with these dims and pointers takes (an adaspec_path other than AUTO), or a
// negative status if a forced path does not fit the shape.
static int resolve_accept_path(const adaspec_accept_dims &d, const void *logits, const void *probs)
{
    const bool fast_ok = accept_fast_path_supported(d, logits, probs);
    const bool stream_ok = accept_stream_path_supported(d, logits, probs);
    const bool two_pass_ok = fast_ok && stream_ok;
    if (d.path == ADASPEC_PATH_FAST && !fast_ok) return ADASPEC_ERR_UNSUPPORTED;
    if (d.path == ADASPEC_PATH_STREAM && !stream_ok) return ADASPEC_ERR_UNSUPPORTED;
    if (d.path == ADASPEC_PATH_TWO_PASS && !two_pass_ok) return ADASPEC_ERR_UNSUPPORTED;
    if (d.path != ADASPEC_PATH_AUTO) return d.path;
    // AUTO.  The two-pass form in row parts does the least work (rows behind a rejection are never read, the
    // sampling step runs on one row per request) and spreads every row over many small workgroups; measured
    // on MI355X it is ahead of the per-row kernels (+ emit kernel) on every benchmark shape: V = 32000, 150
    // rows 16.5 against 21.4 us; V = 128256: 227 rows 28 against 38 us, 380 rows 39 against 63 us, 510 rows
    // 39 against 70 us; all greedy 17.1 against 16.9 us.  Batches it does not take (more than 1024 requests)
    // use the older two-pass pair when there are more rows than compute units or the vocabulary is large; a
    // row that does not fit the registers of one workgroup (V > 131072) goes to the streaming kernel, anything
    // else to the vector kernel.
    if (two_pass_ok && make_accept_plan(d).parts) return ADASPEC_PATH_TWO_PASS;
    if (two_pass_ok && (d.total_q > compute_units() || d.vocab >= 65536)) return ADASPEC_PATH_TWO_PASS;
    if (fast_ok) return ADASPEC_PATH_FAST;
    if (stream_ok) return ADASPEC_PATH_STREAM;
    return ADASPEC_PATH_VECTOR;
}

int adaspec_accept_resolved_path(const void *target_logits, const void *draft_probs,
                                 const adaspec_accept_dims *dims)
{
    const int rc = validate_accept_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    return resolve_accept_path(*dims, target_logits, draft_probs);
}

// workspace == NULL with use_static_scratch: the library's own device array takes its place
static int accept_impl(const void *target_logits, const void *draft_probs,
                       const int32_t *draft_tokens, const float *uniforms,
                       const int32_t *spec_lens, const float *temperature,
                       int32_t *out_tokens, int32_t *out_accept_len,
                       const adaspec_accept_dims *dims,
                       void *workspace, size_t workspace_bytes, bool use_static_scratch, void *stream)
{
    int rc = validate_accept_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    if (use_static_scratch && make_accept_plan(*dims).noalloc_bytes > kNoallocScratchBytes)
        return ADASPEC_ERR_WORKSPACE;           // larger than the built-in scratch: use adaspec_accept
    if (dims->batch == 0) return ADASPEC_OK;
    if (!target_logits || !uniforms || !spec_lens || !temperature || !out_tokens || !out_accept_len ||
        (!workspace && !use_static_scratch))
        return ADASPEC_ERR_NULL;
    if (dims->total_draft > 0 && (!draft_probs || !draft_tokens)) return ADASPEC_ERR_NULL;
    if (use_static_scratch) {
        rc = noalloc_scratch(&workspace);
        if (rc != ADASPEC_OK) return rc;
        workspace_bytes = kNoallocScratchBytes;
    }
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return ADASPEC_ERR_ALIGN;
    const int path = resolve_accept_path(*dims, target_logits, draft_probs);
    if (path < 0) return path;
    const bool two_pass = path == ADASPEC_PATH_TWO_PASS, fast = path == ADASPEC_PATH_FAST,
               streaming = path == ADASPEC_PATH_STREAM;
    AcceptArgs a;
    a.plan = make_accept_plan(*dims);
    if (!use_static_scratch && workspace_bytes < a.plan.total_bytes) return ADASPEC_ERR_WORKSPACE;
    a.logits = target_logits; a.probs = draft_probs; a.draft_tokens = draft_tokens;
    a.uniforms = uniforms; a.spec_lens = spec_lens; a.temperature = temperature;
    a.out_tokens = out_tokens; a.out_accept_len = out_accept_len;
    a.dims = *dims; a.ws = static_cast<char *>(workspace);
    a.stream = static_cast<hipStream_t>(stream);

    // AUTO: rows that the two-pass form in parts can read (any storage types, V up to 524288, aligned) take it in place of
    // the streaming and vector kernels too, which evaluate every row in one workgroup (MI355X, whole call: V = 128256
    // in fp32, 256 rows: vector kernel 746 us, in parts 39.7 us; V = 262144 in bf16, 192 rows: streaming kernel 65 us, in
    // parts 32.3 us).  Forced paths keep their kernels, and so do AUTO calls with other rows or too many requests.
    const bool aligned = aligned16(target_logits) && (dims->total_draft == 0 || aligned16(draft_probs));
    const bool in_parts = a.plan.parts && aligned && (two_pass || (dims->path == ADASPEC_PATH_AUTO && !fast));
    if (two_pass || in_parts) {
        // the statistics of the draft rows, then per request the accept tests, the sampling on the one row
        // that decides its token, and the request's outputs (no emit kernel); both in row parts for up to
        // 1024 requests, larger batches with one workgroup per row and then per request
        if (!record_event(dims->timing_start, dims->timing_stop, true, a.stream)) return ADASPEC_ERR_HIP;
        if (in_parts) {
            if (launch_accept_parts(a, compute_units()) != hipSuccess) return ADASPEC_ERR_HIP;
        } else {
            if (launch_accept_test(a) != hipSuccess) return ADASPEC_ERR_HIP;
            if (launch_accept_resolve(a) != hipSuccess) return ADASPEC_ERR_HIP;
        }
        if (!record_event(dims->timing_start, dims->timing_stop, false, a.stream)) return ADASPEC_ERR_HIP;
        return ADASPEC_OK;
    }
    // the register-resident kernel finds each row's request itself; only the vector kernel needs the plan
    if (!fast && !streaming && launch_accept_plan(a) != hipSuccess) return ADASPEC_ERR_HIP;
    if (!record_event(dims->timing_start, dims->timing_stop, true, a.stream)) return ADASPEC_ERR_HIP;
    hipError_t e = fast ? launch_accept_fast(a) : (streaming ? launch_accept_stream(a) : launch_accept_vector(a));
    if (e != hipSuccess) return ADASPEC_ERR_HIP;
    if (!record_event(dims->timing_start, dims->timing_stop, false, a.stream)) return ADASPEC_ERR_HIP;
    if (launch_accept_emit(a) != hipSuccess) return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_accept(const void *target_logits, const void *draft_probs,
                   const int32_t *draft_tokens, const float *uniforms,
                   const int32_t *spec_lens, const float *temperature,
                   int32_t *out_tokens, int32_t *out_accept_len,
                   const adaspec_accept_dims *dims,
                   void *workspace, size_t workspace_bytes, void *stream)
{
    return accept_impl(target_logits, draft_probs, draft_tokens, uniforms, spec_lens, temperature, out_tokens,
                       out_accept_len, dims, workspace, workspace_bytes, false, stream);
}

int adaspec_accept_noalloc(const void *target_logits, const void *draft_probs,
                           const int32_t *draft_tokens, const float *uniforms,
                           const int32_t *spec_lens, const float *temperature,
                           int32_t *out_tokens, int32_t *out_accept_len,
                           const adaspec_accept_dims *dims, void *stream)
{
    return accept_impl(target_logits, draft_probs, draft_tokens, uniforms, spec_lens, temperature, out_tokens,
                       out_accept_len, dims, nullptr, 0, true, stream);
}

int adaspec_accept_tree(const void *target_logits, const void *draft_probs,
                        const int32_t *draft_tokens, const int32_t *parents, const float *uniforms,
                        const int32_t *spec_lens, const float *temperature,
                        int32_t *out_tokens, int32_t *out_accept_len, int32_t *out_path,
                        const adaspec_accept_dims *dims,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = validate_accept_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    if (dims->path != ADASPEC_PATH_AUTO && dims->path != ADASPEC_PATH_VECTOR && dims->path != ADASPEC_PATH_FAST)
        return ADASPEC_ERR_UNSUPPORTED;
    if (dims->max_spec_len > 63) return ADASPEC_ERR_UNSUPPORTED;
    // (the fast tree kernels take the shapes of the streaming chain kernel: 16-bit rows of one type, V % 8 == 0,
    // V <= 524288, strides % 8 == 0, 16-byte aligned)
    const bool fast_ok = accept_stream_path_supported(*dims, target_logits, draft_probs);
    if (dims->path == ADASPEC_PATH_FAST && !fast_ok) return ADASPEC_ERR_UNSUPPORTED;
    const bool fast = fast_ok && dims->path != ADASPEC_PATH_VECTOR;
    if (dims->batch == 0) return ADASPEC_OK;
    if (!target_logits || !parents || !uniforms || !spec_lens || !temperature || !out_tokens ||
        !out_accept_len || !out_path || !workspace)
        return ADASPEC_ERR_NULL;
    if (dims->total_draft > 0 && (!draft_probs || !draft_tokens)) return ADASPEC_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return ADASPEC_ERR_ALIGN;
    AcceptArgs a;
    a.plan = make_accept_plan(*dims);
    if (workspace_bytes < a.plan.total_bytes) return ADASPEC_ERR_WORKSPACE;
    a.logits = target_logits; a.probs = draft_probs; a.draft_tokens = draft_tokens;
    a.uniforms = uniforms; a.spec_lens = spec_lens; a.temperature = temperature;
    a.out_tokens = out_tokens; a.out_accept_len = out_accept_len;
    a.dims = *dims; a.ws = static_cast<char *>(workspace);
    a.stream = static_cast<hipStream_t>(stream);
    // (the fast kernels find their rows and requests themselves, up to a few thousand requests)
    if ((!fast || tree_fast_needs_plan(*dims)) && launch_accept_plan(a) != hipSuccess) return ADASPEC_ERR_HIP;
    if (!record_event(dims->timing_start, dims->timing_stop, true, a.stream)) return ADASPEC_ERR_HIP;
    if (fast) {
        if (launch_accept_tree_fast(a, parents, compute_units(), out_path) != hipSuccess) return ADASPEC_ERR_HIP;
    } else {
        if (launch_accept_tree_nodes(a, parents) != hipSuccess) return ADASPEC_ERR_HIP;
        if (launch_accept_tree_walk(a, out_path) != hipSuccess) return ADASPEC_ERR_HIP;
    }
    if (!record_event(dims->timing_start, dims->timing_stop, false, a.stream)) return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_kv_compact_path(void *k_pages, void *v_pages, const int32_t *block_table,
                            const int32_t *ctx_lens, const int32_t *spec_lens,
                            const int32_t *out_path, const int32_t *out_accept_len,
                            const adaspec_attn_dims *d, int32_t path_stride, void *stream)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->batch < 0 || d->max_spec_len < 0 || path_stride < d->max_spec_len + 1) return ADASPEC_ERR_DIM;
    if (d->n_kv_heads <= 0 || d->head_dim <= 0 || d->page_size <= 0) return ADASPEC_ERR_DIM;
    if (d->num_pages <= 0 || d->max_pages_per_req <= 0) return ADASPEC_ERR_DIM;
    if (!dtype_ok(d->dtype)) return ADASPEC_ERR_DTYPE;
    if ((d->head_dim * (d->dtype == ADASPEC_F32 ? 4 : 2)) % 16) return ADASPEC_ERR_UNSUPPORTED;
    if (d->batch > 65535) return ADASPEC_ERR_UNSUPPORTED;
    if (d->batch == 0) return ADASPEC_OK;
    if (!k_pages || !v_pages || !block_table || !ctx_lens || !spec_lens || !out_path || !out_accept_len)
        return ADASPEC_ERR_NULL;
    if (!aligned16(k_pages) || !aligned16(v_pages)) return ADASPEC_ERR_ALIGN;
    if (launch_kv_compact_path(k_pages, v_pages, block_table, ctx_lens, spec_lens, out_path, out_accept_len, *d,
                               path_stride, static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_check_ragged_inputs(const int32_t *block_table, const int32_t *ctx_lens,
                                const int32_t *spec_lens, const adaspec_attn_dims *dims,
                                int32_t *err_flags, void *stream)
{
    int rc = validate_attn_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    if (!block_table || !ctx_lens || !spec_lens || !err_flags) return ADASPEC_ERR_NULL;
    if (launch_check_ragged(block_table, ctx_lens, spec_lens, *dims, err_flags,
                            static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_check_accept_inputs(const int32_t *draft_tokens, const int32_t *spec_lens, const float *temperature,
                                const adaspec_accept_dims *dims, int32_t *err_flags, void *stream)
{
    int rc = validate_accept_dims(dims);
    if (rc != ADASPEC_OK) return rc;
    if (!spec_lens || !temperature || !err_flags) return ADASPEC_ERR_NULL;
    if (dims->total_draft > 0 && !draft_tokens) return ADASPEC_ERR_NULL;
    if (launch_check_accept_inputs(draft_tokens, spec_lens, temperature, *dims, err_flags,
                                   static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_check_tree_parents(const int32_t *parents, const int32_t *spec_lens, int32_t batch, int32_t total_q,
                               int32_t max_spec_len, int32_t *err_flags, void *stream)
{
    if (batch < 0 || total_q < batch || max_spec_len < 0) return ADASPEC_ERR_DIM;
    if ((int64_t)total_q > (int64_t)batch * (max_spec_len + 1)) return ADASPEC_ERR_DIM;
    if (max_spec_len > 63) return ADASPEC_ERR_UNSUPPORTED;
    if (!parents || !spec_lens || !err_flags) return ADASPEC_ERR_NULL;
    if (launch_check_tree_parents(parents, spec_lens, batch, total_q, max_spec_len, err_flags,
                                  static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_kv_append(const void *k_new, const void *v_new, void *k_pages, void *v_pages,
                      const int32_t *block_table, const int32_t *ctx_lens,
                      const int32_t *spec_lens, const adaspec_attn_dims *d, void *stream)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->batch < 0 || d->total_q < d->batch || d->max_spec_len < 0) return ADASPEC_ERR_DIM;
    if ((int64_t)d->total_q > (int64_t)d->batch * (d->max_spec_len + 1)) return ADASPEC_ERR_DIM;
    if (d->n_kv_heads <= 0 || d->head_dim <= 0 || d->page_size <= 0) return ADASPEC_ERR_DIM;
    if (d->num_pages <= 0 || d->max_pages_per_req <= 0) return ADASPEC_ERR_DIM;
    if (!dtype_ok(d->dtype)) return ADASPEC_ERR_DTYPE;
    if ((d->head_dim * (d->dtype == ADASPEC_F32 ? 4 : 2)) % 16) return ADASPEC_ERR_UNSUPPORTED;
    if (d->batch == 0) return ADASPEC_OK;
    if (!k_new || !v_new || !k_pages || !v_pages || !block_table || !ctx_lens || !spec_lens)
        return ADASPEC_ERR_NULL;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_pages) || !aligned16(v_pages))
        return ADASPEC_ERR_ALIGN;
    if (launch_kv_append(k_new, v_new, k_pages, v_pages, block_table, ctx_lens, spec_lens, *d,
                         static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

int adaspec_commit(const int32_t *out_tokens, const int32_t *out_accept_len,
                   const int32_t *spec_lens, const int32_t *ctx_lens,
                   const int32_t *next_spec_lens,
                   int32_t *committed_lens, int32_t *next_ctx_lens, int32_t *last_token,
                   int32_t *seq_tokens, int32_t *seq_lens,
                   const adaspec_commit_dims *d, void *stream)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->batch < 0 || d->max_spec_len < 0 || d->seq_stride < 0) return ADASPEC_ERR_DIM;
    if (d->out_stride < d->max_spec_len + 1) return ADASPEC_ERR_DIM;
    if ((seq_tokens == nullptr) != (seq_lens == nullptr)) return ADASPEC_ERR_NULL;
    if (seq_tokens && d->seq_stride <= 0) return ADASPEC_ERR_DIM;
    if (d->batch == 0) return ADASPEC_OK;
    if (!out_tokens || !out_accept_len || !spec_lens || !ctx_lens || !committed_lens || !last_token)
        return ADASPEC_ERR_NULL;
    if (launch_commit(out_tokens, out_accept_len, spec_lens, ctx_lens, next_spec_lens, committed_lens,
                      next_ctx_lens, last_token, seq_tokens, seq_lens, *d,
                      static_cast<hipStream_t>(stream)) != hipSuccess)
        return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

static int validate_draft_dims(const adaspec_draft_dims *d)
{
    if (!d) return ADASPEC_ERR_NULL;
    if (d->rows < 0 || d->vocab <= 0) return ADASPEC_ERR_DIM;
    if (d->logits_row_stride < d->vocab || d->probs_row_stride < d->vocab) return ADASPEC_ERR_DIM;
    if (!dtype_ok(d->logits_dtype) || !dtype_ok(d->probs_dtype)) return ADASPEC_ERR_DTYPE;
    if (d->path < ADASPEC_PATH_AUTO || d->path > ADASPEC_PATH_TWO_PASS || d->path == ADASPEC_PATH_STREAM)
        return ADASPEC_ERR_DIM;
    return ADASPEC_OK;
}

// AUTO of draft sampling, measured on MI355X (us per captured call; three sweeps / register-resident / in parts):
//   V = 8192 bf16    1 row  7.5 / 11.0 /  6.9   128 rows  8.2 / 11.6 /  7.5   256 rows  8.6 / 11.9 /  7.9   300 rows 11.4 / 18.9 / 10.1
//     all greedy            5.9 /      /  6.7             6.4 /      /  7.2             7.0 /      /  7.6             9.1 /      /  9.6
//   V = 16384 bf16   1 row  9.3 / 11.0 /  7.3   128 rows 10.2 / 11.7 /  8.3   256 rows 11.7 / 12.7 /  9.4   300 rows 15.7 / 19.9 / 11.8
//     all greedy            7.5 /      /  7.0             8.5 /      /  7.9             9.7 /      /  8.9            13.2 /      / 11.4
//   V = 32768 bf16   1 row 12.7 / 11.0 /  8.2   128 rows 14.6 / 12.9 / 10.7   256 rows 16.0 / 14.1 / 13.1   300 rows 21.9 / 20.8 / 14.8
//   V = 65536 bf16   1 row 19.5 / 16.5 /  8.7   128 rows 22.6 / 18.6 / 14.6   256 rows 24.9 / 21.2 / 18.4   300 rows 34.9 / 34.7 / 25.0
//   V = 128256 bf16  1 row 31.8 / 26.4 /  8.8   128 rows 39.1 / 32.1 / 18.9   256 rows 43.0 / 33.5 / 31.7   300 rows 62.8 / 57   / 39.9
//     one row more than one workgroup of 1024 threads per compute unit holds: 129 rows in parts 23.0, 160 25.5, 192 27.5
//   V = 12288 fp32   1 row  7.6 /   -  /  7.1   128 rows  9.2 /   -  /  8.2   256 rows 11.9 /   -  / 10.8   300 rows 15.4 /   -  / 12.4
//     all greedy            6.2 /   -  /  6.6             7.5 /   -  /  7.6            10.4 /   -  / 10.1            13.0 /   -  / 11.7
//   V = 50272 fp32   1 row 14.3 /   -  /  8.4   128 rows 21.1 /   -  / 16.2   256 rows 34.1 /   -  / 22.0   300 rows 43.2 /   -  / 26.8
// In parts above V = 12288: below, greedy rows (which the host cannot tell from sampled ones) lose what the others gain.  fp32
// probabilities of 16-bit logits only above 32768: the sweeps' are a little nearer to 64 bits (V = 16384, T = 1: off by 5.8e-8, in parts
// 7.5e-8; V = 50272 1.1e-7 and 6.8e-8).  Without a workspace, or with rows the parts do not take, the register-resident kernel above V = 24576 where it fits, else three sweeps.
constexpr int kDraftPartsAbove = 12288, kDraftPartsAboveWider = 32768, kDraftFastAbove = 24576;
static bool draft_wants_parts(const adaspec_draft_dims &d)
{
    const bool wider = d.probs_dtype == ADASPEC_F32 && d.logits_dtype != ADASPEC_F32;
    return d.vocab > (wider ? kDraftPartsAboveWider : kDraftPartsAbove);
}

// Whether dims may take the form in parts: forced (ADASPEC_PATH_TWO_PASS) for 16-bit logits up to V = 131072; AUTO also
// for fp32 logits and larger vocabularies.
static bool draft_parts_fit(const adaspec_draft_dims &d)
{
    if (!draft_parts_supported(d)) return false;
    const bool small16 = d.logits_dtype != ADASPEC_F32 && d.vocab <= 131072;
    return small16 || (d.path == ADASPEC_PATH_AUTO && draft_wants_parts(d));
}

size_t adaspec_draft_sample_workspace_bytes(const adaspec_draft_dims *d)
{
    if (validate_draft_dims(d) != ADASPEC_OK || d->rows == 0) return 0;
    if (d->vocab % 8 || d->logits_row_stride % 8 || d->probs_row_stride % 8 || !draft_parts_fit(*d)) return 0;
    if (d->path == ADASPEC_PATH_VECTOR || d->path == ADASPEC_PATH_FAST) return 0;
    return draft_parts_workspace_bytes(*d);
}

int adaspec_draft_sample(const void *draft_logits, const float *temperature, const float *uniforms,
                         const int32_t *out_rows, void *draft_probs, int32_t *draft_tokens,
                         float *confidence, const adaspec_draft_dims *d, void *workspace, size_t workspace_bytes,
                         void *stream)
{
    const int rc = validate_draft_dims(d);
    if (rc != ADASPEC_OK) return rc;
    if (d->rows == 0) return ADASPEC_OK;
    if (!draft_logits || !temperature || !uniforms || !draft_probs || !draft_tokens || !confidence)
        return ADASPEC_ERR_NULL;
    if (!aligned16(draft_logits) || !aligned16(draft_probs)) return ADASPEC_ERR_ALIGN;
    if (!draft_sample_supported(*d, draft_logits, draft_probs)) return ADASPEC_ERR_UNSUPPORTED;
    const bool fast_ok = draft_fast_supported(*d);
    const bool split_ok = draft_parts_fit(*d);
    if (d->path == ADASPEC_PATH_FAST && !fast_ok) return ADASPEC_ERR_UNSUPPORTED;
    bool split = false;
    if (d->path == ADASPEC_PATH_TWO_PASS) {
        if (!split_ok) return ADASPEC_ERR_UNSUPPORTED;
        if (!workspace) return ADASPEC_ERR_NULL;
        if (reinterpret_cast<uintptr_t>(workspace) & 255u) return ADASPEC_ERR_ALIGN;
        if (workspace_bytes < draft_parts_workspace_bytes(*d)) return ADASPEC_ERR_WORKSPACE;
        split = true;
    } else if (d->path == ADASPEC_PATH_AUTO) {
        // (probabilities in the logits' place: a workgroup of the split form would have each row alone; us per captured call, in
        // parts / register-resident / three sweeps: V = 128256 bf16 1 row 41.1 / 26.9 / 32.4, 128 44.6 / 30.3 / 39.7; 64 of 50272
        // fp32 38.3 / - / 16.7)
        split = split_ok && draft_wants_parts(*d) && workspace && (draft_probs != draft_logits || out_rows) &&
                !(reinterpret_cast<uintptr_t>(workspace) & 255u) && workspace_bytes >= draft_parts_workspace_bytes(*d);
    }
    const bool fast = !split && fast_ok &&
                      (d->path == ADASPEC_PATH_FAST || (d->path == ADASPEC_PATH_AUTO && d->vocab > kDraftFastAbove));
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!record_event(d->timing_start, d->timing_stop, true, st)) return ADASPEC_ERR_HIP;
    hipError_t e;
    if (split)
        e = launch_draft_parts(draft_logits, temperature, uniforms, out_rows, draft_probs, draft_tokens, confidence, *d,
                               static_cast<char *>(workspace), compute_units(), st);
    else if (fast)
        e = launch_draft_fast(draft_logits, temperature, uniforms, out_rows, draft_probs, draft_tokens, confidence, *d, st);
    else
        e = launch_draft_sample(draft_logits, temperature, uniforms, out_rows, draft_probs, draft_tokens, confidence, *d, st);
    if (e != hipSuccess) return ADASPEC_ERR_HIP;
    if (!record_event(d->timing_start, d->timing_stop, false, st)) return ADASPEC_ERR_HIP;
    return ADASPEC_OK;
}

const char *adaspec_status_string(int status)
{
    switch (status) {
    case ADASPEC_OK: return "ok";
    case ADASPEC_ERR_NULL: return "a required pointer is NULL";
    case ADASPEC_ERR_DIM: return "a dimension is out of range or inconsistent";
    case ADASPEC_ERR_DTYPE: return "unknown or unsupported element type";
    case ADASPEC_ERR_ALIGN: return "pointer or stride is not aligned as required";
    case ADASPEC_ERR_WORKSPACE: return "workspace too small";
    case ADASPEC_ERR_UNSUPPORTED: return "shape not supported by the requested kernel path";
    case ADASPEC_ERR_HIP: return "a HIP call failed";
    default: return "unknown status";
    }
}

int adaspec_version(void) { return 100; }

}  // extern "C"
