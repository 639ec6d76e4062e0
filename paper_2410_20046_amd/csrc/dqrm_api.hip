// C ABI of the DQRM embedding hot path: host-side validation and kernel dispatch.
// Every entry point validates on the host first and enqueues nothing on error.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <mutex>

#include "dqrm.h"
#include "dqrm_device.hpp"
#include "dqrm_fwd.hpp"
#include "dqrm_dedupe.hpp"
#include "dqrm_bwd.hpp"
#include "dqrm_update.hpp"
#include "dqrm_merge.hpp"
#include "dqrm_dense.hpp"
#include "dqrm_step.hpp"

// Scratch of dqrm_embbag_bwd_noalloc: one copy per GPU, held until the process ends.  In host code
// this name is only a handle for hipGetSymbolAddress; kernels receive the address that call returns.
static __device__ __align__(256) unsigned char scratch[DQRM_NOALLOC_SCRATCH_BYTES];

namespace {

thread_local char t_hip_error[256] = "";

int32_t hip_fail(hipError_t e, const char *what)
{
    std::snprintf(t_hip_error, sizeof(t_hip_error), "%s: %s", what, hipGetErrorString(e));
    return DQRM_ERR_HIP;
}

#define DQRM_HIP_CHECK(expr)                                 \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);    \
    } while (0)

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int pow2ceil(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Checks the table descriptor; *total_rows receives R.
int32_t check_tables(const dqrm_tables_t *tb, bool need_packed, int64_t *total_rows)
{
    if (!tb) return DQRM_ERR_INVALID_ARG;
    if (tb->num_tables < 1 || tb->dim < 1) return DQRM_ERR_INVALID_ARG;
    if (!tb->row_offsets_host || !tb->row_offsets_dev || !tb->master || !tb->w_scale) return DQRM_ERR_INVALID_ARG;
    if (need_packed && !tb->packed) return DQRM_ERR_INVALID_ARG;
    if (tb->num_tables > DQRM_MAX_TABLES) return DQRM_ERR_UNSUPPORTED;
    if (tb->dim % 8 != 0 || tb->dim > DQRM_MAX_DIM) return DQRM_ERR_UNSUPPORTED;
    if (!aligned(tb->master, 16) || (tb->packed && !aligned(tb->packed, 4))) return DQRM_ERR_INVALID_ARG;
    const int64_t *ro = tb->row_offsets_host;
    if (ro[0] != 0) return DQRM_ERR_INVALID_ARG;
    for (int t = 0; t < tb->num_tables; ++t) {
        if (ro[t + 1] < ro[t]) return DQRM_ERR_INVALID_ARG;
        if (ro[t + 1] - ro[t] > DQRM_MAX_TABLE_ROWS) return DQRM_ERR_UNSUPPORTED;
    }
    *total_rows = ro[tb->num_tables];
    return DQRM_OK;
}

constexpr int64_t kMaxIndices = 2147483647LL - 2 * DQRM_MAX_TABLES - 64;
// the element-wise kernels index quarter-rows (float4) of the sparse gradient with 32-bit numbers
constexpr int64_t kMaxRowQuarters = 2147483647LL - 4LL * 2048 * 256;

int32_t check_batch(const dqrm_tables_t *tb, const int64_t *indices, const int64_t *offsets, int32_t batch,
                    int64_t num_indices)
{
    if (!offsets || batch < 1 || num_indices < 0) return DQRM_ERR_INVALID_ARG;
    if (num_indices > 0 && !indices) return DQRM_ERR_INVALID_ARG;
    if (num_indices > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    if ((int64_t)batch * tb->num_tables > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    return DQRM_OK;
}

// ---- workspace layout of dqrm_embbag_bwd -------------------------------------
struct WsLayout {
    size_t off_part_info, off_totals, off_part_key, off_part_pos, off_part_start, off_sorted_bag, off_chunk_local, off_single_local, off_chunk_desc, off_chunk_bags,
        off_single_desc, off_seg_count, off_partial_full, off_partial_last, off_absmax_slots, total;
};

// Whether a batch can be partitioned by range (dedupe_partition_kernel): more lookups than one tile, and room for at least 8
// ranges of every table.
bool partitionable(int32_t T, int64_t N) { return N > dqrm::kDdTile && T * 8 <= dqrm::kMaxParts; }

// (table, range) pairs of a batch: only where the tables alone are many is there room for more than kMaxParts
int max_slots(int32_t T) { return 2 * T > dqrm::kMaxParts ? dqrm::kMaxSlots : dqrm::kMaxParts; }

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

WsLayout ws_layout(int32_t T, int32_t D, int64_t N)
{
    WsLayout L{};
    size_t o = 0;
    const size_t n = (size_t)N, t = (size_t)T, slots = (size_t)(N / DQRM_SEG_CHUNK + 2);
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    L.off_part_info = take((size_t)max_slots(T) * 2 * sizeof(int4));
    L.off_totals = take(4 * sizeof(int));
    const size_t big = partitionable(T, N) ? n : 0;
    L.off_part_key = take(big * sizeof(unsigned));
    L.off_part_pos = take(big * sizeof(unsigned short));
    L.off_part_start = take(big ? t * dqrm::kDdTiles * dqrm::kDdRanges * sizeof(unsigned short) : 0);
    L.off_sorted_bag = take(n * sizeof(int));
    // (the lists have a slot even for an empty batch: the summing kernels request their first entries before they
    // know the counts)
    const size_t n1 = n ? n : 1;
    L.off_chunk_local = take(n1 * 16);
    L.off_single_local = take(n1 * 16);
    L.off_chunk_desc = take(n1 * 16);
    L.off_chunk_bags = take((n / 2 + 1) * DQRM_SEG_CHUNK * sizeof(int));
    L.off_single_desc = take(n1 * 16);
    L.off_seg_count = take(slots * sizeof(int));
    L.off_partial_full = take(slots * (size_t)D * sizeof(float));
    L.off_partial_last = take(slots * (size_t)D * sizeof(float));
    L.off_absmax_slots = take(t * dqrm::kAbsmaxSlots * dqrm::kAbsmaxStride * sizeof(float));
    L.total = o;
    return L;
}

dqrm::BwdWs ws_views(void *workspace, const WsLayout &L)
{
    char *b = static_cast<char *>(workspace);
    dqrm::BwdWs w;
    w.part_info = reinterpret_cast<int4 *>(b + L.off_part_info);
    w.totals = reinterpret_cast<int *>(b + L.off_totals);
    w.part_key = reinterpret_cast<unsigned *>(b + L.off_part_key);
    w.part_pos = reinterpret_cast<unsigned short *>(b + L.off_part_pos);
    w.part_start = reinterpret_cast<unsigned short *>(b + L.off_part_start);
    // (needed before the dense list is written, and far smaller: only for more than kDdTile lookups and fewer tables than kMaxParts / 8)
    w.part_bound = reinterpret_cast<unsigned *>(b + L.off_chunk_desc);
    static_assert((size_t)dqrm::kMaxParts / 8 * (dqrm::kDdRanges + 1) * sizeof(unsigned) <= (size_t)dqrm::kDdTile * 16, "it fits");
    w.sorted_bag = reinterpret_cast<int *>(b + L.off_sorted_bag);
    w.chunk_local = reinterpret_cast<int4 *>(b + L.off_chunk_local);
    w.single_local = reinterpret_cast<int4 *>(b + L.off_single_local);
    w.chunk_desc = reinterpret_cast<int4 *>(b + L.off_chunk_desc);
    w.chunk_bags = reinterpret_cast<int *>(b + L.off_chunk_bags);
    w.single_desc = reinterpret_cast<int4 *>(b + L.off_single_desc);
    w.seg_count = reinterpret_cast<int *>(b + L.off_seg_count);
    w.partial_full = reinterpret_cast<float *>(b + L.off_partial_full);
    w.partial_last = reinterpret_cast<float *>(b + L.off_partial_last);
    w.absmax_slots = reinterpret_cast<float *>(b + L.off_absmax_slots);
    return w;
}

int num_cus()
{
    static thread_local int cached_dev = -1, cached = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (dev != cached_dev) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
        cached = v;
        cached_dev = dev;
    }
    return cached;
}

int grid_for(int64_t work_items, int threads, int blocks_per_cu)
{
    int64_t want = (work_items + threads - 1) / threads;
    int64_t cap = (int64_t)num_cus() * blocks_per_cu;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    return (int)want;
}

template <bool EXTRA>
void launch_dedupe(int cap, dim3 grid, hipStream_t st, const dqrm::DedupeArgs &da)
{
    if (cap == 2048)
        hipLaunchKernelGGL((dqrm::dedupe_kernel<256, 2048, false, EXTRA>), grid, dim3(256), 0, st, da);
    else if (cap == 4096)
        hipLaunchKernelGGL((dqrm::dedupe_kernel<512, 4096, false, EXTRA>), grid, dim3(512), 0, st, da);
    else
        hipLaunchKernelGGL((dqrm::dedupe_kernel<1024, 8192, false, EXTRA>), grid, dim3(1024), 0, st, da);
}

template <bool PACKED>
void launch_fwd(int G, dim3 grid, hipStream_t st, const dqrm::FwdArgs &a)
{
    using namespace dqrm;
    switch (G) {
    case 2: hipLaunchKernelGGL((embbag_fwd_kernel<2, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    case 4: hipLaunchKernelGGL((embbag_fwd_kernel<4, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    case 8: hipLaunchKernelGGL((embbag_fwd_kernel<8, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    case 16: hipLaunchKernelGGL((embbag_fwd_kernel<16, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    case 32: hipLaunchKernelGGL((embbag_fwd_kernel<32, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    default: hipLaunchKernelGGL((embbag_fwd_kernel<64, PACKED>), grid, dim3(kFwdThreads), 0, st, a); break;
    }
}

template <bool REUSE>
void launch_segsum(int G, dim3 grid, hipStream_t st, const dqrm::SegArgs &a)
{
    using namespace dqrm;
    switch (G) {
    case 2: hipLaunchKernelGGL((segment_sum_kernel<2, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    case 4: hipLaunchKernelGGL((segment_sum_kernel<4, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    case 8: hipLaunchKernelGGL((segment_sum_kernel<8, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    case 16: hipLaunchKernelGGL((segment_sum_kernel<16, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    case 32: hipLaunchKernelGGL((segment_sum_kernel<32, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    default: hipLaunchKernelGGL((segment_sum_kernel<64, REUSE>), grid, dim3(kSumThreads), 0, st, a); break;
    }
}

template <bool REUSE>
void launch_segsum_multi(int G, dim3 grid, hipStream_t st, const dqrm::SegMulti &m)
{
    using namespace dqrm;
    switch (G) {
    case 2: hipLaunchKernelGGL((segment_sum_multi_kernel<2, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    case 4: hipLaunchKernelGGL((segment_sum_multi_kernel<4, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    case 8: hipLaunchKernelGGL((segment_sum_multi_kernel<8, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    case 16: hipLaunchKernelGGL((segment_sum_multi_kernel<16, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    case 32: hipLaunchKernelGGL((segment_sum_multi_kernel<32, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    default: hipLaunchKernelGGL((segment_sum_multi_kernel<64, REUSE>), grid, dim3(kSumThreads), 0, st, m); break;
    }
}

// Bags of one and a half lookups or more on average: their gradient rows are read more than once.
bool several_lookups(int64_t num_indices, int64_t T, int64_t batch) { return num_indices >= T * batch * 3 / 2; }

int32_t sparse_update_impl(const dqrm_tables_t *tables, int64_t capacity, const int64_t *uniq_rows,
                           const int32_t *table_uniq_offsets, const int8_t *gq, const int32_t *sums,
                           const float *g_scale, float lr, void *stream)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (capacity < 0 || !uniq_rows || !table_uniq_offsets || !g_scale) return DQRM_ERR_INVALID_ARG;
    if (capacity > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    if (capacity * (tables->dim / 4) > kMaxRowQuarters) return DQRM_ERR_UNSUPPORTED;
    dqrm::UpdateArgs a;
    a.master = tables->master;
    a.packed = tables->packed;
    a.w_scale = tables->w_scale;
    a.row_offsets = tables->row_offsets_dev;
    a.uniq_rows = uniq_rows;
    a.tuo = table_uniq_offsets;
    a.gq = gq;
    a.sums = sums;
    a.g_scale = g_scale;
    a.capacity = capacity;
    a.lr = lr;
    a.T = tables->num_tables;
    a.D = tables->dim;
    a.by_q4 = dqrm::FastDiv::make((unsigned)(a.D / 4));
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(dqrm::sparse_update_kernel, dim3(grid_for(capacity * (a.D / 4), dqrm::kEwThreads, 8)),
                       dim3(dqrm::kEwThreads), dqrm::TableLds::bytes(a.T), st, a);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t check_fwd(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch, int64_t num_indices,
                  int32_t mode, const float *out, const int8_t *codes_dbg)
{
    int64_t R = 0;
    if (mode != DQRM_FWD_MASTER && mode != DQRM_FWD_PACKED) return DQRM_ERR_INVALID_ARG;
    int32_t rc = check_tables(tables, mode == DQRM_FWD_PACKED, &R);
    if (rc != DQRM_OK) return rc;
    rc = check_batch(tables, indices, offsets, batch, num_indices);
    if (rc != DQRM_OK) return rc;
    if (!out || !aligned(out, 16) || (codes_dbg && !aligned(codes_dbg, 4))) return DQRM_ERR_INVALID_ARG;
    return DQRM_OK;
}

dqrm::FwdArgs fwd_args(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch, int64_t num_indices,
                       float *out, int8_t *codes_dbg)
{
    dqrm::FwdArgs a;
    a.master = tables->master;
    a.packed = tables->packed;
    a.w_scale = tables->w_scale;
    a.row_offsets = tables->row_offsets_dev;
    a.indices = indices;
    a.offsets = offsets;
    a.out = out;
    a.codes = codes_dbg;
    a.num_indices = num_indices;
    a.T = tables->num_tables;
    a.B = batch;
    a.D = tables->dim;
    a.no_rows = tables->row_offsets_host[a.T] <= 0;
    a.tile_t = 0; // fwd_tiles()
    return a;
}

// the tiles of workgroups of so many threads
dim3 fwd_tiles(dqrm::FwdArgs &a, int threads)
{
    a.tile_t = std::min(a.T, dqrm::kFwdTileT(threads));
    return dim3((unsigned)((a.B + dqrm::kFwdTileB - 1) / dqrm::kFwdTileB), (unsigned)((a.T + a.tile_t - 1) / a.tile_t));
}

int32_t check_dedupe(const dqrm_tables_t *tables, int32_t batch, int32_t num_batches, const dqrm_dedupe_batch_t *batches, size_t workspace_bytes)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (!batches || num_batches < 1) return DQRM_ERR_INVALID_ARG;
    if (num_batches > DQRM_MAX_DEDUPE_BATCHES) return DQRM_ERR_UNSUPPORTED;
    const int T = tables->num_tables, D = tables->dim;
    for (int i = 0; i < num_batches; ++i) {
        const dqrm_dedupe_batch_t &b = batches[i];
        rc = check_batch(tables, b.indices, b.offsets, batch, b.num_indices);
        if (rc != DQRM_OK) return rc;
        if (!b.sorted_pos || !b.uniq_rows || !b.seg_offsets || !b.table_uniq_offsets || !b.num_unique || !b.workspace ||
            !aligned(b.workspace, 256))
            return DQRM_ERR_INVALID_ARG;
        if (b.max_table_lookups < 0) return DQRM_ERR_INVALID_ARG;
        if (workspace_bytes < ws_layout(T, D, b.num_indices).total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
    }
    return DQRM_OK;
}

// What the launches of a sort are given, and which they are.
struct DedupePlan {
    dqrm::DedupeArgs args;
    int64_t max_n, most; // lookups of a batch, of a table, at most
    int cap;             // lookups that a range's workgroup sorts at once
    bool partition, whole, uneven;
    dim3 grid() const { return dim3(args.T, num_batches, (unsigned)(args.parts + (args.extra + args.T - 1) / args.T)); }
    int num_batches;
};

constexpr int kDdFullRanges = 32; // ranges of a partitioned table, if there is room
DedupePlan plan_dedupe(const dqrm_tables_t *tables, int32_t batch, int32_t num_batches, const dqrm_dedupe_batch_t *batches)
{
    const int T = tables->num_tables, D = tables->dim;
    int64_t max_n = 0;
    DedupePlan plan;
    dqrm::DedupeArgs &da = plan.args;
    std::memset(&da, 0, sizeof(da));
    for (int i = 0; i < num_batches; ++i) {
        const dqrm_dedupe_batch_t &b = batches[i];
        dqrm::DedupeBatch &o = da.b[i];
        max_n = std::max(max_n, b.num_indices);
        o.indices = b.indices;
        o.offsets = b.offsets;
        o.N = b.num_indices;
        o.limit = b.max_table_lookups > 0 ? std::min<int32_t>(b.max_table_lookups, DQRM_MAX_TABLE_LOOKUPS)
                                          : DQRM_MAX_TABLE_LOOKUPS;
        o.ws = ws_views(b.workspace, ws_layout(T, D, b.num_indices));
        o.sorted_pos = b.sorted_pos;
        o.tuo = b.table_uniq_offsets;
        o.num_unique = b.num_unique;
        o.uniq_rows = b.uniq_rows;
        o.seg_offsets = b.seg_offsets;
    }
    da.row_offsets = tables->row_offsets_dev;
    da.T = T;
    da.B = batch;
    // How many ranges a table's rows are cut into, and the workgroup: by the lookups of an average table (a table of more
    // is sorted all the same, if need be piece by piece).  Measured (us, with dedupe_finish_kernel):
    //   26 tables x  2048 lookups:  8 ranges of 512 threads 15.7 (1 range 19.1; one 1024-thread workgroup per table, the
    //                               sort without ranges that this replaces: 25)
    //   26 tables x  8192:          8 ranges of 1024 threads 22 (1: 41, 16: 30; without ranges 42)
    //   208 tables x 8192 (eight batches): 1 range 55 (2: 64, 8: 100; without ranges 61)
    //   208 tables x 1024:          1 range 18 (8: 63)
    // so: a workgroup per CU or a little less, at least 256 lookups to a range, and no more than fit the LDS.
    const int64_t avg = (max_n + T - 1) / T, wgs = (int64_t)T * num_batches;
    const int64_t most_parts = dqrm::kMaxParts / T;
    int64_t least_n = max_n;
    for (int i = 0; i < num_batches; ++i) least_n = std::min<int64_t>(least_n, da.b[i].N);
    int64_t most = 0; // lookups of any table
    for (int i = 0; i < num_batches; ++i) most = std::max<int64_t>(most, std::min<int64_t>(da.b[i].N, da.b[i].limit));
    // From two tiles per table on every range's workgroup reading the whole table costs more than sorting the tiles by
    // range first where rows are popular (26 tables, Zipf 1.1 / evenly spread, us, tiles first / everything read: 65536 lookups 112 / 220 and 82 /
    // 110; 24000 57 / 79 and 53 / 39); where the ranges' workgroups leave half of the CUs idle, from three (4 tables, 24000: 38 / 34 and 30 / 29;
    // 32000: 39 / 70 and 33 / 34).
    const bool partition = avg > (wgs * kDdFullRanges * 2 <= num_cus() ? 3 : 2) * dqrm::kDdTile && partitionable(T, least_n);
    // Where the tables alone are workgroups for half of the CUs or more, none is cut (dedupe_table_kernel): 208 x 8192 lookups 60
    // (dedupe_kernel, one range: 67), 1024 x 4096 181 (187); with fewer lookups dedupe_kernel's shorter code counts for more.
    const bool whole = !partition && avg > 2048 && most <= dqrm::kTableCap && num_cus() <= wgs * 2;
    int64_t parts = whole ? 1 : partition ? kDdFullRanges : std::max<int64_t>(std::min<int64_t>({num_cus() / wgs, avg / 256, 16}), (avg - 1) / 8192 * 2);
    parts = std::max<int64_t>(1, std::min(parts, most_parts));
    da.parts = (int)parts;
    da.bags_per_part = (int)((batch + parts - 1) / parts);
    da.by_parts = dqrm::FastDiv::make((unsigned)parts);
    da.even = dqrm::FastDiv::make((unsigned)std::max<int64_t>(1, max_n / ((int64_t)T * batch)));
    // The segment sums of bags of several lookups are faster over a list ordered by chunk length (26 tables x 65536 lookups: by a
    // quarter), those of bags of one over one in sorted order (8 x 26 x 8192, whole steps: 461 us, by length 470; 26 x 8192: 73.2, 74.2).
    da.by_length = several_lookups(max_n, T, batch);
    // A table far above the average would leave its few ranges' workgroups at work alone, each with piece after piece to take,
    // the more so if its popular rows lie close together: a table of more than the LDS holds (and a quarter above the average) has
    // ranges of half the LDS each, as many as that takes, chosen so that they hold about equally many lookups.  The workgroups of
    // those beyond `parts` look up in the tables' boundaries which table is theirs.  Measured (us, with dedupe_finish_kernel; in
    // brackets the `parts` equally wide ranges that every table has otherwise):
    //   255 tables x  128 lookups and one of 65536: 261 (7600); one of 16384: 70 (670)
    //    25 tables x 2048 and one of 65536:          75 (472); 25 x 512 and one of 16384: 51 (135)
    // where no table has that many: 26 x 2048 19.1 (18.5), 26 x 8192 32.5 (31.6).  A bound on a table's lookups spares that.
    // Of a partitioned table the ranges hold about equally many, so half the LDS is enough, and two workgroups share a CU, unless there
    // is a CU for each, or they hold so many that some would overflow it (Zipf 1.1 / evenly spread, us, half / whole: 8 x 65536 76 / 49 and
    // 47 / 42; ranges of 1700, 100 x 17000 89 / 108 and 88 / 112; of 2500, 128 x 20000 142 / 129 and 132 / 136; of 3300, 100 x 32768 173 / 161
    // and 179 / 162; of 4096, 64 x 65536 240 / 200 and 224 / 189).
    const int cap = partition ? (avg > 2560 * parts || wgs * parts <= num_cus() ? 8192 : 4096) : avg <= 512 ? 2048 : (avg <= 4096 && parts > 1 ? 4096 : 8192);
    const int64_t light = std::max<int64_t>(cap, avg + avg / 4);
    const bool uneven = !partition && !whole && most > light;
    if (uneven) {
        const int64_t room = max_slots(T) - T * parts;
        const int64_t per_range = std::max<int64_t>({cap / 2, DQRM_MAX_TABLE_LOOKUPS / dqrm::kDdMaxRanges, room > 0 ? (max_n + room - 1) / room : max_n + 1});
        da.light = (int)light;
        da.per_range = (int)std::min<int64_t>(per_range, DQRM_MAX_TABLE_LOOKUPS);
        // the sum over the tables above `light` of ceil(n / per_range) - parts, at most
        da.extra = (int)std::min(max_n / per_range, max_n / light * std::max<int64_t>(0, (most + per_range - 1) / per_range - parts));
    }
    plan.max_n = max_n, plan.most = most, plan.cap = cap;
    plan.partition = partition, plan.whole = whole, plan.uneven = uneven;
    plan.num_batches = num_batches;
    return plan;
}

void launch_dedupe_sort(const DedupePlan &plan, hipStream_t st)
{
    const dqrm::DedupeArgs &da = plan.args;
    const dim3 grid = plan.grid();
    if (plan.partition) {
        hipLaunchKernelGGL(dqrm::dedupe_partition_kernel, dim3(da.T, plan.num_batches, (unsigned)((plan.most + dqrm::kDdTile - 1) / dqrm::kDdTile)),
                           dim3(dqrm::kDdPartThreads), 0, st, da);
        if (plan.cap == 4096)
            hipLaunchKernelGGL((dqrm::dedupe_kernel<512, 4096, true, false>), grid, dim3(512), 0, st, da);
        else
            hipLaunchKernelGGL((dqrm::dedupe_kernel<1024, 8192, true, false>), grid, dim3(1024), 0, st, da);
    } else if (plan.whole) {
        hipLaunchKernelGGL(dqrm::dedupe_table_kernel, grid, dim3(dqrm::kTableThreads), 0, st, da);
    } else if (plan.uneven) {
        launch_dedupe<true>(plan.cap, grid, st, da);
    } else {
        launch_dedupe<false>(plan.cap, grid, st, da);
    }
}

void launch_dedupe_finish(const DedupePlan &plan, hipStream_t st)
{
    const dqrm::DedupeArgs &da = plan.args;
    // (Up to 4 workgroups per CU for one batch, as many as their LDS allows: 26 x 65536 lookups 283.7 us a step with 2, 279.8 with 4; 26 x
    // 8192 71.1 with either.  8 for eight batches: 256 per batch then; with 512 each the scans in front of the work take 3 us longer.)
    const int finish_blocks = std::min(grid_for(plan.max_n, dqrm::kSegThreads, 4), std::max(1, num_cus() * 8 / plan.num_batches));
    hipLaunchKernelGGL(da.extra > 0 ? dqrm::dedupe_finish_kernel<true> : dqrm::dedupe_finish_kernel<false>,
                       dim3(finish_blocks, plan.num_batches), dim3(dqrm::kSegThreads), dqrm::finish_lds_bytes(da), st, da);
}

int32_t check_segsum(const dqrm_tables_t *tables, int32_t batch, int64_t num_indices, const float *grad_out, const float *values,
                     const void *workspace, size_t workspace_bytes)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (batch < 1 || num_indices < 0) return DQRM_ERR_INVALID_ARG;
    if (num_indices > kMaxIndices || (int64_t)batch * tables->num_tables > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    if (!grad_out || !values || !workspace) return DQRM_ERR_INVALID_ARG;
    if (!aligned(grad_out, 16) || !aligned(values, 16) || !aligned(workspace, 256)) return DQRM_ERR_INVALID_ARG;
    if (workspace_bytes < ws_layout(tables->num_tables, tables->dim, num_indices).total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
    return DQRM_OK;
}

dqrm::SegArgs segsum_args(const dqrm_tables_t *tables, int32_t batch, int64_t num_indices, const float *grad_out, float *values,
                          float *g_absmax, void *workspace)
{
    dqrm::SegArgs sa;
    sa.grad_out = grad_out;
    sa.ws = ws_views(workspace, ws_layout(tables->num_tables, tables->dim, num_indices));
    sa.N = num_indices;
    sa.values = values;
    sa.g_absmax = g_absmax;
    sa.T = tables->num_tables;
    sa.B = batch;
    sa.D = tables->dim;
    return sa;
}

// at most one lane group per four lookups (a window of the chunk list per workgroup, a few singles per group)
int segsum_blocks(int64_t num_indices, int D) { return grid_for((num_indices + 3) / 4 * pow2ceil(D / 4), dqrm::kSumThreads, dqrm::kSumBlocksPerCu); }

void launch_segsum_any(const dqrm::SegArgs &sa, hipStream_t st)
{
    const dim3 grid(segsum_blocks(sa.N, sa.D));
    if (several_lookups(sa.N, sa.T, sa.B))
        launch_segsum<true>(pow2ceil(sa.D / 4), grid, st, sa);
    else
        launch_segsum<false>(pow2ceil(sa.D / 4), grid, st, sa);
}

int32_t check_quant_update(const dqrm_tables_t *tables, int64_t capacity, int64_t num_indices, const float *values,
                           const int64_t *uniq_rows, const int32_t *table_uniq_offsets, const float *g_absmax, const int8_t *gq,
                           const float *g_scale, const void *workspace, size_t workspace_bytes)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (capacity < 0 || num_indices < 0 || !values || !uniq_rows || !table_uniq_offsets || !g_absmax || !gq ||
        !g_scale || !workspace)
        return DQRM_ERR_INVALID_ARG;
    if (capacity > kMaxIndices || num_indices > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    if (!aligned(values, 16) || !aligned(gq, 4) || !aligned(workspace, 256)) return DQRM_ERR_INVALID_ARG;
    if (capacity * (tables->dim / 4) > kMaxRowQuarters) return DQRM_ERR_UNSUPPORTED;
    if (workspace_bytes < ws_layout(tables->num_tables, tables->dim, num_indices).total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
    return DQRM_OK;
}

dqrm::QuantUpdateArgs quant_update_args(const dqrm_tables_t *tables, int64_t capacity, int64_t num_indices, const float *values,
                                        const int64_t *uniq_rows, const int32_t *table_uniq_offsets, float *g_absmax, int8_t *gq,
                                        float *g_scale, float lr, void *workspace)
{
    dqrm::QuantUpdateArgs a;
    a.u.master = tables->master;
    a.u.packed = tables->packed;
    a.u.w_scale = tables->w_scale;
    a.u.row_offsets = tables->row_offsets_dev;
    a.u.uniq_rows = uniq_rows;
    a.u.tuo = table_uniq_offsets;
    a.u.gq = nullptr;
    a.u.sums = nullptr;
    a.u.g_scale = nullptr;
    a.u.capacity = capacity;
    a.u.lr = lr;
    a.u.T = tables->num_tables;
    a.u.D = tables->dim;
    a.u.by_q4 = dqrm::FastDiv::make((unsigned)(a.u.D / 4));
    a.values = values;
    a.absmax_slots = ws_views(workspace, ws_layout(tables->num_tables, tables->dim, num_indices)).absmax_slots;
    a.g_absmax = g_absmax;
    a.gq_out = gq;
    a.g_scale_out = g_scale;
    return a;
}

void launch_quant_update(const dqrm::QuantUpdateArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(dqrm::quant_update_kernel, dim3(grid_for(a.u.capacity * (a.u.D / 4), dqrm::kEwThreads, 8)),
                       dim3(dqrm::kEwThreads), dqrm::TableLds::bytes(a.u.T), st, a);
}

template <int THREADS, int CAP, bool PACKED>
void launch_step_sort_for(const DedupePlan &plan, dqrm::FwdArgs &fa, hipStream_t st)
{
    using namespace dqrm;
    DedupeArgs da = plan.args;
    if (!plan.uneven) da.light = INT_MAX; // (no table has more lookups than the others by far)
    const dim3 tiles = fwd_tiles(fa, THREADS), sort = plan.grid();
    const int sort_groups = (int)(sort.x * sort.z);
    const dim3 grid(sort_groups + tiles.x * tiles.y);
    switch (pow2ceil(fa.D / 4)) {
    case 2: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 2, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    case 4: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 4, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    case 8: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 8, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    case 16: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 16, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    case 32: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 32, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    default: hipLaunchKernelGGL((step_sort_kernel<THREADS, CAP, 64, PACKED>), grid, dim3(THREADS), 0, st, da, fa, sort_groups, (int)tiles.x); break;
    }
}

template <bool PACKED>
void launch_step_sort_any(const DedupePlan &plan, dqrm::FwdArgs &fa, hipStream_t st)
{
    if (plan.cap == 2048)
        launch_step_sort_for<256, 2048, PACKED>(plan, fa, st);
    else if (plan.cap == 4096)
        launch_step_sort_for<512, 4096, PACKED>(plan, fa, st);
    else
        launch_step_sort_for<1024, 8192, PACKED>(plan, fa, st);
}

void launch_step_sort(const DedupePlan &plan, dqrm::FwdArgs &fa, bool packed, hipStream_t st)
{
    if (packed)
        launch_step_sort_any<true>(plan, fa, st);
    else
        launch_step_sort_any<false>(plan, fa, st);
}

// The forward rides along with the sort (us a step, in one launch / in two: 4 tables x 128 lookups x 16 20.8 / 23.3, 26 x 2048 x 16
// 35.4 / 38.6, 13 x 10.5 K x 40 in bags 59.7 / 70.6, 26 x 8192 x 64 67.3 / 71.4, 26 x 16000 x 16 106.1 / 115.2), but for so many large
// bags that its tiles take two rounds behind the sort's workgroups, each of which needs most of a CU's LDS (26 x 64, bags of two, 6000
// samples 90.0 / 94.6, 8192 samples 108.3 / 106.9).
bool step_sorts_with_forward(const DedupePlan &plan, dqrm::FwdArgs fa)
{
    if (plan.partition || plan.whole) return false;
    const dim3 tiles = fwd_tiles(fa, plan.cap / 8);
    return !several_lookups(plan.max_n, fa.T, fa.B) || (int)(tiles.x * tiles.y) <= num_cus() * 3 / 2;
}

// A workgroup per table where a table is little work for one CU: with up to 128 KB of gradient rows to add up it spares two launches and
// several round trips (us a step, one workgroup per table / three launches: 4 x 128 x 16 14.6 / 20.5, 26 x 1024 x 16 24.3 / 32.6,
// 26 x 2048 x 16 33.5 / 36.3, 1 x 2048 x 16 26.9 / 28.2, 200 x 2048 x 16 55.8 / 95.6, 26 x 256 x 128 28.2 / 31.6; 256 KB: 26 x 1024 x 64 38.3 /
// 34.9), of up to 3072 lookups while most CUs have no table (1 x 3000 x 8 30.1 / 30.3, 1 x 4096 x 8 37.0 / 32.7, 26 x 4096 x 8 44.1 / 43.5, 40 x 4096
// x 8 49.1 / 55.2).  The host knows only the average table: a batch whose bags do not all look as if they held equally many lookups may
// have one table with most of them, so all of it is to be little (1 MB in one table: about 50 us against 30).  As many lookups as
// bags, or a multiple, may be unequal all the same, which no user of one lookup per bag or equally many has: 26 x 1024 bags x 16, 27 lookups a bag
// in one table and one in the others, 113 us against 100; 26 x 2048 with all lookups in one table 192 against 156.
bool step_by_table(const DedupePlan &plan, const dqrm::SegArgs &sa)
{
    const int64_t row = sa.D * (int64_t)sizeof(float), T = sa.T, bags = T * sa.B, avg = (sa.N + T - 1) / T;
    return !plan.partition && plan.args.parts <= dqrm::kStepParts && avg * row <= (128 << 10) && (avg <= 3072 || T * 8 > num_cus()) &&
           (sa.N % bags == 0 || sa.N * row <= (1 << 20));
}

void launch_step_table(const DedupePlan &plan, const dqrm::SegArgs &sa, const dqrm::QuantUpdateArgs &qa, hipStream_t st)
{
    using namespace dqrm;
    const StepTableArgs a{plan.args, sa, qa, segsum_blocks(sa.N, sa.D)};
    const dim3 grid(sa.T), threads(kStepThreads);
    switch (pow2ceil(sa.D / 4)) {
    case 2: hipLaunchKernelGGL(step_table_kernel<2>, grid, threads, 0, st, a); break;
    case 4: hipLaunchKernelGGL(step_table_kernel<4>, grid, threads, 0, st, a); break;
    case 8: hipLaunchKernelGGL(step_table_kernel<8>, grid, threads, 0, st, a); break;
    case 16: hipLaunchKernelGGL(step_table_kernel<16>, grid, threads, 0, st, a); break;
    case 32: hipLaunchKernelGGL(step_table_kernel<32>, grid, threads, 0, st, a); break;
    default: hipLaunchKernelGGL(step_table_kernel<64>, grid, threads, 0, st, a); break;
    }
}

// workspace of dqrm_sparse_merge: table offsets of the merged list, and per place the source word, the
// first-of-its-row flag and the flags before it
struct MergeLayout {
    size_t off_base, off_src, off_head, off_excl, off_table_heads, total;
};
MergeLayout merge_layout(int T, int64_t max_total)
{
    MergeLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    const size_t m = (size_t)max_total;
    L.off_base = take(((size_t)T + 1) * sizeof(int32_t));
    L.off_src = take(m * sizeof(int32_t));
    L.off_head = take(m * sizeof(int32_t));
    L.off_excl = take(m * sizeof(int32_t));
    L.off_table_heads = take((size_t)T * sizeof(int32_t));
    L.total = o;
    return L;
}

} // namespace

extern "C" {

const char *dqrm_version(void) { return "0.1"; }

const char *dqrm_last_hip_error(void) { return t_hip_error; }

int32_t dqrm_find_scale(const dqrm_tables_t *tables, void *stream)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int T = tables->num_tables, D = tables->dim;
    // w_scale doubles as the absmax accumulator (bit pattern of a non-negative float)
    hipLaunchKernelGGL(dqrm::fill_u32_kernel, dim3((T + 255) / 256), dim3(256), 0, st,
                       reinterpret_cast<unsigned *>(tables->w_scale), 0u, T);
    const int64_t f4 = R * (D / 4);
    if (f4 > 0) {
        hipLaunchKernelGGL(dqrm::table_absmax_kernel, dim3(grid_for(f4, dqrm::kEwThreads * 4, 16)),
                           dim3(dqrm::kEwThreads), 0, st, tables->master, tables->row_offsets_dev, T, D, tables->w_scale);
    }
    hipLaunchKernelGGL(dqrm::finalize_scale_kernel, dim3((T + 255) / 256), dim3(256), 0, st, tables->w_scale, T);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_pack_int4(const dqrm_tables_t *tables, void *stream)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, true, &R);
    if (rc != DQRM_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int T = tables->num_tables, D = tables->dim;
    const int64_t g8 = R * (D / 8);
    if (g8 > 0) {
        hipLaunchKernelGGL(dqrm::pack_int4_kernel, dim3(grid_for(g8, dqrm::kEwThreads * dqrm::kPackPerThread, 8)), dim3(dqrm::kEwThreads),
                           0, st, tables->master, tables->row_offsets_dev, tables->w_scale, T, D, tables->packed);
    }
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_embbag_fwd(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch,
                        int64_t num_indices, int32_t mode, float *out, int8_t *codes_dbg, void *stream)
{
    const int32_t rc = check_fwd(tables, indices, offsets, batch, num_indices, mode, out, codes_dbg);
    if (rc != DQRM_OK) return rc;
    dqrm::FwdArgs a = fwd_args(tables, indices, offsets, batch, num_indices, out, codes_dbg);
    const dim3 grid = fwd_tiles(a, dqrm::kFwdThreads);
    const int G = pow2ceil(a.D / 4);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (mode == DQRM_FWD_PACKED)
        launch_fwd<true>(G, grid, st, a);
    else
        launch_fwd<false>(G, grid, st, a);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

size_t dqrm_embbag_bwd_workspace_bytes(int32_t num_tables, int32_t dim, int32_t batch, int64_t num_indices)
{
    if (num_tables < 1 || num_tables > DQRM_MAX_TABLES || dim < 8 || dim > DQRM_MAX_DIM || dim % 8 != 0 || batch < 1 ||
        num_indices < 0 || num_indices > kMaxIndices)
        return 0;
    return ws_layout(num_tables, dim, num_indices).total;
}

int32_t dqrm_dedupe_multi(const dqrm_tables_t *tables, int32_t batch, int32_t num_batches,
                          const dqrm_dedupe_batch_t *batches, size_t workspace_bytes, void *stream)
{
    const int32_t rc = check_dedupe(tables, batch, num_batches, batches, workspace_bytes);
    if (rc != DQRM_OK) return rc;
    const DedupePlan plan = plan_dedupe(tables, batch, num_batches, batches);
    hipStream_t st = static_cast<hipStream_t>(stream);
    launch_dedupe_sort(plan, st);
    launch_dedupe_finish(plan, st);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_dedupe(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch,
                    int64_t num_indices, int32_t *sorted_pos, int64_t *uniq_rows, int32_t *seg_offsets,
                    int32_t *table_uniq_offsets, int32_t *num_unique, void *workspace, size_t workspace_bytes,
                    void *stream)
{
    dqrm_dedupe_batch_t b;
    b.indices = indices;
    b.offsets = offsets;
    b.num_indices = num_indices;
    b.sorted_pos = sorted_pos;
    b.uniq_rows = uniq_rows;
    b.seg_offsets = seg_offsets;
    b.table_uniq_offsets = table_uniq_offsets;
    b.num_unique = num_unique;
    b.workspace = workspace;
    b.max_table_lookups = 0;
    return dqrm_dedupe_multi(tables, batch, 1, &b, workspace_bytes, stream);
}

int32_t dqrm_segment_sum(const dqrm_tables_t *tables, int32_t batch, int64_t num_indices, const float *grad_out,
                         float *values, float *g_absmax, void *workspace, size_t workspace_bytes, void *stream)
{
    const int32_t rc = check_segsum(tables, batch, num_indices, grad_out, values, workspace, workspace_bytes);
    if (rc != DQRM_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dqrm::SegArgs sa = segsum_args(tables, batch, num_indices, grad_out, values, g_absmax, workspace);
    launch_segsum_any(sa, st);
    if (g_absmax)
        hipLaunchKernelGGL(dqrm::absmax_finalize_kernel, dim3((sa.T + 255) / 256), dim3(256), 0, st, sa.ws.absmax_slots,
                           sa.T, g_absmax);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_segment_sum_multi(const dqrm_tables_t *tables, int32_t batch, int32_t num_batches,
                               const dqrm_segsum_batch_t *batches, size_t workspace_bytes, void *stream)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (!batches || num_batches < 1 || batch < 1) return DQRM_ERR_INVALID_ARG;
    if (num_batches > DQRM_MAX_DEDUPE_BATCHES) return DQRM_ERR_UNSUPPORTED;
    if ((int64_t)batch * tables->num_tables > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    const int T = tables->num_tables, D = tables->dim;
    int64_t max_n = 0;
    bool any_absmax = false;
    for (int i = 0; i < num_batches; ++i) {
        const dqrm_segsum_batch_t &b = batches[i];
        if (b.num_indices < 0) return DQRM_ERR_INVALID_ARG;
        if (b.num_indices > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
        if (!b.grad_out || !b.values || !b.workspace) return DQRM_ERR_INVALID_ARG;
        if (!aligned(b.grad_out, 16) || !aligned(b.values, 16) || !aligned(b.workspace, 256)) return DQRM_ERR_INVALID_ARG;
        if (workspace_bytes < ws_layout(T, D, b.num_indices).total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
        max_n = std::max(max_n, b.num_indices);
        any_absmax = any_absmax || b.g_absmax != nullptr;
    }
    dqrm::SegMulti sm;
    dqrm::AbsmaxMulti am;
    std::memset(&sm, 0, sizeof(sm));
    std::memset(&am, 0, sizeof(am));
    for (int i = 0; i < num_batches; ++i) {
        const dqrm_segsum_batch_t &b = batches[i];
        dqrm::SegArgs &sa = sm.b[i];
        sa.grad_out = b.grad_out;
        sa.ws = ws_views(b.workspace, ws_layout(T, D, b.num_indices));
        sa.N = b.num_indices;
        sa.values = b.values;
        sa.g_absmax = b.g_absmax;
        sa.T = T, sa.B = batch, sa.D = D;
        am.slots[i] = sa.ws.absmax_slots;
        am.g_absmax[i] = b.g_absmax;
    }
    am.T = T;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int G = pow2ceil(D / 4);
    const int grid_sum = grid_for((max_n + 3) / 4 * G, dqrm::kSumThreads, dqrm::kSumBlocksPerCu);
    if (several_lookups(max_n, T, batch))
        launch_segsum_multi<true>(G, dim3(grid_sum, num_batches), st, sm);
    else
        launch_segsum_multi<false>(G, dim3(grid_sum, num_batches), st, sm);
    if (any_absmax)
        hipLaunchKernelGGL(dqrm::absmax_finalize_multi_kernel, dim3((T + 255) / 256, num_batches), dim3(256), 0, st, am);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_embbag_bwd(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch,
                        int64_t num_indices, const float *grad_out, int32_t *sorted_pos, int64_t *uniq_rows,
                        int32_t *seg_offsets, int32_t *table_uniq_offsets, int32_t *num_unique, float *values,
                        float *g_absmax, void *workspace, size_t workspace_bytes, void *stream)
{
    // validate everything before the first launch
    if (!grad_out || !values || !g_absmax) return DQRM_ERR_INVALID_ARG;
    if (!aligned(grad_out, 16) || !aligned(values, 16)) return DQRM_ERR_INVALID_ARG;
    int32_t rc = dqrm_dedupe(tables, indices, offsets, batch, num_indices, sorted_pos, uniq_rows, seg_offsets,
                             table_uniq_offsets, num_unique, workspace, workspace_bytes, stream);
    if (rc != DQRM_OK) return rc;
    return dqrm_segment_sum(tables, batch, num_indices, grad_out, values, g_absmax, workspace, workspace_bytes, stream);
}

int32_t dqrm_embbag_bwd_noalloc(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets,
                                int32_t batch, int64_t num_indices, const float *grad_out, int32_t *sorted_pos,
                                int64_t *uniq_rows, int32_t *seg_offsets, int32_t *table_uniq_offsets,
                                int32_t *num_unique, float *values, float *g_absmax, void *stream)
{
    // the size check needs only the shape: do it before anything touches the device
    if (!tables) return DQRM_ERR_INVALID_ARG;
    if (tables->num_tables < 1 || tables->dim < 1 || batch < 1 || num_indices < 0) return DQRM_ERR_INVALID_ARG;
    const size_t need = dqrm_embbag_bwd_workspace_bytes(tables->num_tables, tables->dim, batch, num_indices);
    if (need == 0) return DQRM_ERR_UNSUPPORTED;
    if (need > (size_t)DQRM_NOALLOC_SCRATCH_BYTES) {
        std::snprintf(t_hip_error, sizeof(t_hip_error),
                      "dqrm_embbag_bwd_noalloc: this shape needs %zu bytes of scratch, the built-in array holds %zu",
                      need, (size_t)DQRM_NOALLOC_SCRATCH_BYTES);
        return DQRM_ERR_SCRATCH_LIMIT;
    }
    // every GPU holds its own copy of the array at its own address: ask once per device, with that device current
    constexpr int kMaxDevices = 64;
    static void *dev_ptr[kMaxDevices] = {};
    static std::mutex mu;
    int dev = 0;
    DQRM_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return DQRM_ERR_UNSUPPORTED;
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!dev_ptr[dev]) {
            void *p = nullptr;
            DQRM_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            if (!p || !aligned(p, 256)) return hip_fail(hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
            dev_ptr[dev] = p;
        }
        ws = dev_ptr[dev];
    }
    // nothing in the workspace has to start at zero: the dedupe kernels write every counter and slot they or
    // the segment sums read, so the previous call's contents do not matter
    return dqrm_embbag_bwd(tables, indices, offsets, batch, num_indices, grad_out, sorted_pos, uniq_rows, seg_offsets,
                           table_uniq_offsets, num_unique, values, g_absmax, ws, (size_t)DQRM_NOALLOC_SCRATCH_BYTES, stream);
}

int32_t dqrm_grad_quant_int8(int32_t num_tables, int32_t dim, int64_t capacity, const float *values,
                             const int32_t *table_uniq_offsets, const float *g_absmax, int8_t *gq, float *g_scale,
                             void *stream)
{
    if (num_tables < 1 || dim < 1 || capacity < 0) return DQRM_ERR_INVALID_ARG;
    if (!values || !table_uniq_offsets || !g_absmax || !gq || !g_scale) return DQRM_ERR_INVALID_ARG;
    if (num_tables > DQRM_MAX_TABLES || dim % 8 != 0 || dim > DQRM_MAX_DIM) return DQRM_ERR_UNSUPPORTED;
    if (capacity > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    if (!aligned(values, 16) || !aligned(gq, 4)) return DQRM_ERR_INVALID_ARG;
    if (capacity * (dim / 4) > kMaxRowQuarters) return DQRM_ERR_UNSUPPORTED;
    dqrm::QuantArgs a;
    a.values = values;
    a.tuo = table_uniq_offsets;
    a.g_absmax = g_absmax;
    a.gq = gq;
    a.g_scale = g_scale;
    a.capacity = capacity;
    a.T = num_tables;
    a.D = dim;
    a.by_q4 = dqrm::FastDiv::make((unsigned)(dim / 4));
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(dqrm::grad_quant_kernel, dim3(grid_for(capacity * (dim / 4), dqrm::kEwThreads * dqrm::kGqPerThread, 8)),
                       dim3(dqrm::kEwThreads), dqrm::TableLds::bytes(num_tables), st, a);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_grad_quant_int8_multi(int32_t num_tables, int32_t dim, int32_t num_blocks,
                                   const dqrm_quant_block_t *blocks, void *stream)
{
    if (num_tables < 1 || dim < 1 || !blocks || num_blocks < 1) return DQRM_ERR_INVALID_ARG;
    if (num_tables > DQRM_MAX_TABLES || dim % 8 != 0 || dim > DQRM_MAX_DIM) return DQRM_ERR_UNSUPPORTED;
    if (num_blocks > DQRM_MAX_DEDUPE_BATCHES) return DQRM_ERR_UNSUPPORTED;
    int64_t max_cap = 0;
    for (int i = 0; i < num_blocks; ++i) {
        const dqrm_quant_block_t &b = blocks[i];
        if (b.capacity < 0) return DQRM_ERR_INVALID_ARG;
        if (!b.values || !b.table_uniq_offsets || !b.g_absmax || !b.gq || !b.g_scale) return DQRM_ERR_INVALID_ARG;
        if (b.capacity > kMaxIndices || b.capacity * (dim / 4) > kMaxRowQuarters) return DQRM_ERR_UNSUPPORTED;
        if (!aligned(b.values, 16) || !aligned(b.gq, 4)) return DQRM_ERR_INVALID_ARG;
        max_cap = std::max(max_cap, b.capacity);
    }
    dqrm::QuantMulti qm;
    std::memset(&qm, 0, sizeof(qm));
    for (int i = 0; i < num_blocks; ++i) {
        const dqrm_quant_block_t &b = blocks[i];
        dqrm::QuantArgs &a = qm.b[i];
        a.values = b.values;
        a.tuo = b.table_uniq_offsets;
        a.g_absmax = b.g_absmax;
        a.gq = b.gq;
        a.g_scale = b.g_scale;
        a.capacity = b.capacity;
        a.T = num_tables;
        a.D = dim;
        a.by_q4 = dqrm::FastDiv::make((unsigned)(dim / 4));
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(dqrm::grad_quant_multi_kernel,
                       dim3(grid_for(max_cap * (dim / 4), dqrm::kEwThreads * dqrm::kGqPerThread, 8), num_blocks), dim3(dqrm::kEwThreads),
                       dqrm::TableLds::bytes(num_tables), st, qm);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_sparse_update(const dqrm_tables_t *tables, int64_t capacity, const int64_t *uniq_rows,
                           const int32_t *table_uniq_offsets, const int8_t *gq, const float *g_scale, float lr,
                           void *stream)
{
    if (!gq || !aligned(gq, 4)) return DQRM_ERR_INVALID_ARG;
    return sparse_update_impl(tables, capacity, uniq_rows, table_uniq_offsets, gq, nullptr, g_scale, lr, stream);
}

int32_t dqrm_sparse_update_sums(const dqrm_tables_t *tables, int64_t capacity, const int64_t *uniq_rows,
                                const int32_t *table_uniq_offsets, const int32_t *sums, const float *g_scale,
                                float lr, void *stream)
{
    if (!sums || !aligned(sums, 16)) return DQRM_ERR_INVALID_ARG;
    return sparse_update_impl(tables, capacity, uniq_rows, table_uniq_offsets, nullptr, sums, g_scale, lr, stream);
}

size_t dqrm_sparse_merge_workspace_bytes(int32_t num_tables, int32_t dim, int32_t num_blocks, int64_t max_total)
{
    if (num_tables < 1 || num_tables > DQRM_MAX_TABLES || dim < 8 || dim > DQRM_MAX_DIM || dim % 8 != 0 ||
        num_blocks < 1 || num_blocks > DQRM_MAX_DEDUPE_BATCHES || max_total < 0 || max_total > kMaxIndices)
        return 0;
    return merge_layout(num_tables, max_total).total;
}

int32_t dqrm_sparse_merge(const dqrm_tables_t *tables, int32_t num_blocks, const dqrm_sparse_block_t *blocks,
                          int64_t max_total, int64_t *uniq_rows, int32_t *table_uniq_offsets, int32_t *num_unique,
                          int32_t *sums, void *workspace, size_t workspace_bytes, void *stream)
{
    int64_t R = 0;
    int32_t rc = check_tables(tables, false, &R);
    if (rc != DQRM_OK) return rc;
    if (!blocks || num_blocks < 1 || max_total < 0) return DQRM_ERR_INVALID_ARG;
    if (num_blocks > DQRM_MAX_DEDUPE_BATCHES || max_total > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    const int T = tables->num_tables, D = tables->dim;
    if (max_total * (D / 4) > kMaxRowQuarters) return DQRM_ERR_UNSUPPORTED;
    if (!uniq_rows || !table_uniq_offsets || !num_unique || !sums || !workspace) return DQRM_ERR_INVALID_ARG;
    if (!aligned(sums, 16) || !aligned(workspace, 256)) return DQRM_ERR_INVALID_ARG;
    dqrm::MergeArgs ma;
    std::memset(&ma, 0, sizeof(ma));
    int64_t max_cap = 0;
    for (int k = 0; k < num_blocks; ++k) {
        const dqrm_sparse_block_t &b = blocks[k];
        if (!b.uniq_rows || !b.table_uniq_offsets || !b.gq || !aligned(b.gq, 4) || b.capacity < 0)
            return DQRM_ERR_INVALID_ARG;
        if (b.capacity >= (1LL << dqrm::kMergeSrcBits)) return DQRM_ERR_UNSUPPORTED;
        ma.uniq_rows[k] = b.uniq_rows, ma.tuo[k] = b.table_uniq_offsets, ma.gq[k] = b.gq, ma.capacity[k] = b.capacity;
        if (b.capacity > max_cap) max_cap = b.capacity;
    }
    const MergeLayout L = merge_layout(T, max_total);
    if (workspace_bytes < L.total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
    char *ws = static_cast<char *>(workspace);
    ma.n = num_blocks, ma.T = T, ma.D = D, ma.max_total = (int)max_total;
    ma.base = reinterpret_cast<int32_t *>(ws + L.off_base);
    ma.sorted_src = reinterpret_cast<int32_t *>(ws + L.off_src);
    ma.head = reinterpret_cast<int32_t *>(ws + L.off_head);
    ma.local_excl = reinterpret_cast<int32_t *>(ws + L.off_excl);
    ma.table_heads = reinterpret_cast<int32_t *>(ws + L.off_table_heads);
    ma.uniq_rows_out = uniq_rows, ma.tuo_out = table_uniq_offsets, ma.num_unique = num_unique, ma.sums = sums;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per_block = (int)((max_cap + dqrm::kMergeThreads - 1) / dqrm::kMergeThreads);
    hipLaunchKernelGGL(dqrm::merge_rank_kernel, dim3(per_block < 1 ? 1 : per_block, num_blocks), dim3(dqrm::kMergeThreads),
                       dqrm::merge_rank_lds_bytes(T, num_blocks), st, ma);
    hipLaunchKernelGGL(dqrm::merge_scan_kernel, dim3(T), dim3(dqrm::kMergeScanThreads), 0, st, ma);
    hipLaunchKernelGGL(dqrm::merge_sum_kernel, dim3(grid_for(max_total * (D / 4), dqrm::kMergeThreads, 8)),
                       dim3(dqrm::kMergeThreads), dqrm::merge_sum_lds_bytes(T), st, ma);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_quant_update(const dqrm_tables_t *tables, int64_t capacity, int64_t num_indices, const float *values,
                          const int64_t *uniq_rows, const int32_t *table_uniq_offsets, float *g_absmax, int8_t *gq,
                          float *g_scale, float lr, void *workspace, size_t workspace_bytes, void *stream)
{
    const int32_t rc = check_quant_update(tables, capacity, num_indices, values, uniq_rows, table_uniq_offsets, g_absmax, gq, g_scale,
                                          workspace, workspace_bytes);
    if (rc != DQRM_OK) return rc;
    launch_quant_update(quant_update_args(tables, capacity, num_indices, values, uniq_rows, table_uniq_offsets, g_absmax, gq, g_scale, lr,
                                          workspace),
                        static_cast<hipStream_t>(stream));
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_fwd_bwd_step(const dqrm_tables_t *tables, const int64_t *indices, const int64_t *offsets, int32_t batch,
                          int64_t num_indices, int32_t mode, float *out, int8_t *codes_dbg, const float *grad_out, float lr,
                          int64_t capacity, int32_t *sorted_pos, int64_t *uniq_rows, int32_t *seg_offsets,
                          int32_t *table_uniq_offsets, int32_t *num_unique, float *values, float *g_absmax, int8_t *gq,
                          float *g_scale, void *workspace, size_t workspace_bytes, void *stream)
{
    int32_t rc = check_fwd(tables, indices, offsets, batch, num_indices, mode, out, codes_dbg);
    if (rc != DQRM_OK) return rc;
    const dqrm_dedupe_batch_t b{indices, offsets, num_indices, sorted_pos, uniq_rows, seg_offsets, table_uniq_offsets, num_unique, workspace, 0};
    rc = check_dedupe(tables, batch, 1, &b, workspace_bytes);
    if (rc != DQRM_OK) return rc;
    rc = check_segsum(tables, batch, num_indices, grad_out, values, workspace, workspace_bytes);
    if (rc != DQRM_OK) return rc;
    rc = check_quant_update(tables, capacity, num_indices, values, uniq_rows, table_uniq_offsets, g_absmax, gq, g_scale, workspace,
                            workspace_bytes);
    if (rc != DQRM_OK) return rc;

    hipStream_t st = static_cast<hipStream_t>(stream);
    dqrm::FwdArgs fa = fwd_args(tables, indices, offsets, batch, num_indices, out, codes_dbg);
    DedupePlan plan = plan_dedupe(tables, batch, 1, &b);
    const dqrm::SegArgs sa = segsum_args(tables, batch, num_indices, grad_out, values, nullptr, workspace);
    const dqrm::QuantUpdateArgs qa = quant_update_args(tables, capacity, num_indices, values, uniq_rows, table_uniq_offsets, g_absmax, gq,
                                                       g_scale, lr, workspace);
    const bool by_table = step_by_table(plan, sa);
    if (by_table) plan.args.by_length = 0; // (nobody would read the chunks' ranks by length that the sort counts for it)
    if (step_sorts_with_forward(plan, fa)) {
        launch_step_sort(plan, fa, mode == DQRM_FWD_PACKED, st);
    } else {
        const dim3 grid = fwd_tiles(fa, dqrm::kFwdThreads);
        if (mode == DQRM_FWD_PACKED)
            launch_fwd<true>(pow2ceil(fa.D / 4), grid, st, fa);
        else
            launch_fwd<false>(pow2ceil(fa.D / 4), grid, st, fa);
        launch_dedupe_sort(plan, st);
    }
    if (by_table) {
        launch_step_table(plan, sa, qa, st);
    } else {
        launch_dedupe_finish(plan, st);
        launch_segsum_any(sa, st);
        launch_quant_update(qa, st);
    }
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

} // extern "C"

// ---- the dense part of the train step ---------------------------------------------
namespace {

constexpr int kMaxMlpLayers = 16;
constexpr int kDenseMaxSplits = dqrm::kSgdMaxSlices; // slices of the batch dimension in the weight-gradient products

struct DenseLayout {
    // activations: bot_act[l] = output of bottom layer l, R = interaction output, top_act[l] = output of top
    // layer l (the last one is the logit); gradients w.r.t. the layers' pre-activations: bot_dz[l], top_dz[l]
    // (the last top one is the loss gradient), dR w.r.t. the interaction output; per-layer slices of the split
    // weight-gradient products: bot_part[l], top_part[l]
    size_t bot_act[kMaxMlpLayers], top_act[kMaxMlpLayers], R;
    size_t bot_dz[kMaxMlpLayers], top_dz[kMaxMlpLayers], dR;
    size_t bot_part[kMaxMlpLayers], top_part[kMaxMlpLayers];
    // the quantised variants: fake-quantised weights (layers in flat order), flat FP32 gradients, per-tensor maxima
    size_t wq, grads, gmax;
    size_t loss_terms; // per-sample loss
    // [late, late_end): the slices and the flat gradients, which nothing touches before the last input gradient is there.  Until then
    // the quantised weights' codes lie there, layer by layer (LayerCodes), as far as they fit: a workspace that is enough for FP32 weights
    // is enough for them too.  (Slices and gradients are two parameters' room for each, a row of codes and its scale is padded to
    // 64 of them and one: only models of nothing but layers of less than 32 inputs at small batches do not fit whole.)
    size_t late, late_end;
    size_t total;
};

// flat parameter order (see dqrm_dense_quant_t): top layers, then bottom layers
int64_t dense_param_count(const dqrm_dense_model_t *m)
{
    int64_t p = 0;
    for (int l = 0; l < m->top_layers; ++l) p += (int64_t)m->top_dims[l + 1] * (m->top_dims[l] + 1);
    for (int l = 0; l < m->bot_layers; ++l) p += (int64_t)m->bot_dims[l + 1] * (m->bot_dims[l] + 1);
    return p;
}

// Rows of bfloat16 codes are whole slabs of a product's reduction.
constexpr int code_pitch(int in) { return (in + 63) / 64 * 64; }

// A layer's codes at `at`, what rounding the weights adds to them (both [out][pitch], 16 bits), and their rows' scales (a kernel
// reads them 4 at a time).
struct LayerCodes {
    size_t codes, low, scale, end;
    LayerCodes(size_t at, int in, int out)
    {
        const size_t plane = (size_t)out * code_pitch(in) * sizeof(unsigned short);
        codes = at, low = at + plane, scale = low + plane, end = align_up(scale + (size_t)(out + 3) / 4 * 4 * sizeof(float), 256);
    }
};

// The layers' inputs and outputs, bottom MLP first.
template <typename F>
void each_layer(const dqrm_dense_model_t *m, F &&f)
{
    for (int l = 0; l < m->bot_layers; ++l) f(m->bot_dims[l], m->bot_dims[l + 1]);
    for (int l = 0; l < m->top_layers; ++l) f(m->top_dims[l], m->top_dims[l + 1]);
}

// How the weight-gradient products [out][in] of all layers (one launch) are cut: a layer's tiles, 128x128 or 64x64, a workgroup
// each, and the batch dimension in slices of whole slabs of samples.
struct GradCut {
    static constexpr int kSlab = 64; // samples
    int most;         // the largest tile
    int per128, per64; // samples of a slice, by the tile
    int tile(int in, int out) const { return most >= 128 && std::min(in, out) >= 128 ? 128 : 64; }
    int per(int in, int out) const { return tile(in, out) == 128 ? per128 : per64; }
    int splits(int in, int out, int batch) const { return (batch + per(in, out) - 1) / per(in, out); }
};

GradCut grad_cut(const dqrm_dense_model_t *m, int batch)
{
    const int64_t cus = num_cus(), slabs = (batch + GradCut::kSlab - 1) / GradCut::kSlab;
    // A CU has one workgroup at a time: 5 us for its beginning and end, and so many per slab (measured: 512x512 in slices of 2048
    // samples 82 us in tiles of 128, 36 in tiles of 64); a slice costs its partial tiles, written and added up again, at about 4 TB/s.
    constexpr double kUs128 = 2.4, kUs64 = 0.98, kUsFixed = 5;
    auto us_of = [&](int tile, int64_t n) { return kUsFixed + (tile == 128 ? kUs128 : kUs64) * n; };
    GradCut best{};
    double best_us = 0;
    for (int most : {128, 64}) {
        GradCut c{most, 0, 0};
        int64_t tiles[2] = {};   // of 64, of 128
        double params[2] = {};
        each_layer(m, [&](int in, int out) {
            const int t = c.tile(in, out), k = t == 128;
            tiles[k] += (int64_t)((out + t - 1) / t) * ((in + t - 1) / t);
            params[k] += (double)out * (in + 1);
        });
        if (most == 128 && tiles[1] == 0) continue;
        int64_t last = 0;
        for (int s = 1; s <= kDenseMaxSplits; ++s) { // slices of the larger tiles; the smaller ones take no longer
            const int64_t n = (slabs + s - 1) / s;
            if (n == last) continue;
            last = n;
            const double each = us_of(most, n);
            const int64_t n64 = most == 64 ? n : std::max<int64_t>({1, (slabs + kDenseMaxSplits - 1) / kDenseMaxSplits, std::min(slabs, (int64_t)((each - kUsFixed) / kUs64))});
            const int64_t s64 = (slabs + n64 - 1) / n64, s128 = (slabs + n - 1) / n;
            const double work = most == 64 ? (double)(s64 * tiles[0]) : s128 * tiles[1] + s64 * tiles[0] * us_of(64, n64) / each;
            const double us = std::ceil(work / cus) * each + (s64 * params[0] + s128 * params[1]) * 8 / 4e6;
            if (best_us == 0 || us < best_us) best_us = us, best = GradCut{most, (int)n * GradCut::kSlab, (int)n64 * GradCut::kSlab};
        }
    }
    return best;
}

int32_t check_dense_model(const dqrm_dense_model_t *m, int32_t batch)
{
    if (!m || batch < 1) return DQRM_ERR_INVALID_ARG;
    if (m->num_dense < 1 || m->num_tables < 1 || m->dim < 1 || m->bot_layers < 1 || m->top_layers < 1)
        return DQRM_ERR_INVALID_ARG;
    if (!m->bot_dims || !m->bot_w || !m->bot_b || !m->top_dims || !m->top_w || !m->top_b) return DQRM_ERR_INVALID_ARG;
    if (m->bot_layers > kMaxMlpLayers || m->top_layers > kMaxMlpLayers) return DQRM_ERR_UNSUPPORTED;
    const int V = m->num_tables + 1;
    if (V > 64 || (int64_t)V * m->dim > dqrm::kInterMaxZ) return DQRM_ERR_UNSUPPORTED;
    if (m->bot_dims[0] != m->num_dense || m->bot_dims[m->bot_layers] != m->dim) return DQRM_ERR_INVALID_ARG;
    if (m->top_dims[0] != m->dim + V * (V - 1) / 2 || m->top_dims[m->top_layers] != 1) return DQRM_ERR_INVALID_ARG;
    for (int l = 0; l <= m->bot_layers; ++l)
        if (m->bot_dims[l] < 1 || m->bot_dims[l] > 65536) return DQRM_ERR_UNSUPPORTED;
    for (int l = 0; l <= m->top_layers; ++l)
        if (m->top_dims[l] < 1 || m->top_dims[l] > 65536) return DQRM_ERR_UNSUPPORTED;
    for (int l = 0; l < m->bot_layers; ++l)
        if (!m->bot_w[l] || !m->bot_b[l]) return DQRM_ERR_INVALID_ARG;
    for (int l = 0; l < m->top_layers; ++l)
        if (!m->top_w[l] || !m->top_b[l]) return DQRM_ERR_INVALID_ARG;
    if ((int64_t)batch * 65536 > kMaxIndices) return DQRM_ERR_UNSUPPORTED;
    return DQRM_OK;
}

DenseLayout dense_layout(const dqrm_dense_model_t *m, int32_t batch)
{
    DenseLayout L{};
    size_t o = 0;
    auto take = [&](size_t floats) {
        size_t at = o;
        o = align_up(o + floats * sizeof(float), 256);
        return at;
    };
    const GradCut cut = grad_cut(m, batch);
    auto part = [&](int in, int out) { return take((size_t)cut.splits(in, out, batch) * out * (in + 1)); };
    for (int l = 0; l < m->bot_layers; ++l) {
        L.bot_act[l] = take((size_t)batch * m->bot_dims[l + 1]);
        L.bot_dz[l] = take((size_t)batch * m->bot_dims[l + 1]);
    }
    L.R = take((size_t)batch * m->top_dims[0]);
    L.dR = take((size_t)batch * m->top_dims[0]);
    for (int l = 0; l < m->top_layers; ++l) {
        L.top_act[l] = take((size_t)batch * m->top_dims[l + 1]);
        L.top_dz[l] = take((size_t)batch * m->top_dims[l + 1]);
    }
    const size_t P = (size_t)dense_param_count(m);
    L.wq = take(P);
    L.late = o;
    for (int l = 0; l < m->bot_layers; ++l) L.bot_part[l] = part(m->bot_dims[l], m->bot_dims[l + 1]);
    for (int l = 0; l < m->top_layers; ++l) L.top_part[l] = part(m->top_dims[l], m->top_dims[l + 1]);
    L.grads = take(P);
    L.late_end = o;
    L.gmax = take((size_t)dqrm::kMaxGradTensors * dqrm::kGradMaxSlots * dqrm::kGradMaxStride);
    L.loss_terms = take((size_t)batch);
    L.total = o;
    return L;
}

// A workspace for `batch` samples is enough for fewer as well, the last batch of an epoch for instance: fewer samples may be cut into
// more slices (a slab less makes another cut the best one), so this is the most that any number of samples up to `batch`
// takes.  The cut depends on their number of slabs only, and at most 512 of those are allowed (8192 samples: 0.1 ms on the host).
size_t dense_workspace(const dqrm_dense_model_t *m, int32_t batch)
{
    size_t most = 0;
    for (int64_t b = GradCut::kSlab; b < batch + GradCut::kSlab; b += GradCut::kSlab)
        most = std::max(most, dense_layout(m, (int32_t)std::min<int64_t>(b, batch)).total);
    return most;
}

// The tile of a layer's product by planes of bfloat16, or 0: by the fp32 matrix instructions.  Those are left where a wave's 32x32
// tile can have its reduction shared by four waves on otherwise idle SIMDs, and that is long: 512 samples, 512 -> 512, us, fp32 /
// planes: reduction 256: 7.1 / 6.7, 384: 8.2 / 8.1, 512: 8.4 / 9.5; input gradients (B read along j) 256: 7.2 / 7.6, 200: 11.4 / 9.0.
// Elsewhere, reduction 512: 1024x512 10.7 / 9.8, 2048x512 15.7 / 10.8, 8192x512 57 / 28.7.  Of the tiles the one whose rounds over the
// CUs (a workgroup each) take least: 8192x512, 128 / 128x64 / 64: 28.7 / 31.4 / 38.7; 8192x256: 21.8 / 16.0 / 19.6; 2048x512: 20.6 /
// 13.8 / 10.8.
int plane_tile(const dqrm::GemmArgs &g, bool b_wide)
{
    if (g.K < 8 && (!b_wide || (int64_t)g.M * g.K < 8)) return 0; // (an operand with its rows along r is read 8 floats at a time)
    const int64_t cus = num_cus(), tiles32 = (int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32);
    if (tiles32 <= cus && g.K >= (b_wide ? 256 : 384)) return 0;
    auto us = [&](int bm, int bn, int each) { return (((int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) + cus - 1) / cus) * each; };
    const int64_t us64 = us(64, 64, 10), us128x64 = us(128, 64, 16), us128 = us(128, 128, 27);
    if (us128 <= us128x64 && us128 <= us64) return 128;
    return us128x64 < us64 ? 12864 : 64;
}

// A: the reduction index is the unit-stride one.  B_MODE: how B lies in memory and is read (dqrm::kOpRC: likewise; kOpWide: its
// column index j is).
template <int B_MODE>
hipError_t launch_gemm(hipStream_t st, const dqrm::GemmArgs &g)
{
    const int t = plane_tile(g, B_MODE == dqrm::kOpWide);
    if (t && g.codes) {
        const int bm = t == 64 ? 64 : 128, bn = t == 128 ? 128 : 64;
        const dim3 grid(((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn)), block(dqrm::kPlaneThreads);
        if (t == 128)
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::CodeTile128<B_MODE>, B_MODE>), grid, block, 0, st, g);
        else if (t == 64)
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::CodeTile64<B_MODE>, B_MODE>), grid, block, 0, st, g);
        else
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::CodeTile128x64<B_MODE>, B_MODE>), grid, block, 0, st, g);
        return hipGetLastError();
    }
    if (t) {
        const int bm = t == 64 ? 64 : 128, bn = t == 128 ? 128 : 64;
        const dim3 grid(((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn)), block(dqrm::kPlaneThreads);
        if (t == 128)
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::PlaneTile128, B_MODE>), grid, block, 0, st, g);
        else if (t == 64)
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::PlaneTile64, B_MODE>), grid, block, 0, st, g);
        else
            hipLaunchKernelGGL((dqrm::gemm_planes_kernel<dqrm::PlaneTile128x64, B_MODE>), grid, block, 0, st, g);
        return hipGetLastError();
    }
    dqrm::GemmOne one;
    one.p = g;
    // A product with fewer tiles than the chip has SIMDs (4 per CU) leaves some of them idle: let 2 or 4 waves
    // share a tile, each with a slice of the reduction (at least one pair of slabs each), up to one wave per
    // SIMD.  (Measured: beyond that, slices cost more than they bring.)
    const int pairs = g.K / (2 * dqrm::kGemmBK), simds = num_cus() * 4;
    one.total_tiles = ((g.M + 31) / 32) * ((g.N + 31) / 32);
    one.kslices = 1;
    while (one.kslices < 4 && one.total_tiles * one.kslices * 2 <= simds && pairs >= one.kslices * 2) one.kslices *= 2;
    const int waves = one.total_tiles * one.kslices;
    hipLaunchKernelGGL((dqrm::gemm_wave_kernel<B_MODE>), dim3((waves + dqrm::kGemmWaves - 1) / dqrm::kGemmWaves),
                       dim3(dqrm::kGemmThreads), 0, st, one);
    return hipGetLastError();
}

// Samples per workgroup of the short-input layer: two workgroups per CU (4 waves of 2), within the kernel's limits, for wide
// layers; up to 256 outputs (one wave of the workgroup's two) reading the weights costs less than walking more samples does:
// 8192 samples, whole steps, us, at 4 / 8 / 16 samples: 13 -> 64 78.0 / 77.9 / 81.5, 256 100.8 / 101.3 / 100.9, 512 127.8 / 121.1 / 119.0.
int small_k_samples(int batch, int out)
{
    if (out <= 256) return dqrm::kSmallKMinSamples;
    return std::min(dqrm::kSmallKMaxSamples, std::max(dqrm::kSmallKMinSamples, batch / (2 * num_cus())));
}

// the weight gradients of a group of layers in one launch
hipError_t launch_weight_grads(hipStream_t st, dqrm::GemmGroup &grp)
{
    int blocks = 0;
    for (int q = 0; q < grp.count; ++q) {
        dqrm::GemmArgs &g = grp.p[q];
        g.block_begin = blocks;
        blocks += ((g.M + g.tile - 1) / g.tile) * ((g.N + g.tile - 1) / g.tile) * g.splits;
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(dqrm::gemm_split_group_kernel, dim3(blocks), dim3(dqrm::kPlaneThreads), 0, st, grp);
    return hipGetLastError();
}

// The weights that the forward and the input gradients use, and their codes and scales if they are quantised (and there is room).
struct LayerWeights {
    const float *w;
    const unsigned short *codes, *low;
    const float *scale;
};

// Y[B][out] = act(X[B][in] * W[out][in]^T + b)
hipError_t linear_fwd(hipStream_t st, const float *X, const LayerWeights &W, const float *b, float *Y, int B, int in, int out,
                bool relu)
{
    dqrm::GemmArgs g{};
    g.A = X, g.a_si = in, g.a_sr = 1;
    g.B = W.w, g.b_sr = 1, g.b_sj = in;
    g.codes = W.codes, g.low = W.low, g.scale = W.scale, g.c_pitch = code_pitch(in);
    g.C = Y, g.c_si = out;
    g.M = B, g.N = out, g.K = in;
    g.bias = b, g.relu = relu ? 1 : 0;
    return launch_gemm<dqrm::kOpRC>(st, g);
}

// dX[B][in] = (dZ[B][out] * W[out][in]) masked by (mask[B][in] > 0)
hipError_t linear_bwd_input(hipStream_t st, const float *dZ, const LayerWeights &W, const float *mask, float *dX, int B, int in,
                      int out)
{
    dqrm::GemmArgs g{};
    g.A = dZ, g.a_si = out, g.a_sr = 1;
    g.B = W.w, g.b_sr = in, g.b_sj = 1;
    g.codes = W.codes, g.low = W.low, g.scale = W.scale, g.c_pitch = code_pitch(in);
    g.C = dX, g.c_si = in;
    g.M = B, g.N = in, g.K = out;
    g.mask = mask;
    return launch_gemm<dqrm::kOpWide>(st, g);
}

// Whether the interaction of V vectors of D floats goes by the plain kernels: where it would fill only a little of the 32x32 tiles
// that the matrix cores take it in.  Whole steps (13-64-D, x-32-1) of 8192 samples, us, matrix cores / plain, with the share:
//   up to 32 vectors (one tile): 2 x 64 (0.01) 107 / 88, 9 x 16 (0.04) 83 / 76, 12 x 128 (0.14) 148 / 141, 27 x 8 (0.18) 104 / 101,
//                                21 x 16 (0.22) 97.6 / 97.7, 16 x 32 (0.25) 98 / 101, 27 x 16 (0.36) 105 / 110
//   more: 36 x 8 (0.08) 161 / 119, 33 x 32 (0.27) 181 / 160, 50 x 16 (0.31) 216 / 202, 63 x 16 (0.48) 286 / 305; but 33 x 64
//         (0.27) 220 / 226, 46 x 32 (0.52) 219 / 252
bool inter_plain(int V, int D)
{
    const int t = dqrm::inter_tiles(V) * 32;
    const int64_t share = (int64_t)V * V * D * 100, whole = (int64_t)t * t * ((D + 31) / 32 * 32);
    return share < whole * (V > 32 && D <= 32 ? 31 : 22);
}

// Weights (with their padding) of a bottom MLP's last layer that rides along in the interaction, at most.
int inter_lin_floats(int V, int D, int in, int batch)
{
    if (batch > 2048) return dqrm::kInterLinFloats;
    return inter_plain(V, D) && in <= 256 ? dqrm::kInterLinFloatsPlain : dqrm::kInterLinFloatsFew;
}

// The interaction, forward or backward.  On the matrix cores: one wave per sample, as many waves per workgroup as the LDS holds.  Vectors of a
// multiple of 4 floats are read 16 bytes at a time (from any 4-byte boundary).
hipError_t launch_interact(hipStream_t st, const dqrm::InteractArgs &ia, bool backward, int lin_floats)
{
    const int V = ia.T + 1;
    if (inter_plain(V, ia.D)) {
        const size_t lds = sizeof(float) * dqrm::inter_plain_floats(V, ia.D, backward, lin_floats ? ia.lin_k : 0);
        hipLaunchKernelGGL(backward ? dqrm::interact_bwd_plain_kernel : dqrm::interact_fwd_plain_kernel, dim3(ia.B),
                           dim3(dqrm::kInterPlainThreads), lds, st, ia);
        return hipGetLastError();
    }
    const size_t per = sizeof(float) * (backward ? dqrm::inter_wave_floats_bwd(V, ia.D)
                                                 : dqrm::inter_wave_floats(V, ia.D, lin_floats ? ia.lin_k : 0));
    const size_t shared = sizeof(float) * (size_t)lin_floats;
    const int waves = (int)std::min<size_t>(dqrm::kInterWaves, (dqrm::kInterLdsBytes - shared) / per); // (>= 1: at most 37 KB)
    const dim3 grid((ia.B + waves - 1) / waves), block(waves * dqrm::kWave);
    const size_t lds = shared + waves * per;
    void (*k)(dqrm::InteractArgs);
    const bool vec = ia.D % 4 == 0;
    if (V <= 32)
        k = backward ? (vec ? dqrm::interact_bwd_kernel<1, true> : dqrm::interact_bwd_kernel<1, false>)
                     : (vec ? dqrm::interact_fwd_kernel<1, true> : dqrm::interact_fwd_kernel<1, false>);
    else
        k = backward ? (vec ? dqrm::interact_bwd_kernel<2, true> : dqrm::interact_bwd_kernel<2, false>)
                     : (vec ? dqrm::interact_fwd_kernel<2, true> : dqrm::interact_fwd_kernel<2, false>);
    hipLaunchKernelGGL(k, grid, block, lds, st, ia);
    return hipGetLastError();
}

// One layer's weight-gradient product  [dZ^T * X | dZ^T * 1]  ([out][in + 1], the last column is the bias
// gradient) with the batch dimension cut into slices: partials[s][out][in + 1].
dqrm::GemmArgs weight_grad_problem(const float *dZ, const float *X, float *partials, int B, int in, int out, const GradCut &cut)
{
    dqrm::GemmArgs g{};
    g.A = dZ, g.a_si = 1, g.a_sr = out;
    g.B = X, g.b_sr = in, g.b_sj = 1;
    g.M = out, g.N = in, g.K = B;
    g.tile = cut.tile(in, out), g.splits = cut.splits(in, out, B), g.k_per_split = cut.per(in, out), g.P = partials;
    return g;
}

} // namespace

extern "C" {

size_t dqrm_dense_workspace_bytes(const dqrm_dense_model_t *model, int32_t batch)
{
    if (check_dense_model(model, batch) != DQRM_OK) return 0;
    return dense_workspace(model, batch);
}

int64_t dqrm_dense_param_count(const dqrm_dense_model_t *model)
{
    if (check_dense_model(model, 1) != DQRM_OK) return -1;
    return dense_param_count(model);
}

int32_t dqrm_dense_step(const dqrm_dense_model_t *m, int32_t batch, const float *dense_x, const float *emb_out,
                        const float *labels, float lr, float *loss, float *grad_emb, void *workspace,
                        size_t workspace_bytes, void *stream)
{
    return dqrm_dense_step_quant(m, nullptr, batch, dense_x, emb_out, labels, lr, loss, grad_emb, workspace,
                                 workspace_bytes, stream);
}

int32_t dqrm_dense_step_quant(const dqrm_dense_model_t *m, const dqrm_dense_quant_t *quant, int32_t batch,
                              const float *dense_x, const float *emb_out, const float *labels, float lr, float *loss,
                              float *grad_emb, void *workspace, size_t workspace_bytes, void *stream)
{
    int32_t rc = check_dense_model(m, batch);
    if (rc != DQRM_OK) return rc;
    const int wbits = quant ? quant->weight_bits : 0, gbits = quant ? quant->grad_bits : 0;
    if ((wbits != 0 && wbits != 4 && wbits != 8) || (gbits != 0 && gbits != 8)) return DQRM_ERR_UNSUPPORTED;
    if (gbits == 8 && !quant->grad_scale) return DQRM_ERR_INVALID_ARG;
    if (quant && quant->grad_buffer && gbits != 0) return DQRM_ERR_UNSUPPORTED; // FP32 gradient buffers only
    if (!dense_x || !emb_out || !labels || !loss || !grad_emb || !workspace || !aligned(workspace, 256))
        return DQRM_ERR_INVALID_ARG;
    const DenseLayout L = dense_layout(m, batch);
    if (workspace_bytes < L.total) return DQRM_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    auto F = [&](size_t off) { return reinterpret_cast<float *>(ws + off); };
    const int B = batch, T = m->num_tables, D = m->dim;

    // ---- the weights the forward and the input gradients use: the model's, or their fake-quantised copies
    LayerWeights top_wf[kMaxMlpLayers], bot_wf[kMaxMlpLayers];
    for (int l = 0; l < m->top_layers; ++l) top_wf[l] = {m->top_w[l], nullptr, nullptr, nullptr};
    for (int l = 0; l < m->bot_layers; ++l) bot_wf[l] = {m->bot_w[l], nullptr, nullptr, nullptr};
    if (wbits) {
        float *wq = quant->wq ? quant->wq : F(L.wq);
        size_t free = L.late;
        dqrm::FqGroup fq{};
        fq.qmax = (float)((1 << (wbits - 1)) - 1);
        int rows = 0;
        auto flush_fq = [&]() -> hipError_t {
            if (fq.count == 0) return hipSuccess;
            fq.total_rows = rows;
            hipLaunchKernelGGL(dqrm::mlp_fake_quant_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, fq);
            fq.count = 0;
            rows = 0;
            return hipGetLastError();
        };
        auto add_fq = [&](const float *W, LayerWeights *wf, int in, int out) -> hipError_t {
            hipError_t e = hipSuccess;
            if (fq.count == dqrm::kGemmMaxGroup) e = flush_fq();
            dqrm::FqLayer &q = fq.l[fq.count++];
            q.W = W, q.Wq = wq, q.out = out, q.in = in, q.row_begin = rows, q.pitch = code_pitch(in);
            q.codes = q.low = nullptr, q.scale = nullptr;
            const LayerCodes at(free, in, out);
            if (at.end <= L.late_end) {
                q.codes = reinterpret_cast<unsigned short *>(ws + at.codes), q.low = reinterpret_cast<unsigned short *>(ws + at.low);
                q.scale = F(at.scale);
                free = at.end;
            }
            rows += out;
            *wf = {wq, q.codes, q.low, q.scale};
            wq += (size_t)out * in;
            return e;
        };
        for (int l = 0; l < m->top_layers; ++l)
            DQRM_HIP_CHECK(add_fq(m->top_w[l], &top_wf[l], m->top_dims[l], m->top_dims[l + 1]));
        for (int l = 0; l < m->bot_layers; ++l)
            DQRM_HIP_CHECK(add_fq(m->bot_w[l], &bot_wf[l], m->bot_dims[l], m->bot_dims[l + 1]));
        DQRM_HIP_CHECK(flush_fq());
    }

    // ---- forward
    // The bottom MLP's last layer rides along in the interaction kernels while its weights are few (64 -> 16 in the
    // paper's Kaggle model; every sample reads them all), a little more of them at small batches, and a first layer with a
    // short reduction (the 13 dense features) has a kernel of its own: both are all launch cost as products on the matrix
    // cores.  (On the matrix cores, 4160 to 4352 floats, us, products -> riding: 256 -> 16 and 26 tables at 256 samples 105.6 ->
    // 99.8, 2048: 157 -> 154, 8192: 404 -> 410; 64 -> 64 and 32 tables at 2048 102.5 -> 97.7, 4096: 144 -> 148.  In the plain
    // kernels, 8320 floats, 256 -> 32 at 64: 51.2 -> 46.9, 1024: 54.5 -> 50.1, 8192: 104 -> 120; 512 -> 32 at 64: 53.7 -> 58.5.)
    const int bl_last = m->bot_layers - 1;
    const int lin_floats = (int)std::min<int64_t>((int64_t)D * dqrm::inter_lin_pitch(m->bot_dims[bl_last]), 1 << 20);
    const bool ride = lin_floats <= inter_lin_floats(T + 1, D, m->bot_dims[bl_last], B);
    const float *x = dense_x;
    for (int l = 0; l < m->bot_layers - (ride ? 1 : 0); ++l) {
        const int in = m->bot_dims[l], out = m->bot_dims[l + 1];
        if (in <= dqrm::kSmallKMax && out % 4 == 0 && aligned(m->bot_b[l], 16)) {
            dqrm::SmallKArgs sk{};
            sk.X = x, sk.W = bot_wf[l].w, sk.bias = m->bot_b[l], sk.Y = F(L.bot_act[l]), sk.B = B, sk.N = out, sk.K = in, sk.relu = 1;
            sk.samples = small_k_samples(B, out);
            hipLaunchKernelGGL(dqrm::linear_small_k_kernel, dim3((B + sk.samples - 1) / sk.samples),
                               dim3(dqrm::kSmallKThreads), 0, st, sk);
            DQRM_HIP_CHECK(hipGetLastError());
        } else {
            DQRM_HIP_CHECK(linear_fwd(st, x, bot_wf[l], m->bot_b[l], F(L.bot_act[l]), B, in, out, true));
        }
        x = F(L.bot_act[l]);
    }
    dqrm::InteractArgs ia{};
    ia.bot = ride ? F(L.bot_act[bl_last]) : x, ia.emb = emb_out, ia.R = F(L.R), ia.B = B, ia.T = T, ia.D = D;
    if (ride) {
        ia.lin_x = x, ia.lin_w = bot_wf[bl_last].w, ia.lin_b = m->bot_b[bl_last], ia.lin_y = F(L.bot_act[bl_last]);
        ia.lin_k = m->bot_dims[bl_last];
    }
    DQRM_HIP_CHECK(launch_interact(st, ia, false, ride ? lin_floats : 0));
    x = F(L.R);
    const int last = m->top_layers - 1;
    for (int l = 0; l < last; ++l) {
        DQRM_HIP_CHECK(linear_fwd(st, x, top_wf[l], m->top_b[l], F(L.top_act[l]), B, m->top_dims[l], m->top_dims[l + 1], true));
        x = F(L.top_act[l]);
    }
    // the last layer (one output), the loss, and the gradient back to that layer's input in one kernel
    unsigned *gmax = reinterpret_cast<unsigned *>(ws + L.gmax);
    dqrm::HeadArgs ha{};
    ha.X = x, ha.w = top_wf[last].w, ha.bias = m->top_b[last], ha.y = labels;
    ha.z = F(L.top_act[last]), ha.dz = F(L.top_dz[last]), ha.terms = F(L.loss_terms);
    ha.dX = last > 0 ? F(L.top_dz[last - 1]) : F(L.dR);
    ha.relu_input = last > 0; // the input of top layer l > 0 is a ReLU output; the interaction output is not
    ha.B = B, ha.in = m->top_dims[last];
    ha.zero = gmax, ha.nzero = gbits ? dqrm::kMaxGradTensors * dqrm::kGradMaxSlots : 0, ha.zstride = dqrm::kGradMaxStride;
    hipLaunchKernelGGL(dqrm::head_kernel, dim3((B + 3) / 4), dim3(256), 0, st, ha);
    DQRM_HIP_CHECK(hipGetLastError());

    // ---- backward: the chain of input gradients first (dZ = gradient w.r.t. a layer's pre-activation) ...
    for (int l = last - 1; l >= 0; --l) {
        const float *in_act = l > 0 ? F(L.top_act[l - 1]) : F(L.R);
        float *dX = l > 0 ? F(L.top_dz[l - 1]) : F(L.dR);
        DQRM_HIP_CHECK(linear_bwd_input(st, F(L.top_dz[l]), top_wf[l], l > 0 ? in_act : nullptr, dX, B,
                                        m->top_dims[l], m->top_dims[l + 1]));
    }
    const float *bot_out = F(L.bot_act[bl_last]);
    ia.bot = bot_out, ia.dR = F(L.dR), ia.dbot = F(L.bot_dz[bl_last]), ia.demb = grad_emb, ia.bot_mask = bot_out;
    const bool ride_back = ride && bl_last > 0; // (a first layer's input gradient is not needed)
    if (ride_back) ia.lin_mask = F(L.bot_act[bl_last - 1]), ia.lin_dx = F(L.bot_dz[bl_last - 1]);
    DQRM_HIP_CHECK(launch_interact(st, ia, true, 0));
    for (int l = bl_last - (ride_back ? 1 : 0); l > 0; --l)
        DQRM_HIP_CHECK(linear_bwd_input(st, F(L.bot_dz[l]), bot_wf[l], F(L.bot_act[l - 1]), F(L.bot_dz[l - 1]), B,
                                        m->bot_dims[l], m->bot_dims[l + 1]));

    // ... then every layer's weight gradient in one launch and the SGD step in another (the input gradients
    // above used the weights of before the step)
    const GradCut cut = grad_cut(m, B);
    dqrm::GemmGroup wg{};
    dqrm::SgdGroup sg{};
    sg.lr = lr;
    if (quant && quant->grad_buffer)
        sg.buffer = quant->grad_buffer, sg.buffer_add = quant->buffer_add != 0, sg.buffer_update = quant->buffer_update != 0;
    if (gbits) {
        sg.grads = quant->grads ? quant->grads : F(L.grads);
        sg.err = quant->grad_error;
        sg.codes = quant->grad_codes;
        sg.gmax_bits = gmax;
        sg.grad_scale = quant->grad_scale;
    }
    long long flat = 0;
    int tensor = 0;
    hipError_t launch_err = hipSuccess;
    auto flush = [&](bool ends_step) {
        if (wg.count == 0 && !ends_step) return;
        if (ends_step) sg.loss_terms = F(L.loss_terms), sg.loss = loss, sg.batch = B; // one more block
        hipError_t e = launch_weight_grads(st, wg);
        if (e != hipSuccess && launch_err == hipSuccess) launch_err = e;
        // (8 workgroups to each CU, the one with the loss among them: one more would start when the others end)
        const unsigned blocks = (unsigned)std::min<long long>((sg.total + 255) / 256, num_cus() * 8 - 1);
        const dim3 last_grid(blocks + (ends_step ? 1u : 0u));
        if (gbits) {
            if (blocks) hipLaunchKernelGGL(dqrm::grad_sum_absmax_kernel, dim3(blocks), dim3(256), 0, st, sg);
            hipLaunchKernelGGL(dqrm::grad_quant_ec_kernel, last_grid, dim3(256), 0, st, sg);
        } else {
            hipLaunchKernelGGL(dqrm::sgd_from_partials_kernel, last_grid, dim3(256), 0, st, sg);
        }
        e = hipGetLastError();
        if (e != hipSuccess && launch_err == hipSuccess) launch_err = e;
        wg.count = 0;
        sg.count = 0;
        sg.total = 0;
    };
    auto add_layer = [&](const float *dZ, const float *X, float *W, float *b, float *part, int in, int out) {
        if (wg.count == dqrm::kGemmMaxGroup) flush(false);
        const dqrm::GemmArgs g = weight_grad_problem(dZ, X, part, B, in, out, cut);
        wg.p[wg.count++] = g;
        dqrm::SgdLayer &s = sg.l[sg.count++];
        s.P = part, s.W = W, s.b = b, s.S = g.splits, s.out = out, s.in = in, s.elem_begin = sg.total;
        s.flat_begin = flat, s.tensor0 = tensor;
        s.by_cols = dqrm::FastDiv::make((unsigned)in + 1u);
        if ((long long)out * (in + 1) > 2147483647LL) s.by_cols.d = 0;
        sg.total += (long long)out * (in + 1);
        flat += (long long)out * (in + 1);
        tensor += 2;
    };
    for (int l = 0; l < m->top_layers; ++l)
        add_layer(F(L.top_dz[l]), l > 0 ? F(L.top_act[l - 1]) : F(L.R), m->top_w[l], m->top_b[l], F(L.top_part[l]),
                  m->top_dims[l], m->top_dims[l + 1]);
    for (int l = 0; l < m->bot_layers; ++l)
        add_layer(F(L.bot_dz[l]), l > 0 ? F(L.bot_act[l - 1]) : dense_x, m->bot_w[l], m->bot_b[l], F(L.bot_part[l]),
                  m->bot_dims[l], m->bot_dims[l + 1]);
    flush(true);
    DQRM_HIP_CHECK(launch_err);
    DQRM_HIP_CHECK(hipGetLastError());
    return DQRM_OK;
}

int32_t dqrm_check_status(void *stream, int32_t *first_bad_table, int64_t *first_bad_index)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    DQRM_HIP_CHECK(hipStreamSynchronize(st));
    dqrm::DeviceStatus h;
    DQRM_HIP_CHECK(hipMemcpyFromSymbol(&h, HIP_SYMBOL(dqrm::g_status), sizeof(h), 0, hipMemcpyDeviceToHost));
    if (h.code != 0) {
        dqrm::DeviceStatus z{0, 0, 0};
        DQRM_HIP_CHECK(hipMemcpyToSymbol(HIP_SYMBOL(dqrm::g_status), &z, sizeof(z), 0, hipMemcpyHostToDevice));
    }
    if (first_bad_table) *first_bad_table = h.code ? h.table : -1;
    if (first_bad_index) *first_bad_index = h.code ? h.value : -1;
    return h.code;
}


} // extern "C"
