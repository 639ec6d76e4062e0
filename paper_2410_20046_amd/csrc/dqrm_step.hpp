// dqrm_fwd_bwd_step: the kernels of a whole step of the tables, where more can go into a launch than the calls it stands for
// can put there one by one.
//
// step_sort_kernel: the forward and the sort of the batch (dqrm_dedupe.hpp, kernel 1) need nothing of each other, so they share a
//   launch: the first workgroups sort, the others are the forward's tiles.
// step_table_kernel: behind the sort, for tables of few lookups: a workgroup per table takes it from the sort's lists to its updated
//   rows (what dedupe_finish_kernel, segment_sum_kernel and quant_update_kernel do in three launches).
#pragma once

#include "dqrm_bwd.hpp"
#include "dqrm_dedupe.hpp"
#include "dqrm_fwd.hpp"
#include "dqrm_update.hpp"

namespace dqrm {

// Bound by the sort's chains (dedupe_kernel), as long as the forward's tiles fit beside them: a workgroup of either kind has the
// same threads and one piece of LDS.  26 tables x 2048 lookups x 16: 12.3 us against 4.4 + 11.6 in two launches.
template <int THREADS, int CAP, int G, bool PACKED>
__global__ __launch_bounds__(THREADS) void step_sort_kernel(DedupeArgs d, FwdArgs f, int sort_groups, int tiles_b)
{
    constexpr size_t kDedupe = sizeof(DedupeLds<THREADS, CAP>), kFwd = sizeof(FwdLds<THREADS>);
    __shared__ __align__(16) char lds[kDedupe > kFwd ? kDedupe : kFwd];
    const int b = (int)blockIdx.x;
    if (b < sort_groups) { // (workgroup-uniform)
        dedupe_body<THREADS, CAP, false, true>(d, *reinterpret_cast<DedupeLds<THREADS, CAP> *>(lds), b % d.T, 0, b / d.T);
    } else {
        const int i = b - sort_groups;
        embbag_fwd_body<THREADS, G, PACKED>(f, *reinterpret_cast<FwdLds<THREADS> *>(lds), i % tiles_b, i / tiles_b);
    }
}

constexpr int kStepThreads = 1024, kStepWaves = kStepThreads / kWave;
constexpr int kStepParts = 64;         // ranges of a table, at most: a lane each
constexpr int kStepLongSegments = 2048; // segments of more than one chunk
static_assert(kDdMaxRanges <= kStepParts && DQRM_MAX_TABLE_LOOKUPS / (DQRM_SEG_CHUNK + 1) < kStepLongSegments, "room for a table's lists");
constexpr int kStepSingles = 4;        // singles a group has in flight
constexpr int kStepLongBatch = 8;      // chunk sums of a segment of more than one chunk that a lane has in flight
constexpr int kStepRows = 4096;        // segments whose rows stay in LDS for the update
constexpr int kStepPerThread = 4;      // float4 elements of the update that a thread has in flight

struct StepTableArgs {
    DedupeArgs d; // (one batch)
    SegArgs s;
    QuantUpdateArgs q;
    int sum_blocks; // workgroups that segment_sum_kernel would have
};

// Bound by a chain of about ten round trips of a microsecond (counts, lists, bags, rows, parked sums, values, weights) and, from
// about 100 KB of rows per table on, by what one CU can have in flight.  The lists it reads are each range's own, in their places; the
// dense ones are written beside the sums, so that the workspace serves a later dqrm_segment_sum (the chunks in sorted order, also
// where dedupe_finish_kernel puts the long ones first: a sum over few chunks gains nothing by that).  Rows of the update stay in
// LDS, which lets its weights, the only data that come from far, be requested before the long segments are added up.  More loads to a
// thread in flight, or the first ones of both lists requested together, cost more in registers and code than they save.
// 4 tables x 128 lookups x 16: the step 20.5 -> 14.6 us (passes one behind the other, code warm); 26 x 2048 x 16: 36.3 -> 33.5.
template <int G>
__global__ __launch_bounds__(kStepThreads) void step_table_kernel(StepTableArgs a)
{
    constexpr int kGroups = kStepThreads / G;
    constexpr int kSums = 5; // before my table: segments, chunks, singles, further ranges; my further ranges
    __shared__ int s_sum[kSums][kStepWaves];
    __shared__ int4 s_info[2 * kStepParts]; // part_info of my ranges; the further ones by their number, modulo kStepParts
    __shared__ int s_base[kStepParts], s_uniq[kStepParts + 1], s_chunk[kStepParts + 1], s_single[kStepParts + 1];
    __shared__ unsigned s_max[kAbsmaxSlots];
    __shared__ int4 s_long[kStepLongSegments]; // sorted position of the head, chunks, global segment, slot of the maximum
    __shared__ unsigned s_row[kStepRows];
    __shared__ int s_longs;

    const DedupeBatch &bt = a.d.b[0];
    const BwdWs &ws = bt.ws;
    const int t = (int)blockIdx.x, T = a.d.T, parts = a.d.parts, D = a.s.D;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    if (tid < kAbsmaxSlots) s_max[tid] = 0u;
    if (tid == kWave) s_longs = 0;

    // ---- what the tables before mine have, and my ranges' lists
    const int V = T * parts;
    {
        int sum[kSums] = {};
        auto count = [&](int v, int table, bool further, const int4 &x) {
            if (table < t) sum[0] += x.y, sum[1] += x.z, sum[2] += x.w, sum[3] += further;
            if (table == t) sum[4] += further, s_info[further ? kStepParts + ((v - V) & (kStepParts - 1)) : v - t * parts] = x;
        };
        for (int v = tid; v < V; v += kStepThreads) count(v, (int)a.d.by_parts.div((unsigned)v), false, ws.part_info[2 * v]);
        const int more = a.d.extra > 0 ? min(ws.totals[3], a.d.extra) : 0;
        for (int v = V + tid; v < V + more; v += kStepThreads) // (a further range knows its place in the order of all, and with it its table)
            count(v, (int)a.d.by_parts.div((unsigned)(ws.part_info[2 * v + 1].w - (v - V))) - 1, true, ws.part_info[2 * v]);
#pragma unroll
        for (int k = 0; k < kSums; ++k) {
            const int incl = wave_incl_scan_add(sum[k], lane);
            if (lane == kWave - 1) s_sum[k][wave] = incl;
        }
    }
    __syncthreads();
    auto total = [&](int k) {
        return __builtin_amdgcn_readlane(wave_incl_scan_add(lane < kStepWaves ? s_sum[k][lane] : 0, lane), kStepWaves - 1);
    };
    const int u0 = total(0), c0 = total(1), single0 = total(2), e0 = total(3), np = parts + total(4);
    int U, C, S;
    { // (every wave by itself; the first one leaves it in LDS)
        const int4 x = lane < parts ? s_info[lane] : lane < np ? s_info[kStepParts + ((e0 + lane - parts) & (kStepParts - 1))] : make_int4(0, 0, 0, 0);
        const int u = wave_incl_scan_add(x.y, lane), c = wave_incl_scan_add(x.z, lane), s = wave_incl_scan_add(x.w, lane);
        U = __builtin_amdgcn_readlane(u, kWave - 1), C = __builtin_amdgcn_readlane(c, kWave - 1), S = __builtin_amdgcn_readlane(s, kWave - 1);
        if (wave == 0) s_base[lane] = x.x, s_uniq[lane] = u - x.y, s_chunk[lane] = c - x.z, s_single[lane] = s - x.w;
    }
    if (tid == 0) {
        bt.tuo[t] = u0;
        if (t == T - 1) {
            bt.tuo[T] = u0 + U;
            *bt.num_unique = u0 + U;
            bt.seg_offsets[u0 + U] = (int32_t)bt.N;
            ws.totals[0] = c0 + C;
            ws.totals[1] = u0 + U;
            ws.totals[2] = single0 + S;
        }
    }
    __syncthreads();

    // ---- segment sums; the dense lists beside them
    const int lg = tid & (G - 1), grp = tid / G, leader = lane & ~(G - 1);
    const int col = lg * 4;
    const bool col_ok = col < D;
    const unsigned tD = (unsigned)T * (unsigned)D;
    const float *grad = a.s.grad_out + (unsigned)t * (unsigned)D + (col_ok ? col : 0);
    auto add_max = [&](int slot, float v) {
        const unsigned b = __float_as_uint(v);
        if (b > s_max[slot]) atomicMax(s_max + slot, b);
    };
    auto file_row = [&](int j, int pos, int row) { // (by one lane of the group)
        bt.uniq_rows[j] = (int64_t)(unsigned)row;
        bt.seg_offsets[j] = pos;
        if (j - u0 < kStepRows) s_row[j - u0] = (unsigned)row;
    };
    for (int i0 = grp; __builtin_amdgcn_readfirstlane(i0) < S; i0 += kStepSingles * kGroups) {
        int4 d[kStepSingles]; // {sorted position, bag, segment, row}
        int j[kStepSingles];
        float4 r[kStepSingles];
#pragma unroll
        for (int k = 0; k < kStepSingles; ++k) {
            const int i = min(i0 + k * kGroups, S - 1), p = table_of(s_single, np, i);
            d[k] = ws.single_local[s_base[p] + (i - s_single[p])];
            j[k] = u0 + s_uniq[p];
        }
#pragma unroll
        for (int k = 0; k < kStepSingles; ++k) r[k] = load_row_f4<true>(grad + (uint64_t)(unsigned)d[k].y * tD);
#pragma unroll
        for (int k = 0; k < kStepSingles; ++k) {
            const int i = i0 + k * kGroups;
            if (i >= S) continue;
            j[k] += d[k].z;
            if (lg == 0) {
                file_row(j[k], d[k].x, d[k].w);
                ws.single_desc[single0 + i] = make_int4(d[k].y, j[k], t, 0);
            }
            if (col_ok) {
                *reinterpret_cast<float4 *>(a.s.values + (int64_t)j[k] * D + col) = r[k];
                add_max(single_absmax_slot(single0 + i, a.sum_blocks, G), f4_absmax(r[k]));
            }
        }
    }
    for (int c = grp; __builtin_amdgcn_readfirstlane(c) < C; c += kGroups) {
        const bool live = c < C;
        const int cc = min(c, C - 1), p = table_of(s_chunk, np, cc);
        const int4 d = ws.chunk_local[s_base[p] + (cc - s_chunk[p])];
        const int len = min(desc_len(d), DQRM_SEG_CHUNK), kchunk = desc_kchunk(d), nchunks = desc_nchunks(d);
        const int j = u0 + s_uniq[p] + (d.z & 0xFFFF), place = c0 + cc;
        int my_bags[kChunkIdsPerLane(G)]; // (past the chunk's end: its last bag again)
#pragma unroll
        for (int q = 0; q < kChunkIdsPerLane(G); ++q) my_bags[q] = ws.sorted_bag[d.x + min(q * G + lg, len - 1)];
        const int wave_len = __builtin_amdgcn_readfirstlane(wave_max_int(len));
        const float4 acc = sum_chunk<G, true>(my_bags, len, wave_len, leader, grad, tD);
        if (!live) continue;
#pragma unroll
        for (int q = 0; q < kChunkIdsPerLane(G); ++q)
            if (q * G + lg < DQRM_SEG_CHUNK) ws.chunk_bags[(int64_t)place * DQRM_SEG_CHUNK + q * G + lg] = my_bags[q];
        const int slot = chunk_absmax_slot(place, a.sum_blocks, G);
        if (lg == 0) {
            ws.chunk_desc[place] = make_int4(d.x, d.y, j, t);
            if (kchunk == 0) {
                file_row(j, d.x, d.w);
                if (nchunks > 1) s_long[atomicAdd(&s_longs, 1)] = make_int4(d.x, nchunks, j, slot);
            }
        }
        if (!col_ok) continue;
        if (nchunks > 1) {
            *reinterpret_cast<float4 *>(partial_slot(ws, d.x - kchunk * DQRM_SEG_CHUNK, kchunk, nchunks, D) + col) = acc;
        } else {
            *reinterpret_cast<float4 *>(a.s.values + (int64_t)j * D + col) = acc;
            add_max(slot, f4_absmax(acc));
        }
    }
    __syncthreads();

    // ---- the first rows of the update are requested now: they are the ones that come from memory
    const unsigned q4 = a.q.u.by_q4.d;
    const unsigned elements = (unsigned)max((int64_t)0, min((int64_t)U, a.q.u.capacity - u0)) * q4;
    const int64_t r0 = a.d.row_offsets[t];
    float4 w[kStepPerThread];
    auto element = [&](unsigned first, int k) { return min(first + k * kStepThreads + tid, elements - 1); };
    auto place_of = [&](unsigned e) { // of element e of the table's values in the master table
        const unsigned u = a.q.u.by_q4.div(e);
        return (r0 + (u < kStepRows ? (int64_t)s_row[u] : bt.uniq_rows[u0 + u])) * q4 + (e - u * q4);
    };
    auto request_weights = [&](unsigned first) {
#pragma unroll
        for (int k = 0; k < kStepPerThread; ++k)
            if (first + k * kStepThreads < elements) w[k] = reinterpret_cast<const float4 *>(a.q.u.master)[place_of(element(first, k))]; // (workgroup-uniform)
    };
    request_weights(0);

    // ---- segments of more than one chunk
    const int longs = s_longs;
    for (int m = grp; __builtin_amdgcn_readfirstlane(m) < longs; m += kGroups) {
        const int4 e = s_long[min(m, longs - 1)];
        const int wave_n = __builtin_amdgcn_readfirstlane(wave_max_int(e.y));
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int k0 = 0; k0 < wave_n; k0 += kStepLongBatch) {
            float4 v[kStepLongBatch];
#pragma unroll
            for (int q = 0; q < kStepLongBatch; ++q)
                v[q] = *reinterpret_cast<const float4 *>(partial_slot(ws, e.x, min(k0 + q, e.y - 1), e.y, D) + (col_ok ? col : 0));
#pragma unroll
            for (int q = 0; q < kStepLongBatch; ++q)
                if (k0 + q < e.y) acc = k0 + q == 0 ? v[q] : f4_add(acc, v[q]);
        }
        // (the maximum is of the whole row, as segment_sum_kernel takes it: NaN only if all of a narrow row is, else hidden by the others)
        float row_max = col_ok ? f4_absmax(acc) : 0.0f;
        if (G >= 16) row_max = fmaxf(row_max, 0.0f);
#pragma unroll
        for (int o = G / 2; o >= 1; o >>= 1) row_max = fmaxf(row_max, __shfl_xor(row_max, o, kWave));
        if (m < longs) {
            if (col_ok) *reinterpret_cast<float4 *>(a.s.values + (int64_t)e.z * D + col) = acc;
            if (lg == 0) add_max(e.w, row_max);
        }
    }
    __syncthreads();

    // ---- scale, codes, update
    float amax = 0.0f;
#pragma unroll
    for (int k = 0; k < kAbsmaxSlots; ++k) amax = fmaxf(amax, __uint_as_float(s_max[k]));
    const Scale gs(scale_from_absmax(amax, 127.0f));
    Scale wsc(1.0f, 1.0f);
    if (a.q.u.packed) wsc = Scale(a.q.u.w_scale[t]);
    if (tid < kAbsmaxSlots) *absmax_slot(ws.absmax_slots, t, tid) = __uint_as_float(s_max[tid]);
    if (tid == 0) {
        a.q.g_absmax[t] = amax;
        a.q.g_scale_out[t] = gs.s;
    }
    float4 *values = reinterpret_cast<float4 *>(a.s.values) + (int64_t)u0 * q4;
    for (unsigned first = 0; first < elements; first += kStepThreads * kStepPerThread) {
        if (first > 0) request_weights(first);
        float4 v[kStepPerThread];
#pragma unroll
        for (int k = 0; k < kStepPerThread; ++k)
            if (first + k * kStepThreads < elements) v[k] = values[element(first, k)];
#pragma unroll
        for (int k = 0; k < kStepPerThread; ++k) {
            const unsigned e = first + k * kStepThreads + tid;
            if (e >= elements) continue;
            const int64_t at = place_of(e);
            const int q0 = int8_code(v[k].x, gs), q1 = int8_code(v[k].y, gs), q2 = int8_code(v[k].z, gs), q3 = int8_code(v[k].w, gs);
            reinterpret_cast<unsigned *>(a.q.gq_out)[(int64_t)u0 * q4 + e] = pack_bytes(q0, q1, q2, q3);
            const float4 x = sgd_step(w[k], q0, q1, q2, q3, gs.s, a.q.u.lr);
            reinterpret_cast<float4 *>(a.q.u.master)[at] = x;
            if (a.q.u.packed) reinterpret_cast<unsigned short *>(a.q.u.packed)[at] = encode4(x, wsc);
        }
    }
}

} // namespace dqrm
