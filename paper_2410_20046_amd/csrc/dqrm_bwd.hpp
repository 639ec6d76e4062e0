// Segment sums: the "specified sparsity" gradient of Sec. 4.3 / the gradient-quantisation appendix, from the work lists
// that dqrm_dedupe leaves in the workspace (dqrm_dedupe.hpp).
//
// segment_sum_kernel: one lane group per chunk (<= DQRM_SEG_CHUNK consecutive contributions of one segment) adds its
//   gradient rows left to right.  A segment of one chunk is final.  The chunks of a longer segment park their sums and
//   count themselves in on the segment's counter; the wave of the chunk that arrives last adds the segment's chunk sums
//   in chunk order.  Which wave that is depends on scheduling; what it computes does not.
// absmax_finalize_kernel: folds the per-table maxima.
// segment_sum_multi_kernel / absmax_finalize_multi_kernel: the same for several batches in one launch.
#pragma once

#include "dqrm_dedupe.hpp"
#include "dqrm_device.hpp"

namespace dqrm {

constexpr int kSumThreads = 256;   // segment_sum_kernel
constexpr int kSegBatch = 16;      // gradient rows requested before the first is added
constexpr int kSumBlocksPerCu = 4; // grid of segment_sum_kernel, in workgroups per CU (128 registers per lane)

// ---------------------------------------------------------------------------
// dqrm_segment_sum: chunk sums, then the combine of long segments, then absmax.

struct SegArgs {
    const float *grad_out;
    BwdWs ws;
    float *values;
    float *g_absmax;
    int64_t N;
    int T, B, D;
};

__device__ __forceinline__ float4 f4_add(float4 a, float4 b)
{
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// 16 bytes of a gradient row.  With bags of one lookup a row is added into one segment and read once: by a streaming load, so that
// it does not push the lists and sums that are read again out of the caches (62.3 -> 60.7 us per step that way).  A row of a
// bag of several lookups (REUSE) is read once for each, and is to stay in the cache (26 tables x 65536 lookups in bags of 8: the step
// 341 -> 321 us with plain loads).
template <bool REUSE>
__device__ __forceinline__ float4 load_row_f4(const float *p)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    if (REUSE) return *reinterpret_cast<const float4 *>(p);
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float f4_absmax(float4 a)
{
    return fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w)));
}

// Per-block maxima of |values| by table, kept in LDS (bit patterns of
// non-negative floats order like unsigned integers) and flushed once per block.
struct BlockAbsmax {
    unsigned *s_max; // [T] in LDS
    __device__ __forceinline__ void init(unsigned *lds, int T)
    {
        s_max = lds;
        for (int k = threadIdx.x; k < T; k += blockDim.x) s_max[k] = 0u;
        // the caller synchronises before the first add()
    }
    __device__ __forceinline__ void add(int t, float v)
    {
        const unsigned b = __float_as_uint(v);
        if (b > s_max[t]) atomicMax(s_max + t, b);
    }
    // all threads of the block; publishes the block's maxima
    __device__ __forceinline__ void flush(float *slots, int T)
    {
        __syncthreads();
        for (int k = threadIdx.x; k < T; k += blockDim.x) {
            const unsigned b = s_max[k];
            if (b != 0u)
                atomicMax(reinterpret_cast<unsigned *>(absmax_slot(slots, k, blockIdx.x & (kAbsmaxSlots - 1))), b);
        }
    }
};

// entries of a chunk's bag list that each lane of a group of g lanes holds
constexpr int kChunkIdsPerLane(int g) { return (DQRM_SEG_CHUNK + g - 1) / g; }

// The chunk's bag list: each lane fetches its share once (the whole 32-entry record, whatever the chunk's
// length: the list sits at a place known from the chunk's index, so no descriptor is needed to ask for it).
template <int G>
__device__ __forceinline__ void load_chunk_bags(const SegArgs &a, int c, int lg, int (&my_bags)[kChunkIdsPerLane(G)])
{
    const int *bags = a.ws.chunk_bags + (int64_t)c * DQRM_SEG_CHUNK;
#pragma unroll
    for (int q = 0; q < kChunkIdsPerLane(G); ++q) {
        const int i = q * G + lg;
        my_bags[q] = i < DQRM_SEG_CHUNK ? bags[i] : 0;
    }
}

// Sum of one chunk: its gradient rows, left to right.
//
// Every load of a batch is issued before the first is used, and none sits under a
// per-lane branch: a lane without a row at position i reads the row of bag 0
// instead and leaves it out of the sum.  (With loads under divergent branches the
// compiler cannot count the loads in flight and waits for all of them before each
// next one.)  `wave_len` is the longest chunk among the wave's groups: batches
// and quarters of batches beyond it are skipped by the whole wave.
template <int G, bool REUSE>
__device__ __forceinline__ float4 sum_chunk(const int (&my_bags)[kChunkIdsPerLane(G)], int len, int wave_len, int leader,
                                            const float *g0, unsigned tD)
{
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int kBatch = kSegBatch, kQuarter = kBatch / 4;
#pragma unroll
    for (int i0 = 0; i0 < DQRM_SEG_CHUNK; i0 += kBatch) {
        if (i0 < wave_len) {
            float4 g[kBatch];
#pragma unroll
            for (int q0 = 0; q0 < kBatch; q0 += kQuarter) {
                if (q0 == 0 || i0 + q0 < wave_len) {
#pragma unroll
                    for (int q = q0; q < q0 + kQuarter; ++q) {
                        const int i = i0 + q;
                        int b = __shfl(my_bags[i / G], leader + (i % G), kWave); // the group passes the bags round
                        b = i < len ? b : 0;
                        g[q] = load_row_f4<REUSE>(g0 + (uint64_t)(unsigned)b * tD);
                    }
                } else {
#pragma unroll
                    for (int q = q0; q < q0 + kQuarter; ++q) g[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int i = i0 + q;
                if (i < len) acc = (i == 0) ? g[q] : f4_add(acc, g[q]);
            }
        }
    }
    return acc;
}

// Where the sum of chunk k of a segment of more than one chunk is parked: full chunks are disjoint runs of
// DQRM_SEG_CHUNK sorted positions, so (position / DQRM_SEG_CHUNK) names them uniquely; the last chunk of a
// segment is filed under the slot of the segment's first chunk, in a second array.  The segment's arrival
// counter sits at the first chunk's slot number too.
__device__ __forceinline__ float *partial_slot(const BwdWs &ws, int head_pos, int k, int nchunks, int D)
{
    return k == nchunks - 1 ? ws.partial_last + (int64_t)(head_pos / DQRM_SEG_CHUNK) * D
                            : ws.partial_full + (int64_t)(head_pos / DQRM_SEG_CHUNK + k) * D;
}

// Parked chunk sums and arrival counters are the only data that one workgroup of this kernel hands to another.
// They travel by device-scope atomic stores, loads and adds (each coherent across the chip by itself: they go
// past the caches that are private to a part of the chip), in this order: a chunk's sum is stored and the
// stores are waited for; then the chunk is counted in; the wave that sees the count complete then loads the
// sums.  No fence is used: a device-scope release or acquire writes back or drops whole caches, which costs more
// than the entire kernel when thousands of waves do it.
__device__ __forceinline__ void park_f4(float *p, float4 v)
{
    unsigned long long *to = reinterpret_cast<unsigned long long *>(p); // (16-byte aligned)
    auto two = [](float a, float b) { return (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32); };
    __hip_atomic_store(to + 0, two(v.x, v.y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(to + 1, two(v.z, v.w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kCombineBatch = 64; // chunk sums of one column requested together

// The sum of a segment of `nchunks` > 1 chunks, 64 columns of it from `base` on: its parked chunk sums, left to right, by a whole
// wave; lane l ends with column base + combine_col(l).  A load is 16 bytes a lane, of four chunks' rows (a sixteenth of the lanes
// each); the four are then turned, so that a lane has one column of all four.  The loads' cache policy is that of a device-scope
// atomic load.  Those past the last full chunk or the last column read that one again: every address lies in the segment's own
// rows (the whole offset is in the vector one, the part that the hardware checks).  (4 bytes a lane, 64 loads per trip: a segment of
// 300 chunks took 20 to 30 us beside the others' work, now 9 to 13; the kernel at 26 tables x 8192 lookups of bags of one 24.4 -> 22.2 us.)
__device__ __forceinline__ int combine_col(int lane) { return 4 * (lane & 15) + (lane >> 4); }

__device__ __forceinline__ float combine_columns(const BwdWs &ws, int head_pos, int nchunks, int D, int base, int lane)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int kAgentScope = 16; // sc1
    constexpr int kLoads = kCombineBatch / 4;
    const int full = nchunks - 1; // chunks filed under their positions (at most 2047 rows of 1 KB); the last one is elsewhere
    const int64_t slot = (int64_t)(head_pos / DQRM_SEG_CHUNK) * D;
    const float last = __hip_atomic_load(ws.partial_last + slot + min(base + combine_col(lane), D - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(ws.partial_full + slot, 0, full * D * (int)sizeof(float), 0x00020000);
    const int row = D * (int)sizeof(float), col = min(base + 4 * (lane & 15), D - 4) * (int)sizeof(float);
    int at = (lane >> 4) * row + col;
    const int at_last = (full - 1) * row + col;
    float acc = 0.f;
    for (int k0 = 0; k0 < full; k0 += kCombineBatch) {
        u32x4 v[kLoads];
#pragma unroll
        for (int q0 = 0; q0 < kLoads; q0 += 4)
            if (q0 == 0 || k0 + 4 * q0 < full) // (wave-uniform)
#pragma unroll
                for (int q = q0; q < q0 + 4; ++q) {
                    v[q] = __builtin_amdgcn_raw_buffer_load_b128(rows, min(at, at_last), 0, kAgentScope);
                    at += 4 * row;
                    asm volatile("" : "+v"(at)); // (one offset, not 16 in as many registers)
                }
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            if (k0 + 4 * q < full) {
                const u32x2 a = __builtin_amdgcn_permlane32_swap(v[q][0], v[q][2], false, false);
                const u32x2 b = __builtin_amdgcn_permlane32_swap(v[q][1], v[q][3], false, false);
                const u32x2 c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
                const unsigned sums[4] = {c[0], c[1], d[0], d[1]};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + 4 * q + k < full) acc = (k0 + 4 * q + k == 0) ? __uint_as_float(sums[k]) : acc + __uint_as_float(sums[k]);
            }
        }
    }
    return acc + last;
}

// One column of such a sum for rows narrower than a wave: the wave's lanes are split among several segments, so `head_pos` and
// `nchunks` differ from lane to lane (nchunks = 0: a lane without a column to add).  All lanes go through the
// motions up to `wave_n`, the largest nchunks in the wave; a lane past its own last chunk asks for that chunk again.
__device__ __forceinline__ float combine_column_shared_wave(const BwdWs &ws, int head_pos, int nchunks, int wave_n, int D,
                                                            int col)
{
    float acc = 0.f;
    for (int k0 = 0; k0 < wave_n; k0 += kCombineBatch) {
        float pv[kCombineBatch];
#pragma unroll
        for (int q = 0; q < kCombineBatch; ++q) {
            pv[q] = 0.f;
            if (k0 + q < wave_n) {
                const float *p = nchunks > 0 ? partial_slot(ws, head_pos, min(k0 + q, nchunks - 1), nchunks, D) + col
                                             : ws.partial_full;
                pv[q] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
#pragma unroll
        for (int q = 0; q < kCombineBatch; ++q)
            if (k0 + q < nchunks) acc = (k0 + q == 0) ? pv[q] : acc + pv[q];
    }
    return acc;
}

// Work of one workgroup of kSumThreads / G lane groups:
//  * singles (rows looked up once: a plain copy of one gradient row), a few per
//    group, spread evenly over all groups of the grid;
//  * chunks, one per lane group and round.  The sum of a segment's only chunk is
//    final.  The sum of a chunk of a longer segment is parked; the chunk then counts
//    itself in, and if it completes its segment's count, its whole wave (a lane per
//    column) adds the segment's parked sums in chunk order, stores the row of
//    `values`, and clears the counter for the next use.
// No load sits under a per-lane branch: a group without work goes through the
// motions on bag 0 of table 0 and stores nothing.
constexpr int kSinglesPerGroup = 4;

// The slot that a maximum of single i, or of chunk c of a list of any order, is flushed to with `blocks` workgroups and G lanes to a
// group.  A slot whose maximum is NaN counts as none, so where there are NaN it matters which values share one.  (A segment of more
// than one chunk has one maximum, of its whole row, which is flushed to the slot of any of its chunks: whichever arrives last.  In a list
// ordered by length the places inside a class are dealt as the sort's lanes arrive, so there it is open which values share a slot.)
__device__ __forceinline__ int single_absmax_slot(int i, int blocks, int G)
{
    const unsigned groups = (unsigned)(kSumThreads / G);
    return (int)((unsigned)i / kSinglesPerGroup % (blocks * groups) / groups) & (kAbsmaxSlots - 1);
}
__device__ __forceinline__ int chunk_absmax_slot(int c, int blocks, int G)
{
    const unsigned groups = (unsigned)(kSumThreads / G), waves = kSumThreads / kWave;
    const unsigned g = (unsigned)c % (blocks * groups);
    return (int)(G < 16 ? g % (blocks * waves) / waves : g / groups) & (kAbsmaxSlots - 1);
}

template <int G, bool REUSE>
__device__ __forceinline__ void segment_sum_body(const SegArgs &a)
{
    constexpr int kGroups = kSumThreads / G; // lane groups per workgroup
    __shared__ unsigned s_max[DQRM_MAX_TABLES];
    const int T = a.T, D = a.D;
    BlockAbsmax amax;
    amax.init(s_max, T);

    const int lg = threadIdx.x & (G - 1);
    const int grp = (int)threadIdx.x / G;
    const int col = lg * 4;
    const bool col_ok = col < D;
    const float *grad_col = a.grad_out + (col_ok ? col : 0); // lanes beyond the row read column 0 and store nothing
    const int lane = threadIdx.x & (kWave - 1);
    const int leader = lane & ~(G - 1);
    const unsigned tD = (unsigned)T * (unsigned)D;
    const int cap = (int)a.N;       // both lists have N slots, so descriptors may be requested before the counts are known
    const int cap_chunks = cap / 2; // a chunk has at least two lookups
    const int ngroups = (int)gridDim.x * kGroups;
    const int gi = (int)blockIdx.x * kGroups + grp;

    // ---- requests that need no count: the first chunk's descriptor and bag list, the first singles
    // Wide rows: consecutive chunks for the groups of a wave (they are alike in length, so few lanes idle).  Narrow
    // rows (many groups per wave): the wave's groups take chunks a whole grid's waves apart, or the chunks of a small
    // table's rows would all complete their segments in one wave, which adds them up a few per round trip.
    int c = gi;
    if constexpr (G < 16) {
        constexpr int kWavesPerBlock = kSumThreads / kWave, kGroupsPerWave = kWave / G;
        c = ((int)blockIdx.x * kWavesPerBlock + (int)threadIdx.x / kWave) + (grp % kGroupsPerWave) * ((int)gridDim.x * kWavesPerBlock);
    }
    int4 d = make_int4(0, 0, 0, 0);
    int my_bags[kChunkIdsPerLane(G)] = {};
    if (c < cap_chunks) {
        d = a.ws.chunk_desc[c];
        load_chunk_bags<G>(a, c, lg, my_bags);
    }
    int s0 = gi * kSinglesPerGroup;
    int4 sd[kSinglesPerGroup];
#pragma unroll
    for (int k = 0; k < kSinglesPerGroup; ++k) sd[k] = a.ws.single_desc[min(s0 + k, max(cap - 1, 0))];
    const int C = min(a.ws.totals[0], cap_chunks), S = min(a.ws.totals[2], cap);
    __syncthreads(); // s_max is cleared

    // ---- singles: the wave's first group holds the lowest positions
    while (__builtin_amdgcn_readfirstlane(s0) < S) {
        float4 r[kSinglesPerGroup];
        int4 cur[kSinglesPerGroup];
#pragma unroll
        for (int k = 0; k < kSinglesPerGroup; ++k) {
            cur[k] = s0 + k < S ? sd[k] : make_int4(0, 0, 0, 0);
            r[k] = load_row_f4<REUSE>(grad_col + (uint64_t)(unsigned)cur[k].x * tD + (unsigned)cur[k].z * (unsigned)D);
        }
        const int s_next = s0 + ngroups * kSinglesPerGroup;
#pragma unroll
        for (int k = 0; k < kSinglesPerGroup; ++k) sd[k] = a.ws.single_desc[min(s_next + k, cap - 1)];
#pragma unroll
        for (int k = 0; k < kSinglesPerGroup; ++k) {
            if (s0 + k < S && col_ok) {
                *reinterpret_cast<float4 *>(a.values + (int64_t)cur[k].y * D + col) = r[k];
                amax.add(cur[k].z, f4_absmax(r[k]));
            }
        }
        s0 = s_next;
    }

    // ---- chunks: the wave's first group holds the lowest index
    while (__builtin_amdgcn_readfirstlane(c) < C) {
        const int c_next = c + ngroups;
        int4 d_next = make_int4(0, 0, 0, 0);
        int next_bags[kChunkIdsPerLane(G)] = {};
        if (__builtin_amdgcn_readfirstlane(c_next) < C) { // whole wave or none; groups past C - 1 read slots that exist
            d_next = a.ws.chunk_desc[min(c_next, cap_chunks - 1)];
            load_chunk_bags<G>(a, min(c_next, cap_chunks - 1), lg, next_bags);
        }
        const bool live = c < C;
        int len = live ? desc_len(d) : 0;
        len = len > DQRM_SEG_CHUNK ? DQRM_SEG_CHUNK : len;
        const int wave_len = __builtin_amdgcn_readfirstlane(wave_max_int(len));
        const int nchunks = desc_nchunks(d), kchunk = desc_kchunk(d);
        const int t = live ? d.w : 0;
        const float4 acc = sum_chunk<G, REUSE>(my_bags, len, wave_len, leader, grad_col + (unsigned)t * (unsigned)D, tD);
        const bool parks = live && nchunks > 1;
        const int head_pos = d.x - kchunk * DQRM_SEG_CHUNK; // sorted position of the segment's head
        if (live && col_ok) {
            if (parks) {
                park_f4(partial_slot(a.ws, head_pos, kchunk, nchunks, D) + col, acc);
            } else {
                *reinterpret_cast<float4 *>(a.values + (int64_t)d.z * D + col) = acc;
                amax.add(t, f4_absmax(acc));
            }
        }
        if (__any(parks)) { // wave-uniform
            // the parked sums have reached the chip-wide level before any of this wave's chunks is counted in
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            int before = -1;
            if (parks && lg == 0)
                before = __hip_atomic_fetch_add(a.ws.seg_count + head_pos / DQRM_SEG_CHUNK, 1, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::: "memory"); // (the loads below stay below)
            // the groups whose chunk completed its segment's count: the wave adds up their segments
            unsigned long long todo = __ballot(parks && lg == 0 && before == nchunks - 1);
            if constexpr (G >= 16) { // a row fills the wave: a lane per column, the segments one by one
                while (todo != 0ull) {
                    const int src = __ffsll((long long)todo) - 1;
                    todo &= todo - 1ull;
                    const int s_head = __builtin_amdgcn_readlane(head_pos, src), s_n = __builtin_amdgcn_readlane(nchunks, src);
                    const int s_seg = __builtin_amdgcn_readlane(d.z, src), s_t = __builtin_amdgcn_readlane(d.w, src);
                    float m = 0.0f;
                    for (int base = 0; base < D; base += kWave) {
                        const float sum = combine_columns(a.ws, s_head, s_n, D, base, lane);
                        const int cc = base + combine_col(lane);
                        if (cc < D) {
                            a.values[(int64_t)s_seg * D + cc] = sum;
                            m = fmaxf(m, fabsf(sum));
                        }
                    }
                    m = wave_max(m);
                    if (lane == 0) {
                        amax.add(s_t, m);
                        // (ready for another run of the segment sums on the same dedupe)
                        __hip_atomic_store(a.ws.seg_count + s_head / DQRM_SEG_CHUNK, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            } else { // narrow rows: 4 G lanes per segment, 16 / G segments in one round trip
                constexpr int kLanesPerSeg = 4 * G, kSegsPerPass = kWave / kLanesPerSeg;
                const int slot = lane / kLanesPerSeg, cc = lane % kLanesPerSeg;
                while (todo != 0ull) {
                    int src = -1;
#pragma unroll
                    for (int j = 0; j < kSegsPerPass; ++j) {
                        if (todo != 0ull) {
                            if (slot == j) src = __ffsll((long long)todo) - 1;
                            todo &= todo - 1ull;
                        }
                    }
                    const int from = src < 0 ? 0 : src;
                    const int s_head = __shfl(head_pos, from, kWave);
                    const int n_from = __shfl(nchunks, from, kWave);
                    const int s_n = src >= 0 && cc < D ? n_from : 0;
                    const int s_seg = __shfl(d.z, from, kWave), s_t = __shfl(d.w, from, kWave);
                    const int wave_n = __builtin_amdgcn_readfirstlane(wave_max_int(s_n));
                    const float sum = combine_column_shared_wave(a.ws, s_head, s_n, wave_n, D, cc);
                    if (s_n > 0) a.values[(int64_t)s_seg * D + cc] = sum;
                    float m = s_n > 0 ? fabsf(sum) : 0.0f;
#pragma unroll
                    for (int o = kLanesPerSeg / 2; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
                    if (src >= 0 && cc == 0) {
                        amax.add(s_t, m);
                        __hip_atomic_store(a.ws.seg_count + s_head / DQRM_SEG_CHUNK, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
        c = c_next;
        d = d_next;
#pragma unroll
        for (int q = 0; q < kChunkIdsPerLane(G); ++q) my_bags[q] = next_bags[q];
    }
    amax.flush(a.ws.absmax_slots, T);
}

template <int G, bool REUSE>
__global__ __launch_bounds__(kSumThreads, 4) void segment_sum_kernel(SegArgs a)
{
    segment_sum_body<G, REUSE>(a);
}

// The segment sums of several batches in one launch (blockIdx.y picks the batch): small batches, such as the
// micro-batches of simulated data parallelism, are a chain of dependent round trips with little else to do, and
// several of them side by side cost hardly more than one.
struct SegMulti {
    SegArgs b[DQRM_MAX_DEDUPE_BATCHES];
};

template <int G, bool REUSE>
__global__ __launch_bounds__(kSumThreads, 4) void segment_sum_multi_kernel(SegMulti m)
{
    segment_sum_body<G, REUSE>(m.b[blockIdx.y]);
}

// g_absmax[t] = max over the table's slots
// (and clears them, so that the segment sums may be repeated on the same dedupe)
__device__ __forceinline__ void absmax_finalize_body(float *__restrict__ slots, int T, float *__restrict__ g_absmax)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    float v[kAbsmaxSlots];
#pragma unroll
    for (int k = 0; k < kAbsmaxSlots; ++k) v[k] = *absmax_slot(slots, t, k);
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < kAbsmaxSlots; ++k) {
        m = fmaxf(m, v[k]);
        *absmax_slot(slots, t, k) = 0.0f;
    }
    g_absmax[t] = m;
}

__global__ void absmax_finalize_kernel(float *__restrict__ slots, int T, float *__restrict__ g_absmax)
{
    absmax_finalize_body(slots, T, g_absmax);
}

struct AbsmaxMulti {
    float *slots[DQRM_MAX_DEDUPE_BATCHES];
    float *g_absmax[DQRM_MAX_DEDUPE_BATCHES]; // an entry may be null: that batch's maxima are not wanted
    int T;
};

__global__ void absmax_finalize_multi_kernel(AbsmaxMulti m)
{
    if (m.g_absmax[blockIdx.y]) absmax_finalize_body(m.slots[blockIdx.y], m.T, m.g_absmax[blockIdx.y]);
}

} // namespace dqrm
