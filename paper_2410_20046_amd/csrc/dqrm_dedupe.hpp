// dqrm_dedupe: sort a batch's lookups by (table, row, position), find the distinct rows, and build the work lists of
// the segment sums (the sparse-tensor coalescing of Sec. 4.3).  It needs only the batch's indices.
//
// Kernel 1 (dedupe_kernel; dedupe_table_kernel where the tables alone fill the chip): the rows of a table are cut into `parts` ranges, one workgroup per (batch, table, range).
//   A workgroup reads all of its table's lookups, keeps those of its range in lookup order (LDS), counts those below
//   it (that is where its piece of the sorted order starts: no workgroup waits for another), sorts what it kept with a
//   stable LSD radix sort in LDS, and writes its piece of the sorted order and its own lists of chunks and singles.
//   A range with more lookups than the LDS holds is taken in pieces, and a table with far more than the others has further ranges.
//   Tables of very many lookups are first sorted by range, a tile of lookups per workgroup (dedupe_partition_kernel), so
//   that a range's workgroup reads only its own.
// Kernel 2 (dedupe_finish_kernel): turns the workgroups' counts into offsets (there are at most kMaxParts of them,
//   every workgroup repeats the scan), writes the index-only outputs (unique rows, segment offsets, table offsets,
//   count) and one dense list of 16-byte chunk descriptors over all tables.
#pragma once

#include "dqrm_device.hpp"

namespace dqrm {

constexpr int kMaxParts = 1024;    // (table, range) pairs per batch where every table has equally many ranges, at most
constexpr int kMaxSlots = 1280;    // with the further ranges of tables of very many lookups
constexpr int kDdSample = 512;     // lookups of such a table that its ranges are chosen by
constexpr int kDdMaxRanges = 64;   // its ranges, at most
constexpr int kDdTile = 8192;      // lookups of a table that a workgroup of dedupe_partition_kernel takes
constexpr int kDdTiles = DQRM_MAX_TABLE_LOOKUPS / kDdTile; // of a table, at most
constexpr int kDdRanges = 64;      // ranges of a partitioned table, at most
constexpr int kDdPartThreads = 1024;
constexpr int kDdPartSample = 256; // lookups of a partitioned table that its ranges are chosen by
constexpr int kSegThreads = 256;   // dedupe_finish_kernel
static_assert(DQRM_MAX_TABLES <= kMaxParts && DQRM_MAX_TABLE_LOOKUPS <= 65536 && DQRM_MAX_TABLE_LOOKUPS / DQRM_SEG_CHUNK < 4096,
              "a part per table at least; positions inside a table are 16 bits; the chunk descriptor holds 12 bits of chunk count");

// Views into the caller's workspace (all device pointers).
struct BwdWs {
    // [kMaxSlots][2] per (table, range), those every table has first: {first sorted position, segments, chunks other than
    // singles, singles}, then how many chunks of each length class there are, 16 bits each, and in w (of a further range) its place
    // in the order of all
    int4 *part_info;
    // the lookups of tiles of kDdTile, each sorted by range (dedupe_partition_kernel; only for batches of more than kDdTile)
    unsigned *part_key;       // [N]   rows (or the number of rows, for a bad index)
    unsigned short *part_pos; // [N]   positions inside the table
    unsigned short *part_start; // [T][kDdTiles][kDdRanges] first item of each range inside the tile
    unsigned *part_bound;     // [T][kDdRanges + 1] first row of each range, and the number of rows + 1 (in chunk_desc's place)
    int *sorted_bag;          // [N]   bag of every sorted lookup
    int4 *chunk_local;        // [N]   chunk lists of the parts (each starts at the part's first sorted position)
    int4 *single_local;       // [N]   their lists of singles: {sorted position, bag, segment, row}
    int4 *chunk_desc;         // [N]   dense chunk list over all tables, as the summing kernels read it
    int *chunk_bags;          // [N/2 + 1][32] bags of chunk c's lookups, so that they can be read before its descriptor
    int4 *single_desc;        // [N]   dense list of singles: {bag, global segment, table, -}
    int *totals;              // [4]   chunks, segments, singles; further ranges (if there can be any)
    int *seg_count;           // [N/32 + 2] chunks of a segment of more than one chunk that have parked their sum, filed
                              //       under (sorted position of the segment's head / 32); zero between uses
    float *partial_full;      // [(N/32 + 2) * D] sum of a full chunk of a segment of more than one chunk
    float *partial_last;      // [(N/32 + 2) * D] sum of the last chunk of such a segment
    float *absmax_slots;      // [T][kAbsmaxSlots] running maxima, one 128-byte line per entry
};

// A chunk = up to DQRM_SEG_CHUNK consecutive sorted lookups of one segment.  Its
// descriptor is one 16-byte record, so that the summing kernels need a single
// load to know their work:
//   x  global sorted position of the chunk's first lookup
//   y  len (bits 0..7) | index of the chunk inside its segment (bits 8..19) |
//      chunks in the segment (bits 20..31)
//   z  index of the segment inside its part (bits 0..15) | rank of the chunk among the part's chunks of its length class
//   w  table-local row of the segment
__device__ __forceinline__ int4 make_chunk_desc(int gstart, int len, int kchunk, int nchunks, int seg, int rank, unsigned row)
{
    return make_int4(gstart, len | (kchunk << 8) | (nchunks << 20), seg | (rank << 16), (int)row);
}
// The dense list is in sorted order, or (DedupeArgs::by_length) the long chunks of all tables come first: the groups of a wave of the
// summing kernel then add up chunks of about the same length, and the segments of many chunks, which one wave finishes after
// all of theirs, are not the last ones at work (26 tables x 65536 lookups: segment sums with the
// short chunks first 95 us, the long ones first 90).
constexpr int kChunkClasses = 5;
__device__ __forceinline__ int chunk_class(int len) { return len > 24 ? 0 : len > 16 ? 1 : len > 8 ? 2 : len > 4 ? 3 : 4; }
__device__ __forceinline__ int desc_len(const int4 &d) { return d.y & 0xFF; }
__device__ __forceinline__ int desc_kchunk(const int4 &d) { return (d.y >> 8) & 0xFFF; }
__device__ __forceinline__ int desc_nchunks(const int4 &d) { return (int)((unsigned)d.y >> 20); }

// One launch can dedupe several batches (blockIdx.y picks the batch).
struct DedupeBatch {
    const int64_t *indices;
    const int64_t *offsets;
    int64_t N;
    int limit; // lookups a table may have: DQRM_MAX_TABLE_LOOKUPS or the caller's smaller bound
    BwdWs ws;
    int32_t *sorted_pos;
    int32_t *tuo;
    int32_t *num_unique;
    int64_t *uniq_rows;
    int32_t *seg_offsets;
};
struct DedupeArgs {
    DedupeBatch b[DQRM_MAX_DEDUPE_BATCHES];
    const int64_t *row_offsets;
    int T, B;
    int parts; // ranges per table, T * parts <= kMaxParts
    int bags_per_part; // ceil(B / parts)
    int light;         // a table of more lookups has its ranges chosen by a sample, and further ones
    int per_range;     // as far as it has fewer than one per so many lookups
    int extra;         // further ranges of all tables of a batch, at most (0: no table can have any)
    int by_length;     // the order of the dense chunk list, see chunk_class
    FastDiv by_parts;
    FastDiv even; // by the lookups of a bag if all bags of the launch hold equally many (a guess), else by 1
};

// bits set below my lane / up to and including it
__device__ __forceinline__ int mask_rank(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// the last bag b of [0, B) with off(b) <= p, for a non-decreasing off with off(0) <= p
template <typename Off>
__device__ __forceinline__ int find_bag(Off off, int B, int p)
{
    int bag = 0;
    for (int step = 1 << (31 - __clz(B)); step >= 1; step >>= 1) {
        const int b = bag + step;
        if (b < B && (int)off(b) <= p) bag = b;
    }
    return bag;
}

// The bags of a table's lookups: where they all hold equally many (`even`, a guess) a lookup's bag follows from its position;
// otherwise it is found among the bags' first positions, every 2^sparse-th of them in LDS, and then among those between.
struct BagSearch {
    const int64_t *bag_offsets; // of the table, B + 1
    long long lo;               // its first lookup
    int B, sparse;
    bool even;

    // a bag of [b_lo, b_hi) that does not lie behind the one in front of it and inside the table's n lookups, or -1
    template <int THREADS>
    __device__ __forceinline__ int disorder(int b_lo, int b_hi, int n, int tid) const
    {
        int bad = -1;
        for (int b0 = b_lo + tid; b0 < b_hi; b0 += 4 * THREADS) { // (four at a time, all requested before the first is looked at)
            long long s[4], e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = min(b0 + q * THREADS, b_hi - 1);
                s[q] = bag_offsets[b];
                e[q] = bag_offsets[b + 1];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (s[q] < lo || e[q] > lo + n || s[q] > e[q]) bad = min(b0 + q * THREADS, b_hi - 1);
        }
        return bad;
    }
    template <int THREADS>
    __device__ __forceinline__ void stage(unsigned short *soff, int tid) const
    {
        for (int b = tid; b << sparse < B; b += THREADS) {
            const long long s = bag_offsets[b << sparse] - lo;
            soff[b] = (unsigned short)(s < 0 ? 0 : (s > 65535 ? 65535 : (int)s));
        }
    }
    // (after a wrong guess nothing is staged)
    __device__ __forceinline__ int find(const unsigned short *soff, int p) const
    {
        if (even) return find_bag([&](int b) { return bag_offsets[b] - lo; }, B, p);
        const int hint = p < 65535 ? find_bag([&](int b) { return soff[b]; }, ((B - 1) >> sparse) + 1, p) << sparse : 0;
        if (sparse == 0 && p < 65535) return hint; // (position 65535 cannot be told from an empty bag at 65536 in 16 bits)
        return hint + find_bag([&](int b) { return bag_offsets[hint + b] - lo; }, p < 65535 ? min(1 << sparse, B - hint) : B, p);
    }
};

// A table's lookups [lo, lo + n) in the batch, by its bags' offsets; n = 0 if they make no sense or are too many (then
// bad_code / bad_value say why), or if an earlier table has some of them.
struct TableExtent {
    long long lo;
    int n, bad_code;
    long long bad_value;
};

// All threads of the workgroup call this (t: wave-uniform; s_back: an LDS word per wave).  Tables share lookups only where a
// boundary between tables lies before the one in front of it (the table that it ends reports that): whether there is one before
// t is looked up for all tables at once, and only then is t compared with each of them.
template <int THREADS>
__device__ __forceinline__ TableExtent table_extent(const int64_t *offsets, int t, int B, int64_t N, int limit, int tid, int *s_back)
{
    constexpr int kWaves = THREADS / kWave;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // (by every wave for itself while that is one step: the workgroup has nothing to wait for then)
    const bool by_wave = t <= kWave;
    bool back = false;
    for (int s = by_wave ? lane : tid; s < t; s += THREADS) back |= offsets[(long long)s * B] > offsets[(long long)(s + 1) * B];
    const long long lo = offsets[(long long)t * B], hi = offsets[(long long)(t + 1) * B];
    const bool bad = lo < 0 || hi > N || lo > hi, many = !bad && hi - lo > limit;
    TableExtent x;
    x.bad_code = bad ? DQRM_ERR_BAD_OFFSETS : (many ? DQRM_ERR_CAPACITY : 0);
    x.bad_value = bad ? lo : hi - lo;
    x.n = bad || many ? 0 : (int)(hi - lo);
    x.lo = lo < 0 ? 0 : (lo > N ? N : lo);
    bool any_back = __any(back);
    if (!by_wave) {
        if (lane == 0) s_back[wave] = any_back;
        __syncthreads();
        any_back = __any(s_back[lane & (kWaves - 1)]); // (the number of waves is a power of two)
    }
    if (any_back) {
        bool shared = false;
        for (int s = lane; s < t; s += kWave) {
            const long long l = offsets[(long long)s * B], h = offsets[(long long)(s + 1) * B];
            shared |= l >= 0 && l <= h && h <= N && h - l <= limit && l < hi && lo < h;
        }
        if (__any(shared)) x.n = 0;
    }
    x.n = __builtin_amdgcn_readfirstlane(x.n); // (wave-uniform, and known to be)
    return x;
}

// Further ranges of a table of n lookups.  Together a batch's tables have no more than DedupeArgs::extra (host) where their
// boundaries are in order; where they are not, none has any.
__device__ __forceinline__ int extra_ranges(const DedupeArgs &a, int n)
{
    return n > a.light ? max((n + a.per_range - 1) / a.per_range - a.parts, 0) : 0;
}

// The e-th further range of a batch: its table and its number among the table's ranges (table -1: there are fewer).  The first
// one's workgroup leaves in totals[3] how many there are.  All threads of the workgroup call this; s_w: an LDS word per wave,
// s_found: two.
template <int THREADS>
__device__ __forceinline__ int2 find_extra(const DedupeArgs &a, const DedupeBatch &bt, int e, int tid, int *s_w, int *s_found)
{
    constexpr int kWaves = THREADS / kWave;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int per = (a.T + THREADS - 1) / THREADS; // consecutive tables per thread
    bool back = false;
    auto count_of = [&](int t) {
        const long long lo = bt.offsets[(long long)t * a.B], hi = bt.offsets[(long long)(t + 1) * a.B];
        back |= lo > hi;
        return lo >= 0 && lo <= hi && hi <= bt.N && hi - lo <= bt.limit ? extra_ranges(a, (int)(hi - lo)) : 0;
    };
    int mine = 0;
#pragma unroll 1
    for (int t = tid * per; t < min((tid + 1) * per, a.T); ++t) mine += count_of(t);
    const int incl = wave_incl_scan_add(mine, lane);
    if (tid == 0) s_found[0] = -1;
    if (lane == kWave - 1) s_w[wave] = incl;
    const bool any_back = __syncthreads_or(back ? 1 : 0) != 0;
    const int waves_incl = wave_incl_scan_add(lane < kWaves ? s_w[lane] : 0, lane);
    const int total = __builtin_amdgcn_readlane(waves_incl, kWaves - 1);
    int before = incl - mine + (wave > 0 ? __builtin_amdgcn_readlane(waves_incl, max(wave - 1, 0)) : 0);
    if (e == 0 && tid == 0) bt.ws.totals[3] = any_back ? 0 : total;
    if (e >= before && e < before + mine) // (one thread)
#pragma unroll 1
        for (int t = tid * per; t < min((tid + 1) * per, a.T); ++t) {
            const int count = count_of(t);
            if (e >= before && e < before + count) s_found[0] = t, s_found[1] = a.parts + e - before;
            before += count;
        }
    __syncthreads();
    const int2 r = make_int2(__builtin_amdgcn_readfirstlane(s_found[0]), __builtin_amdgcn_readfirstlane(s_found[1]));
    return any_back ? make_int2(-1, 0) : r;
}

// Range `part` of `ranges` of a table of very many lookups, [x, y): between two of kDdSample of its keys (s_sample, all
// written), so that the ranges hold about equally many lookups wherever in the table the popular rows lie.  A key that
// bounds several ranges has the first of them to itself.  All threads of the workgroup call this.
template <int THREADS>
__device__ __forceinline__ uint2 sampled_range(const unsigned *s_sample, int part, int ranges, unsigned rows_t, int tid, unsigned *s_split)
{
#pragma unroll 1
    for (int j = tid; j < kDdSample; j += THREADS) {
        const unsigned k = s_sample[j];
        int rank = 0;
#pragma unroll 2
        for (int i = 0; i < kDdSample; i += 4) {
            const uint4 o = *reinterpret_cast<const uint4 *>(s_sample + i);
            rank += (o.x < k || (o.x == k && i < j)) + (o.y < k || (o.y == k && i + 1 < j)) + (o.z < k || (o.z == k && i + 2 < j)) +
                    (o.w < k || (o.w == k && i + 3 < j));
        }
#pragma unroll
        for (int b = -1; b < 2; ++b) // the keys that bound this range and the one before it
            if ((part + b) > 0 && part + b < ranges && rank == (part + b) * kDdSample / ranges) s_split[b + 1] = k;
    }
    __syncthreads();
    auto bound = [&](int b) { // of part + b and the range in front of it
        const int p = part + b;
        if (p <= 0) return 0u;
        if (p >= ranges) return rows_t + 1u;
        return s_split[b + 1] + (p > 1 && s_split[b + 1] == s_split[b] ? 1u : 0u);
    };
    return make_uint2(bound(0), bound(1));
}

// A wave-uniform number that the compiler takes for a new one.  (Two unrolled loops that leave at the same round would
// otherwise be compiled as one path per round through both.)
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}
// the same for a number of the lane
__device__ __forceinline__ int opaque_lane(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The lanes of the wave whose digit of `bits` bits equals mine (all 64 lanes active).  Per bit: the lanes whose bit is set
// (ballot) against my own bit spread over a word (0 or all ones, a signed one-bit field extract): the lanes whose bit
// equals mine are ~(ballot ^ mine), and gfx950 folds that and the running AND into one three-input bit operation per
// 32-bit half.  (Measured against a table of lane masks in LDS, one atomic OR and one read per lane: that took 15 % longer
// over a whole sort, the conflicts of frequent digits cost more than the ballots.)
__device__ __forceinline__ unsigned long long match_digit(unsigned d, int bits)
{
    unsigned lo = ~0u, hi = ~0u;
    for (int b = 0; b < bits; ++b) {
        unsigned mine = (unsigned)(int)__builtin_amdgcn_sbfe(d, b, 1);
        asm volatile("" : "+v"(mine)); // (keeps the compiler from deriving the ballot from d again: a shift more per bit)
        const unsigned long long bal = __ballot(mine != 0u);
        lo &= ~((unsigned)bal ^ mine);
        hi &= ~((unsigned)(bal >> 32) ^ mine);
    }
    return ((unsigned long long)hi << 32) | lo;
}

// Where the items of each digit go, for the wave's items of a sorting pass: after the items of smaller digits and those
// of the same digit in earlier waves.  cnt: a row of 256 counts per wave (complete); a lane owns four digits.  Every wave
// adds up all rows by itself, which saves the barriers of a shared scan.  *starts = the digits' first places.
template <int WAVES>
__device__ __forceinline__ uint2 digit_places(const unsigned short *cnt, int wave, int lane, uint2 *starts)
{
    unsigned all01 = 0, all23 = 0, my01 = 0, my23 = 0; // (two 16-bit sums a word: at most 8192 each)
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint2 c = *reinterpret_cast<const uint2 *>(cnt + w * 256 + 4 * lane);
        if (w < wave) {
            my01 += c.x;
            my23 += c.y;
        }
        all01 += c.x;
        all23 += c.y;
    }
    const unsigned n0 = all01 & 0xFFFFu, n1 = all01 >> 16, n2 = all23 & 0xFFFFu, n3 = all23 >> 16;
    const unsigned sum = n0 + n1 + n2 + n3;
    const unsigned e0 = (unsigned)wave_incl_scan_add((int)sum, lane) - sum, e1 = e0 + n0, e2 = e1 + n1, e3 = e2 + n2;
    *starts = make_uint2(e0 | (e1 << 16), e2 | (e3 << 16));
    return make_uint2(starts->x + my01, starts->y + my23);
}

// Tables of many lookups: dedupe_kernel would read all of them in every range's workgroup.  Here a workgroup takes a tile
// of kDdTile lookups and sorts it by range (one stable pass of the radix sort), so that a range's workgroup finds its
// lookups in one run per tile.  Where a sample, the same for all tiles of a table, shows popular rows the ranges lie between its keys: they
// hold about equally many lookups, so a range's workgroup can be half as large, and two share a CU.  Where it shows none they are
// equally wide, which evenly spread lookups fill better than a sample of so few can tell (8 of the sample to a range).  The whole
// sort, us, Zipf 1.1 / 1.05 / evenly spread: 26 x 65536 lookups, equally wide 174 / 210 / 110, by the sample in any case 124 / 112 / 125, as it is
// now 112 / 100 / 82; 8 x 65536 138 / 89 / 43, 75 / 72 / 86, 47 / 46 / 41.  Bound by vector instructions, of which a workgroup has one CU's: the
// ranks by quarters and a search past whose last range no key lies took 18.7 -> 16.2 us of it at 26 x 65536.  (A sample of 512 has four times
// the comparisons, 8 us more.  The items' loop not unrolled, for a kernel of 7.6 instead of 10.7 KB: 18.3.)
__global__ __launch_bounds__(kDdPartThreads) void dedupe_partition_kernel(DedupeArgs args)
{
    constexpr int kWaves = kDdPartThreads / kWave, kItems = kDdTile / kDdPartThreads;
    __shared__ __align__(16) unsigned s_key[kDdTile];
    __shared__ unsigned short s_pos[kDdTile];
    __shared__ __align__(16) unsigned short cnt[kWaves * 256], place[kWaves * 256];
    __shared__ int s_back[kWaves];
    __shared__ unsigned s_split[kDdRanges], s_bound[kDdRanges + 1];
    __shared__ int s_hits[kDdRanges], s_rank[kDdPartSample];
    const DedupeBatch &bt = args.b[blockIdx.y];
    const int t = blockIdx.x, tile = blockIdx.z, B = args.B;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const unsigned rows_t = (unsigned)(args.row_offsets[t + 1] - args.row_offsets[t]);
    const TableExtent x = table_extent<kDdPartThreads>(bt.offsets, t, B, bt.N, bt.limit, tid, s_back); // (its problems: dedupe_kernel reports them)
    const int len = min(kDdTile, x.n - tile * kDdTile);
    if (len <= 0) return;
    const int rounds = (len + kDdPartThreads - 1) / kDdPartThreads;
    const int wave_at = wave * rounds * kWave;
    const char *src = reinterpret_cast<const char *>(bt.indices + x.lo + tile * kDdTile);
    const long long sample = bt.indices[x.lo + (unsigned)(tid % kDdPartSample) * (unsigned)x.n / kDdPartSample];
    long long raw[kItems];
    const int rounds_1 = opaque(rounds);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (r >= rounds_1) break;
        raw[r] = *reinterpret_cast<const long long *>(src + (unsigned)min(wave_at + r * kWave + lane, len - 1) * 8u);
    }
    // the sample, its ranks (four threads to a key), the ranges between
    const int parts = args.parts;
    if (tid < kDdPartSample) s_key[tid] = (unsigned long long)sample < rows_t ? (unsigned)sample : rows_t, s_rank[tid] = 0;
    if (tid < kDdRanges) s_split[tid] = 0u, s_hits[tid] = 0;
    __syncthreads();
    // Ranges of equal width do where the sample is spread over them as chance would (four standard deviations of a count), or where
    // each is one row: no two of them can be better.
    const unsigned share = args.by_parts.div(rows_t) + 1u;
    if (tid < kDdPartSample) atomicAdd(&s_hits[s_key[tid] / share], 1);
    __syncthreads();
    static_assert(kDdRanges == kWave, "a lane each");
    const float expected = (float)kDdPartSample * (float)share / (float)rows_t;
    const float per_share = 1.0f / (float)share;
    const bool equal = __builtin_amdgcn_readfirstlane(share == 1u || wave_max_int(s_hits[lane]) <= (int)(expected + 4.0f * sqrtf(expected)));
    if (!equal) {
        // A wave has 64 keys and compares them with a quarter of the sample: a key counts those below it, and the equal ones in front of
        // it, which are all of an earlier quarter and none of a later one.
        const int mine = wave % 4 * kWave, quarter = wave / 4 * kWave, j = mine + lane;
        const unsigned k = s_key[j];
        int rank = 0;
        static_assert(kDdPartThreads == 4 * kDdPartSample && kDdPartSample == 4 * kWave, "quarters");
        if (quarter == mine) { // (wave-uniform)
#pragma unroll 4
            for (int i = 0; i < kWave; ++i) rank += s_key[quarter + i] < k + (i < lane ? 1u : 0u);
        } else {
            const unsigned limit = k + (quarter < mine ? 1u : 0u);
#pragma unroll 4
            for (int i = 0; i < kWave; i += 4) {
                const uint4 o = *reinterpret_cast<const uint4 *>(s_key + quarter + i);
                rank += (o.x < limit) + (o.y < limit) + (o.z < limit) + (o.w < limit);
            }
        }
        atomicAdd(&s_rank[j], rank);
        __syncthreads();
        if (tid < kDdPartSample) {
            const int r = s_rank[tid], p = (r * parts + kDdPartSample - 1) / kDdPartSample; // the range that it would be the first key of
            if (p > 0 && p < parts && p * kDdPartSample / parts == r) s_split[p] = k;
        }
    }
    __syncthreads();
    // (a key that bounds several ranges has the first of them to itself)
    if (tid <= kDdRanges) {
        unsigned b = equal ? min((unsigned)tid * share, rows_t + 1u) : tid == 0 ? 0u : tid == parts ? rows_t + 1u : 0u;
        if (!equal && tid > 0 && tid < parts) b = s_split[tid] + (tid > 1 && s_split[tid] == s_split[tid - 1] ? 1u : 0u);
        if (tid > parts) b = ~0u; // (no range)
        s_bound[tid] = b;
        if (tile == 0 && tid <= parts) bt.ws.part_bound[(int64_t)t * (kDdRanges + 1) + tid] = b;
    }
    __syncthreads();
    unsigned short *my_cnt = cnt + wave * 256, *my_place = place + wave * 256;
    *reinterpret_cast<uint2 *>(my_cnt + 4 * lane) = make_uint2(0u, 0u);
    const int bits = 32 - __clz(args.parts); // (the digit `parts` is the padding's)
    unsigned key[kItems], rank[kItems]; // rank: place inside the wave's items of the digit, digit in the upper half
    bool bad_index = false;
    long long bad_value = 0;
    const int rounds_2 = opaque(rounds);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (r >= rounds_2) break;
        const bool exists = wave_at + r * kWave + lane < len;
        key[r] = (unsigned long long)raw[r] < rows_t ? (unsigned)raw[r] : rows_t;
        if (exists && key[r] == rows_t) bad_index = true, bad_value = raw[r];
        int d = 0;
        if (equal) { // key / share: at most 63, so the rounded quotient is at most one off
            d = (int)((float)key[r] * per_share);
            const int rest = (int)(key[r] - (unsigned)d * share);
            d += rest < 0 ? -1 : (rest >= (int)share ? 1 : 0);
        } else { // the last range that begins at or before it
#pragma unroll
            for (int step = kDdRanges / 2; step >= 1; step >>= 1) d = s_bound[d + step] <= key[r] ? d + step : d; // (past the last one: no key)
        }
        if (!exists) d = args.parts; // (padding: after every range)
        const unsigned long long peers = match_digit((unsigned)d, bits);
        const unsigned prev = my_cnt[d];
        const int before = mask_rank(peers);
        rank[r] = (prev + (unsigned)before) | ((unsigned)d << 16);
        if (before == 0) my_cnt[d] = (unsigned short)(prev + (unsigned)__popcll(peers));
    }
    if (bad_index) report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, bad_value);
    __syncthreads();
    uint2 starts;
    *reinterpret_cast<uint2 *>(my_place + 4 * lane) = digit_places<kWaves>(cnt, wave, lane, &starts);
    if (wave == 0 && 4 * lane < kDdRanges)
        *reinterpret_cast<uint2 *>(bt.ws.part_start + ((int64_t)t * kDdTiles + tile) * kDdRanges + 4 * lane) = starts;
    const int rounds_3 = opaque(rounds);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        if (r >= rounds_3) break;
        const unsigned to = my_place[rank[r] >> 16] + (rank[r] & 0xFFFFu);
        s_key[to] = key[r];
        s_pos[to] = (unsigned short)(wave_at + r * kWave + lane);
    }
    __syncthreads();
    unsigned *out_key = bt.ws.part_key + x.lo + tile * kDdTile;
    unsigned short *out_pos = bt.ws.part_pos + x.lo + tile * kDdTile;
    for (int i = tid; i < len; i += kDdPartThreads) {
        out_key[i] = s_key[i];
        out_pos[i] = (unsigned short)(tile * kDdTile + s_pos[i]);
    }
}

constexpr int kDdStack = 192;     // pending range ends
constexpr int kDdPivotDepth = 96; // pending ranges beyond which a range is halved instead of split at a sampled row
static_assert(kDdPivotDepth + 2 + 32 <= kDdStack, "halving ends at a range of one row");

// (The loops over a thread's items leave at the first round that does not exist, and those after the sort are not
// unrolled: most launches have one or two rounds, every line of code is fetched anew by every launch, and a kernel
// this short waits for its code as much as for its data.)
// PARTITIONED: the table's lookups come from dedupe_partition_kernel, a run of this range per tile.
// EXTRA: a table may have more than DedupeArgs::light lookups (a kernel of its own, as the others pay for its code otherwise).
// LDS of such a workgroup
template <int THREADS, int CAP>
struct DedupeLds {
    static constexpr int kWaves = THREADS / kWave;
    // the kept lookups, twice (a sorting pass moves them from one half to the other): key relative to the range, position
    // inside the table
    alignas(16) unsigned key[2][CAP + 4];
    unsigned short pos[2][CAP], rank[CAP];
    // digit counters, a row of 256 per wave, and where the wave's items of each digit go
    alignas(16) unsigned short cnt[kWaves * 256], place[kWaves * 256];
    unsigned long long heads[CAP / kWave];
    int scan[2][kWaves];
    int4 x[kWaves];
    int cls[kChunkClasses]; // chunks of each length class so far
    unsigned stack[kDdStack];
    unsigned pivot;
    int back[kWaves];
};

// block_x: the table, block_y: the batch, block_z: the range
template <int THREADS, int CAP, bool PARTITIONED, bool EXTRA>
__device__ __forceinline__ void dedupe_body(const DedupeArgs &args, DedupeLds<THREADS, CAP> &lds, int block_x, int block_y, int block_z)
{
    constexpr int kWaves = THREADS / kWave, kCap = CAP;
    constexpr int kDdItems = CAP / THREADS; // lookups a thread requests at a time, and sorts
    static_assert(kCap % THREADS == 0 && kCap <= 8192, "ranks are 16 bits");
    auto &s_key = lds.key;
    auto &s_pos = lds.pos;
    auto &s_rank = lds.rank;
    auto &cnt = lds.cnt;
    auto &place = lds.place;
    auto &s_heads = lds.heads;
    auto &s_scan = lds.scan;
    auto &s_x = lds.x;
    auto &s_class = lds.cls;
    auto &s_stack = lds.stack;
    auto &s_pivot = lds.pivot;
    auto &s_back = lds.back;

    const DedupeBatch &bt = args.b[block_y];
    const int64_t *__restrict__ indices = bt.indices;
    const int64_t *__restrict__ offsets = bt.offsets;
    const int B = args.B;
    const int64_t N = bt.N;
    const BwdWs &ws = bt.ws;
    int32_t *__restrict__ sorted_pos = bt.sorted_pos;

    int t = block_x, part = block_z; // consecutive workgroups: different tables
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    if (EXTRA && part >= args.parts) {
        const int e = (part - args.parts) * args.T + t;
        if (e >= args.extra) return;
        const int2 r = find_extra<THREADS>(args, bt, e, tid, s_scan[0], s_scan[1]);
        if (r.x < 0) return;
        t = r.x, part = r.y;
        __syncthreads(); // (s_scan is free again)
    }

    const unsigned rows_t = (unsigned)(args.row_offsets[t + 1] - args.row_offsets[t]); // host: <= DQRM_MAX_TABLE_ROWS

    const int64_t *__restrict__ bag_offsets = offsets + (long long)t * B;
    uint2 bound = make_uint2(0u, 0u); // (requested with the boundaries of the tables; of no meaning for a table without lookups)
    if constexpr (PARTITIONED) {
        const unsigned *at = ws.part_bound + (int64_t)t * (kDdRanges + 1) + part;
        bound = make_uint2(at[0], at[1]);
    }
    const TableExtent x = table_extent<THREADS>(offsets, t, B, N, bt.limit, tid, s_back);
    const long long lo = x.lo;
    const int n = x.n, base = (int)lo;
    // A problem of the data is kept here and reported at one place (one problem per thread and kind of work is enough: only
    // the first of all is recorded).
    int bad_code = part == 0 && tid == 0 ? x.bad_code : 0;
    long long bad_value = x.bad_value;

    // My range of the keys [0, rows_t]: a row, or rows_t for a lookup whose index is out of range (those sort after
    // every row, and the part that holds them reports them).  The ranges of most tables are equally wide,
    // those of a partitioned one as dedupe_partition_kernel chose them.
    const unsigned share = args.by_parts.div(rows_t) + 1u;
    unsigned range_lo = min((unsigned)part * share, rows_t + 1u), range_hi = min(range_lo + share, rows_t + 1u);
    static_assert(!PARTITIONED || !EXTRA, "a partitioned table has no further ranges");
    if constexpr (PARTITIONED) {
        range_lo = n > 0 ? (unsigned)__builtin_amdgcn_readfirstlane((int)bound.x) : 0u;
        range_hi = n > 0 ? (unsigned)__builtin_amdgcn_readfirstlane((int)bound.y) : 0u;
    }
    bool sampled = EXTRA && n > args.light;
    if (__builtin_expect(sampled, 0)) {
        bool back = false;
#pragma unroll 1
        for (int s = tid; s < args.T; s += THREADS) back |= offsets[(long long)s * B] > offsets[(long long)(s + 1) * B];
        sampled = !__syncthreads_or(back ? 1 : 0);
    }
    if (__builtin_expect(sampled, 0)) {
        unsigned *s_sample = s_key[1];
#pragma unroll 1
        for (int j = tid; j < kDdSample; j += THREADS) { // (n is at least kDdSample: host)
            const long long v = indices[lo + (unsigned)j * (unsigned)n / kDdSample];
            s_sample[j] = (unsigned long long)v < rows_t ? (unsigned)v : rows_t;
        }
        __syncthreads();
        const uint2 r = sampled_range<THREADS>(s_sample, part, args.parts + extra_ranges(args, n), rows_t, tid, s_stack);
        range_lo = (unsigned)__builtin_amdgcn_readfirstlane((int)r.x), range_hi = (unsigned)__builtin_amdgcn_readfirstlane((int)r.y);
        __syncthreads(); // (the LDS is free again)
    }

    // The lookups to look at: all of the table's, or those of my range, tile by tile: item i of tile w's run is item
    // run_first[w] + i of mine and lies at run_from[w] + i (both wave-uniform).
    int count = n, run_below = 0;
    int run_first[kDdTiles], run_from[kDdTiles];
    if constexpr (PARTITIONED) {
        const int tile_len = min(kDdTile, n - lane * kDdTile); // (lanes are tiles)
        int s = 0, e = 0;
        if (lane < kDdTiles && tile_len > 0) {
            const unsigned short *st = ws.part_start + ((int64_t)t * kDdTiles + lane) * kDdRanges;
            s = min((int)st[part], tile_len);
            e = part + 1 < args.parts ? min((int)st[part + 1], tile_len) : tile_len;
        }
        const int incl = wave_incl_scan_add(e - s, lane), below_incl = wave_incl_scan_add(s, lane);
        const int first = incl - (e - s), from = base + lane * kDdTile + s - first;
        count = __builtin_amdgcn_readlane(incl, kDdTiles - 1);
        run_below = __builtin_amdgcn_readlane(below_incl, kDdTiles - 1);
#pragma unroll
        for (int w = 0; w < kDdTiles; ++w) {
            run_first[w] = __builtin_amdgcn_readlane(first, w);
            run_from[w] = __builtin_amdgcn_readlane(from, w);
        }
    }
    // a wave's share of a scan step: as few rounds as the step's lookups need
    const int scan_rounds = (min(count, kDdItems * THREADS) + THREADS - 1) / THREADS;
    const int scan_step = scan_rounds * THREADS;
    // The keys of a step's lookups, wave-striped (item r of a lane: wave_first + r * 64 + lane, so that a wave's items
    // are consecutive); requested one step ahead.  Lookups past the end re-read the last one.
    const int wave_first = wave * scan_rounds * kWave;
    const int64_t *__restrict__ my_indices = indices + base;
    struct Lookup {
        long long index;   // not PARTITIONED: as given
        unsigned row, pos; // PARTITIONED: checked, and where it was
    };
    Lookup raw[kDdItems];
    auto request = [&](int i, Lookup &l) {
        i = min(i, count - 1);
        if constexpr (PARTITIONED) {
            int at = run_from[0]; // (by differences: a choice among the runs' starts becomes an array in scratch memory, and every request waits)
#pragma unroll
            for (int w = 1; w < kDdTiles; ++w) at += i >= run_first[w] ? run_from[w] - run_from[w - 1] : 0;
            l.row = ws.part_key[at + i];
            l.pos = ws.part_pos[at + i];
        } else {
            l.index = *reinterpret_cast<const long long *>(reinterpret_cast<const char *>(my_indices) + (unsigned)i * 8u);
        }
    };
    auto row_of = [&](const Lookup &l) {
        if constexpr (PARTITIONED) return l.row;
        return (unsigned long long)l.index < rows_t ? (unsigned)l.index : rows_t;
    };
    auto request_step = [&](int i0, int lane) {
#pragma unroll
        for (int r = 0; r < kDdItems; ++r) raw[r] = Lookup{}; // (or what a step leaves alone would stay alive from the one before)
        const int scan_rounds_4 = opaque(scan_rounds);
#pragma unroll
        for (int r = 0; r < kDdItems; ++r) {
            if (r >= scan_rounds_4) break;
            request(i0 + r * kWave + lane, raw[r]);
        }
    };
    if (range_lo < range_hi && count > 0) request_step(wave_first, lane);

    // ---- bags.  The parts share the check of their order.  Where the bags hold equally many lookups each (the usual
    // batches), the bag of a lookup is guessed and the guess looked up; otherwise it is found among the
    // bags' first positions: in LDS, all of them or (if they do not fit) some, and then among those between where they are.
    const bool even = (unsigned long long)args.even.d * (unsigned)B == (unsigned)n; // (host: the divisor is N / (T B))
    const BagSearch bags{bag_offsets, lo, B, max(0, 32 - __clz((B - 1) / kCap)), even};
    if (n > 0) {
        const int b_lo = min(args.bags_per_part * part, B), b_hi = min(b_lo + args.bags_per_part, B);
        const int b = bags.disorder<THREADS>(b_lo, b_hi, n, tid);
        if (b >= 0) bad_code = DQRM_ERR_BAD_OFFSETS, bad_value = (long long)t * B + b;
    }
    if (bad_code != 0) report(bad_code, t, bad_value);
    if (part == 0 && tid < kAbsmaxSlots) *absmax_slot(ws.absmax_slots, t, tid) = 0.0f;
    if (tid < kChunkClasses) s_class[tid] = 0; // (read after more barriers)
    int n_uniq = 0, n_chunk = 0, n_single = 0; // this part's lists so far
    int part_base = -1;                        // first sorted position of the part
    unsigned cur = range_lo, end = range_hi;
    int depth = 0;
    bool requested = true; // the first keys are on their way
    const int tid_ = tid;
    while (cur < end) {
        // (Nearly always one round, and its arrays start at zero: what an unfinished loop leaves undefined would be carried
        // from round to round.  Nothing that depends on the lane is worth keeping in registers for the next round either.)
        const int tid = opaque_lane(tid_), lane = tid & (kWave - 1);
        // ---- 1. the lookups of [cur, end), in lookup order, to LDS; how many lie below -----------------------------
        const unsigned width = end - cur;
        if (!requested && count > 0) request_step(wave_first, lane);
        requested = false;
        int m = 0, below = run_below;
        // (a partitioned range of one row is known to hold just that row: if it is long, it need not be looked over first)
        const bool known = PARTITIONED && range_hi - range_lo == 1u && count > kCap;
        if (known) m = count;
        for (int i0 = known ? count : 0, par = 0; i0 < count; i0 += scan_step, par ^= 1) {
            unsigned key[kDdItems] = {}, pos[kDdItems] = {};
            bool bad_index = false;
            int mine = 0; // kept (low half) and below (high half), each at most 512 a wave and 8192 a workgroup
            const int scan_rounds_5 = opaque(scan_rounds);
#pragma unroll
            for (int r = 0; r < kDdItems; ++r) {
                if (r >= scan_rounds_5) break;
                key[r] = row_of(raw[r]);
                pos[r] = raw[r].pos;
                if (i0 + wave_first + r * kWave + lane >= count) key[r] = ~0u; // no lookup: in no range and below none
                if (!PARTITIONED && key[r] == rows_t && end > rows_t) bad_index = true, bad_value = raw[r].index;
                mine += __popcll(__ballot(key[r] - cur < width));
                mine += __popcll(__ballot(key[r] < cur)) << 16;
            }
            if (bad_index) report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, bad_value);
            if (i0 + scan_step < count) request_step(i0 + scan_step + wave_first, lane);
            if (lane == 0) s_scan[par][wave] = mine;
            __syncthreads();
            const int x = lane < kWaves ? s_scan[par][lane] : 0;
            const int incl = wave_incl_scan_add(x, lane);
            const int total = __builtin_amdgcn_readlane(incl, kWaves - 1);
            int dst = m + ((__builtin_amdgcn_readlane(incl, wave) - mine) & 0xFFFF);
            const int scan_rounds_6 = opaque(scan_rounds);
#pragma unroll
            for (int r = 0; r < kDdItems; ++r) {
                if (r >= scan_rounds_6) break;
                const bool in = key[r] - cur < width;
                const unsigned long long mask = __ballot(in);
                const int d = dst + mask_rank(mask);
                if (in && d < kCap) {
                    s_key[0][d] = key[r] - cur;
                    s_pos[0][d] = (unsigned short)(PARTITIONED ? pos[r] : (unsigned)(i0 + wave_first + r * kWave + lane));
                }
                dst += __popcll(mask);
            }
            m += total & 0xFFFF;
            below += total >> 16;
        }
        __syncthreads();
        const int at = base + below; // sorted position of the range's first lookup
        if (part_base < 0) part_base = at;

        if (m > kCap && width > 1) {
            // ---- more than fits: three ranges around a row from the middle of what was kept (a row so hot that it
            // alone overflows the LDS is that row sooner or later, and a range of one row needs no sort)
            unsigned pivot = cur + width / 2;
            const bool sampled = depth < kDdPivotDepth;
            if (sampled) {
                if (wave == 0) {
                    const unsigned k = s_key[0][lane * (kCap / kWave)];
                    int rank = 0;
                    for (int j = 0; j < kWave; ++j) {
                        const unsigned o = (unsigned)__builtin_amdgcn_readlane((int)k, j);
                        rank += o < k || (o == k && j < lane);
                    }
                    if (rank == kWave / 2) s_pivot = k;
                }
                __syncthreads();
                pivot = cur + s_pivot;
            }
            if (tid == 0) s_stack[depth] = end;
            ++depth;
            if (sampled && pivot + 1 < end) {
                if (tid == 0) s_stack[depth] = pivot + 1;
                ++depth;
            }
            __syncthreads();
            if (sampled && pivot == cur) { // the first of the three is empty: go on with the row itself
                --depth;
                end = s_stack[depth];
            } else {
                end = pivot;
            }
            __syncthreads();
            continue;
        }

        if (m > kCap) {
            // ---- one row (or the bad indices) with more lookups than the LDS holds: they are in order as they come
            const bool valid = cur < rows_t;
            unsigned short *soff = reinterpret_cast<unsigned short *>(s_key[0]);
            if (!even) {
                bags.stage<THREADS>(soff, tid); // (what was kept of the lookups is not needed)
                __syncthreads();
            }
            int done = 0;
            request_step(wave_first, lane);
            for (int i0 = 0, par = 0; i0 < count; i0 += scan_step, par ^= 1) {
                unsigned long long in[kDdItems] = {};
                int pos[kDdItems] = {}, mine = 0;
                const int scan_rounds_7 = opaque(scan_rounds);
#pragma unroll
                for (int r = 0; r < kDdItems; ++r) {
                    if (r >= scan_rounds_7) break;
                    const int i = i0 + wave_first + r * kWave + lane;
                    in[r] = __ballot(i < count && row_of(raw[r]) == cur);
                    pos[r] = PARTITIONED ? (int)raw[r].pos : i;
                    mine += __popcll(in[r]);
                }
                if (i0 + scan_step < count) request_step(i0 + scan_step + wave_first, lane);
                if (lane == 0) s_scan[par][wave] = mine;
                __syncthreads(); // (and the step before this one has been written out)
                const int incl = wave_incl_scan_add(lane < kWaves ? s_scan[par][lane] : 0, lane);
                int dst = __builtin_amdgcn_readlane(incl, wave) - mine;
                const int scan_rounds_8 = opaque(scan_rounds);
#pragma unroll
                for (int r = 0; r < kDdItems; ++r) {
                    if (r >= scan_rounds_8) break;
                    if ((in[r] >> lane) & 1ull) s_pos[0][dst + mask_rank(in[r])] = (unsigned short)pos[r];
                    dst += __popcll(in[r]);
                }
                __syncthreads();
                const int kept = __builtin_amdgcn_readlane(incl, kWaves - 1);
                for (int k = tid; k < kept; k += THREADS) {
                    const int p = s_pos[0][k], d = at + done + k;
                    sorted_pos[d] = base + p;
                    int bag = (int)args.even.div((unsigned)p);
                    if (!even || bag_offsets[bag] > lo + p || lo + p >= bag_offsets[bag + 1]) bag = bags.find(soff, p);
                    if (valid) ws.sorted_bag[d] = bag;
                }
                done += kept;
            }
            if (valid) {
                const int nchunks = (m + DQRM_SEG_CHUNK - 1) / DQRM_SEG_CHUNK;
                const int last_len = m - (nchunks - 1) * DQRM_SEG_CHUNK, last_class = chunk_class(last_len);
                constexpr int kFull = 0; // class of a full chunk
                const int long_rank = s_class[kFull], last_rank = last_class == kFull ? long_rank + nchunks - 1 : s_class[last_class];
                for (int c = tid; c < nchunks; c += THREADS)
                    ws.chunk_local[part_base + n_chunk + c] =
                        make_chunk_desc(at + c * DQRM_SEG_CHUNK, c + 1 < nchunks ? DQRM_SEG_CHUNK : last_len, c, nchunks, n_uniq,
                                        c + 1 < nchunks ? long_rank + c : last_rank, cur);
                __syncthreads();
                if (tid == 0) {
                    ws.seg_count[at / DQRM_SEG_CHUNK] = 0;
                    s_class[kFull] += nchunks - 1;
                    s_class[last_class] += 1;
                }
                n_uniq += 1;
                n_chunk += nchunks;
            }
        } else if (m > 0) {
            // ---- 2. stable LSD radix sort of the m items, at most 8 bits per pass ------------------------------------
            const int rounds = (m + THREADS - 1) / THREADS; // 1 .. kDdItems, the same for the whole workgroup
            const int wave_at = wave * rounds * kWave;      // this wave's first item
            const int nbits = width > 1 && m > 1 ? 32 - __clz(width - 1) : 0;
            const int passes = (nbits + 7) / 8;
            const int bits = passes > 0 ? (nbits + passes - 1) / passes : 0;
            const unsigned digit_mask = (1u << bits) - 1u;
            unsigned short *my_cnt = cnt + wave * 256, *my_place = place + wave * 256;
            int half = 0;
            if (passes > 0) // padding: the largest digit in every pass and last in line, so it stays last
                for (int i = m + tid; i < rounds * THREADS; i += THREADS) s_key[0][i] = ~0u;
            for (int p = 0; p < passes; ++p, half ^= 1) {
                const int shift = bits * p;
                const unsigned *from_key = s_key[half];
                const unsigned short *from_pos = s_pos[half];
                unsigned *to_key = s_key[half ^ 1];
                unsigned short *to_pos = s_pos[half ^ 1];
                // (a wave's row of counters is its own: no barrier between clearing and counting)
                *reinterpret_cast<uint2 *>(my_cnt + 4 * lane) = make_uint2(0u, 0u);
                if (p == 0) __syncthreads(); // the padding is there
#pragma unroll 1
                for (int i = wave_at + lane, r = 0; r < rounds; ++r, i += kWave) {
                    const unsigned d = (from_key[i] >> shift) & digit_mask;
                    const unsigned long long peers = match_digit(d, bits);
                    const unsigned prev = my_cnt[d];
                    const int rank = mask_rank(peers);
                    s_rank[i] = (unsigned short)(prev + (unsigned)rank); // rank inside the wave's items of this digit
                    if (rank == 0) my_cnt[d] = (unsigned short)(prev + (unsigned)__popcll(peers));
                }
                __syncthreads();
                uint2 starts;
                *reinterpret_cast<uint2 *>(my_place + 4 * lane) = digit_places<kWaves>(cnt, wave, lane, &starts);
#pragma unroll 1
                for (int i = wave_at + lane, r = 0; r < rounds; ++r, i += kWave) {
                    const unsigned k = from_key[i];
                    const int to = my_place[(k >> shift) & digit_mask] + s_rank[i];
                    to_key[to] = k;
                    to_pos[to] = from_pos[i];
                }
                __syncthreads();
            }
            const unsigned *skey = s_key[half];
            const unsigned short *spos = s_pos[half];
            // the room of the keys' other half: the segments' first items, then the bags' first positions
            unsigned short *shead = reinterpret_cast<unsigned short *>(s_key[half ^ 1]), *soff = shead + kCap + 2;
            // the guessed bags' offsets are requested now, for all items at once, and looked at when the heads are known
            long long bag_lo[kDdItems] = {}, bag_hi[kDdItems] = {};
            if (even) {
                const int rounds_9 = opaque(rounds);
#pragma unroll
                for (int r = 0; r < kDdItems; ++r) {
                    if (r >= rounds_9) break;
                    const int i = wave_at + r * kWave + lane;
                    const unsigned g = args.even.div(i < m ? spos[i] : 0u); // below B, as the position is below n
                    bag_lo[r] = bag_offsets[g];
                    bag_hi[r] = bag_offsets[g + 1u];
                }
            } else {
                bags.stage<THREADS>(soff, tid);
            }

            // ---- 3. segment heads --------------------------------------------------------------------------------------
            const unsigned bad_key = rows_t - cur; // (what the bad indices carry; at least width where there can be none)
            int wave_heads = 0, wave_valid = 0;
#pragma unroll 1
            for (int r = 0; r < rounds; ++r) {
                const int i = wave_at + r * kWave + lane;
                const unsigned k = skey[i], prev = skey[max(i - 1, 0)];
                const bool valid = k < bad_key && i < m;
                const unsigned long long heads = __ballot(valid && (i == 0 || k != prev));
                if (lane == 0) s_heads[wave * rounds + r] = heads;
                wave_heads += __popcll(heads);
                wave_valid += __popcll(__ballot(valid));
            }
            if (lane == 0) s_x[wave] = make_int4(wave_heads, wave_valid, 0, 0);
            __syncthreads();
            int heads_before, seg_count, valid_count; // (the valid items come first)
            {
                const int4 x = s_x[lane & (kWaves - 1)];
                const int incl = wave_incl_scan_add(lane < kWaves ? (x.x | (x.y << 16)) : 0, lane);
                const int total = __builtin_amdgcn_readlane(incl, kWaves - 1);
                seg_count = total & 0xFFFF;
                valid_count = total >> 16;
                heads_before = (__builtin_amdgcn_readlane(incl, wave) & 0xFFFF) - wave_heads;
            }
            {
                int seg = heads_before;
#pragma unroll 1
                for (int r = 0; r < rounds; ++r) {
                    const unsigned long long heads = s_heads[wave * rounds + r];
                    if ((heads >> lane) & 1ull) shead[seg + mask_rank(heads)] = (unsigned short)(wave_at + r * kWave + lane);
                    seg += __popcll(heads);
                }
            }
            if (tid == 0) shead[seg_count] = (unsigned short)valid_count; // end of the last segment
            // bags (the guessed ones first; bags of other lengths that happen to add up to the same number are searched)
            bool search = !even;
            if (even) {
                const int rounds_10 = opaque(rounds);
#pragma unroll
                for (int r = 0; r < kDdItems; ++r) {
                    if (r >= rounds_10) break;
                    const int i = wave_at + r * kWave + lane, p = i < m ? (int)spos[i] : 0;
                    const int bag = (int)args.even.div((unsigned)p);
                    search |= bag_lo[r] > lo + p || lo + p >= bag_hi[r];
                    s_rank[i] = (unsigned short)bag;
                    if (i < valid_count) ws.sorted_bag[at + i] = bag;
                }
            } else {
                __syncthreads(); // (the staged offsets)
            }
            if (search) {
#pragma unroll 1
                for (int i = wave_at + lane, r = 0; r < rounds; ++r, i += kWave) {
                    const int bag = bags.find(soff, i < m ? (int)spos[i] : 0);
                    s_rank[i] = (unsigned short)bag;
                    if (i < valid_count) ws.sorted_bag[at + i] = bag;
                }
            }
            __syncthreads();

            // ---- 4. the part's piece of the sorted order and its lists.  Chunk heads: every DQRM_SEG_CHUNK-th item of a
            // segment, counted from its head.  Two classes, listed separately: "single" = a row looked up exactly once (the
            // common case, no summation needed), and all others.  Both lists in sorted order: counted first, then written.
            // (In the order in which the waves get there, the segment sums of 26 tables x 8192 lookups of one bag each take
            // 28.5 us instead of 25.4.)
            int chunk_at = 0, single_at = 0;
            for (int writes = 0; writes < 2; ++writes) {
                int seg_before = heads_before - 1, wave_chunks = 0, wave_singles = 0;
#pragma unroll 1
                for (int r = 0; r < rounds; ++r) {
                    const unsigned long long heads = s_heads[wave * rounds + r];
                    const int i = wave_at + r * kWave + lane;
                    const bool valid = i < valid_count;
                    const int seg = max(seg_before + mask_rank(heads) + (int)((heads >> lane) & 1ull), 0);
                    seg_before += __popcll(heads);
                    const int start = shead[seg], seg_end = shead[min(seg + 1, seg_count)];
                    const bool chead = valid && ((i - start) % DQRM_SEG_CHUNK) == 0;
                    const bool single = chead && i == start && seg_end == i + 1;
                    const unsigned long long singles = __ballot(single), chunks = __ballot(chead && !single);
                    if (writes) { // (wave-uniform)
                        const int p = i < m ? (int)spos[i] : 0;
                        // (more bags than 16 bits tell: this thread's own store is read back)
                        const int bag = B <= 65536 ? (int)s_rank[i] : (valid ? ws.sorted_bag[at + i] : 0);
                        const unsigned row = cur + skey[i];
                        if (i < m) sorted_pos[at + i] = base + p;
                        if (single)
                            ws.single_local[single_at + wave_singles + mask_rank(singles)] = make_int4(at + i, bag, n_uniq + seg, (int)row);
                        if (chead && !single) {
                            const int nchunks = (seg_end - start + DQRM_SEG_CHUNK - 1) / DQRM_SEG_CHUNK;
                            const int len = min(DQRM_SEG_CHUNK, seg_end - i);
                            ws.chunk_local[chunk_at + wave_chunks + mask_rank(chunks)] =
                                make_chunk_desc(at + i, len, (i - start) / DQRM_SEG_CHUNK, nchunks, n_uniq + seg,
                                                args.by_length ? atomicAdd(&s_class[chunk_class(len)], 1) : 0, row);
                            // the arrival counter of a segment of more than one chunk starts at zero
                            if (i == start && nchunks > 1) ws.seg_count[(at + i) / DQRM_SEG_CHUNK] = 0;
                        }
                    }
                    wave_chunks += __popcll(chunks);
                    wave_singles += __popcll(singles);
                }
                if (writes) break;
                if (lane == 0) s_x[wave] = make_int4(wave_chunks, wave_singles, 0, 0);
                __syncthreads();
                const int4 x = s_x[lane & (kWaves - 1)];
                const int incl = wave_incl_scan_add(lane < kWaves ? (x.x | (x.y << 16)) : 0, lane); // (at most 8192 each)
                const int total = __builtin_amdgcn_readlane(incl, kWaves - 1), before = __builtin_amdgcn_readlane(incl, wave);
                chunk_at = part_base + n_chunk + (before & 0xFFFF) - wave_chunks;
                single_at = part_base + n_single + (before >> 16) - wave_singles;
                n_chunk += total & 0xFFFF;
                n_single += total >> 16;
            }
            n_uniq += seg_count;
        }

        // ---- the next pending range
        cur = end;
        if (depth > 0) {
            __syncthreads(); // (the LDS is free again)
            --depth;
            end = s_stack[depth];
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int e = (block_z - args.parts) * args.T + block_x; // (a further range's number; the others have none)
        const bool further = EXTRA && block_z >= args.parts;
        int4 *info = ws.part_info + 2 * (further ? args.T * args.parts + e : t * args.parts + block_z);
        const int w = further ? (t + 1) * args.parts + e : 0;
        info[0] = make_int4(max(part_base, 0), n_uniq, n_chunk, n_single);
        info[1] = make_int4(s_class[0] | (s_class[1] << 16), s_class[2] | (s_class[3] << 16), s_class[4], w);
    }
}

template <int THREADS, int CAP, bool PARTITIONED, bool EXTRA>
__global__ __launch_bounds__(THREADS) void dedupe_kernel(DedupeArgs args)
{
    __shared__ DedupeLds<THREADS, CAP> lds;
    dedupe_body<THREADS, CAP, PARTITIONED, EXTRA>(args, lds, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Kernel 1 for launches with a workgroup per CU or more before any table is cut into ranges (several batches side by side) and at
// most kTableCap lookups in a table: a workgroup sorts a whole table.  There is nothing to look for and nothing to piece together,
// so a thread's items stay in registers between the sort's passes (the LDS holds them once) and every loop over them is unrolled.
// Bound by the chains of a workgroup that has its CU to itself: LDS round trips between barriers, and fetching its code.
// 208 tables x 8192 lookups (eight batches of 26): 40.5 us, dedupe_kernel with one range 45; with dedupe_finish_kernel 60.0 (67.3);
// x 16384 lookups: 106 (155, two ranges).
constexpr int kTableThreads = 1024, kTableCap = 16384;

__global__ __launch_bounds__(kTableThreads) void dedupe_table_kernel(DedupeArgs args)
{
    constexpr int THREADS = kTableThreads, kWaves = THREADS / kWave, kItems = kTableCap / THREADS;
    __shared__ __align__(16) unsigned s_key[kTableCap];
    __shared__ unsigned short s_pos[kTableCap], s_head[kTableCap + 2]; // s_head: sorted index of each segment's head, and the last one's end
    // digit counters, a row of 256 per wave, and where the wave's items of each digit go; later the bags' first positions
    __shared__ __align__(16) unsigned short s_digits[2][kWaves * 256];
    __shared__ int s_x[kWaves], s_back[kWaves], s_class[kChunkClasses];

    const DedupeBatch &bt = args.b[blockIdx.y];
    const BwdWs &ws = bt.ws;
    const int t = blockIdx.x, B = args.B, tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const unsigned rows_t = (unsigned)(args.row_offsets[t + 1] - args.row_offsets[t]); // host: <= DQRM_MAX_TABLE_ROWS
    const TableExtent x = table_extent<THREADS>(bt.offsets, t, B, bt.N, bt.limit, tid, s_back);
    const long long lo = x.lo;
    const int n = x.n, base = (int)lo; // host: n <= kTableCap
    const int64_t *__restrict__ bag_offsets = bt.offsets + (long long)t * B;
    // items, wave-striped: number r of a lane is item first + r * 64 of the table
    const int rounds = (n + THREADS - 1) / THREADS, first = wave * rounds * kWave + lane;
    auto each = [&](auto &&body) {
#pragma unroll
        for (int r = 0; r < kItems; ++r)
            if (r < rounds) body(r, first + r * kWave);
    };
    long long raw[kItems];
    each([&](int r, int i) { raw[r] = bt.indices[lo + min(i, n - 1)]; });

    const bool even = (unsigned long long)args.even.d * (unsigned)B == (unsigned)n;
    const BagSearch bags{bag_offsets, lo, B, max(0, 32 - __clz((B - 1) / (2 * kWaves * 256))), even};
    int bad_code = tid == 0 ? x.bad_code : 0;
    long long bad_value = x.bad_value;
    if (n > 0) {
        const int b = bags.disorder<THREADS>(0, B, n, tid);
        if (b >= 0) bad_code = DQRM_ERR_BAD_OFFSETS, bad_value = (long long)t * B + b;
    }
    if (bad_code != 0) report(bad_code, t, bad_value);
    if (tid < kAbsmaxSlots) *absmax_slot(ws.absmax_slots, t, tid) = 0.0f;
    if (tid < kChunkClasses) s_class[tid] = 0; // (read after more barriers)

    // ---- 1. stable LSD radix sort of the rows (or the number of rows, for a bad index), at most 8 bits per pass
    unsigned key[kItems], pos[kItems]; // pos: in the upper half the rank inside the wave's items of the digit
    bool bad_index = false;
    each([&](int r, int i) {
        const bool good = (unsigned long long)raw[r] < rows_t;
        if (!good && i < n) bad_index = true, bad_value = raw[r];
        // (padding: the largest digit in every pass and last in line, so it stays last)
        key[r] = i < n ? (good ? (unsigned)raw[r] : rows_t) : ~0u;
        pos[r] = (unsigned)i;
    });
    if (bad_index) report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, bad_value);
    const int nbits = 32 - __clz(rows_t | 1u), passes = (nbits + 7) / 8, bits = (nbits + passes - 1) / passes;
    const unsigned digit_mask = (1u << bits) - 1u;
    unsigned short *my_cnt = s_digits[0] + wave * 256, *my_place = s_digits[1] + wave * 256;
#pragma unroll 1
    for (int p = 0; p < passes; ++p) {
        const int shift = bits * p;
        // (a wave's row of counters is its own: no barrier between clearing and counting)
        *reinterpret_cast<uint2 *>(my_cnt + 4 * lane) = make_uint2(0u, 0u);
        each([&](int r, int) {
            const unsigned d = (key[r] >> shift) & digit_mask;
            const unsigned long long peers = match_digit(d, bits);
            const unsigned prev = my_cnt[d];
            const int rank = mask_rank(peers);
            pos[r] = (pos[r] & 0xFFFFu) | ((prev + (unsigned)rank) << 16);
            if (rank == 0) my_cnt[d] = (unsigned short)(prev + (unsigned)__popcll(peers));
        });
        __syncthreads(); // (and every thread has its items of the pass before)
        uint2 starts;
        *reinterpret_cast<uint2 *>(my_place + 4 * lane) = digit_places<kWaves>(s_digits[0], wave, lane, &starts);
        each([&](int r, int) {
            const int to = my_place[(key[r] >> shift) & digit_mask] + (int)(pos[r] >> 16);
            s_key[to] = key[r];
            s_pos[to] = (unsigned short)pos[r];
        });
        __syncthreads();
        each([&](int r, int i) {
            key[r] = s_key[i];
            pos[r] = s_pos[i];
        });
    }

    // ---- 2. bags: the guessed ones' offsets are requested now and looked at when the heads are known (half the words: a good
    // offset fits them, and others have been reported)
    int bag_lo[kItems], bag_hi[kItems];
    if (even)
        each([&](int r, int i) {
            const unsigned g = args.even.div(i < n ? pos[r] : 0u); // below B, as the position is below n
            bag_lo[r] = (int)bag_offsets[g];
            bag_hi[r] = (int)bag_offsets[g + 1u];
        });
    else
        bags.stage<THREADS>(s_digits[0], tid); // (all waves are through with the digits)

    // ---- 3. segment heads (the valid items come first)
    unsigned long long heads[kItems];
    int wave_heads = 0, wave_valid = 0;
    each([&](int r, int i) {
        const unsigned prev = s_key[max(i - 1, 0)];
        const bool valid = key[r] < rows_t; // (padding is not)
        heads[r] = __ballot(valid && (i == 0 || key[r] != prev));
        wave_heads += __popcll(heads[r]);
        wave_valid += __popcll(__ballot(valid));
    });
    if (lane == 0) s_x[wave] = wave_heads | (wave_valid << 16);
    __syncthreads();
    const int incl = wave_incl_scan_add(lane < kWaves ? s_x[lane] : 0, lane); // (at most 16384 each)
    const int total = __builtin_amdgcn_readlane(incl, kWaves - 1);
    const int seg_count = total & 0xFFFF, valid_count = total >> 16;
    const int heads_before = (__builtin_amdgcn_readlane(incl, wave) & 0xFFFF) - wave_heads;
    int seg_at = heads_before;
    each([&](int r, int i) {
        if ((heads[r] >> lane) & 1ull) s_head[seg_at + mask_rank(heads[r])] = (unsigned short)i;
        seg_at += __popcll(heads[r]);
    });
    if (tid == 0) s_head[seg_count] = (unsigned short)valid_count; // end of the last segment
    bool search = !even;
    if (even)
        each([&](int r, int i) {
            const int p = i < n ? (int)pos[r] : 0;
            search |= bag_lo[r] > base + p || base + p >= bag_hi[r];
            bag_lo[r] = (int)args.even.div((unsigned)p);
        });
    __syncthreads();
    if (search) // (bags of other lengths that happen to add up to the same number are searched)
        each([&](int r, int i) { bag_lo[r] = bags.find(s_digits[0], i < n ? (int)pos[r] : 0); });

    // ---- 4. the sorted order and the lists.  Chunk heads: every DQRM_SEG_CHUNK-th item of a segment, counted from its head; a
    // row looked up exactly once is a "single" and listed separately.  Both lists in sorted order: counted first, then written.
    unsigned info[kItems]; // segment's first item (bits 0..14), its end (bits 15..29), single (bit 30), chunk (bit 31)
    int wave_chunks = 0, wave_singles = 0;
    seg_at = heads_before - 1;
    each([&](int r, int i) {
        const int seg = max(seg_at + mask_rank(heads[r]) + (int)((heads[r] >> lane) & 1ull), 0);
        seg_at += __popcll(heads[r]);
        const int start = s_head[seg], end = s_head[min(seg + 1, seg_count)];
        const bool chead = i < valid_count && ((i - start) % DQRM_SEG_CHUNK) == 0, single = chead && i == start && end == i + 1;
        info[r] = (unsigned)start | ((unsigned)end << 15) | (single ? 1u << 30 : 0u) | (chead && !single ? 1u << 31 : 0u);
        wave_singles += __popcll(__ballot(single));
        wave_chunks += __popcll(__ballot(chead && !single));
    });
    __syncthreads(); // (s_x is free again)
    if (lane == 0) s_x[wave] = wave_chunks | (wave_singles << 16);
    __syncthreads();
    const int list_incl = wave_incl_scan_add(lane < kWaves ? s_x[lane] : 0, lane);
    const int list_total = __builtin_amdgcn_readlane(list_incl, kWaves - 1), before = __builtin_amdgcn_readlane(list_incl, wave);
    int chunk_at = base + (before & 0xFFFF) - wave_chunks, single_at = base + (before >> 16) - wave_singles;
    seg_at = heads_before - 1;
    each([&](int r, int i) {
        const int seg = max(seg_at + mask_rank(heads[r]) + (int)((heads[r] >> lane) & 1ull), 0);
        seg_at += __popcll(heads[r]);
        const int start = (int)(info[r] & 0x7FFFu), end = (int)((info[r] >> 15) & 0x7FFFu);
        const bool single = (info[r] >> 30) & 1u, chunk = info[r] >> 31;
        const unsigned long long singles = __ballot(single), chunks = __ballot(chunk);
        if (i < n) bt.sorted_pos[base + i] = base + (int)pos[r];
        if (i < valid_count) ws.sorted_bag[base + i] = bag_lo[r];
        if (single) ws.single_local[single_at + mask_rank(singles)] = make_int4(base + i, bag_lo[r], seg, (int)key[r]);
        if (chunk) {
            const int nchunks = (end - start + DQRM_SEG_CHUNK - 1) / DQRM_SEG_CHUNK, len = min(DQRM_SEG_CHUNK, end - i);
            ws.chunk_local[chunk_at + mask_rank(chunks)] =
                make_chunk_desc(base + i, len, (i - start) / DQRM_SEG_CHUNK, nchunks, seg,
                                args.by_length ? atomicAdd(&s_class[chunk_class(len)], 1) : 0, key[r]);
            // the arrival counter of a segment of more than one chunk starts at zero
            if (i == start && nchunks > 1) ws.seg_count[(base + i) / DQRM_SEG_CHUNK] = 0;
        }
        single_at += __popcll(singles);
        chunk_at += __popcll(chunks);
    });
    __syncthreads();
    if (tid == 0) {
        ws.part_info[2 * t] = make_int4(base, seg_count, list_total & 0xFFFF, list_total >> 16);
        ws.part_info[2 * t + 1] = make_int4(s_class[0] | (s_class[1] << 16), s_class[2] | (s_class[3] << 16), s_class[4], 0);
    }
}

// ---------------------------------------------------------------------------
// Kernel 2 of dqrm_dedupe: the parts' lists -> one dense, global chunk list and the index-only outputs (unique rows,
// segment offsets, table offsets, count).
//
// Dense chunk descriptor, as the summing kernels read it:
//   x  global sorted position of the chunk's first lookup
//   y  len | index of the chunk inside its segment | chunks in the segment (as above)
//   z  global index of the segment (row of `values`)
//   w  table
// Dense single descriptor: x bag, y global index of the segment, z table.
// its dynamic LDS
inline size_t finish_lds_bytes(const DedupeArgs &a)
{
    const size_t most = a.extra ? (size_t)a.T * a.parts + a.extra : (size_t)kMaxParts;
    return sizeof(int) * ((3 + kChunkClasses) * (most + 1) + most) + (a.extra ? 2 * sizeof(unsigned short) * most : 0);
}

template <bool EXTRA>
__global__ __launch_bounds__(kSegThreads) void dedupe_finish_kernel(DedupeArgs args)
{
    const DedupeBatch &a = args.b[blockIdx.y];
    const BwdWs &ws = a.ws;
    // exclusive sums over the parts in their order: segments, chunks, singles, chunks of each class (V + 1 entries each); the
    // parts' first sorted positions; with further ranges, the parts' tables and which part_info is whose
    constexpr int kSums = 3 + kChunkClasses, kWaves = kSegThreads / kWave;
    extern __shared__ int finish_lds[]; // finish_lds_bytes()
    __shared__ int s_w[kSums][kWaves];
    const int T = args.T, parts = args.parts, most = EXTRA ? T * parts + args.extra : kMaxParts; // (a constant where it can be: every access pays for it)
    int *s_base = finish_lds + kSums * (most + 1);
    unsigned short *s_table = reinterpret_cast<unsigned short *>(s_base + most), *s_order = s_table + most;
    auto s_sum = [&](int k) { return finish_lds + k * (most + 1); };
    const int *s_uniq = s_sum(0), *s_chunk = s_sum(1), *s_single = s_sum(2);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    int V = T * parts;
    // (requested beside the number of further ranges, which is nearly always zero)
    int per = (V + kSegThreads - 1) / kSegThreads; // consecutive parts per thread
    int4 x = ws.part_info[2 * min(tid * per, V - 1)], y = ws.part_info[2 * min(tid * per, V - 1) + 1];
    const int more = EXTRA ? __builtin_amdgcn_readfirstlane(ws.totals[3]) : 0;
    if (EXTRA && __builtin_expect(more > 0, 0)) {
        // a further range knows its place, and with it its table; another one comes behind the further ones of earlier tables
        int *table = finish_lds; // (the sums are not there yet)
        for (int e = tid; e < more; e += kSegThreads) {
            const int place = ws.part_info[2 * (V + e) + 1].w;
            table[e] = (int)args.by_parts.div((unsigned)(place - e)) - 1;
            s_order[place] = (unsigned short)(V + e);
            s_table[place] = (unsigned short)table[e];
        }
        __syncthreads();
        for (int v = tid; v < V; v += kSegThreads) {
            const int t = (int)args.by_parts.div((unsigned)v);
            int lo = 0, hi = more; // the first one of table t or behind it
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (table[mid] < t) lo = mid + 1;
                else hi = mid;
            }
            s_order[v + lo] = (unsigned short)v;
            s_table[v + lo] = (unsigned short)t;
        }
        __syncthreads();
        V += more;
        per = (V + kSegThreads - 1) / kSegThreads;
        const int id = s_order[min(tid * per, V - 1)];
        x = ws.part_info[2 * id], y = ws.part_info[2 * id + 1];
    }
    auto table_of_part = [&](int v) { return EXTRA && more > 0 ? (int)s_table[v] : (int)args.by_parts.div((unsigned)v); };
    {
        const int first = tid * per, end = min(first + per, V);
        int mine[kSums] = {}, c[kSums];
        auto counts = [&](int v) { // of part v, into c
            if (v > first || per > 1) {
                const int id = EXTRA && more > 0 ? s_order[v] : v;
                x = ws.part_info[2 * id], y = ws.part_info[2 * id + 1];
            }
            c[0] = x.y, c[1] = x.z, c[2] = x.w;
            c[3] = y.x & 0xFFFF, c[4] = (int)((unsigned)y.x >> 16), c[5] = y.y & 0xFFFF, c[6] = (int)((unsigned)y.y >> 16), c[7] = y.z;
            s_base[v] = x.x;
        };
        static_assert(kChunkClasses == 5, "counts");
        for (int v = first; v < end; ++v) {
            counts(v);
#pragma unroll
            for (int k = 0; k < kSums; ++k) mine[k] += c[k];
        }
        int before[kSums];
#pragma unroll
        for (int k = 0; k < kSums; ++k) {
            const int incl = wave_incl_scan_add(mine[k], lane);
            if (lane == kWave - 1) s_w[k][wave] = incl;
            before[k] = incl - mine[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSums; ++k)
#pragma unroll
            for (int w = 0; w < kWaves; ++w) before[k] += w < wave ? s_w[k][w] : 0;
        for (int v = first; v < end; ++v) {
            if (per > 1) counts(v); // (one part per thread: they are still here)
#pragma unroll
            for (int k = 0; k < kSums; ++k) {
                s_sum(k)[v] = before[k];
                before[k] += c[k];
                if (v == V - 1) s_sum(k)[V] = before[k];
            }
        }
        __syncthreads();
    }
    const int C = s_chunk[V], U = s_uniq[V], S = s_single[V];
    if (blockIdx.x == 0) {
        if (EXTRA && more > 0)
            for (int v = tid; v < V; v += kSegThreads) {
                if (v == 0 || s_table[v] != s_table[v - 1]) a.tuo[s_table[v]] = s_uniq[v];
            }
        else
            for (int k = tid; k < T; k += kSegThreads) a.tuo[k] = s_uniq[k * parts];
        if (tid == 0) {
            a.tuo[T] = U;
            *a.num_unique = U;
            a.seg_offsets[U] = (int32_t)a.N;
            ws.totals[0] = C;
            ws.totals[1] = U;
            ws.totals[2] = S;
        }
    }
    const int at = (int)(blockIdx.x * kSegThreads) + tid, step = (int)(gridDim.x * kSegThreads);
    // Chunks, kChunksPerWave consecutive ones per wave: their descriptors (a lane each, the other lanes along for the
    // ride), then the bags of their lookups at a place that depends on the chunk's index alone (a chunk has at least
    // two lookups, so there are at most N / 2 chunks): half a wave per chunk.
    constexpr int kChunksPerWave = 8;
    for (int c0 = at / kWave * kChunksPerWave; c0 < C; c0 += step / kWave * kChunksPerWave) {
        const int c = min(c0 + (lane & (kChunksPerWave - 1)), C - 1);
        const int v = table_of(s_chunk, V, c);
        const int4 d = ws.chunk_local[s_base[v] + (c - s_chunk[v])];
        const int j = s_uniq[v] + (d.z & 0xFFFF);
        // its place in the dense list; by length: after the chunks of longer classes, then those of its own in earlier parts
        int place = c;
        if (args.by_length) {
            const int cls = chunk_class(desc_len(d));
            place = s_sum(3 + cls)[v] + (int)((unsigned)d.z >> 16);
#pragma unroll
            for (int k = 0; k + 1 < kChunkClasses; ++k) place += k < cls ? s_sum(3 + k)[V] : 0;
        }
        if (lane < kChunksPerWave && c0 + lane < C) {
            if (desc_kchunk(d) == 0) { // first chunk of its segment: d.x is the segment's head
                a.uniq_rows[j] = (int64_t)(unsigned)d.w;
                a.seg_offsets[j] = d.x;
            }
            ws.chunk_desc[place] = make_int4(d.x, d.y, j, table_of_part(v));
        }
        int bag[kChunksPerWave / 2], to[kChunksPerWave / 2];
        const int i = lane & (DQRM_SEG_CHUNK - 1);
#pragma unroll
        for (int q = 0; q < kChunksPerWave / 2; ++q) {
            const int from = 2 * q + (lane >> 5);
            const int x = __shfl(d.x, from, kWave), len = __shfl(desc_len(d), from, kWave);
            to[q] = __shfl(place, from, kWave);
            bag[q] = ws.sorted_bag[x + min(i, len - 1)];
        }
#pragma unroll
        for (int q = 0; q < kChunksPerWave / 2; ++q)
            if (c0 + 2 * q + (lane >> 5) < C) // (past the chunk's end: its last bag again)
                ws.chunk_bags[(int64_t)to[q] * DQRM_SEG_CHUNK + i] = bag[q];
    }
    for (int c = at; c < S; c += step) {
        const int v = table_of(s_single, V, c);
        const int4 d = ws.single_local[s_base[v] + (c - s_single[v])]; // {sorted position, bag, segment, row}
        const int j = s_uniq[v] + d.z;
        a.uniq_rows[j] = (int64_t)(unsigned)d.w;
        a.seg_offsets[j] = d.x;
        ws.single_desc[c] = make_int4(d.y, j, table_of_part(v), 0);
    }
}

} // namespace dqrm
