// Forward: gather -> INT4 fake-quant -> sum-pool (Sec. 3.1 and Sec. 4.1 of the paper).
//
// A workgroup owns a tile of kFwdTileB consecutive samples x up to kFwdTileT
// consecutive tables (32 of embbag_fwd_kernel's).  The index arrays are table-major (bag = t * B + b), the
// output is sample-major (slot = b * T + t): with 16 samples per tile every
// 128-byte line of `offsets` / `indices` is read by one workgroup only, and with
// all tables in the tile (T <= kFwdTileT) the workgroup's output is one
// contiguous piece of `out`.  Three phases, each one memory round trip deep, so
// the dependent chain offsets -> index -> row is paid once per workgroup:
//   A  one thread per bag (sample fastest, so the reads coalesce) reads the
//      bag's extent and first index, checks them, and leaves the row's byte
//      offset, the table scale and the output slot in LDS, filed in output order;
//   B  groups of G = pow2ceil(D/4) lanes walk the tile in output order; lane l
//      of a group owns columns 4l..4l+3 (one 16-byte store per row).  The first
//      rows of a whole batch of slots are requested before any is used;
//   C  `out = 0 + s * q` is stored.  Tiles with a bag of more than one lookup take the
//      general path instead: the tile's index lists are turned into checked row
//      offsets in LDS by all threads (one more round trip for the whole tile), then
//      every bag's rows are requested kFwdBagBatch at a time and added in order
//      (packed rows of many bags: by fwd_bags, 8 codes of a row to a lane).
// The per-column sum is the plain left-to-right sum over the bag, so no
// cross-lane reduction is needed and the result does not depend on the mapping.
#pragma once

#include "dqrm_device.hpp"

namespace dqrm {

constexpr int kFwdTileB = 16;                      // samples per tile
constexpr int kFwdThreads = 512;                   // of embbag_fwd_kernel; a workgroup has as many slots for bags as threads
constexpr int kFwdTileT(int threads) { return threads / kFwdTileB; } // tables per tile, at most
constexpr int kFwdBatch = 16;                      // first rows in flight per lane
constexpr int kFwdLookupsPerSlot = 8;              // lookups of a tile whose row offsets fit in LDS (general bags), over its slots
constexpr int kFwdBagBatch = 8;                    // rows of one bag in flight per lane (general bags)

struct FwdArgs {
    const float *master;
    const uint8_t *packed;
    const float *w_scale;
    const int64_t *row_offsets;
    const int64_t *indices;
    const int64_t *offsets;
    float *out;
    int8_t *codes;
    int64_t num_indices;
    int T, B, D;
    int tile_t;  // tables per tile: min(T, kFwdTileT); the tiles' grid = (ceil(B / kFwdTileB), ceil(T / tile_t))
    int no_rows; // the tables hold no row at all: nothing may be read from them
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void store_codes(int8_t *codes, int64_t i, int D, int col, float4 q)
{
    char4 c = make_char4((signed char)(int)q.x, (signed char)(int)q.y, (signed char)(int)q.z, (signed char)(int)q.w);
    *reinterpret_cast<char4 *>(codes + i * D + col) = c;
}

// The raw bytes of 4 consecutive elements of one row as they come from memory:
// two packed bytes, or four fp32 values.
template <bool PACKED> struct RowPiece;
template <> struct RowPiece<true> {
    unsigned v;
    __device__ __forceinline__ void load(const char *p) { v = *reinterpret_cast<const unsigned short *>(p); }
    __device__ __forceinline__ float4 codes(Scale) const
    {
        // the builtin's result is typed unsigned although the extract sign-extends
        return make_float4((float)(int)__builtin_amdgcn_sbfe((int)v, 0, 4), (float)(int)__builtin_amdgcn_sbfe((int)v, 4, 4),
                           (float)(int)__builtin_amdgcn_sbfe((int)v, 8, 4), (float)(int)__builtin_amdgcn_sbfe((int)v, 12, 4));
    }
};
template <> struct RowPiece<false> {
    float4 w;
    __device__ __forceinline__ void load(const char *p) { w = *reinterpret_cast<const float4 *>(p); }
    __device__ __forceinline__ float4 codes(Scale s) const
    {
        return make_float4((float)int4_code(w.x, s), (float)int4_code(w.y, s), (float)int4_code(w.z, s),
                           (float)int4_code(w.w, s));
    }
};

// The slots of the tile in output order when no bag has more than one lookup (the usual batch):
// out = 0 + s * q, nothing else to add.  A slot without a valid lookup reads row 0 and multiplies by 0;
// the addition turns a -0 product into the +0 of an empty sum.  Slots from `live` on do not exist
// (samples beyond the batch); their LDS entries read as "no lookup".
template <int THREADS, int G, bool PACKED>
__device__ __forceinline__ void fwd_single_lookup_tile(const char *tab, const int64_t *s_off, const Scale *s_scale,
                                                       const float *s_mul, const int *s_slot, int grp, float *out_col,
                                                       int D, int live)
{
    constexpr int kGroups = THREADS / G;
    constexpr int kIters = (THREADS + kGroups - 1) / kGroups;
    constexpr int kBatch = kIters < kFwdBatch ? kIters : kFwdBatch;
    for (int k0 = 0; k0 * kGroups < live; k0 += kBatch) {
        RowPiece<PACKED> piece[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = min((k0 + k) * kGroups + grp, THREADS - 1);
            piece[k].load(tab + s_off[i]);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = (k0 + k) * kGroups + grp;
            if (i < live) {
                const float m = s_mul[i];
                const float4 q = piece[k].codes(s_scale[i]);
                const f32x4 v = {0.f + m * q.x, 0.f + m * q.y, 0.f + m * q.z, 0.f + m * q.w};
                // (plain stores: the consumer of `out`, the dense part of the model, runs next and finds it in the caches)
                *reinterpret_cast<f32x4 *>(out_col + (size_t)(unsigned)s_slot[i] * D) = v;
            }
        }
    }
}

// The bags of packed rows of a tile whose lookups' row offsets lie in LDS.  A group of lanes walks its bags kFwdBagBatch lookups at a time, the next
// ones (of the same bag or of the next) requested before the present ones are added: what bounds it is the chain of these round
// trips, 416 bags of a tile over the workgroup's groups.  8 codes to a lane make the groups half as wide and twice as many as for
// one lookup per bag, where the 16-byte stores decide.  No load is under a branch: a lookup past the bag's end or with a bad index
// reads row 0 and enters the sum as 0 * q, which leaves the sum as it is.
// Bags of 0 to 8 lookups, 26 x 8192 x 64, packed: 34.0 -> 24 us in a kernel trace (a pass among others 31.6 -> 22.9); bags of 8: 41.4 -> 38.
template <int THREADS, int G>
__device__ __forceinline__ void fwd_bags(const FwdArgs &a, const int64_t *s_loff, const int *s_pos, const int *s_len, const int64_t *s_beg,
                                         const int *s_slot, const Scale *s_scale, int live, int tid)
{
    constexpr int kCols = 8, kLanes = G / 2, kGroups = THREADS / kLanes;
    const int col = (tid & (kLanes - 1)) * kCols;
    if (col >= a.D) return; // lanes beyond the row
    const char *tab = reinterpret_cast<const char *>(a.packed) + (col >> 1);
    struct Batch {
        int i, j0, len;
        unsigned piece[kFwdBagBatch]; // 8 codes each
        unsigned valid; // bit per lookup
    };
    auto request = [&](Batch &b, int i, int j0) {
        b.i = i, b.j0 = j0, b.valid = 0u;
        b.len = i < live ? s_len[i] : 0;
        const int pos = i < live ? s_pos[i] : 0;
#pragma unroll
        for (int j = 0; j < kFwdBagBatch; ++j) {
            const int64_t off = s_loff[max(pos + min(j0 + j, b.len - 1), 0)];
            const bool valid = j0 + j < b.len && off >= 0;
            b.valid |= valid ? 1u << j : 0u;
            b.piece[j] = *reinterpret_cast<const unsigned *>(tab + (valid ? off : 0));
        }
    };
    float acc[kCols] = {};
    auto add = [&](const Batch &b) { // and the bag's end
        const float s = s_scale[b.i].s;
#pragma unroll
        for (int j = 0; j < kFwdBagBatch; ++j) {
            const float m = (b.valid >> j) & 1u ? s : 0.0f;
            float q[kCols];
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                q[k] = (float)(int)__builtin_amdgcn_sbfe((int)b.piece[j], 4 * k, 4);
                acc[k] = acc[k] + m * q[k];
            }
            if (a.codes && (b.valid >> j) & 1u)
#pragma unroll
                for (int k = 0; k < kCols; k += 4)
                    store_codes(a.codes, s_beg[b.i] + b.j0 + j, a.D, col + k, make_float4(q[k], q[k + 1], q[k + 2], q[k + 3]));
        }
        if (b.j0 + kFwdBagBatch >= b.len) {
            float *to = a.out + (size_t)(unsigned)s_slot[b.i] * a.D + col;
#pragma unroll
            for (int k = 0; k < kCols; k += 4) {
                const f32x4 v = {acc[k], acc[k + 1], acc[k + 2], acc[k + 3]};
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(to + k));
                acc[k] = acc[k + 1] = acc[k + 2] = acc[k + 3] = 0.0f;
            }
        }
    };
    // one step: `now` is added while `then`, what comes after it, travels; false if nothing comes after it in the whole wave
    auto step = [&](const Batch &now, Batch &then) {
        const bool more = now.j0 + kFwdBagBatch < now.len;
        const int i = more ? now.i : now.i + kGroups;
        if (!__any(i < live)) {
            if (now.i < live) add(now);
            return false;
        }
        request(then, i, more ? now.j0 + kFwdBagBatch : 0);
        if (now.i < live) add(now);
        return true;
    };
    Batch x, y;
    request(x, tid / kLanes, 0);
    while (step(x, y) && step(y, x)) {
    }
}

// LDS of a workgroup; an entry per slot of its tile
template <int THREADS>
struct FwdLds {
    int64_t off[THREADS]; // byte offset of the first lookup's row in the table (0 if none / invalid)
    int64_t beg[THREADS]; // position of the bag's first lookup
    int len[THREADS];     // lookups in the bag
    int tab[THREADS];
    int slot[THREADS];    // output slot b * T + t (below 2^31: checked on the host)
    Scale scale[THREADS]; // table scale (and its reciprocal)
    float mul[THREADS];   // table scale, or 0 when the first lookup is absent or invalid
    int general;          // some bag of the tile has more than one lookup
    int64_t loff[THREADS * kFwdLookupsPerSlot]; // general bags: row byte offset of every lookup of the tile, -1 if bad
    int pos[THREADS];     // ... where slot i's list starts in loff
    int w[THREADS / kWave];
};

// Tile (block_x, block_y)
template <int THREADS, int G, bool PACKED>
__device__ __forceinline__ void embbag_fwd_body(const FwdArgs &a, FwdLds<THREADS> &lds, int block_x, int block_y)
{
    auto &s_off = lds.off;
    auto &s_beg = lds.beg;
    auto &s_len = lds.len;
    auto &s_tab = lds.tab;
    auto &s_slot = lds.slot;
    auto &s_scale = lds.scale;
    auto &s_mul = lds.mul;
    auto &s_general = lds.general;
    auto &s_loff = lds.loff;
    auto &s_pos = lds.pos;
    auto &s_w = lds.w;

    const int tid = threadIdx.x;
    const int b0 = block_x * kFwdTileB, t0 = block_y * a.tile_t;
    const int nb = min(kFwdTileB, a.B - b0), nt = min(a.tile_t, a.T - t0); // samples / tables of this tile
    const int live = nb * nt;                                              // its slots, a prefix in output order
    const int row_bytes = PACKED ? (a.D >> 1) : a.D * 4;
    if (tid == 0) s_general = 0;
    __syncthreads();

    // ---- phase A: one bag per thread, sample fastest ---------------------------
    {
        const int s = tid; // (as many slots as threads)
        const int bl = s % kFwdTileB, tl = s / kFwdTileB;
        const bool exists = bl < nb && tl < nt;
        // output-order index inside the tile; the entries past `live` are filled with "no lookup"
        int i = bl * nt + tl;
        if (!exists) i = tl < nt ? live + (bl - nb) * nt + tl : s;
        int64_t off = 0, beg = 0;
        int len = 0;
        const int t = exists ? t0 + tl : 0, b = b0 + bl;
        float sc = 1.0f, mul = 0.0f;
        if (exists) {
            const int64_t bag = (int64_t)t * a.B + b;
            int64_t lo = a.offsets[bag], hi = a.offsets[bag + 1];
            if (lo < 0 || hi > a.num_indices || lo > hi) {
                report(DQRM_ERR_BAD_OFFSETS, t, bag);
                lo = hi = 0;
            }
            if (hi - lo > 0x7fffffff) hi = lo + 0x7fffffff;
            beg = lo;
            len = (int)(hi - lo);
            sc = a.w_scale[t];
            if (len > 0) {
                const int64_t idx = a.indices[lo];
                const int64_t r0 = a.row_offsets[t], r1 = a.row_offsets[t + 1];
                if (idx >= 0 && idx < r1 - r0) {
                    off = (r0 + idx) * row_bytes;
                    mul = sc;
                } else {
                    report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, idx);
                }
                if (len > 1) s_general = 1;
            }
        }
        s_off[i] = off;
        s_beg[i] = beg;
        s_len[i] = len;
        s_tab[i] = t;
        s_slot[i] = exists ? b * a.T + t : 0;
        // the packed rows hold codes already: no quotient, no reciprocal
        s_scale[i] = PACKED ? Scale(sc, 0.0f) : Scale(sc);
        s_mul[i] = mul;
    }
    __syncthreads();

    // ---- general bags: the tile's lookups as checked row offsets in LDS ------------------
    const bool general = s_general != 0 || a.codes != nullptr || a.no_rows != 0;
    bool staged = false;
    if (general && !a.no_rows) {
        // position of every slot's list in s_loff (slots in output order; a slot per thread)
        const int my_len = tid < live ? s_len[tid] : 0;
        int total;
        const int pos = block_excl_scan_add<THREADS / kWave>(my_len, tid & (kWave - 1), tid / kWave, s_w, &total);
        s_pos[tid] = pos;
        staged = total <= THREADS * kFwdLookupsPerSlot; // block-uniform
        if (staged && my_len > 0) {
            const int t = s_tab[tid];
            const int64_t r0 = a.row_offsets[t], r1 = a.row_offsets[t + 1];
            const int64_t beg = s_beg[tid];
            for (int j0 = 0; j0 < my_len; j0 += kFwdBagBatch) {
                int64_t idx[kFwdBagBatch];
#pragma unroll
                for (int j = 0; j < kFwdBagBatch; ++j) idx[j] = a.indices[beg + min(j0 + j, my_len - 1)];
#pragma unroll
                for (int j = 0; j < kFwdBagBatch; ++j) {
                    if (j0 + j >= my_len) break;
                    int64_t off = -1;
                    if (idx[j] >= 0 && idx[j] < r1 - r0)
                        off = (r0 + idx[j]) * row_bytes;
                    else
                        report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, idx[j]);
                    s_loff[pos + j0 + j] = off;
                }
            }
        }
        __syncthreads();
    }

    // ---- phases B and C ------------------------------------------------------------
    // Packed rows, and several bags to a group: by groups of half as many lanes (fwd_bags).  With one bag or less to a group their lanes
    // only have twice the work: 16000 bags of 3 lookups x 64, one table, 7.7 us here and 8.6 there; bags of up to 6, 2 tables x 10901 x
    // 40, 7.9 and 8.0.  Of master rows a lane takes 16 bytes either way, and their codes' arithmetic, not the round trips, takes the
    // time: 20 tables x 4001 bags of up to 6 lookups x 32 14.8 here, 15.9 with the next rows requested ahead.
    if (PACKED && staged && live > 2 * (THREADS / G)) {
        fwd_bags<THREADS, G>(a, s_loff, s_pos, s_len, s_beg, s_slot, s_scale, live, tid);
        return;
    }
    constexpr int kGroups = THREADS / G; // groups per workgroup
    const int lg = tid & (G - 1);
    const int grp = tid / G;
    const int col = lg * 4;
    if (col >= a.D) return; // lanes beyond the row (D / 4 not a power of two) have nothing to do from here on
    const char *tab = PACKED ? reinterpret_cast<const char *>(a.packed) + (col >> 1)
                             : reinterpret_cast<const char *>(a.master + col);
    float *out_col = a.out + col;

    if (!general) {
        fwd_single_lookup_tile<THREADS, G, PACKED>(tab, s_off, s_scale, s_mul, s_slot, grp, out_col, a.D, live);
        return;
    }

    if (staged) {
        // A bag's rows kFwdBagBatch at a time, none under a branch: a lookup past the bag's end or with a bad
        // index reads row 0 and enters the sum as 0 * q, which leaves the sum as it is.
        for (int i = grp; i < live; i += kGroups) {
            const Scale sq = s_scale[i];
            const int len = s_len[i], pos = s_pos[i];
            const int64_t beg = s_beg[i];
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int j0 = 0; j0 < len; j0 += kFwdBagBatch) {
                RowPiece<PACKED> piece[kFwdBagBatch];
                float m[kFwdBagBatch];
#pragma unroll
                for (int j = 0; j < kFwdBagBatch; ++j) {
                    const int64_t off = s_loff[pos + min(j0 + j, len - 1)];
                    m[j] = (j0 + j < len && off >= 0) ? sq.s : 0.0f;
                    piece[j].load(tab + (off >= 0 ? off : 0));
                }
#pragma unroll
                for (int j = 0; j < kFwdBagBatch; ++j) {
                    const float4 q = piece[j].codes(sq);
                    acc.x = acc.x + m[j] * q.x;
                    acc.y = acc.y + m[j] * q.y;
                    acc.z = acc.z + m[j] * q.z;
                    acc.w = acc.w + m[j] * q.w;
                    if (a.codes && m[j] != 0.0f) store_codes(a.codes, beg + j0 + j, a.D, col, q);
                }
            }
            const f32x4 v = {acc.x, acc.y, acc.z, acc.w};
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(out_col + (size_t)(unsigned)s_slot[i] * a.D));
        }
        return;
    }

    // general bags of a tile with too many lookups for LDS, or tables without rows: one lookup at a time
    for (int i = grp; i < live; i += kGroups) {
        const Scale sq = s_scale[i];
        const float s = sq.s;
        const int len = s_len[i];
        const int64_t beg = s_beg[i];
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (len > 0 && !a.no_rows) {
            const int t = s_tab[i];
            const int64_t r0 = a.row_offsets[t], r1 = a.row_offsets[t + 1];
            for (int64_t p = beg; p < beg + len; ++p) {
                const int64_t idx = a.indices[p];
                if (idx < 0 || idx >= r1 - r0) {
                    if (lg == 0 && p > beg) report(DQRM_ERR_INDEX_OUT_OF_RANGE, t, idx); // (the first one: phase A)
                    continue;
                }
                RowPiece<PACKED> piece;
                piece.load(tab + (r0 + idx) * row_bytes);
                const float4 q = piece.codes(sq);
                acc.x = acc.x + s * q.x;
                acc.y = acc.y + s * q.y;
                acc.z = acc.z + s * q.z;
                acc.w = acc.w + s * q.w;
                if (a.codes) store_codes(a.codes, p, a.D, col, q);
            }
        }
        const f32x4 v = {acc.x, acc.y, acc.z, acc.w};
        __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(out_col + (size_t)(unsigned)s_slot[i] * a.D));
    }
}

template <int G, bool PACKED>
__global__ __launch_bounds__(kFwdThreads) void embbag_fwd_kernel(FwdArgs a)
{
    __shared__ FwdLds<kFwdThreads> lds;
    embbag_fwd_body<kFwdThreads, G, PACKED>(a, lds, blockIdx.x, blockIdx.y);
}

} // namespace dqrm
