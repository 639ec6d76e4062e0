// The dense part of the DLRM train step (model-architecture table of the paper):
// bottom MLP -> pairwise-dot interaction with the pooled embeddings -> top MLP ->
// sigmoid + mean binary cross-entropy, its backward, and plain SGD on the MLP
// weights.  FP32 throughout (the paper's "MLP in FP32" variant): the matrix
// products of long reductions over few tiles and the interaction run on the fp32
// matrix instructions, all others on the bfloat16 ones with their operands as
// sums of three bfloat16 (gemm_planes_tile).
#pragma once

#include <type_traits>

#include "dqrm_device.hpp"

namespace dqrm {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// C(i,j) = epilogue( sum_r A(i,r) * B(r,j) ), all operands addressed with
// explicit strides so that one kernel serves X*W^T and dY*W (and dY^T*X, split).
//
// One wave owns a 32x32 tile of C: it keeps the tile in the 16 accumulator
// registers of v_mfma_f32_32x32x2_f32 and walks the reduction in slabs of 32.
// In a slab, lane l = (h, w) with w = l % 32, h = l / 32 holds
// A(i0 + w, r0 + 16 h + s) and B(r0 + 16 h + s, j0 + w) for s = 0..15 and issues
// 16 products, the s-th pairing r0 + s (lanes h = 0) with r0 + 16 + s (lanes
// h = 1): every r of the slab is used once, in an order that is the same for
// both operands.  Two slabs are in flight from memory, and the slab after the
// current one is brought into that register layout while the current one is
// multiplied.
//
// How an operand's slab reaches the register layout depends on its memory layout
// (the kOp* forms below; A's is kOpRC): read along its unit-stride index with 16-byte
// loads and passed through a per-wave piece of LDS, or, when the 32-wide index is
// the unit-stride one, also with 4-byte loads straight into place.  Nothing assumes
// an alignment beyond 4 bytes.  No load sits under a branch: indices past the
// edge are clamped and the value is replaced by 0.
//
// With kslices > 1 the waves of a workgroup share tiles and add their accumulators
// through LDS.
//
// These are the products of few tiles with a long reduction; the others go by
// gemm_planes_tile below.
struct GemmArgs {
    const float *A;
    long long a_si, a_sr;
    const float *B;
    long long b_sr, b_sj;
    float *C; // C(i, j) at C[i * c_si + j]
    long long c_si;
    int M, N, K;
    const float *bias; // [N] added per column j, or null
    const float *mask; // same addressing as C: result multiplied by (mask > 0), or null
    int relu;          // max(x, 0) after the bias
    // A split product (a weight gradient): slice z of the reduction covers r in [z * k_per_split, ...) and goes to P[z][M][N + 1], its
    // last column the sums of A(i, r) over r; sgd_from_partials_kernel adds the slices in order.  Several of them share
    // one launch: the workgroups are dealt over the tiles of all.
    int splits, k_per_split;
    float *P;
    // Or B as integers times a scale: quantised weights.  B(r, j) = scale[j] * code (kOpRC) or scale[r] * code (kOpWide); the codes lie
    // in rows of c_pitch bfloat16 (16-byte aligned, filled up with zeros; along r or along j, as B's), the scales 16-byte aligned.
    // low (kOpRC), laid out as they are: what rounding scale * code to a float added to it, in units of the scale.
    const unsigned short *codes, *low;
    const float *scale;
    int c_pitch;
    int tile;        // 64 or 128
    int block_begin; // first workgroup of this problem in a group (filled by the launcher)
};

constexpr int kGemmMaxGroup = 16;
struct GemmGroup {
    GemmArgs p[kGemmMaxGroup];
    int count;
};

constexpr int kGemmThreads = 256;
constexpr int kGemmWaves = kGemmThreads / kWave;
constexpr int kGemmBK = 32;      // reduction slab
constexpr int kGemmPitch = 36;   // LDS row pitch of a turned slab (floats): rows stay 16-byte aligned

struct SlabRegs {
    float v[16];
};

// Wide-contiguous operand: element (wide, r) at base[wide + r * sr], clamped form (the last partial slab, tiles of operands narrower
// than 32).  Lane (h, w) reads r = r0 + 16 h + s, s = 0..15, of its own wide index, which the caller has clamped.
__device__ __forceinline__ void slab_load_direct(SlabRegs &x, const float *base, long long sr, int wide, int r0, int r_end, int h)
{
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int r = r0 + 16 * h + s;
        const int rc = min(r, r_end - 1);
        const float val = base[wide + (long long)rc * sr];
        x.v[s] = r < r_end ? val : 0.0f;
    }
}

// Reduction-contiguous operand: element (wide, r) at base[wide * sw + r], clamped form.  Step 1: lane l reads
// r = r0 + l % 32 of the tile's rows 2 it + l / 32, it = 0..15 (first_wide = the tile's first wide index,
// n_wide = the operand's extent in that index).
__device__ __forceinline__ void slab_load_along_r(SlabRegs &x, const float *base, long long sw, int first_wide,
                                                  int n_wide, int r0, int r_end, int lane)
{
    const int r = r0 + (lane & 31);
    const int rc = min(r, r_end - 1);
#pragma unroll
    for (int it = 0; it < 16; ++it) {
        const int wide = min(first_wide + 2 * it + (lane >> 5), n_wide - 1);
        const float val = base[(long long)wide * sw + rc];
        x.v[it] = r < r_end ? val : 0.0f;
    }
}

// step 2: through the wave's LDS piece into the product layout
__device__ __forceinline__ void slab_turn(SlabRegs &x, const SlabRegs &st, float *lds, int lane)
{
#pragma unroll
    for (int it = 0; it < 16; ++it) lds[(2 * it + (lane >> 5)) * kGemmPitch + (lane & 31)] = st.v[it];
    // (same wave: the LDS operations complete in order, no barrier needed)
    const float4 *row = reinterpret_cast<const float4 *>(lds + (lane & 31) * kGemmPitch + 16 * (lane >> 5));
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
        const float4 q = row[s4];
        x.v[4 * s4 + 0] = q.x, x.v[4 * s4 + 1] = q.y, x.v[4 * s4 + 2] = q.z, x.v[4 * s4 + 3] = q.w;
    }
}

// How the whole slabs of an operand are read (template parameters of the kernels):
//   kOpRC    the reduction index is the unit-stride one: 16-byte loads along it, turned through LDS
//   kOpWide  the 32-wide index is the unit-stride one: 16-byte loads along it, through LDS: only for tiles whose 32 wide
//            indices all exist
// The last partial slab, and kOpWide tiles of operands narrower than 32, take the clamped 4-byte path instead.
enum { kOpRC = 0, kOpWide = 1 };

// four floats that are only known to start on a 4-byte boundary (a 16-byte global load needs no more)
typedef float Float4Dw __attribute__((ext_vector_type(4), aligned(4)));

// `first_wide`: the tile's first wide index, `n_wide`: the operand's extent in it (kOpRC reads row n_wide - 1 in
// place of the rows past it; kOpWide needs all 32 to exist)
template <int MODE>
__device__ __forceinline__ void slab_fetch_fast(SlabRegs &st, const float *base, long long sw, long long sr,
                                                int first_wide, int n_wide, int r0, int lane)
{
    // lane l reads four consecutive floats (l % 8) * 4 .. + 3 of lines l / 8 + 8 it, it = 0..3; a line is a
    // row of the operand (kOpRC: along r) or one reduction index (kOpWide: along the wide index)
    const int line = lane >> 3, c4 = (lane & 7) * 4;
    if (MODE == kOpRC) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = min(first_wide + line + 8 * it, n_wide - 1);
            const Float4Dw q = *reinterpret_cast<const Float4Dw *>(base + (long long)row * sw + (r0 + c4));
            st.v[4 * it + 0] = q.x, st.v[4 * it + 1] = q.y, st.v[4 * it + 2] = q.z, st.v[4 * it + 3] = q.w;
        }
    } else {
        const float *p = base + (long long)(r0 + line) * sr + (first_wide + c4);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const Float4Dw q = *reinterpret_cast<const Float4Dw *>(p + (long long)(8 * it) * sr);
            st.v[4 * it + 0] = q.x, st.v[4 * it + 1] = q.y, st.v[4 * it + 2] = q.z, st.v[4 * it + 3] = q.w;
        }
    }
}

// staging registers of a whole slab -> product layout
template <int MODE>
__device__ __forceinline__ void slab_settle_fast(SlabRegs &x, const SlabRegs &st, float *lds, int lane)
{
    const int line = lane >> 3, c4 = (lane & 7) * 4;
#pragma unroll
    for (int it = 0; it < 4; ++it)
        *reinterpret_cast<float4 *>(lds + (line + 8 * it) * kGemmPitch + c4) =
            make_float4(st.v[4 * it + 0], st.v[4 * it + 1], st.v[4 * it + 2], st.v[4 * it + 3]);
    // (same wave: the LDS operations complete in order, no barrier needed)
    const int w = lane & 31, h = lane >> 5;
    if (MODE == kOpRC) { // LDS holds [wide][r]: 16 consecutive r of my wide index
        const float4 *row = reinterpret_cast<const float4 *>(lds + w * kGemmPitch + 16 * h);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const float4 q = row[s4];
            x.v[4 * s4 + 0] = q.x, x.v[4 * s4 + 1] = q.y, x.v[4 * s4 + 2] = q.z, x.v[4 * s4 + 3] = q.w;
        }
    } else { // LDS holds [r][wide]: my wide index of 16 consecutive r
#pragma unroll
        for (int s = 0; s < 16; ++s) x.v[s] = lds[(16 * h + s) * kGemmPitch + w];
    }
}

// LDS of the workgroup: per wave, the pieces through which A and B are turned
constexpr int kGemmTurnFloats = 32 * kGemmPitch;
constexpr int kGemmLdsFloats = kGemmWaves * 2 * kGemmTurnFloats;

// the tile `local` (and, with ks > 1, the slice wave % ks of its reduction) of problem g, by one wave
template <int B_MODE>
__device__ __forceinline__ void gemm_wave_tile(const GemmArgs &g, int local, bool live, int ks, int wave, int lane,
                                               float *lds_all)
{
    constexpr bool B_RC = B_MODE == kOpRC;
    const int kz = wave & (ks - 1);
    const int tiles_j = (g.N + 31) / 32;
    const int i_first = (local / tiles_j) * 32, j_first = (local % tiles_j) * 32; // first row / column this tile stores
    // this wave's part of the reduction
    const int k_per_wave = ks > 1 ? ((g.K + 2 * kGemmBK * ks - 1) / (2 * kGemmBK * ks)) * (2 * kGemmBK) : g.K;
    const int r_begin = kz * k_per_wave;
    const int r_end = live ? min(g.K, r_begin + k_per_wave) : r_begin;
    const int w = lane & 31, h = lane >> 5;

    // The last tile of a dimension that is not a multiple of 32 is moved back so that it ends at the edge: it
    // recomputes a few rows / columns of its neighbour, stores only its own, and reads whole slabs like any
    // other.  Operands narrower than 32 cannot: their tiles re-read the last row / column (clamped indices)
    // and those results are not stored.
    const int i0 = (i_first + 32 > g.M && g.M >= 32) ? g.M - 32 : i_first;
    const int j0 = (j_first + 32 > g.N && g.N >= 32) ? g.N - 32 : j_first;
    // whole slabs can be read the fast way (kOpWide: only if the tile's 32 columns all exist)
    const bool whole = B_RC || j0 + 32 <= g.N;
    const int jb = min(j0 + w, g.N - 1);
    float *lds_a = lds_all + wave * 2 * kGemmTurnFloats, *lds_b = lds_a + kGemmTurnFloats;
    // (requested now, used in the epilogue)
    const float bias_j = g.bias ? g.bias[min(j0 + w, g.N - 1)] : 0.0f;
    // ... and so is the mask of this lane's 16 outputs (rows and columns past the edge re-read the last ones)
    float mask_v[16];
    if (g.mask) {
        const int mj = min(j0 + w, g.N - 1);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            mask_v[v] = g.mask[(long long)min(i0 + 8 * (v >> 2) + 4 * h + (v & 3), g.M - 1) * g.c_si + mj];
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) mask_v[v] = 1.0f;
    }

    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    // Two slabs are in flight while a third is multiplied: sa[q] / sb[q] receive slab n with n % 2 == q as it
    // comes from memory, a / b hold the current slab in product layout.
    SlabRegs a, b, sa[2], sb[2];
    auto fetch_safe = [&](int q, int r0) {
        slab_load_along_r(sa[q], g.A, g.a_si, i0, g.M, r0, r_end, lane);
        if (B_RC)
            slab_load_along_r(sb[q], g.B, g.b_sj, j0, g.N, r0, r_end, lane);
        else
            slab_load_direct(sb[q], g.B, g.b_sr, jb, r0, r_end, h);
    };
    auto fetch_fast = [&](int q, int r0) { // whole tile, whole slab
        slab_fetch_fast<kOpRC>(sa[q], g.A, g.a_si, g.a_sr, i0, g.M, r0, lane);
        slab_fetch_fast<B_MODE>(sb[q], g.B, g.b_sj, g.b_sr, j0, g.N, r0, lane);
    };
    auto settle_fast = [&](int q) {
        slab_settle_fast<kOpRC>(a, sa[q], lds_a, lane);
        slab_settle_fast<B_MODE>(b, sb[q], lds_b, lane);
    };
    auto settle = [&](int q) { // staging registers of the clamped path -> product layout
        slab_turn(a, sa[q], lds_a, lane);
        if (B_RC)
            slab_turn(b, sb[q], lds_b, lane);
        else
            b = sb[q];
    };
    auto products = [&]() {
#pragma unroll
        for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[s], b.v[s], acc, 0, 0, 0);
    };

    // Pairs of whole slabs of a whole tile.  The loop bodies below have no branch and every fetch is
    // unconditional, so that the loads in flight are the same, in number and order, on entry and on the way
    // round: only then does the compiler wait for exactly the slab it needs.  (A fetch past the fast part
    // re-reads its last pair of slabs: harmless.)
    int r0 = r_begin;
    const int r_pairs = whole ? r_begin + (r_end - r_begin) / (2 * kGemmBK) * (2 * kGemmBK) : r_begin;
    if (r0 < r_pairs) {
        const int r_last = r_pairs - 2 * kGemmBK;
        // a2 / b2: the slab after the current one is brought into product layout while the current one is
        // multiplied (the matrix core runs on its own once a product is issued; the LDS traffic of the turn
        // goes out in its shadow)
        SlabRegs a2, b2;
        fetch_fast(0, r0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_fast(1, r0 + kGemmBK);
        __builtin_amdgcn_sched_barrier(0);
        settle_fast(0);
        __builtin_amdgcn_sched_barrier(0);
        for (; r0 < r_pairs; r0 += 2 * kGemmBK) {
            const int rn = min(r0 + 2 * kGemmBK, r_last);
            fetch_fast(0, rn);
            __builtin_amdgcn_sched_barrier(0);
            slab_settle_fast<kOpRC>(a2, sa[1], lds_a, lane);
            slab_settle_fast<B_MODE>(b2, sb[1], lds_b, lane);
            products();
            __builtin_amdgcn_sched_barrier(0);
            fetch_fast(1, rn + kGemmBK);
            __builtin_amdgcn_sched_barrier(0);
            slab_settle_fast<kOpRC>(a, sa[0], lds_a, lane);
            slab_settle_fast<B_MODE>(b, sb[0], lds_b, lane);
#pragma unroll
            for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a2.v[s], b2.v[s], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // what is left: at most one whole and one partial slab of a whole tile, or everything of a clamped tile
    // (past the end: clamped addresses, zeros, and a product that adds nothing)
    if (r0 < r_end) {
        fetch_safe(0, r0);
        fetch_safe(1, r0 + kGemmBK);
        for (; r0 < r_end; r0 += 2 * kGemmBK) {
            settle(0);
            fetch_safe(0, r0 + 2 * kGemmBK);
            products();
            settle(1);
            fetch_safe(1, r0 + 3 * kGemmBK);
            products();
        }
    }

    // the slices of a tile meet: slice 0 adds the others' accumulators in order and goes on alone
    if (ks > 1) {
        float *mine = lds_a;
        if (kz > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) mine[v * kWave + lane] = acc[v];
        }
        __syncthreads();
        if (kz > 0 || !live) return;
        for (int k = 1; k < ks; ++k) {
            const float *other = lds_a + k * 2 * kGemmTurnFloats;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += other[v * kWave + lane];
        }
    }

    // accumulator layout: lane l holds column j = l % 32 and rows 8*(v/4) + 4*(l/32) + v%4, v = 0..15
    const int j = j0 + w;
    if (j < j_first || j >= g.N) return; // (a moved tile stores only its own columns and rows)
    const float bj = bias_j;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int i = i0 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (i < i_first || i >= g.M) continue;
        float x = acc[v] + bj;
        if (g.relu) x = fmaxf(x, 0.0f);
        const long long off = (long long)i * g.c_si + j;
        x = mask_v[v] > 0.0f ? x : 0.0f;
        g.C[off] = x;
    }
}

// ---- products of many tiles: three bfloat16 planes per operand ---------------------------------------------------
// The fp32 matrix instructions run at a sixteenth of the bfloat16 ones' rate.  A float of 2^-103 or more is exactly the sum of a
// bfloat16, the bfloat16 nearest to what that leaves, and a third one's rest (three planes of 8 significant bits each; of smaller floats
// the third plane may be subnormal or nothing).  Of the nine products of two such sums the six largest are taken, each exact, and
// added up in fp32 by the matrix cores, 16 of the reduction at a time: 6 x 32 matrix-core cycles for what takes 8 x 64 in fp32.  The
// three left out are 2^-24 of a product at most, half a rounding of fp32, and far less on average.  The products of the first
// planes have an accumulator of their own, which is rounded once per 16 of the reduction: measured on normal random data, the
// error against 64 bits is a third of what the fp32 instructions' is (8192x512x512: 1.3e-7 and 4.05e-7 of the 2-norm).
//
// A workgroup of 8 waves has a tile of BM x BN; the reduction goes by slabs of BK.  The threads read a slab as floats (two slabs
// ahead), split them once for the whole workgroup and leave the planes in LDS, 8 consecutive r of a row to a 16-byte
// vector, in one of two buffers while the waves multiply from the other: one barrier per slab.  Two waves to a SIMD, as one alone
// is bound by the 5.5 cycles that each of its instructions takes to issue: their splitting and LDS traffic goes out beside the
// other's products.
//
// Not finite: an infinity's planes are infinity and NaN, and a float next to the largest rounds up to one.  A wave with a sum that is
// not finite adds its part of the tile up again in plain fp32, on the fp32 matrix instructions with operands straight from memory,
// and the lanes concerned take that, so that infinities and NaN come out as they do there.  It costs only what has them: one sample, its tiles; a
// model that has diverged altogether, the dense step of the Terabyte shape, 8192 samples, all NaN: 768 us (finite: 366); every such lane by
// itself, a float at a time: 2389; the fp32 matrix instructions alone: 636.
typedef __bf16 Bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 Bf16x8 __attribute__((ext_vector_type(8)));
typedef float Float2 __attribute__((ext_vector_type(2)));

constexpr int kPlanes = 3;
constexpr int kPlaneThreads = 512, kPlaneWaves = kPlaneThreads / kWave;

// The shape of a workgroup's work.  KH: the parts of a slab's reduction that go to different waves (their sums meet at the end);
// the waves of a part lie 2 x (4 / KH) over the tile.
// BP: planes of B.
template <int BM_, int BN_, int BK_, int KH_, int BP_ = kPlanes>
struct PlaneTile {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, KH = KH_, BP = BP_;
    static constexpr int WN = kPlaneWaves / KH / 2, FM = BM / 64; // a wave's product: FM x 1 tiles of 32 x 32
    static_assert(BN == 32 * WN && BK / 16 % KH == 0, "a wave has one tile of columns");
    // bytes of LDS between the groups of 8 r of a plane (a write's 8 lanes at a time are BK / 8 groups of as many rows as that
    // takes), of a plane, of a slab
    static constexpr int pitch(int rows) { return rows * 16 + (BK == 32 ? 32 : 16); }
    static constexpr int plane(int rows) { return pitch(rows) * (BK / 8); }
    static constexpr int kRoom = (KH == 1 ? 64 : BM) * (BN + 4) * 4; // the tile leaves through it
    static constexpr int kPlaneBytes = kPlanes * plane(BM) + BP * plane(BN), kSlabBytes = kPlaneBytes > kRoom ? kPlaneBytes : kRoom;
};
using PlaneTile128 = PlaneTile<128, 128, 32, 1>;
using PlaneTile128x64 = PlaneTile<128, 64, 64, 2>;
using PlaneTile64 = PlaneTile<64, 64, 64, 2>;

// a pair of floats -> a pair of bfloat16 (round to nearest even), and what that leaves of them (exact)
__device__ __forceinline__ unsigned split_pair(float &x0, float &x1)
{
    const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector((Float2){x0, x1}, Bf16x2));
    x0 -= __uint_as_float(h << 16);
    x1 -= __uint_as_float(h & 0xFFFF0000u);
    return h;
}

// The tiles of products with quantised weights, by B's mode.
constexpr int kCodePlanes(int mode) { return mode == kOpRC ? 2 : 1; }
template <int MODE> using CodeTile128 = PlaneTile<128, 128, 32, 1, kCodePlanes(MODE)>;
template <int MODE> using CodeTile128x64 = PlaneTile<128, 64, 64, 2, kCodePlanes(MODE)>;
template <int MODE> using CodeTile64 = PlaneTile<64, 64, 64, 2, kCodePlanes(MODE)>;

// The float (or what T is) `bytes` behind a wave-uniform address.  The offset is hidden from the loop around it, or the compiler would add
// the two once before the loop and then the slab's address to that 64-bit sum beside every load: an instruction each, and twice the registers.
template <typename T>
__device__ __forceinline__ T load_at(const void *base, unsigned &bytes)
{
    asm("" : "+v"(bytes));
    return *reinterpret_cast<const T *>(static_cast<const char *>(base) + bytes);
}

// One operand's part of a tile, as one thread reads it: ROWS wide indices, 8 consecutive r of each slab in an item.
// kOpRC: the reduction index is the unit-stride one; kOpWide: the wide one is.
// SCALED (kOpRC): every element is multiplied by scale[r].
template <int MODE, int ROWS, int BK, bool SCALED = false>
struct PlaneOperand {
    static constexpr int kGroups = BK / 8, kItems = ROWS * kGroups / kPlaneThreads;
    static constexpr int kRowsPerItem = kPlaneThreads / kGroups, kGroupsPerItem = kPlaneThreads / ROWS; // kOpRC; kOpWide
    const float *tile;     // the tile's first wide index, r = 0 (wave-uniform)
    const float *slabs;    // where fetch() starts from: there, or where the operand starts
    long long sr;          // kOpWide: between lines
    // In bytes (a 32-bit byte offset beside a scalar address takes no instruction of its own: 32 of 134 vector instructions a slab of the
    // weight gradients).  kOpRC: of the items' rows; kOpWide: of the first item's lines (kept, as adding a line's length 8 times
    // costs two instructions beside each load)
    unsigned off[MODE == kOpRC ? kItems : 8];
    int row, kg;           // of the first item
    float v[2][kItems][8]; // two slabs on their way
    const float *scale;    // from this thread's first r on (whole slabs; otherwise of no meaning)
    float sv[2][SCALED ? 8 : 1];

    // `first`: the tile's first wide index; those past `count` re-read the last.  `whole`: the reduction has a whole slab; otherwise
    // nobody looks at what fetch() reads, and it reads the operand's first 8 floats (kOpRC; it has as many: host) or its first line.
    __device__ __forceinline__ void init(const float *base, long long sw, long long sr_, int first, int count, bool whole, int tid)
    {
        if (MODE == kOpRC) {
            sr = sw;
            row = tid / kGroups, kg = tid % kGroups;
            tile = base + (long long)first * sw;
            slabs = whole ? tile : base;
#pragma unroll
            for (int c = 0; c < kItems; ++c) {
                off[c] = ((unsigned)(min(first + row + c * kRowsPerItem, count - 1) - first) * (unsigned)sw + 8u * kg) * 4u;
                if (!whole) off[c] = 0u;
            }
        } else {
            sr = whole ? sr_ : 0;
            row = tid % ROWS, kg = tid / ROWS;
            tile = slabs = base + first;
#pragma unroll
            for (int k = 0; k < 8; ++k) off[k] = ((8u * kg + k) * (unsigned)sr + (unsigned)min(row, count - 1 - first)) * 4u;
        }
    }
    __device__ __forceinline__ void init_scale(const float *s, bool whole) { scale = whole ? s + 8 * kg : s; }
    // a whole slab
    __device__ __forceinline__ void fetch(int q, int r0)
    {
#pragma unroll
        for (int c = 0; c < kItems; ++c) {
            if (MODE == kOpRC) {
                const Float4Dw lo = load_at<Float4Dw>(slabs + r0, off[c]), hi = load_at<Float4Dw>(slabs + r0 + 4, off[c]);
#pragma unroll
                for (int k = 0; k < 4; ++k) v[q][c][k] = lo[k], v[q][c][4 + k] = hi[k];
            } else {
                const float *p = slabs + (long long)(r0 + 8 * c * kGroupsPerItem) * sr;
#pragma unroll
                for (int k = 0; k < 8; ++k) v[q][c][k] = load_at<float>(p, off[k]);
            }
        }
        if constexpr (SCALED) {
            const float4 lo = *reinterpret_cast<const float4 *>(scale + r0), hi = *reinterpret_cast<const float4 *>(scale + r0 + 4);
            sv[q][0] = lo.x, sv[q][1] = lo.y, sv[q][2] = lo.z, sv[q][3] = lo.w;
            sv[q][4] = hi.x, sv[q][5] = hi.y, sv[q][6] = hi.z, sv[q][7] = hi.w;
        }
    }
    // the partial slab: r past `r_end` re-reads the one before it and counts as 0
    __device__ __forceinline__ void fetch_tail(int q, int r0, int r_end, long long line, int first, int count, bool whole_slabs)
    {
#pragma unroll
        for (int c = 0; c < kItems; ++c) {
            const int r_item = r0 + 8 * (kg + (MODE == kOpRC ? 0 : c * kGroupsPerItem));
            const int at = min(first + row + (MODE == kOpRC ? c * kRowsPerItem : 0), count - 1) - first;
            const float *p = tile + (MODE == kOpRC ? at * sr : at);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int r = r_item + k, rc = min(r, r_end - 1);
                const float t = p[MODE == kOpRC ? rc : rc * line];
                v[q][c][k] = r < r_end ? t : 0.0f;
                if constexpr (SCALED) sv[q][k] = scale[min(r, r_end - 1) - (whole_slabs ? 8 * kg : 0)];
            }
        }
    }
    // split and leave in LDS
    __device__ __forceinline__ void put(int q, char *lds)
    {
        constexpr int kPitch = ROWS * 16 + (BK == 32 ? 32 : 16);
#pragma unroll
        for (int c = 0; c < kItems; ++c) {
            char *at = lds + (kg + (MODE == kOpRC ? 0 : c * kGroupsPerItem)) * kPitch + (row + (MODE == kOpRC ? c * kRowsPerItem : 0)) * 16;
            float t[8], low[8]; // low: what a product with the scale lost when it was rounded
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                t[k] = SCALED ? v[q][c][k] * sv[q][k] : v[q][c][k];
                if (SCALED) low[k] = __builtin_fmaf(v[q][c][k], sv[q][k], -t[k]);
            }
#pragma unroll
            for (int p = 0; p < kPlanes; ++p) {
                uint4 o;
                o.x = split_pair(t[0], t[1]), o.y = split_pair(t[2], t[3]), o.z = split_pair(t[4], t[5]), o.w = split_pair(t[6], t[7]);
                if (SCALED && p == 0)
#pragma unroll
                    for (int k = 0; k < 8; ++k) t[k] += low[k];
                *reinterpret_cast<uint4 *>(at + p * kPitch * kGroups) = o;
            }
        }
    }
    __device__ __forceinline__ float sum(int q) const // (kOpWide: of one row)
    {
        float s = 0.0f;
#pragma unroll
        for (int c = 0; c < kItems; ++c)
            s += ((v[q][c][0] + v[q][c][1]) + (v[q][c][2] + v[q][c][3])) + ((v[q][c][4] + v[q][c][5]) + (v[q][c][6] + v[q][c][7]));
        return s;
    }
};

// The same of an operand whose planes lie in memory as they are (GemmArgs::codes and low).
template <int MODE, int ROWS, int BK>
struct CodeOperand {
    static constexpr int kGroups = BK / 8, kItems = ROWS * kGroups / kPlaneThreads;
    static constexpr int kRowsPerItem = kPlaneThreads / kGroups, kGroupsPerItem = kPlaneThreads / ROWS; // kOpRC; kOpWide
    const unsigned short *slabs; // the tile's first wide index, r = 0
    const unsigned short *low;   // kOpRC: the second plane's
    long long pitch;             // kOpWide: between lines
    unsigned off[MODE == kOpRC ? kItems : 1]; // bytes; kOpRC: of the items' rows; kOpWide: of the first line's row
    int row, kg;
    unsigned v[2][kItems][8]; // kOpRC: two planes; kOpWide: a code each

    // `whole`: the reduction has a whole slab; otherwise fetch() reads the first line over and over (kOpWide), and nobody looks at it
    __device__ __forceinline__ void init(const unsigned short *base, const unsigned short *base_low, int pitch_, int first, int count, bool whole, int tid)
    {
        pitch = pitch_;
        if (MODE == kOpRC) {
            row = tid / kGroups, kg = tid % kGroups;
            slabs = base + (long long)first * pitch;
            low = base_low + (long long)first * pitch;
#pragma unroll
            for (int c = 0; c < kItems; ++c) off[c] = ((unsigned)(min(first + row + c * kRowsPerItem, count - 1) - first) * (unsigned)pitch + 8u * kg) * 2u;
        } else {
            row = tid % ROWS, kg = tid / ROWS;
            slabs = base + first;
            if (!whole) pitch = 0;
            off[0] = (8u * kg * (unsigned)pitch + (unsigned)min(row, count - 1 - first)) * 2u;
        }
    }
    __device__ __forceinline__ void fetch(int q, int r0)
    {
#pragma unroll
        for (int c = 0; c < kItems; ++c) {
            if constexpr (MODE == kOpRC) {
                const uint4 t = load_at<uint4>(slabs + r0, off[c]), u = load_at<uint4>(low + r0, off[c]);
                v[q][c][0] = t.x, v[q][c][1] = t.y, v[q][c][2] = t.z, v[q][c][3] = t.w;
                v[q][c][4] = u.x, v[q][c][5] = u.y, v[q][c][6] = u.z, v[q][c][7] = u.w;
            } else {
                const unsigned short *line = slabs + (long long)(r0 + 8 * c * kGroupsPerItem) * pitch;
#pragma unroll
                for (int k = 0; k < 8; ++k, line += pitch) v[q][c][k] = load_at<unsigned short>(line, off[0]);
            }
        }
    }
    // the partial slab: kOpRC reads on in the row's zeros, kOpWide the last line again (A has zeros there)
    __device__ __forceinline__ void fetch_tail(int q, int r0, int r_end, int line, int first, int count)
    {
        if constexpr (MODE == kOpRC) {
            fetch(q, r0);
        } else {
#pragma unroll
            for (int c = 0; c < kItems; ++c)
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    v[q][c][k] = slabs[(unsigned)min(r0 + 8 * (kg + c * kGroupsPerItem) + k, r_end - 1) * (unsigned)line + (unsigned)min(row, count - 1 - first)];
        }
    }
    __device__ __forceinline__ void put(int q, char *lds)
    {
        constexpr int kPitch = ROWS * 16 + (BK == 32 ? 32 : 16);
#pragma unroll
        for (int c = 0; c < kItems; ++c) {
            const unsigned(&x)[8] = v[q][c];
            char *at = lds + (kg + (MODE == kOpRC ? 0 : c * kGroupsPerItem)) * kPitch + (row + (MODE == kOpRC ? c * kRowsPerItem : 0)) * 16;
            if constexpr (MODE == kOpRC) {
                *reinterpret_cast<uint4 *>(at) = make_uint4(x[0], x[1], x[2], x[3]);
                *reinterpret_cast<uint4 *>(at + kPitch * kGroups) = make_uint4(x[4], x[5], x[6], x[7]);
            } else {
                *reinterpret_cast<uint4 *>(at) = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16));
            }
        }
    }
};

// Where a request past the last slab of a reduction of k starts.  Codes and scales are read 16 bytes at a time from addresses that
// are multiples of that, eight r by eight; floats from any.
constexpr __host__ __device__ int last_slab(int k, int bk, bool codes)
{
    const int r = k > bk ? k - bk : 0;
    return codes ? r / 8 * 8 : r;
}
static_assert(last_slab(415, 32, true) == 376 && last_slab(367, 64, true) == 296 && last_slab(33, 32, true) == 0 && last_slab(512, 32, true) == 480 &&
              last_slab(415, 32, false) == 383 && last_slab(20, 32, true) == 0, "inside the reduction, and of a whole vector");

// Tile `local` of product g (one slice of its reduction, and the rows' sums beside it, if SPLIT).  lds0, lds1: kSlabBytes each.
template <typename TILE, int A_MODE, int B_MODE, bool SPLIT>
__device__ __forceinline__ void gemm_planes_tile(const GemmArgs &g, int local, char *lds0, char *lds1)
{
    constexpr int BM = TILE::BM, BN = TILE::BN, BK = TILE::BK, KH = TILE::KH, FM = TILE::FM, WN = TILE::WN;
    constexpr int kA = TILE::plane(BM), kB = TILE::plane(BN), kPitchA = TILE::pitch(BM), kPitchB = TILE::pitch(BN);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int w = lane & 31, h = lane >> 5, kh = wave / (2 * WN), wm = wave & 1, wn = (wave >> 1) % WN;
    const int tiles_j = (g.N + BN - 1) / BN, tiles_i = (g.M + BM - 1) / BM;
    const int z = SPLIT ? local / (tiles_i * tiles_j) : 0;
    local -= z * tiles_i * tiles_j;
    const int i0 = local / tiles_j * BM, j0 = local % tiles_j * BN;
    const int r_begin = SPLIT ? min(z * g.k_per_split, g.K) : 0, r_end = SPLIT ? min(r_begin + g.k_per_split, g.K) : g.K;

    constexpr int BP = TILE::BP;
    constexpr bool CODES = BP < kPlanes;
    static_assert(!CODES || (A_MODE == kOpRC && !SPLIT), "quantised weights");
    PlaneOperand<A_MODE, BM, BK, CODES && B_MODE == kOpWide> a;
    std::conditional_t<CODES, CodeOperand<B_MODE, BN, BK>, PlaneOperand<B_MODE, BN, BK>> b;
    a.init(g.A, g.a_si, g.a_sr, i0, g.M, g.K >= BK, tid);
    float col_scale = 1.0f;
    if constexpr (CODES) {
        b.init(g.codes, g.low, g.c_pitch, j0, g.N, g.K >= BK, tid);
        if (B_MODE == kOpWide) a.init_scale(g.scale, g.K >= BK);
        else col_scale = g.scale[min(j0 + 32 * wn + w, g.N - 1)];
    } else {
        b.init(g.B, g.b_sj, g.b_sr, j0, g.N, g.K >= BK, tid);
    }
    floatx16 acc[FM], rest[FM]; // the first planes' products, and the smaller ones
#pragma unroll
    for (int m = 0; m < FM; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[m][v] = rest[m][v] = 0.0f;
    float row_sum = 0.0f;

    // The slabs in their order: the partial one first, if there is one (it is read in another way, and the loop below has no
    // branch).  Requests past the last slab read some slab of the operands that exists, and nobody looks at it.
    const int whole = (r_end - r_begin) / BK, tail = r_end - r_begin - whole * BK;
    const int slabs = whole + (tail > 0), r_slab = r_begin - (tail > 0 ? BK : 0), r_last = last_slab(g.K, BK, CODES);
    auto fetch = [&](int q, int s) {
        const int r0 = min(r_slab + s * BK, r_last);
        a.fetch(q, r0);
        b.fetch(q, r0);
    };
    auto put = [&](int q, int s, char *lds) {
        a.put(q, lds);
        b.put(q, lds + kPlanes * kA);
        if (SPLIT) row_sum += __uint_as_float(__float_as_uint(a.sum(q)) & (unsigned)((s - slabs) >> 31)); // (no branch)
    };
    // a slab's planes, as the matrix cores take them
    constexpr int kSteps = BK / 16 / KH;
    struct Fragments {
        Bf16x8 a[kSteps][kPlanes][FM], b[kSteps][BP];
    };
    auto read = [&](Fragments &f, const char *lds) {
        const char *la = lds + (2 * kSteps * kh + h) * kPitchA + (32 * FM * wm + w) * 16;
        const char *lb = lds + kPlanes * kA + (2 * kSteps * kh + h) * kPitchB + (32 * wn + w) * 16;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int p = kPlanes - 1; p >= 0; --p) {
#pragma unroll
                for (int m = 0; m < FM; ++m)
                    f.a[s][p][m] = *reinterpret_cast<const Bf16x8 *>(la + p * kA + 2 * s * kPitchA + m * 32 * 16);
                if (p < BP) f.b[s][p] = *reinterpret_cast<const Bf16x8 *>(lb + p * kB + 2 * s * kPitchB);
            }
    };
    auto products = [&](const Fragments &f) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int sum = kPlanes - 1; sum >= 0; --sum)
#pragma unroll
                for (int p = sum < BP ? 0 : sum + 1 - BP; p <= sum; ++p)
#pragma unroll
                    for (int m = 0; m < FM; ++m) {
                        if (CODES && p > 0 && sum > p) continue; // (the rounding of a weight by A's first plane only)
                        floatx16 &to = sum > 0 ? rest[m] : acc[m];
                        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[s][p][m], f.b[s][sum - p], to, 0, 0, 0);
                    }
    };
    if (slabs > 0) { // (the whole workgroup, or none of it)
        if (tail > 0) {
            a.fetch_tail(0, r_end - tail, r_end, g.a_sr, i0, g.M, g.K >= BK);
            if constexpr (CODES) b.fetch_tail(0, r_end - tail, r_end, g.c_pitch, j0, g.N);
            else b.fetch_tail(0, r_end - tail, r_end, g.b_sr, j0, g.N, g.K >= BK);
        } else {
            fetch(0, 0);
        }
        fetch(1, 1);
        put(0, 0, lds0);
        fetch(0, 2);
        __syncthreads();
        // while slab s is multiplied, s + 1 is split and written to LDS, s + 2 and s + 3 are on their way
        for (int s = 0; s < slabs; s += 2) {
            Fragments f;
            read(f, lds0);
            put(1, s + 1, lds1);
            fetch(1, s + 3);
            products(f);
            __syncthreads();
            if (s + 1 < slabs) {
                read(f, lds1);
                put(0, s + 2, lds0);
                fetch(0, s + 4);
                products(f);
                __syncthreads();
            }
        }
    }

    // lane l holds column l % 32 of its products and rows 8 (v / 4) + 4 (l / 32) + v % 4
    const int i_lane = 32 * FM * wm + 4 * h, j_lane = 32 * wn + w;
    float finite = 0.0f;
#pragma unroll
    for (int m = 0; m < FM; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (CODES && B_MODE == kOpRC) acc[m][v] = __builtin_fmaf(acc[m][v], col_scale, rest[m][v] * col_scale); // (a rounding, as without the scale)
            else acc[m][v] += rest[m][v];
            finite = __builtin_fmaf(acc[m][v], 0.0f, finite);
        }
    if (__builtin_expect(__any(finite != 0.0f), 0)) { // (NaN: the whole wave's part again, and the lanes concerned take it)
#pragma unroll
        for (int m = 0; m < FM; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) rest[m][v] = 0.0f;
        const float *pb = g.B + (long long)min(j0 + j_lane, g.N - 1) * g.b_sj;
        const float *pa[FM];
#pragma unroll
        for (int m = 0; m < FM; ++m) pa[m] = g.A + (long long)min(i0 + 32 * (FM * wm + m) + w, g.M - 1) * g.a_si;
        constexpr int kPart = BK / KH;
#pragma unroll 1
        for (int r0 = r_begin + kPart * kh; r0 < r_end; r0 += BK) { // the wave's part of each slab
            // lane (h, w): r0 + h kPart / 2 .. of its row and its column, 0 past the end
            float av[FM][kPart / 2], bv[kPart / 2];
            auto load = [&](float *to, const float *p, long long line, bool along_r) {
                const int r1 = r0 + kPart / 2 * h;
                if (along_r && r0 + kPart <= r_end) {
#pragma unroll
                    for (int k = 0; k < kPart / 2; k += 4) {
                        const Float4Dw t = *reinterpret_cast<const Float4Dw *>(p + r1 + k);
                        to[k] = t[0], to[k + 1] = t[1], to[k + 2] = t[2], to[k + 3] = t[3];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kPart / 2; ++k) {
                        const float t = p[min(r1 + k, r_end - 1) * line];
                        to[k] = r1 + k < r_end ? t : 0.0f;
                    }
                }
            };
            load(bv, pb, g.b_sr, B_MODE == kOpRC);
#pragma unroll
            for (int m = 0; m < FM; ++m) load(av[m], pa[m], g.a_sr, A_MODE == kOpRC);
#pragma unroll
            for (int k = 0; k < kPart / 2; ++k)
#pragma unroll
                for (int m = 0; m < FM; ++m) rest[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[m][k], bv[k], rest[m], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < FM; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][v] = finite != 0.0f ? rest[m][v] : acc[m][v];
    }

    // The tile goes through LDS: 16 bytes to a thread, and a loop of little code (a launch fetches every line of its code anew).
    // KH = 1: rows 0..63 lie in lds0, the others in lds1; KH = 2: either has a part's sums.
    constexpr int kPitch = BN + 4, kCols = BN / 4, kRows = kPlaneThreads / kCols;
    static_assert(KH == 2 || BM == 128, "the tile fits the slabs' room");
    float *tile0 = reinterpret_cast<float *>(lds0), *tile1 = reinterpret_cast<float *>(lds1); // (every read is behind a barrier)
    {
        float *at = ((KH == 1 ? wm : kh) ? tile1 : tile0) + (KH == 1 ? 4 * h : i_lane) * kPitch + j_lane;
#pragma unroll
        for (int m = 0; m < FM; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) at[(32 * m + 8 * (v >> 2) + (v & 3)) * kPitch] = acc[m][v];
    }
    const int col = tid % kCols * 4, j = j0 + col, row = tid / kCols;
    float *out = SPLIT ? g.P + (long long)z * g.M * (g.N + 1) : g.C;
    const long long pitch = SPLIT ? g.N + 1 : g.c_si;
    const bool full = j + 4 <= g.N;
    float bias[4] = {};
    if (!SPLIT && g.bias) {
#pragma unroll
        for (int n = 0; n < 4; ++n) bias[n] = g.bias[min(j + n, g.N - 1)];
    }
    __syncthreads();
#pragma unroll 4
    for (int k = 0; k < BM / kRows; ++k) {
        const int r = row + k * kRows, i = i0 + r;
        const long long at = (long long)min(i, g.M - 1) * pitch + j;
        float4 t = *reinterpret_cast<const float4 *>((KH == 1 && r >= 64 ? tile1 - 64 * kPitch : tile0) + r * kPitch + col);
        if (KH == 2) {
            const float4 u = *reinterpret_cast<const float4 *>(tile1 + r * kPitch + col);
            t.x += u.x, t.y += u.y, t.z += u.z, t.w += u.w;
        }
        float x[4] = {t.x, t.y, t.z, t.w};
        if (!SPLIT) {
            Float4Dw mask = {1.0f, 1.0f, 1.0f, 1.0f};
            if (g.mask) { // (one load, except at the last columns: those past the edge are not stored)
                if (full)
                    mask = *reinterpret_cast<const Float4Dw *>(g.mask + at);
                else
#pragma unroll
                    for (int n = 0; n < 4; ++n) mask[n] = g.mask[at - j + min(j + n, g.N - 1)];
            }
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                x[n] += bias[n];
                if (g.relu) x[n] = fmaxf(x[n], 0.0f);
                x[n] = mask[n] > 0.0f ? x[n] : 0.0f;
            }
        }
        if (i < g.M) {
            if (full)
                *reinterpret_cast<Float4Dw *>(out + at) = (Float4Dw){x[0], x[1], x[2], x[3]};
            else
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    if (j + n < g.N) out[at + n] = x[n];
        }
    }
    if (SPLIT) { // the rows' sums: several threads have a part of each
        constexpr int kParts = kPlaneThreads / BM;
        __syncthreads();
        tile0[tid] = row_sum; // (kOpWide: row tid % BM)
        __syncthreads();
        if (j0 == 0 && tid < BM && i0 + tid < g.M) {
            float s = tile0[tid];
#pragma unroll
            for (int k = 1; k < kParts; ++k) s += tile0[k * BM + tid];
            out[(long long)(i0 + tid) * pitch + g.N] = s;
        }
    }
}

// Workgroups are dealt to the eight parts of the chip in turn, each with a second-level cache of its own: neighbouring tiles, which
// share rows of A, go to the same one.
__device__ __forceinline__ int xcd_chunk(int id, int count)
{
    const int each = count / kXcds, more = count % kXcds, xcd = id % kXcds;
    return xcd * each + min(xcd, more) + id / kXcds;
}

// Products with quantised weights take the same way with other planes for B.  A code is an integer of at most 8 bits, which one
// bfloat16 holds exactly: three products instead of six, and nothing to split in B (44 vector instructions of a thread's 90 a slab).  The
// row's scale is taken out of the sum (forward: the output's column) or goes into A as that is split, with what the product loses
// (input gradients).  The quantised weight is scale * code rounded to a float: that rounding, up to 2^-24 of it, is a second plane of the
// forward, without which parameter gradients' error against 64 bits is 4 % larger (16 models, geometric mean / median: embedding
// gradients 1.68e-7 by six products, parameter gradients 6.00e-8; so 1.66e-7 and 5.73e-8).  In the train step of the Terabyte shape,
// 8192 samples, us: forward 128x128 26.8 -> 21.2, 128x64 17.8 -> 16.2; input gradients 128x128 26.1 -> 22.4.
template <typename TILE, int B_MODE>
__global__ __launch_bounds__(kPlaneThreads) void gemm_planes_kernel(GemmArgs g)
{
    // (two arrays: the compiler knows that what is read from one is not what is written to the other)
    __shared__ __align__(16) char lds0[TILE::kSlabBytes], lds1[TILE::kSlabBytes];
    gemm_planes_tile<TILE, kOpRC, B_MODE, false>(g, xcd_chunk((int)blockIdx.x, (int)gridDim.x), lds0, lds1);
}

// With kslices > 1 the waves of a workgroup meet at a barrier inside: a wave past the last tile stays, takes the
// last tile with an empty reduction and stores nothing.
struct GemmOne {
    GemmArgs p;
    int total_tiles, kslices;
};

// one product per launch
template <int B_MODE>
__global__ __launch_bounds__(kGemmThreads) void gemm_wave_kernel(GemmOne one)
{
    __shared__ __align__(16) float lds[kGemmLdsFloats];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); // wave-uniform, and known to be
    const int ks = one.kslices;
    const int tile = ((int)blockIdx.x * kGemmWaves + wave) / ks;
    const bool live = tile < one.total_tiles;
    if (!live && ks == 1) return;
    gemm_wave_tile<B_MODE>(one.p, min(tile, one.total_tiles - 1), live, ks, wave, lane, lds);
}

// Several split products in one launch (kOpWide operands): the weight gradients of all layers, a workgroup per tile.
// Measured: the Terabyte shape's layers at batch 8192 (12.4 GFLOP) 85-89 us in the step's kernel trace, the Kaggle shape's at 2048
// (1.96 GFLOP) 20-22; on the fp32 matrix instructions 171 and 34.5.
__global__ __launch_bounds__(kPlaneThreads) void gemm_split_group_kernel(GemmGroup grp)
{
    constexpr int kLds = PlaneTile128::kSlabBytes > PlaneTile64::kSlabBytes ? PlaneTile128::kSlabBytes : PlaneTile64::kSlabBytes;
    __shared__ __align__(16) char lds0[kLds], lds1[kLds];
    const int id = xcd_chunk((int)blockIdx.x, (int)gridDim.x); // (a slice's tiles share their operands' rows)
    int pi = 0;
#pragma unroll 1
    for (int q = 1; q < grp.count; ++q)
        if (id >= grp.p[q].block_begin) pi = q;
    const GemmArgs &g = grp.p[pi];
    const int local = id - g.block_begin;
    if (g.tile == 128)
        gemm_planes_tile<PlaneTile128, kOpWide, kOpWide, true>(g, local, lds0, lds1);
    else
        gemm_planes_tile<PlaneTile64, kOpWide, kOpWide, true>(g, local, lds0, lds1);
}

// ---- a layer with a short input (the bottom MLP's first: 13 dense features) -------------------------------
// Y[b][o] = act(sum_k X[b][k] * W[o][k] + bias[o]) for K <= kSmallKMax: a product with a reduction this short is
// all launch and edge handling on the matrix cores.  A thread owns four consecutive outputs: their 4 K weights stay
// in registers while the thread walks the workgroup's samples, whose inputs sit in LDS.
constexpr int kSmallKMax = 16;
constexpr int kSmallKThreads = 128;
// Samples per workgroup, from the least to the most (small_k_samples()).  Every workgroup reads all weights, in 4 K loads a
// thread whose lanes lie 16 K bytes apart: 64 cache lines each, which cost more than everything else at 4 samples of a
// large batch: 8192x13 -> 512 takes 21.7 us with 4 samples to a workgroup, 12.9 with 16 (2048 samples, 4: 8.2).
constexpr int kSmallKMinSamples = 4, kSmallKMaxSamples = 16;
struct SmallKArgs {
    const float *X, *W, *bias;
    float *Y;
    int B, N, K, relu, samples; // N a multiple of 4, bias and Y 16-byte aligned (host)
};

__global__ __launch_bounds__(kSmallKThreads) void linear_small_k_kernel(SmallKArgs a)
{
    __shared__ float xs[kSmallKMaxSamples * kSmallKMax];
    const int N = a.N, K = a.K;
    const int b0 = (int)blockIdx.x * a.samples, nb = min(a.samples, a.B - b0); // samples <= kSmallKMaxSamples (host)
    for (int e = threadIdx.x; e < a.samples * kSmallKMax; e += kSmallKThreads) {
        const int bl = e / kSmallKMax, k = e % kSmallKMax;
        xs[e] = (bl < nb && k < K) ? a.X[(long long)(b0 + bl) * K + k] : 0.0f;
    }
    __syncthreads();
    for (int o = (int)threadIdx.x * 4; o < N; o += kSmallKThreads * 4) {
        // (4-byte loads: a row of an odd number of floats starts on no wider boundary; all 4 K are requested at once,
        // past K the last weight is read again and meets a zero input)
        float wr[4][kSmallKMax];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < kSmallKMax; ++k) wr[r][k] = a.W[(long long)(o + r) * K + min(k, K - 1)];
        const float4 bias = *reinterpret_cast<const float4 *>(a.bias + o);
        for (int bl = 0; bl < nb; ++bl) {
            float acc[4] = {bias.x, bias.y, bias.z, bias.w};
#pragma unroll
            for (int k = 0; k < kSmallKMax; ++k) {
                const float xv = xs[bl * kSmallKMax + k]; // zero past K
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = __builtin_fmaf(xv, wr[r][k], acc[r]);
            }
            if (a.relu) {
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = fmaxf(acc[r], 0.0f);
            }
            *reinterpret_cast<float4 *>(a.Y + (long long)(b0 + bl) * N + o) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
    }
}

// ---- the head: last linear layer (one output), sigmoid, binary cross-entropy, gradient w.r.t. its input ----
// z = X[b] . w + bias;  p = 1 / (1 + exp(-z));  term_b = -(y log max(p, 1e-12) + (1-y) log max(1-p, 1e-12));
// dz = (p - y) / B;  dX[b][k] = dz * w[k], masked by X[b][k] > 0 when X is a ReLU output.
// One wave per sample.  The mean of the terms is taken by loss_sum_block in the step's last kernel.
// (Block 0 also clears the `nzero` words at `zero`: the per-tensor gradient maxima of the INT8-gradient path,
// which are accumulated later in the same step.)
struct HeadArgs {
    const float *X;    // [B][in] input of the last top layer
    const float *w;    // [in] its weights (the ones the forward uses)
    const float *bias; // [1]
    const float *y;    // [B] labels
    float *z;          // [B] logits
    float *dz;         // [B]
    float *terms;      // [B] per-sample loss
    float *dX;         // [B][in]
    int relu_input;
    int B, in;
    unsigned *zero; // nzero words, zstride apart
    int nzero, zstride;
};

__global__ __launch_bounds__(256) void head_kernel(HeadArgs a)
{
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < a.nzero; k += 256) a.zero[(long long)k * a.zstride] = 0u;
    const int lane = threadIdx.x & (kWave - 1);
    const int b = (int)blockIdx.x * (256 / kWave) + (int)threadIdx.x / kWave;
    if (b >= a.B) return;
    const float *x = a.X + (long long)b * a.in;
    float s = 0.0f;
    for (int k = lane; k < a.in; k += kWave) s += x[k] * a.w[k];
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) s += __shfl_xor(s, d, kWave); // (every lane ends with the same sum)
    const float z = s + a.bias[0];
    const float p = 1.0f / (1.0f + expf(-z));
    const float yy = a.y[b];
    const float dz = (p - yy) / (float)a.B;
    if (lane == 0) {
        a.z[b] = z;
        a.dz[b] = dz;
        a.terms[b] = -(yy * logf(fmaxf(p, 1e-12f)) + (1.0f - yy) * logf(fmaxf(1.0f - p, 1e-12f)));
    }
    float *dx = a.dX + (long long)b * a.in;
    for (int k = lane; k < a.in; k += kWave) {
        const float g = dz * a.w[k];
        dx[k] = (!a.relu_input || x[k] > 0.0f) ? g : 0.0f;
    }
}

// loss = mean of the per-sample terms, by one block of 256 threads (fixed order: strided partial sums, then a tree)
__device__ __forceinline__ void loss_sum_block(const float *terms, int B, float *loss)
{
    __shared__ float part[256];
    float s = 0.0f;
    for (int b = threadIdx.x; b < B; b += 256) s += terms[b];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = part[0] / (float)B;
}

// SGD step from the split products of [dZ^T * X | dZ^T * 1], all layers in one launch:
// layer q's P is [S][out][in + 1];  W[o][i] -= lr * sum_s P[s][o][i],  b[o] -= lr * sum_s P[s][o][in]
// (slices added in order).  elem_begin[q] = first element of layer q in the launch's flat index space.
struct SgdLayer {
    const float *P;
    float *W, *b;
    int S, out, in;
    long long elem_begin; // first element of the layer in this launch's index space
    long long flat_begin; // ... in the model's flat parameter order (see dqrm_dense_quant_t)
    int tensor0;          // index of the layer's weight tensor in that order (its bias is tensor0 + 1)
    FastDiv by_cols;      // by in + 1, where the layer has fewer than 2^31 elements (else by_cols.d is 0)
};
struct SgdGroup {
    SgdLayer l[kGemmMaxGroup];
    int count;
    long long total;
    float lr;
    // INT8 gradients with error compensation (distributed-training section): flat arrays over the model
    float *grads;        // [P] this step's FP32 gradients (before the residual is added)
    float *err;          // [P] residuals carried between steps, or null
    int8_t *codes;       // [P] INT8 codes out, or null
    unsigned *gmax_bits; // [tensors][kGradMaxSlots][kGradMaxStride] running max |g + e| per tensor (word 0 of each line), as bit
                         // patterns, zeroed before the step
    float *grad_scale;   // [tensors] out
    // Simulated data parallelism (FP32 gradients): the gradient is added to (or starts) the caller's buffer, flat
    // over the model like `grads`, and the parameters take the step from the buffer, or none at all
    float *buffer;     // [P], or null
    int buffer_add;    // the buffer already holds earlier micro-batches
    int buffer_update; // this micro-batch ends its group: parameter <- parameter - lr * buffer
    // The launch that ends the step has one more block than the parameters need: it turns the per-sample loss
    // terms into the mean (null otherwise).
    const float *loss_terms; // [batch]
    float *loss;
    int batch;
};

// blocks that work on the parameters; the extra one, if any, does its job here and the caller returns
__device__ __forceinline__ bool sgd_extra_block(const SgdGroup &grp, int &blocks)
{
    blocks = gridDim.x;
    if (!grp.loss_terms) return false;
    blocks -= 1;
    if ((int)blockIdx.x < blocks) return false;
    loss_sum_block(grp.loss_terms, grp.batch, grp.loss);
    return true;
}

// The layers' descriptions in LDS, for lanes of different layers: read by a lane's own index from the kernel's arguments, every field
// is a round trip to memory (0.77 M parameters: grad_sum_absmax_kernel 12.7 -> 9.7 us; 0.48 M: sgd_from_partials_kernel 7.7 -> 6.1).
__device__ __forceinline__ void stage_layers(const SgdGroup &grp, SgdLayer *layers)
{
    const unsigned *from = reinterpret_cast<const unsigned *>(grp.l);
    unsigned *to = reinterpret_cast<unsigned *>(layers);
    for (int k = threadIdx.x; k < grp.count * (int)(sizeof(SgdLayer) / sizeof(unsigned)); k += 256) to[k] = from[k];
}

// which layer of the group element e belongs to, and where inside it
struct SgdElem {
    int q, o, i; // layer, output row, input column (i == in: the bias)
    long long le;
};
__device__ __forceinline__ SgdElem sgd_elem(const SgdGroup &grp, const SgdLayer *layers, long long e)
{
    SgdElem r;
    r.q = 0;
#pragma unroll 1
    for (int k = 1; k < grp.count; ++k)
        if (e >= grp.l[k].elem_begin) r.q = k;
    const SgdLayer &L = layers[r.q];
    r.le = e - L.elem_begin;
    r.o = L.by_cols.d ? (int)L.by_cols.div((unsigned)r.le) : (int)(r.le / (L.in + 1));
    r.i = (int)(r.le - (long long)r.o * (L.in + 1));
    return r;
}

constexpr int kSgdMaxSlices = 16; // slices of a split product, at most (the host's limit)

// the slices of one element, added in order; all of them are requested before the first is used, four at a time as far as there are any
// (a slice index past the last re-reads the last slice and is left out)
__device__ __forceinline__ float sum_partials(const SgdLayer &L, long long le)
{
    const long long per = (long long)L.out * (L.in + 1);
    float p[kSgdMaxSlices];
#pragma unroll
    for (int z0 = 0; z0 < kSgdMaxSlices; z0 += 4)
        if (z0 < L.S) // (the same in the whole wave, but where a layer ends)
#pragma unroll
            for (int z = z0; z < z0 + 4; ++z) p[z] = L.P[(long long)min(z, L.S - 1) * per + le];
    float s = 0.0f;
#pragma unroll
    for (int z = 0; z < kSgdMaxSlices; ++z)
        if (z < L.S) s += p[z];
    return s;
}

__global__ __launch_bounds__(256) void sgd_from_partials_kernel(SgdGroup grp)
{
    __shared__ SgdLayer s_layers[kGemmMaxGroup];
    int blocks;
    if (sgd_extra_block(grp, blocks)) return;
    stage_layers(grp, s_layers);
    __syncthreads();
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < grp.total; e += (long long)blocks * 256) {
        const SgdElem x = sgd_elem(grp, s_layers, e);
        const SgdLayer &L = s_layers[x.q];
        float s = sum_partials(L, x.le);
        if (grp.buffer) {
            float *slot = grp.buffer + L.flat_begin + x.le;
            if (grp.buffer_add) s = *slot + s;
            *slot = s;
            if (!grp.buffer_update) continue;
        }
        if (x.i < L.in)
            L.W[(long long)x.o * L.in + x.i] = L.W[(long long)x.o * L.in + x.i] - grp.lr * s;
        else
            L.b[x.o] = L.b[x.o] - grp.lr * s;
    }
}

// INT8 gradients, pass 1: the FP32 gradient of every parameter (slices added in order) goes to `grads`,
// and the maximum of |gradient + residual| of every tensor to gmax_bits (per-block maxima in LDS first).
constexpr int kMaxGradTensors = 2 * 2 * 16; // weights and bias of at most 16 + 16 layers
constexpr int kGradMaxSlots = 16;           // lines per tensor, a workgroup uses line blockIdx % 16: a large tensor's
                                            // ~700 workgroups would otherwise queue up at one line
constexpr int kGradMaxStride = 32;          // words between two maxima: one 128-byte line each (same-line
                                            // atomics from many workgroups serialise at the memory side)
__global__ __launch_bounds__(256) void grad_sum_absmax_kernel(SgdGroup grp)
{
    __shared__ unsigned s_max[kMaxGradTensors];
    __shared__ SgdLayer s_layers[kGemmMaxGroup];
    for (int k = threadIdx.x; k < kMaxGradTensors; k += 256) s_max[k] = 0u;
    stage_layers(grp, s_layers);
    __syncthreads();
    // a thread keeps the running maximum of the tensor it is in and hands it over when the tensor changes
    int cur_t = -1;
    float cur_max = 0.0f;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < grp.total; e += (long long)gridDim.x * 256) {
        const SgdElem x = sgd_elem(grp, s_layers, e);
        const SgdLayer &L = s_layers[x.q];
        const float s = sum_partials(L, x.le);
        const long long f = L.flat_begin + x.le;
        grp.grads[f] = s;
        const float gp = grp.err ? s + grp.err[f] : s;
        const int t = L.tensor0 + (x.i < L.in ? 0 : 1);
        if (t != cur_t) {
            if (cur_t >= 0 && cur_max > 0.0f) atomicMax(s_max + cur_t, __float_as_uint(cur_max));
            cur_t = t;
            cur_max = 0.0f;
        }
        cur_max = fmaxf(cur_max, fabsf(gp));
    }
    // usually the whole wave ends in one tensor: one LDS atomic per wave
    const int tt = wave_max_int(cur_t);
    if (__all(cur_t < 0 || cur_t == tt)) {
        const float m = wave_max(cur_max);
        if ((threadIdx.x & (kWave - 1)) == 0 && tt >= 0 && m > 0.0f) atomicMax(s_max + tt, __float_as_uint(m));
    } else if (cur_t >= 0 && cur_max > 0.0f) {
        atomicMax(s_max + cur_t, __float_as_uint(cur_max));
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kMaxGradTensors; k += 256)
        if (s_max[k] != 0u)
            atomicMax(grp.gmax_bits + (k * kGradMaxSlots + (int)(blockIdx.x % kGradMaxSlots)) * kGradMaxStride, s_max[k]);
}

// pass 2: g' = g + e;  s = max(max|g'| / 127, 1e-8);  code = clamp(rint(g' / s), -128, 127);
// e <- g' - s * code;  parameter <- parameter - lr * (s * code)   (every operation rounded on its own)
__global__ __launch_bounds__(256) void grad_quant_ec_kernel(SgdGroup grp)
{
    __shared__ Scale s_scale[kMaxGradTensors];
    __shared__ SgdLayer s_layers[kGemmMaxGroup];
    int blocks;
    if (sgd_extra_block(grp, blocks)) return;
    stage_layers(grp, s_layers);
    __syncthreads();
    // the tensors of this launch's layers
    for (int k = threadIdx.x; k < 2 * grp.count; k += 256) {
        const int t = s_layers[k >> 1].tensor0 + (k & 1);
        unsigned m[kGradMaxSlots], mx = 0u;
#pragma unroll
        for (int q = 0; q < kGradMaxSlots; ++q) m[q] = grp.gmax_bits[(t * kGradMaxSlots + q) * kGradMaxStride];
#pragma unroll
        for (int q = 0; q < kGradMaxSlots; ++q) mx = max(mx, m[q]); // (non-negative floats order like their bits)
        const float gs = scale_from_absmax(__uint_as_float(mx), 127.0f);
        s_scale[t] = Scale(gs);
        if (blockIdx.x == 0) grp.grad_scale[t] = gs;
    }
    __syncthreads();
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < grp.total; e += (long long)blocks * 256) {
        const SgdElem x = sgd_elem(grp, s_layers, e);
        const SgdLayer &L = s_layers[x.q];
        const long long f = L.flat_begin + x.le;
        const Scale sc = s_scale[L.tensor0 + (x.i < L.in ? 0 : 1)];
        float *p = x.i < L.in ? L.W + (long long)x.o * L.in + x.i : L.b + x.o;
        const float g = grp.grads[f], w = *p; // (the parameter too before anything is stored)
        const float gp = grp.err ? g + grp.err[f] : g;
        const int c = int8_code_fresh(gp, sc); // the scale comes from the maximum of these very values
        if (grp.codes) grp.codes[f] = (int8_t)c;
        const float deq = sc.s * (float)c;
        if (grp.err) grp.err[f] = gp - deq;
        const float step = grp.lr * deq;
        *p = w - step;
    }
}

// ---- channel-wise fake quantisation of the linear layers' weights (model-quantisation appendix) ------
// One scale per output row: s_o = max(max_i |W[o][i]| / qmax, 1e-8), Wq[o][i] = s_o * clamp(rint(W[o][i] / s_o)).
// One wave per row, all layers in one launch.
struct FqLayer {
    const float *W;
    float *Wq;
    unsigned short *codes, *low; // [out][pitch] bfloat16, zeros from `in` on; low: see GemmArgs; null: not wanted
    float *scale;          // [out], if they are
    int out, in, row_begin, pitch;
};
struct FqGroup {
    FqLayer l[kGemmMaxGroup];
    int count, total_rows;
    float qmax; // 7 or 127; the lowest code is -qmax - 1
};

__global__ __launch_bounds__(256) void mlp_fake_quant_kernel(FqGroup grp)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int row = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (256 / kWave) + threadIdx.x / kWave));
    if (row >= grp.total_rows) return;
    int q = 0;
#pragma unroll 1
    for (int k = 1; k < grp.count; ++k)
        if (row >= grp.l[k].row_begin) q = k;
    const FqLayer &L = grp.l[q];
    const float *w = L.W + (long long)(row - L.row_begin) * L.in;
    float *wq = L.Wq + (long long)(row - L.row_begin) * L.in;
    const long long code_row = (long long)(row - L.row_begin) * L.pitch;
    float m = 0.0f;
    for (int i = lane; i < L.in; i += kWave) m = fmaxf(m, fabsf(w[i]));
    m = wave_max(m);
    const Scale sc(scale_from_absmax(m, grp.qmax));
    for (int i = lane; i < L.in; i += kWave) {
        // a fresh scale: no quotient beyond qmax (1 + 2^-23)
        const int c = code_i<false>(w[i], sc, -grp.qmax - 1.0f, grp.qmax);
        const float v = sc.s * (float)c;
        wq[i] = v;
        if (!L.codes) continue; // (wave-uniform)
        L.low[code_row + i] = (unsigned short)(__float_as_uint(__builtin_fmaf(-sc.s, (float)c, v) * sc.y) >> 16);
        L.codes[code_row + i] = (unsigned short)(__float_as_uint((float)c) >> 16); // (exact: 8 bits)
    }
    if (!L.codes) return;
    for (int i = L.in + lane; i < L.pitch; i += kWave) L.codes[code_row + i] = L.low[code_row + i] = 0;
    if (lane == 0) L.scale[row - L.row_begin] = sc.s;
}

// ---- pairwise-dot interaction ---------------------------------------------------
// Z[b] = [bottom-MLP output, table 0 .. table T-1], V = T + 1 vectors of width D.
// R[b] = [Z[b][0] (D values), dot(Z[b][i], Z[b][j]) for i = 1..V-1, j = 0..i-1, row-major].
struct InteractArgs {
    const float *bot; // [B][D]
    const float *emb; // [B][T][D]
    float *R;         // [B][D + V(V-1)/2]
    const float *dR;  // backward: gradient w.r.t. R
    float *dbot;      // [B][D]
    float *demb;      // [B][T][D]
    const float *bot_mask; // the bottom MLP's last activation (ReLU mask for dbot), or null
    int B, T, D;
    // The bottom MLP's last layer, when it is small enough to ride along (lin_w != null): the forward kernel computes
    // bot[b] = relu(lin_x[b] * lin_w^T + lin_b) itself (and stores it to lin_y for the backward pass); the backward
    // kernel goes on from dbot to that layer's input gradient, lin_dx[b] = (dbot[b] * lin_w) masked by lin_mask > 0.
    const float *lin_x;    // [B][lin_k] input of that layer
    const float *lin_w;    // [D][lin_k]
    const float *lin_b;    // [D]
    float *lin_y;          // [B][D] its output
    const float *lin_mask; // [B][lin_k] backward: the layer's input if that is a ReLU output, or null
    float *lin_dx;         // [B][lin_k] backward: gradient w.r.t. the pre-activation of the layer before, or null
    int lin_k;
};

constexpr int kInterThreads = 256; // at most; a wave per sample
constexpr int kInterWaves = kInterThreads / kWave;
constexpr int kInterMaxV = 64;      // vectors per sample, at most (host)
constexpr int kInterMaxZ = 64 * 64; // V * D floats, at most (host)
constexpr int kInterLdsBytes = 64 * 1024; // of a workgroup, at most

// Layout of a wave's LDS: the sample's vectors, rows of Dp = D rounded up to 8 floats (zeros past D) and a pitch of
// Dp + 4 (the lanes of a wave read 16 bytes of different rows: a pitch that is a multiple of the bank count would put
// them all into the same banks); the backward kernel adds the symmetric matrix of pair gradients.
__host__ __device__ inline int inter_dp(int D) { return (D + 7) & ~7; }
__host__ __device__ inline int inter_pitch(int D) { return inter_dp(D) + 4; }
__host__ __device__ inline int inter_tiles(int V) { return (V + 31) / 32; }
__host__ __device__ inline int inter_sp(int V) { return 32 * inter_tiles(V) + 4; } // pitch of the pair-gradient matrix
// The bottom MLP's last layer rides along in these kernels while its weights are few: every sample's wave reads them all
// (from LDS in the forward, from the first-level cache in the backward).  Rows of 4 * odd floats: the 16 outputs that a
// wave computes at a time then start in different banks.
__host__ __device__ inline int inter_lin_pitch(int K)
{
    const int q = (K + 3) / 4;
    return 4 * (q | 1);
}
// weights (with their padding) of a layer that rides along, at most (host): of any batch, of a small one, of a small one in the
// plain kernels
constexpr int kInterLinFloats = 4096, kInterLinFloatsFew = 4608, kInterLinFloatsPlain = 8704;
// floats of LDS per wave: forward (lin_k: the riding layer's input width, or 0), backward
__host__ __device__ inline int inter_wave_floats(int V, int D, int lin_k)
{
    return V * inter_pitch(D) + (lin_k ? inter_lin_pitch(lin_k) : 0);
}
__host__ __device__ inline int inter_wave_floats_bwd(int V, int D)
{
    return V * inter_pitch(D) + 32 * inter_tiles(V) * inter_sp(V);
}

// pair index p -> (i, j), i > j, p = i(i-1)/2 + j
__device__ __forceinline__ void pair_of(int p, int &i, int &j)
{
    i = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)p)) * 0.5f);
    while (i * (i - 1) / 2 > p) --i;
    while ((i + 1) * i / 2 <= p) ++i;
    j = p - i * (i - 1) / 2;
}

// What the lanes of a wave wrote to their LDS may be read by its other lanes from here on: the wave's LDS operations
// complete in order, so this only keeps the compiler from moving them.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Vectors 1 .. T of a sample (T * D consecutive floats) into rows 1 .. T of z, by one wave.  request() asks for the first
// kAhead loads per lane, so that they travel beside whatever else the kernel needs first; settle() does the rest.
template <bool VEC>
struct InterRows {
    static constexpr int kAhead = 8;
    Float4Dw q[kAhead];
    const float *emb;
    int cols, count, lane;

    __device__ __forceinline__ void load(int e0)
    {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int e = min(e0 + k * kWave, count - 1);
            if (VEC)
                q[k] = *reinterpret_cast<const Float4Dw *>(emb + 4ll * e);
            else
                q[k][0] = emb[e];
        }
    }
    __device__ __forceinline__ void request(const float *from, int T, int D, int my_lane)
    {
        emb = from, lane = my_lane, cols = VEC ? D / 4 : D, count = T * cols;
        load(lane);
    }
    __device__ __forceinline__ void settle(float *z, int pitch)
    {
        const int dr = kWave / cols, dc = kWave - dr * cols;
        int r = lane / cols, c = lane - r * cols;
        for (int e0 = lane;;) {
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                if (e0 + k * kWave < count) {
                    float *at = z + (1 + r) * pitch + (VEC ? 4 * c : c);
                    if (VEC)
                        *reinterpret_cast<float4 *>(at) = make_float4(q[k][0], q[k][1], q[k][2], q[k][3]);
                    else
                        *at = q[k][0];
                }
                r += dr, c += dc;
                if (c >= cols) c -= cols, ++r;
            }
            e0 += kAhead * kWave;
            if (e0 >= count) break;
            load(e0);
        }
    }
};

// One wave per sample, V <= 32 NT.  The pair products are the lower triangle of Z * Z^T on the matrix cores; both operands
// are the same registers (lane l holds Z[l % 32][.] as a row of A and as a column of B), read from LDS 16 bytes at a
// time.  Rows past V re-read the last vector: their products are not stored.  A tile's product s pairs the elements s and
// Dp / 2 + s of the vectors.
// What bounds it: reading the embeddings (54.5 MB at 27 vectors of 64 x 8192 samples).  There, with the bottom MLP's last layer
// (256 -> 64) as a product of its own: 22 us (kernel alone); dot products with a thread each and that layer's weights read again
// for every sample took 90 us.
template <int NT, bool VEC>
__global__ __launch_bounds__(kInterThreads) void interact_fwd_kernel(InteractArgs a)
{
    extern __shared__ __align__(16) float inter_lds[]; // weights of the riding layer, then inter_wave_floats() per wave
    const int V = a.T + 1, D = a.D, Dp = inter_dp(D), pitch = inter_pitch(D), K = a.lin_k;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), waves = (int)blockDim.x / kWave;
    const int lp = inter_lin_pitch(K), lin = a.lin_w ? D * lp : 0;
    const int b = (int)blockIdx.x * waves + wave;
    const bool live = b < a.B;
    float *z = inter_lds + lin + wave * inter_wave_floats(V, D, a.lin_w ? K : 0);
    const long long bc = min(b, a.B - 1);
    InterRows<VEC> rows;
    rows.request(a.emb + bc * a.T * D, a.T, D, lane);
    const float *first = a.lin_w ? a.lin_x + bc * K : a.bot + bc * D; // input of the riding layer, or vector 0 itself
    const int nf = a.lin_w ? K : D;
    const float f0 = first[min(lane, nf - 1)];
    if (a.lin_w) { // (all waves of the workgroup)
        for (int e = threadIdx.x; e < D * K; e += blockDim.x) {
            const int d = e / K;
            inter_lds[d * lp + (e - d * K)] = a.lin_w[e];
        }
        __syncthreads();
    }
    if (!live) return;
    float *r = a.R + (long long)b * (D + V * (V - 1) / 2);
    rows.settle(z, pitch);
    if (a.lin_w) {
        float *x = z + V * pitch; // lp floats
        if (lane < K) x[lane] = f0;
        for (int k = lane + kWave; k < K; k += kWave) x[k] = first[k];
        wave_lds_order();
        // 4 lanes per output, each a strided quarter of the sum
        for (int d0 = 0; d0 < D; d0 += kWave / 4) {
            const int d = d0 + (lane >> 2), part = lane & 3;
            const float *w = inter_lds + min(d, D - 1) * lp;
            const float bias = a.lin_b[min(d, D - 1)];
            float s = 0.0f;
            for (int k = part; k < K; k += 4) s = __builtin_fmaf(x[k], w[k], s);
            s += __shfl_xor(s, 1, kWave);
            s += __shfl_xor(s, 2, kWave);
            if (part == 0 && d < D) {
                const float y = fmaxf(s + bias, 0.0f);
                z[d] = y;
                a.lin_y[(long long)b * D + d] = y;
                r[d] = y;
            }
        }
    } else {
        if (lane < D) z[lane] = r[lane] = f0;
        for (int d = lane + kWave; d < D; d += kWave) z[d] = r[d] = first[d];
    }
    if (Dp != D)
        for (int e = lane; e < V * (Dp - D); e += kWave) z[e / (Dp - D) * pitch + D + e % (Dp - D)] = 0.0f;
    wave_lds_order();
    const int w = lane & 31, h = lane >> 5;
    floatx16 acc[NT == 1 ? 1 : 3]; // tiles (0, 0), (1, 0), (1, 1)
#pragma unroll
    for (int t = 0; t < (NT == 1 ? 1 : 3); ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
    const float *z0 = z + min(w, V - 1) * pitch + h * (Dp / 2), *z1 = z + min(32 + w, V - 1) * pitch + h * (Dp / 2);
#pragma unroll 4
    for (int s = 0; s < Dp / 2; s += 4) {
        const float4 q4 = *reinterpret_cast<const float4 *>(z0 + s);
        const float q[4] = {q4.x, q4.y, q4.z, q4.w};
        if (NT == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(q[k], q[k], acc[0], 0, 0, 0);
        } else {
            const float4 p4 = *reinterpret_cast<const float4 *>(z1 + s);
            const float p[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(q[k], q[k], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[k], q[k], acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(p[k], p[k], acc[2], 0, 0, 0);
            }
        }
    }
    // lane l holds column j = l % 32 and rows 8 (v / 4) + 4 (l / 32) + v % 4 of a tile
#pragma unroll
    for (int t = 0; t < (NT == 1 ? 1 : 3); ++t) {
        const int i0 = t == 0 ? 0 : 32, j = (t == 2 ? 32 : 0) + w;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int i = i0 + 8 * (v >> 2) + 4 * h + (v & 3);
            if (i < V && j < i) r[D + i * (i - 1) / 2 + j] = acc[t][v];
        }
    }
}

// dZ[i] = sum over j != i of dP(i, j) * Z[j]  (+ dR[0..D) for i = 0): the pair gradients are spread into a symmetric
// matrix S with a zero diagonal (and zeros past V), and dZ = S * Z goes to the matrix cores, a wave per sample (vectors past
// V are zeros in both).
// What bounds it: reading the embeddings and writing their gradients (109 MB at 27 vectors of 64 x 8192 samples).  There:
// 35 us; a thread per element with the sum from LDS took 86 us.
template <int NT, bool VEC>
__global__ __launch_bounds__(kInterThreads) void interact_bwd_kernel(InteractArgs a)
{
    extern __shared__ __align__(16) float inter_lds[]; // inter_wave_floats_bwd() per wave
    const int V = a.T + 1, D = a.D, pitch = inter_pitch(D), sp = inter_sp(V);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int b = (int)blockIdx.x * ((int)blockDim.x / kWave) + wave;
    if (b >= a.B) return; // (no barrier below)
    float *S = inter_lds + wave * inter_wave_floats_bwd(V, D), *z = S + 32 * NT * sp;
    const int P = V * (V - 1) / 2;
    const float *dr = a.dR + (long long)b * (D + P);
    // everything is requested before the first wait
    InterRows<VEC> rows;
    rows.request(a.emb + (long long)b * a.T * D, a.T, D, lane);
    constexpr int kPairsAhead = 8;
    float g[kPairsAhead];
#pragma unroll
    for (int k = 0; k < kPairsAhead; ++k) g[k] = dr[D + min(lane + k * kWave, P - 1)];
    const float f0 = a.bot[(long long)b * D + min(lane, D - 1)];
    for (int e = lane; e < 32 * NT * sp / 4; e += kWave) reinterpret_cast<float4 *>(S)[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    wave_lds_order();
    auto spread = [&](int p, float x) {
        int i, j;
        pair_of(p, i, j);
        S[i * sp + j] = x;
        S[j * sp + i] = x;
    };
#pragma unroll
    for (int k = 0; k < kPairsAhead; ++k)
        if (lane + k * kWave < P) spread(lane + k * kWave, g[k]);
    for (int p = lane + kPairsAhead * kWave; p < P; p += kWave) spread(p, dr[D + p]);
    rows.settle(z, pitch);
    if (lane < D) z[lane] = f0;
    for (int d = lane + kWave; d < D; d += kWave) z[d] = a.bot[(long long)b * D + d];
    wave_lds_order();
    const int w = lane & 31, h = lane >> 5;
    float mine[NT][NT][16]; // this lane's 16 elements of S per tile: row l % 32, columns 16 (l / 32) + s
#pragma unroll
    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
        for (int tk = 0; tk < NT; ++tk)
#pragma unroll
            for (int s = 0; s < 16; s += 4) {
                const float4 q = *reinterpret_cast<const float4 *>(S + (32 * ti + w) * sp + 32 * tk + 16 * h + s);
                mine[ti][tk][s] = q.x, mine[ti][tk][s + 1] = q.y, mine[ti][tk][s + 2] = q.z, mine[ti][tk][s + 3] = q.w;
            }
    for (int d0 = 0; d0 < D; d0 += 32) {
        const int d = d0 + w;
        const bool in = d < D;
        const float *zc = z + min(d, D - 1);
        floatx16 acc[NT];
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ti][v] = 0.0f;
#pragma unroll
        for (int tk = 0; tk < NT; ++tk) {
            float x[16];
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int k = 32 * tk + 16 * h + s;
                const float q = zc[min(k, V - 1) * pitch];
                x[s] = k < V ? q : 0.0f;
            }
#pragma unroll
            for (int s = 0; s < 16; ++s)
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
                    acc[ti] = __builtin_amdgcn_mfma_f32_32x32x2f32(mine[ti][tk][s], x[s], acc[ti], 0, 0, 0);
        }
        // lane l holds column d = d0 + l % 32 and rows 8 (v / 4) + 4 (l / 32) + v % 4 of a tile
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * ti + 8 * (v >> 2) + 4 * h + (v & 3);
                if (!in || i >= V) continue;
                if (i == 0) {
                    const long long off = (long long)b * D + d;
                    float s = acc[ti][v] + dr[d];
                    if (a.bot_mask) s = a.bot_mask[off] > 0.0f ? s : 0.0f;
                    a.dbot[off] = s;
                    z[d] = s; // (this column of z has been used: the gradient w.r.t. bot takes row 0's place)
                } else {
                    a.demb[((long long)b * a.T + (i - 1)) * D + d] = acc[ti][v];
                }
            }
    }
    if (a.lin_w && a.lin_dx) { // on to the input gradient of the bottom MLP's last layer
        wave_lds_order();
        const int K = a.lin_k;
        for (int k = lane; k < K; k += kWave) {
            float s = 0.0f;
            for (int d = 0; d < D; ++d) s = __builtin_fmaf(z[d], a.lin_w[(long long)d * K + k], s);
            if (a.lin_mask) s = a.lin_mask[(long long)b * K + k] > 0.0f ? s : 0.0f;
            a.lin_dx[(long long)b * K + k] = s;
        }
    }
}

// ---- the plain kernels: few or short vectors (inter_plain()) ------------------------------------------------------
// The matrix cores' tiles would be mostly padding, and a wave per sample a long way for the little there is to do: a sample has a
// workgroup, whose threads take pairs (forward) or elements (backward).  Bound by that chain of a sample (loads, LDS, the riding
// layer, stores) and the instructions of 128 threads per sample.  9 vectors of 16, 8192 samples, with a layer 32 -> 16 riding
// along: 8.7 and 11.8 us; the kernels above take 10.5 and 17.9.
constexpr int kInterPlainThreads = 128;
// floats of dynamic LDS (at most 33 KB)
inline int inter_plain_floats(int V, int D, bool backward, int lin_k)
{
    return (backward ? V * D + V * (V | 1) + D : V * (D + 1)) + lin_k;
}

__global__ __launch_bounds__(kInterPlainThreads) void interact_fwd_plain_kernel(InteractArgs a)
{
    // rows one float apart from a multiple of the bank count: the lanes of a wave read different rows at the
    // same d, and with a pitch of D = 16 all of them would fall into two banks
    extern __shared__ __align__(16) float inter_lds[]; // V * (D + 1) (+ lin_k) floats (inter_plain_floats)
    float *z = inter_lds;
    const int b = blockIdx.x, V = a.T + 1, D = a.D, pitch = D + 1;
    if (a.lin_w) {
        // the embeddings travel while the layer is computed: 8 threads per output, each a strided eighth of the sum
        for (int e = D + (int)threadIdx.x; e < V * D; e += kInterPlainThreads) {
            const int i = e / D, d = e - i * D;
            z[i * pitch + d] = a.emb[(long long)b * a.T * D + (e - D)];
        }
        float *xin = inter_lds + V * pitch; // lin_k floats
        const int K = a.lin_k;
        for (int k = threadIdx.x; k < K; k += kInterPlainThreads) xin[k] = a.lin_x[(long long)b * K + k];
        __syncthreads();
        for (int e0 = 0; e0 < D * 8; e0 += kInterPlainThreads) { // (kInterPlainThreads is a multiple of 8: teams stay whole)
            const int e = e0 + (int)threadIdx.x;
            const int d = min(e >> 3, D - 1), part = e & 7;
            const float *w = a.lin_w + (long long)d * K;
            float s = 0.0f;
            for (int k = part; k < K; k += 8) s = __builtin_fmaf(xin[k], w[k], s);
            s += __shfl_xor(s, 1, kWave);
            s += __shfl_xor(s, 2, kWave);
            s += __shfl_xor(s, 4, kWave);
            if (part == 0 && e < D * 8) {
                const float y = fmaxf(s + a.lin_b[d], 0.0f);
                z[d] = y;
                a.lin_y[(long long)b * D + d] = y;
            }
        }
    } else {
        for (int e = threadIdx.x; e < V * D; e += kInterPlainThreads) {
            const int i = e / D, d = e - i * D;
            z[i * pitch + d] = e < D ? a.bot[(long long)b * D + e] : a.emb[(long long)b * a.T * D + (e - D)];
        }
    }
    __syncthreads();
    const int P = V * (V - 1) / 2, W = D + P;
    float *r = a.R + (long long)b * W;
    for (int e = threadIdx.x; e < W; e += kInterPlainThreads) {
        if (e < D) {
            r[e] = z[e];
        } else {
            int i, j;
            pair_of(e - D, i, j);
            const float *zi = z + i * pitch, *zj = z + j * pitch;
            float s = 0.0f;
            for (int d = 0; d < D; ++d) s += zi[d] * zj[d];
            r[e] = s;
        }
    }
}

// The pair gradients are spread into a symmetric matrix with a zero diagonal first, so that an element's sum runs over all j (in the
// order 0 .. V-1) without a case distinction.
__global__ __launch_bounds__(kInterPlainThreads) void interact_bwd_plain_kernel(InteractArgs a)
{
    extern __shared__ __align__(16) float inter_lds[]; // V * D + V * (V | 1) + D floats (inter_plain_floats)
    const int b = blockIdx.x, V = a.T + 1, D = a.D, vp = V | 1; // odd pitch
    float *z = inter_lds, *dpf = inter_lds + V * D, *dzl = dpf + V * vp; // dzl: D floats, the gradient w.r.t. bot
    const int P = V * (V - 1) / 2, W = D + P;
    for (int e = threadIdx.x; e < V * D; e += kInterPlainThreads)
        z[e] = e < D ? a.bot[(long long)b * D + e] : a.emb[(long long)b * a.T * D + (e - D)];
    const float *dr = a.dR + (long long)b * W;
    for (int p = threadIdx.x; p < P; p += kInterPlainThreads) {
        int i, j;
        pair_of(p, i, j);
        const float g = dr[D + p];
        dpf[i * vp + j] = g;
        dpf[j * vp + i] = g;
    }
    for (int i = threadIdx.x; i < V; i += kInterPlainThreads) dpf[i * vp + i] = 0.0f;
    __syncthreads();
    for (int e = threadIdx.x; e < V * D; e += kInterPlainThreads) {
        const int i = e / D, d = e - i * D;
        float s = (i == 0) ? dr[d] : 0.0f;
        const float *row = dpf + i * vp, *col = z + d;
        for (int j = 0; j < V; ++j) s += row[j] * col[j * D];
        if (i == 0) {
            const long long off = (long long)b * D + d;
            if (a.bot_mask) s = a.bot_mask[off] > 0.0f ? s : 0.0f;
            a.dbot[off] = s;
            dzl[d] = s;
        } else {
            a.demb[(long long)b * a.T * D + (e - D)] = s;
        }
    }
    if (a.lin_w && a.lin_dx) { // on to the input gradient of the bottom MLP's last layer
        __syncthreads();
        const int K = a.lin_k;
        for (int k = threadIdx.x; k < K; k += kInterPlainThreads) {
            float s = 0.0f;
            for (int d = 0; d < D; ++d) s = __builtin_fmaf(dzl[d], a.lin_w[(long long)d * K + k], s);
            if (a.lin_mask) s = a.lin_mask[(long long)b * K + k] > 0.0f ? s : 0.0f;
            a.lin_dx[(long long)b * K + k] = s;
        }
    }
}

} // namespace dqrm
