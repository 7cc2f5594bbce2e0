// Keyframe-query attention for gfx950 (CDNA4).
//
// Method (Sec. 3.2.3-3.2.4; App. B.2): at a step where only keyframes are
// denoised, the query tokens of the M keyframes attend over the keys and
// values of all T frames. Per head: out = softmax(Q_kf K^T / sqrt(d)) V.
//
// bf16 kernel design:
//  * A workgroup of 8 waves owns one (head, 256-row query tile); each wave
//    owns 32 query rows. Query rows are gathered straight from the keyframe
//    tokens (row r reads token kf[r / N] * N + r % N), so the gather is fused
//    and non-keyframe query rows are never read.
//  * Scores are computed transposed, S^T = K Q^T, with
//    v_mfma_f32_32x32x16_bf16: K rows are the A operand (from LDS), the
//    wave's query rows the B operand (held in registers for the whole loop).
//    In the 32x32 accumulator layout every lane then holds 16 scores of ONE
//    query column, so the softmax max and sum are in-lane reductions plus one
//    exchange with the lane 32 apart.
//  * The probabilities are already in the B-operand layout of the second
//    product, O^T = V^T P^T: the lane's 16 accumulators become two bf16x8
//    operands without any data movement. The V^T A operands are read from
//    the natural [key][dim] V tile with transposing LDS reads; the key order
//    inside an operand follows the accumulator layout (a reduction index may
//    be permuted freely as long as both operands agree).
//  * K and V tiles (64 keys; 128 at head dimension 64) go from HBM straight into LDS (buffer loads
//    with an LDS destination: no staging registers, no LDS write
//    instructions), double-buffered so the next tile streams in while the
//    current one is computed; the buffer range check zero-fills keys >= S and
//    the last tile masks their scores.
//  * Online softmax in the log2 domain with fp32 state, taken against a
//    reference that is a past row maximum: the row maximum of a tile is only
//    computed when the tile's row sum shows that a probability outgrew the
//    reference (first tile, or a jump by a factor of ~256), so the common tile
//    costs no max reduction. P is rounded to bf16 for the matrix cores and the
//    row sum adds those same rounded values.
//  * Workgroup ids are mapped XCD-aware: consecutive ids go round-robin to the
//    device's X XCDs (8 on MI355X), so tile = (id % X) * per_xcd + id / X gives
//    each XCD a contiguous, head-major range of tiles and the workgroups
//    resident on one XCD stream the same head's K/V through that XCD's L2.
//  * Split-key tail (when the caller provides a workspace): one workgroup
//    fills a CU, so a launch of n tiles runs in ceil(n / CUs) rounds (256 CUs
//    on MI355X; the count is queried from the device) and the
//    last round may leave most CUs idle. The tiles beyond the last full round
//    are then split along the keys into parts that run as extra workgroups;
//    each part writes its unnormalised (O, m, l) in fp32, and a small kernel
//    combines the parts of a tile (max of the references, rescaled sums).
//  * Small launches (when the caller provides a workspace or names the static
//    scratch): attn_bf16_small_kernel, 32 rows a workgroup, the keys shared out
//    among its waves; the rule is at small_pays.
//  * Frame-level key/value mask (the frame-list form): the key loop walks the
//    listed frames' keys end to end, a tile that reaches past a frame taking its
//    last keys from the next listed one (in tiles that never cross a frame where
//    that does not pay or fit: list_walk); masked frames are never read.
//  * Projected keys and values at a skipped step (the cache form; App. B.2):
//    the key loop walks all frames in frame-aligned tiles; a tile of a cached
//    frame loads that frame's two cached hidden states h_before and h_after
//    instead of K and V, and the workgroup forms
//    h = fmaf(alpha, h_after, (1 - alpha) h_before), rounded once to bf16, in
//    LDS as both the key tile and the value tile, so the projected keys and
//    values are never written to HBM.
// The fp32 kernels are in rf_attention_f32.hip.
#include <atomic>

#include "rf_device.h"
#include "rf_list_walk.h"

namespace rf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Data moves as 32-bit words; bf16 vectors are only ever formed by a
// whole-vector bitcast of a u32x4 (or of one scalar word) right before the
// instruction that consumes them.

// Tunables (compile-time): waves per workgroup (each owns 32 query rows), keys
// per LDS tile (at head dimension 128, and at 64), the largest row partial sum of a tile accepted before the
// softmax reference is rebased (so every probability stays below it), and how
// many LDS fragments the matrix core reads ahead.
#ifndef RF_ATTN_WAVES
#define RF_ATTN_WAVES 8
#endif
#ifndef RF_ATTN_BC
#define RF_ATTN_BC 64
#endif
#ifndef RF_ATTN_BC64
#define RF_ATTN_BC64 128
#endif
#ifndef RF_ATTN_REBASE_BOUND
#define RF_ATTN_REBASE_BOUND 256.0f
#endif
#ifndef RF_ATTN_K_LEAD
#define RF_ATTN_K_LEAD 4
#endif
#ifndef RF_ATTN_V_LEAD
#define RF_ATTN_V_LEAD 3
#endif

constexpr int kWaves = RF_ATTN_WAVES;
constexpr int kThreads = 64 * kWaves;
constexpr int kBr = 32 * kWaves;   // query rows per workgroup
// Keys per LDS tile. At head dimension 64 a tile of 64 keys carries half the
// matrix work of one at 128 for the same softmax, barrier and loop overhead, so
// it takes twice the keys (the registers and LDS that head dimension leaves free
// hold them).
__host__ __device__ constexpr int key_tile(int head_dim) { return head_dim == 64 ? RF_ATTN_BC64 : RF_ATTN_BC; }
// Split-key tail: the most parts a tail tile is cut into and the fewest key
// tiles a part has by the plan, which counts a frame list's tiles without any that
// crosses a frame (walked end to end there may be about half as many, and a part
// is that much shorter; list_walk sees to it that none is empty). A round of whole
// tiles fills the device's compute units (one workgroup per CU), queried at launch.
constexpr int kMaxSplit = 8;
constexpr int kMinKvPerSplit = 8;
constexpr float kRebaseBound = RF_ATTN_REBASE_BOUND;   // largest tile row sum kept without a rebase
static_assert(key_tile(64) % 32 == 0 && key_tile(128) % 32 == 0, "key tile must be a multiple of 32");

struct AttnKArgs {
    const uint16_t *q;
    const uint16_t *k;
    const uint16_t *v;
    uint16_t *out;
    int64_t S;
    int64_t N;
    int64_t Mq;
    int32_t heads;
    int32_t n_qtiles;
    int32_t total_tiles;    // tiles computed whole (all tiles when there is no split)
    int32_t per_xcd;
    int32_t xcds;           // XCDs of the device: workgroup id i runs on XCD i % xcds
    int32_t grid_direct;    // workgroups of the whole tiles (per_xcd * xcds)
    int32_t split;          // parts per tail tile (0: no split)
    int32_t kv_per_split;   // key tiles per part
    float *ws_o;            // [tail tile * split + part][kBr][D] unnormalised O
    float *ws_ml;           // [tail tile * split + part][kBr][2] reference max (log2 domain), row sum
    float scale_log2;   // log2(e) / sqrt(d)
    int32_t kf[kMaxFrames];
    // key/value frame list: the keys are the tokens of frames kvf[0..n_kv), in
    // list_tiles key tiles: end to end (tiles_per_frame = 0; a tile may run from
    // one frame into the next listed one), or in tiles that never cross a frame
    // (ceil(N / key tile) a frame, its last one partial; always in the cache form)
    int32_t n_kv;
    int32_t tiles_per_frame;
    int32_t list_tiles;
    // frame-list form: the listed frames; cache form (all T frames walked): per
    // frame the two cache slots (h_before | h_after << 16), or -1 when the frame
    // takes its keys and values from k and v
    int32_t kvf[kMaxFrames];
    const uint16_t *store;           // cache form: [slot][N][heads][head_dim] cached hidden states
    float calpha[kMaxFrames];        // cache form: each cached frame's weight alpha
};

// Kernel arguments travel in the kernarg segment: keep them within 4 KB.
static_assert(sizeof(AttnKArgs) <= 4096, "attention kernel arguments exceed 4 KB");

// Forms of the bf16 kernel's key loop.
constexpr int kFormDense = 0;    // all S tokens in order
constexpr int kFormFrames = 1;   // the tokens of the listed frames a.kvf, end to end
constexpr int kFormCache = 2;    // all frames; cached frames give projected keys = values
constexpr int kFormAligned = 3;  // the tokens of the listed frames, in tiles that never cross a frame

// Two floats -> two bf16 (round to nearest even) packed low-first in a word.
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    const bf16x2_t v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ inline bf16x8_t as_bf16x8(u32x4_t w) { return __builtin_bit_cast(bf16x8_t, w); }

// lo + hi of a packed bf16 pair, accumulated in fp32 (v_dot2 against (1, 1)).
__device__ __forceinline__ float add_bf16x2(uint32_t word, float acc) {
    const bf16x2_t one = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, word), one, acc, false);
}

// LDS tile layout. A tile holds kBc keys of one head, K and V each in natural
// [key][dim] order with unpadded rows of 2*D bytes, so that the global->LDS
// loads can write whole 1 KB wave-chunks at consecutive addresses (lane l of a
// load lands at chunk + 16 l). Bank conflicts on the reads are removed by
// permuting the 16-byte slots of each row with an XOR of a key-dependent mask:
//   K: slot = chunk ^ kswz(key) makes the 16 lanes of one 128-bit read pass
//      (16 consecutive keys, same chunk) hit 16 different slot positions of
//      the 256-byte bank window;
//   V: slot = chunk ^ vswz(key) makes the 32 lanes of one transposing 64-bit
//      read pass (4 keys x 64 bytes) hit 8 different 32-byte positions.
template <int D>
struct TileLayout {
    static constexpr int kBc = key_tile(D);            // keys per tile
    static constexpr int kRow = 2 * D;                 // bytes per key row
    static constexpr int kSlots = kRow / 16;           // 16-byte slots per row
    static constexpr int kRowsPerWin = 256 / kRow;     // rows per 256-byte bank window
    static constexpr int kTileBytes = kBc * kRow;
    static constexpr int kRowsPerLoad = 1024 / kRow;   // rows one wave-wide 16-byte load fills
    static constexpr int kLoads = kTileBytes / 1024;   // wave-wide loads per tensor per tile
    __host__ __device__ static constexpr int kswz(int key) { return (key / kRowsPerWin) % kSlots; }
    __host__ __device__ static constexpr int vswz(int key) { return 4 * ((key / kRowsPerWin) % (kSlots / 4)); }
};

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;

// S^T = K Q^T for one tile of kNB 32-key blocks. kofs[kk] is this lane's byte
// offset of its K fragment for reduction step kk inside block 0. The K
// fragments are read through a ring RF_ATTN_K_LEAD fragments ahead of the
// matrix core; the scheduling groups pin that order: LEAD reads, then
// (1 MFMA, 1 read) pairs, then the last LEAD MFMAs.
template <int D, int kNB>
__device__ __forceinline__ void scores_tile(const uint8_t *kb, const int (&kofs)[D / 16],
                                            const u32x4_t (&qf)[D / 16], f32x16_t (&sacc)[kNB]) {
    constexpr int kSteps = D / 16;
    constexpr int kNF = kNB * kSteps;
    constexpr int kLead = RF_ATTN_K_LEAD < kNF ? RF_ATTN_K_LEAD : kNF;
    u32x4_t ring[kLead];
    auto rd = [&](int i) {
        const int b = i / kSteps, kk = i % kSteps;
        return *reinterpret_cast<const u32x4_t *>(kb + kofs[kk] + b * 32 * TileLayout<D>::kRow);
    };
#pragma unroll
    for (int i = 0; i < kLead; ++i) ring[i] = rd(i);
#pragma unroll
    for (int i = 0; i < kNF; ++i) {
        const int b = i / kSteps, kk = i % kSteps;
        const f32x16_t c = kk == 0 ? f32x16_t{} : sacc[b];
        sacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ring[i % kLead]), as_bf16x8(qf[kk]), c,
                                                          0, 0, 0);
        if (i + kLead < kNF) ring[i % kLead] = rd(i + kLead);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, kLead, 0);
#pragma unroll
    for (int i = 0; i < kNF - kLead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kLead, 0);
}

// One A operand of O^T = V^T P^T: dims db*32 + (lane % 32) of the 16 keys
// c*16 .. c*16+15, in the key order of the probability operand (elements 0..3:
// keys c*16 + grp*4 + 0..3, elements 4..7: keys c*16 + 8 + grp*4 + 0..3).
// Each half is one transposing read: the 16 lanes of a group fetch 8 bytes of
// 4 key rows and the hardware redistributes them so lane i receives dim i of
// all four keys.
template <int D>
__device__ __forceinline__ u32x4_t vt_operand(const uint8_t *vb, int vofs, int c) {
    constexpr int kRow = TileLayout<D>::kRow;
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4_t *)(vb + vofs + c * 16 * kRow));
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4_t *)(vb + vofs + (c * 16 + 8) * kRow));
    const u32x2_t l2 = __builtin_bit_cast(u32x2_t, lo), h2 = __builtin_bit_cast(u32x2_t, hi);
    return __builtin_shufflevector(l2, h2, 0, 1, 2, 3);
}

// O^T += V^T P^T for one tile; operands are read RF_ATTN_V_LEAD ahead.
template <int D, int kNB>
__device__ __forceinline__ void pv_tile(const uint8_t *vb, const int (&vofs)[D / 32],
                                        const u32x4_t (&pw)[2 * kNB], f32x16_t (&oacc)[D / 32]) {
    constexpr int kNF = 2 * kNB * (D / 32);
    constexpr int kLead = RF_ATTN_V_LEAD < kNF ? RF_ATTN_V_LEAD : kNF;
    u32x4_t ring[kLead];
    auto rd = [&](int i) {
        const int c = i / (D / 32), db = i % (D / 32);
        return vt_operand<D>(vb, vofs[db], c);
    };
#pragma unroll
    for (int i = 0; i < kLead; ++i) ring[i] = rd(i);
#pragma unroll
    for (int i = 0; i < kNF; ++i) {
        const int c = i / (D / 32), db = i % (D / 32);
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ring[i % kLead]), as_bf16x8(pw[c]),
                                                           oacc[db], 0, 0, 0);
        if (i + kLead < kNF) ring[i % kLead] = rd(i + kLead);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * kLead, 0);
#pragma unroll
    for (int i = 0; i < kNF - kLead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kLead, 0);
}

// The reference of a row's rebased tile (log2 domain): its running maximum so far,
// of which mx is this tile's. Probabilities are exp2(fma(score, scale, -reference)),
// so where the rounding of mx * scale is worth 2^6 and more (from about 2^31 on, where
// the largest score itself would give inf or 0), and where every score is -inf, the
// reference is at least -2^30: such low scores then give 0, and the next tile that
// has an ordinary one rebases the row. A walk over the keys, or a part of one, may
// begin with whole tiles of them.
__device__ __forceinline__ float rebased_reference(float m_run, float mx, float sl2) {
    const float m = mx * sl2, m_new = fmaxf(m_run, m);
    return fabsf(fmaf(mx, sl2, -m)) < 64.0f ? m_new : fmaxf(m_new, -0x1p30f);
}

// Query fragments: B operand of S^T = K Q^T (fused keyframe gather).
template <int D>
__device__ __forceinline__ void load_queries(const AttnKArgs &a, int64_t row, int head, int grp,
                                             u32x4_t (&qf)[D / 16]) {
    if (row < a.Mq) {
        const int64_t f = row / a.N;
        const int64_t tok = static_cast<int64_t>(a.kf[f]) * a.N + (row - f * a.N);
        const uint16_t *qp = a.q + (tok * a.heads + head) * D + grp * 8;
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) qf[kk] = *reinterpret_cast<const u32x4_t *>(qp + kk * 16);
    } else {
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) qf[kk] = u32x4_t{0u, 0u, 0u, 0u};
    }
}

// LDS byte offsets of a lane's K fragment (block 0, step kk) and of its V^T operand halves.
template <int D>
__device__ __forceinline__ void fragment_offsets(int lane, int (&kofs)[D / 16], int (&vofs)[D / 32]) {
    using L = TileLayout<D>;
    const int col = lane & 31, grp = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) kofs[kk] = col * L::kRow + (((2 * kk) ^ grp ^ L::kswz(col)) * 16);
    const int g16 = (lane >> 4) & 1, j = lane & 15;
    const int rr = grp * 4 + j / 4;   // key row within each 8-key half of a 16-key group
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
        vofs[db] = rr * L::kRow + (((2 * db + g16) ^ (L::vswz(rr) / 2)) * 32) + 8 * (j % 4);
}

// Per-tile pipeline, double-buffered LDS, one barrier per tile:
//   issue the global->LDS loads of tile t+1 into the buffer tile t-1 used
//   math on tile t
//   wait for this wave's loads, barrier (tile t+1 visible, tile t released)
// The loads go through raw buffer resources rebased per tile in scalar
// registers whose range ends at the tile's last valid key, so the hardware
// range check zero-fills the keys past it (keys >= S, or past the end of a
// frame in the frame-masked form) and their scores are masked. The loop is
// unrolled by two so every LDS access names its buffer statically.
// kForm: kFormDense, kFormFrames or kFormAligned (the keys are the tokens of the
// frames a.kvf, a frame-level mask) or kFormCache (every frame, cached frames projected).
template <int D, int kForm>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void attn_bf16_kernel(const AttnKArgs a) {
    constexpr bool kKvList = kForm != kFormDense;   // a frame list's tiles
    using L = TileLayout<D>;
    constexpr int kBc = L::kBc;
    constexpr int kNB = kBc / 32;                       // 32-key score blocks per tile
    constexpr int kLoadsPerWave = L::kLoads / kWaves;
    static_assert(L::kLoads % kWaves == 0, "tile loads must split evenly over the waves");

    __shared__ __attribute__((aligned(1024))) uint8_t k0[L::kTileBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t k1[L::kTileBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t v0[L::kTileBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t v1[L::kTileBytes];

    const int bid = blockIdx.x;
    int tile, part = -1;
    if (bid < a.grid_direct) {
        tile = (bid % a.xcds) * a.per_xcd + bid / a.xcds;
        if (tile >= a.total_tiles) return;
    } else {   // a part of a tail tile (tail tiles follow the whole ones in tile order)
        const int u = bid - a.grid_direct;
        const int tt = u / a.split;
        part = u - tt * a.split;
        tile = a.total_tiles + tt;
    }
    const int head = tile / a.n_qtiles;
    const int qt = tile - head * a.n_qtiles;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, grp = lane >> 5;
    const int64_t rs = static_cast<int64_t>(a.heads) * D;   // token stride in elements

    const int64_t row = static_cast<int64_t>(qt) * kBr + wave * 32 + col;
    u32x4_t qf[D / 16];
    load_queries<D>(a, row, head, grp, qf);

    // ---- per-lane offsets, fixed for the whole loop ----
    // global byte offsets (from the tile's first key) of this lane's 16 bytes in each load
    int kgo[kLoadsPerWave], vgo[kLoadsPerWave];
#pragma unroll
    for (int i = 0; i < kLoadsPerWave; ++i) {
        const int key = (wave * kLoadsPerWave + i) * L::kRowsPerLoad + lane / L::kSlots;
        const int slot = lane % L::kSlots;
        kgo[i] = static_cast<int>(key * rs * 2) + (slot ^ L::kswz(key)) * 16;
        vgo[i] = static_cast<int>(key * rs * 2) + (slot ^ L::vswz(key)) * 16;
    }
    int kofs[D / 16], vofs[D / 32];
    fragment_offsets<D>(lane, kofs, vofs);

    f32x16_t oacc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.0f;
    // m_run: reference max (log2 domain) the probabilities are taken against
    // (a past row maximum; see the softmax below).
    float m_run = -__builtin_huge_valf();
    float l_run = 0.0f;   // this lane's partial row sum

    const uint16_t *kbase = a.k + static_cast<int64_t>(head) * D;
    const uint16_t *vbase = a.v + static_cast<int64_t>(head) * D;
    // bytes from a head's first element to one past the last element it owns
    const int64_t head_bytes = ((a.S - 1) * rs + D) * 2;

    // Tile t: its first key's token, the bytes from there to the end of its last
    // valid key, and the number of valid keys (at most kBc).
    // Cache form: slots >= 0 for a tile of a cached frame (before | after << 16),
    // its rows' offset inside the frame and the frame's weight.
    struct Geom {
        int64_t tok0, left;
        int32_t valid;
        int32_t first, delta;   // frame list: ListTile's
        int32_t slots;
        int64_t frame_off;
        float alpha;
    };
    int64_t t_begin = 0, t_end = kKvList ? a.list_tiles : (a.S + kBc - 1) / kBc;
    if (part >= 0) {
        t_begin = static_cast<int64_t>(part) * a.kv_per_split;
        if (t_begin + a.kv_per_split < t_end) t_end = t_begin + a.kv_per_split;
    }
    [[maybe_unused]] auto walker = [&]() {
        if constexpr (kForm == kFormFrames) return ListWalker<kBc, AttnKArgs>(a, t_begin);
        else return 0;
    }();
    auto geom = [&](int64_t t) {
        Geom g;
        g.slots = -1;
        g.frame_off = 0;
        g.alpha = 0.0f;
        if constexpr (kForm == kFormCache) {
            const int32_t m = static_cast<int32_t>(t) / a.tiles_per_frame;
            const int64_t o = (t - static_cast<int64_t>(m) * a.tiles_per_frame) * kBc;
            g.tok0 = static_cast<int64_t>(m) * a.N + o;
            g.slots = a.kvf[m];
            g.frame_off = o;
            g.alpha = a.calpha[m];
            g.valid = static_cast<int32_t>(a.N - o < kBc ? a.N - o : kBc);
            g.left = ((g.valid - 1) * rs + D) * 2;
        } else if constexpr (kForm == kFormAligned) {
            const ListTile l = aligned_tile<kBc>(a, t);
            g.tok0 = l.tok0;
            g.valid = l.valid;
            g.left = ((g.valid - 1) * rs + D) * 2;
        } else if constexpr (kForm == kFormFrames) {
            const ListTile l = walker.take(a, rs);   // (called tile after tile)
            g.tok0 = l.tok0;
            g.valid = l.valid;
            g.first = l.first;
            g.delta = l.delta;
            g.left = ((g.valid - 1) * rs + D) * 2 + l.delta;
        } else {
            g.tok0 = t * kBc;
            g.left = head_bytes - g.tok0 * rs * 2;
            g.valid = static_cast<int32_t>(a.S - g.tok0 < kBc ? a.S - g.tok0 : kBc);
        }
        return g;
    };

    auto issue = [&](const Geom &g, uint8_t *kdst, uint8_t *vdst) {
        // The resources start at the tile's first key; their range ends at its last valid
        // key (clamped to 2^31 - 1: a tile never reaches that far past its first key).
        const int32_t rec = __builtin_amdgcn_readfirstlane(
            static_cast<int32_t>(g.left < 0x7fffffffLL ? g.left : 0x7fffffffLL));
        if constexpr (kForm == kFormCache) {
            if (g.slots >= 0) {
                // a cached frame: h_before into the key buffer, h_after into the value
                // buffer, both in the key layout (project_tile then writes both tiles)
                const uint16_t *hb = a.store + ((g.slots & 0xffff) * a.N + g.frame_off) * rs + head * D;
                const uint16_t *ha = a.store + ((g.slots >> 16) * a.N + g.frame_off) * rs + head * D;
                const __amdgpu_buffer_rsrc_t br =
                    __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(hb), 0, rec, kBufferWord3);
                const __amdgpu_buffer_rsrc_t ar =
                    __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(ha), 0, rec, kBufferWord3);
#pragma unroll
                for (int i = 0; i < kLoadsPerWave; ++i) {
                    const int chunk = (wave * kLoadsPerWave + i) * 1024;
                    load_lds16(br, (lds_void_t *)(kdst + chunk), kgo[i]);
                    load_lds16(ar, (lds_void_t *)(vdst + chunk), kgo[i]);
                }
                return;
            }
        }
        const __amdgpu_buffer_rsrc_t kr =
            __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(kbase + g.tok0 * rs), 0, rec, kBufferWord3);
        const __amdgpu_buffer_rsrc_t vr =
            __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(vbase + g.tok0 * rs), 0, rec, kBufferWord3);
        if constexpr (kForm == kFormFrames) {
            if (g.delta != 0) {
#pragma unroll
                for (int i = 0; i < kLoadsPerWave; ++i) {
                    const int chunk = (wave * kLoadsPerWave + i) * 1024;
                    const int key = (wave * kLoadsPerWave + i) * L::kRowsPerLoad + lane / L::kSlots;
                    const int next = key >= g.first ? g.delta : 0;
                    load_lds16(kr, (lds_void_t *)(kdst + chunk), kgo[i] + next);
                    load_lds16(vr, (lds_void_t *)(vdst + chunk), vgo[i] + next);
                }
                return;
            }
        }
#pragma unroll
        for (int i = 0; i < kLoadsPerWave; ++i) {
            const int chunk = (wave * kLoadsPerWave + i) * 1024;
            load_lds16(kr, (lds_void_t *)(kdst + chunk), kgo[i]);
            load_lds16(vr, (lds_void_t *)(vdst + chunk), vgo[i]);
        }
    };

    // Cache form: the projected state of a cached frame's tile, formed in LDS.
    // The key buffer holds h_before and the value buffer h_after, both in the key
    // layout; each wave owns whole key rows (kBc / 8 of them), reads its rows' 16-byte
    // slots of both, and writes h = fmaf(alpha, h_after, (1 - alpha) h_before),
    // rounded once to bf16, back into the key buffer at the same slot and into the
    // value buffer at the slot the value layout puts it. A wave's LDS instructions
    // run in order and no other wave touches its rows, so its reads see the loaded
    // states before its writes replace them. The caller's barrier then publishes
    // both tiles.
    auto project_tile = [&](uint8_t *kb, uint8_t *vb, float alpha) {
        constexpr int kRowsPerWave = kBc / kWaves;
        constexpr int kPerLane = kRowsPerWave * L::kSlots / 64;
        static_assert(kRowsPerWave * L::kSlots % 64 == 0, "a wave's rows must split evenly over its lanes");
        const float oma = 1.0f - alpha;
        u32x4_t hv[kPerLane];
        int pk[kPerLane], pv[kPerLane];
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            const int sidx = lane * kPerLane + i;
            const int key = wave * kRowsPerWave + sidx / L::kSlots;
            const int slot = sidx % L::kSlots;
            pk[i] = key * L::kRow + (slot ^ L::kswz(key)) * 16;
            pv[i] = key * L::kRow + (slot ^ L::vswz(key)) * 16;
            const u32x4_t b = *reinterpret_cast<const u32x4_t *>(kb + pk[i]);
            const u32x4_t af = *reinterpret_cast<const u32x4_t *>(vb + pk[i]);
            u32x4_t h;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = fmaf(alpha, __uint_as_float(af[e] << 16), oma * __uint_as_float(b[e] << 16));
                const float hi = fmaf(alpha, __uint_as_float(af[e] & 0xffff0000u),
                                      oma * __uint_as_float(b[e] & 0xffff0000u));
                h[e] = pack_bf16x2(lo, hi);
            }
            hv[i] = h;
        }
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
            *reinterpret_cast<u32x4_t *>(kb + pk[i]) = hv[i];
            *reinterpret_cast<u32x4_t *>(vb + pv[i]) = hv[i];
        }
    };
    // after a tile's loads are visible: form the projected tile if the frame is cached
    auto settle_tile = [&](const Geom &g, uint8_t *kb, uint8_t *vb) {
        if constexpr (kForm == kFormCache) {
            if (g.slots >= 0) {
                project_tile(kb, vb, g.alpha);
                __syncthreads();
            }
        }
    };

    const float sl2 = a.scale_log2;
    auto compute = [&](int32_t valid, const uint8_t *kb, const uint8_t *vb) {
        // ---- S^T = K Q^T : 32-key blocks ----
        f32x16_t sacc[kNB];
        scores_tile<D, kNB>(kb, kofs, qf, sacc);
        // accumulator r of block b holds key b*32 + (r/4)*8 + grp*4 + r%4 for query `col`
        if (valid < kBc) {
#pragma unroll
            for (int b = 0; b < kNB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = b * 32 + (r / 4) * 8 + grp * 4 + (r % 4);
                    if (key >= valid) sacc[b][r] = -__builtin_huge_valf();
                }
        }

        // ---- online softmax (log2 domain), reference max moved only when needed ----
        // p = exp2(s * scale - m_run) against the current reference m_run. The
        // reference is a past row maximum, so p may exceed 1; that is harmless (O / l
        // does not depend on the reference and floating-point relative precision does
        // not depend on scale) until p grows large. The row sum bounds every p of the
        // tile, so a row whose tile sum exceeds kRebaseBound takes the exact
        // path: this tile's row maximum becomes the reference, O and l are
        // rescaled and P is recomputed. The first tile (m_run = -inf gives
        // p = inf) always takes it; afterwards it is rare.
        u32x4_t pw[2 * kNB];
        auto probs = [&]() {
            // probabilities, packed as the B operand of O^T = V^T P^T:
            // operand c takes accumulators 8*(c%2) .. 8*(c%2)+7 of block c/2.
            // The row sum adds the bf16-rounded values the matrix core consumes,
            // in four independent partial sums (a single chain of dependent adds
            // would hold up the end of the softmax).
            float lsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int b = 0; b < kNB; ++b)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const float p0 = fast_exp2(fmaf(sacc[b][r], sl2, -m_run));
                    const float p1 = fast_exp2(fmaf(sacc[b][r + 1], sl2, -m_run));
                    const uint32_t word = pack_bf16x2(p0, p1);
                    lsp[(r / 2) % 4] = add_bf16x2(word, lsp[(r / 2) % 4]);
                    pw[b * 2 + r / 8][(r % 8) / 2] = word;
                }
            return ((lsp[0] + lsp[1]) + lsp[2]) + lsp[3];
        };
        float ls = probs();
        // decided per query row (its two lanes agree), so a row's result depends on
        // its own scores only, whichever rows share the wave
        if (!(halves_sum(ls) <= kRebaseBound)) {   // rare; both lanes of a row take it
            float mx = -__builtin_huge_valf();
#pragma unroll
            for (int b = 0; b < kNB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[b][r]);
            const float m_new = rebased_reference(m_run, halves_max(mx), sl2);
            const float corr = fast_exp2(m_run - m_new);   // 0 on the first tile
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= corr;
            ls = probs();
        }
        l_run += ls;

        // ---- O^T += V^T P^T ----
        pv_tile<D, kNB>(vb, vofs, pw, oacc);
    };
    auto tile_done = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads have reached LDS
        __syncthreads();
    };

    Geom cur = geom(t_begin);
    issue(cur, k0, v0);
    tile_done();
    settle_tile(cur, k0, v0);
    for (int64_t t = t_begin; t < t_end; t += 2) {
        Geom nxt = cur;
        if (t + 1 < t_end) {
            nxt = geom(t + 1);
            issue(nxt, k1, v1);
        }
        compute(cur.valid, k0, v0);
        tile_done();
        if (t + 1 >= t_end) break;
        // (a projected tile is formed while no load is in flight, so its barrier
        // waits for nothing but the projection itself)
        settle_tile(nxt, k1, v1);
        if (t + 2 < t_end) {
            cur = geom(t + 2);
            issue(cur, k0, v0);
        }
        compute(nxt.valid, k1, v1);
        tile_done();
        if (t + 2 < t_end) settle_tile(cur, k0, v0);
    }

    l_run = halves_sum(l_run);
    if (part >= 0) {
        // ---- a part of a tail tile: unnormalised O and (m, l) for the combine kernel ----
        if (row < a.Mq) {
            const int64_t slot = static_cast<int64_t>(tile - a.total_tiles) * a.split + part;
            const int64_t r = slot * kBr + wave * 32 + col;
            float *po = a.ws_o + r * D;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const int rr = g4 * 4;
                    *reinterpret_cast<f32x4_t *>(po + db * 32 + g4 * 8 + grp * 4) =
                        f32x4_t{oacc[db][rr], oacc[db][rr + 1], oacc[db][rr + 2], oacc[db][rr + 3]};
                }
            if (grp == 0) *reinterpret_cast<f32x2_t *>(a.ws_ml + r * 2) = f32x2_t{m_run, l_run};
        }
        return;
    }

    // ---- epilogue: normalise, round to bf16, store the compact row ----
    if (row < a.Mq) {
        const float inv = 1.0f / l_run;
        uint16_t *op = a.out + row * rs + static_cast<int64_t>(head) * D;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                // accumulator r holds dimension db*32 + (r/4)*8 + grp*4 + r%4
                const int r = g4 * 4;
                const u32x2_t w = {pack_bf16x2(oacc[db][r] * inv, oacc[db][r + 1] * inv),
                                   pack_bf16x2(oacc[db][r + 2] * inv, oacc[db][r + 3] * inv)};
                *reinterpret_cast<u32x2_t *>(op + db * 32 + g4 * 8 + grp * 4) = w;
            }
    }
}

// ---------------------------------------------------------------------------
// Small launches: a workgroup owns 32 query rows of one head and its 8 waves
// share out the keys, wave w taking tiles w, w + 8, ...; the parts are merged
// through LDS at the end. Each wave streams its tiles into LDS of its own (one K
// and one V buffer: the next K is fetched while this tile's softmax and second
// product run, the next V under the next tile's scores), so the loop has no
// barrier and no second kernel follows.
// What bounds it: a CU reads K and V once per 32 rows instead of once per 256,
// 32 FLOP per byte through its L1, which is half of what the matrix cores could
// take; a launch that leaves most CUs idle in 256-row tiles has that to spare.
// Kernel and combine against this one: 9 frames of 17 x 31, 5 heads x 64, three
// keyframes 31.1 -> 19.0 us (504 TFLOP/s); 13 of 16 x 16, 8 x 64, four 27.1 ->
// 15.6; 9 of 10 x 13, 3 x 128, three 24.5 -> 11.5. 182 vector registers at head
// dimension 128, 166 at 64, where the compiler also spills 6 scalar registers (14
// with a frame list) to vector lanes.
// ---------------------------------------------------------------------------

constexpr int kSmallRows = 32;
// 8 KB of K and of V a tile at either head dimension: 128 KB of LDS
__host__ __device__ constexpr int small_key_tile(int head_dim) { return head_dim == 64 ? 64 : 32; }

// The softmax of attn_bf16_kernel's tiles (there it stays inside the kernel: called
// as this function, the compiler's schedule of its head dimension 64 form loses
// 4 %, 1001 against 1040 TFLOP/s).
template <int D, int kNB>
__device__ __forceinline__ void softmax_tile(f32x16_t (&sacc)[kNB], int32_t valid, int grp, float sl2, float &m_run,
                                             float &l_run, f32x16_t (&oacc)[D / 32], u32x4_t (&pw)[2 * kNB]) {
    if (valid < 32 * kNB) {
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (b * 32 + (r / 4) * 8 + grp * 4 + r % 4 >= valid) sacc[b][r] = -__builtin_huge_valf();
    }
    auto probs = [&]() {
        float lsp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = fast_exp2(fmaf(sacc[b][r], sl2, -m_run));
                const float p1 = fast_exp2(fmaf(sacc[b][r + 1], sl2, -m_run));
                const uint32_t word = pack_bf16x2(p0, p1);
                lsp[(r / 2) % 4] = add_bf16x2(word, lsp[(r / 2) % 4]);
                pw[b * 2 + r / 8][(r % 8) / 2] = word;
            }
        return ((lsp[0] + lsp[1]) + lsp[2]) + lsp[3];
    };
    float ls = probs();
    if (!(halves_sum(ls) <= kRebaseBound)) {
        float mx = -__builtin_huge_valf();
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[b][r]);
        const float m_new = rebased_reference(m_run, halves_max(mx), sl2);
        const float corr = fast_exp2(m_run - m_new);
        m_run = m_new;
        l_run *= corr;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= corr;
        ls = probs();
    }
    l_run += ls;
}

template <int D, bool kFrames>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void attn_bf16_small_kernel(const AttnKArgs a) {
    using L = TileLayout<D>;
    constexpr int kBc = small_key_tile(D);
    constexpr int kNB = kBc / 32;
    constexpr int kTileBytes = kBc * L::kRow;
    constexpr int kLoads = kTileBytes / 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t ks[kWaves * kTileBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t vs[kWaves * kTileBytes];
    __shared__ float ml[kWaves][kSmallRows][2];

    const int bid = blockIdx.x;
    const int tile = (bid % a.xcds) * a.per_xcd + bid / a.xcds;
    if (tile >= a.total_tiles) return;
    const int head = tile / a.n_qtiles;
    const int qt = tile - head * a.n_qtiles;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, grp = lane >> 5;
    const int64_t rs = static_cast<int64_t>(a.heads) * D;
    uint8_t *kb = ks + wave * kTileBytes;
    uint8_t *vb = vs + wave * kTileBytes;

    u32x4_t qf[D / 16];
    load_queries<D>(a, static_cast<int64_t>(qt) * kSmallRows + col, head, grp, qf);
    int kofs[D / 16], vofs[D / 32];
    fragment_offsets<D>(lane, kofs, vofs);
    int kgo[kLoads], vgo[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int key = i * L::kRowsPerLoad + lane / L::kSlots;
        const int slot = lane % L::kSlots;
        kgo[i] = static_cast<int>(key * rs * 2) + (slot ^ L::kswz(key)) * 16;
        vgo[i] = static_cast<int>(key * rs * 2) + (slot ^ L::vswz(key)) * 16;
    }
    f32x16_t oacc[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.0f;
    float m_run = -__builtin_huge_valf(), l_run = 0.0f;

    struct Geom {
        int64_t tok0;
        int32_t valid;
    };
    auto geom = [&](int64_t t) {
        Geom g;
        int64_t left;
        if constexpr (kFrames) {
            const int32_t m = static_cast<int32_t>(t) / a.tiles_per_frame;
            const int64_t o = (t - static_cast<int64_t>(m) * a.tiles_per_frame) * kBc;
            g.tok0 = static_cast<int64_t>(a.kvf[m]) * a.N + o;
            left = a.N - o;
        } else {
            g.tok0 = t * kBc;
            left = a.S - g.tok0;
        }
        g.valid = static_cast<int32_t>(left < kBc ? left : kBc);
        return g;
    };
    // the resource starts at the tile's first key and ends at its last valid one
    auto issue = [&](const Geom &g, const uint16_t *tensor, const int (&go)[kLoads], uint8_t *dst) {
        const int32_t rec = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(((g.valid - 1) * rs + D) * 2));
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            uniform_ptr(tensor + g.tok0 * rs + static_cast<int64_t>(head) * D), 0, rec, kBufferWord3);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) load_lds16(r, (lds_void_t *)(dst + i * 1024), go[i]);
    };

    const int64_t n = kFrames ? a.list_tiles : (a.S + kBc - 1) / kBc;
    if (wave < n) {
        Geom g = geom(wave);
        issue(g, a.k, kgo, kb);
        issue(g, a.v, vgo, vb);
        for (int64_t t = wave; t < n; t += kWaves) {
            // (past the last tile it is fetched again and not used: with the loads on every
            // path the waits below can be counted instead of draining both tensors)
            const Geom nxt = geom(t + kWaves < n ? t + kWaves : t);
            wait_loads<kLoads>();   // K is there; V may still be in flight
            f32x16_t sacc[kNB];
            scores_tile<D, kNB>(kb, kofs, qf, sacc);
            wait_lds_reads();       // K is read: its buffer is free
            issue(nxt, a.k, kgo, kb);
            u32x4_t pw[2 * kNB];
            softmax_tile<D, kNB>(sacc, g.valid, grp, a.scale_log2, m_run, l_run, oacc, pw);
            wait_loads<kLoads>();   // V is there; the next K may still be in flight
            pv_tile<D, kNB>(vb, vofs, pw, oacc);
            wait_lds_reads();
            issue(nxt, a.v, vgo, vb);
            g = nxt;
        }
        wait_loads<0>();   // nothing lands in the buffers any more
    }

    // ---- merge: dimensions 0..63 of a wave's O rows go into its own K buffer, 64..127
    // into its V buffer, 256 bytes a row, their 16-byte units permuted by row % 16 ----
    const float l = halves_sum(l_run);
    if (grp == 0) {
        ml[wave][col][0] = m_run;
        ml[wave][col][1] = l;
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const int unit = ((db % 2) * 8 + g4 * 2 + grp) ^ (col & 15);
            *reinterpret_cast<f32x4_t *>((db < 2 ? kb : vb) + col * 256 + unit * 16) =
                f32x4_t{oacc[db][g4 * 4], oacc[db][g4 * 4 + 1], oacc[db][g4 * 4 + 2], oacc[db][g4 * 4 + 3]};
        }
    __syncthreads();
    const int r = tid / 16, unit = tid % 16;   // 512 threads: 32 rows x 16 units
    const int64_t row = static_cast<int64_t>(qt) * kSmallRows + r;
    if (row >= a.Mq) return;
    float m = ml[0][r][0];
#pragma unroll
    for (int p = 1; p < kWaves; ++p) m = fmaxf(m, ml[p][r][0]);
    float wgt[kWaves], lsum = 0.0f;
#pragma unroll
    for (int p = 0; p < kWaves; ++p) {
        wgt[p] = fast_exp2(ml[p][r][0] - m);
        lsum = fmaf(wgt[p], ml[p][r][1], lsum);
    }
    const float inv = 1.0f / lsum;
    uint16_t *op = a.out + row * rs + static_cast<int64_t>(head) * D + unit * 4;
#pragma unroll
    for (int half = 0; half < D / 64; ++half) {
        f32x4_t x = {};
#pragma unroll
        for (int p = 0; p < kWaves; ++p) {
            const f32x4_t y = *reinterpret_cast<const f32x4_t *>((half == 0 ? ks : vs) + p * kTileBytes + r * 256 +
                                                                 (unit ^ (r & 15)) * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = fmaf(wgt[p], y[e], x[e]);
        }
        const u32x2_t w = {pack_bf16x2(x[0] * inv, x[1] * inv), pack_bf16x2(x[2] * inv, x[3] * inv)};
        *reinterpret_cast<u32x2_t *>(op + half * 64) = w;
    }
}

// ---------------------------------------------------------------------------
// Combine of the split tail: for each row of a tail tile, the parts' reference
// maxima m_p (log2 domain), row sums l_p and unnormalised outputs O_p give
//   m = max_p m_p,  out = sum_p 2^(m_p - m) O_p / sum_p 2^(m_p - m) l_p,
// rounded to bf16. Each thread owns 8 output dimensions of one row.
// ---------------------------------------------------------------------------

struct CombineArgs {
    const float *ws_o;
    const float *ws_ml;
    uint16_t *out;
    int64_t Mq;
    int32_t heads;
    int32_t n_qtiles;
    int32_t first_tail;   // tile index of the first tail tile
    int32_t split;
};

constexpr int kCombineThreads = 256;

template <int D>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(const CombineArgs a) {
    constexpr int kTpr = D / 8;                       // threads per row
    constexpr int kRows = kCombineThreads / kTpr;     // rows per workgroup
    constexpr int kGroups = kBr / kRows;              // workgroups per tail tile
    const int tt = blockIdx.x / kGroups;
    const int r = (blockIdx.x - tt * kGroups) * kRows + threadIdx.x / kTpr;
    const int c8 = threadIdx.x % kTpr;
    const int tile = a.first_tail + tt;
    const int head = tile / a.n_qtiles;
    const int qt = tile - head * a.n_qtiles;
    const int64_t row = static_cast<int64_t>(qt) * kBr + r;
    if (row >= a.Mq) return;
    const int64_t base = static_cast<int64_t>(tt) * a.split * kBr + r;   // slot of part 0 of this row
    float m = -__builtin_huge_valf();
    for (int p = 0; p < a.split; ++p) m = fmaxf(m, a.ws_ml[(base + static_cast<int64_t>(p) * kBr) * 2]);
    float l = 0.0f, o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.0f;
    for (int p = 0; p < a.split; ++p) {
        const int64_t slot = base + static_cast<int64_t>(p) * kBr;
        const f32x2_t ml = *reinterpret_cast<const f32x2_t *>(a.ws_ml + slot * 2);
        const float wgt = fast_exp2(ml[0] - m);
        l = fmaf(wgt, ml[1], l);
        const f32x4_t *po = reinterpret_cast<const f32x4_t *>(a.ws_o + slot * D + c8 * 8);
        const f32x4_t x0 = po[0], x1 = po[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = fmaf(wgt, x0[e], o[e]);
            o[e + 4] = fmaf(wgt, x1[e], o[e + 4]);
        }
    }
    const float inv = 1.0f / l;
    const int64_t rs = static_cast<int64_t>(a.heads) * D;
    const u32x4_t w = {pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv),
                       pack_bf16x2(o[4] * inv, o[5] * inv), pack_bf16x2(o[6] * inv, o[7] * inv)};
    *reinterpret_cast<u32x4_t *>(a.out + row * rs + static_cast<int64_t>(head) * D + c8 * 8) = w;
}

}  // namespace

hipError_t device_geometry(DeviceGeometry *out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<int64_t> cached[kMaxDevices];   // (cus << 32 | xcds), 0 until queried
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int64_t v = cached[dev].load(std::memory_order_relaxed);
    if (v == 0) {
        int cus = 0, xcds = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipDeviceGetAttribute(&xcds, hipDeviceAttributeNumberOfXccs, dev);
        if (e != hipSuccess || xcds < 1) xcds = 1;   // no XCD count reported: one L2 domain
        if (cus < 1) return hipErrorInvalidDevice;
        if (xcds > cus) xcds = cus;
        v = (static_cast<int64_t>(cus) << 32) | static_cast<uint32_t>(xcds);
        cached[dev].store(v, std::memory_order_relaxed);
    }
    out->cus = static_cast<int32_t>(v >> 32);
    out->xcds = static_cast<int32_t>(v & 0xffffffff);
    return hipSuccess;
}

AttnSplit attention_split(int64_t Mq, int32_t heads, int32_t head_dim, int64_t N, int64_t S, int32_t n_kv,
                          int32_t cus, int32_t walk_frames) {
    AttnSplit sp{};
    const int64_t total = (Mq + kBr - 1) / kBr * heads;
    const int64_t kBc = key_tile(head_dim);
    const int64_t kv_tiles = n_kv > 0 ? static_cast<int64_t>(n_kv) * ((N + kBc - 1) / kBc) : (S + kBc - 1) / kBc;
    const int64_t tail = total % cus;
    sp.n_tiles = total;
    sp.n_direct = total;
    if (tail == 0) return sp;
    // tail time in rounds of whole tiles for s parts: ceil(tail * s / CUs) / s
    int best_s = 1;
    double best = 1.0;
    for (int s = 2; s <= kMaxSplit && kv_tiles / s >= kMinKvPerSplit; ++s) {
        const double cost = static_cast<double>((tail * s + cus - 1) / cus) / s;
        if (cost < best - 1e-9) {
            best = cost;
            best_s = s;
        }
    }
    if (best_s == 1) return sp;
    sp.n_direct = total - tail;
    sp.n_tail = tail;
    sp.split = best_s;
    // (the cache form's frame-aligned walk has at least kv_tiles tiles: its parts keep kMinKvPerSplit)
    const int64_t walk = walk_frames > 0 ? static_cast<int64_t>(walk_frames) * ((N + kBc - 1) / kBc) : kv_tiles;
    sp.kv_per_split = (walk + best_s - 1) / best_s;
    sp.ws_bytes = tail * best_s * kBr * (static_cast<int64_t>(head_dim) * 4 + 8);
    return sp;
}

// Whether the small kernel ends earlier than whole tiles and a split tail, by their
// times in us, counted in rounds of the device: a round of whole tiles has a fixed
// part, which grows with the rows that its tiles hold, and the time of each key tile
// walked; a split has a second kernel and the parts' results, written and read again;
// a round of small tiles has a fixed part and the tiles of its busiest wave. The
// counts are fitted to the times of both at 4,300 drawn launches (1 to 33 frames of up
// to 2,048 tokens, 1 to 48 heads, dense and frame lists, most of them ragged; rms
// error 7-8 %), and the small kernel has to come out 7 % shorter: of 2,681 that then
// take it six are behind by more than 4 % (9 at most; without the fixed parts 314
// were, by up to 94 %), and the choice loses 0.6 % to the better of the two on average.
// Whole tiles against small ones, us:
//   9 frames of 17 x 31, 5 x 128, three keyframes (35 in sevenths; 250)   37.3   32.7
//   21 of 16 x 16, 12 x 64, five (60 in quarters; 480)                    34.5   36.9
//   13 of 16 x 16, 12 x 128, four (48 in fifths; 384)                     36.8   43.9
//   3 of 22 x 13, 31 x 64, two (93; 558)                                  19.6   20.6
//   5 of 10 x 14, 43 x 128, four (129; 774 in four rounds)                25.1   34.9
//   one listed of 2 of 21 x 47, 40 x 64, one (160; 1,240 in five)         22.8   33.6
struct SmallCost {
    double round, rows, tile;                // whole tiles: a round, the more of it at full rows, a key tile
    double split, parts;                     // a split: the second kernel, 256 parts' results
    double small, small_round, small_tile;   // small tiles: the launch's difference, a round, a wave's key tile
};
constexpr SmallCost kSmallCost64{4.4, 2.1, 1.90, 2.9, 4.9, 1.0, 3.3, 1.30};
constexpr SmallCost kSmallCost128{4.1, 4.8, 1.50, 1.9, 9.5, 0.4, 4.6, 1.25};
constexpr double kSmallShorter = 0.93;

bool small_pays(const AttnSplit &sp, int64_t Mq, int32_t heads, int32_t head_dim, int64_t key_tiles,
                int64_t small_key_tiles, int32_t cus) {
    const SmallCost &c = head_dim == 64 ? kSmallCost64 : kSmallCost128;
    const int64_t parts = sp.n_tail * sp.split;
    const double rounds = static_cast<double>((sp.n_direct + cus - 1) / cus);
    const double part_rounds = static_cast<double>((parts + cus - 1) / cus);
    const double walks = rounds + (sp.split > 0 ? part_rounds / sp.split : 0.0);   // of all keys
    const double rows = Mq < kBr ? static_cast<double>(Mq) / kBr : 1.0;            // of a tile's
    const double whole = (rounds + part_rounds) * (c.round + c.rows * rows) + walks * key_tiles * c.tile +
                         (sp.split > 0 ? c.split + c.parts * parts / 256 : 0.0);
    const int64_t small_tiles = (Mq + kSmallRows - 1) / kSmallRows * heads;
    const double small_rounds = static_cast<double>((small_tiles + cus - 1) / cus);
    const double wave_tiles = static_cast<double>((small_key_tiles + kWaves - 1) / kWaves);
    return c.small + small_rounds * (c.small_round + c.small_tile * wave_tiles) < kSmallShorter * whole;
}

// End to end (no partial tile but the last) where that saves a tile, a tile meets at
// most two frames, all offsets inside a tile fit 32 bits, and `split` equal parts are
// all non-empty. 6 frames of 30 x 52, 12 x 128: 147 tiles of 64 instead of 150, 489 ->
// 480 us; 5 of 30 x 52, 24 x 64: 417 -> 388; 11 of 10 x 13, 24 x 64: 55.5 -> 42.7.
// Where it saves none the walk alone costs 1-2 %: 10 of 16 x 16, 24 x 64, without
// splitting: 43.8 us aligned, 44.5 end to end; 3 of 64 x 64, 4 x 128: 272, 275.5; one
// of 1 x 22, 31 x 128: 5.8, 6.0.
// The small kernel keeps to frames: its waves take every eighth tile, and finding
// one by division costs it 3-5 % where no tile is saved.
ListWalk list_walk(const AttnParams &p, int64_t bc, int64_t split) {
    const int64_t per_frame = (p.N + bc - 1) / bc, token = static_cast<int64_t>(p.heads) * p.head_dim * 2;
    const ListWalk aligned{per_frame, p.n_kv * per_frame};
    if (p.N < bc || p.N > 0x3fffffffLL / p.n_kv) return aligned;
    int64_t gap = 0;
    for (int i = 0; i + 1 < p.n_kv; ++i) gap = p.kvf[i + 1] - p.kvf[i] - 1 > gap ? p.kvf[i + 1] - p.kvf[i] - 1 : gap;
    if ((gap * p.N + bc) * token > 0x7fffffffLL) return aligned;
    const int64_t tiles = (p.n_kv * p.N + bc - 1) / bc;
    if (tiles == aligned.tiles) return aligned;
    if (split > 0 && tiles <= (split - 1) * (split - 1)) return aligned;
    return ListWalk{0, tiles};
}

bool attention_shares_keys(const AttnParams &p, const AttnSplit &sp) {
    const int64_t Mq = static_cast<int64_t>(p.M) * p.N;
    if (p.cache_form) return false;
    if (p.dtype == RF_F32) return f32_split_pays(Mq, p.heads, p.geo.cus);
    const int64_t bc = key_tile(p.head_dim), bc_small = small_key_tile(p.head_dim);
    const int64_t small_tiles =
        p.n_kv > 0 ? p.n_kv * ((p.N + bc_small - 1) / bc_small) : (p.S + bc_small - 1) / bc_small;
    const int64_t tiles = p.n_kv > 0 ? list_walk(p, bc, sp.split).tiles : (p.S + bc - 1) / bc;
    return small_pays(sp, Mq, p.heads, p.head_dim, tiles, small_tiles, p.geo.cus);
}

hipError_t launch_attention(const AttnParams &p, hipStream_t stream) {
    const int64_t Mq = static_cast<int64_t>(p.M) * p.N;
    if (p.dtype == RF_F32) return launch_attention_f32(p, stream);
    AttnKArgs a{};
    a.q = static_cast<const uint16_t *>(p.q);
    a.k = static_cast<const uint16_t *>(p.k);
    a.v = static_cast<const uint16_t *>(p.v);
    a.out = static_cast<uint16_t *>(p.out);
    a.S = p.S;
    a.N = p.N;
    a.Mq = Mq;
    a.heads = p.heads;
    const int64_t nq = (Mq + kBr - 1) / kBr;
    const int32_t xcds = p.geo.xcds;
    if (p.geo.cus < 1 || xcds < 1 || xcds > 64) return hipErrorInvalidValue;
    AttnSplit sp{};
    sp.n_direct = nq * p.heads;
    const int32_t walk = p.cache_form ? static_cast<int32_t>(p.S / p.N) : 0;
    if (p.ws) {
        sp = attention_split(Mq, p.heads, p.head_dim, p.N, p.S, p.n_kv, p.geo.cus, walk);
        if (sp.split > 0 && p.ws_bytes < sp.ws_bytes) return hipErrorInvalidValue;
    }
    const bool small = p.split_keys && attention_shares_keys(p, sp);
    if (small) {
        sp = AttnSplit{};
        sp.n_direct = (Mq + kSmallRows - 1) / kSmallRows * p.heads;
    }
    const int64_t total = sp.n_direct;
    const int64_t per_xcd = (total + xcds - 1) / xcds;
    if (nq * p.heads > 0x7fffffffLL / 64) return hipErrorInvalidConfiguration;
    // per-lane load offsets inside a tile are 32-bit: a whole launch's tile must span < 2 GiB of
    // token rows (a small launch's tile is half of it, but what is refused does not depend on the form)
    if (static_cast<int64_t>(p.heads) * p.head_dim * 2 * key_tile(p.head_dim) >= 0x7fffffffLL)
        return hipErrorInvalidConfiguration;
    const int64_t kBc = small ? small_key_tile(p.head_dim) : key_tile(p.head_dim);
    a.n_qtiles = static_cast<int32_t>(small ? (Mq + kSmallRows - 1) / kSmallRows : nq);
    a.total_tiles = static_cast<int32_t>(total);
    a.per_xcd = static_cast<int32_t>(per_xcd);
    a.xcds = xcds;
    a.grid_direct = static_cast<int32_t>(per_xcd * xcds);
    a.split = static_cast<int32_t>(sp.split);
    a.kv_per_split = static_cast<int32_t>(sp.kv_per_split);
    const int64_t n_parts = sp.n_tail * sp.split;
    if (sp.split > 0) {
        a.ws_o = static_cast<float *>(p.ws);
        a.ws_ml = a.ws_o + n_parts * kBr * p.head_dim;
    }
    a.scale_log2 = static_cast<float>(1.4426950408889634 / sqrt(static_cast<double>(p.head_dim)));
    for (int i = 0; i < p.M; ++i) a.kf[i] = p.kf[i];
    a.n_kv = p.n_kv;
    for (int i = 0; i < p.n_kv; ++i) a.kvf[i] = p.kvf[i];
    ListWalk lw{(p.N + kBc - 1) / kBc, walk * ((p.N + kBc - 1) / kBc)};
    if (p.n_kv > 0 && small) {
        lw.tiles = p.n_kv * lw.per_frame;
    } else if (p.n_kv > 0) {
        lw = list_walk(p, kBc, sp.split);
        if (sp.split > 0) a.kv_per_split = static_cast<int32_t>((lw.tiles + sp.split - 1) / sp.split);
    }
    if ((p.n_kv > 0 || p.cache_form) && lw.tiles > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.tiles_per_frame = static_cast<int32_t>(lw.per_frame);
    a.list_tiles = static_cast<int32_t>(lw.tiles);
    if (p.cache_form) {
        a.n_kv = walk;
        for (int i = 0; i < walk; ++i) {
            a.kvf[i] = p.cslot[i];
            a.calpha[i] = p.calpha[i];
        }
        a.store = static_cast<const uint16_t *>(p.store);
    }
    const dim3 grid(static_cast<uint32_t>(per_xcd * xcds + n_parts)), block(kThreads);
    if (small) {
        const bool frames = p.n_kv > 0;
        if (p.head_dim == 128 && frames) hipLaunchKernelGGL((attn_bf16_small_kernel<128, true>), grid, block, 0, stream, a);
        else if (p.head_dim == 128) hipLaunchKernelGGL((attn_bf16_small_kernel<128, false>), grid, block, 0, stream, a);
        else if (frames) hipLaunchKernelGGL((attn_bf16_small_kernel<64, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_bf16_small_kernel<64, false>), grid, block, 0, stream, a);
    } else if (p.cache_form) {
        if (p.head_dim == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, kFormCache>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, kFormCache>), grid, block, 0, stream, a);
    } else if (p.n_kv > 0 && a.tiles_per_frame > 0) {
        if (p.head_dim == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, kFormAligned>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, kFormAligned>), grid, block, 0, stream, a);
    } else if (p.n_kv > 0) {
        if (p.head_dim == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, kFormFrames>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, kFormFrames>), grid, block, 0, stream, a);
    } else {
        if (p.head_dim == 128) hipLaunchKernelGGL((attn_bf16_kernel<128, kFormDense>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_bf16_kernel<64, kFormDense>), grid, block, 0, stream, a);
    }
    if (sp.split == 0) return hipGetLastError();
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    CombineArgs c{};
    c.ws_o = a.ws_o;
    c.ws_ml = a.ws_ml;
    c.out = a.out;
    c.Mq = Mq;
    c.heads = p.heads;
    c.n_qtiles = a.n_qtiles;
    c.first_tail = a.total_tiles;
    c.split = a.split;
    const int rows_per_wg = kCombineThreads / (p.head_dim / 8);
    const dim3 cgrid(static_cast<uint32_t>(sp.n_tail * (kBr / rows_per_wg))), cblock(kCombineThreads);
    if (p.head_dim == 128) hipLaunchKernelGGL(attn_combine_kernel<128>, cgrid, cblock, 0, stream, c);
    else hipLaunchKernelGGL(attn_combine_kernel<64>, cgrid, cblock, 0, stream, c);
    return hipGetLastError();
}

}  // namespace rf
