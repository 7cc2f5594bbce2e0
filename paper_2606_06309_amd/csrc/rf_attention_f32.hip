// fp32 keyframe-query attention for gfx950: fp32 inputs, products, sums and
// outputs throughout, on the fp32 matrix instructions.
//
// What bounds it: the fp32 matrix cores (157 TFLOP/s, 154 in a large library
// product on the same card; a wave's v_mfma_f32_32x32x2_f32 takes 64 cycles and
// one 4-byte operand per lane, so a 16-byte LDS read feeds four of them and
// neither LDS, the vector pipe nor memory is near its limit). 5 keyframes of 13
// frames of 30 x 52 tokens, 12 heads x 128: 7.34 ms = 132 TFLOP/s, where two
// lanes per row and vector fused multiply-adds took 57.6 ms (16.9 TFLOP/s); its
// 732 workgroups make 2.86 rounds of the compute units, 95 % of three.
//
// Common to both kernels:
//  * Scores are computed transposed, S^T = K Q^T, 32 keys x 32 query rows at a
//    time: K rows from LDS are the A operand, the wave's query rows (held in
//    registers) the B operand. Lane l holds query column l % 32; lanes l and
//    l ^ 32 share it and hold 16 of the 32 scores each, in the order key =
//    (r / 4) * 8 + (l / 32) * 4 + r % 4.
//  * That is the B operand of O^T = V^T P^T as it stands: step r of the second
//    product takes accumulator r, whose two half-waves hold two different keys,
//    and the V rows of the same two keys. The dimension a row of O^T stands for
//    may be chosen freely, so lane i takes dimensions i * D/32 .. + D/32 - 1 and
//    one wide LDS read of a V row feeds all D/32 products of a step.
//  * K and V tiles go from memory straight into LDS (buffer loads with an LDS
//    destination), V in natural order, the 16-byte slots of a K row permuted by
//    key % 16 so that the 16 lanes of a read pass hit 16 different slots. The
//    buffer resource's range ends at the tile's last valid key: keys past it
//    read as zero and their scores are masked.
//  * Online softmax against the exact running row maximum, subtracted before
//    the scale so that the largest score gives exactly 1.
//
// attn_f32_tile_kernel: a workgroup of 4 waves owns 128 query rows, the waves
// share double-buffered tiles (64 KB of LDS), two workgroups per compute unit.
// A row meets the same keys in the same order whichever launch it is part of.
//
// attn_f32_split_kernel (calls that allow a split): a workgroup owns 32 query
// rows and its waves share out the key tiles among themselves: wave w takes
// tiles w, w + kParts, ...; the parts are merged through LDS at the end. Each
// wave streams its tiles into LDS of its own (one K and one V buffer: the next
// K is fetched while this tile's softmax and second product run, the next V
// under the next tile's scores), so the loop has no barrier. Small launches
// then fill four times as many compute units.
#include "rf_device.h"

namespace rf {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct AttnF32Args {
    const float *q;
    const float *k;
    const float *v;
    float *out;
    int64_t S;
    int64_t N;
    int64_t Mq;
    int32_t heads;
    int32_t n_qtiles;
    int32_t total_tiles;
    int32_t per_xcd;
    int32_t xcds;              // XCDs of the device: workgroup id i runs on XCD i % xcds
    float scale_log2;          // log2(e) / sqrt(d)
    int32_t kf[kMaxFrames];
    // > 0: the keys are the tokens of frames kvf[0..n_kv), walked frame by frame
    // in tiles that never cross a frame
    int32_t n_kv;
    int32_t tiles_per_frame;
    int32_t kvf[kMaxFrames];
};

// An LDS tile of kKeys keys of one head: K and V each [key][dim], 4 * D bytes a row.
template <int D, int kKeys>
struct F32Tile {
    static constexpr int kRow = 4 * D;
    static constexpr int kSlots = kRow / 16;
    static constexpr int kBytes = kKeys * kRow;
    static constexpr int kRowsPerLoad = 1024 / kRow;   // rows one wave-wide 16-byte load fills
    static constexpr int kLoads = kBytes / 1024;       // wave-wide loads per tensor
};

// One wave's state: 32 query rows, their running softmax and O^T.
template <int D>
struct F32Wave {
    static constexpr int kDb = D / 32;      // 32-row blocks of O^T, and floats per V read
    f32x4_t qf[D / 8];
    f32x16_t o[kDb];
    float m;      // running row maximum of the raw scores
    float l;      // this lane's part of the row sum
};

template <int D>
__device__ __forceinline__ void load_queries(const AttnF32Args &a, int64_t row, int head, int grp, F32Wave<D> &w) {
    if (row < a.Mq) {
        const int64_t f = row / a.N;
        const int64_t tok = static_cast<int64_t>(a.kf[f]) * a.N + (row - f * a.N);
        const float *qp = a.q + (tok * a.heads + head) * D + grp * 4;
#pragma unroll
        for (int c = 0; c < D / 8; ++c) w.qf[c] = *reinterpret_cast<const f32x4_t *>(qp + c * 8);
    } else {
#pragma unroll
        for (int c = 0; c < D / 8; ++c) w.qf[c] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int db = 0; db < F32Wave<D>::kDb; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) w.o[db][r] = 0.0f;
    w.m = -__builtin_huge_valf();
    w.l = 0.0f;
}

// First token and number of valid keys of tile t (at most kKeys).
struct F32Geom {
    int64_t tok0;
    int32_t valid;
};
template <int kKeys>
__device__ __forceinline__ F32Geom tile_geom(const AttnF32Args &a, int64_t t) {
    F32Geom g;
    int64_t left;
    if (a.n_kv > 0) {
        const int32_t m = static_cast<int32_t>(t) / a.tiles_per_frame;
        const int64_t o = (t - static_cast<int64_t>(m) * a.tiles_per_frame) * kKeys;
        g.tok0 = static_cast<int64_t>(a.kvf[m]) * a.N + o;
        left = a.N - o;
    } else {
        g.tok0 = t * kKeys;
        left = a.S - g.tok0;
    }
    g.valid = static_cast<int32_t>(left < kKeys ? left : kKeys);
    return g;
}

// Loads i0 .. i0 + kN - 1 of a tile into LDS: load i fills kRowsPerLoad rows at dst + 1024 i.
template <int D, int kKeys, bool kSwizzle, int kN>
__device__ __forceinline__ void issue_rows(const AttnF32Args &a, const float *tensor, int head, const F32Geom &g,
                                           uint8_t *dst, int i0, int lane) {
    using L = F32Tile<D, kKeys>;
    const int64_t rs = static_cast<int64_t>(a.heads) * D;   // token stride in elements
    // the resource starts at the tile's first key and ends at its last valid one
    const int32_t rec = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(((g.valid - 1) * rs + D) * 4));
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(tensor + g.tok0 * rs + static_cast<int64_t>(head) * D), 0, rec, kBufferWord3);
    const int sub = lane / L::kSlots, slot = lane % L::kSlots;
    // slot ^ (key % 16) of key = key0 + sub, key0 a multiple of kRowsPerLoad: (slot ^ sub) ^ (key0 % 16)
    const int at = static_cast<int>(sub * rs * 4) + (kSwizzle ? slot ^ sub : slot) * 16;
    const int step = static_cast<int>(L::kRowsPerLoad * rs * 4);
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        const int key0 = (i0 + i) * L::kRowsPerLoad;
        load_lds16(r, (lds_void_t *)(dst + (i0 + i) * 1024), (kSwizzle ? at ^ ((key0 & 15) * 16) : at) + (i0 + i) * step);
    }
}

// Scores of the 32 keys at kb (a K tile's rows, slots permuted by key % 16).
template <int D>
__device__ __forceinline__ f32x16_t f32_scores(const uint8_t *kb, int col, int grp, const f32x4_t (&qf)[D / 8]) {
    const uint8_t *row = kb + col * (4 * D);
    const int base = (grp ^ (col & 15)) * 16;
    f32x16_t s = {};
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
        const f32x4_t kf = *reinterpret_cast<const f32x4_t *>(row + (base ^ (c * 32)));
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[c][e], s, 0, 0, 0);
    }
    return s;
}

// Softmax of 32 keys' scores (the first `valid` of them count): s becomes the
// probabilities against the new running maximum, O and l are rescaled to it.
template <int D>
__device__ __forceinline__ void f32_softmax(F32Wave<D> &w, f32x16_t &s, int valid, int grp, float sl2) {
    if (valid < 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if ((r / 4) * 8 + grp * 4 + r % 4 >= valid) s[r] = -__builtin_huge_valf();
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(w.m, halves_max(mx));
    // rows whose maximum stays keep O and l as they are (their factor is exactly 1)
    if (__builtin_amdgcn_ballot_w64(mx > w.m) != 0) {
        const float corr = mx > w.m ? fast_exp2((w.m - mx) * sl2) : 1.0f;   // 0 on the first tile
        w.l *= corr;
#pragma unroll
        for (int db = 0; db < F32Wave<D>::kDb; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) w.o[db][r] *= corr;
        w.m = mx;
    }
    // a row whose scores so far are all -inf takes 0 as its reference: its probabilities are 0
    const float ref = mx == -__builtin_huge_valf() ? 0.0f : mx;
    float sum[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        s[r] = fast_exp2((s[r] - ref) * sl2);
        sum[r / 4] = r % 4 == 0 ? s[r] : sum[r / 4] + s[r];
    }
    w.l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
}

// O^T += V^T P^T for the 32 keys whose V rows are at vb.
template <int D>
__device__ __forceinline__ void f32_pv(F32Wave<D> &w, const uint8_t *vb, const f32x16_t &p, int col, int grp) {
    constexpr int kDb = F32Wave<D>::kDb;
    typedef float vread_t __attribute__((ext_vector_type(kDb)));
    const uint8_t *lane0 = vb + grp * 4 * (4 * D) + col * (4 * kDb);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const vread_t v = *reinterpret_cast<const vread_t *>(lane0 + ((r / 4) * 8 + r % 4) * (4 * D));
#pragma unroll
        for (int db = 0; db < kDb; ++db)
            w.o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[db], p[r], w.o[db], 0, 0, 0);
    }
}

template <int D>
__device__ __forceinline__ int64_t key_tiles(const AttnF32Args &a, int keys) {
    return a.n_kv > 0 ? static_cast<int64_t>(a.n_kv) * a.tiles_per_frame : (a.S + keys - 1) / keys;
}

// Workgroup id -> (head, query tile): consecutive ids go round-robin to the
// XCDs, so each XCD gets a contiguous head-major range whose workgroups stream
// the same head's K and V through that XCD's L2. false: no tile for this id.
__device__ __forceinline__ bool f32_tile(const AttnF32Args &a, int &head, int &qt) {
    const int bid = blockIdx.x;
    const int tile = (bid % a.xcds) * a.per_xcd + bid / a.xcds;
    if (tile >= a.total_tiles) return false;
    head = tile / a.n_qtiles;
    qt = tile - head * a.n_qtiles;
    return true;
}

constexpr int kTileWaves = 4;
constexpr int kTileRows = 32 * kTileWaves;
// 16 KB of K and of V a tile at either head dimension
template <int D> constexpr int kTileKeys = D == 128 ? 32 : 64;

template <int D>
__global__ __launch_bounds__(64 * kTileWaves) __attribute__((amdgpu_waves_per_eu(2)))
void attn_f32_tile_kernel(const AttnF32Args a) {
    constexpr int kKeys = kTileKeys<D>;
    using L = F32Tile<D, kKeys>;
    constexpr int kLoadsPerWave = L::kLoads / kTileWaves;
    __shared__ __attribute__((aligned(1024))) uint8_t k0[L::kBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t k1[L::kBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t v0[L::kBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t v1[L::kBytes];
    int head, qt;
    if (!f32_tile(a, head, qt)) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, grp = lane >> 5;
    const int64_t row = static_cast<int64_t>(qt) * kTileRows + wave * 32 + col;
    F32Wave<D> w;
    load_queries<D>(a, row, head, grp, w);

    auto issue = [&](const F32Geom &g, uint8_t *kd, uint8_t *vd) {
        issue_rows<D, kKeys, true, kLoadsPerWave>(a, a.k, head, g, kd, wave * kLoadsPerWave, lane);
        issue_rows<D, kKeys, false, kLoadsPerWave>(a, a.v, head, g, vd, wave * kLoadsPerWave, lane);
    };
    auto compute = [&](int valid, const uint8_t *kb, const uint8_t *vb) {
#pragma unroll
        for (int b = 0; b < kKeys / 32; ++b) {
            if (b > 0 && valid <= b * 32) break;
            f32x16_t s = f32_scores<D>(kb + b * 32 * L::kRow, col, grp, w.qf);
            f32_softmax<D>(w, s, valid - b * 32, grp, a.scale_log2);
            f32_pv<D>(w, vb + b * 32 * L::kRow, s, col, grp);
        }
    };
    auto tile_done = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads have reached LDS
        __syncthreads();
    };
    const int64_t n = key_tiles<D>(a, kKeys);
    F32Geom cur = tile_geom<kKeys>(a, 0);
    issue(cur, k0, v0);
    tile_done();
    for (int64_t t = 0; t < n; t += 2) {
        F32Geom nxt = cur;
        if (t + 1 < n) {
            nxt = tile_geom<kKeys>(a, t + 1);
            issue(nxt, k1, v1);
        }
        compute(cur.valid, k0, v0);
        tile_done();
        if (t + 1 >= n) break;
        if (t + 2 < n) {
            cur = tile_geom<kKeys>(a, t + 2);
            issue(cur, k0, v0);
        }
        compute(nxt.valid, k1, v1);
        tile_done();
    }
    const float inv = 1.0f / halves_sum(w.l);
    if (row < a.Mq) {
        constexpr int kDb = F32Wave<D>::kDb;
        typedef float vread_t __attribute__((ext_vector_type(kDb)));
        float *op = a.out + (row * a.heads + head) * D;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            vread_t x;
#pragma unroll
            for (int db = 0; db < kDb; ++db) x[db] = w.o[db][r] * inv;
            *reinterpret_cast<vread_t *>(op + ((r / 4) * 8 + grp * 4 + r % 4) * kDb) = x;
        }
    }
}

// Waves that share out the keys: 128 KB of private K and V buffers either way.
template <int D> constexpr int kParts = D == 128 ? 4 : 8;
constexpr int kSplitKeys = 32;
constexpr int kSplitRows = 32;

template <int D>
__global__ __launch_bounds__(64 * kParts<D>) __attribute__((amdgpu_waves_per_eu(kParts<D> / 4)))
void attn_f32_split_kernel(const AttnF32Args a) {
    constexpr int kP = kParts<D>;
    constexpr int kDb = F32Wave<D>::kDb;
    using L = F32Tile<D, kSplitKeys>;
    typedef float vread_t __attribute__((ext_vector_type(kDb)));
    __shared__ __attribute__((aligned(1024))) uint8_t ks[kP * L::kBytes];
    __shared__ __attribute__((aligned(1024))) uint8_t vs[kP * L::kBytes];
    __shared__ float ml[kP][kSplitRows][2];
    int head, qt;
    if (!f32_tile(a, head, qt)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, grp = lane >> 5;
    uint8_t *kb = ks + wave * L::kBytes;
    uint8_t *vb = vs + wave * L::kBytes;
    F32Wave<D> w;

    load_queries<D>(a, static_cast<int64_t>(qt) * kSplitRows + col, head, grp, w);
    const int64_t n = key_tiles<D>(a, kSplitKeys);
    if (wave < n) {
        F32Geom g = tile_geom<kSplitKeys>(a, wave);
        issue_rows<D, kSplitKeys, true, L::kLoads>(a, a.k, head, g, kb, 0, lane);
        issue_rows<D, kSplitKeys, false, L::kLoads>(a, a.v, head, g, vb, 0, lane);
        for (int64_t t = wave; t < n; t += kP) {
            // (past the last tile it is fetched again and not used: with the loads on every
            // path the waits below can be counted instead of draining both tensors)
            const F32Geom nxt = tile_geom<kSplitKeys>(a, t + kP < n ? t + kP : t);
            wait_loads<L::kLoads>();   // K is there; V may still be in flight
            f32x16_t s = f32_scores<D>(kb, col, grp, w.qf);
            wait_lds_reads();          // K is read: its buffer is free
            issue_rows<D, kSplitKeys, true, L::kLoads>(a, a.k, head, nxt, kb, 0, lane);
            f32_softmax<D>(w, s, g.valid, grp, a.scale_log2);
            wait_loads<L::kLoads>();   // V is there; the next K may still be in flight
            f32_pv<D>(w, vb, s, col, grp);
            wait_lds_reads();
            issue_rows<D, kSplitKeys, false, L::kLoads>(a, a.v, head, nxt, vb, 0, lane);
            g = nxt;
        }
        wait_loads<0>();   // nothing lands in the buffers any more
    }

    // ---- merge: every wave's O rows into its own K buffer, units permuted by row % 16 ----
    const float l = halves_sum(w.l);
    if (grp == 0) {
        ml[wave][col][0] = w.m;
        ml[wave][col][1] = l;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        vread_t x;
#pragma unroll
        for (int db = 0; db < kDb; ++db) x[db] = w.o[db][r];
        const int unit = ((r / 4) * 8 + grp * 4 + r % 4) ^ (col & 15);
        *reinterpret_cast<vread_t *>(kb + col * L::kRow + unit * (4 * kDb)) = x;
    }
    __syncthreads();
    constexpr int kUnits = kSplitRows * 32;   // of kDb floats
    for (int u = tid; u < kUnits; u += 64 * kP) {
        const int r = u / 32, unit = u % 32;
        const int64_t row = static_cast<int64_t>(qt) * kSplitRows + r;
        if (row >= a.Mq) break;
        float m = ml[0][r][0];
#pragma unroll
        for (int p = 1; p < kP; ++p) m = fmaxf(m, ml[p][r][0]);
        float lsum = 0.0f;
        vread_t x = {};
#pragma unroll
        for (int p = 0; p < kP; ++p) {
            const float wgt = fast_exp2((ml[p][r][0] - m) * a.scale_log2);
            lsum = fmaf(wgt, ml[p][r][1], lsum);
            const vread_t y = *reinterpret_cast<const vread_t *>(ks + p * L::kBytes + r * L::kRow +
                                                                 (unit ^ (r & 15)) * (4 * kDb));
#pragma unroll
            for (int db = 0; db < kDb; ++db) x[db] = fmaf(wgt, y[db], x[db]);
        }
        const float inv = 1.0f / lsum;
#pragma unroll
        for (int db = 0; db < kDb; ++db) x[db] *= inv;
        *reinterpret_cast<vread_t *>(a.out + (row * a.heads + head) * D + unit * kDb) = x;
    }
}

}  // namespace

hipError_t launch_attention_f32(const AttnParams &p, hipStream_t stream) {
    const int64_t Mq = static_cast<int64_t>(p.M) * p.N;
    const int32_t cus = p.geo.cus, xcds = p.geo.xcds;
    if (cus < 1 || xcds < 1 || xcds > 64) return hipErrorInvalidValue;
    AttnF32Args a{};
    a.q = static_cast<const float *>(p.q);
    a.k = static_cast<const float *>(p.k);
    a.v = static_cast<const float *>(p.v);
    a.out = static_cast<float *>(p.out);
    a.S = p.S;
    a.N = p.N;
    a.Mq = Mq;
    a.heads = p.heads;
    a.scale_log2 = static_cast<float>(1.4426950408889634 / sqrt(static_cast<double>(p.head_dim)));
    for (int i = 0; i < p.M; ++i) a.kf[i] = p.kf[i];
    a.n_kv = p.n_kv;
    for (int i = 0; i < p.n_kv; ++i) a.kvf[i] = p.kvf[i];

    const bool split = p.split_keys && attention_shares_keys(p, AttnSplit{});
    const int64_t rows = split ? kSplitRows : kTileRows;
    const int64_t keys = split ? kSplitKeys : (p.head_dim == 128 ? kTileKeys<128> : kTileKeys<64>);
    const int64_t nq = (Mq + rows - 1) / rows;
    // (65,535 heads also keep the byte offsets inside a tile of 64 x 64 or 32 x 128 below 2 GiB)
    if (p.heads > 65535 || nq > 0x7fffffffLL / 64 / p.heads) return hipErrorInvalidConfiguration;
    const int64_t tpf = (p.N + keys - 1) / keys;
    if (p.n_kv > 0 && tpf * p.n_kv > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.tiles_per_frame = static_cast<int32_t>(tpf < 0x7fffffffLL ? tpf : 0x7fffffffLL);   // read for a frame list only
    a.n_qtiles = static_cast<int32_t>(nq);
    a.total_tiles = static_cast<int32_t>(nq * p.heads);
    a.xcds = xcds;
    a.per_xcd = (a.total_tiles + xcds - 1) / xcds;
    const dim3 grid(static_cast<uint32_t>(a.per_xcd) * static_cast<uint32_t>(xcds));
    if (split) {
        if (p.head_dim == 128)
            hipLaunchKernelGGL(attn_f32_split_kernel<128>, grid, dim3(64 * kParts<128>), 0, stream, a);
        else
            hipLaunchKernelGGL(attn_f32_split_kernel<64>, grid, dim3(64 * kParts<64>), 0, stream, a);
    } else {
        if (p.head_dim == 128) hipLaunchKernelGGL(attn_f32_tile_kernel<128>, grid, dim3(64 * kTileWaves), 0, stream, a);
        else hipLaunchKernelGGL(attn_f32_tile_kernel<64>, grid, dim3(64 * kTileWaves), 0, stream, a);
    }
    return hipGetLastError();
}

// Whole tiles of 128 rows keep a compute unit busy for one unit of time each;
// tiles of 32 rows with the keys shared out take a quarter of it. The split
// form is taken where its rounds of the device end at least a tenth earlier
// (it reads K and V four times as often).
bool f32_split_pays(int64_t Mq, int32_t heads, int32_t cus) {
    const int64_t whole = (Mq + kTileRows - 1) / kTileRows * heads;
    const int64_t parts = (Mq + kSplitRows - 1) / kSplitRows * heads;
    const int64_t t_whole = 4 * ((whole + cus - 1) / cus), t_split = (parts + cus - 1) / cus;
    return 10 * t_split < 9 * t_whole;
}

}  // namespace rf
