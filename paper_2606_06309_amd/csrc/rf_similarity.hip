// Cosine similarity between latent frames for gfx950 (content-aware keyframe
// selection: Eq. (1) compares frames by cosine similarity, Sec. 3.1; Alg. 1).
//
// The frames of a batch element form a matrix X = [T][F] (F = C*H*W elements,
// channel after channel); the similarity is the Gram matrix G = X X^T scaled
// by the frame norms. F is large (10^5 .. 10^6) and T small (<= 256), so the
// work is a reduction over F, split over the workgroups of the device:
//  1. gram_mfma_kernel (at most 64 frames): a wave walks chunks of 64 elements,
//     loads all frames' elements of a chunk into registers (the next chunk's while
//     this one is summed), widens them to fp64 once and accumulates every pair of
//     4-frame blocks with v_mfma_f64_4x4x4_4b in fp64 (fp32 x fp32 products are
//     exact there). The partial Gram blocks of a workgroup go to the workspace.
//     What bounds it: for 33 frames 45 block pairs x 16 cycles per 16 elements of
//     a SIMD (75 TFLOP/s of 78.6; 4x4 blocks lose 9 % of it to padding where 16x16
//     ones would lose half, and run at 47), 4.4 us at 33 frames of 16 x 90 x 160,
//     beside 30 MB of reads and the start and end of two launches. The vector form
//     it replaces widened 32 operands for 64 fused multiply-adds. That shape:
//     26.4 -> 17.8 us in all, fp32; bf16 32.3 -> 17.2.
//     gram_wide_kernel (more frames) stages one chunk of all frames in LDS and
//     sums 4x4 blocks with vector instructions.
//  2. gram_reduce_kernel: a workgroup per 4x4 block pair sums the partials of
//     all runs in a fixed order (deterministic) into the cosines, or above 64
//     frames into the Gram matrix, which
//  3. cosine_normalize_kernel, one workgroup per batch element, turns into
//     G_ij / (max(|x_i|, eps) * max(|x_j|, eps)) in place.
#include <utility>

#include "rf_internal.h"

namespace rf {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = 64;             // feature elements a wave takes at a time (at most 64 frames)
constexpr int kRunChunk = 256;         // elements the number of runs is counted in (at most 64 frames)
constexpr int kTileFloats = 16384;     // LDS floats of one staged chunk (more than 64 frames; 64 KB)
constexpr int kMaxWideChunk = 256;     // feature elements of one (more than 64 frames)
constexpr double kNormFloor = 1e-8;
constexpr int64_t kMaxWorkgroups = 512;      // partial-Gram workgroups per launch the workspace holds
constexpr int kNarrowFrames = 64;            // padded frame count of the matrix-core path

typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct PartialArgs {
    const void *x;
    double *ws;
    int64_t plane;
    int64_t chunks_per_plane;
    int64_t n_chunks;         // per batch element
    int64_t n_runs;           // workgroups (partial Gram blocks) per batch element
    int32_t C, T, Tp, NB, NBP, L;
};

template <bool kBf16>
__device__ inline float load_elem(const void *x, int64_t i) {
    if (kBf16) return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(x)[i]) << 16);
    return static_cast<const float *>(x)[i];
}

// Block pair index -> (bi, bj), bi <= bj, enumerated row after row.
__device__ inline void block_pair(int bp, int NB, int &bi, int &bj) {
    int row = 0, rem = bp;
    while (rem >= NB - row) {
        rem -= NB - row;
        ++row;
    }
    bi = row;
    bj = row + rem;
}

// ---- at most 64 frames: fp64 matrix cores ----

// Four consecutive elements of one frame, as loaded: planes of any size put
// them at any element's alignment.
template <bool kBf16>
struct Quad;
template <>
struct Quad<false> {
    struct __attribute__((packed, aligned(4))) Raw { float v[4]; };
    float v[4];
    __device__ __forceinline__ void load(const void *x, int64_t i) {
        const Raw r = *reinterpret_cast<const Raw *>(static_cast<const float *>(x) + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = r.v[e];
    }
    __device__ __forceinline__ void load_part(const void *x, int64_t i, int n) {   // the first n of them
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < n ? load_elem<false>(x, i + e) : 0.0f;
    }
    __device__ __forceinline__ float get(int e) const { return v[e]; }
};
template <>
struct Quad<true> {
    struct __attribute__((packed, aligned(2))) Raw { uint32_t w[2]; };
    uint32_t w[2];
    __device__ __forceinline__ void load(const void *x, int64_t i) {
        const Raw r = *reinterpret_cast<const Raw *>(static_cast<const uint16_t *>(x) + i);
        w[0] = r.w[0];
        w[1] = r.w[1];
    }
    __device__ __forceinline__ void load_part(const void *x, int64_t i, int n) {
        const uint16_t *p = static_cast<const uint16_t *>(x) + i;
        w[0] = (n > 0 ? p[0] : 0u) | (n > 1 ? static_cast<uint32_t>(p[1]) << 16 : 0u);
        w[1] = (n > 2 ? p[2] : 0u) | (n > 3 ? static_cast<uint32_t>(p[3]) << 16 : 0u);
    }
    __device__ __forceinline__ float get(int e) const {
        return __uint_as_float(e % 2 ? w[e / 2] & 0xffff0000u : w[e / 2] << 16);
    }
};

// kNB = NB blocks of 4 frames. v_mfma_f64_4x4x4_4b multiplies four independent
// 4x4 blocks over 4 elements each: lane l gives row l % 4 of both operands, so a
// register that holds frame 4 b + l % 4 at element slot l / 4 is the A operand of
// every pair (b, .) and the B operand of every pair (., b), and the four blocks
// of an instruction are four quarters of the elements.
template <int kNB, bool kBf16>
__global__ __launch_bounds__(kThreads) void gram_mfma_kernel(const PartialArgs a) {
    constexpr int kNBP = kNB * (kNB + 1) / 2;
    constexpr int kGroup = 16;   // block pairs summed over the waves at a time
    __shared__ double red[kGroup * kThreads];
    const int64_t b = blockIdx.x / a.n_runs;
    const int64_t rn = blockIdx.x - b * a.n_runs;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t waves = a.n_runs * (kThreads / 64);
    const int64_t gw = rn * (kThreads / 64) + wave;
    const int64_t c0 = gw * a.n_chunks / waves, c1 = (gw + 1) * a.n_chunks / waves;

    // this lane's frame of each block (rows past the last frame repeat it: their
    // entries are never written) and its elements inside a chunk
    const int slot = 4 * (lane / 4);
    const int64_t lane_off = (lane % 4) * a.plane + slot;
    const int last = 4 * (kNB - 1) + lane % 4;
    const int64_t last_off = (last < a.T ? last : a.T - 1) * a.plane + slot;
    auto fetch = [&](int64_t chunk, Quad<kBf16> (&x)[kNB]) {
        const int64_t c = chunk / a.chunks_per_plane;
        const int64_t p0 = (chunk - c * a.chunks_per_plane) * kChunk;
        const int64_t base = (b * a.C + c) * a.T * a.plane + p0;
        if (p0 + kChunk <= a.plane) {
#pragma unroll
            for (int f = 0; f < kNB; ++f)
                x[f].load(a.x, base + (f < kNB - 1 ? 4 * f * a.plane + lane_off : last_off));
        } else {
            const int64_t left = a.plane - p0 - slot;
            const int n = static_cast<int>(left < 0 ? 0 : left < 4 ? left : 4);
#pragma unroll
            for (int f = 0; f < kNB; ++f)
                x[f].load_part(a.x, base + (f < kNB - 1 ? 4 * f * a.plane + lane_off : last_off), n);
        }
    };
    double acc[kNBP];
#pragma unroll
    for (int i = 0; i < kNBP; ++i) acc[i] = 0.0;
    auto sum = [&](const Quad<kBf16> (&x)[kNB]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double v[kNB];
#pragma unroll
            for (int f = 0; f < kNB; ++f) v[f] = static_cast<double>(x[f].get(e));
            int i = 0;
#pragma unroll
            for (int bi = 0; bi < kNB; ++bi)
#pragma unroll
                for (int bj = bi; bj < kNB; ++bj, ++i)
                    acc[i] = __builtin_amdgcn_mfma_f64_4x4x4f64(v[bi], v[bj], acc[i], 0, 0, 0);
        }
    };
    Quad<kBf16> x0[kNB], x1[kNB];
    if (c0 < c1) fetch(c0, x0);
    for (int64_t chunk = c0; chunk < c1; chunk += 2) {
        if (chunk + 1 < c1) fetch(chunk + 1, x1);
        sum(x0);
        if (chunk + 1 >= c1) break;
        if (chunk + 2 < c1) fetch(chunk + 2, x0);
        sum(x1);
    }

    // sum over the waves and the four blocks; lane 16 i + 4 q + j holds entry (i, j) of block q
    double *dst = a.ws + (b * a.n_runs + rn) * kNBP * 16;
#pragma unroll
    for (int g = 0; g < kNBP; g += kGroup) {
        constexpr int kAll = kNBP;
        const int n = kAll - g < kGroup ? kAll - g : kGroup;
        if (g > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < kGroup; ++i)
            if (g + i < kAll) red[i * kThreads + tid] = acc[g + i < kAll ? g + i : 0];
        __syncthreads();
        if (tid < n * 16) {
            const double *src = red + (tid / 16) * kThreads + (tid % 16) / 4 * 16 + tid % 4;
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w)
#pragma unroll
                for (int q = 0; q < 4; ++q) s += src[w * 64 + q * 4];
            dst[g * 16 + tid] = s;
        }
    }
}

// ---- more than 64 frames ----

// The chunk of all T frames is staged in LDS as [element][frame] (frames padded
// with zeros to a multiple of 4); a thread walks several block pairs and writes
// each one's 16 sums when done. A run is one chunk. What bounds it is the latency of
// a thread's LDS reads before its sums (few frames past 64 leave a workgroup one pair
// a thread): reading four elements ahead, one video of 16 planes, 80 frames of 2 x 4:
// 41.1 -> 37.3 us in all; 80 of 52 x 160: 100.2 -> 93.4; 200 of 30 x 52: 141 -> 138.
template <bool kBf16>
__global__ __launch_bounds__(kThreads) void gram_wide_kernel(const PartialArgs a) {
    extern __shared__ __attribute__((aligned(16))) float tile[];   // Tp * L floats (<= kTileFloats)
    const int64_t b = blockIdx.x / a.n_runs;
    const int64_t rn = blockIdx.x - b * a.n_runs;
    const int tid = threadIdx.x;
    double *dst = a.ws + (b * a.n_runs + rn) * a.NBP * 16;
    const int64_t c = rn / a.chunks_per_plane;
    const int64_t p0 = (rn - c * a.chunks_per_plane) * a.L;
    const int64_t frame0 = (b * a.C + c) * a.T;
    for (int idx = tid; idx < a.Tp * a.L; idx += kThreads) {
        const int f = idx / a.L, k = idx - f * a.L;
        float v = 0.0f;
        if (f < a.T && p0 + k < a.plane) v = load_elem<kBf16>(a.x, (frame0 + f) * a.plane + p0 + k);
        tile[k * a.Tp + f] = v;
    }
    __syncthreads();
    const f32x4_t *t4 = reinterpret_cast<const f32x4_t *>(tile);
    const int row4 = a.Tp / 4;
    for (int bp = tid; bp < a.NBP; bp += kThreads) {
        int bi, bj;
        block_pair(bp, a.NB, bi, bj);
        double acc[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0;
        // four elements (L is a multiple of 16) are summed while the next four are read
        f32x4_t u[4], w[4];
        auto read = [&](int k, f32x4_t (&x)[4], f32x4_t (&y)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = t4[(k + j) * row4 + bi];
                y[j] = t4[(k + j) * row4 + bj];
            }
        };
        read(0, u, w);
        for (int k = 0; k < a.L; k += 4) {
            f32x4_t un[4], wn[4];
            read(k + 4 < a.L ? k + 4 : k, un, wn);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[r * 4 + q] =
                            fma(static_cast<double>(u[j][r]), static_cast<double>(w[j][q]), acc[r * 4 + q]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u[j] = un[j];
                w[j] = wn[j];
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[bp * 16 + e] = acc[e];
    }
}

struct ReduceArgs {
    const double *ws;
    double *sim;
    int64_t n_runs;
    int32_t T, NB, NBP;
};

// One workgroup per (batch element, block pair): kReduceLanes lanes per Gram
// entry sum the runs' partials with stride kReduceLanes, then the lane sums
// are added in a tree. kCosine: the workgroup also sums the two diagonal blocks
// of its frames, in the same order as their own workgroups do, and writes the
// cosines, so no launch follows (the partials of at most 512 runs are read
// three times instead of once: a few hundred KB from L2); otherwise the Gram
// entries, for cosine_normalize_kernel.
constexpr int kReduceThreads = 1024;
constexpr int kReduceLanes = kReduceThreads / 16;

template <bool kCosine>
__global__ __launch_bounds__(kReduceThreads) void gram_reduce_kernel(const ReduceArgs a) {
    constexpr int kSums = kCosine ? 3 : 1;
    __shared__ double part[kSums][kReduceThreads / 64][16];
    __shared__ double total[kSums][16];
    const int64_t b = blockIdx.x / a.NBP;
    const int bp = static_cast<int>(blockIdx.x - b * a.NBP);
    const int tid = threadIdx.x, e = tid % 16, lane = tid / 16;
    int bi, bj;
    block_pair(bp, a.NB, bi, bj);
    // block pair (i, i) follows the i rows of NB, NB - 1, ... pairs before it
    const int diag_i = bi * a.NB - bi * (bi - 1) / 2, diag_j = bj * a.NB - bj * (bj - 1) / 2;
    const double *src = a.ws + b * a.n_runs * a.NBP * 16 + e;
    const int64_t run = static_cast<int64_t>(a.NBP) * 16;
    double s[kSums];
#pragma unroll
    for (int k = 0; k < kSums; ++k) s[k] = 0.0;
#pragma unroll 4
    for (int64_t r = lane; r < a.n_runs; r += kReduceLanes) {
        s[0] += src[r * run + bp * 16];
        if constexpr (kCosine) {
            s[1] += src[r * run + diag_i * 16];
            s[2] += src[r * run + diag_j * 16];
        }
    }
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
        s[k] += __shfl_xor(s[k], 16);
        s[k] += __shfl_xor(s[k], 32);
        if (tid % 64 < 16) part[k][tid / 64][e] = s[k];
    }
    __syncthreads();
    if (tid < kSums * 16) {
        double v[kReduceThreads / 64];
#pragma unroll
        for (int w = 0; w < kReduceThreads / 64; ++w) v[w] = part[lane][w][e];
#pragma unroll
        for (int n = kReduceThreads / 128; n > 0; n /= 2)
#pragma unroll
            for (int w = 0; w < n; ++w) v[w] += v[w + n];
        total[lane][e] = v[0];
    }
    __syncthreads();
    const int i = 4 * bi + e / 4, j = 4 * bj + e % 4;
    if (tid < 16 && i <= j && j < a.T) {
        double g = total[0][e];
        if constexpr (kCosine) {
            const double ni = sqrt(total[1][e / 4 * 5]), nj = sqrt(total[2][e % 4 * 5]);
            g /= (ni > kNormFloor ? ni : kNormFloor) * (nj > kNormFloor ? nj : kNormFloor);
        }
        double *out = a.sim + b * a.T * a.T;
        out[static_cast<int64_t>(i) * a.T + j] = g;
        out[static_cast<int64_t>(j) * a.T + i] = g;
    }
}

__global__ __launch_bounds__(kThreads) void cosine_normalize_kernel(double *sim, int32_t T) {
    __shared__ double norm[kMaxFrames];
    double *g = sim + static_cast<int64_t>(blockIdx.x) * T * T;
    for (int i = threadIdx.x; i < T; i += kThreads) {
        const double n = sqrt(g[static_cast<int64_t>(i) * T + i]);
        norm[i] = n > kNormFloor ? n : kNormFloor;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < T * T; idx += kThreads) {
        const int i = idx / T, j = idx - i * T;
        g[idx] = g[idx] / (norm[i] * norm[j]);
    }
}

template <int kNB, bool kBf16>
void launch_mfma(const PartialArgs &a, dim3 grid, hipStream_t stream) {
    hipLaunchKernelGGL((gram_mfma_kernel<kNB, kBf16>), grid, dim3(kThreads), 0, stream, a);
}

// gram_mfma_kernel of 1..16 frame blocks
template <bool kBf16, int... kNB>
void launch_mfma_of(const PartialArgs &a, dim3 grid, hipStream_t stream, std::integer_sequence<int, kNB...>) {
    static constexpr void (*const launch[])(const PartialArgs &, dim3, hipStream_t) = {
        launch_mfma<kNB + 1, kBf16>...};
    launch[a.NB - 1](a, grid, stream);
}

}  // namespace

SimGeometry similarity_geometry(int32_t B, int32_t C, int32_t T, int64_t plane) {
    SimGeometry g{};
    g.Tp = (T + 3) / 4 * 4;
    g.NB = g.Tp / 4;
    g.NBP = g.NB * (g.NB + 1) / 2;
    const bool wide = g.Tp > kNarrowFrames;
    const int L = (kTileFloats / g.Tp) / 16 * 16;
    g.L = !wide ? kChunk : L < kMaxWideChunk ? L : kMaxWideChunk;
    g.chunks_per_plane = (plane + g.L - 1) / g.L;
    g.n_chunks = static_cast<int64_t>(C) * g.chunks_per_plane;
    // The workspace holds at most kMaxWorkgroups runs over the whole batch and at
    // least one per batch element; one per chunk above 64 frames.
    const int64_t per_b = kMaxWorkgroups / B > 0 ? kMaxWorkgroups / B : 1;
    const int64_t units = wide ? g.n_chunks : static_cast<int64_t>(C) * ((plane + kRunChunk - 1) / kRunChunk);
    const int64_t run = wide ? 1 : (units + per_b - 1) / per_b;
    g.n_runs = (units + run - 1) / run;
    g.workspace_bytes = static_cast<int64_t>(B) * g.n_runs * g.NBP * 16 * static_cast<int64_t>(sizeof(double));
    // Up to 16 frames a chunk is bound by its loads and two workgroups per compute
    // unit keep more of them in flight (5 videos of 13 frames of 61 x 105, 16
    // channels: 11.9 us against 12.7 with one); with more, the matrix instructions
    // of one wave fill a SIMD, and fewer partials are summed with one (33 frames of
    // 90 x 160: 17.8 us against 18.8; 48 frames: 24.8 against 31.3). Where a wave
    // then walks more than kLongWalk chunks its loads and its matrix instructions add
    // up, and two workgroups overlap them as long as the registers hold two waves a
    // SIMD, that is up to 44 frames in fp32 and 48 in bf16 (one against two, many calls
    // back to back over two sets of buffers, 16 x 90 x 160; 33 frames, fp32: 36 videos
    // 272 us, 236; 12: 97.6, 88.7; 5, 17.6 chunks: 46.5, 45.2; 2, 7 chunks: 25.8, 27.0; 40
    // frames: 5 videos 53.6, 52.4; 20: 188, 165; bf16 49.0, 47.9; 186, 163; 44: 61.3, 59.7;
    // 215, 192; bf16 55.9, 54.5; 213, 188; 48: fp32 68.3, 76.0; 243, 244; bf16 63.6, 62.7;
    // 243, 215). Two are taken up to 36 frames; 37 to 44, and to 48 in bf16, keep one for
    // the present, 2-12 % above two.
    constexpr int64_t kLongWalk = 16;
    const int64_t one_per_cu = kMaxWorkgroups / 2 / B > 0 ? kMaxWorkgroups / 2 / B : 1;
    const bool long_walk = g.NB <= 9 && g.n_chunks * B > kLongWalk * (kMaxWorkgroups / 2) * (kThreads / 64);
    if (!wide && g.NB > 4 && !long_walk && g.n_runs > one_per_cu) g.n_runs = one_per_cu;
    return g;
}

hipError_t launch_similarity(const SimParams &p, hipStream_t stream) {
    const SimGeometry g = similarity_geometry(p.B, p.C, p.T, p.plane);
    PartialArgs a{};
    a.x = p.latents;
    a.ws = p.workspace;
    a.plane = p.plane;
    a.chunks_per_plane = g.chunks_per_plane;
    a.n_chunks = g.n_chunks;
    a.n_runs = g.n_runs;
    a.C = p.C;
    a.T = p.T;
    a.Tp = g.Tp;
    a.NB = g.NB;
    a.NBP = g.NBP;
    a.L = g.L;
    const int64_t blocks = static_cast<int64_t>(p.B) * g.n_runs;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const dim3 grid(static_cast<uint32_t>(blocks)), block(kThreads);
    const bool wide = g.Tp > kNarrowFrames, bf16 = p.dtype == RF_BF16;
    if (wide) {
        const size_t lds = static_cast<size_t>(g.Tp) * g.L * sizeof(float);
        if (bf16) hipLaunchKernelGGL(gram_wide_kernel<true>, grid, block, lds, stream, a);
        else hipLaunchKernelGGL(gram_wide_kernel<false>, grid, block, lds, stream, a);
    } else {
        constexpr std::make_integer_sequence<int, kNarrowFrames / 4> blocks_of_4{};
        if (bf16) launch_mfma_of<true>(a, grid, stream, blocks_of_4);
        else launch_mfma_of<false>(a, grid, stream, blocks_of_4);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    ReduceArgs r{};
    r.ws = p.workspace;
    r.sim = p.sim;
    r.n_runs = g.n_runs;
    r.T = p.T;
    r.NB = g.NB;
    r.NBP = g.NBP;
    const int64_t rblocks = static_cast<int64_t>(p.B) * g.NBP;
    if (rblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const dim3 rgrid(static_cast<uint32_t>(rblocks)), rblock(kReduceThreads);
    if (!wide) {
        hipLaunchKernelGGL(gram_reduce_kernel<true>, rgrid, rblock, 0, stream, r);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(gram_reduce_kernel<false>, rgrid, rblock, 0, stream, r);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cosine_normalize_kernel, dim3(static_cast<uint32_t>(p.B)), block, 0, stream, p.sim, p.T);
    return hipGetLastError();
}

}  // namespace rf
