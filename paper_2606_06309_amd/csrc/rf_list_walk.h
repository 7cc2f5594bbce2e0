// The walk over a frame list's keys in key tiles: its plan (host) and its steps
// (device; the host runs them in tests).
#pragma once

#include <hip/hip_runtime.h>

#include "rf_internal.h"

namespace rf {

// How a frame list's keys are cut into tiles of bc.
struct ListWalk {
    int64_t per_frame;   // tiles of a frame, 0: the frames' keys lie end to end
    int64_t tiles;
};
// For tiles of bc keys; `split` parts of the split tail walk them (0: none).
ListWalk list_walk(const AttnParams &p, int64_t bc, int64_t split);

// A tile of a frame list: its first key's token, its valid keys, and the key
// from which its keys belong to the next listed frame, `delta` bytes further on
// than consecutive tokens would be (0: none, or the frames are neighbours).
struct ListTile {
    int64_t tok0;
    int32_t valid, first, delta;
};
// Tile t of a list walked in tiles that never cross a frame.
// Args: the fields N, n_kv, tiles_per_frame and kvf of AttnKArgs.
template <int kBc, class Args>
__host__ __device__ __forceinline__ ListTile aligned_tile(const Args &a, int64_t t) {
    const int32_t m = static_cast<int32_t>(t) / a.tiles_per_frame;
    const int64_t o = (t - static_cast<int64_t>(m) * a.tiles_per_frame) * kBc;
    return ListTile{static_cast<int64_t>(a.kvf[m]) * a.N + o, static_cast<int32_t>(a.N - o < kBc ? a.N - o : kBc),
                    kBc, 0};
}

// The tiles of a list walked end to end, one after the other from tile t on, without
// a division or a wait for a frame id at each: the id of the frame after the current
// one is fetched when the current one is entered, long before a tile reaches it (with
// both at every tile: 500 us where this takes 490, 6 frames of 30 x 52, 12 x 128).
template <int kBc, class Args>
struct ListWalker {
    int64_t o;             // the next tile's offset in its frame
    int32_t m;             // and that frame's place in the list
    int32_t frame, next;   // ids of frames m and m + 1 (next: any listed one after the last)
    __host__ __device__ __forceinline__ ListWalker(const Args &a, int64_t t) {
        m = static_cast<int32_t>(t) * kBc / static_cast<int32_t>(a.N);
        o = t * kBc - m * a.N;
        frame = a.kvf[m];
        next = a.kvf[m + 1 < a.n_kv ? m + 1 : m];
    }
    __host__ __device__ __forceinline__ ListTile take(const Args &a, int64_t rs) {
        ListTile g;
        const int64_t left = a.N - o;   // keys of this frame from here on
        g.tok0 = frame * a.N + o;
        g.first = kBc;
        g.delta = 0;
        g.valid = static_cast<int32_t>(left < kBc ? left : kBc);
        o += kBc;
        if (__builtin_expect(o >= a.N, 0)) {   // (out of the common tile's way: 527 us against 533)
            o = kBc - left;
            if (o > 0 && m + 1 < a.n_kv) {
                g.first = static_cast<int32_t>(left);
                g.valid = kBc;
                // (a frame holds a tile: the next one does not end before this tile does)
                g.delta = static_cast<int32_t>((next - frame - 1) * a.N * rs * 2);
            }
            ++m;
            frame = next;
            next = a.kvf[m + 1 < a.n_kv ? m + 1 : a.n_kv - 1];
        }
        return g;
    }
};

}  // namespace rf
