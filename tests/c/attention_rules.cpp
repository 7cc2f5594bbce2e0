/* Host rules of the attention launch, called in the library itself: which sizes
   are refused, and the walk over a frame list's keys, tile by tile and part by
   part, against the listed tokens one after the other. Prints "ok <checks>";
   exits 1 at the first mismatch. */
#include <cstdio>
#include <random>
#include <vector>

#include "rf_internal.h"
#include "rf_list_walk.h"

static int checks;
#define CHECK(cond)                                                                     \
    do {                                                                                \
        ++checks;                                                                       \
        if (!(cond)) return std::printf("line %d: %s\n", __LINE__, #cond), 1;           \
    } while (0)

// M = 1 frame of N tokens over T frames, every pointer NULL: only for launches that are refused.
static rf::AttnParams sizes(int T, int64_t N, int heads, int head_dim, int split_keys) {
    rf::AttnParams p{};
    p.M = 1;
    p.N = N;
    p.S = N * T;
    p.heads = heads;
    p.head_dim = head_dim;
    p.dtype = RF_BF16;
    p.split_keys = split_keys;
    p.geo.cus = 256;
    p.geo.xcds = 8;
    return p;
}

// Rows of a whole launch's key tile that span 2 GiB or more are refused, also
// where a small launch's own tile would stay below it.
static int heads_limit() {
    for (int head_dim : {64, 128}) {
        const int heads = 131072;   // 128 keys x 64 or 64 keys x 128, 2 bytes: 2 GiB
        for (int split_keys : {0, 1})
            for (int more : {0, 1, 65536})
                CHECK(rf::launch_attention(sizes(16, 32, heads + more, head_dim, split_keys), nullptr) ==
                      hipErrorInvalidConfiguration);
    }
    return 0;
}

struct WalkArgs {   // what the kernel's arguments hold of a walk
    int64_t N;
    int32_t n_kv, tiles_per_frame;
    int32_t kvf[rf::kMaxFrames];
};

static rf::AttnParams list(const std::vector<int> &frames, int64_t N, int heads, int head_dim) {
    rf::AttnParams p = sizes(256, N, heads, head_dim, 1);
    p.n_kv = static_cast<int32_t>(frames.size());
    for (int i = 0; i < p.n_kv; ++i) p.kvf[i] = frames[i];
    return p;
}

// The tiles that `split` parts (0: one walk) of the launch take, in order: every
// part begins at a tile, no offset inside a tile passes 32 bits, and the keys are
// the listed tokens. end_to_end: whether the walk has to lie end to end.
template <int kBc>
static int walk(const rf::AttnParams &p, int64_t split, bool end_to_end) {
    const rf::ListWalk lw = rf::list_walk(p, kBc, split);
    CHECK((lw.per_frame == 0) == end_to_end);
    CHECK(lw.tiles == (end_to_end ? (p.n_kv * p.N + kBc - 1) / kBc : p.n_kv * ((p.N + kBc - 1) / kBc)));
    WalkArgs a{};
    a.N = p.N;
    a.n_kv = p.n_kv;
    a.tiles_per_frame = static_cast<int32_t>(lw.per_frame);
    for (int i = 0; i < p.n_kv; ++i) a.kvf[i] = p.kvf[i];
    const int64_t rs = static_cast<int64_t>(p.heads) * p.head_dim;
    const int64_t parts = split > 0 ? split : 1, step = (lw.tiles + parts - 1) / parts;
    int64_t n = 0;   // keys met so far
    for (int64_t part = 0; part < parts; ++part) {
        const int64_t begin = part * step, end = begin + step < lw.tiles ? begin + step : lw.tiles;
        CHECK(begin < end);
        WalkArgs e = a;
        e.n_kv = end_to_end ? a.n_kv : 1;   // (the walker is made for walks end to end only)
        rf::ListWalker<kBc, WalkArgs> walker(e, end_to_end ? begin : 0);
        for (int64_t t = begin; t < end; ++t) {
            const rf::ListTile g = end_to_end ? walker.take(a, rs) : rf::aligned_tile<kBc>(a, t);
            CHECK(g.valid > 0 && g.valid <= kBc);
            CHECK(g.delta >= 0 && (kBc * rs) * 2 + g.delta <= 0x7fffffffLL);
            for (int key = 0; key < g.valid; ++key, ++n) {
                const int64_t tok = g.tok0 + key + (key >= g.first ? g.delta / (rs * 2) : 0);
                if (tok != p.kvf[n / p.N] * p.N + n % p.N || n / p.N >= p.n_kv) CHECK(!"a listed token");
            }
            CHECK(g.delta % (rs * 2) == 0);
        }
    }
    CHECK(n == p.n_kv * p.N);
    return 0;
}

template <int kBc>
static int walks(int head_dim) {
    std::mt19937 rng(17);
    for (int64_t N : {1, 2, 31, 63, 64, 65, 96, 127, 128, 129, 130, 191, 200, 255, 256, 257, 527})
        for (int round = 0; round < 40; ++round) {
            std::vector<int> frames;
            const int every = 1 + static_cast<int>(rng() % 4);
            for (int f = static_cast<int>(rng() % 5); f < 256 && frames.size() < 1 + rng() % 40; f += 1 + rng() % every)
                frames.push_back(f);
            const rf::AttnParams p = list(frames, N, 3, head_dim);
            const int64_t tiles = (p.n_kv * N + kBc - 1) / kBc;
            const bool saves = N >= kBc && tiles < p.n_kv * ((N + kBc - 1) / kBc);
            if (walk<kBc>(p, 0, saves)) return 1;
            // the parts that the split plan gives launches of these keys, at tails of any size
            for (int32_t cus : {7, 64, 256})
                for (int64_t Mq : {int64_t(1), N, 5 * N, 100 * N}) {
                    const rf::AttnSplit sp = rf::attention_split(Mq, p.heads, head_dim, N, p.S, p.n_kv, cus);
                    if (sp.split == 0) continue;
                    if (walk<kBc>(p, sp.split, saves && tiles > (sp.split - 1) * (sp.split - 1))) return 1;
                    // the plan's figure, in tiles that do not cross a frame, is the most a part has
                    CHECK((rf::list_walk(p, kBc, sp.split).tiles + sp.split - 1) / sp.split <= sp.kv_per_split);
                }
        }
    return 0;
}

// Parts of an end-to-end walk are all non-empty from (split - 1)^2 + 1 tiles on,
// and stay in frame-aligned tiles below.
static int guard_on_parts() {
    for (int64_t split = 2; split <= 8; ++split)
        for (int64_t tiles : {(split - 1) * (split - 1), (split - 1) * (split - 1) + 1}) {
            std::vector<int> frames;   // of 64 keys and a key more: n frames are n tiles up to n = 63
            for (int i = 0; i < tiles - 1; ++i) frames.push_back(2 * i);
            if (frames.size() < 2) continue;   // (one frame: the same tiles either way)
            const rf::AttnParams p = list(frames, 65, 2, 128);
            const int64_t walked = (static_cast<int64_t>(frames.size()) * 65 + 63) / 64;
            CHECK(walked == tiles);
            if (walk<64>(p, split, tiles > (split - 1) * (split - 1))) return 1;
        }
    return 0;
}

// Offsets inside a tile that reaches past a gap of frames fit 32 bits: 24 heads x
// 128 are 6,144 bytes a token, so 97 frames of 3,600 tokens and a tile of 64 still
// fit and 98 do not.
static int guard_on_gaps() {
    for (int gap : {96, 97, 98, 99}) {
        if (walk<64>(list({0, gap + 1, gap + 2}, 3600, 24, 128), 0, gap <= 97)) return 1;
        if (walk<64>(list({0, 1, gap + 2}, 3600, 24, 128), 2, gap <= 97)) return 1;
        if (walk<128>(list({0, gap + 1}, 3600, 48, 64), 0, gap <= 97)) return 1;
    }
    // exactly at the bound, and the next above: (3 N + 64) tokens of 256 bytes against 2^31 - 1
    if (walk<64>(list({0, 4}, 2796181, 1, 128), 0, true)) return 1;
    if (walk<64>(list({0, 4}, 2796182, 1, 128), 0, false)) return 1;
    return 0;
}

int main() {
    if (heads_limit() || walks<64>(128) || walks<128>(64) || guard_on_parts() || guard_on_gaps()) return 1;
    std::printf("ok %d\n", checks);
    return 0;
}
