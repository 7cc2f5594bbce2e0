/* Host rules of the attention launch, called in the library itself: which sizes
   are refused. Prints "ok <checks>"; exits 1 at the first mismatch. */
#include <cstdio>

#include "rf_internal.h"

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

int main() {
    if (heads_limit()) return 1;
    std::printf("ok %d\n", checks);
    return 0;
}
