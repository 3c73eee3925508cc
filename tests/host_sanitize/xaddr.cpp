// Every activation load of a wave of the 64-bit form (XRows<MB, true>) lies
// inside X, and the chunks that the matrix cores use are the row's own.
#include <cstdio>

#include "bdl_xaddr.h"

int main() {
    long long bad = 0, n = 0;
    const int ks[] = {1, 2, 3, 4, 5, 8, 9, 17, 64, 65, 1025};
    const int ts[] = {1, 2, 15, 16, 17, 31, 32, 33, 100, 32768};
    for (int KS : ks)
        for (int T : ts)
            for (int packed = 0; packed < 2; ++packed)
                for (int c = 0; c < 8; ++c)
                    for (int last = 0; last < 20; ++last) {
                        const int t = T - 1 - last, K = 32 * KS, NP = (KS + 1) / 2;
                        if (t < 0) break;
                        const long long bytes = packed ? (T + 15) / 16 * (long long)KS * 1024 : (long long)T * K * 2;
                        for (int g = 0; g < NP; ++g) {
                            const long long at = bdl::x_chunk_offset(packed, t, K, c) + bdl::x_pair_offset(packed, K, c, g);
                            bad += at < 0 || at + 16 > bytes;
                            const int step = 2 * g + c / 4, in = 8 * (c % 4);      // k-step and its input
                            const long long want = packed ? ((long long)(t / 16) * KS + step) * 1024 + (t % 16 + 2 * in) * 16
                                                          : ((long long)t * K + 32 * step + in) * 2;
                            bad += step < KS && at != want;
                            ++n;
                        }
                    }
    std::printf("%lld loads, %lld bad\n", n, bad);
    return bad != 0;
}
