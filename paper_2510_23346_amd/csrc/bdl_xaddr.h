// Where a wave's activation loads lie (host and device: the host checks the
// bounds of what the kernels compute).
#pragma once

namespace bdl {

// Activations are loaded in pairs of k-steps, 16 bytes (a chunk) per lane:
// chunk c (0 .. 7) of a row's pair holds its inputs 8 c .. 8 c + 7, so chunks
// 4 .. 7 are the second k-step.  X is row-major [T x K], or packed in
// fragments (1 KB per 16 rows and k-step, rows padded to 16).

// byte offset of chunk c of row t's pair 0
constexpr long long x_chunk_offset(bool packed, int t, int K, int c) {
    return packed ? ((long long)(t >> 4) * (K >> 5) + (c >> 2)) * 1024 + ((t & 15) + 16 * (c & 3)) * 16
                  : (long long)t * K * 2 + c * 16;
}

// bytes from there to the same chunk of pair g.  The last pair of an odd number
// of k-steps has no second one: its chunks 4 .. 7 (which nothing uses) take
// chunks 0 .. 3 again, so that no load leaves X.
constexpr long long x_pair_offset(bool packed, int K, int c, int g) {
    return (long long)g * (packed ? 2048 : 128) -
           (((K >> 5) & 1) && g == (K >> 6) && c >= 4 ? (packed ? 1024 : 64) : 0);
}

}  // namespace bdl
