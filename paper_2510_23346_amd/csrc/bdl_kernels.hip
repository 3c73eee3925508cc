// HIP kernels of the BD-LoRA shard forward for gfx950 (MI355X).
//
// A forward launch of one token batch over P projections (all sharing the
// tokens' adapter ids) that the decode launch does not take runs these kernels
// on the caller's stream (medium batches swap step 3 for the medium-batch GEMM
// and its epilogue in bdl_gemm.hip, large ones for the large-tile GEMMs there;
// step 3 is left with what those do not take above 256 tokens):
//
//  1. prep_kernel   -- workgroup 0 plans the batch: validates ids and groups
//                      tokens by adapter (counting sort over slots), and
//                      writes ready-to-use work descriptors for the other two
//                      kernels (shrink items; per row tile, the adapter
//                      octets to expand).  The other workgroups copy the
//                      activations X into the MFMA fragment layout.
//  2. shrink_kernel -- Z = scale * X A for every adapter group (the LoRA
//                      "shrink", matmul_3 / matmul_5 of the paper's Fig. 2/3,
//                      step "Z <- X A" of Alg. 1 and Alg. 2).  Each group's
//                      factor A^T is streamed once; the group's token rows are
//                      gathered.
//  3. gemm_kernel   -- out = X W_s^T + Z B for each output tile: the base
//                      product (matmul_1 / matmul_2) with the LoRA "expand"
//                      (matmul_4 / matmul_6) and the add (add_1 / add_2)
//                      fused, one bf16 store per output (Alg. 1 / Alg. 2,
//                      steps "Y_adapter <- Z B" and "Y <- Y + Y_adapter").
//
// Both GEMM-shaped kernels use 8 waves per workgroup that split the K loop
// into contiguous ranges and reduce through LDS in a fixed order, so results
// are bitwise reproducible.  Their operands are read in the 1 KB fragment
// layout (see bdl_device.h).  The expand runs as extra MFMA k-steps: for the
// adapters present in the tile, 8-rank pieces ("octets") of B^T are the B
// operand and the matching Z entries (zero for tokens of other adapters) the
// A operand.  Z is kept as a pair of bf16 numbers (hi + lo, about 16
// significant bits) and multiplied in two MFMAs, so the intermediate adds no
// bf16-sized error to the LoRA term.
#include "bdl_device.h"

namespace bdl {

constexpr int kStages = 3;                    // k-steps of loads kept in flight per wave

// --------------------------------------------------------------------------
// 2. shrink: Z[t, sigma * r8max + j] = scale_a * sum_k X[t, k] A_a,sigma[k, j]
//    work unit = (projection, shrink item of 16 MB tokens of one adapter,
//    chunk of 16 NB columns of A^T_cat)
//
//    A resident set of workgroups takes the units (projection in the order
//    sorder, longest K first; item; chunk) one at a time from a counter that
//    the plan zeroes, so the long units start first and no workgroup is spent
//    on the host's padding of the item count; the next unit's number is
//    fetched while the current one runs.  Eight waves split K; a wave's A^T
//    and X (pairs of k-steps, see XRows) run through a ring of D pairs.  A
//    projection whose columns all fit the smaller chunk (NBS blocks: one
//    slice) takes that, the others the larger (NBL: q, k and v from one pass
//    over X).
//
//    Bound by X and A^T from the caches and HBM, by round trips on small
//    batches.  Against the form before (rows gathered as MFMA operands, a
//    cache line per lane; 16 x 16 units up to 512 tokens, with K split over
//    the XCDs and a second launch for scattered adapters), kernel trace: 8B
//    layer, 150 tokens 18 -> 14 us, 333 tokens 30 -> 21 us, 4096 tokens 54
//    -> 47 us (119 MB of X: 2.5 TB/s); 70B, 256 tokens over 128 adapters,
//    beside the base product, 99 (both launches) -> 102 us, the step 155 ->
//    148 us; 70B, 4288 tokens, 117 us as before.
// --------------------------------------------------------------------------

// LDS (u32x4): the waves' X buffers, then (overlaid) their sums
constexpr int shrink_lds(int mb, int nb) { return kWaves * 64 * mb * (nb > 2 ? nb : 2); }

template <int MB, int NB, bool BIG>
__device__ __forceinline__ void shrink_unit(const FwdArgs& a, const ProjLaunch& P, const int4& it, int chunk, u32x4* lds) {
    constexpr int D0 = 144 / (8 * (MB + NB)), D = D0 > 8 ? 8 : D0 < 2 ? 2 : D0;      // pairs in flight
    const int w = wave_id(), l = threadIdx.x & 63;
    const int slot = it.x, nrows = it.z, r8s = it.w, ncols = P.n_slices * r8s, cb0 = chunk * NB;
    const float sc = a.scale[slot];
    const int* prow = a.perm + it.y;
    const int KS = P.K >> 5, NP = (KS + 1) >> 1, nblk = (ncols + 15) >> 4;
    const uint16_t* abase = a.pool + (size_t)slot * a.slot_stride + P.a_off;
    __amdgpu_buffer_rsrc_t ra[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) ra[cb] = buf_rsrc(abase + frag_index(min(cb0 + cb, nblk - 1), 0, KS), KS * 1024u);
    int g0, n;                                         // this wave's pairs
    wave_krange(NP, w, &g0, &n);
    XRows<MB, BIG> x;
    auto row = [=](int r) { return prow[min(r, nrows - 1)]; };
    if (P.X)
        x.init(P.X, P.K, a.T, lds + w * MB * 128, row);
    else
        x.init_packed(P.Xp, P.K, a.T, lds + w * MB * 128, row);
    f32x4 acc[MB][NB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 av[D][2][NB], xv[D][MB][2];
    auto load = [&](int d, int i) __attribute__((always_inline)) {
        const bool ok = i < n;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
                av[d][e][cb] = buf16(ra[cb], ok ? (unsigned)(2 * (g0 + i) + e) * 1024u + l * 16u : kOob);
        x.load(xv[d], g0 + i, ok);
    };
    auto comp = [&](int d, int i) __attribute__((always_inline)) {
        x.put(xv[d]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (2 * (g0 + i) + e >= KS) continue;      // an odd K's last pair holds one k-step
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                const u32x4 xf = x.get(rb, e);
#pragma unroll
                for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = mfma(av[d][e][cb], xf, acc[rb][cb]);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d);
    int i = 0;
    for (; i + D < n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            comp(d, i + d);
            load(d, i + d + D);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (i + d < n) comp(d, i + d);
    // the waves' sums in lane order (fragment (rb, cb) of wave w at
    // ((w MB + rb) NB + cb) 64 + lane), added in wave order
    f32x4* const red = reinterpret_cast<f32x4*>(lds);
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) red[((w * MB + rb) * NB + cb) * 64 + l] = acc[rb][cb];
    __syncthreads();
    constexpr int FR = MB * NB * 64;
    for (int e = threadIdx.x; e < FR; e += kThreads) {
        f32x4 v = red[e];
#pragma unroll
        for (int ww = 1; ww < kWaves; ++ww) v += red[ww * FR + e];
        // 4 consecutive rows of A^T (ranks of one octet) of one token
        const int fr = e >> 6, ln = e & 63, rb = fr / NB, cb = fr - rb * NB;
        const int r = rb * 16 + (ln & 15), vr = (cb0 + cb) * 16 + 4 * (ln >> 4);
        if (r < nrows && vr < ncols) {
            const int t = prow[r], sig = vr / r8s, j = vr - sig * r8s;
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float z = sc * v[q];
                hi[q] = f2bf(z);
                lo[q] = f2bf(z - bf2f((uint16_t)hi[q]));
            }
            uint16_t* zp = P.Z + (size_t)t * P.zs + sig * a.r8max + j;
            *reinterpret_cast<uint2*>(zp) = make_uint2(hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16));
            *reinterpret_cast<uint2*>(zp + P.zplane) = make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
        }
    }
    __syncthreads();
}

template <int MB, int NBS, int NBL, bool BIG>
__global__ __launch_bounds__(kThreads) void shrink_kernel(FwdArgs) {
    const FwdArgs& a = kernel_args<FwdArgs>();
    __shared__ u32x4 lds[shrink_lds(MB, NBL)];
    __shared__ int s_unit[2];
    // (clamped: the plan writes at most items_bound items)
    const int n_items = min(a.meta[1], a.items_bound);
    int total = 0;
    for (int q = 0; q < a.n_proj; ++q) total += n_items * a.schunks[q];
    int u = blockIdx.x;                                // the first unit needs no counter
    for (int turn = 0; u < total; ++turn) {
        int next = 0;
        if (threadIdx.x == 0) next = (int)gridDim.x + atomicAdd(a.queue, 1);
        int p = a.sorder[0];
        for (int ps = 0; ps + 1 < a.n_proj && u >= n_items * a.schunks[p]; ++ps) {
            u -= n_items * a.schunks[p];
            p = a.sorder[ps + 1];
        }
        const ProjLaunch& P = a.p[p];
        const int item = u / a.schunks[p], chunk = u - item * a.schunks[p];
        const int4 it = a.items[item];
        const bool small = P.n_slices * a.r8max <= 16 * NBS;
        if (chunk * 16 * (small ? NBS : NBL) < P.n_slices * it.w) {
            if (NBS == NBL || !small)
                shrink_unit<MB, NBL, BIG>(a, P, it, chunk, lds);
            else
                shrink_unit<MB, NBS, BIG>(a, P, it, chunk, lds);
        }
        if (threadIdx.x == 0) s_unit[turn & 1] = next;
        __syncthreads();
        u = s_unit[turn & 1];
    }
}

// workgroups of the shrink kernel that the device holds at once (cached)
template <int MB, int NBS, int NBL, bool BIG>
int shrink_resident() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, cu = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, shrink_kernel<MB, NBS, NBL, BIG>, kThreads, 0) != hipSuccess)
            return 0;
        n = cu * (per > 1 ? per : 1);
    }
    return n;
}

hipError_t launch_shrink(const FwdArgs& a, int mb, int nb, hipStream_t s) {
    if (!a.queue) return hipErrorInvalidValue;
    long long total = 0;
    bool big = false;                    // X beyond 32-bit offsets (only with more than 512 tokens)
    for (int i = 0; i < a.n_proj; ++i) {
        if (a.sorder[i] < 0 || a.sorder[i] >= a.n_proj || a.schunks[i] < 1) return hipErrorInvalidValue;
        big = big || (long long)((a.T + 15) / 16 * 16) * a.p[i].K * 2 >= 0x7fffff00LL;
        total += (long long)a.items_bound * a.schunks[i];
    }
    if (total <= 0) return hipSuccess;
#define BDL_SHRINK_CASE(M, NS, NL, BG)                                                                    \
    if (mb == M && nb == NL && big == BG) {                                                               \
        const int r = shrink_resident<M, NS, NL, BG>();                                                   \
        if (r <= 0) return hipErrorInvalidValue;                                                          \
        const dim3 grid((unsigned)(total < r ? total : r));                                               \
        hipLaunchKernelGGL((shrink_kernel<M, NS, NL, BG>), grid, dim3(kThreads), 0, s, a);                \
        return hipGetLastError();                                                                         \
    }
    BDL_SHRINK_CASE(1, 1, 3, false) BDL_SHRINK_CASE(1, 2, 6, false) BDL_SHRINK_CASE(1, 4, 4, false)
    BDL_SHRINK_CASE(2, 1, 3, false) BDL_SHRINK_CASE(2, 2, 6, false) BDL_SHRINK_CASE(4, 4, 4, false)
    BDL_SHRINK_CASE(2, 1, 3, true) BDL_SHRINK_CASE(2, 2, 6, true) BDL_SHRINK_CASE(4, 4, 4, true)
#undef BDL_SHRINK_CASE
    return hipErrorInvalidValue;
}

// --------------------------------------------------------------------------
// 3. base GEMM with fused expand
// --------------------------------------------------------------------------

template <int MB, int NB>
__global__ __launch_bounds__(kThreads) void gemm_kernel(FwdArgs a) {
    constexpr int MT = MB * 16, NT = NB * 16, LD = NT + 4;
    __shared__ float red[4 * MT * LD];
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15;

    const int bid = blockIdx.x;
    int p = 0;
    while (p + 1 < a.n_proj && bid >= a.p[p + 1].tile_base) ++p;
    const ProjLaunch& P = a.p[p];
    const int local = bid - P.tile_base;
    const int mt = local / P.tiles_n, nt = local - mt * P.tiles_n;
    const int m0 = mt * MT, n0 = nt * NT;
    const int T = a.T, N = P.N, K = P.K;

    // expand inputs that do not depend on the base product: fetched first
    const int* codes = a.tile_oct + (size_t)mt * a.oct_cap;
    int code = codes[4 * w + (l >> 4)];
    int rvid[MB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        const int row = m0 + rb * 16 + lr;
        rvid[rb] = row < T ? a.vid[row] : -1;
    }

    // ---- base product X W_s^T over this wave's k-steps
    const int KS = K >> 5;
    const int nrb = (T + 15) >> 4, ncb = N >> 4;
    const uint16_t* ap[MB];
    const uint16_t* bp[NB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) ap[rb] = P.Xp + frag_index(min(mt * MB + rb, nrb - 1), 0, KS) + l * 8;
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) bp[cb] = P.W + frag_index(min(nt * NB + cb, ncb - 1), 0, KS) + l * 8;
    f32x4 acc[MB][NB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    int k0, nk;
    wave_krange(KS, w, &k0, &nk);
    if (P.Ws) {
        // INT4 base: same tile, the raw q on the matrix cores, scales in fp32
        const char* wq[NB];
        const uint16_t* wsc[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            const int blk = min(nt * NB + cb, ncb - 1);
            wq[cb] = reinterpret_cast<const char*>(P.W) + (size_t)blk * KS * kInt4FragBytes + l * 4;
            wsc[cb] = P.Ws + (size_t)blk * (KS / kInt4Group) * 16 + lr;
        }
        if (nk > 0) mma_range_int4<MB, NB, kStages>(acc, ap, wq, wsc, k0, nk);
    } else if (nk > 0) {
        mma_range<MB, NB, kStages>(acc, ap, bp, k0, nk, kFrag, kFrag);
    }

    // ---- expand: acc += Zhat B over the tile's octets (masked per token)
    int sig[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        const int c = n0 + cb * 16;
        int sgm = 0;
        while (sgm + 1 < P.n_slices && c >= P.slice_col[sgm + 1]) ++sgm;
        sig[cb] = sgm;
    }
    const u32x4 zero4 = u32x4{0u, 0u, 0u, 0u};
    for (int e = w;;) {
        if (!__any(code >= 0)) break;
        const int slot = code >> 12, r8s = (code >> 4) & 0xff, j0 = (code & 15) * 8;
        u32x4 bv[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            const int col = min(n0 + cb * 16 + lr, N - 1);
            bv[cb] = code >= 0 ? ld16(a.pool + (size_t)slot * a.slot_stride + P.b_off +
                                      (size_t)col * r8s + j0)
                               : zero4;
        }
        u32x4 zh[MB], zl[MB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            if (cb == 0 || sig[cb] != sig[cb - 1]) {
#pragma unroll
                for (int rb = 0; rb < MB; ++rb) {
                    const bool match = code >= 0 && rvid[rb] == slot;
                    const uint16_t* zp = P.Z + (size_t)(m0 + rb * 16 + lr) * P.zs + sig[cb] * a.r8max + j0;
                    zh[rb] = match ? ld16(zp) : zero4;
                    zl[rb] = match ? ld16(zp + P.zplane) : zero4;
                }
            }
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                acc[rb][cb] = mfma(zh[rb], bv[cb], acc[rb][cb]);
                acc[rb][cb] = mfma(zl[rb], bv[cb], acc[rb][cb]);
            }
        }
        e += kWaves;
        if (4 * e + 4 > a.oct_cap) break;
        code = codes[4 * e + (l >> 4)];
    }

    // ---- reduce the 8 waves and store bf16 (or fp32), two columns per thread
    reduce_waves<MB, NB>(acc, red);
    for (int idx = threadIdx.x; idx < MT * NT / 2; idx += kThreads) {
        const int r = idx / (NT / 2), c = (idx - r * (NT / 2)) * 2;
        const int row = m0 + r, col = n0 + c;
        if (row < T && col < N) {
            if (P.out_f32) {
                *reinterpret_cast<float2*>(P.out_f32 + (size_t)row * N + col) =
                    float2{red[r * LD + c], red[r * LD + c + 1]};
            } else {
                const uint32_t v = (uint32_t)f2bf(red[r * LD + c]) | ((uint32_t)f2bf(red[r * LD + c + 1]) << 16);
                *reinterpret_cast<uint32_t*>(P.out + (size_t)row * N + col) = v;
            }
        }
    }
}

hipError_t launch_gemm(const FwdArgs& a, int mb, int nb, hipStream_t s) {
    const dim3 grid(a.total_tiles), block(kThreads);
    if (a.total_tiles <= 0) return hipSuccess;
#define BDL_GEMM_CASE(M, NN)                                                   \
    if (mb == M && nb == NN) {                                                 \
        hipLaunchKernelGGL((gemm_kernel<M, NN>), grid, block, 0, s, a);        \
        return hipGetLastError();                                              \
    }
    // (batches above 256 tokens only: always 64 rows)
    BDL_GEMM_CASE(4, 1) BDL_GEMM_CASE(4, 2) BDL_GEMM_CASE(4, 4)
#undef BDL_GEMM_CASE
    return hipErrorInvalidValue;
}

// --------------------------------------------------------------------------
// packing (off the per-batch path)
// --------------------------------------------------------------------------

// rows-major [rows x K] -> fragment layout with rows padded to 16 (zeros)
__global__ void pack_rows_kernel(const uint16_t* src, uint16_t* dst, int rows, int K, long long frags) {
    const int l = threadIdx.x & 63;
    const int KS = K >> 5;
    for (long long f = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6; f < frags;
         f += ((long long)gridDim.x * blockDim.x) >> 6) {
        const int rb = (int)(f / KS), ks = (int)(f - (long long)rb * KS);
        const int row = rb * 16 + (l & 15);
        u32x4 v = u32x4{0u, 0u, 0u, 0u};
        if (row < rows) v = ld16(src + (size_t)row * K + ks * 32 + (l >> 4) * 8);
        *reinterpret_cast<u32x4*>(dst + (size_t)f * kFrag + l * 8) = v;
    }
}

hipError_t launch_pack_rows(const uint16_t* src, uint16_t* dst, int rows, int K, hipStream_t s) {
    const long long frags = (long long)((rows + 15) / 16) * (K / 32);
    if (frags == 0) return hipSuccess;
    long long blocks = (frags + 3) / 4;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src, dst, rows, K, frags);
    return hipGetLastError();
}

__global__ void copy_kernel(const uint16_t* src, uint16_t* dst, long long pieces) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < pieces; i += (long long)gridDim.x * blockDim.x)
        *reinterpret_cast<u32x4*>(dst + i * 8) = ld16(src + i * 8);
}

hipError_t launch_copy(const uint16_t* src, uint16_t* dst, long long elems, hipStream_t s) {
    if (elems < 8 || elems % 8) return hipErrorInvalidValue;
    const long long blocks = (elems / 8 + 255) / 256;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, src, dst, elems / 8);
    return hipGetLastError();
}

// INT4 base weight: nn.Linear rows of nibbles (low nibble = even input) and
// bf16 scales [N x K/128] -> the forward layout (one 32-bit word per lane and
// k-step, then the scales grouped per 16-column block).  Thread = one word or
// one scale.
__global__ void pack_int4_kernel(const uint8_t* q, const uint16_t* scales, uint32_t* dst_w, uint16_t* dst_s, int N,
                                 int K) {
    const long long words = (long long)N * K / 8, nsc = (long long)N * (K / 128);
    const int KS = K >> 5, G = K >> 7;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < words + nsc;
         i += (long long)gridDim.x * blockDim.x) {
        if (i < words) {
            const int l = (int)(i & 63);
            const long long f = i >> 6;
            const int rb = (int)(f / KS), ks = (int)(f - (long long)rb * KS);
            const int n = rb * 16 + (l & 15), k0 = ks * 32 + (l >> 4) * 8;
            const uint8_t* src = q + (size_t)n * (K / 2) + k0 / 2;
            uint32_t w = 0;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const uint32_t nib = (src[v >> 1] >> (4 * (v & 1))) & 15u;
                w |= nib << (4 * (v >> 1) + 16 * (v & 1));
            }
            dst_w[i] = w;
        } else {
            const long long j = i - words;
            const int c = (int)(j & 15);
            const long long r = j >> 4;
            const int rb = (int)(r / G), g = (int)(r - (long long)rb * G);
            dst_s[j] = scales[(size_t)(rb * 16 + c) * G + g];
        }
    }
}

hipError_t launch_pack_int4(const uint8_t* q, const uint16_t* scales, uint32_t* dst_w, uint16_t* dst_s, int N,
                            int K, hipStream_t s) {
    const long long total = (long long)N * K / 8 + (long long)N * (K / 128);
    if (total == 0) return hipSuccess;
    long long blocks = (total + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(pack_int4_kernel, dim3((unsigned)blocks), dim3(256), 0, s, q, scales, dst_w, dst_s, N, K);
    return hipGetLastError();
}

// slot tables of consecutive adapter slots, written in stream order after
// their slabs
__global__ void set_slots_kernel(int* r8, float* scale, int* loaded, SlotBatch b) {
    const int i = threadIdx.x;
    if (i < b.n) {
        r8[b.first + i] = b.r8[i];
        scale[b.first + i] = b.scale[i];
        loaded[b.first + i] = 1;
    }
}

hipError_t launch_set_slots(int* r8, float* scale, int* loaded, const SlotBatch& b, hipStream_t s) {
    if (b.n < 1 || b.n > kMaxSlotBatch) return hipErrorInvalidValue;
    hipLaunchKernelGGL(set_slots_kernel, dim3(1), dim3(64), 0, s, r8, scale, loaded, b);
    return hipGetLastError();
}

// adapter: paper layout -> pool layout
//   stage = [A_0 .. A_{S-1} | B_0 .. B_{S-1}],  A_s [K x r], B_s [r x n_s]
//   dst_a = A^T_cat in fragment layout: row s*r8 + j of A^T_cat is column j
//           of A_s (zero for j >= r), rows padded to a multiple of 16
//   dst_b = B^T_cat [N x r8] row-major: row n is column n of its slice's B
struct PackArgs {
    uint16_t* dst_a;
    uint16_t* dst_b;
    const uint16_t* stage;
    int K, S, rank, r8, N;
    int slice_out[kMaxSlices];
    int slice_col[kMaxSlices + 1];
};

__global__ void pack_adapter_kernel(PackArgs a) {
    const int KS = a.K >> 5;
    const int arows = a.S * a.r8;
    const long long na = (long long)((arows + 15) / 16) * KS * kFrag;
    const long long nb = (long long)a.N * a.r8;
    const long long a_elems = (long long)a.S * a.K * a.rank;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < na + nb;
         i += (long long)gridDim.x * blockDim.x) {
        if (i < na) {
            const long long f = i / kFrag;
            const int e = (int)(i - f * kFrag), l = e >> 3, q = e & 7;
            const int rb = (int)(f / KS), ks = (int)(f - (long long)rb * KS);
            const int row = rb * 16 + (l & 15), k = ks * 32 + (l >> 4) * 8 + q;
            uint16_t v = 0;
            if (row < arows) {
                const int s = row / a.r8, j = row - s * a.r8;
                if (j < a.rank) v = a.stage[(long long)s * a.K * a.rank + (long long)k * a.rank + j];
            }
            a.dst_a[i] = v;
        } else {
            const long long q = i - na;
            const int n = (int)(q / a.r8), j = (int)(q - (long long)n * a.r8);
            int s = 0;
            while (s + 1 < a.S && n >= a.slice_col[s + 1]) ++s;
            long long boff = a_elems;
            for (int u = 0; u < s; ++u) boff += (long long)a.rank * a.slice_out[u];
            uint16_t v = 0;
            if (j < a.rank) v = a.stage[boff + (long long)j * a.slice_out[s] + (n - a.slice_col[s])];
            a.dst_b[q] = v;
        }
    }
}

hipError_t launch_pack_adapter(uint16_t* dst_a, uint16_t* dst_b, const uint16_t* stage, int K, int n_slices,
                               const int* slice_out, int rank, int r8, hipStream_t s) {
    PackArgs a;
    a.dst_a = dst_a;
    a.dst_b = dst_b;
    a.stage = stage;
    a.K = K;
    a.S = n_slices;
    a.rank = rank;
    a.r8 = r8;
    int col = 0;
    for (int i = 0; i < kMaxSlices; ++i) a.slice_out[i] = i < n_slices ? slice_out[i] : 0;
    for (int i = 0; i <= kMaxSlices; ++i) {
        a.slice_col[i] = col;
        if (i < n_slices) col += slice_out[i];
    }
    a.N = col;
    const long long total = (long long)((n_slices * r8 + 15) / 16) * (K / 32) * kFrag + (long long)col * r8;
    if (total == 0) return hipSuccess;
    long long blocks = (total + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(pack_adapter_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace bdl
