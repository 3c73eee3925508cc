// Internal device helpers of the BD-LoRA shard kernels (gfx950, wave64).
//
// Matrix-core primitive: v_mfma_f32_16x16x32_bf16.  Lane l of a wave holds
//   A operand: row (l % 16), 8 consecutive k starting at 8 * (l / 16)
//   B operand: col (l % 16), the same 8 k
//   C/D      : col (l % 16), rows 4 * (l / 16) + i, i = 0..3
// Both operands are read straight from row-major, K-contiguous memory
// (activations [rows x K], nn.Linear weights [cols x K], transposed LoRA
// factors), one 16-byte load per lane per 16x32 block.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdl_launch.h"
#include "bdl_xaddr.h"

namespace bdl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// word 3 of a raw buffer resource on gfx950 (32-bit untyped data)
constexpr int kRawBufferWord3 = 0x00020000;

constexpr int kWaves = 8;                 // waves per workgroup (split K)
constexpr int kThreads = kWaves * 64;

__device__ __forceinline__ u32x4 ld16(const uint16_t* p) {
    return *reinterpret_cast<const u32x4*>(p);
}

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// fp32 -> bf16 bits, round to nearest, ties to even (finite inputs; NaN kept NaN)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// wave index as a scalar (uniform) value
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// MFMA fragment layout.  A K-contiguous matrix with rows padded to a
// multiple of 16 is stored as 1 KB fragments, fragment (rb, ks) holding the
// operand of one 16-row block for one 32-wide k-step exactly as the 64 lanes
// load it: element [(rb * KS + ks) * 512 + lane * 8 + i] is
// M[16 rb + lane % 16][32 ks + 8 (lane / 16) + i].  Weights, packed
// activations and the pool's A^T factors use it, so every operand load of a
// wave reads 1 KB of contiguous memory.
constexpr int kFrag = 512;                  // elements per fragment

__device__ __forceinline__ size_t frag_index(int rb, int ks, int KS) {
    return ((size_t)rb * KS + ks) * kFrag;
}

// Wave-level K loop over the contiguous k-step range [k0, k0 + n), n >= 1.
// ap[rb] / bp[cb] point at this lane's element of k-step 0; consecutive
// k-steps are sa / sb elements apart.  D stages of loads stay in flight: the
// loads of k-step i + D are issued right after the MFMAs of k-step i.  Load
// addresses are clamped to the last k-step, so the steady-state loop issues
// the same loads every iteration and each load's only consumer is the next
// iteration (the compiler cannot sink it next to its use); the last n % D
// k-steps are consumed after the loop.
template <int MB, int NB, int D>
__device__ __forceinline__ void mma_range(f32x4 (&acc)[MB][NB], const uint16_t* const (&ap)[MB],
                                          const uint16_t* const (&bp)[NB], int k0, int n, int sa,
                                          int sb) {
    u32x4 a[D][MB], b[D][NB];
    const int last = k0 + n - 1;
    auto load = [&](int d, int ks) {
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) b[d][cb] = ld16(bp[cb] + (size_t)ks * sb);
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) a[d][rb] = ld16(ap[rb] + (size_t)ks * sa);
    };
    auto comp = [&](int d) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = mfma(a[d][rb], b[d][cb], acc[rb][cb]);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, min(k0 + d, last));
    int i = 0;
    for (; i + D <= n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            comp(d);
            load(d, min(k0 + i + d + D, last));
        }
    }
    const int rem = n - i;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < rem) comp(d);
}

// INT4 base weights.  One 32-bit word per lane and k-step holds the 8 values
// of the lane's B operand as nibbles q + 8, value i in bits 4 (i/2) + 16 (i%2).
// Each nibble u becomes the bf16 number 128 + u (exponent of 128, u in the low
// mantissa bits), which is exact; an extra MFMA against -136 removes the
// offset, so the matrix cores see exactly sum_k x_k q_k for the k-step.  The
// group scale is applied in fp32 to that k-step's product.  (The 64-row kernel;
// the decode launch and the large tiles take the form after it.)
constexpr int kInt4Group = 4;                 // k-steps per scale group (128 inputs)
constexpr int kInt4FragBytes = 256;           // one k-step of one 16-column block

__device__ __forceinline__ u32x4 unpack_int4(uint32_t w) {
    return u32x4{(w & 0x000F000Fu) | 0x43004300u, ((w >> 4) & 0x000F000Fu) | 0x43004300u,
                 ((w >> 8) & 0x000F000Fu) | 0x43004300u, ((w >> 12) & 0x000F000Fu) | 0x43004300u};
}

__device__ __forceinline__ u32x4 int4_offset_operand() {
    return u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};   // bf16 -136 x 8
}

// The same with 16 + u (u in the mantissa bits 6..3) and an offset of -24: one
// more shift per fragment, and the offset's rounding is 5.7 times smaller,
// for sums over a pair of k-steps or a whole scale group.
// (m = 0x00780078 and c = 0x41804180 in registers: one and-or per word then)
__device__ __forceinline__ u32x4 unpack_int4_16(uint32_t w, uint32_t m, uint32_t c) {
    return u32x4{((w << 3) & m) | c, ((w >> 1) & m) | c, ((w >> 5) & m) | c, ((w >> 9) & m) | c};
}

__device__ __forceinline__ u32x4 int4_offset16_operand() {
    return u32x4{0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u};   // bf16 -24 x 8
}

// acc[rb][cb] += s_cb * (x_rb . q_cb) for one k-step: xa = activation
// fragments, q[cb] = the INT4 words, sc[cb] = bf16 scale bits (low half).
template <int MB, int NB>
__device__ __forceinline__ void mma_int4_kstep(f32x4 (&acc)[MB][NB], const u32x4 (&xa)[MB], const uint32_t (&q)[NB],
                                               const uint32_t (&sc)[NB]) {
    const u32x4 off = int4_offset_operand();
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 w[NB];
    float s[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        w[cb] = unpack_int4(q[cb]);
        s[cb] = __uint_as_float(sc[cb] << 16);
    }
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        const f32x4 corr = mfma(xa[rb], off, zero);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            const f32x4 t = mfma(xa[rb], w[cb], corr);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[rb][cb][i] = fmaf(s[cb], t[i], acc[rb][cb][i]);
        }
    }
}

// mma_range for an INT4 B operand: wq[cb] points at this lane's word of
// k-step 0 of block cb (k-steps kInt4FragBytes apart), ws[cb] at the block's
// scale of group 0 for this lane's column (groups 16 entries apart).
template <int MB, int NB, int D>
__device__ __forceinline__ void mma_range_int4(f32x4 (&acc)[MB][NB], const uint16_t* const (&ap)[MB],
                                               const char* const (&wq)[NB], const uint16_t* const (&ws)[NB],
                                               int k0, int n) {
    u32x4 a[D][MB];
    uint32_t q[D][NB], sc[D][NB];
    const int last = k0 + n - 1;
    auto load = [&](int d, int ks) {
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
            q[d][cb] = *reinterpret_cast<const uint32_t*>(wq[cb] + (size_t)ks * kInt4FragBytes);
            sc[d][cb] = ws[cb][(ks / kInt4Group) * 16];
        }
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) a[d][rb] = ld16(ap[rb] + (size_t)ks * kFrag);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, min(k0 + d, last));
    int i = 0;
    for (; i + D <= n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            mma_int4_kstep<MB, NB>(acc, a[d], q[d], sc[d]);
            load(d, min(k0 + i + d + D, last));
        }
    }
    const int rem = n - i;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < rem) mma_int4_kstep<MB, NB>(acc, a[d], q[d], sc[d]);
}

// The kernel's by-value argument where the launch put it.  (Named as a
// parameter and indexed with a projection number that depends on the
// workgroup, it would be copied to scratch memory first.)
template <class T>
__device__ __forceinline__ const T& kernel_args() {
    return *(const T*)(const __attribute__((address_space(4))) T*)__builtin_amdgcn_kernarg_segment_ptr();
}

constexpr unsigned kOob = 0x7ffffff0u;      // byte offset past every buffer: the load returns zeros

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, kRawBufferWord3);
}

__device__ __forceinline__ u32x4 buf16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

// Activations.  A wave takes the caller's row-major X in pairs of k-steps: 16
// rows x 128 bytes with two loads in which eight lanes cover a row's line
// (lanes 16 rows apart, as the MFMA operand wants them, would touch a line per
// lane), through its own buffer in LDS, from which the operand fragments
// are read.  Lane l takes row 8 h + l / 8 and chunk (l mod 8) ^
// swizzle(row), so that both sides hit distinct banks.
__device__ __forceinline__ int x_swz(int r) { return ((r >> 1) ^ ((r & 1) << 2)) & 7; }

// BIG: X of 2 GB or more, beyond a buffer's 32-bit offsets (64-bit addresses,
// which no bounds check guards: every load lies inside X by x_pair_offset, and
// one that is not wanted repeats the row's first pair, unused).
template <int MB, bool BIG = false>
struct XRows {
    __amdgpu_buffer_rsrc_t rx;
    unsigned ro[MB][2];     // byte offset of this lane's chunk of pair 0
    unsigned st;            // bytes from one pair to the next
    const char* rp[BIG ? MB : 1][2];   // BIG: the chunk's address instead,
    int kx, ch[2];          // the inputs of a row and the chunk
    bool pk;                // and whether X is packed
    u32x4* buf;             // this wave's MB x 128 pieces
    int pos[2];             // where this lane's operand of k-step e of a pair lies in a row block

    // row(i): the X row of row i of the MB 16-row blocks
    template <class Row>
    __device__ __forceinline__ void init(const uint16_t* X, int K, int T, u32x4* lds, Row row) {
        const int l = threadIdx.x & 63;
        rx = buf_rsrc(X, (unsigned)T * K * 2u);
        buf = lds;
        st = 128u;
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = 8 * h + (l >> 3);
                const unsigned c = (unsigned)((l & 7) ^ x_swz(r)) * 16u;
                if constexpr (BIG)
                    rp[rb][h] = reinterpret_cast<const char*>(X) + x_chunk_offset(false, row(rb * 16 + r), K, (int)c >> 4);
                else
                    ro[rb][h] = (unsigned)row(rb * 16 + r) * K * 2u + c;
            }
        init_pos(K, false);
    }
    // the same from X in the fragment layout (rows padded to 16)
    template <class Row>
    __device__ __forceinline__ void init_packed(const uint16_t* Xp, int K, int T, u32x4* lds, Row row) {
        const int l = threadIdx.x & 63;
        const unsigned KS = (unsigned)K >> 5;
        rx = buf_rsrc(Xp, (unsigned)((T + 15) >> 4) * KS * 1024u);
        buf = lds;
        st = 2048u;
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = 8 * h + (l >> 3), c = (l & 7) ^ x_swz(r), t = row(rb * 16 + r);
                const unsigned o = (unsigned)((t & 15) + 16 * (c & 3)) * 16u + (unsigned)(c >> 2) * 1024u;
                if constexpr (BIG)
                    rp[rb][h] = reinterpret_cast<const char*>(Xp) + x_chunk_offset(true, t, K, c);
                else
                    ro[rb][h] = (unsigned)(t >> 4) * KS * 1024u + o;
            }
        init_pos(K, true);
    }
    __device__ __forceinline__ void init_pos(int K, bool packed) {
        const int l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
        if constexpr (BIG) {
            kx = K;
            pk = packed;
#pragma unroll
            for (int h = 0; h < 2; ++h) ch[h] = (l & 7) ^ x_swz(8 * h + (l >> 3));
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) pos[e] = (lr >> 3) * 64 + (lr & 7) * 8 + ((4 * e + lg) ^ x_swz(lr));
    }
    // pair g (its k-steps 2 g, 2 g + 1); ok false: zeros, no memory traffic
    __device__ __forceinline__ void load(u32x4 (&v)[MB][2], int g, bool ok) const {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (BIG)
                    v[rb][h] = *reinterpret_cast<const u32x4*>(rp[rb][h] + x_pair_offset(pk, kx, ch[h], ok ? g : 0));
                else
                    v[rb][h] = buf16(rx, ok ? ro[rb][h] + (unsigned)g * st : kOob);
            }
    }
    // (the wave's LDS operations run in order, so one buffer does: a pair is
    // written after the last one's reads; the fences keep the compiler's order)
    __device__ __forceinline__ void put(const u32x4 (&v)[MB][2]) const {
        const int l = threadIdx.x & 63;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int h = 0; h < 2; ++h) buf[rb * 128 + h * 64 + l] = v[rb][h];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __device__ __forceinline__ u32x4 get(int rb, int e) const { return buf[rb * 128 + pos[e]]; }
};

// minimum / bitwise or over the 64 lanes of a wave, as a uniform value
__device__ __forceinline__ int wave_min(int v) {
    constexpr int kMax = 0x7fffffff;
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ unsigned wave_or(unsigned v) {
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
    v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// inclusive prefix sum over the 64 lanes of a wave (DPP row shifts, then row
// broadcasts of lanes 15 and 31)
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

__device__ __forceinline__ int wave_total(int incl) { return __builtin_amdgcn_readlane(incl, 63); }

// Contiguous k-step range of wave w when KS k-steps are split over kWaves.
__device__ __forceinline__ void wave_krange(int KS, int w, int* k0, int* n) {
    const int q = KS / kWaves, r = KS - q * kWaves;
    *k0 = w * q + min(w, r);
    *n = q + (w < r ? 1 : 0);
}

// Deterministic reduction of the 8 waves' accumulators of one MT x NT tile
// (MT = 16 MB, NT = 16 NB) through LDS: (w0+w4)+(w2+w6) + (w1+w5)+(w3+w7).
// On return red[r * (NT + 4) + c] holds the tile sum for every thread.
// red must hold 4 * MT * (NT + 4) floats.
template <int MB, int NB>
__device__ __forceinline__ void reduce_waves(f32x4 (&acc)[MB][NB], float* red) {
    constexpr int NT = NB * 16, MT = MB * 16, LD = NT + 4, REG = MT * LD;
    const int w = wave_id(), l = threadIdx.x & 63;
    auto put = [&](float* dst) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    dst[(rb * 16 + 4 * (l >> 4) + i) * LD + cb * 16 + (l & 15)] = acc[rb][cb][i];
    };
    auto add = [&](const float* src) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[rb][cb][i] += src[(rb * 16 + 4 * (l >> 4) + i) * LD + cb * 16 + (l & 15)];
    };
    if (w >= 4) put(red + (w - 4) * REG);
    __syncthreads();
    if (w < 4) add(red + w * REG);
    __syncthreads();
    if (w >= 2 && w < 4) put(red + (w - 2) * REG);
    __syncthreads();
    if (w < 2) add(red + w * REG);
    __syncthreads();
    if (w == 1) put(red);
    __syncthreads();
    if (w == 0) {
        add(red);
        put(red);
    }
    __syncthreads();
}

}  // namespace bdl
