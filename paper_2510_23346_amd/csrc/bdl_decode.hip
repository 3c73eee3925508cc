// Decode path (batches of at most kDecodeMaxT tokens): one launch.
//
// Workgroups, in launch order:
//   shrink  Z = scale * X A for each token's own adapter (step "Z <- X A" of
//           Alg. 1 / Alg. 2), one or four 16-row blocks of A^T and 16 tokens
//           at a time;
//   main    out = X W_s + Z B: each owns some columns over the whole K (its
//           waves split K and meet in LDS), adds the expand (steps "Y_adapter
//           <- Z B", "Y <- Y + Y_adapter") as extra MFMA k-steps and stores
//           bf16 once.  No partial sum leaves the CU.
// A main workgroup streams its weights at once; only before the expand it
// waits for its projection's shrink workgroups (flags in device memory, see
// raise_flag).  Those are launched first and are usually done by then; a wait
// that runs past a time limit (other work can hold the CUs that they need)
// ends with the workgroup computing that Z itself, so that no workgroup ever
// depends on another one being scheduled.
#include "bdl_device.h"

namespace bdl {

// A producer workgroup raises its own 64-bit flag in device memory once its
// stores have reached memory: the flag takes the launch's tag.  (One counter
// that all producers add to costs about 40 ns per addition.)  What a
// producer writes for others is whole cache lines, written through; no cache
// of a consumer can hold an older copy, since nothing reads that memory
// earlier in the launch and a launch starts with its caches invalidated.
//
// The tag is the number of the launch among those on this pool's flags, so that
// no flag needs a reset, also where a captured launch is replayed.  Every
// workgroup keeps its own count of them (a.count): it reads its word, which
// no other one touches in the launch, and at its end writes it back one higher,
// with its share of the words that no workgroup of this launch has; so after
// every launch all words agree.  (8B layer, one token: 15.9 us; 15.6 with the
// packet's number in its queue and the queue's address for a tag, which repeat
// where a new queue gets an old one's address; 24.6 with the id that HSA gives
// each queue, which lies in host memory; 16.6 with one count for all, raised by
// the last workgroup that has read it: a wave's later loads wait behind the
// atomic operation's answer.)  The packet's number still stands beside the
// count: it costs nothing, and tells launches apart where calls on one pool
// overlapped against the rules.
extern "C" __device__ unsigned long long bdl_dispatch_id() __asm("llvm.amdgcn.dispatch.id");

__device__ __forceinline__ unsigned launch_no(const DecArgs& a) { return a.count[blockIdx.x] + 1; }

// one wave, once it has the number
__device__ __forceinline__ void count_launch(const DecArgs& a, unsigned no) {
    const int l = threadIdx.x & 63, s0 = gridDim.x + blockIdx.x * a.count_share;
    if (l == 0) a.count[blockIdx.x] = no;
    for (int i = s0 + l; i < min(s0 + a.count_share, a.counts); i += 64) a.count[i] = no;
}

__device__ __forceinline__ unsigned long long launch_tag(unsigned no) {
    return (unsigned long long)no << 32 | (unsigned)bdl_dispatch_id();
}

// every wave of a producer: its stores have reached memory
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void raise_flag(const DecArgs& a, int i, unsigned no) {
    __hip_atomic_store(a.flags + i, launch_tag(no), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// one wave: wait for flags i0 .. i0 + n - 1, whose workgroups have about `units`
// to do per `share` of them; false when the time limit for that passed
__device__ __forceinline__ bool wait_flags(const DecArgs& a, int i0, int n, unsigned no, int units, int share) {
    if (a.wait_ticks == 0) return false;
    const int l = threadIdx.x & 63;
    const unsigned long long tag = launch_tag(no), t0 = __builtin_amdgcn_s_memrealtime();
    for (int i = 0; i < n;) {
        const unsigned long long f = __hip_atomic_load(a.flags + i0 + min(i + l, n - 1), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
        if (__all(f == tag)) {
            i += 64;
        } else {
            if ((__builtin_amdgcn_s_memrealtime() - t0) * share > (unsigned long long)a.wait_ticks * (share + units)) return false;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return true;
}

// z as three bf16 numbers whose sum is exactly z (8 significant bits each,
// cut towards zero so that nothing overflows); the parts of an infinity or a
// NaN past the first are zero
__device__ __forceinline__ void split3(float z, uint32_t (&b)[3]) {
    const uint32_t u = __float_as_uint(z), h = u & 0xffff0000u;
    const bool fin = (u & 0x7f800000u) != 0x7f800000u;
    const float r = fin ? z - __uint_as_float(h) : 0.f;
    const uint32_t m = __float_as_uint(r) & 0xffff0000u;
    const float q = r - __uint_as_float(m);
    b[0] = h >> 16;
    b[1] = m >> 16;
    b[2] = __float_as_uint(q) >> 16;
}

// The plan of T <= 64 tokens from t0 on, computed by one wave (lane t holds
// token t0 + t):
// ids checked against the loaded slots, the adapters in use in ascending slot
// order ("groups"; at most act_max of them: any past that bound, possible
// only when a captured forward replays after more adapters were loaded, are
// treated as none and raise the error flag).  Pools of at most 64 slots keep
// the slot tables in lanes (one load round trip) and send each slot in use to
// the lane of its rank among them; larger pools look the tables up per token
// and take the smallest remaining slot per pass.
struct PlanLoads {
    int lt, rt, id;
};

struct Plan {
    int n;          // groups (uniform)
    int gs, gr;     // lane g: slot and padded rank of group g (0 from the count on)
    int vid, mine;  // lane t: validated id and group of token t (-1: none)
    bool bad;       // some id named no adapter (uniform)
};

__device__ __forceinline__ PlanLoads dec_plan_loads(const DecArgs& a, int t0, int T) {
    const int l = threadIdx.x & 63;
    const bool small = a.max_slots <= 64;
    PlanLoads r;
    r.lt = small && l < a.max_slots ? a.loaded[l] : 0;
    r.rt = small && l < a.max_slots ? a.r8[l] : 0;
    r.id = -1;
    if (a.ids) {
        if (l < T) r.id = a.ids[t0 + l];
    } else {
        // segments in token order: the last one starting at or before t
        for (int i = 0; i < a.n_seg; ++i)
            if (t0 + l >= a.seg_start[i]) r.id = a.seg_slot[i];
        if (l >= T) r.id = -1;
    }
    return r;
}

__device__ __forceinline__ Plan dec_plan(const DecArgs& a, const PlanLoads& ld, int T) {
    const int l = threadIdx.x & 63;
    const bool in = l < T;
    const bool small = a.max_slots <= 64;
    const int lt = ld.lt, rt = ld.rt, id = ld.id;
    const bool in_range = id >= 0 && id < a.max_slots;
    int lv, r8v;
    if (small) {
        lv = __shfl(lt, in_range ? id : 0);
        r8v = __shfl(rt, in_range ? id : 0);
        if (!in_range) lv = r8v = 0;
    } else {
        lv = in_range ? a.loaded[id] : 0;
        r8v = in_range ? a.r8[id] : 0;
    }
    bool ok = in_range && lv != 0;
    bool bad = __ballot(in && !ok && id != -1) != 0ull;
    int g = 0, mine = -1, gs = 0, gr = 0;
    const int v = ok ? id : -1;
    if (small) {
        const unsigned long long bit = ok ? 1ull << v : 0ull;
        const unsigned long long used =
            (unsigned long long)wave_or((unsigned)bit) | ((unsigned long long)wave_or((unsigned)(bit >> 32)) << 32);
        g = __popcll(used);
        // lane l holds slot l: a slot in use goes to the lane of its rank
        // among them, the other lanes to the lanes from g on (together a
        // permutation of the 64 lanes)
        const int below = __popcll(used & ((1ull << l) - 1ull));
        const int to = ((used >> l) & 1ull) ? below : g + (l - below);
        gs = __builtin_amdgcn_ds_permute(to * 4, l);
        gr = __builtin_amdgcn_ds_permute(to * 4, rt);
        if (ok) mine = __popcll(used & (bit - 1ull));
    } else {
        unsigned long long rem = __ballot(ok);
        while (rem) {
            const int m = wave_min(((rem >> l) & 1ull) ? v : 0x7fffffff);
            const bool eq = ok && v == m;
            if (eq) mine = g;
            // slot m's rank: held by every lane whose token uses it
            const int rm = __builtin_amdgcn_readlane(r8v, __ffsll((long long)__ballot(eq)) - 1);
            if (l == g) {
                gs = m;
                gr = rm;
            }
            ++g;
            rem &= ~__ballot(eq);
        }
    }
    if (g > a.act_max) {
        const bool over = ok && mine >= a.act_max;
        bad = bad || __ballot(over) != 0ull;
        if (over) {
            ok = false;
            mine = -1;
        }
        g = a.act_max;
    }
    if (l >= g) gs = gr = 0;
    return Plan{__builtin_amdgcn_readfirstlane(g), gs, gr, ok ? v : -1, mine, bad};
}

// shrink items per group (lane g): its tokens, 16 at a time.  cnt: 64 ints of
// this wave's LDS
__device__ __forceinline__ int dec_items(const Plan& pl, int* cnt) {
    const int l = threadIdx.x & 63;
    cnt[l] = 0;
    __builtin_amdgcn_wave_barrier();
    if (pl.mine >= 0) atomicAdd(&cnt[pl.mine], 1);
    __builtin_amdgcn_wave_barrier();
    return (cnt[l] + 15) >> 4;
}

// Z of row group g
__device__ __forceinline__ uint16_t* dec_z(const DecArgs& a, const DecProj& P, int g) {
    return P.Z + (size_t)g * P.nbA * a.rows * kDecZLine;
}

// Z of row blocks c0 .. c0 + nb - 1 (nb <= NBA) of A^T for 16 tokens (row block
// rb) of group ai, stored as one 128-byte line per (block, token): three planes
// of 16 bf16 numbers.  The workgroup's waves split K; a wave's loads run
// through a ring of D pairs of k-steps; the tokens are the MFMA's columns.
// One block a workgroup gives the shortest launch while the workgroups are
// resident at once, four read X once for all and are a fourth as many (see
// DecArgs::merge).
constexpr int kShrinkMerge = 4;

template <int NW, int NBA>
__device__ __forceinline__ void dec_shrink(const DecArgs& a, const DecProj& P, const Plan& pl, int ai, int rb, int c0,
                                           int nb, const uint16_t* X, uint16_t* Z, int T, u32x4* lds) {
    constexpr int D = NBA == 1 ? 8 : 4;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
    const int slot = __builtin_amdgcn_readlane(pl.gs, ai);
    const float sc = a.scale[slot];
    // the adapter's tokens in ascending order: lane i gets the i-th
    const unsigned long long m = __ballot(pl.mine == ai), lt = (1ull << l) - 1ull;
    const int cnt = __popcll(m), below = __popcll(m & lt);
    const int toks = __builtin_amdgcn_ds_permute((pl.mine == ai ? below : cnt + (l - below)) * 4, l);
    const int t = __shfl(toks, min(rb * 16 + lr, cnt - 1));      // the token of this lane's MFMA column

    const int KS = P.K >> 5, NP = (KS + 1) >> 1, g0 = NP * w / NW, n = NP * (w + 1) / NW - g0;
    __amdgpu_buffer_rsrc_t ra[NBA];                               // (blocks past nb: of no size)
#pragma unroll
    for (int b = 0; b < NBA; ++b)
        ra[b] = buf_rsrc(a.pool + (size_t)slot * a.slot_stride + P.a_off + frag_index(c0 + min(b, nb - 1), 0, KS),
                         b < nb ? KS * 1024u : 0u);
    XRows<1> x;
    x.init(X, P.K, T, lds + w * 128, [=](int r) { return __shfl(toks, min(rb * 16 + r, cnt - 1)); });
    f32x4 acc[NBA];
#pragma unroll
    for (int b = 0; b < NBA; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 av[D][2][NBA], xv[D][1][2];
    auto load = [&](int d, int i) __attribute__((always_inline)) {
        const bool ok = i < n;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int b = 0; b < NBA; ++b)
                av[d][e][b] = buf16(ra[b], ok ? (unsigned)(2 * (g0 + i) + e) * 1024u + l * 16u : kOob);
        x.load(xv[d], g0 + i, ok);
    };
    auto comp = [&](int d, int i) __attribute__((always_inline)) {
        x.put(xv[d]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (2 * (g0 + i) + e >= KS) continue;    // an odd K's last pair holds one k-step
            const u32x4 xf = x.get(0, e);
#pragma unroll
            for (int b = 0; b < NBA; ++b) acc[b] = mfma(av[d][e][b], xf, acc[b]);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d);
    __builtin_amdgcn_sched_barrier(0);                // every load above is in flight before the first MFMA
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
    f32x4* const red = reinterpret_cast<f32x4*>(lds) + (NBA == 1 ? NW * 128 : 0);
    if (NBA > 1) __syncthreads();                     // every wave is past its X buffer, which red overlays
#pragma unroll
    for (int b = 0; b < NBA; ++b) red[(b * NW + w) * 64 + l] = acc[b];
    __syncthreads();
    // wave b, block b: lane = 4 consecutive rows of A^T (ranks of one octet) of one token
    if (w < nb) {
        f32x4 v = red[w * NW * 64 + l];
#pragma unroll
        for (int q = 1; q < NW; ++q) v += red[(w * NW + q) * 64 + l];
        if (rb * 16 + lr < cnt) {
            uint32_t b[4][3];
#pragma unroll
            for (int e = 0; e < 4; ++e) split3(sc * v[e], b[e]);
            uint16_t* z = Z + ((size_t)(c0 + w) * a.rows + t) * kDecZLine + 4 * lg;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                __hip_atomic_store(reinterpret_cast<unsigned long long*>(z + 16 * q),
                                   (unsigned long long)(b[0][q] | (b[1][q] << 16)) |
                                       ((unsigned long long)(b[2][q] | (b[3][q] << 16)) << 32),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        stores_done();
    }
    __syncthreads();
}

// K loop of column blocks C0 .. C0 + NC - 1 of the wave, bf16 base: part kq
// of kparts of K, in pairs of k-steps through a ring of D pairs of loads
// (those past the part's end return zeros without touching memory).  pre runs
// once the ring's first loads are issued, mid before its last pass.
template <int MB, int NB, int C0, int NC, class Pre, class Mid>
__device__ __forceinline__ void dec_k_bf16(f32x4 (&acc)[MB][NB], const DecProj* const (&Pc)[NB], const int (&blk)[NB],
                                           const XRows<MB>& x, int KS, int kq, int kparts, Pre pre, Mid mid) {
    constexpr int D = MB <= 1 ? 4 : 2;
    const int l = threadIdx.x & 63, NP = (KS + 1) >> 1, g0 = NP * kq / kparts, n = NP * (kq + 1) / kparts - g0;
    __amdgpu_buffer_rsrc_t rw[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) rw[c] = buf_rsrc(Pc[C0 + c]->W + frag_index(blk[C0 + c], 0, KS), KS * 1024u);
    u32x4 wv[D][2][NC], xv[D][MB][2];
    auto load = [&](int d, int i) __attribute__((always_inline)) {
        const bool ok = i < n;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                wv[d][e][c] = buf16(rw[c], ok ? (unsigned)(2 * (g0 + i) + e) * 1024u + l * 16u : kOob);
        x.load(xv[d], g0 + i, ok);
    };
    auto comp = [&](int d, int i) __attribute__((always_inline)) {
        x.put(xv[d]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (2 * (g0 + i) + e >= KS) continue;    // an odd K's last pair holds one k-step
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                const u32x4 xf = x.get(rb, e);
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[rb][C0 + c] = mfma(wv[d][e][c], xf, acc[rb][C0 + c]);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d);
    pre();
    int i = 0;
    for (; i + D < n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            comp(d, i + d);
            load(d, i + d + D);
        }
    }
    mid();
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (i + d < n) comp(d, i + d);
}

// The same on an INT4 base, in scale groups of 4 k-steps.  With q + 8 held as
// 16 + (q + 8), the sum of x (24 + q) over a pair of k-steps, begun at
// -24 sum x, is sum x q; the group's scale is applied to it in fp32.  (Begun
// there, so that no large sum is rounded: the two added up over a whole group
// apart, with 128 + (q + 8), were 4 times less exact, and 10 times with
// activations of mean 1.)
template <int MB, int NB, int C0, int NC, class Pre, class Mid>
__device__ __forceinline__ void dec_k_int4(f32x4 (&acc)[MB][NB], const DecProj* const (&Pc)[NB], const int (&blk)[NB],
                                           const XRows<MB>& x, int KS, int kq, int kparts, Pre pre, Mid mid) {
    constexpr int D = MB <= 2 ? 2 : 1;                // groups of activations in flight
    constexpr int DW = 2;                             // groups of weights in flight
    const int l = threadIdx.x & 63, lg = l >> 4, G = KS >> 2, g0 = G * kq / kparts, n = G * (kq + 1) / kparts - g0;
    __amdgpu_buffer_rsrc_t rw[NC], rs[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const DecProj& P = *Pc[C0 + c];
        rw[c] = buf_rsrc(reinterpret_cast<const char*>(P.W) + (size_t)blk[C0 + c] * KS * kInt4FragBytes,
                         KS * (unsigned)kInt4FragBytes);
        rs[c] = buf_rsrc(P.Ws + (size_t)blk[C0 + c] * G * 16, G * 32u);
    }
    uint32_t q[DW][NC][4];
    u32x4 xv[D][2][MB][2];
    uint2 sc[DW][NC];
    auto load_w = [&](int d, int i) __attribute__((always_inline)) {
        const unsigned g = g0 + i;
        const unsigned wo = i < n ? g * (4u * kInt4FragBytes) + l * 4u : kOob;
        const unsigned so = i < n ? g * 32u + lg * 8u : kOob;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                q[d][c][j] = __builtin_amdgcn_raw_buffer_load_b32(rw[c], (int)wo, j * kInt4FragBytes, 0);
            sc[d][c] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rs[c], (int)so, 0, 0));
        }
    };
    auto load_x = [&](int d, int h, int i) __attribute__((always_inline)) { x.load(xv[d][h], 2 * (g0 + i) + h, i < n); };
    const u32x4 off = int4_offset16_operand();
    uint32_t um = 0x00780078u, uc = 0x41804180u;
    asm("" : "+v"(um), "+v"(uc));
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    auto comp = [&](int dw, int dx, int next) __attribute__((always_inline)) {
        float s[NC][4];
        u32x4 wf[NC][4];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            s[c][0] = __uint_as_float(sc[dw][c].x << 16);
            s[c][1] = __uint_as_float(sc[dw][c].x & 0xffff0000u);
            s[c][2] = __uint_as_float(sc[dw][c].y << 16);
            s[c][3] = __uint_as_float(sc[dw][c].y & 0xffff0000u);
#pragma unroll
            for (int j = 0; j < 4; ++j) wf[c][j] = unpack_int4_16(q[dw][c][j], um, uc);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            x.put(xv[dx][h]);
            if (next >= 0) load_x(dx, h, next);
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                const u32x4 x0 = x.get(rb, 0), x1 = x.get(rb, 1);
                const f32x4 corr = mfma(off, x1, mfma(off, x0, zero));
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const f32x4 t = mfma(wf[c][2 * h + 1], x1, mfma(wf[c][2 * h], x0, corr));
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[rb][C0 + c][i] = fmaf(s[c][i], t[i], acc[rb][C0 + c][i]);
                }
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DW; ++d) load_w(d, d);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        load_x(d, 0, d);
        load_x(d, 1, d);
    }
    pre();
    int i = 0;
    for (; i + DW < n; i += DW) {
#pragma unroll
        for (int d = 0; d < DW; ++d) {
            comp(d, d % D, i + d + D);
            load_w(d, i + d + DW);
        }
    }
    mid();
#pragma unroll
    for (int d = 0; d < DW; ++d)
        if (i + d < n) comp(d, d % D, d + D < DW ? i + d + D : -1);
}

// Main workgroup: NW waves = ncg column groups x kparts parts of K (the host
// picks kparts per projection); a wave takes NB column blocks of 16
// (PAIR, the gated MLP: block 0 of gate and the same block of up) and all MB
// row blocks of the batch.  Its weight and activation fragments run through a
// ring of k-steps.  The K-parts also share the expand's turns and meet in LDS
// once.
//
// What bounds it: HBM (the base weight and the used adapters' A, each read
// once) and, around it, the launch's own start and end.  8B layer shard, weights from HBM,
// kernel trace, against the three launches this replaces (plan and packing;
// split-K sums of 11.9 MB in fp32 partial tiles; epilogue), which took one
// tile of 64 columns through memory between them:
//   1 token, 1 adapter                  25.2 -> 12.8 us (54.5 MB of weights: 4.3 TB/s)
//   16 tokens, 8 adapters of rank 16           17.2 us
//   37 tokens, ranks 8 and 64           44.1 -> 31.4 us
//   64 tokens, 26 adapters of rank 16   39.8 -> 30.4 us (75.4 MB: 2.5 TB/s)
//   the same on an INT4 base            40.2 -> 24.6 us
// At 64 tokens a workgroup moves 2 bytes of activations per byte of weight
// through its CU; two pairs of k-steps in flight per wave are what the
// registers hold (three waves per SIMD instead of two spill: 126 us).  One
// counter per projection instead of flags cost 5 us, packing the activations
// first (in the same launch) 5 us, a launch of its own for the shrink 7-10.
// ZS: the wave's column blocks read different Z (gate and up, or a slice that
// ends inside a pair of blocks).
template <int NW, int MB, int NB, bool Q4, bool PAIR, bool ZS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void dec_main_kernel(DecArgs) {
    const DecArgs& a = kernel_args<DecArgs>();
    static_assert(!PAIR || (NB == 2 && ZS), "gate and up");
    constexpr int XB = NW * MB * 128, RB = NW * MB * NB * 64, SB = NW * 64 * kShrinkMerge;   // the waves' X buffers; their sums; shrink
    __shared__ u32x4 lds[XB > RB ? (XB > SB ? XB : SB) : (RB > SB ? RB : SB)];
    f32x4* const red = reinterpret_cast<f32x4*>(lds);
    __shared__ int s_cnt[NW][64];
    __shared__ int s_vid[64];
    // row block << 25 | slot << 12 | r8 << 4 | octet, -1 padded to whole turns (a token has one adapter)
    __shared__ int s_oct[kDecodeMaxT * kMaxRank8 / 8 + 4 * MB];
    __shared__ int s_info[3];                                // turns; outcome of the wait; turns of one row block each
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lg = l >> 4;
    const int bid = blockIdx.x;

    if (bid < a.groups * a.n_shrink) {
        const int g = bid / a.n_shrink, sb = bid - g * a.n_shrink, t0 = g * a.rows, T = min(a.rows, a.T - t0);
        const unsigned no = launch_no(a);
        const Plan pl = dec_plan(a, dec_plan_loads(a, t0, T), T);
        if (sb == 0 && pl.bad && threadIdx.x == 0) atomicOr(a.err, 1);
        int p = 0;
#pragma unroll
        for (int q = 1; q < kMaxProjs; ++q)
            if (q < a.n_proj && sb >= a.shrink_base[q]) p = q;
        const DecProj& P = a.p[p];
        // what there is to do, adapter after adapter: its items (16 tokens) times
        // its blocks of A^T (times four of them, merged).  Mostly one each; the
        // host counts the workgroups by the adapters that it knows
        const int nb = (P.n_slices * pl.gr + 15) >> 4, ng = a.merge ? (nb + kShrinkMerge - 1) / kShrinkMerge : nb;
        const int units = dec_items(pl, s_cnt[w]) * ng, incl = wave_incl_scan(units);
        for (int u = sb - a.shrink_base[p]; u < wave_total(incl); u += P.n_shrink) {
            const int ai = __ffsll((long long)__ballot(incl > u)) - 1, nga = __builtin_amdgcn_readlane(ng, ai);
            const int k = u - (__builtin_amdgcn_readlane(incl, ai) - __builtin_amdgcn_readlane(units, ai)), rb = k / nga, c = k - rb * nga;
            if (a.merge)
                dec_shrink<NW, kShrinkMerge>(a, P, pl, ai, rb, c * kShrinkMerge,
                                             min(__builtin_amdgcn_readlane(nb, ai) - c * kShrinkMerge, kShrinkMerge),
                                             P.X + (size_t)t0 * P.K, dec_z(a, P, g), T, lds);
            else
                dec_shrink<NW, 1>(a, P, pl, ai, rb, c, 1, P.X + (size_t)t0 * P.K, dec_z(a, P, g), T, lds);
        }
        if (threadIdx.x == 0) raise_flag(a, bid, no);
        if (w == 0) count_launch(a, no);
        return;
    }

    // the row groups of a tile run on one XCD (workgroup b runs on XCD b mod 8)
    // close together, so that its L2 serves the weights to all but the first
    const int mb0 = bid - a.groups * a.n_shrink, per = 8 * a.groups, m8 = mb0 / per, in8 = mb0 - m8 * per;
    const int mbid = a.groups == 1 ? mb0 : m8 * 8 + (in8 & 7), g = a.groups == 1 ? 0 : in8 >> 3;
    if (mbid >= a.n_main) {
        if (w == 0) count_launch(a, launch_no(a));
        return;
    }
    const int t0 = g * a.rows, T = min(a.rows, a.T - t0);
    int p = 0;
    if constexpr (!PAIR) {
#pragma unroll
        for (int q = 1; q < kMaxProjs; ++q)
            if (q < a.n_proj && mbid >= a.tile_base[q]) p = q;
    }
    const DecProj P = a.p[p], P1 = a.p[PAIR ? 1 : p];
    const int kparts = P.kparts, ncg = NW >> __builtin_ctz(kparts), cg = w >> __builtin_ctz(kparts), kq = w - cg * kparts;
    const int KS = P.K >> 5, nWb = P.N >> 4, tile = mbid - (PAIR ? 0 : a.tile_base[p]);
    // this wave's column blocks (clamped at the projection's edge; not stored)
    int blk[NB];
    const DecProj* Pc[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        blk[cb] = min(PAIR ? tile * ncg + cg : (tile * ncg + cg) * NB + cb, nWb - 1);
        Pc[cb] = PAIR && cb == 1 ? &P1 : &P;
    }
    int sig[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
        sig[cb] = 0;
#pragma unroll
        for (int q = 1; q < kMaxSlices; ++q)
            if (q < Pc[cb]->n_slices && blk[cb] * 16 >= Pc[cb]->slice_col[q]) sig[cb] = q;
    }
    f32x4 acc[MB][NB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    XRows<MB> x;
    const int last = T - 1;
    x.init(P.X + (size_t)t0 * P.K, P.K, T, lds + w * MB * 128, [last](int r) { return min(r, last); });

    // wave 0 plans the batch (its loads go ahead of the weights')
    PlanLoads ld = PlanLoads{0, 0, -1};
    unsigned no = 0;
    if (w == 0 && a.act_max > 0) ld = dec_plan_loads(a, t0, T);
    // Expand turn: 4 octets of the adapters in use (lane group lg takes
    // octet lg; tokens of other adapters see zeros, which cost no traffic:
    // their loads are past the end of Z).  Either the octets of all adapters,
    // each turn for every row block; or, row block after row block, those of
    // the adapters that have tokens there (`own`), which is less where most
    // adapters have tokens in few row blocks (1B layer, 64 tokens, 64 adapters of
    // rank 64: 170 -> 86 us).  The first turns' B^T are loaded during the K loop.
    constexpr int NZ = ZS ? NB : 1;                   // Z's of a turn
    constexpr int E = ZS ? 2 : 3;                     // turns in flight, one row block each
    struct TurnB {
        u32x4 b[NB];
        int cd;
    };
    struct TurnZ {
        u32x4 z[MB][3];
    };
    struct TurnO {
        u32x4 z[NZ][3];
        int rb;
    };
    TurnB tb[E];
    int turns = 0;
    bool own = false;
    auto load_b = [&](TurnB& t, int e) __attribute__((always_inline)) {
        t.cd = e < turns ? s_oct[4 * e + lg] : -1;
        const int slot = t.cd >= 0 ? (t.cd >> 12) & 0x1fff : 0, r8s = t.cd >= 0 ? (t.cd >> 4) & 0xff : 0, j0 = t.cd >= 0 ? (t.cd & 15) * 8 : 0;
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
            t.b[cb] = ld16(a.pool + (size_t)slot * a.slot_stride + Pc[cb]->b_off + (size_t)(blk[cb] * 16 + lr) * r8s + j0);
    };
    // Z of block q's projection and slice, for the tokens of row block rb
    auto load_z3 = [&](u32x4 (&z)[3], int cd, int q, int rb) __attribute__((always_inline)) {
        const int vr = sig[q] * ((cd >> 4) & 0xff) + (cd & 15) * 8;              // row of A^T
        const __amdgpu_buffer_rsrc_t rz = buf_rsrc(dec_z(a, *Pc[q], g), (unsigned)(Pc[q]->nbA * a.rows * kDecZLine * 2));
        const unsigned zo = (unsigned)(((vr >> 4) * a.rows + rb * 16 + lr) * kDecZLine + (vr & 15)) * 2u;
        const bool mine = cd >= 0 && s_vid[rb * 16 + lr] == ((cd >> 12) & 0x1fff);
#pragma unroll
        for (int i = 0; i < 3; ++i) z[i] = buf16(rz, mine ? zo + i * 32u : kOob);
    };
    auto load_z = [&](TurnZ& t, int cd, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) load_z3(t.z[rb], cd, q, rb);
    };
    auto load_zo = [&](TurnO& t, int cd) __attribute__((always_inline)) {
        t.rb = max(__builtin_amdgcn_readfirstlane(cd) >> 25, 0);                 // (lane 0 has the turn's first octet)
#pragma unroll
        for (int q = 0; q < NZ; ++q) load_z3(t.z[q], cd, q, t.rb);
    };
    auto use = [&](const u32x4& b, const TurnZ& z, int cb) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int i = 0; i < 3; ++i) acc[rb][cb] = mfma(b, z.z[rb][i], acc[rb][cb]);
    };
    auto use_own = [&](const TurnB& b, const TurnO& z) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
            if (MB == 1 || z.rb == rb) {
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int i = 0; i < 3; ++i) acc[rb][cb] = mfma(b.b[cb], z.z[ZS ? cb : 0][i], acc[rb][cb]);
            }
    };
    auto pre = [&]() __attribute__((always_inline)) {
        if (w == 0) no = launch_no(a);
        if (w == 0 && a.act_max > 0) {
            const Plan pl = dec_plan(a, ld, T);
            s_vid[l] = pl.vid;
            const int c = pl.gr >> 3;
            const int incl = wave_incl_scan(c), total = wave_total(incl);
            int at = 0, ow = MB == 1;
            // (few turns are not worth the count: 8B, 50 tokens a row group over 8
            // adapters, a microsecond a launch)
            if (MB > 1 && total > 64) {
                // lane g: the row blocks that hold tokens of its adapter, and octets
                // before its own in each of them (two 16-bit sums a scan)
                s_cnt[0][l] = 0;
                __builtin_amdgcn_wave_barrier();
                if (pl.mine >= 0) atomicOr(&s_cnt[0][pl.mine], 1 << (l >> 4));
                __builtin_amdgcn_wave_barrier();
                const int in = s_cnt[0][l];
                int sum[(MB + 1) / 2], tot[(MB + 1) / 2], first[MB], n = 0;
#pragma unroll
                for (int h = 0; h < (MB + 1) / 2; ++h) {
                    const int v = ((in >> (2 * h)) & 1 ? c : 0) | ((in >> (2 * h + 1)) & 1 ? c << 16 : 0);
                    sum[h] = wave_incl_scan(v);
                    tot[h] = wave_total(sum[h]);
                    sum[h] -= v;
                }
#pragma unroll
                for (int rb = 0; rb < MB; ++rb) {
                    first[rb] = n;
                    n += (((tot[rb >> 1] >> (16 * (rb & 1))) & 0xffff) + 3) >> 2;
                }
                // (loads of a turn)
                ow = n * (NB + 3 * NZ) < ((total + 3) >> 2) * (NB + 3 * NZ * MB);
                if (ow) {
#pragma unroll
                    for (int rb = 0; rb < MB; ++rb) {
                        const int o = 4 * first[rb] + ((sum[rb >> 1] >> (16 * (rb & 1))) & 0xffff);
                        const int end = (tot[rb >> 1] >> (16 * (rb & 1))) & 0xffff;
                        if ((in >> rb) & 1)
                            for (int j = 0; j < c; ++j) s_oct[o + j] = (rb << 25) | (pl.gs << 12) | (pl.gr << 4) | j;
                        if (l < ((-end) & 3)) s_oct[4 * first[rb] + end + l] = -1;
                    }
                    at = n;
                }
            }
            if (MB == 1 || !ow) {
                for (int j = 0; j < c; ++j) s_oct[incl - c + j] = (pl.gs << 12) | (pl.gr << 4) | j;
                if (l < 4) s_oct[total + l] = -1;
                at = (total + 3) >> 2;
            }
            if (l == 0) {
                s_info[0] = at;
                s_info[2] = ow;
            }
        }
    };
    auto mid = [&]() __attribute__((always_inline)) {
        if (a.act_max > 0) {
            __syncthreads();
            turns = s_info[0];
            own = MB == 1 || s_info[2];
#pragma unroll
            for (int d = 0; d < E; ++d)
                if (kq + d * kparts < turns && (d < 2 || own)) load_b(tb[d], kq + d * kparts);
        }
    };
    auto none = []() {};
    if constexpr (Q4 && PAIR) {
        if (Pc[0]->Ws && Pc[1]->Ws) {
            dec_k_int4<MB, NB, 0, 2>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
        } else if (Pc[0]->Ws) {
            // one of gate and up on an INT4 base, the other bf16
            dec_k_int4<MB, NB, 0, 1>(acc, Pc, blk, x, KS, kq, kparts, none, none);
            dec_k_bf16<MB, NB, 1, 1>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
        } else {
            dec_k_bf16<MB, NB, 0, 1>(acc, Pc, blk, x, KS, kq, kparts, none, none);
            if (Pc[1]->Ws)
                dec_k_int4<MB, NB, 1, 1>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
            else
                dec_k_bf16<MB, NB, 1, 1>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
        }
    } else if (Q4 && P.Ws) {
        dec_k_int4<MB, NB, 0, NB>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
    } else {
        dec_k_bf16<MB, NB, 0, NB>(acc, Pc, blk, x, KS, kq, kparts, pre, mid);
    }

    if (turns > 0) {
        if (w == 0) {
            // (the two projections of a pair have their shrink workgroups side by side)
            const int i0 = a.shrink_base[p], i1 = p + (PAIR ? 2 : 1) < a.n_proj ? a.shrink_base[p + (PAIR ? 2 : 1)] : a.n_shrink;
            // (a limit for each unit that a shrink workgroup takes: an expand turn's
            // 4 octets of ranks are 2 blocks of A^T a slice)
            const bool ok = wait_flags(a, g * a.n_shrink + i0, i1 - i0, no, 2 * P.n_slices * turns, P.n_shrink);
            if (l == 0) s_info[1] = ok;
        }
        __syncthreads();
        if (!s_info[1]) {
            // this tile's projections, every item
            const Plan mine = dec_plan(a, dec_plan_loads(a, t0, T), T);
            const int nit = dec_items(mine, s_cnt[w]);
            for (int q = 0; q < (PAIR ? 2 : 1); ++q) {
                const DecProj& Q = a.p[p + q];
                for (int ai = 0; ai < mine.n; ++ai) {
                    const int nb = (Q.n_slices * __builtin_amdgcn_readlane(mine.gr, ai) + 15) >> 4;
                    const int items = __builtin_amdgcn_readlane(nit, ai);
                    for (int rb = 0; rb < items; ++rb)
                        for (int c = 0; c < nb; ++c)
                            dec_shrink<NW, 1>(a, Q, mine, ai, rb, c, 1, Q.X + (size_t)t0 * Q.K, dec_z(a, Q, g), T, lds);
                }
            }
        }
        asm volatile("" ::: "memory");
        const int nt = (turns - kq + kparts - 1) >> __builtin_ctz(kparts);      // this wave's turns (kparts: a power of 2)
        if (nt > 0 && own) {
            TurnO to[E];
#pragma unroll
            for (int d = 0; d < E; ++d)
                if (d < nt) load_zo(to[d], tb[d].cd);
            int i = 0;
            for (; i + 2 * E <= nt; i += E) {
#pragma unroll
                for (int d = 0; d < E; ++d) {
                    use_own(tb[d], to[d]);
                    load_b(tb[d], kq + (i + d + E) * kparts);
                    load_zo(to[d], tb[d].cd);
                }
            }
#pragma unroll
            for (int d = 0; d < E; ++d)
                if (i + d < nt) {
                    use_own(tb[d], to[d]);
                    if (i + d + E < nt) {
                        load_b(tb[d], kq + (i + d + E) * kparts);
                        load_zo(to[d], tb[d].cd);
                    }
                }
#pragma unroll
            for (int d = 0; d < E; ++d)
                if (i + E + d < nt) use_own(tb[d], to[d]);
        } else if (MB > 1 && nt > 0) {
            TurnZ z0, z1;
            if (nt < 2) load_b(tb[1], turns);
            if constexpr (ZS) {
                // a Z of each block, one after the other
                static_assert(NB == 2, "block 0 and block 1");
                load_z(z0, tb[0].cd, 0);
                for (int e = kq; e < turns; e += kparts) {
                    load_z(z1, tb[0].cd, 1);
                    use(tb[0].b[0], z0, 0);
                    load_z(z0, tb[1].cd, 0);              // of the next turn (none: zeros)
                    use(tb[0].b[1], z1, 1);
                    tb[0] = tb[1];
                    if (e + 2 * kparts < turns) load_b(tb[1], e + 2 * kparts);
                }
            } else {
                auto use_all = [&](const TurnB& b, const TurnZ& z) __attribute__((always_inline)) {
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb) use(b.b[cb], z, cb);
                };
                load_z(z0, tb[0].cd, 0);
                load_z(z1, tb[1].cd, 0);
                for (int e = kq; e < turns; e += 2 * kparts) {
                    use_all(tb[0], z0);
                    if (e + 2 * kparts < turns) {
                        load_b(tb[0], e + 2 * kparts);
                        load_z(z0, tb[0].cd, 0);
                    }
                    if (e + kparts >= turns) break;
                    use_all(tb[1], z1);
                    if (e + 3 * kparts < turns) {
                        load_b(tb[1], e + 3 * kparts);
                        load_z(z1, tb[1].cd, 0);
                    }
                }
            }
        }
    }
    if (w == 0) count_launch(a, no);
    // the K-parts meet: fragment (w, rb, cb) in lane order, added in part order
    __syncthreads();                                  // every wave is past its X buffer, which red overlays
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) red[((w * MB + rb) * NB + cb) * 64 + l] = acc[rb][cb];
    __syncthreads();
    constexpr int NS = PAIR ? 1 : NB;                 // stored blocks per column group
    for (int e = threadIdx.x; e < ncg * MB * NS * 64; e += (64 * NW)) {
        // lane ln of fragment (rb, cb): token 16 rb + ln mod 16, columns 4 (ln / 16) + i
        const int ln = e & 63, f = e >> 6, cb = f % NS, rb = (f / NS) % MB, g = f / (NS * MB);
        const int t = rb * 16 + (ln & 15), b = (tile * ncg + g) * NS + cb, col = b * 16 + 4 * (ln >> 4);
        if (t >= T || b >= nWb) continue;
        const f32x4* src = red + ((g * kparts * MB + rb) * NB + cb) * 64 + ln;
        f32x4 v = src[0];
        for (int q = 1; q < kparts; ++q) v += src[q * MB * NB * 64];
        if constexpr (PAIR) {
            f32x4 u = src[64];
            for (int q = 1; q < kparts; ++q) u += src[q * MB * NB * 64 + 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = v[i] / (1.f + __expf(-v[i])) * u[i];
        }
        const uint2 o = make_uint2((uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                                   (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16));
        // out, or the MLP intermediate H (the second projection's input)
        *reinterpret_cast<uint2*>((a.h_dst ? a.h_dst : P.out) + (size_t)(t0 + t) * P.N + col) = o;
    }
}

template <int MB, int NW>
static hipError_t launch_mb(DecArgs& a, bool q4, hipStream_t s) {
    // column blocks of a wave in different slices
    bool zs = false;
    for (int i = 0; i < a.n_proj; ++i)
        for (int q = 1; q < a.p[i].n_slices; ++q) zs = zs || a.p[i].slice_col[q] % (16 * kDecNB) != 0;
    const dim3 grid(a.groups * (a.n_shrink + (a.groups == 1 ? a.n_main : (a.n_main + 7) / 8 * 8)));
    if ((long long)grid.x > a.counts) return hipErrorInvalidValue;
    a.count_share = (a.counts - (int)grid.x + (int)grid.x - 1) / (int)grid.x;
#define BDL_DEC_CASE(Q, R, Z) hipLaunchKernelGGL((dec_main_kernel<NW, MB, kDecNB, Q, R, Z>), grid, dim3(64 * NW), 0, s, a)
    if (a.pair) {
        if (q4) BDL_DEC_CASE(true, true, true); else BDL_DEC_CASE(false, true, true);
    } else if (zs) {
        if (q4) BDL_DEC_CASE(true, false, true); else BDL_DEC_CASE(false, false, true);
    } else {
        if (q4) BDL_DEC_CASE(true, false, false); else BDL_DEC_CASE(false, false, false);
    }
#undef BDL_DEC_CASE
    return hipGetLastError();
}

hipError_t launch_dec_main(DecArgs& a, int mb, hipStream_t s) {
    if (a.n_main <= 0 || a.n_shrink < 1 || a.T < 1 || a.rows > mb * 16 || a.rows > kDecodeMaxT ||
        a.groups != (a.T + a.rows - 1) / a.rows || !a.flags || !a.count) return hipErrorInvalidValue;
    bool q4 = false;
    for (int i = 0; i < a.n_proj; ++i) {
        q4 = q4 || a.p[i].Ws != nullptr;
        if (a.p[i].kparts < 1 || (a.p[i].kparts & (a.p[i].kparts - 1)) || dec_waves(mb) % a.p[i].kparts) return hipErrorInvalidValue;
    }
    switch (mb) {
        case 1: return launch_mb<1, dec_waves(1)>(a, q4, s);
        case 2: return launch_mb<2, dec_waves(2)>(a, q4, s);
        case 3: return launch_mb<3, dec_waves(3)>(a, q4, s);
        case 4: return launch_mb<4, dec_waves(4)>(a, q4, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace bdl
