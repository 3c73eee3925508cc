// Launch descriptors shared by the host side of the library and its kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdlora.h"

namespace bdl {

constexpr int kMaxProjs = 8;
constexpr int kMaxSlices = 4;
constexpr int kMaxSlots = 8192;
constexpr int kMaxRank8 = 128;       // largest supported rank, rounded up to 8
constexpr int kPlanLdsTokens = 8192; // plan keeps validated ids in LDS up to this batch size
constexpr int kPlanWaveGroups = 256;  // plan: placement by all waves for at most this many adapters
constexpr int kPlanParMaxSlots = 4096; // ... in pools of at most this many slots (its LDS counts)
constexpr int kMaxSeg = BDLORA_MAX_SEGMENTS;   // segments of a batch given in run-length form
constexpr int kBigM = 256, kBigN = 256;   // output tile of the large-tile base GEMM (prefill)
constexpr int kBigPartSlots = 256;        // fp32 partial tiles of the large-tile GEMM's split tiles
constexpr int kBigPartElems = kBigM * kBigN;
constexpr int kMidMaxT = 256;             // medium-batch base GEMM: largest batch (all rows in one tile)

// One projection of a forward launch.
struct ProjLaunch {
    const uint16_t* X;        // [T x K] bf16 activations (row-major); null: an intermediate, in Xp only
    const uint16_t* Xp;       // packed activations, fragment layout, rows padded to 16
    int x_rowmajor;           // large-tile and medium-batch paths: the GEMM reads X (row-major, rows
                              // gathered by token) and Xp is not written; else Xp.  (The shrink reads
                              // X wherever there is one.)
    const uint16_t* W;        // packed base weight, fragment layout ([N x K] nn.Linear rows)
    const uint16_t* Ws;       // INT4 base: its scales (null for a bf16 base)
    uint16_t* out;            // [T x N] bf16
    float* out_f32;           // when set: the output in fp32 [T x N] instead of out
    uint16_t* Z;              // [2 x max_tokens x zs] workspace: scale * X A per slice as a
                              // bf16 pair (hi plane, then lo plane at Z + zplane)
    long long zplane;         // elements between the hi and the lo plane
    int K, N, n_slices, zs;
    int slice_col[kMaxSlices + 1];   // first column of each slice; [n_slices] = N
    long long a_off, b_off;   // element offsets of packed A^T_cat and of B^T_cat in a slot
    int tiles_n;              // base GEMM: column tiles of this projection
    int tile_base;            // base GEMM: first flattened tile (large tiles: work item) of this projection
    int ksplit;               // large-tile / medium-batch GEMM: k-ranges per tile (1: not split)
    int fix_base;             // large-tile GEMM: first split tile of this projection in the fix-up order
    int fix_count;            // large-tile GEMM: split tiles of this projection (0 when ksplit is 1)
    int part_base;            // large-tile GEMM: first partial tile of this projection's split tiles;
                              // medium-batch GEMM: first work item (= partial tile) of this projection
    int col_base;             // medium-batch GEMM: first 64-column epilogue tile of this projection
};

// Everything one forward launch needs (passed by value as a kernel argument).
struct FwdArgs {
    ProjLaunch p[kMaxProjs];
    int n_proj;
    int T;
    const uint16_t* pool;     // adapter slabs
    long long slot_stride;    // elements per slot
    int r8max;                // per-slice Z stride (elements)
    const float* scale;       // [max_slots]
    const int* vid;           // [T] validated ids
    const int* perm;          // [T] tokens grouped by adapter
    const int* rowtok;        // large-tile GEMM: token of each tile row (adapter order), or null
    const int* rowslot;       // medium-batch GEMM: (rank8 << 16) | slot of each such row, -1 for none
    const int4* items;        // shrink items {slot, first perm index, rows, r8}
    const int* meta;          // [1] number of shrink items
    int items_bound;          // shrink: upper bound on items
    int* queue;               // shrink: unit counter, zeroed by the plan (meta[2])
    int sorder[kMaxProjs];    // shrink: projections in unit order (longest K first)
    int schunks[kMaxProjs];   // shrink: column chunks of an item, by projection (not by unit order)
    const int* tile_oct;      // expand octet codes per row tile (-1 padded)
    int oct_cap;              // entries per row tile in tile_oct
    int tiles_m;              // base GEMM: row tiles
    int total_tiles;          // base GEMM: flattened tiles (large tiles: work items) over all projections
    float* bigpart;           // large-tile GEMM: fp32 partials of split tiles (kBigPartSlots tiles)
    int total_fix;            // large-tile GEMM: split tiles over all projections
    int mid_rb, mid_nb;       // medium-batch GEMM: 16-row blocks per tile, 16-column blocks per wave
    int mid_items;            // medium-batch GEMM: work items (tile x k-range) over all projections
    int mid_col_tiles;        // medium-batch GEMM: 64-column epilogue tiles over all projections
    int max_slots;            // pool slots
    // MLP intermediate (large-tile and medium-batch launches of the MLP's
    // first projections): -1 writes out / out_f32; BDLORA_ACT_NONE writes
    // H = projection 0's output, BDLORA_ACT_SILU_MUL H = silu(projection 0)
    // * projection 1 (gate and up of equal shape; their tiles are paired so
    // one workgroup holds both), in bf16 into h_dst in the fragment layout of
    // the second projection's input (rows = tokens, h_KS k-steps)
    int mlp_act;
    uint16_t* h_dst;
    int h_KS;
};

// Activation packing job of the prep launch.
struct PackJob {
    const uint16_t* src;      // [rows x K] row-major
    uint16_t* dst;            // fragment layout, rows padded to a multiple of 16
    int rows, K;
    int frag_base;            // first fragment of this job in the launch's numbering
};

// Prep launch: workgroup 0 plans the batch, the others pack activations.
struct PrepArgs {
    const int* ids;           // [T] per-token ids, or null: the batch is given by the segments below
    int T;
    int n_seg;                // segments (ids null): token t takes seg_slot[i] of the last i with
    int seg_start[kMaxSeg];   // seg_start[i] <= t (the host checked that they tile 0..T-1)
    int seg_slot[kMaxSeg];
    const int* loaded;
    const int* r8;            // [max_slots]
    int max_slots;
    int mts;                  // shrink rows per item
    int gemm_mt;              // base GEMM row tile (<= 64)
    int oct_cap;
    int* vid;
    int* perm;
    int* rowtok;              // optional [T]: the adapted tokens in perm order, then the others in order
    int* rowslot;             // optional [T], with rowtok: (rank8 << 16) | slot of each row's adapter, -1 for none
    int oct_perm;             // 1: octet lists for the 64-row blocks of rowtok order (large-tile GEMM)
    int* gslot;
    int* gstart;
    int* gcount;
    int4* items;
    int* tile_oct;
    int* meta;                // [0] groups, [1] shrink items, [2] the shrink's unit counter (zeroed)
    int* err;
    PackJob jobs[kMaxProjs];
    int n_jobs;
    int total_frags;
};

// ---- decode path (T <= kDecodeMaxT) ----------------------------------------
// One launch: shrink and main workgroups (bdl_decode.hip).
constexpr int kDecodeMaxT = BDLORA_DECODE_MAX_T;
constexpr int kRowsMaxT = 256;       // largest batch that takes it, in row groups of up to kDecodeMaxT
constexpr int kDecNB = 2;            // 16-column blocks per wave of a main workgroup
// Waves per workgroup for mb blocks of 16 tokens.  The registers allow two
// waves per SIMD, so four-wave workgroups leave room for shrink and main ones
// on a CU together (64 tokens, 26 adapters: 29.7 against 29.5 us; 32 tokens:
// 21.8 against 25.1); with one block, mostly few adapters, eight waves halve
// each wave's share of K (one token: 13.9 against 15.4 us).
constexpr int dec_waves(int mb) { return mb == 1 ? 8 : 4; }
constexpr int kDecZLine = 64;        // elements of Z per (16-row block of A^T, token): one 128-byte line

struct DecProj {
    const uint16_t* X;        // activations [T x K], row-major
    const uint16_t* W;        // packed base weight
    const uint16_t* Ws;       // INT4 base: its scales (null for a bf16 base)
    uint16_t* out;            // [T x N] bf16
    uint16_t* Z;              // [groups][nbA][rows][kDecZLine] scale * X A: per 16-row block of A^T and
                              // token three planes of 16 bf16 numbers that sum to the fp32 value (the
                              // rest unused)
    int K, N, n_slices;
    int slice_col[kMaxSlices + 1];
    long long a_off, b_off;
    int nbA;                  // A^T_cat blocks of an adapter of the pool's largest rank
    int n_shrink;             // shrink workgroups (of each row group; at least one)
    int kparts;               // parts of K per column group of a main workgroup (1, 2, 4 or 8)
};

struct DecArgs {
    // what a workgroup reads first
    int groups, rows;               // row groups, each planned by itself: group g holds the tokens
                                    // [g rows, (g + 1) rows) of the batch (rows <= kDecodeMaxT)
    int n_shrink, n_main;           // workgroups of each kind and group, in launch order (n_shrink >= 1:
                                    // the first also reports invalid ids)
    int n_proj;
    int shrink_base[kMaxProjs];     // first shrink workgroup of each projection
    int tile_base[kMaxProjs];       // first main workgroup of each projection
    int T;
    int act_max;              // adapter positions of the launch: the host's bound on the adapters in
                              // use; the plan treats those past it (slot order) as none and raises *err
    int max_slots;
    int merge;                // shrink workgroups take four blocks of A^T (else one)
    int pair;                 // gated MLP: projections 0 and 1 share the tiles of 0, H = silu(0) * 1
    unsigned wait_ticks;      // longest wait for a producer (100 MHz ticks a turn; 0: none), then its work is done here
    unsigned long long* flags;   // [groups][n_shrink] launch tags (bdl_decode.hip, launch_tag)
    unsigned* count;          // [counts] launches on these flags so far, a word per workgroup (counts: at
    int counts;               // least the workgroups of any launch on them)
    int count_share;          // words past the launch's workgroups per workgroup (set by launch_dec_main)
    const int* ids;           // [T] per-token slot ids, or null: the segments below
    const int* loaded;        // [max_slots] nonzero: the slot holds an adapter
    const int* r8;            // [max_slots] padded rank of each slot
    const uint16_t* pool;
    long long slot_stride;
    const float* scale;       // [max_slots]
    uint16_t* h_dst;          // when set: the output is the MLP intermediate H [T x N], written here
    int* err;                 // sticky error flag
    DecProj p[kMaxProjs];
    int n_seg;                // segments (ids null): token t takes seg_slot[i] of the last i with
    int seg_start[kRowsMaxT];     // seg_start[i] <= t (the host checked that they tile 0..T-1)
    int seg_slot[kRowsMaxT];
};
static_assert(sizeof(DecArgs) <= 4096, "kernel arguments");

// Host-side launchers (bdl_kernels.hip, bdl_prep.hip, bdl_decode.hip).
hipError_t launch_dec_main(DecArgs& a, int mb, hipStream_t s);
hipError_t launch_prep(const PrepArgs& a, hipStream_t s);
hipError_t launch_shrink(const FwdArgs& a, int mb, int nb, hipStream_t s);
// column blocks of the shrink's chunks for a projection of cols = n_slices * r8max columns (shape mb x nb)
constexpr int shrink_blocks(int nb, int cols) { return nb == 6 ? (cols <= 32 ? 2 : 6) : nb == 3 ? (cols <= 16 ? 1 : 3) : nb; }
hipError_t launch_gemm(const FwdArgs& a, int mb, int nb, hipStream_t s);
hipError_t launch_gemm_big(const FwdArgs& a, hipStream_t s);
hipError_t launch_gemm_mid(const FwdArgs& a, hipStream_t s);
hipError_t launch_mid_epi(const FwdArgs& a, hipStream_t s);
hipError_t launch_pack_adapter(uint16_t* dst_a, uint16_t* dst_b, const uint16_t* stage, int K,
                               int n_slices, const int* slice_out, int rank, int r8, hipStream_t s);
hipError_t launch_copy(const uint16_t* src, uint16_t* dst, long long elems, hipStream_t s);   // elems: a multiple of 8
hipError_t launch_pack_rows(const uint16_t* src, uint16_t* dst, int rows, int K, hipStream_t s);
// rank and scale tables of up to kMaxSlotBatch consecutive slots (kernel argument)
constexpr int kMaxSlotBatch = 64;
struct SlotBatch {
    int first, n;
    int r8[kMaxSlotBatch];
    float scale[kMaxSlotBatch];
};
hipError_t launch_set_slots(int* r8, float* scale, int* loaded, const SlotBatch& b, hipStream_t s);
hipError_t launch_pack_int4(const uint8_t* q, const uint16_t* scales, uint32_t* dst_w, uint16_t* dst_s, int N,
                            int K, hipStream_t s);
hipError_t launch_mlp_pack(const float* G, const float* U, uint16_t* dst, int T, int N, hipStream_t s);

// Static scratch of the allocation-free decode entry point (bdl_static.hip).
constexpr long long kStaticScratchBytes = BDLORA_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
// Take the address of the current device's copy (call once per device, with
// it current; later calls return at once).
hipError_t static_scratch_init(int device);
// That address (null before static_scratch_init succeeded on the device).
void* static_scratch(int device);

}  // namespace bdl
