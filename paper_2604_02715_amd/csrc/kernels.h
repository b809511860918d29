// Device-side structures and kernel launchers of libfluxmoe.so (decode side: decode_args.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "decode_args.h"
#include "ffn_plan.h"

namespace fluxmoe {

// ---------------------------------------------------------------- expert FFN
struct FfnArgs {
    const uint16_t* tokens;      // BF16 [T][H]
    const int32_t* topk_ids;     // [T][K]
    const float* topk_w;         // [T][K]
    const int32_t* page_table;   // this layer's row: [n_experts]
    const uint16_t* slots13;     // type-1 arena
    const uint16_t* slots2;      // type-2 arena
    float* out;                  // [T][H]
    uint32_t T, K, H, F, E;
    uint32_t flags;
    // workspace carve-up (device)
    int32_t* expert_count;       // [E + 1]
    int32_t* expert_offset;      // [E + 2]
    int32_t* sorted_pair;        // [pairs_cap]  pair index (t * K + k), grouped by expert
    int32_t* pair_pos;           // [pairs_cap]  position of a pair in sorted order, -1 = skipped
    int4* tile_rec;              // [tiles_cap]  (expert, first sorted row, rows, slot); rows = 0 past the last tile
    int32_t* n_tiles;            // [2]  row tiles; K splits of the first product that work (256 x 256 tiles)
    int32_t* chunk_count;        // [n_chunks][E] in the place of hbuf, which is written later.  Large batches: pairs per (chunk of kRouteChunkPairs pairs, expert),
                                 // turned into the chunk's first position inside the expert's rows by the grouping kernel
    uint16_t* hbuf;              // BF16 [pairs_cap][F]
    float* ybuf;                 // FP32 [ksplit][pairs_cap][H]; with ksplit1 > 1 the first product's partial sums
                                 // [ksplit1][pairs_cap][2][F] (gate, up) lie here before the second product runs
    float* part;                 // where the strip kernels' first product puts its partial sums: ybuf, or behind y where the second product
                                 // adds them up itself (few_fused)
    float* tail;                 // partial sums of the last round of the second product's 256 x 256 tiles (last_round_kernel), nullptr: not split
    uint32_t* error_word;
    uint32_t n_chunks;           // 0: the grouping kernel counts and scatters the pairs itself (one workgroup)
    uint32_t pairs_cap, tiles_cap, m_tile, ksplit;
    uint32_t ksplit1;            // most K splits of the first product (the launch covers as many, first_splits says how many work).
                                 // 1: SwiGLU in its epilogue, more: FP32 partial sums that swiglu_reduce_kernel adds up
    uint32_t split_tiles;        // up to so many row tiles ksplit1 splits work
    uint32_t n_cus;
    uint32_t halves;             // non-zero (strip kernels, m_tile 128): a workgroup of the first product has one strip and its
                                 // pairs of wavefronts half of the k range each, instead of two strips
    uint32_t g1_xcd;             // non-zero (strip kernels): the first product's column workgroups of a row tile share an XCD
    uint32_t identity;           // non-zero: one expert in slot 0 takes every token with gate 1 (K = 1, E = 1); topk_ids,
                                 // topk_w and page_table are not read
    uint32_t tiled;              // non-zero: LDS-tiled kernels (m_tile 256, or 128 for tiles of 128 x 128), else strip kernels
    uint32_t tiled_sn_log2;      // set per launch by launch_ffn: log2 of the columns of the LDS-direct kernels' super-tile
    uint32_t tiled_total;        // set per launch by launch_ffn: tile numbers of the LDS-direct kernel's launch
    uint32_t ring1, ring2;       // non-zero (identity): rows of a tile of gemm_ring_kernel in the first and second product
    uint32_t direct;             // set by launch_ffn: the second product writes the output itself (identity, unsplit)
    uint32_t tiled_group;        // super-rows of the LDS-direct gate/up kernel that share a column block in time;
                                 // 0 = launch_ffn derives it from the rows per expert
};

// What launch_ffn goes by and no kernel reads, kept out of their arguments
struct FfnCall : FfnArgs {
    uint32_t tiled_waves;        // variant of the LDS-tiled kernels: 2 LDS-direct loads, 8 or 4
                                 // wavefronts with register-staged loads
    uint32_t tiled_persist;      // LDS-direct kernels: workgroups per CU-sized round that walk through the tiles (1 = 256
                                 // workgroups), 0 = one workgroup per tile
    uint32_t few;                // non-zero (strip kernels, at most kFewPairs pairs): the first product's workgroups group the pairs
    uint32_t few2;               // non-zero: gemm2_few_kernel is the second product
    uint32_t few_fused;          // it also adds up the first product's partial sums
    uint32_t mapped;             // experts of the layer known to be resident, 0 = not known
};

// hook(user, kind, begin, stream) is called around every kernel when timing is on
// (kinds: 1 grouping, 2 gate/up product + SwiGLU, 3 down product, 4 combine)
typedef void (*SpanHook)(void* user, int kind, int begin, hipStream_t stream);
// done: completes with the call's last kernel; routed: with the kernel that reads the page table last (nullptr: none).
// done is attached to its launch (none of either for the shared expert); routed too if attach_routed, else it is recorded behind it (stream capture).
hipError_t launch_ffn(const FfnCall& call, int n_cus, hipStream_t stream, hipEvent_t done, hipEvent_t routed, bool attach_routed,
                      SpanHook hook, void* user);
// gemm_ring_kernel (ffn_ring.hip) for the first or second product
hipError_t launch_ring(const FfnArgs& args, int product, hipStream_t stream);
hipError_t launch_mfma_probe(const void* operands, float* out, uint32_t n_workgroups, uint32_t iters,
                             hipStream_t stream);
// The decode kernel's launch shape and memory accesses without its work (probe_kernels.hip): n_blocks blocks of
// 4096 bytes read, stream_mix_out_bytes(n_blocks, small) bytes written (small or small + 128 bytes per block).
uint64_t stream_mix_out_bytes(uint64_t n_blocks, uint32_t small);
hipError_t launch_stream_mix(void* dst, const void* src, uint32_t n_blocks, uint32_t small, int waves_per_wg,
                             uint32_t per_wave, uint32_t order, uint32_t n_workgroups, hipStream_t stream);

}  // namespace fluxmoe
