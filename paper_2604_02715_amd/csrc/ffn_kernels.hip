// Routed SwiGLU expert FFN over page-table addressed slots (gfx950, BF16 MFMA, FP32 acc).
//
// The paper runs an unchanged fused-MoE kernel on the materialized tensors (Sec. 5; tensor
// types of Sec. 4.1 "Formal model": fused gate/up [2][H][F] and down [F][H]); it gives no
// kernel design, so this one is built for decode-shaped batches on MI355X, where every
// expert sees few tokens and the FFN is bound by streaming the expert's weights once:
//
//   route_sort   one workgroup: counting sort of the (token, k) pairs by expert, skipping
//                pairs whose expert has no slot; emits one record per row tile (expert, first
//                row, rows, slot), tiles with the most rows first
//   gemm1        per (row tile, 128-column strip): a = X W1 and b = X W3 on two wavefronts
//                with v_mfma_f32_16x16x32_bf16, h = silu(a) * b rounded to BF16; with few row tiles
//                per (row tile, strip, K split), and swiglu_reduce adds the splits and applies SwiGLU
//   gemm2        per (row tile, 128-column strip, K split): y = h W2, FP32 partial sums
//   combine      out[t] = sum_k gate[t][k] * sum_splits y[pos(t,k)]   (fixed order)
//
// Weights stay row-major [K][N] in the slots (placement is bit-exact by contract), while
// MFMA wants 8 consecutive k per lane.  Each lane therefore loads 8 rows x 16 bytes (8
// columns) straight from HBM, fully coalesced along N, and transposes its 8x8 tile in
// registers with v_perm_b32; MFMA number c of a step uses column c of every lane's tile,
// so output column j of that MFMA is column 8 * j + c of the strip.  Weights never pass
// through LDS and every weight byte is read exactly once per row tile; LDS holds only the
// tile's activations, shared by the four wavefronts of a workgroup.
// Batches with more rows per expert than one 128-row tile go to the LDS-tiled kernels
// further down (gemm_d2l_kernel and its register-staged predecessors), which are bound by
// the matrix cores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ffn_device.h"
#include "kernels.h"

namespace fluxmoe {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

union Frag {
    uint4 u;
    bf16x8 v;
};

constexpr int kStrip = 128;        // output columns per wavefront
constexpr int kChunk = 32;         // k per MFMA step
constexpr uint32_t kRoutedPairs = kFewPairs;
constexpr int kNonTemporal = 2;    // cache policy operand of the buffer loads: bit 1 = nt

// ------------------------------------------------------------------ routing / grouping
// K splits of the first product that work (the launch covers ksplit1), for weight strips and tiles of 128 x 128
__device__ __forceinline__ uint32_t first_splits(const FfnArgs& a, uint32_t n_tiles) { return n_tiles <= a.split_tiles ? a.ksplit1 : 1u; }
// and for tiles of 256 x 256 into n_tiles[1], by one wavefront of the grouping kernel with a candidate in each lane: done by
// the product's workgroups it held each back for half a microsecond, and there are up to seven for a CU (131 -> 144 us a call).
__device__ __forceinline__ void choose_splits(const FfnArgs& a, uint32_t n_tiles, uint32_t rows, uint32_t lane) {
    uint32_t k = lane + 1;
    float cost = k <= a.ksplit1 ? tiled_cost(SplitShape{a.H, a.F, a.n_cus}, n_tiles, rows, k) : 3e38f;
    for (int d = 4; d > 0; d >>= 1) {        // at most 8 splits
        const float c2 = __shfl_xor(cost, d);
        const uint32_t k2 = uint32_t(__shfl_xor(int(k), d));
        if (c2 < cost || (c2 == cost && k2 < k)) { cost = c2; k = k2; }
    }
    if (lane == 0) a.n_tiles[1] = int32_t(n_tiles <= a.split_tiles ? a.ksplit1 : k);
}

// Row tiles are handed out by size class: the body a tile runs and the time it takes grow with its rows,
// and a launch ends when its last workgroup does, so the tiles with the most rows are numbered (and
// therefore started) first and the many small ones fill in behind them.
constexpr int kTileClasses = 5;
__device__ __forceinline__ int tile_class(int32_t rows) {
    return rows > 96 ? 0 : (rows > 64 ? 1 : (rows > 32 ? 2 : (rows > 16 ? 3 : 4)));
}

// Exclusive prefix sums over the 1024 threads of a workgroup for N values per thread at once; total[i]
// receives the sum of v[i] over all threads.  tot: N * 17 ints of LDS.  Contains barriers.
template <int N>
__device__ __forceinline__ void block_scan_excl(const int32_t (&v)[N], int32_t (&excl)[N], int32_t (&total)[N], int32_t* tot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = v[i];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t y = __shfl_up(x[i], d, 64);
            if (lane >= d) x[i] += y;
        }
        if (lane == 63) tot[i * 17 + wave] = x[i];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int32_t w = lane < 16 ? tot[i * 17 + lane] : 0;
            int32_t xs = w;
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                const int32_t y = __shfl_up(xs, d, 64);
                if (lane >= d) xs += y;
            }
            if (lane < 16) tot[i * 17 + lane] = xs - w;
            if (lane == 15) tot[i * 17 + 16] = xs;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        excl[i] = x[i] - v[i] + tot[i * 17 + wave];
        total[i] = tot[i * 17 + 16];
    }
    __syncthreads();
}

// Large batches: one workgroup per chunk of kRouteChunkPairs pairs counts its pairs per expert
// (route_count_kernel), the single workgroup of route_sort_kernel<true> adds the chunks up, turns each
// chunk's count into the chunk's first position inside the expert's rows and does the scans and the tile
// records, and one workgroup per chunk puts its pairs in place (route_scatter_kernel).  The positions a
// chunk's pairs get depend only on the chunk, not on which workgroup runs first.
__device__ __forceinline__ int32_t route_classify(const FfnArgs& a, int32_t e, const int32_t* slot_of, bool report) {
    if (e < 0 || uint32_t(e) >= a.E) {
        if (report) atomicOr(a.error_word, 2u);
        return -1;
    }
    if (slot_of[e] < 0) {
        if (report && !(a.flags & 2u)) atomicOr(a.error_word, 2u);
        return -1;
    }
    return e;
}

__global__ __launch_bounds__(1024) void route_count_kernel(FfnArgs a) {
    extern __shared__ int32_t sh[];          // count[E]
    const uint32_t pairs = a.T * a.K, first = blockIdx.x * kRouteChunkPairs;
    for (uint32_t e = threadIdx.x; e < a.E; e += 1024) sh[e] = 0;
    __syncthreads();
    for (uint32_t p = first + threadIdx.x; p < min(pairs, first + kRouteChunkPairs); p += 1024) {
        const int32_t e = route_classify(a, a.topk_ids[p], a.page_table, true);
        if (e >= 0) atomicAdd(&sh[e], 1);
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < a.E; e += 1024) a.chunk_count[size_t(blockIdx.x) * a.E + e] = sh[e];
}

__global__ __launch_bounds__(1024) void route_scatter_kernel(FfnArgs a) {
    extern __shared__ int32_t sh[];          // cursor[E]
    const uint32_t pairs = a.T * a.K, first = blockIdx.x * kRouteChunkPairs;
    for (uint32_t e = threadIdx.x; e < a.E; e += 1024) sh[e] = a.expert_offset[e] + a.chunk_count[size_t(blockIdx.x) * a.E + e];
    __syncthreads();
    for (uint32_t p = first + threadIdx.x; p < min(pairs, first + kRouteChunkPairs); p += 1024) {
        const int32_t e = route_classify(a, a.topk_ids[p], a.page_table, false);
        int32_t pos = -1;
        if (e >= 0) {
            pos = atomicAdd(&sh[e], 1);
            a.sorted_pair[pos] = int32_t(p);
        }
        a.pair_pos[p] = pos;
    }
}

template <bool CHUNKED, bool CHOOSE>
__global__ __launch_bounds__(1024) void route_sort_kernel(FfnArgs a) {
    extern __shared__ int32_t sh[];          // count[E], cursor[E], slot[E], scan scratch
    int32_t* count = sh;
    int32_t* cursor = sh + a.E;
    int32_t* slot_of = sh + 2 * a.E;         // this layer's page-table row: every later look-up is an LDS read
    int32_t* scratch = sh + 3 * a.E;
    __shared__ int32_t class_total[kTileClasses];
    const int tid = threadIdx.x;
    const uint32_t pairs = a.T * a.K;
    const int32_t m = int32_t(a.m_tile);
    for (uint32_t e = tid; e < a.E; e += 1024) { count[e] = 0; slot_of[e] = a.page_table[e]; }
    if (tid < kTileClasses) class_total[tid] = 0;
    // the first pairs' expert ids are fetched while the page-table row is on its way
    constexpr int kKept = 8;
    int32_t kept[kKept];
#pragma unroll
    for (int i = 0; i < kKept; ++i) {
        const uint32_t p = tid + 1024u * i;
        kept[i] = (!CHUNKED && p < pairs) ? a.topk_ids[p] : -1;
    }
    if (CHUNKED) {
        // the chunks' counts, added up per expert; each is replaced by the sum of the chunks before it
        for (uint32_t e = tid; e < a.E; e += 1024) {
            int32_t run = 0;
            for (uint32_t c = 0; c < a.n_chunks; ++c) {
                const int32_t v = a.chunk_count[size_t(c) * a.E + e];
                a.chunk_count[size_t(c) * a.E + e] = run;
                run += v;
            }
            count[e] = run;
        }
    }
    __syncthreads();
    // a thread's first kKept pairs stay in registers for the scatter at the end (expert, or -1 for a pair
    // that is skipped); batches with more pairs per thread read the rest again
    auto classify = [&](int32_t e, bool report) { return route_classify(a, e, slot_of, report); };
    if (!CHUNKED) {
#pragma unroll
        for (int i = 0; i < kKept; ++i) {
            const uint32_t p = tid + 1024u * i;
            kept[i] = p < pairs ? classify(kept[i], true) : -1;
            if (kept[i] >= 0) atomicAdd(&count[kept[i]], 1);
        }
        for (uint32_t p = tid + 1024u * kKept; p < pairs; p += 1024) {
            const int32_t e = classify(a.topk_ids[p], true);
            if (e >= 0) atomicAdd(&count[e], 1);
        }
    }
    __syncthreads();
    // Tiles per class over all experts, needed before the tiles of the first 1024 experts can be numbered.  With one
    // round (at most 1024 experts) the round's own scan delivers them; otherwise they are summed here
    // (integer sums: the order of the additions does not matter).
    const bool one_round = a.E <= 1024;
    if (!one_round) {
        for (uint32_t e = tid; e < a.E; e += 1024) {
            const int32_t c = count[e];
            if (c >= m) atomicAdd(&class_total[tile_class(m)], c / m);
            if (c % m) atomicAdd(&class_total[tile_class(c % m)], 1);
        }
        __syncthreads();
    }
    int32_t class_base[kTileClasses];        // first tile number of each class; advanced round by round
    int32_t n_tiles = 0;
#pragma unroll
    for (int k = 0; k < kTileClasses; ++k) { class_base[k] = n_tiles; n_tiles += class_total[k]; }
    int32_t row_base = 0;
    // experts in rounds of 1024, one per thread: exclusive scans of its rows and of its tiles in each class
    for (uint32_t base = 0; base < a.E; base += 1024) {
        const uint32_t e = base + tid;
        const int32_t c = (e < a.E) ? count[e] : 0;
        const int32_t full = c / m, rem = c % m;
        const int k_full = tile_class(m), k_rem = tile_class(rem);
        int32_t v[1 + kTileClasses], excl[1 + kTileClasses], total[1 + kTileClasses];
        v[0] = c;
#pragma unroll
        for (int k = 0; k < kTileClasses; ++k) v[1 + k] = (k == k_full ? full : 0) + ((rem && k == k_rem) ? 1 : 0);
        block_scan_excl(v, excl, total, scratch);
        if (one_round) {
            n_tiles = 0;
#pragma unroll
            for (int k = 0; k < kTileClasses; ++k) { class_base[k] = n_tiles; n_tiles += total[1 + k]; }
        }
        if (e < a.E) {
            const int32_t row_excl = row_base + excl[0];
            a.expert_offset[e] = row_excl;
            a.expert_count[e] = c;
            cursor[e] = row_excl;
            const int32_t slot = c ? slot_of[e] : -1;
            int32_t at_full = 0, at_rem = 0;
#pragma unroll
            for (int k = 0; k < kTileClasses; ++k) {
                if (k == k_full) at_full = class_base[k] + excl[1 + k];
                if (k == k_rem) at_rem = class_base[k] + excl[1 + k] + (k == k_full ? full : 0);
            }
            for (int32_t i = 0; i < full; ++i)
                if (uint32_t(at_full + i) < a.tiles_cap) a.tile_rec[at_full + i] = make_int4(int32_t(e), row_excl + i * m, m, slot);
            if (rem && uint32_t(at_rem) < a.tiles_cap) a.tile_rec[at_rem] = make_int4(int32_t(e), row_excl + full * m, rem, slot);
        }
        row_base += total[0];
#pragma unroll
        for (int k = 0; k < kTileClasses; ++k) class_base[k] += total[1 + k];
    }
    // the records past the last tile read as empty tiles
    for (uint32_t i = uint32_t(min(n_tiles, int32_t(a.tiles_cap))) + tid; i < a.tiles_cap; i += 1024) a.tile_rec[i] = make_int4(0, 0, 0, -1);
    if (tid == 0) {
        a.expert_offset[a.E] = row_base;
        a.n_tiles[0] = min(n_tiles, int32_t(a.tiles_cap));
    }
    if (CHOOSE && tid < 64) choose_splits(a, uint32_t(n_tiles), uint32_t(row_base), uint32_t(tid));
    if (CHUNKED) return;                     // route_scatter_kernel puts the pairs in place
    __syncthreads();
    auto place = [&](uint32_t p, int32_t e) {
        int32_t pos = -1;
        if (e >= 0) {
            pos = atomicAdd(&cursor[e], 1);
            a.sorted_pair[pos] = int32_t(p);
        }
        a.pair_pos[p] = pos;
    };
#pragma unroll
    for (int i = 0; i < kKept; ++i) {
        const uint32_t p = tid + 1024u * i;
        if (p < pairs) place(p, kept[i]);
    }
    for (uint32_t p = tid + 1024u * kKept; p < pairs; p += 1024) place(p, classify(a.topk_ids[p], false));
}

// The rows of an expert in the order of their pairs, for a split last round.  Grouping puts them where its atomics happen to arrive, and no result
// depends on that while every tile sums alike; where some of an expert's tiles are summed in parts, a row's tile decides the order of
// its sum.  Rows that share one tile stay as they are.  A workgroup per expert, a stretch of the pairs to each wavefront: bound by its launch and one
// trip to memory, on which the first 512 pairs of a stretch and the expert's place go together; what they were found to be is kept.  8192 pairs of 8 experts
// 4.4 us; the call without / with it 2645 / 2648 us (2671 / 2681 where the pairs were read twice and after the expert's place).
__global__ __launch_bounds__(1024) void route_order_kernel(FfnArgs a) {
    __shared__ uint32_t found[16];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, pairs = a.T * a.K;
    const int32_t e = int32_t(blockIdx.x);
    if (last_round((uint32_t(a.n_tiles[0]) + 3) / 4 * ((a.H + 2047) / 2048)).parts == 1) return;
    const uint32_t stretch = (pairs + 1023) / 1024 * 64, first = min(pairs, wave * stretch), last = min(pairs, first + stretch);
    auto look = [&](uint32_t base, uint64_t (&mine)[8]) __attribute__((always_inline)) {
        int32_t id[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) id[i] = a.topk_ids[min(base + 64 * i + lane, pairs - 1)];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) mine[i] = __ballot(base + 64 * i + lane < last && id[i] == e);
    };
    uint64_t kept[8], more[8];
    look(first, kept);
    const uint32_t rows = uint32_t(a.expert_count[e]), row0 = uint32_t(a.expert_offset[e]);
    if (rows <= a.m_tile) return;                            // uniform
    uint32_t n = 0;
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) n += uint32_t(__popcll(kept[i]));
    for (uint32_t base = first + 512; base < last; base += 512) {
        look(base, more);
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) n += uint32_t(__popcll(more[i]));
    }
    if (lane == 0) found[wave] = n;
    __syncthreads();
    uint32_t at = row0;
    for (uint32_t w = 0; w < wave; ++w) at += found[w];
    auto place = [&](uint32_t base, const uint64_t (&mine)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) {
            const uint32_t p = base + 64 * i + lane, pos = at + uint32_t(__popcll(mine[i] & ((1ull << lane) - 1)));
            if (((mine[i] >> lane) & 1) && pos < row0 + rows) {
                a.sorted_pair[pos] = int32_t(p);
                a.pair_pos[p] = int32_t(pos);
            }
            at += uint32_t(__popcll(mine[i]));
        }
    };
    place(first, kept);
    for (uint32_t base = first + 512; base < last; base += 512) {
        look(base, more);
        place(base, more);
    }
}

// The shared expert: every token once, in order, on the one expert in slot 0.  What route_sort_kernel would find out
// from T identical ids is known, so the lists are written by as many workgroups
// as they need and nothing is counted (gemm_ring_kernel needs none).
__global__ __launch_bounds__(256) void route_identity_kernel(FfnArgs a) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < a.T) {
        a.sorted_pair[i] = int32_t(i);
        a.pair_pos[i] = int32_t(i);
    }
    const uint32_t n_tiles = (a.T + a.m_tile - 1) / a.m_tile;
    if (i < a.tiles_cap) {
        const uint32_t row0 = i * a.m_tile;
        a.tile_rec[i] = i < n_tiles ? make_int4(0, int32_t(row0), int32_t(min(a.m_tile, a.T - row0)), 0) : make_int4(0, 0, 0, -1);
    }
    if (i == 0) {
        a.expert_count[0] = int32_t(a.T);
        a.expert_offset[0] = 0;
        a.expert_offset[1] = int32_t(a.T);
        a.n_tiles[0] = int32_t(n_tiles);
        a.n_tiles[1] = int32_t(a.ksplit1);
    }
}

// ------------------------------------------------------------------ strip GEMM core
__device__ __forceinline__ uint32_t comp(const uint4& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// k chunks per wavefront held in the register ring (one being multiplied, the rest in flight)
template <int MI> struct RingDepth { static constexpr int value = MI >= 8 ? 2 : (MI >= 4 ? 3 : 4); };

// Shared A blocks: the four wavefronts of a workgroup multiply the same rows of A, so a block of
// kABlock k values of the tile's rows is loaded once per workgroup into LDS (two buffers) instead of
// once per wavefront from L2 (where it costs 0.75 bytes of requests per weight byte streamed).
constexpr int kABlock = 128;                 // k per block = 4 chunks

// acc += a * b (v_mfma_f32_16x16x32_bf16) with the accumulator pinned to the AGPR half of the register
// file.  Written as assembly because with the builtin the register allocator, short of VGPRs for
// 192 accumulators plus the load ring, parks ring registers in AGPRs and moves them back (more
// v_accvgpr moves than MFMAs in the ring loop).  The matrix-core hazards the compiler would cover
// are covered here: s_nop 1 gives the two wait states between a VALU write of an operand (the
// v_perm transposes, the v_accvgpr_write zeroing) and the MFMA that reads it; mfma_drain() must
// run before anything but another mfma16 reads an accumulator (the compiler, which must not spill or copy one within eight wait
// states of it, does not know: tests/test_mfma_hazards.py looks through the machine code).  volatile keeps the statements in
// program order (loads and LDS reads stay where the source puts them relative to the MFMAs).
__device__ __forceinline__ void mfma16(f32x4& acc, const bf16x8& a, const bf16x8& b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// 2 x 16 wait states: more than the 18 the longest matrix instruction needs before its result may
// be read by a vector, memory or LDS instruction
__device__ __forceinline__ void mfma_drain() {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// One wavefront's product C[16*MI rows][128 columns] = A[rows][k range] * B[k range][strip].
template <int MI>
struct StripGemm {
    f32x4 acc[MI][8];

    static constexpr int kABufElems = 16 * MI * kABlock;     // one LDS buffer (rows of 256 bytes)

    // B rows come through buffer loads: one descriptor per expert matrix (scalar registers), one
    // VGPR with the lane's byte offset inside a chunk, and the row's byte offset as the scalar
    // offset operand - no vector arithmetic per load.  row0_bytes: offset of the chunk's first row.
    // The loads carry the non-temporal hint (cache policy bit 1): a decode-shaped batch reads every
    // weight byte once, and without the hint the stream pushes the activations, h and the partial
    // sums out of the caches (measured: 6 to 10 % more weight bytes per second with it).
    __device__ __forceinline__ static void load_b(uint4 (&b)[8], __amdgpu_buffer_rsrc_t rsrc, uint32_t voff,
                                                  uint32_t row0_bytes, uint32_t row_bytes) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, row0_bytes + uint32_t(r) * row_bytes, kNonTemporal);
            b[r] = make_uint4(v.x, v.y, v.z, v.w);
        }
    }

    // column c of the lane's 8 x 8 tile
    __device__ __forceinline__ static Frag column(const uint4 (&b)[8], int c) {
        Frag f;
        const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
        f.u.x = __builtin_amdgcn_perm(comp(b[1], c >> 1), comp(b[0], c >> 1), sel);
        f.u.y = __builtin_amdgcn_perm(comp(b[3], c >> 1), comp(b[2], c >> 1), sel);
        f.u.z = __builtin_amdgcn_perm(comp(b[5], c >> 1), comp(b[4], c >> 1), sel);
        f.u.w = __builtin_amdgcn_perm(comp(b[7], c >> 1), comp(b[6], c >> 1), sel);
        return f;
    }

    __device__ __forceinline__ void mma_b(const uint4 (&b)[8], const uint4 (&a)[MI]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const Frag f = column(b, c);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                Frag fa;
                fa.u = a[mi];
                mfma16(acc[mi][c], fa.v, f.v);
            }
        }
    }

    // The first n_blocks * kABlock k values of the range with A shared through LDS.  Every wavefront
    // of the four in the workgroup must call this with the same abase, k_begin and n_blocks (it
    // contains barriers).
    // A: a block is 16 MI rows x 128 k; it goes from global memory straight into LDS
    // (global_load_lds_dwordx4: no registers, no LDS write instructions), one instruction per
    // wavefront per 16 rows: lane (tid / 16, tid % 16) brings one 16-byte piece of row 16 i + tid / 16.
    // Such a load fills 1 KiB contiguously, so rows are 256 bytes apart with no padding; to keep the
    // 16-byte fragment reads of 16 consecutive rows on different banks, position p of row r holds
    // piece p ^ (r % 16).  abase is uniform over the workgroup; aoff[i] is the thread's byte offset of
    // piece (tid % 16) ^ (tid / 16 % 16) of row 16 i + tid / 16 (clamped to the tile's last row).
    // B: bmat points at the [k_rows][ldb] matrix (uniform over the wavefront, under 4 GiB), col is the
    // lane's first column; a four-deep register ring as in run().
    // HALVES: the two pairs of wavefronts multiply different k of the same columns.  A buffer then holds two blocks, one
    // after the other; pair `half` takes the second of each two if it is 1.  n_blocks counts pairs of blocks.
    template <bool HALVES>
    __device__ __forceinline__ void run_shared(const uint8_t* abase, const uint32_t (&aoff)[MI], uint16_t* abuf,
                                               const uint16_t* bmat, uint32_t k_rows, uint32_t col, uint32_t ldb,
                                               uint32_t k_begin, uint32_t n_blocks, int lane, int wave, uint32_t half) {
        if (n_blocks == 0) return;
        const uint32_t kg = 8u * (uint32_t(lane) >> 4);
        const uint32_t row_bytes = 2u * ldb;
        // descriptor word 3 = 0x00020000: raw 32-bit data format of this architecture family
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(bmat), 0, int(k_rows * row_bytes), 0x00020000);
        const uint32_t voff = kg * row_bytes + 2u * col;
        const uint32_t first_bytes = k_begin * row_bytes;
        const uint32_t chunk_bytes = uint32_t(kChunk) * row_bytes;
        // fragment of chunk c, tile mi: row 16 mi + lane % 16, piece 4 c + lane / 16
        const int a_fr = (lane & 15) * (2 * kABlock) + 16 * ((lane >> 4) ^ (lane & 15));   // bytes; ^ 64 c, + 4096 mi
        const uint8_t* const abuf8 = reinterpret_cast<const uint8_t*>(abuf);
        const uint32_t abuf_lds = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)abuf));
        uint4 bst[4][8];
        constexpr uint32_t kBlockBytes = uint32_t(kABufElems) * 2, kBufBytes = kBlockBytes * (HALVES ? 2 : 1);
        const uint32_t my_block = HALVES ? half * kBlockBytes : 0u;
        // M0 carries the LDS destination of an LDS-direct load and is read when the instruction
        // issues; the compiler reserves it, so its value is put back
        auto a_dma = [&](uint32_t blk, uint32_t buf_bytes) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < (HALVES ? 2 : 1) * MI; ++n) {
                const int i = n % MI, sub = n / MI;
                const uint8_t* src = abase + (size_t(k_begin) + (size_t(blk) * (HALVES ? 2 : 1) + sub) * kABlock) * 2;
                uint32_t saved_m0;
                const uint32_t dst = abuf_lds + buf_bytes + uint32_t(sub) * kBlockBytes + uint32_t(i * 4 + wave) * 1024u;
                asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                             : "=&s"(saved_m0) : "v"(aoff[i]), "s"(src), "s"(dst) : "memory");
            }
        };
        // the wavefront's chunk number L (four to a block) -> byte offset of its first row
        auto chunk_at = [&](uint32_t L) __attribute__((always_inline)) {
            return first_bytes + (HALVES ? ((L >> 2) * 2 + half) * 4 + (L & 3u) : L) * chunk_bytes;
        };
        // one block of four chunks; PREFETCH: all four B loads three chunks ahead are inside the
        // shared range and the next A block exists
        auto block = [&](uint32_t cur_bytes, uint32_t nxt_bytes, uint32_t blk, auto PREFETCH) __attribute__((always_inline)) {
            if (PREFETCH.value) a_dma(blk + 1, nxt_bytes);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t chunk = blk * 4 + c;
                if (PREFETCH.value || chunk + 3 < n_blocks * 4) load_b(bst[(c + 3) & 3], rsrc, voff, chunk_at(chunk + 3), row_bytes);
                uint4 af[MI];
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
                    af[mi] = *reinterpret_cast<const uint4*>(abuf8 + cur_bytes + my_block + ((a_fr ^ (64 * c)) + 4096 * mi));
                mma_b(bst[c], af);
            }
            // the A block fetched above was issued before this block's 32 B loads and loads return in
            // order: at most the 24 newest (three chunks of B) may still be in flight
            if (PREFETCH.value) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
            __syncthreads();
        };
        a_dma(0, 0);
#pragma unroll
        for (int c = 0; c < 3; ++c) load_b(bst[c], rsrc, voff, chunk_at(uint32_t(c)), row_bytes);
        asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
        __syncthreads();
        uint32_t blk = 0;
        for (; blk + 1 < n_blocks; ++blk)
            block((blk & 1) * kBufBytes, ((blk + 1) & 1) * kBufBytes, blk, std::integral_constant<bool, true>{});
        block((blk & 1) * kBufBytes, ((blk + 1) & 1) * kBufBytes, blk, std::integral_constant<bool, false>{});
        mfma_drain();
    }

    struct Stage {
        uint4 b[8];      // the lane's 8 rows x 8 columns of B
        uint4 a[MI];     // the lane's A fragments (8 consecutive k of one row per 16-row tile)
    };

    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[mi][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    __device__ __forceinline__ static void load(Stage& st, const uint16_t* const (&arow)[MI],
                                                const uint16_t* bcol, size_t ldb, uint32_t k0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) st.b[r] = load_stream16(bcol + size_t(k0 + r) * ldb);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) st.a[mi] = *reinterpret_cast<const uint4*>(arow[mi] + k0);
    }

    __device__ __forceinline__ void mma(const Stage& st) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            Frag f;
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
            f.u.x = __builtin_amdgcn_perm(comp(st.b[1], c >> 1), comp(st.b[0], c >> 1), sel);
            f.u.y = __builtin_amdgcn_perm(comp(st.b[3], c >> 1), comp(st.b[2], c >> 1), sel);
            f.u.z = __builtin_amdgcn_perm(comp(st.b[5], c >> 1), comp(st.b[4], c >> 1), sel);
            f.u.w = __builtin_amdgcn_perm(comp(st.b[7], c >> 1), comp(st.b[6], c >> 1), sel);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                Frag fa;
                fa.u = st.a[mi];
                mfma16(acc[mi][c], fa.v, f.v);
            }
        }
    }

    // k range a multiple of 8.  bcol must point at 8 existing columns for every lane (callers
    // clamp lanes past the edge).  A ring of 3-4 register stages keeps all but one chunk
    // of 32 k in flight while that one is multiplied: with one wavefront per SIMD that is what
    // covers HBM latency.  A k range that is not a multiple of 32 ends with one chunk in
    // which the lanes past the end contribute zeros.
    __device__ __forceinline__ void run(const uint16_t* const (&arow)[MI], const uint16_t* bcol,
                                        size_t ldb, uint32_t k_begin, uint32_t k_end, int lane) {
        constexpr int kStages = RingDepth<MI>::value;
        if (k_begin >= k_end) return;
        const uint32_t kg = 8u * (uint32_t(lane) >> 4);
        const uint32_t n = (k_end - k_begin) / kChunk;
        const uint32_t kb = k_begin + kg;
        Stage st[kStages];
#pragma unroll
        for (int s = 0; s < kStages - 1; ++s)
            if (uint32_t(s) < n) load(st[s], arow, bcol, ldb, kb + s * kChunk);
        // Steady state without branches: a conditional load inside the loop makes the compiler
        // wait for the newest loads at the join (it must assume the path that issued none), which
        // serialises the ring.  Rounds in which every load is in range run unconditionally; the
        // last rounds take the guarded form.
        uint32_t base = 0;
        for (; base + 2 * kStages - 2 < n; base += kStages) {
#pragma unroll
            for (int s = 0; s < kStages; ++s) {
                load(st[(s + kStages - 1) % kStages], arow, bcol, ldb, kb + (base + s + kStages - 1) * kChunk);
                mma(st[s]);
            }
        }
        for (; base < n; base += kStages) {
#pragma unroll
            for (int s = 0; s < kStages; ++s) {
                const uint32_t i = base + s;
                if (i < n) {
                    if (i + kStages - 1 < n)
                        load(st[(s + kStages - 1) % kStages], arow, bcol, ldb, kb + (i + kStages - 1) * kChunk);
                    mma(st[s]);
                }
            }
        }
        const uint32_t k_full = k_begin + n * kChunk;
        if (k_full < k_end) {
            const uint4 z = make_uint4(0, 0, 0, 0);
            Stage t;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) t.a[mi] = z;
#pragma unroll
            for (int r = 0; r < 8; ++r) t.b[r] = z;
            if (k_full + kg < k_end) load(t, arow, bcol, ldb, k_full + kg);
            mma(t);
        }
        mfma_drain();
    }
};

struct TileInfo {
    int32_t expert, row0, rows, slot;
};

// One 16-byte load: route_sort_kernel or route_identity_kernel wrote (expert, first row, rows, slot) for every tile number below
// tiles_cap, with rows = 0 past the last tile.
__device__ __forceinline__ bool tile_info(const FfnArgs& a, uint32_t tile, TileInfo& t) {
    const int4 r = a.tile_rec[tile];
    t.expert = r.x; t.row0 = r.y; t.rows = r.z; t.slot = r.w;
    return t.rows > 0 && t.slot >= 0;
}

// h[row][n] = bf16( silu(x W1) * (x W3) ).  A workgroup is two pairs of wavefronts; each
// pair owns one 128-column strip: the even wavefront multiplies by W1 (gate), the odd one by
// W3 (up), the odd one hands its accumulators over through LDS and the even one applies
// SwiGLU and stores.  Splitting the two matrices over two wavefronts halves the accumulator
// registers per wavefront, which is what leaves room for the deep load ring.
// LISTED: the tile's pairs are in pair_list (LDS), row by row; otherwise they are read from a.sorted_pair.
// HALVES: the workgroup has one strip, and its two pairs of wavefronts take half of the k range each: as many bytes in
// flight per workgroup, twice the workgroups, no empty second strip where their number is odd, and no partial sums.
// 64 experts of H 2880 F 360, 333 tokens, top-4 (three strips; split two ways over K before): 115 -> 106 us a call with the
// numbering of workgroups below, one token's top-10 of 512 experts (H 2048 F 512) 28.9 -> 28.4.
template <int MI, bool LISTED, bool HALVES, bool SPLIT>
__device__ __forceinline__ void gemm1_swiglu_body(const FfnArgs& a, const TileInfo& t, float (*xch)[64], uint16_t* abuf, const int32_t* pair_list,
                                                  uint32_t col_wg, uint32_t split, uint32_t n_split) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));   // uniform: scalar address arithmetic
    const int pair = wave >> 1;
    const int mat_id = wave & 1;
    const uint32_t strip = HALVES ? col_wg : col_wg * 2 + pair;
    const uint32_t n0 = strip * kStrip + 8u * (lane & 15);
    const bool col_ok = n0 < a.F;                 // strips past F still run (barrier below)

    const uint16_t* arow[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int32_t r = min(mi * 16 + (lane & 15), t.rows - 1);
        const int32_t pr = LISTED ? pair_list[r] : a.sorted_pair[t.row0 + r];
        const uint32_t tok = uint32_t(pr) / a.K;
        arow[mi] = a.tokens + size_t(tok) * a.H;
    }
    const size_t mat = size_t(a.H) * a.F;
    const uint16_t* w = a.slots13 + size_t(t.slot) * 2 * mat + size_t(mat_id) * mat;

    // the thread's pieces of the shared A blocks: row 16 i + tid / 16, piece (tid % 16) ^ (tid / 16 % 16)
    const uint32_t piece = (threadIdx.x & 15u) ^ ((threadIdx.x >> 4) & 15u);
    uint32_t aoff[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int32_t r = min(i * 16 + int(threadIdx.x >> 4), t.rows - 1);
        const int32_t pr = LISTED ? pair_list[r] : a.sorted_pair[t.row0 + r];
        aoff[i] = 2u * ((uint32_t(pr) / a.K) * a.H + 8u * piece);          // the launcher checks T * H * 2 < 4 GiB
    }
    // K split `split` multiplies k rows [k_begin, k_end): whole A blocks, the last split what remains
    constexpr uint32_t kUnit = HALVES ? 2 * kABlock : kABlock;
    const uint32_t k_per = SPLIT ? ((a.H + n_split - 1) / n_split + kUnit - 1) / kUnit * kUnit : a.H;
    const uint32_t k_begin = SPLIT ? min(a.H, split * k_per) : 0u;
    const uint32_t k_end = min(a.H, k_begin + k_per);
    StripGemm<MI> g;
    g.zero();
    const uint32_t n_blocks = (k_end - k_begin) / kUnit;
    g.template run_shared<HALVES>(reinterpret_cast<const uint8_t*>(a.tokens), aoff, abuf, w, a.H, col_ok ? n0 : a.F - 8, a.F, k_begin, n_blocks, lane, wave, uint32_t(pair));
    // what is left is less than a block, or two with HALVES: one to each pair, the tail to the second (written as a remainder,
    // so that the compiler knows how short it is and drops the long loop of run())
    uint32_t left = (k_end - k_begin) % kUnit, k_left = k_end - left;
    if (HALVES) {
        const uint32_t first = min(left, uint32_t(kABlock));
        if (pair == 0) left = first;
        else { k_left += first; left -= first; }
    }
    g.run(arow, w + (col_ok ? n0 : a.F - 8), a.F, k_left, k_left + left, lane);

    if (HALVES) {                                 // the second pair's sums are added to the first's
        mfma_drain();
        if (pair == 1) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int c = 0; c < 8; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) xch[mat_id * (MI * 32) + (mi * 8 + c) * 4 + r][lane] = g.acc[mi][c][r];
        }
        __syncthreads();
        if (pair == 0) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int c = 0; c < 8; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) g.acc[mi][c][r] += xch[mat_id * (MI * 32) + (mi * 8 + c) * 4 + r][lane];
        }
        __syncthreads();                          // the memory is used again below
    }

    if (SPLIT && n_split > 1) {                   // partial sums of both matrices, added up by swiglu_reduce_kernel
        if (!col_ok || (HALVES && pair == 1)) return;
        float* part = a.part + (size_t(split) * a.pairs_cap + size_t(t.row0)) * 2 * a.F + size_t(mat_id) * a.F + n0;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t row = mi * 16 + 4 * (lane >> 4) + r;
                if (row >= t.rows) continue;
                float4* dst = reinterpret_cast<float4*>(part + size_t(uint32_t(row)) * 2 * a.F);
                dst[0] = make_float4(g.acc[mi][0][r], g.acc[mi][1][r], g.acc[mi][2][r], g.acc[mi][3][r]);
                dst[1] = make_float4(g.acc[mi][4][r], g.acc[mi][5][r], g.acc[mi][6][r], g.acc[mi][7][r]);
            }
        return;
    }
    if (mat_id == 1 && !(HALVES && pair == 1)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) xch[pair * (MI * 32) + (mi * 8 + c) * 4 + r][lane] = g.acc[mi][c][r];
    }
    __syncthreads();
    if (mat_id == 1 || !col_ok || (HALVES && pair == 1)) return;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int32_t row = mi * 16 + 4 * (lane >> 4) + r;
            if (row >= t.rows) continue;
            float hv[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float ga = g.acc[mi][c][r];
                const float up = xch[pair * (MI * 32) + (mi * 8 + c) * 4 + r][lane];
                hv[c] = swiglu(ga, up);
            }
            uint4 o;
            o.x = pack_bf16_rne(hv[0], hv[1]);
            o.y = pack_bf16_rne(hv[2], hv[3]);
            o.z = pack_bf16_rne(hv[4], hv[5]);
            o.w = pack_bf16_rne(hv[6], hv[7]);
            *reinterpret_cast<uint4*>(a.hbuf + size_t(t.row0 + row) * a.F + n0) = o;
        }
}

// Row tiles hold up to 16 MI rows so that an expert's weights are streamed once even when routing is
// skewed (an expert with 231 of 2560 pairs next to hundreds with five); a tile with fewer rows takes a
// body compiled for fewer 16-row MFMA tiles (less matrix work per chunk, same registers reserved).
// ROUTE (at most kRoutedPairs pairs): there is no grouping kernel in front; every workgroup groups the pairs for itself, a
// pair per lane, and the first ones write the lists the later kernels read.  A decode step of a token or two is launches:
// the grouping kernel was 6 of the 34 us of one token's top-10 of 512 experts (H 2048, F 512), 29 without it.
// Tiles are the distinct experts in order of first appearance (one tile each: no more rows than a strip tile holds).
// SPLIT: a launch that may split K.  Without it the store of partial sums is not compiled in: next to the other epilogue it
// costs the 128-row kernel 61 spilled registers instead of 8 (8 experts of H 4096 F 14336, 128 rows each: 794 -> 775 us a call).
template <int MI, bool ROUTE, bool HALVES, bool SPLIT>
__global__ __launch_bounds__(256) void gemm1_swiglu_kernel(FfnArgs a) {
    // the accumulator exchange of the epilogue ([pair][mi, c, r][lane] floats) reuses the memory of
    // the shared A blocks: every wavefront has passed the last block's barrier by then
    constexpr size_t kXchBytes = sizeof(float) * 2 * MI * 8 * 4 * 64;
    constexpr size_t kABytes = sizeof(uint16_t) * (HALVES ? 4 : 2) * StripGemm<MI>::kABufElems;
    __shared__ __align__(16) uint8_t smem[kXchBytes > kABytes ? kXchBytes : kABytes];
    __shared__ int32_t pair_list[ROUTE ? kRoutedPairs : 1];
    float (*xch)[64] = reinterpret_cast<float (*)[64]>(smem);
    uint16_t* abuf = reinterpret_cast<uint16_t*>(smem);
    TileInfo t;
    // column workgroup, K split, row tile: the three dimensions of the grid, or (a.g1_xcd) numbered as in gemm2_kernel so that
    // the column workgroups of a (tile, split) share an XCD and find the tile's activations, and where rows of the weights
    // are not whole 128-byte lines the line that two strips share, in its L2
    // The tiles come last: the numbers past the last tile are then the last ones and every XCD gets its share of the others (160 experts of
    // H 5120 F 1536, one token, top-8, five splits: 240 of 270 workgroups have work; with the splits last 86 us a call, now 69).  In several rounds, splits
    // last / tiles last: 8 of H 4568 F 6480, 5 tokens, top-8 306 / 289, of H 4584 F 10616, 7 497 / 469, 32 of H 4824 F 1160, 6, top-6 168 / 167, but 60 of
    // H 3968 F 4864, 8 tokens 119 / 122, 290 of H 4608 F 872, 41 tokens 156 / 160.
    uint32_t col_wg = blockIdx.x, tile_no = blockIdx.z, split = blockIdx.y;
    if (!ROUTE && a.g1_xcd) {
        const uint32_t n_cw = HALVES ? (a.F + kStrip - 1) / kStrip : (a.F + 2 * kStrip - 1) / (2 * kStrip);
        const uint32_t xcd = blockIdx.x % 8u, q = blockIdx.x / 8u;
        col_wg = q % n_cw;
        const uint32_t unit = (q / n_cw) * 8u + xcd;
        if (unit >= a.tiles_cap * a.ksplit1) return;
        tile_no = unit / a.ksplit1;
        split = unit % a.ksplit1;
    }
    const uint32_t n_tiles_all = SPLIT && !ROUTE ? uint32_t(a.n_tiles[0]) : 0u;      // travels together with the tile's record
    if (ROUTE) {
        static_assert(!ROUTE || (16 * MI >= int(kRoutedPairs) && kRoutedPairs == 64), "a pair per lane, an expert's pairs in one tile");
        const int lane = threadIdx.x & 63;
        const uint32_t pairs = a.T * a.K, tile = tile_no;
        const bool lists = blockIdx.x == 0 && split == 0;                   // uniform
        const int32_t id = uint32_t(lane) < pairs ? a.topk_ids[lane] : -1;
        const bool known = id >= 0 && uint32_t(id) < a.E;
        const int32_t slot = known ? a.page_table[id] : -1;
        const bool valid = slot >= 0;
        const uint64_t valid_mask = __ballot(valid);
        // the first valid pair with the same expert
        int leader = lane;
        for (int q = int(pairs) - 1; q >= 0; --q)
            if (__builtin_amdgcn_readlane(id, q) == id) leader = q;
        const uint64_t leaders = __ballot(valid && leader == lane);
        const uint32_t n_tiles = uint32_t(__popcll(leaders));
        if (lists && tile == 0 && threadIdx.x < 64) {
            if (uint32_t(lane) < pairs && !valid && (!known || !(a.flags & 2u))) atomicOr(a.error_word, 2u);
            // position of the lane's pair: pairs of earlier experts, then its own expert's earlier pairs
            int32_t pos = 0;
            for (uint32_t q = 0; q < pairs; ++q) {
                const int lq = __builtin_amdgcn_readlane(leader, q);
                if (((valid_mask >> q) & 1u) && (lq < leader || (lq == leader && int(q) < lane))) ++pos;
            }
            if (uint32_t(lane) < pairs) a.pair_pos[lane] = valid ? pos : -1;
            if (lane == 0) {
                a.expert_offset[a.E] = int32_t(__popcll(valid_mask));
                a.n_tiles[0] = int32_t(n_tiles);
            }
        }
        if (tile >= n_tiles) {
            if (lists && threadIdx.x == 0) a.tile_rec[tile] = make_int4(0, 0, 0, -1);
            return;
        }
        uint64_t rest = leaders;
        for (uint32_t i = 0; i < tile; ++i) rest &= rest - 1;
        const int first = __builtin_ctzll(rest);
        const uint64_t mine = __ballot(valid && leader == first);
        t.expert = __builtin_amdgcn_readlane(id, first);
        t.slot = __builtin_amdgcn_readlane(slot, first);
        t.rows = __popcll(mine);
        t.row0 = __popcll(__ballot(valid && leader < first));
        if (lists && threadIdx.x == 0) a.tile_rec[tile] = make_int4(t.expert, t.row0, t.rows, t.slot);
        if (threadIdx.x < 64 && valid && leader == first) pair_list[__popcll(mine & ((1ull << lane) - 1ull))] = lane;
        __syncthreads();
    } else if (!tile_info(a, tile_no, t)) {
        return;                                       // uniform over the workgroup
    }
    const uint32_t n_split = !SPLIT ? 1u : (ROUTE ? a.ksplit1 : first_splits(a, n_tiles_all));
    if (SPLIT && split >= n_split) return;
    if (MI > 1 && t.rows <= 16) gemm1_swiglu_body<1, ROUTE, HALVES, SPLIT>(a, t, xch, abuf, pair_list, col_wg, split, n_split);
    else if (MI > 2 && t.rows <= 32) gemm1_swiglu_body<2, ROUTE, HALVES, SPLIT>(a, t, xch, abuf, pair_list, col_wg, split, n_split);
    else if (MI > 4 && t.rows <= 64) gemm1_swiglu_body<4, ROUTE, HALVES, SPLIT>(a, t, xch, abuf, pair_list, col_wg, split, n_split);
    else if (MI > 6 && t.rows <= 96) gemm1_swiglu_body<6, ROUTE, HALVES, SPLIT>(a, t, xch, abuf, pair_list, col_wg, split, n_split);
    else gemm1_swiglu_body<MI, ROUTE, HALVES, SPLIT>(a, t, xch, abuf, pair_list, col_wg, split, n_split);
}

// y[split][row][n] = h[row][k range] W2[k range][n]
template <int MI>
__device__ __forceinline__ void gemm2_body(const FfnArgs& a, const TileInfo& t, uint16_t* abuf, uint32_t col_wg, uint32_t split) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const uint32_t strip = col_wg * 4 + wave;
    const uint32_t n0 = strip * kStrip + 8u * (lane & 15);
    const bool col_ok = n0 < a.H;                 // wavefronts past the last strip still run (barriers below)
    const uint32_t k_per = ((a.F + a.ksplit - 1) / a.ksplit + kChunk - 1) / kChunk * kChunk;
    const uint32_t k_begin = min(a.F, split * k_per);
    const uint32_t k_end = min(a.F, k_begin + k_per);

    const uint16_t* arow[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int32_t r = min(mi * 16 + (lane & 15), t.rows - 1);
        arow[mi] = a.hbuf + size_t(t.row0 + r) * a.F;
    }
    const uint16_t* w2 = a.slots2 + size_t(t.slot) * a.F * a.H;

    // the thread's pieces of the shared A blocks, as byte offsets from the tile's first row of h
    const uint32_t piece = (threadIdx.x & 15u) ^ ((threadIdx.x >> 4) & 15u);
    uint32_t aoff[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int32_t r = min(i * 16 + int(threadIdx.x >> 4), t.rows - 1);
        aoff[i] = 2u * (uint32_t(r) * a.F + 8u * piece);
    }
    StripGemm<MI> g;
    g.zero();
    const uint32_t n_blocks = (k_end - k_begin) / kABlock;
    g.template run_shared<false>(reinterpret_cast<const uint8_t*>(a.hbuf + size_t(t.row0) * a.F), aoff, abuf, w2, a.F, col_ok ? n0 : a.H - 8, a.H,
                 k_begin, n_blocks, lane, wave, 0);
    g.run(arow, w2 + (col_ok ? n0 : a.H - 8), a.H, k_begin + n_blocks * kABlock, k_end, lane);

    if (!col_ok) return;
    float* y = a.ybuf + size_t(split) * a.pairs_cap * a.H;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int32_t row = mi * 16 + 4 * (lane >> 4) + r;
            if (row >= t.rows) continue;
            float4 lo = make_float4(g.acc[mi][0][r], g.acc[mi][1][r], g.acc[mi][2][r], g.acc[mi][3][r]);
            float4 hi = make_float4(g.acc[mi][4][r], g.acc[mi][5][r], g.acc[mi][6][r], g.acc[mi][7][r]);
            float4* dst = reinterpret_cast<float4*>(y + size_t(t.row0 + row) * a.H + n0);
            dst[0] = lo;
            dst[1] = hi;
        }
}

template <int MI>
__global__ __launch_bounds__(256) void gemm2_kernel(FfnArgs a) {
    __shared__ __align__(16) uint16_t abuf[2 * StripGemm<MI>::kABufElems];
    // One-dimensional grid.  Workgroups go to the 8 XCDs round robin, so workgroup L runs on XCD L % 8; the
    // column workgroups of one (tile, K split) all read the same rows of h, so they are numbered to land on
    // one XCD back to back and find those rows in its L2 (on 8 XCDs each would fetch them from HBM again).
    const uint32_t n_cw = (a.H + 4 * kStrip - 1) / (4 * kStrip);
    const uint32_t xcd = blockIdx.x % 8u, q = blockIdx.x / 8u;
    const uint32_t col_wg = q % n_cw;
    const uint32_t pair = (q / n_cw) * 8u + xcd;             // (tile, split), tile-major
    if (pair >= a.tiles_cap * a.ksplit) return;
    const uint32_t tile = pair / a.ksplit, split = pair % a.ksplit;
    TileInfo t;
    if (!tile_info(a, tile, t)) return;
    if (MI > 1 && t.rows <= 16) gemm2_body<1>(a, t, abuf, col_wg, split);
    else if (MI > 2 && t.rows <= 32) gemm2_body<2>(a, t, abuf, col_wg, split);
    else if (MI > 4 && t.rows <= 64) gemm2_body<4>(a, t, abuf, col_wg, split);
    else if (MI > 6 && t.rows <= 96) gemm2_body<6>(a, t, abuf, col_wg, split);
    else gemm2_body<MI>(a, t, abuf, col_wg, split);
}

// The second product of a call of few pairs, bound by its start-up and by how many CUs have work: a workgroup has one strip of 128
// columns of one expert and its four wavefronts a quarter of the k range each, so a token's ten experts of F 512 give 160 workgroups
// where four strips to a workgroup and two K splits gave 80, and there are no partial sums to write (27.8 -> 26.0 us a call).
// FUSED: the first product's partial sums are added up here, each wavefront its own quarter's, while its first weights are on
// their way: one launch less (26.0 -> 24.3).  For up to four tokens: every strip's workgroup repeats the sums of its expert's rows.
// Combining in the workgroup that is the last of its strip was tried: with device-wide fences 33, with stores and loads that pass the
// L2s by 24.0, which is not worth depending on.
template <int MI, bool FUSED>
__device__ __forceinline__ void gemm2_few_body(const FfnArgs& a, const TileInfo& t, uint32_t row_first, uint8_t* smem, uint32_t strip, uint32_t split) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const uint32_t n0 = strip * kStrip + 8u * (lane & 15);
    const bool col_ok = n0 < a.H;
    const uint32_t col = col_ok ? n0 : a.H - 8;
    const uint32_t k_per = ((a.F + a.ksplit - 1) / a.ksplit + kChunk - 1) / kChunk * kChunk;
    const uint32_t k_lo = min(a.F, split * k_per), k_hi = min(a.F, k_lo + k_per);
    const uint32_t quarter = ((k_per + 3) / 4 + kChunk - 1) / kChunk * kChunk;
    const uint32_t k_begin = min(k_hi, k_lo + uint32_t(wave) * quarter), k_end = min(k_hi, k_begin + quarter);
    const int32_t rows = min(int32_t(16 * MI), t.rows - int32_t(row_first));
    const uint16_t* w2 = a.slots2 + size_t(t.slot) * a.F * a.H;
    StripGemm<MI> g;
    f32x4 sums[8];                               // FUSED: through the compiler's MFMA, which needs no pinned accumulators here
    if constexpr (FUSED) {
        static_assert(!FUSED || MI == 1, "up to four tokens");
#pragma unroll
        for (int c = 0; c < 8; ++c) sums[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto mma = [&](const uint4 (&b)[8], const uint4& af) __attribute__((always_inline)) {
            Frag fa;
            fa.u = af;
#pragma unroll
            for (int c = 0; c < 8; ++c) sums[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa.v, StripGemm<MI>::column(b, c).v, sums[c], 0, 0, 0);
        };
        const uint32_t row_bytes = 2u * a.H;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w2), 0, int(a.F * row_bytes), 0x00020000);
        const uint32_t voff = 8u * (uint32_t(lane) >> 4) * row_bytes + 2u * col, chunk_bytes = uint32_t(kChunk) * row_bytes;
        // whole chunks of 32 k, and what is left of F behind the last of them
        const uint32_t n = (k_end - k_begin) / kChunk, k_tail = k_begin + n * kChunk;
        uint4 b[4][8];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (uint32_t(s) < n) StripGemm<MI>::load_b(b[s], rsrc, voff, k_begin * row_bytes + uint32_t(s) * chunk_bytes, row_bytes);
        const uint32_t n_split = a.ksplit1;
        // h of this quarter in LDS, 16 rows of `pitch` elements
        const uint32_t pitch = quarter + 8;
        uint16_t* const hs = reinterpret_cast<uint16_t*>(smem) + uint32_t(wave) * 16u * pitch;
        for (uint32_t kb = 0; kb < k_end - k_begin; kb += 128) {
            const uint32_t k = kb + 4u * (lane & 31);
            for (int32_t r2 = 0; r2 < rows; r2 += 2) {
                const int32_t r = r2 + (lane >> 5);
                const float* part = a.part + (size_t(t.row0) + row_first + uint32_t(min(r, rows - 1))) * 2 * a.F + min(k_begin + k, a.F - 4);
                float gs[4] = {0.f, 0.f, 0.f, 0.f}, us[4] = {0.f, 0.f, 0.f, 0.f};
                for (uint32_t s0 = 0; s0 < n_split; s0 += 4) {
                    float4 gv[4], uv[4];
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) {
                        const float* at = part + size_t(min(s0 + i, n_split - 1)) * a.pairs_cap * 2 * a.F;
                        gv[i] = *reinterpret_cast<const float4*>(at);
                        uv[i] = *reinterpret_cast<const float4*>(at + a.F);
                    }
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i)
                        if (s0 + i < n_split) {
                            gs[0] += gv[i].x; gs[1] += gv[i].y; gs[2] += gv[i].z; gs[3] += gv[i].w;
                            us[0] += uv[i].x; us[1] += uv[i].y; us[2] += uv[i].z; us[3] += uv[i].w;
                        }
                }
                if (k < k_end - k_begin && r < rows)
                    *reinterpret_cast<uint2*>(hs + uint32_t(r) * pitch + k) = make_uint2(pack_bf16_rne(swiglu(gs[0], us[0]), swiglu(gs[1], us[1])),
                                                                                         pack_bf16_rne(swiglu(gs[2], us[2]), swiglu(gs[3], us[3])));
            }
        }
        asm volatile("" ::: "memory");           // the wavefront's own LDS writes and reads stay in order
        const uint16_t* const ha = hs + uint32_t(min(lane & 15, rows - 1)) * pitch + 8u * (uint32_t(lane) >> 4);
        for (uint32_t base = 0; base < n; base += 4) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (base + s >= n) break;
                mma(b[s], *reinterpret_cast<const uint4*>(ha + (base + s) * kChunk));
                if (base + s + 4 < n) StripGemm<MI>::load_b(b[s], rsrc, voff, k_begin * row_bytes + (base + s + 4) * chunk_bytes, row_bytes);
            }
        }
        if (k_tail < k_end) {                    // (lanes past the end contribute zeros)
            uint4 af = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 8; ++r) b[0][r] = af;
            if (k_tail + 8u * (uint32_t(lane) >> 4) < k_end) {
                StripGemm<MI>::load_b(b[0], rsrc, voff, k_tail * row_bytes, row_bytes);
                af = *reinterpret_cast<const uint4*>(ha + n * kChunk);
            }
            mma(b[0], af);
        }
        __syncthreads();                         // the memory is used again below
    } else {
        g.zero();
        const uint16_t* arow[MI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) arow[mi] = a.hbuf + (size_t(t.row0) + row_first + uint32_t(min(mi * 16 + (lane & 15), rows - 1))) * a.F;
        g.run(arow, w2 + col, a.H, k_begin, k_end, lane);
    }

    float* const y = a.ybuf + (size_t(split) * a.pairs_cap + size_t(t.row0) + row_first) * a.H;
    float (*xch)[64] = reinterpret_cast<float (*)[64]>(smem);
    if constexpr (MI == 1) {
        // the four wavefronts' sums through LDS: each adds up two of the lane's eight columns, in the order of k
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) xch[wave * 32 + c * 4 + r][lane] = FUSED ? sums[c][r] : g.acc[0][c][r];
        __syncthreads();
        if (col_ok) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t row = 4 * (lane >> 4) + r;
                if (row >= rows) continue;
                float v[2];
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const int at = (2 * wave + d) * 4 + r;
                    v[d] = ((xch[at][lane] + xch[32 + at][lane]) + xch[64 + at][lane]) + xch[96 + at][lane];
                }
                *reinterpret_cast<float2*>(y + size_t(uint32_t(row)) * a.H + n0 + 2 * wave) = make_float2(v[0], v[1]);
            }
        }
    } else {
        // wavefronts 2 and 3 hand their sums to 0 and 1, then 1 to 0
#pragma unroll
        for (int from = 2; from >= 1; from >>= 1) {
            if (wave >= from && wave < 2 * from) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int c = 0; c < 8; ++c)
#pragma unroll
                        for (int r = 0; r < 4; ++r) xch[(wave - from) * (MI * 32) + (mi * 8 + c) * 4 + r][lane] = g.acc[mi][c][r];
            }
            __syncthreads();
            if (wave < from) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int c = 0; c < 8; ++c)
#pragma unroll
                        for (int r = 0; r < 4; ++r) g.acc[mi][c][r] += xch[wave * (MI * 32) + (mi * 8 + c) * 4 + r][lane];
            }
            __syncthreads();
        }
        if (wave == 0 && col_ok) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t row = mi * 16 + 4 * (lane >> 4) + r;
                    if (row >= rows) continue;
                    float4* dst = reinterpret_cast<float4*>(y + size_t(uint32_t(row)) * a.H + n0);
                    dst[0] = make_float4(g.acc[mi][0][r], g.acc[mi][1][r], g.acc[mi][2][r], g.acc[mi][3][r]);
                    dst[1] = make_float4(g.acc[mi][4][r], g.acc[mi][5][r], g.acc[mi][6][r], g.acc[mi][7][r]);
                }
        }
    }
}

template <int MI, bool FUSED>
__global__ __launch_bounds__(256, MI == 1 ? 2 : 1) void gemm2_few_kernel(FfnArgs a) {
    extern __shared__ __align__(16) uint8_t few_smem[];
    TileInfo t;
    if (!tile_info(a, blockIdx.z, t)) return;
    for (uint32_t r = 0; r < uint32_t(t.rows); r += 16 * MI) {
        if (r) __syncthreads();
        if (MI > 1 && t.rows <= 16) gemm2_few_body<1, FUSED>(a, t, r, few_smem, blockIdx.x, blockIdx.y);
        else gemm2_few_body<MI, FUSED>(a, t, r, few_smem, blockIdx.x, blockIdx.y);
    }
}

// h[row][n] = bf16( silu(gate) * up ), gate and up summed over the K splits of the first product in split order.
// Bound by its launch at the sizes that split (a few hundred kilobytes to 30 MB of sums, still in the caches): a launch
// of its own is cheaper than the device-wide fence a last-arriver scheme inside the product would take.
__global__ __launch_bounds__(256) void swiglu_reduce_kernel(FfnArgs a) {
    const uint32_t per_row = a.F / 8;
    const uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x;
    const uint32_t row = uint32_t(i / per_row), n0 = 8u * uint32_t(i % per_row);
    uint32_t n_split = a.ksplit1, rows = a.T;
    if (!a.identity) {                           // the two loads travel together
        const uint32_t found = uint32_t(a.n_tiles[a.tiled && a.m_tile == 256 ? 1 : 0]);
        rows = uint32_t(a.expert_offset[a.E]);
        n_split = a.tiled && a.m_tile == 256 ? found : first_splits(a, found);
    }
    if (n_split == 1 || row >= rows) return;       // h is there already; rows past the pairs whose expert is mapped
    float g[8], u[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) g[c] = u[c] = 0.f;
    const float* part = a.part + size_t(row) * 2 * a.F + n0;
    for (uint32_t sp = 0; sp < n_split; ++sp, part += size_t(a.pairs_cap) * 2 * a.F) {
        const float4 g0 = *reinterpret_cast<const float4*>(part), g1 = *reinterpret_cast<const float4*>(part + 4);
        const float4 u0 = *reinterpret_cast<const float4*>(part + a.F), u1 = *reinterpret_cast<const float4*>(part + a.F + 4);
        g[0] += g0.x; g[1] += g0.y; g[2] += g0.z; g[3] += g0.w; g[4] += g1.x; g[5] += g1.y; g[6] += g1.z; g[7] += g1.w;
        u[0] += u0.x; u[1] += u0.y; u[2] += u0.z; u[3] += u0.w; u[4] += u1.x; u[5] += u1.y; u[6] += u1.z; u[7] += u1.w;
    }
    uint4 o;
    o.x = pack_bf16_rne(swiglu(g[0], u[0]), swiglu(g[1], u[1]));
    o.y = pack_bf16_rne(swiglu(g[2], u[2]), swiglu(g[3], u[3]));
    o.z = pack_bf16_rne(swiglu(g[4], u[4]), swiglu(g[5], u[5]));
    o.w = pack_bf16_rne(swiglu(g[6], u[6]), swiglu(g[7], u[7]));
    *reinterpret_cast<uint4*>(a.hbuf + size_t(row) * a.F + n0) = o;
}

// ------------------------------------------------------------------ large row tiles (MFMA bound)
// When an expert sees hundreds of rows (prefill-shaped batches, the shared expert) the FFN is
// bound by the matrix cores, not by weight streaming, and operands must be reused from LDS.
// Workgroup tile 256 rows x 256 columns, k step 64, eight wavefronts as 4 (rows) x 2 (columns),
// two per SIMD so that one wavefront's LDS and barrier waits hide behind the other's MFMAs.
// Each wavefront owns 64 x 128 as 2 x 4 tiles of v_mfma_f32_32x32x16_bf16 (128 accumulator
// registers).  A rows (k contiguous) go to LDS as they are; B arrives row-major [k][n], so
// each lane transposes an 8 (k) x 4 (n) tile in registers (v_perm_b32) and writes [n][k] rows,
// after which both operands are read as 16-byte k-contiguous fragments.  LDS rows are padded
// by 16 bytes (conflict-free 16-byte reads); column c of a lane's tile goes to an LDS row
// chosen so that the 64 lanes of a write hit consecutive rows.  Two LDS buffers, one barrier
// per k step; the registers hold step s + 1 while step s is multiplied, are written to the
// other buffer between the MFMAs of step s and at once reloaded with step s + 2.
// Workgroups are numbered so that the 32 that run together on one XCD (one per CU) form a
// 4 x 8 block of tiles and share operand slices in that XCD's L2.
// MODE 1: the 256 tile columns are 128 of W1 and the same 128 of W3; a wavefront holds gate
// and up values of the same elements and applies SwiGLU in registers.  MODE 2: y = h W2.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kTM = 256, kTK = 64, kLdsPitch = kTK + 8;   // pitch in BF16 elements
constexpr uint32_t kSuperM = 4, kSuperN = 8;              // tiles per super-tile (one XCD's 32 CUs)

template <int MODE>
__global__ __launch_bounds__(512) void gemm_tiled_kernel(FfnArgs a) {
    extern __shared__ __align__(16) uint16_t lds[];
    const uint32_t K = MODE == 1 ? a.H : a.F;
    const uint32_t N = MODE == 1 ? a.F : a.H;               // columns of one B matrix
    const uint32_t ncols_tile = MODE == 1 ? 128u : 256u;     // distinct output columns per tile
    const uint32_t n_ct = (N + ncols_tile - 1) / ncols_tile;
    const uint32_t n_rt = uint32_t(a.n_tiles[0]);
    const uint32_t n_sn = (n_ct + kSuperN - 1) / kSuperN;
    const uint32_t xcd = blockIdx.x % 8u, jj = blockIdx.x / 8u;
    const uint32_t st = (jj / (kSuperM * kSuperN)) * 8u + xcd;
    const uint32_t within = jj % (kSuperM * kSuperN);
    const uint32_t row_tile = (st / n_sn) * kSuperM + within / kSuperN;
    const uint32_t col_tile = (st % n_sn) * kSuperN + within % kSuperN;
    if (row_tile >= n_rt || col_tile >= n_ct) return;
    TileInfo t;
    if (!tile_info(a, row_tile, t)) return;
    const uint32_t n_base = col_tile * ncols_tile;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int q = lane & 31;
    constexpr int kTile = kTM * kLdsPitch;                   // LDS: [buffer][A tile | B tile]

    // global -> register staging.  A: 8 lanes cover one row's 64 k; rows tid / 8 + 64 i.
    const uint16_t* a_src[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int32_t r = min(int32_t(tid >> 3) + 64 * i, t.rows - 1);
        if (MODE == 1) {
            const int32_t pr = a.sorted_pair[t.row0 + r];
            a_src[i] = a.tokens + size_t(uint32_t(pr) / a.K) * a.H + 8 * (tid & 7);
        } else {
            a_src[i] = a.hbuf + size_t(t.row0 + r) * a.F + 8 * (tid & 7);
        }
    }
    const int a_dst = (tid >> 3) * kLdsPitch + 8 * (tid & 7);          // + 64 i rows
    // B: the lane's tile: 4 consecutive columns, 8 rows k = 8 (tid / 64) ..
    const uint32_t cg = tid & 63;
    const uint32_t bk = 8u * (tid >> 6);
    const uint16_t* b_src;
    int b_dst_row;                                           // + c * (MODE 1 ? 32 : 64) rows
    {
        const size_t mat = size_t(a.H) * a.F;
        if (MODE == 1) {
            const uint32_t col = min(n_base + 4u * (cg & 31u), N - 4);
            b_src = a.slots13 + size_t(t.slot) * 2 * mat + (cg >= 32 ? mat : 0) + col;
            b_dst_row = int(cg >> 5) * 128 + int(cg & 31);
        } else {
            const uint32_t col = min(n_base + 4u * cg, N - 4);
            b_src = a.slots2 + size_t(t.slot) * mat + col;
            b_dst_row = int(cg);
        }
    }
    constexpr int b_dst_step = MODE == 1 ? 32 : 64;
    const int b_dst = kTile + b_dst_row * kLdsPitch + int(bk);

    f32x16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // LDS fragment offsets of this wavefront (k-contiguous 16-byte reads).
    // MODE 2: B tile j = LDS rows 32 (4 wn + j) + q: column 4 (32 (j & 1) + q) + 2 wn + j / 2
    // MODE 1: j = 0, 1 gate, j = 2, 3 up: rows 128 (j / 2) + 32 (2 wn + j % 2) + q: column 4 q + 2 wn + j % 2
    const int kfrag = 8 * (lane >> 5);
    const int a_frag = (wm * 64 + q) * kLdsPitch + kfrag;                // + 32 i rows
    int b_frag[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = MODE == 1 ? ((j >> 1) * 128 + (2 * wn + (j & 1)) * 32 + q) : ((4 * wn + j) * 32 + q);
        b_frag[j] = kTile + row * kLdsPitch + kfrag;
    }

    u32x4 ga[4];
    u32x2 gb[8];
    const uint32_t n_steps = K / kTK;
    // item n of a step's 12 global loads: 0..3 the lane's A rows, 4..11 the 8 k rows of its B tile
    auto gload_item = [&](uint32_t k0, int n) __attribute__((always_inline)) {
        if (n < 4) ga[n] = *reinterpret_cast<const u32x4*>(a_src[n] + k0);
        else gb[n - 4] = *reinterpret_cast<const u32x2*>(b_src + size_t(k0 + bk + (n - 4)) * N);
    };
    // item n of a step's 8 LDS writes: 0..3 A rows, 4..7 column c = n - 4 of the transposed B tile
    auto lstore_item = [&](uint16_t* buf, int n) __attribute__((always_inline)) {
        if (n < 4) {
            *reinterpret_cast<u32x4*>(buf + a_dst + 64 * n * kLdsPitch) = ga[n];
        } else {
            const int c = n - 4;
            u32x4 v;
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
            v.x = __builtin_amdgcn_perm(gb[1][c >> 1], gb[0][c >> 1], sel);
            v.y = __builtin_amdgcn_perm(gb[3][c >> 1], gb[2][c >> 1], sel);
            v.z = __builtin_amdgcn_perm(gb[5][c >> 1], gb[4][c >> 1], sel);
            v.w = __builtin_amdgcn_perm(gb[7][c >> 1], gb[6][c >> 1], sel);
            *reinterpret_cast<u32x4*>(buf + b_dst + c * b_dst_step * kLdsPitch) = v;
        }
    };
    bf16x8 fa[2][2], fb[2][4];
    // item n of the 6 fragment reads of sub-step ks into register set `set`
    auto lfrag_item = [&](const uint16_t* buf, int ks, int set, int n) __attribute__((always_inline)) {
        if (n < 2) fa[set][n] = *reinterpret_cast<const bf16x8*>(buf + a_frag + 32 * n * kLdsPitch + ks * 16);
        else fb[set][n - 2] = *reinterpret_cast<const bf16x8*>(buf + b_frag[n - 2] + ks * 16);
    };
    auto mfma_item = [&](int set, int n) __attribute__((always_inline)) {
        const int i = n >> 2, j = n & 3;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
    };

    // One k step.  STORE: refill the other buffer from the staging registers; LOAD: fetch step
    // s + 2 into them; NEXT: read the first fragments of the other buffer after the barrier.
    // A workgroup moves 64 KB per step through the vector memory path (64 B/clk per CU) and again
    // into LDS; issued in one burst, those instructions hold the issuing wavefronts for over a
    // thousand cycles while the matrix cores idle.  They are therefore issued one at a time
    // between the MFMAs (the scheduling barriers keep that order): the fragments of sub-step
    // ks + 1 and the 8 LDS writes during sub-step 0, the 12 global loads during sub-steps 1 and 2.
    // The step's barrier sits before the MFMAs of sub-step 3, which cover the first fragment
    // reads from the other buffer.
    auto step = [&](const uint16_t* cur, uint16_t* nxt, uint32_t k_next, auto STORE, auto LOAD, auto NEXT) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 8; ++n) {                         // sub-step 0 (set 0)
            mfma_item(0, n);
            if (n < 6) lfrag_item(cur, 1, 1, n);
            if (STORE.value) lstore_item(nxt, n);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < 8; ++n) {                         // sub-step 1 (set 1)
            mfma_item(1, n);
            if (n < 6) lfrag_item(cur, 2, 0, n);
            if (LOAD.value && n >= 2) gload_item(k_next, n - 2);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < 8; ++n) {                         // sub-step 2 (set 0)
            mfma_item(0, n);
            if (n < 6) lfrag_item(cur, 3, 1, n);
            if (LOAD.value && n >= 2) gload_item(k_next, 6 + n - 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();                       // all reads of cur are in registers, nxt is complete
#pragma unroll
        for (int n = 0; n < 8; ++n) {                         // sub-step 3 (set 1)
            mfma_item(1, n);
            if (NEXT.value && n < 6) lfrag_item(nxt, 0, 0, n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;

#pragma unroll
    for (int n = 0; n < 12; ++n) gload_item(0, n);
#pragma unroll
    for (int n = 0; n < 8; ++n) lstore_item(lds, n);
    if (n_steps > 1) {
#pragma unroll
        for (int n = 0; n < 12; ++n) gload_item(kTK, n);
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 6; ++n) lfrag_item(lds, 0, 0, n);
    {
        uint16_t* cur = lds;
        uint16_t* nxt = lds + 2 * kTile;
        uint32_t s = 0;
        for (; s + 2 < n_steps; ++s) {
            step(cur, nxt, (s + 2) * kTK, Yes{}, Yes{}, Yes{});
            uint16_t* tmp = cur; cur = nxt; nxt = tmp;
        }
        if (s + 1 < n_steps) {
            step(cur, nxt, 0, Yes{}, No{}, Yes{});
            uint16_t* tmp = cur; cur = nxt; nxt = tmp;
        }
        step(cur, nxt, 0, No{}, No{}, No{});
    }

    // epilogue.  D layout of the 32x32 MFMA: column q = lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int32_t row = wm * 64 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (row >= t.rows) continue;
            if (MODE == 1) {
                const uint32_t col = n_base + 4u * q + 2u * wn;      // two adjacent columns
                if (col >= N) continue;
                const uint32_t packed = pack_bf16_rne(swiglu(acc[i][0][r], acc[i][2][r]), swiglu(acc[i][1][r], acc[i][3][r]));
                *reinterpret_cast<uint32_t*>(a.hbuf + size_t(t.row0 + row) * a.F + col) = packed;
            } else {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const uint32_t col = n_base + 4u * (32 * half + q) + 2u * wn;
                    if (col >= N) continue;
                    *reinterpret_cast<float2*>(a.ybuf + size_t(t.row0 + row) * a.H + col) =
                        make_float2(acc[i][half][r], acc[i][half + 2][r]);
                }
            }
        }
}

// The same tiling with four wavefronts, one per SIMD, each owning 128 x 128 (4 x 4 MFMA tiles, 256
// accumulator registers).  LDS fragment traffic per flop falls by a third against the 64 x 128
// wavefront tile (a 128 x 128 tile reads 256 fragment rows per k for 16384 multiply-adds, the
// 64 x 128 one 192 for 8192), which is what bounds the eight-wavefront kernel.  With a single
// wavefront per SIMD nothing hides a wait, so the loop is software pipelined inside the
// wavefront: the fragments of sub-step ks + 1 are read while sub-step ks is multiplied, the
// refill of the other LDS buffer and the global loads of step s + 2 are spread over the MFMAs of
// sub-steps 0 and 1, and the step's only barrier sits before the MFMAs of sub-step 3, which then
// cover the first fragment reads from the other buffer.
template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_tiled4_kernel(FfnArgs a) {
    extern __shared__ __align__(16) uint16_t lds[];
    const uint32_t K = MODE == 1 ? a.H : a.F;
    const uint32_t N = MODE == 1 ? a.F : a.H;
    const uint32_t ncols_tile = MODE == 1 ? 128u : 256u;
    const uint32_t n_ct = (N + ncols_tile - 1) / ncols_tile;
    const uint32_t n_rt = uint32_t(a.n_tiles[0]);
    const uint32_t n_sn = (n_ct + kSuperN - 1) / kSuperN;
    const uint32_t xcd = blockIdx.x % 8u, jj = blockIdx.x / 8u;
    const uint32_t st = (jj / (kSuperM * kSuperN)) * 8u + xcd;
    const uint32_t within = jj % (kSuperM * kSuperN);
    const uint32_t row_tile = (st / n_sn) * kSuperM + within / kSuperN;
    const uint32_t col_tile = (st % n_sn) * kSuperN + within % kSuperN;
    if (row_tile >= n_rt || col_tile >= n_ct) return;
    TileInfo t;
    if (!tile_info(a, row_tile, t)) return;
    const uint32_t n_base = col_tile * ncols_tile;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int q = lane & 31;
    constexpr int kTile = kTM * kLdsPitch;

    // global -> register staging.  A: 8 lanes cover one row's 64 k; rows tid / 8 + 32 i.
    const uint16_t* a_base = MODE == 1 ? a.tokens : a.hbuf + size_t(uint32_t(t.row0)) * a.F;
    uint32_t a_off[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int32_t r = min(int32_t(tid >> 3) + 32 * i, t.rows - 1);
        if (MODE == 1) {
            const int32_t pr = a.sorted_pair[t.row0 + r];
            a_off[i] = (uint32_t(pr) / a.K) * a.H + 8 * (tid & 7);
        } else {
            a_off[i] = uint32_t(r) * a.F + 8 * (tid & 7);
        }
    }
    const int a_dst = (tid >> 3) * kLdsPitch + 8 * (tid & 7);          // + 32 i rows
    // B: two lane tiles of 4 consecutive columns x 8 k rows: k = 8 (tid / 64) + 32 u
    const uint32_t cg = tid & 63;
    const uint32_t bk = 8u * (tid >> 6);
    const uint16_t* b_src;
    int b_dst_row;
    {
        const size_t mat = size_t(a.H) * a.F;
        if (MODE == 1) {
            const uint32_t col = min(n_base + 4u * (cg & 31u), N - 4);
            b_src = a.slots13 + size_t(t.slot) * 2 * mat + (cg >= 32 ? mat : 0) + col;
            b_dst_row = int(cg >> 5) * 128 + int(cg & 31);
        } else {
            const uint32_t col = min(n_base + 4u * cg, N - 4);
            b_src = a.slots2 + size_t(t.slot) * mat + col;
            b_dst_row = int(cg);
        }
    }
    constexpr int b_dst_step = MODE == 1 ? 32 : 64;
    const int b_dst = kTile + b_dst_row * kLdsPitch + int(bk);

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int kfrag = 8 * (lane >> 5);
    const int a_frag = (wm * 128 + q) * kLdsPitch + kfrag;              // + 32 i rows
    // B tile j of this wavefront: MODE 2 rows 32 (4 wn + j) + q; MODE 1 rows 128 (j / 2) + 32 (2 wn + j % 2) + q
    const int b_frag = kTile + (MODE == 1 ? (2 * wn * 32 + q) : (4 * wn * 32 + q)) * kLdsPitch + kfrag;
    auto b_frag_off = [](int j) { return (MODE == 1 ? ((j >> 1) * 128 + (j & 1) * 32) : (j * 32)) * kLdsPitch; };

    u32x4 ga[8];
    u32x2 gb[2][8];
    const uint32_t n_steps = K / kTK;
    // item n of a step's 24 global loads: 0..7 the lane's A rows, 8..23 the 2 x 8 k rows of its B tiles
    auto gload_item = [&](uint32_t k0, int n) __attribute__((always_inline)) {
        if (n < 8) ga[n] = *reinterpret_cast<const u32x4*>(a_base + a_off[n] + k0);
        else gb[(n - 8) >> 3][(n - 8) & 7] =
                 *reinterpret_cast<const u32x2*>(b_src + size_t(k0 + bk + 32 * ((n - 8) >> 3) + ((n - 8) & 7)) * N);
    };
    // item n of a step's 16 LDS writes: 0..7 A rows, 8..15 column c of transposed B tile u
    auto lstore_item = [&](uint16_t* buf, int n) __attribute__((always_inline)) {
        if (n < 8) {
            *reinterpret_cast<u32x4*>(buf + a_dst + 32 * n * kLdsPitch) = ga[n];
        } else {
            const int u = (n - 8) >> 2, c = (n - 8) & 3;
            u32x4 v;
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
            v.x = __builtin_amdgcn_perm(gb[u][1][c >> 1], gb[u][0][c >> 1], sel);
            v.y = __builtin_amdgcn_perm(gb[u][3][c >> 1], gb[u][2][c >> 1], sel);
            v.z = __builtin_amdgcn_perm(gb[u][5][c >> 1], gb[u][4][c >> 1], sel);
            v.w = __builtin_amdgcn_perm(gb[u][7][c >> 1], gb[u][6][c >> 1], sel);
            *reinterpret_cast<u32x4*>(buf + b_dst + 32 * u + c * b_dst_step * kLdsPitch) = v;
        }
    };
    bf16x8 fa[2][4], fb[2][4];
    // item n of the 8 fragment reads of sub-step ks into register set `set`
    auto lfrag_item = [&](const uint16_t* buf, int ks, int set, int n) __attribute__((always_inline)) {
        if (n < 4) fa[set][n] = *reinterpret_cast<const bf16x8*>(buf + a_frag + 32 * n * kLdsPitch + ks * 16);
        else fb[set][n - 4] = *reinterpret_cast<const bf16x8*>(buf + b_frag + b_frag_off(n - 4) + ks * 16);
    };
    auto mfma_item = [&](int set, int n) __attribute__((always_inline)) {
        const int i = n >> 2, j = n & 3;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
    };

    // One k step.  STORE: refill the other buffer from the staging registers; LOAD: fetch step
    // s + 2 into them; NEXT: read the first fragments of the other buffer after the barrier.
    // Every memory instruction is issued between two MFMAs (the scheduling barriers keep that
    // order): the fragments of sub-step ks + 1 during sub-step ks, the 16 LDS writes during
    // sub-step 0, the 24 global loads during sub-steps 1 and 2.
    auto step = [&](const uint16_t* cur, uint16_t* nxt, uint32_t k_next, auto STORE, auto LOAD, auto NEXT) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 16; ++n) {                        // sub-step 0 (set 0)
            mfma_item(0, n);
            if (n < 8) lfrag_item(cur, 1, 1, n);
            if (STORE.value) lstore_item(nxt, n);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < 16; ++n) {                        // sub-step 1 (set 1)
            mfma_item(1, n);
            if (n < 8) lfrag_item(cur, 2, 0, n);
            if (LOAD.value && n >= 4) gload_item(k_next, n - 4);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < 16; ++n) {                        // sub-step 2 (set 0)
            mfma_item(0, n);
            if (n < 8) lfrag_item(cur, 3, 1, n);
            if (LOAD.value && n >= 4) gload_item(k_next, 12 + n - 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();                       // all reads of cur are in registers, nxt is complete
#pragma unroll
        for (int n = 0; n < 16; ++n) {                        // sub-step 3 (set 1)
            mfma_item(1, n);
            if (NEXT.value && n < 8) lfrag_item(nxt, 0, 0, n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;

#pragma unroll
    for (int n = 0; n < 24; ++n) gload_item(0, n);
#pragma unroll
    for (int n = 0; n < 16; ++n) lstore_item(lds, n);
    if (n_steps > 1) {
#pragma unroll
        for (int n = 0; n < 24; ++n) gload_item(kTK, n);
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 8; ++n) lfrag_item(lds, 0, 0, n);
    uint16_t* cur = lds;
    uint16_t* nxt = lds + 2 * kTile;
    uint32_t s = 0;
    for (; s + 2 < n_steps; ++s) {
        step(cur, nxt, (s + 2) * kTK, Yes{}, Yes{}, Yes{});
        uint16_t* tmp = cur; cur = nxt; nxt = tmp;
    }
    if (s + 1 < n_steps) {
        step(cur, nxt, 0, Yes{}, No{}, Yes{});
        uint16_t* tmp = cur; cur = nxt; nxt = tmp;
    }
    step(cur, nxt, 0, No{}, No{}, No{});

#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int32_t row = wm * 128 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (row >= t.rows) continue;
            if (MODE == 1) {
                const uint32_t col = n_base + 4u * q + 2u * wn;
                if (col >= N) continue;
                const uint32_t packed = pack_bf16_rne(swiglu(acc[i][0][r], acc[i][2][r]), swiglu(acc[i][1][r], acc[i][3][r]));
                *reinterpret_cast<uint32_t*>(a.hbuf + size_t(t.row0 + row) * a.F + col) = packed;
            } else {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const uint32_t col = n_base + 4u * (32 * half + q) + 2u * wn;
                    if (col >= N) continue;
                    *reinterpret_cast<float2*>(a.ybuf + size_t(t.row0 + row) * a.H + col) =
                        make_float2(acc[i][half][r], acc[i][half + 2][r]);
                }
            }
        }
}

// Third variant of the tiled kernel: both operands go from global memory straight into LDS
// (global_load_lds, 16 bytes per lane, no register staging, no LDS write instructions) and B stays
// row-major [k][n] there; its MFMA fragments are formed by the transposing LDS read
// (ds_read_b64_tr_b16: within 16 lanes, lane L receives element L % 4 of the four 8-byte groups that
// lanes L / 4, 4 + L / 4, 8 + L / 4, 12 + L / 4 point at).  Because an LDS-direct load fills 1 KiB
// contiguously (lane l at +16 l), rows cannot be padded; bank conflicts are avoided by choosing
// which global piece each lane fetches: A rows (128 bytes = 8 pieces) hold piece p ^ ((row >> 1) & 7)
// at position p; B rows (512 bytes = 8 units of 32 columns) hold unit u ^ (k & 3) at position u.
// LDS: [A stage 0 | A stage 1 | B stage 0 | B stage 1 | B stage 2], 32 KiB each = all 160 KiB.  Same
// eight wavefronts, wave tiles and sub-step schedule as gemm_tiled_kernel.  (Tiles of 128 x 128: B rows of 256 bytes = 4 units,
// stages of 16 KiB, 80 KiB in all.)
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
// Measurement aid, compile time only (python -m paper_2604_02715_amd.build -DFLUXMOE_D2L_PROBE=<bits>): parts of
// gemm_d2l_kernel's k loop left out to see what each costs.  The results are wrong with any bit set; every
// access that remains is one the full kernel makes too.  1: fragments are read from LDS once per tile only;
// 2: no A loads after the prologue; 4: no B loads after the prologue; 8: no waits for loads inside the loop
// (one wait after it); 16: every B load fetches the tile's first k block (stays cache resident).
#ifndef FLUXMOE_D2L_PROBE
#define FLUXMOE_D2L_PROBE 0
#endif

constexpr uint32_t kTailBlock = 256 * 256;       // floats of a tile's partial sums

// y of the last round's tiles += their other parts of K, in the order of k.  A workgroup has 16 rows of a tile.  Bound by its launch (5 us where
// nothing was split) and by the parts' bytes, 60 MB at most, still in the caches: 8 us on 8 experts of H 4096, 4096 tokens, top-2, three
// parts of two super-tiles.
__global__ __launch_bounds__(256) void last_round_kernel(FfnArgs a) {
    const uint32_t n_rt = uint32_t(a.n_tiles[0]), n_ct = (a.H + 255) / 256, n_sn = (n_ct + 7) / 8;
    const LastRound last = last_round((n_rt + 3) / 4 * n_sn);
    const uint32_t st = last.first + blockIdx.z, within = blockIdx.y;
    const uint32_t row_tile = st / n_sn * 4 + within / 8, col_tile = st % n_sn * 8 + within % 8;
    TileInfo t;
    if (last.parts == 1 || row_tile >= n_rt || col_tile >= n_ct || !tile_info(a, row_tile, t)) return;
    const uint32_t col = 4u * (threadIdx.x & 63u);
    if (col_tile * 256 + col >= a.H) return;
    for (int32_t row = int32_t(blockIdx.x * 16 + (threadIdx.x >> 6)); row < min(t.rows, int32_t(blockIdx.x * 16 + 16)); row += 4) {
        float4* const y = reinterpret_cast<float4*>(a.ybuf + (size_t(t.row0) + uint32_t(row)) * a.H + col_tile * 256 + col);
        float4 s = *y;
        const float* part = a.tail + (size_t(blockIdx.z) * (last.parts - 1) * 32u + within) * kTailBlock + uint32_t(row) * 256u + col;
        for (uint32_t k = 1; k < last.parts; ++k, part += 32 * size_t(kTailBlock)) {
            const float4 v = *reinterpret_cast<const float4*>(part);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        *y = s;
    }
}

// WALK: a workgroup takes several tiles one after the other (see the tile loop at the end); without it the
// launch has one workgroup per tile number and the code for the upcoming tile falls away.
// MODE 1: h = SwiGLU(X W1, X W3).  MODE 2: y = h W2, K split ksplit ways.  MODE 3: the first product with K split
// up to ksplit1 ways, FP32 partial sums of gate and up instead of h (swiglu_reduce_kernel adds them up), or h if that is 1.
// TILE: rows and columns of a workgroup's tile.  256: one workgroup per CU (160 KiB of LDS).  128, with WAVES = 4 as 2 x 2
// of 64 x 64: two per CU, a quarter of the work per tile, for products whose 256 x 256 tiles leave most CUs without one.
// STREAM: the weight loads carry the non-temporal hint.
// RAGGED: K of either product may be any multiple of 8; the pieces of the last step that lie past its end come from zeros.
// ROWS: the tiles are taken row by row and not in super-tiles.  LAST: the last round may be split (a.tail); instances of its own, since
// the look-up costs the others registers.
template <int MODE, int WAVES, bool WALK, int TILE, bool STREAM = false, bool RAGGED = false, bool ROWS = false, bool LAST = false>
__global__ __launch_bounds__(WAVES * 64, TILE == 128 ? 2 : 1) void gemm_d2l_kernel(FfnArgs a) {
    static_assert(!LAST || (MODE == 2 && !WALK && WAVES == 8 && TILE == 256), "a second product with long K");
    constexpr bool kFirst = MODE != 2;                       // gate/up operands: rows gathered from the tokens, two weight matrices
    static_assert(MODE != 3 || !WALK, "the split first product has few tiles");
    // WAVES = 8: wavefronts 4 (rows) x 2 (columns), 64 x 128 each, two per SIMD.  WAVES = 4: 2 x 2,
    // 128 x 128 each (256 accumulator registers), one per SIMD: a third less LDS read traffic per MFMA.
    constexpr int kRowTiles = WAVES == 8 || TILE == 128 ? 2 : 4;   // 32-row MFMA tiles per wavefront
    constexpr int kColTiles = TILE == 256 ? 4 : 2;           // 32-column MFMA tiles per wavefront
    // Wavefront row wm of kWaveRows multiplies the 32-row groups wm, wm + kWaveRows, ... of the tile, so that the groups a tile
    // has rows for are spread over the SIMDs; the others are neither fetched nor multiplied (k_loop below).
    constexpr int kWaveRows = TILE / 32 / kRowTiles;
    constexpr int kStageBytes = TILE * 128;                  // one operand, one step: TILE rows (columns) x 64 k
    constexpr int kRowB = TILE * 2;                          // bytes of a k row of B
    constexpr int kDma = kStageBytes / 1024 / WAVES;         // 1 KiB loads per wavefront, operand and step
    constexpr int kMfma = kColTiles * kRowTiles;             // MFMAs per sub-step
    constexpr int kDmaEvery = kMfma / kDma;                  // MFMAs between two loads of a sub-step
    constexpr int kFrag = kRowTiles + 2 * kColTiles;         // fragment reads per sub-step
    constexpr uint32_t kHalfTile = TILE / 2;                 // gate columns of a tile of the first product, as many up columns
    static_assert(WAVES == 8 || WAVES == 4, "wavefront layouts");
    static_assert(TILE == 256 || (TILE == 128 && WAVES == 4 && !WALK), "tile sizes");
    extern __shared__ __align__(16) uint16_t lds[];
    const uint32_t K = kFirst ? a.H : a.F;
    const uint32_t N = kFirst ? a.F : a.H;
    const uint32_t ncols_tile = kFirst ? kHalfTile : uint32_t(TILE);
    const uint32_t n_ct = (N + ncols_tile - 1) / ncols_tile;
    const uint32_t n_rt = uint32_t(a.n_tiles[0]);
    // Super-tile of this launch: 32 tiles (one per CU of an XCD) as sm rows x sn columns, sn a power of two
    // chosen by the launcher so that the column tiles fill whole super-tiles where they can.
    const uint32_t sn_log2 = a.tiled_sn_log2, sn = 1u << sn_log2, sm = 32u >> sn_log2;
    const uint32_t n_sn = (n_ct + sn - 1) >> sn_log2;
    // Workgroups go to the 8 XCDs round robin, so (super-tile, K split) pair number p runs on XCD
    // p % 8: the splits of one super-tile land on different XCDs
    const uint32_t n_split = MODE == 2 ? a.ksplit : (MODE == 1 ? 1u : (TILE == 256 ? uint32_t(a.n_tiles[1]) : first_splits(a, n_rt)));
    // Super-tiles are taken in groups of tiled_group super-rows (the row tiles of about one expert): for
    // each column block of the group, its super-rows run next to each other in time on different XCDs,
    // so the expert's weights for that column block leave HBM once and the other XCDs find them in the
    // memory-side cache, while the group's activations stay there across the column blocks.
    // (The second product has two column blocks at most and measured no gain: it keeps super-row order.)
    const uint32_t group = a.tiled_group;
    const uint32_t per_group = group * n_sn;
    // Tile number L -> (row tile, column tile, K split); false when the number names no tile.  A workgroup
    // takes the numbers blockIdx.x, blockIdx.x + gridDim.x, ...; gridDim.x is a multiple of 256 (or covers
    // all numbers), so all of them lie on the XCD that runs this workgroup and at the same place of
    // successive super-tiles.
    const uint32_t total = a.tiled_total;
    const LastRound last = LAST ? last_round(((n_rt + sm - 1) / sm) * n_sn) : LastRound{0u, 1u};
    auto locate_unchecked = [&](uint32_t L, uint32_t& row_tile, uint32_t& col_tile, uint32_t& split) __attribute__((always_inline)) {
        const uint32_t xcd = L % 8u, jj = L / 8u;
        const uint32_t pair = (jj / 32u) * 8u + xcd;
        uint32_t st = pair / n_split;
        split = pair % n_split;
        if (last.parts > 1 && pair >= last.first) {
            st = last.first + (pair - last.first) / last.parts;
            split = (pair - last.first) % last.parts;
        }
        const uint32_t within = jj % 32u;
        if (ROWS) {                                          // an XCD's 32 tiles one after the other, row by row
            const uint32_t tile = st * 32u + within;
            row_tile = tile / n_ct;
            col_tile = tile % n_ct;
            return;
        }
        const uint32_t grp = st / per_group, in_grp = st % per_group;
        row_tile = (grp * group + in_grp % group) * sm + (within >> sn_log2);
        col_tile = (in_grp / group) * sn + (within & (sn - 1u));
    };
    auto locate = [&](uint32_t L, uint32_t& row_tile, uint32_t& col_tile, uint32_t& split) __attribute__((always_inline)) {
        locate_unchecked(L, row_tile, col_tile, split);
        return row_tile < n_rt && col_tile < n_ct;
    };
    // A tile number together with what locate() says about it (the divisions in there are done on the
    // vector unit and take a third of a microsecond: once per tile is enough).
    struct TileId { uint32_t L, row_tile, col_tile, split; };
    // first number >= L of this workgroup's sequence that names a tile (L >= total when there is none)
    auto first_tile_from = [&](uint32_t L) __attribute__((always_inline)) {
        TileId id{L, 0, 0, 0};
        if (!WALK) {
            if (!(id.L < total && locate(id.L, id.row_tile, id.col_tile, id.split))) id.L = total;
            return id;
        }
        while (id.L < total && !locate(id.L, id.row_tile, id.col_tile, id.split)) id.L += gridDim.x;
        return id;
    };
    // its record (one 16-byte load; numbers past the end read record 0, which exists)
    auto load_rec = [&](const TileId& id) __attribute__((always_inline)) {
        return a.tile_rec[id.L < total ? id.row_tile : 0u];
    };

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int a_rows = 8 * kDma * wave;                      // first row of A this wavefront fetches: none if the tile ends before it
    // The lane number as a value the compiler cannot trace back to threadIdx: what the per-tile set-up code
    // derives from it is then computed again for every tile instead of being held in registers across the
    // k loop, where registers are short.
    auto fresh_lane = [&]() __attribute__((always_inline)) {
        int x = tid;
        asm volatile("" : "+v"(x));
        return x & 63;
    };
    uint8_t* const lds_b8 = reinterpret_cast<uint8_t*>(lds);
    const size_t mat = size_t(a.H) * a.F;
    const uint32_t n_steps_all = RAGGED ? (K + kTK - 1) / kTK : K / kTK;

    // What a tile's loads need: the lane's byte offsets of its LDS-direct loads (kDma for A, kDma for B
    // per step) from bases that are uniform over the workgroup, the step range, where the results go.
    struct TileState {
        uint32_t a_off[kDma], b_off[kDma];   // until finish_state(): a_off = pair numbers of the lane's rows as loaded
                                             // (first product) or their rows in the tile (second), b_off unset
        const uint8_t* a_base;
        const uint8_t* b_base;
        int32_t rows, row0;
        uint32_t n_base, split, n_steps;
        uint32_t tail;                       // 1 + number of the last round's block of partial sums, 0: the sums go to y
        uint32_t k_left;                     // RAGGED: k from the tile's first to the end of K
        bool valid;
    };
    // rec: the tile's record, loaded earlier.  Issues the gather of the rows' pair numbers (first product);
    // finish_state() turns them into offsets where the tile's first loads are issued, so that nothing waits
    // for the gather in between.
    auto make_state = [&](const TileId& id, const int4& rec, TileState& s) __attribute__((always_inline)) {
        const uint32_t col_tile = id.col_tile, split = id.split;
        s.valid = id.L < total;
        s.rows = __builtin_amdgcn_readfirstlane(rec.z);
        s.row0 = __builtin_amdgcn_readfirstlane(rec.y);
        const int32_t slot = __builtin_amdgcn_readfirstlane(rec.w);
        s.valid = s.valid && s.rows > 0 && slot >= 0;
        if (!s.valid) { s.rows = 1; s.row0 = 0; }
        s.n_base = col_tile * ncols_tile;
        s.split = split;
        // (a super-tile of the last round: the host lets it be split where K has steps enough)
        const bool tail = last.parts > 1 && (id.L / 256u) * 8u >= last.first;
        const uint32_t n_parts = tail ? last.parts : n_split;
        if (LAST) s.tail = tail && split > 0 ? (id.L / 256u * 8u + id.L % 8u - last.first) / last.parts * (last.parts - 1) + split : 0u;
        // split K: this tile multiplies steps [step_lo, step_hi) of the K / 64
        // and writes its own FP32 partial, which combine_kernel or swiglu_reduce_kernel sums in split order
        const uint32_t step_lo = uint32_t(uint64_t(n_steps_all) * split / n_parts);
        const uint32_t step_hi = uint32_t(uint64_t(n_steps_all) * (split + 1) / n_parts);
        const uint32_t k_begin = step_lo * kTK;
        if (RAGGED) s.k_left = K - k_begin;
        s.n_steps = MODE == 1 ? 0u : step_hi - step_lo;        // >= 1: the host keeps the splits <= K / 64
        // rows of h are counted from the tile's first: offsets inside all of h would not fit 32 bits
        s.a_base = MODE == 1 ? nullptr
                             : reinterpret_cast<const uint8_t*>(MODE == 3 ? a.tokens : a.hbuf + size_t(uint32_t(s.row0)) * a.F) + size_t(k_begin) * 2;
        const int lane = fresh_lane();
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int r_lds = 8 * (wave * kDma + i) + (lane >> 3);                 // row of the A tile
            const int32_t r = min(r_lds, s.rows - 1);
            s.a_off[i] = kFirst ? uint32_t(a.sorted_pair[s.row0 + r]) : uint32_t(r);
        }
        const size_t slot_u = s.valid ? size_t(slot) : 0u;
        s.b_base = reinterpret_cast<const uint8_t*>(
            MODE == 1 ? a.slots13 + slot_u * 2 * mat : (MODE == 3 ? a.slots13 + slot_u * 2 * mat : a.slots2 + slot_u * mat) + size_t(k_begin) * N);
    };
    auto finish_state = [&](TileState& s) __attribute__((always_inline)) {
        const int lane = fresh_lane();
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int r_lds = 8 * (wave * kDma + i) + (lane >> 3);              // row of the A tile
            const int piece = (lane & 7) ^ ((r_lds >> 1) & 7);                  // global 16-byte piece held at position lane & 7
            const uint32_t row_elems = kFirst ? (s.a_off[i] / a.K) * a.H : s.a_off[i] * a.F;
            s.a_off[i] = 2u * (row_elems + 8u * piece);
        }
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int k_lds = (1024 / kRowB) * (wave * kDma + i) + lane / (kRowB / 16);   // k row of the B tile
            const int pp = lane & (kRowB / 16 - 1);                             // physical 16-byte piece in the row
            const int unit = (pp >> 2) ^ (k_lds & 3);                           // logical unit of 32 columns
            const uint32_t c = 32u * unit + 8u * (pp & 3);                      // column inside the tile
            uint32_t elems;
            if (kFirst) elems = (c >= kHalfTile ? uint32_t(mat) : 0u) + min(s.n_base + (c & (kHalfTile - 1u)), N - 8);
            else elems = min(s.n_base + c, N - 8);
            s.b_off[i] = 2u * (elems + uint32_t(k_lds) * N);
        }
    };
    // stage_off: 0 or kStageBytes, uniform.  The load is written as inline assembly on purpose: with
    // the compiler's builtin, every later LDS read waits for all outstanding LDS-direct loads
    // (it cannot see that they go to the other stage), which serialises the whole step.  Here the
    // only waits are the explicit ones before the barriers.
    const uint32_t lds_base = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
    // (M0 carries the LDS destination and is read when the instruction issues; it is a register the
    // compiler reserves, so its previous value is put back.)
    auto dma16 = [&](const uint8_t* gptr, uint32_t lds_addr) __attribute__((always_inline)) {
        uint32_t saved_m0;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "v"(gptr), "s"(lds_addr) : "memory");
    };
    auto dma16_nt = [&](const uint8_t* gptr, uint32_t lds_addr) __attribute__((always_inline)) {
        uint32_t saved_m0;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt\n\ts_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "v"(gptr), "s"(lds_addr) : "memory");
    };
    // a_stage_off / b_stage_off: byte offset of the destination stage inside the operand's region, uniform
    auto dma_a = [&](const TileState& s, uint32_t k0, int a_stage_off, int n) __attribute__((always_inline)) {
        // (MODE 1 does not split K: its A base and step count are the same for every tile)
        const uint8_t* base = MODE == 1 ? reinterpret_cast<const uint8_t*>(a.tokens) : s.a_base;
        const uint8_t* src = base + size_t(k0) * 2 + s.a_off[n];
        if (RAGGED && k0 + kTK > (MODE == 1 ? K : s.k_left)) {              // uniform
            const int lane = fresh_lane(), r_lds = 8 * (wave * kDma + n) + (lane >> 3);
            if (k0 + 8u * ((lane & 7) ^ ((r_lds >> 1) & 7)) >= (MODE == 1 ? K : s.k_left)) src = reinterpret_cast<const uint8_t*>(&g_zero_piece);
        }
        dma16(src, lds_base + a_stage_off + (wave * kDma + n) * 1024);
    };
    auto dma_b = [&](const TileState& s, uint32_t k0, int b_stage_off, int n) __attribute__((always_inline)) {
        const uint8_t* src = s.b_base + size_t((FLUXMOE_D2L_PROBE & 16) ? 0u : k0) * N * 2 + s.b_off[n];
        if (RAGGED && k0 + kTK > (MODE == 1 ? K : s.k_left)) {
            const int lane = fresh_lane();
            if (k0 + uint32_t((1024 / kRowB) * (wave * kDma + n) + lane / (kRowB / 16)) >= (MODE == 1 ? K : s.k_left)) src = reinterpret_cast<const uint8_t*>(&g_zero_piece);
        }
        if (STREAM) dma16_nt(src, lds_base + 2 * kStageBytes + b_stage_off + (wave * kDma + n) * 1024);
        else dma16(src, lds_base + 2 * kStageBytes + b_stage_off + (wave * kDma + n) * 1024);
    };
    auto steps_of = [&](const TileState& s) __attribute__((always_inline)) { return MODE == 1 ? n_steps_all : s.n_steps; };
    // a tile's first loads: A and B of steps 0 and 1 into stages 0 and 1 (B of step 2 is issued by step 0)
    auto prime = [&](const TileState& s) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < kDma; ++n) { if (a_rows < s.rows) dma_a(s, 0, 0, n); dma_b(s, 0, 0, n); }
        if (steps_of(s) > 1) {
#pragma unroll
            for (int n = 0; n < kDma; ++n) { if (a_rows < s.rows) dma_a(s, kTK, kStageBytes, n); dma_b(s, kTK, kStageBytes, n); }
        }
    };

    // ---- fragment addresses (bytes from the start of stage 0 of the operand's region); the k loop moves
    // them from stage to stage, so every tile starts from these values again
    int a_addr[kRowTiles][4];
    int b_addr[kColTiles];
    f32x16 acc[kRowTiles][kColTiles];
    int b_next_delta = kStageBytes;
    int a_own = 0, b_own = 0;                                // byte offsets of the current step's stages
    auto begin_tile = [&]() __attribute__((always_inline)) {
        const int lane = fresh_lane();
        const int q = lane & 31, h = lane >> 5;
        const int e = (lane & 15) >> 2, g = lane & 3, nh = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i) {
            const int R = 32 * (wm + kWaveRows * i) + q;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a_addr[i][ks] = R * 128 + 16 * ((2 * ks + h) ^ ((R >> 1) & 7));
        }
        // B fragment j of sub-step ks, read t: row 16 ks + 8 h + 4 t + e, unit u(j) ^ e, bytes 32 nh + 8 g
#pragma unroll
        for (int j = 0; j < kColTiles; ++j) {
            // the wavefront's columns as units: gate and up units of the same h columns, or kColTiles in a row
            const int unit = TILE == 128 ? (kFirst ? wn + 2 * j : 2 * wn + j) ^ e
                                         : (kFirst ? ((((2 * wn + (j & 1)) ^ e)) + 4 * (j >> 1)) : (4 * wn + (j ^ e)));
            b_addr[j] = 2 * kStageBytes + (8 * h + e) * kRowB + 64 * unit + 32 * nh + 8 * g;
        }
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int j = 0; j < kColTiles; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        b_next_delta = kStageBytes;
        a_own = 0;
        b_own = 0;
    };

    bf16x8 fa[2][kRowTiles];
    i16x4 fb_lo[2][kColTiles], fb_hi[2][kColTiles];
    // item n of the kFrag fragment reads of sub-step ks from `stage` into register set `set`: first the
    // A tiles, then the two halves (k 0..3 and 4..7 of the lane's 8) of the four B fragments
    // OTHER: read from the next step's stage instead of the one the address registers point at
    // (A: the other of two stages; B: b_next_delta bytes further in its ring of three)
    auto lfrag_item = [&](int other, int ks, int set, int n, int rows_act) __attribute__((always_inline)) {
        if (n < kRowTiles) {
            if (n >= rows_act) return;
            fa[set][n] = *reinterpret_cast<const bf16x8*>(lds_b8 + (a_addr[n][ks] ^ (other ? kStageBytes : 0)));
        } else {
            const int j = (n - kRowTiles) >> 1, tt = (n - kRowTiles) & 1;
            const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_i16x4*)(lds_b8 + ((b_addr[j] + (other ? b_next_delta : 0)) + ks * 16 * kRowB + tt * 4 * kRowB)));
            if (tt == 0) fb_lo[set][j] = v; else fb_hi[set][j] = v;
        }
    };
    typedef short i16x8 __attribute__((ext_vector_type(8)));
    auto mfma_item = [&](int set, int n) __attribute__((always_inline)) {
        const int i = n / kColTiles, j = n % kColTiles;
        const i16x8 full = __builtin_shufflevector(fb_lo[set][j], fb_hi[set][j], 0, 1, 2, 3, 4, 5, 6, 7);
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], __builtin_bit_cast(bf16x8, full), acc[i][j], 0, 0, 0);
    };

    // Step s multiplies A stage s % 2 and B stage s % 3.  After its barrier nobody reads those
    // stages any more, so sub-step 3 issues the A loads of step s + 2 into the same A stage and
    // sub-step 0 of the next step issues the B loads of step s + 3 into the same B stage: B, whose
    // first reader in an XCD goes to HBM, is fetched two steps ahead, A (mostly L2 hits) one.
    // Loads return in order, so waiting until at most 4 are outstanding before the barrier of
    // step s leaves only the B loads of step s + 2 in flight.
    // LOAD_B: B of step s + 2 (issued in sub-step 0); LOAD_A: A of step s + 2 (after the barrier);
    // NEXT: another step follows.  After the barrier of a tile's last step all five stages are free: that
    // step issues the first loads of the workgroup's next tile (`upcoming`, if it has one) behind its last
    // MFMAs, and they travel while the epilogue runs.
    auto step = [&](const TileState& cur, TileState& upcoming, uint32_t k0, auto LOAD_B, auto LOAD_A, auto NEXT, auto ACT) __attribute__((always_inline)) {
        const int b_plus2 = b_own >= kStageBytes ? b_own - kStageBytes : b_own + 2 * kStageBytes;   // stage of step s + 2
        // one sub-step: the MFMAs of register set `set`, between them the fragment reads of sub-step
        // next_ks into the other set (other = 1: from the next step's stages) and this step's share of loads
        auto sub = [&](int set, int other, int next_ks, auto READ, auto DMA_B, auto DMA_A) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < kMfma; ++n) {
                if (n < kColTiles * ACT.value) mfma_item(set, n);
                if (READ.value && ACT.value && n < kFrag && !(FLUXMOE_D2L_PROBE & 1)) lfrag_item(other, next_ks, set ^ 1, n, ACT.value);
                if (DMA_B.value && n % kDmaEvery == kDmaEvery - 1 && !(FLUXMOE_D2L_PROBE & 4)) dma_b(cur, k0 + 2 * kTK, b_plus2, n / kDmaEvery);
                if (DMA_A.value && n % kDmaEvery == kDmaEvery - 1 && a_rows < cur.rows && !(FLUXMOE_D2L_PROBE & 2)) dma_a(cur, k0 + 2 * kTK, a_own, n / kDmaEvery);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (READ.value && ACT.value && !(FLUXMOE_D2L_PROBE & 1)) {
#pragma unroll
                for (int n = kMfma; n < kFrag; ++n) lfrag_item(other, next_ks, set ^ 1, n, ACT.value);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        using T = std::integral_constant<bool, true>;
        using F = std::integral_constant<bool, false>;
        sub(0, 0, 1, T{}, LOAD_B, F{});                       // sub-step 0
        sub(1, 0, 2, T{}, F{}, F{});                          // sub-step 1
        sub(0, 0, 3, T{}, F{}, F{});                          // sub-step 2
        if (!(FLUXMOE_D2L_PROBE & 8)) {
            if (LOAD_B.value) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kDma) : "memory");   // all but this step's own B loads have landed
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();                                      // all reads of this step's stages are in registers
        sub(1, 1, 0, NEXT, F{}, LOAD_A);                      // sub-step 3
        if (WALK && !NEXT.value && upcoming.valid) { finish_state(upcoming); prime(upcoming); }
        // advance to the next step's stages
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a_addr[i][ks] ^= kStageBytes;
#pragma unroll
        for (int j = 0; j < kColTiles; ++j) b_addr[j] += b_next_delta;
        a_own ^= kStageBytes;
        b_own = b_own == 2 * kStageBytes ? 0 : b_own + kStageBytes;
        b_next_delta = b_own == 2 * kStageBytes ? -2 * kStageBytes : kStageBytes;
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;

    auto epilogue = [&](const TileState& c) __attribute__((always_inline)) {
    const int lane = fresh_lane();
    const int q = lane & 31, h = lane >> 5;
    // epilogue.  D layout of the 32x32 MFMA: column q = lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4;
    // fragment j of this wavefront holds tile columns 128 wn + 32 j + q (MODE 2) or, in MODE 1,
    // gate (j = 0, 1) and up (j = 2, 3) of h columns 64 wn + 32 (j & 1) + q
    if (MODE == 1 || (MODE == 3 && n_split == 1)) {
        // a lane holds one h column; neighbouring lanes swap values (DPP) so that even lanes store
        // columns (q, q + 1) of an even row and odd lanes columns (q - 1, q) of the next row: 4-byte
        // stores instead of 2-byte ones
        // v_perm_b32(other, own, sel): selector bytes 0..3 pick from own, 4..7 from other
        const uint32_t pair_sel = (q & 1) ? 0x03020706u : 0x05040100u;
        // one 64-bit address per stored row; the two column groups of a row lie 64 bytes apart
        const uint32_t col0 = c.n_base + (TILE / 4u) * wn + (q & ~1);
        uint16_t* const hlane = a.hbuf + size_t(c.row0) * a.F + col0;
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const int32_t row = 32 * (wm + kWaveRows * i) + (r >> 2) * 8 + h * 4 + (r & 3) + (q & 1);
                uint16_t* const hrow = hlane + size_t(uint32_t(row)) * a.F;
#pragma unroll
                for (int j = 0; j < kColTiles / 2; ++j) {
                    // own = (row r, row r + 1) of this lane's column; the neighbouring lane's pair comes by DPP
                    // (quad_perm 1,0,3,2); an even lane keeps both lanes' row-r values, an odd lane both
                    // lanes' row-(r + 1) values, lower column first: one byte permute with a per-lane selector
                    const uint32_t own = pack_bf16_rne(swiglu(acc[i][j][r], acc[i][j + kColTiles / 2][r]),
                                                       swiglu(acc[i][j][r + 1], acc[i][j + kColTiles / 2][r + 1]));
                    const uint32_t other = uint32_t(__builtin_amdgcn_update_dpp(0, int(own), 0xB1, 0xF, 0xF, true));
                    const uint32_t packed = __builtin_amdgcn_perm(other, own, pair_sel);
                    if (row < c.rows && col0 + 32u * j < N)
                        *reinterpret_cast<uint32_t*>(hrow + 32 * j) = packed;
                }
            }
    } else if (MODE == 3) {
        // partial sums: row r of split s at [s][r][gate | up][F]
        constexpr int kGate = kColTiles / 2;                 // column tiles of each matrix
        const uint32_t col0 = c.n_base + (TILE / 4u) * wn + q;
        float* const plane = a.ybuf + (size_t(c.split) * a.pairs_cap + size_t(c.row0)) * 2 * a.F + col0;
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int32_t row = 32 * (wm + kWaveRows * i) + (r >> 2) * 8 + h * 4 + (r & 3);
                if (row >= c.rows) continue;
                float* const prow = plane + size_t(uint32_t(row)) * 2 * a.F;
#pragma unroll
                for (int j = 0; j < kColTiles; ++j) {
                    if (col0 + 32u * (j % kGate) >= N) continue;
                    prow[(j / kGate) * a.F + 32 * (j % kGate)] = acc[i][j][r];
                }
            }
    } else {
        // one 64-bit address per stored row; the four column groups of a row lie 128 bytes apart
        // (or, a.direct, the output: one split, row r is token r with gate 1)
        const uint32_t col0 = c.n_base + (TILE / 2u) * wn + q;
        const bool direct = (WAVES == 8 || TILE == 128) && a.direct;
        float* ylane = direct ? a.out + size_t(c.row0) * a.H + col0 : a.ybuf + (size_t(c.split) * a.pairs_cap + size_t(c.row0)) * a.H + col0;
        uint32_t pitch = a.H;
        if (LAST && last.parts > 1) {
            if (c.tail) {
                ylane = a.tail + (size_t(c.tail - 1) * 32u + blockIdx.x / 8u % 32u) * kTailBlock + (col0 - c.n_base);
                pitch = 256;
            } else {
                ylane = a.ybuf + size_t(c.row0) * a.H + col0;
            }
        }
        if (direct && (a.flags & 1u)) {
#pragma unroll
            for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int32_t row = min(32 * (wm + kWaveRows * i) + (r >> 2) * 8 + h * 4 + (r & 3), c.rows - 1);
#pragma unroll
                    for (int j = 0; j < kColTiles; ++j)
                        if (col0 + 32u * j < N) acc[i][j][r] += ylane[size_t(uint32_t(row)) * a.H + 32 * j];
                }
        }
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int32_t row = 32 * (wm + kWaveRows * i) + (r >> 2) * 8 + h * 4 + (r & 3);
                if (row >= c.rows) continue;
                float* const yrow = ylane + size_t(uint32_t(row)) * pitch;
#pragma unroll
                for (int j = 0; j < kColTiles; ++j) {
                    if (col0 + 32u * j >= N) continue;
                    yrow[32 * j] = acc[i][j][r];
                }
            }
    }
    };

    // ACT: how many of the wavefront's row groups the tile has rows for (all, half, or none: then it takes part in the loads
    // and barriers only).  160 experts of H 5120 F 1536 with 205 rows each: 2081 -> 2052 us a call;
    // 8 of H 4096 F 14336, 1024 rows each, and a pass in waves over 128 of H 2048 F 512: no change beyond the runs' spread.
    auto k_loop = [&](const TileState& cur, TileState& upcoming, auto ACT) __attribute__((always_inline)) {
        if (ACT.value) {
#pragma unroll
            for (int n = 0; n < kFrag; ++n) lfrag_item(0, 0, 0, n, ACT.value);
            if (FLUXMOE_D2L_PROBE & 1) {
#pragma unroll
                for (int n = 0; n < kFrag; ++n) lfrag_item(0, 1, 1, n, ACT.value);
            }
        }
        uint32_t s = 0;
        const uint32_t n_steps = steps_of(cur);
        for (; s + 2 < n_steps; ++s) step(cur, upcoming, s * kTK, Yes{}, Yes{}, Yes{}, ACT);
        if (s + 1 < n_steps) step(cur, upcoming, s * kTK, No{}, No{}, Yes{}, ACT);
        step(cur, upcoming, 0, No{}, No{}, No{}, ACT);
    };

    // ---- the workgroup's tiles.  Three of them are in the pipeline: `cur` is multiplied; `nxt` has had its
    // record read and its row gather issued (the values are first touched when its loads are issued at the
    // end of cur's k loop); the record of the one after is on its way.
    // (the record of the workgroup's own number is requested before anything looks at the tile count, which
    // is itself a load: the two travel together instead of one after the other)
    int4 rec_own;
    {
        TileId own{blockIdx.x, 0, 0, 0};
        uint32_t c, sp;
        locate_unchecked(own.L, own.row_tile, c, sp);
        rec_own = a.tile_rec[min(own.row_tile, a.tiles_cap - 1u)];
    }
    const TileId none{total, 0, 0, 0};
    TileId id_cur = first_tile_from(blockIdx.x);
    TileId id_nxt = WALK ? first_tile_from(id_cur.L < total ? id_cur.L + gridDim.x : total) : none;
    int4 rec_nxt = WALK ? load_rec(id_nxt) : make_int4(0, 0, 0, -1);
    TileState cur, nxt;
    make_state(id_cur, id_cur.L == blockIdx.x ? rec_own : load_rec(id_cur), cur);
    nxt.valid = false;
    bool primed = false;                                     // cur's first loads were issued by the tile before it
    while (id_cur.L < total) {
        TileId id_after = none;
        int4 rec_after = make_int4(0, 0, 0, -1);
        if (WALK) {
            id_after = first_tile_from(id_nxt.L < total ? id_nxt.L + gridDim.x : total);
            rec_after = load_rec(id_after);                 // the one load between cur's first loads and the wait below
        }
        // The upcoming tile's row gather is issued here, a whole k loop before its values are needed: issued
        // later (between the steady steps and the last two) the in-order wait of the next step stalls on it
        // (measured: 10 % of the first product's time).
        if (WALK) make_state(id_nxt, rec_nxt, nxt);
        if (cur.valid) {
            begin_tile();
            if (!primed) {
                finish_state(cur);
                prime(cur);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            } else {
                // loads return in order: cur's first loads are older than the record load and the gather just issued
                asm volatile("s_waitcnt vmcnt(%0)" :: "n"(MODE == 1 ? 1 + kDma : 1) : "memory");
            }
            __syncthreads();
            if (32 * (wm + kWaveRows * (kRowTiles / 2)) < cur.rows) k_loop(cur, nxt, std::integral_constant<int, kRowTiles>{});
            else if (32 * wm < cur.rows) k_loop(cur, nxt, std::integral_constant<int, kRowTiles / 2>{});
            else k_loop(cur, nxt, std::integral_constant<int, 0>{});
            if (FLUXMOE_D2L_PROBE & 8) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); __syncthreads(); }
            epilogue(cur);
        }
        if (!WALK) break;
        primed = cur.valid && nxt.valid;
        cur = nxt;
        id_cur = id_nxt;
        id_nxt = id_after;
        rec_nxt = rec_after;
    }
}

// out[t][:] (+)= sum_k gate * sum_split y
// STREAM: y is read and the output written with the non-temporal hint (combine_streams).
// IDENTITY: the shared expert, row t is token t with gate 1.
template <uint32_t kGroup, bool STREAM, bool IDENTITY = false>
__global__ __launch_bounds__(256) void combine_kernel(FfnArgs a) {
    const uint32_t tok = blockIdx.y;
    const uint32_t h = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (h >= a.H) return;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    float* o = a.out + size_t(tok) * a.H + h;
    if (a.flags & 1u) s = *reinterpret_cast<const float4*>(o);
    // kGroup pairs of the token at a time (the launcher takes the smallest of 2, 4, 8, 16 that covers top-k,
    // 16 beyond): their positions and gates are fetched together, then their rows of y, so that the loads
    // overlap instead of following each other pair by pair.  A skipped pair, and a place of the group past
    // top-k, reads row 0 (a cache hit) and adds nothing; the sums run over the splits and then over k, in that
    // order, whatever the group size.
    for (uint32_t k0 = 0; k0 < a.K; k0 += kGroup) {
        int32_t pos[kGroup];
        float gate[kGroup];
        // a.identity is never set where it is asked here; the question keeps the compiler from spilling gates as they arrive, with a wait
        // for each (4096 tokens, an eighth of 512 experts of H 2048, top-10: 34.6 us, without it 37.1; positions and gates in loops of their
        // own 35.2)
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) {
            const bool in = k0 + j < a.K;
            pos[j] = IDENTITY ? int32_t(tok) : (in ? a.pair_pos[tok * a.K + k0 + j] : -1);
            gate[j] = in ? (IDENTITY || a.identity ? 1.f : a.topk_w[tok * a.K + k0 + j]) : 0.f;
        }
        float4 y[kGroup];
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) y[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint32_t sp = 0; sp < a.ksplit; ++sp) {
            float4 v[kGroup];
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                const float* at = a.ybuf + (size_t(sp) * a.pairs_cap + uint32_t(max(pos[j], 0))) * a.H + h;
                if (STREAM) {
                    const uint4 w = load_stream16(at);
                    v[j] = make_float4(__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w));
                } else {
                    v[j] = *reinterpret_cast<const float4*>(at);
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                if (pos[j] >= 0) { y[j].x += v[j].x; y[j].y += v[j].y; y[j].z += v[j].z; y[j].w += v[j].w; }
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) {
            if (pos[j] >= 0) { s.x += gate[j] * y[j].x; s.y += gate[j] * y[j].y; s.z += gate[j] * y[j].z; s.w += gate[j] * y[j].w; }
        }
    }
    if (STREAM) store_stream16(o, make_uint4(__float_as_uint(s.x), __float_as_uint(s.y), __float_as_uint(s.z), __float_as_uint(s.w)));
    else *reinterpret_cast<float4*>(o) = s;
}

// Measurement aid: nothing but independent 32x32x16 BF16 MFMAs (16 accumulators per wavefront, one
// wavefront per SIMD) on operands read once from `in`: what the matrix cores sustain on this chip
// for a given operand content, with no memory traffic in the loop.
__global__ __launch_bounds__(256) void mfma_probe_kernel(const u32x4* in, float* out, uint32_t iters) {
    f32x16 acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    union { u32x4 u; bf16x8 v; } fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        fa[i].u = in[(threadIdx.x * 8 + i) & 4095];
        fb[i].u = in[(threadIdx.x * 8 + 4 + i + blockIdx.x) & 4095];
    }
    for (uint32_t it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i * 4 + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].v, fb[j].v, acc[i * 4 + j], 0, 0, 0);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += acc[i][r];
    out[blockIdx.x * 256 + threadIdx.x] = sum;
}

}  // namespace

hipError_t launch_mfma_probe(const void* operands, float* out, uint32_t n_workgroups, uint32_t iters,
                             hipStream_t stream) {
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(n_workgroups), dim3(256), 0, stream,
                       static_cast<const u32x4*>(operands), out, iters);
    return hipGetLastError();
}

hipError_t launch_ffn(const FfnCall& call, int n_cus, hipStream_t stream, hipEvent_t done, hipEvent_t routed, bool attach_routed,
                      SpanHook hook, void* user) {
    (void)n_cus;
    if (call.T == 0) return hipSuccess;
    if (call.identity && (done || routed)) return hipErrorInvalidValue;      // the shared expert's calls have no event to complete
    FfnArgs a = call;
    auto mark = [&](int kind, int begin) { if (hook) hook(user, kind, begin, stream); };
    const size_t sh = (3 * size_t(a.E) + 1024) * sizeof(int32_t);
    // strip kernels, few pairs: the first product's workgroups do the grouping
    const bool routes_itself = call.few != 0;
    if (routes_itself && (a.identity || a.tiled || a.m_tile < kRoutedPairs || uint64_t(a.T) * a.K > kRoutedPairs)) return hipErrorInvalidValue;
    const hipEvent_t with_routing = attach_routed ? routed : nullptr;
    auto record_routed = [&]() { return routed && !attach_routed ? hipEventRecord(routed, stream) : hipSuccess; };
    // (F > 2048: the second product does not walk)
    if (a.identity || !a.tiled || a.m_tile != 256 || call.tiled_waves != 2 || a.ksplit != 1 || a.F <= 2048 || !last_round_pays(uint64_t(a.T) * a.K, call.mapped, a.E, a.H, a.F))
        a.tail = nullptr;
    const bool chooses = a.tiled && a.m_tile == 256 && a.ksplit1 > 1;
    if (routes_itself) a.split_tiles = ~0u;                         // few rows, and the lists are not there yet: as planned
    const bool grouping = a.identity ? !a.ring1 : !routes_itself;
    if (grouping) mark(1, 1);
    if (!grouping) {
    } else if (a.identity) {
        hipLaunchKernelGGL(route_identity_kernel, dim3((std::max(a.T, a.tiles_cap) + 255) / 256), dim3(256), 0, stream, a);
    } else if (a.n_chunks) {
        hipLaunchKernelGGL(route_count_kernel, dim3(a.n_chunks), dim3(1024), size_t(a.E) * sizeof(int32_t), stream, a);
        if (chooses) hipLaunchKernelGGL((route_sort_kernel<true, true>), dim3(1), dim3(1024), sh, stream, a);
        else hipLaunchKernelGGL((route_sort_kernel<true, false>), dim3(1), dim3(1024), sh, stream, a);
        launch_done(route_scatter_kernel, dim3(a.n_chunks), dim3(1024), size_t(a.E) * sizeof(int32_t), stream, with_routing, a);
    } else {
        launch_done(chooses ? route_sort_kernel<false, true> : route_sort_kernel<false, false>, dim3(1), dim3(1024), sh, stream, with_routing, a);
    }
    if (a.tail) hipLaunchKernelGGL(route_order_kernel, dim3(a.E), dim3(1024), 0, stream, a);
    if (grouping) {
        mark(1, 0);
        if (hipError_t e = record_routed(); e != hipSuccess) return e;
    }
    auto launch_combine = [&](dim3 grid) {
        const bool streams = combine_streams(uint64_t(a.ksplit) * a.T * a.K * a.H * sizeof(float), call.mapped, a.E);
        auto launch = [&](auto plain, auto stream_y) { launch_done(streams ? stream_y : plain, grid, dim3(256), 0, stream, done, a); };
        if (a.identity) launch(combine_kernel<1, false, true>, combine_kernel<1, true, true>);
        else if (a.K <= 2) launch(combine_kernel<2, false>, combine_kernel<2, true>);
        else if (a.K <= 4) launch(combine_kernel<4, false>, combine_kernel<4, true>);
        else if (a.K <= 8) launch(combine_kernel<8, false>, combine_kernel<8, true>);
        else launch(combine_kernel<16, false>, combine_kernel<16, true>);
    };
    auto launch_reduce = [&]() {
        const uint64_t n = uint64_t(a.pairs_cap) * (a.F / 8);
        if (a.ksplit1 > 1) hipLaunchKernelGGL(swiglu_reduce_kernel, dim3(uint32_t((n + 255) / 256)), dim3(256), 0, stream, a);
    };
    if (a.ksplit1 == 0 || (a.ksplit1 > 1 && a.ksplit1 > a.H / kTK)) return hipErrorInvalidValue;
    const uint32_t strips1 = (a.F + kStrip - 1) / kStrip;
    const uint32_t strips2 = (a.H + kStrip - 1) / kStrip;
    if (a.halves && (a.tiled || a.m_tile != 128)) return hipErrorInvalidValue;
    const uint32_t cols1 = a.halves ? strips1 : (strips1 + 1) / 2;
    const dim3 g1 = a.g1_xcd && !routes_itself ? dim3((a.tiles_cap * a.ksplit1 + 7) / 8 * 8 * cols1, 1, 1) : dim3(cols1, a.ksplit1, a.tiles_cap);
    const dim3 g2(((a.tiles_cap * a.ksplit + 7) / 8 * 8) * ((strips2 + 3) / 4), 1, 1);
    a.direct = a.identity && a.ksplit == 1 && (a.ring2 || (a.tiled && call.tiled_waves == 2));
    if (a.ring1) {
        mark(2, 1);
        if (hipError_t e = launch_ring(a, 1, stream); e != hipSuccess) return e;
        launch_reduce();
        mark(2, 0);
        mark(3, 1);
        if (hipError_t e = launch_ring(a, 2, stream); e != hipSuccess) return e;
        mark(3, 0);
        if (a.direct) return hipSuccess;
        mark(4, 1);
        launch_combine(dim3((a.H / 4 + 255) / 256, a.T, 1));
        mark(4, 0);
        return hipGetLastError();
    }
    const bool stream_b = !a.identity && !(a.flags & 2u) && weights_stream(a.E, a.H, a.F, uint64_t(a.T) * a.K, a.m_tile);
    if (a.tiled) {
        const size_t lds_bytes = 4 * size_t(kTM) * kLdsPitch * sizeof(uint16_t);
        const bool four = call.tiled_waves == 4;
        const bool small = a.m_tile == 128;                         // LDS-direct loads, tiles of 128 x 128
        const bool d2l4 = call.tiled_waves == 1;                       // LDS-direct loads, four wavefronts of 128 x 128
        const bool d2l = call.tiled_waves == 2 || d2l4;
        if (!d2l && a.ksplit != 1) return hipErrorInvalidValue;     // only the LDS-direct kernels split K
        if (call.tiled_waves != 2 && (a.ksplit1 != 1 || small)) return hipErrorInvalidValue;
        if (!small && a.m_tile != 256) return hipErrorInvalidValue;
        if (a.ksplit == 0 || a.ksplit > std::max(1u, a.F / kTK)) return hipErrorInvalidValue;
        const bool ragged = a.H % kTK != 0 || a.F % kTK != 0;
        if (ragged && (call.tiled_waves != 2 || small)) return hipErrorInvalidValue;        // only the eight-wavefront LDS-direct kernels take a partial step
        static bool attr_set = false;
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled_kernel<1>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled_kernel<2>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled4_kernel<1>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled4_kernel<2>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            for (const void* f : {reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256, true, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256, true, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, true, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<3, 8, false, 256, false, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256, false, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256, true, false, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256, false, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256, true, false, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, false, false, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, true, false, false, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, false, true, false, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, true, true, false, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 8, true, 256, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, true, 256, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 8, false, 256, true>)}) {
                e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
                if (e != hipSuccess) return e;
            }
            for (const void* f : {reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 4, false, 128>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 4, false, 128>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 4, false, 128, true>), reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 4, false, 128, true>),
                                  reinterpret_cast<const void*>(&gemm_d2l_kernel<3, 4, false, 128>)}) {
                e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 81920);
                if (e != hipSuccess) return e;
            }
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<3, 8, false, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<1, 4, false, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_d2l_kernel<2, 4, false, 256>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
        auto pick = [&](auto plain, auto streams, auto partial, auto both) { return ragged ? (stream_b ? both : partial) : (stream_b ? streams : plain); };
        mark(2, 1);
        // register-staged kernels: super-tiles of 4 x 8 tiles, super-row order
        auto grid_for = [&](uint32_t n_ct) {
            const uint32_t n_sm = (a.tiles_cap + kSuperM - 1) / kSuperM;
            const uint32_t n_sn = (n_ct + kSuperN - 1) / kSuperN;
            const uint32_t supers = (n_sm * n_sn + 7) / 8 * 8;                // whole rounds over the 8 XCDs
            return dim3(supers * kSuperM * kSuperN, 1, 1);
        };
        // LDS-direct kernels.  A launch whose workgroups walk through the tiles takes as the super-tile's
        // column count the power of two (8, 4, 16, 2 in that order of preference) that leaves the fewest empty
        // places in the last column block: a workgroup whose place is empty there has nothing to do while the
        // others work (H 5120 / F 1536, 12 column tiles of the first product: 4 x 8 super-tiles 10.2 ms,
        // 8 x 4 8.1 ms at 2048 rows per expert).  With one workgroup per tile the dispatcher fills the holes
        // and 4 x 8 measured best.  A group is about one expert's super-rows (first product only; at most 8,
        // one per XCD).  Sets the launch's fields in `a`.
        const uint64_t pairs_all = uint64_t(a.T) * a.K;
        const uint64_t avg_rows = pairs_all / std::max<uint64_t>(1, std::min<uint64_t>(a.E, pairs_all));
        bool in_rows = false;                                       // of the launch that d2l_all was asked for last
        auto d2l_all = [&](uint32_t n_ct, uint32_t n_split, bool grouped, bool walk) {
            in_rows = walk && !ragged && tiles_by_rows(n_ct, avg_rows, grouped ? call.tiled_group : 0u);
            if (in_rows) {
                a.tiled_sn_log2 = 3;
                a.tiled_group = 1;
                return dim3((a.tiles_cap * n_ct + 255) / 256 * 256, 1, 1);
            }
            uint32_t best_log2 = 3, best_pad = ~0u;
            for (uint32_t lg : {3u, 2u, 4u, 1u}) {
                if (!walk && lg != 3u) continue;
                const uint32_t pad = ((n_ct + (1u << lg) - 1) >> lg << lg) - n_ct;
                if (pad < best_pad) { best_pad = pad; best_log2 = lg; }
            }
            a.tiled_sn_log2 = best_log2;
            const uint32_t sm = 32u >> best_log2;
            const uint64_t per_super_row = uint64_t(a.m_tile) * sm;
            a.tiled_group = !grouped ? 1u : uint32_t(std::min<uint64_t>(8, std::max<uint64_t>(1,
                call.tiled_group ? call.tiled_group : (avg_rows + per_super_row / 2) / per_super_row)));
            const uint32_t n_sm = ((a.tiles_cap + sm - 1) / sm + a.tiled_group - 1) / a.tiled_group * a.tiled_group;
            const uint32_t n_sn = (n_ct + (1u << best_log2) - 1) >> best_log2;
            const uint32_t supers = (n_sm * n_sn * n_split + 7) / 8 * 8;      // whole rounds over the 8 XCDs
            return dim3(supers * 32u, 1, 1);
        };
        // LDS-direct kernels: the launch covers `tiled_total` tile numbers; a workgroup walks through the numbers
        // blockIdx.x, + gridDim.x, ... and overlaps a tile's epilogue with the next one's first loads.  One
        // workgroup fits on a CU, so the first product runs tiled_persist x 256 workgroups (a multiple of 256
        // keeps a workgroup's numbers on its XCD); with tiled_persist = 0, and for the second product where its tiles are
        // long, one workgroup per number.  Measured on the first product of H 5120 / F 1536, 2048 rows per expert: 7 % (its
        // tiles need a row gather first); on H 4096 / F 14336 under 1 %.  The fixed hand-out loses when the last column block of
        // a super-tile row is partly empty (workgroups with no tile there idle), hence the choice of shapes above.
        auto d2l_grid = [&](const dim3& all, bool walk) {
            a.tiled_total = all.x;
            const uint32_t cap = call.tiled_persist * 256u;
            return (walk && call.tiled_persist && all.x > cap) ? dim3(cap, 1, 1) : all;
        };
        if (small) {
            const dim3 g = d2l_grid(d2l_all((a.F + 63) / 64, a.ksplit1, false, false), false);
            if (a.ksplit1 > 1) hipLaunchKernelGGL((gemm_d2l_kernel<3, 4, false, 128>), g, dim3(256), 81920, stream, a);
            else hipLaunchKernelGGL((stream_b ? gemm_d2l_kernel<1, 4, false, 128, true> : gemm_d2l_kernel<1, 4, false, 128>), g, dim3(256), 81920, stream, a);
        }
        else if (d2l4) { const dim3 g = d2l_grid(d2l_all((a.F + 127) / 128, 1, true, false), false); hipLaunchKernelGGL((gemm_d2l_kernel<1, 4, false, 256>), g, dim3(256), 163840, stream, a); }
        else if (d2l && a.ksplit1 > 1) { const dim3 g = d2l_grid(d2l_all((a.F + 127) / 128, a.ksplit1, false, false), false); hipLaunchKernelGGL((ragged ? gemm_d2l_kernel<3, 8, false, 256, false, true> : gemm_d2l_kernel<3, 8, false, 256>), g, dim3(512), 163840, stream, a); }
        else if (d2l) { const dim3 g = d2l_grid(d2l_all((a.F + 127) / 128, 1, true, call.tiled_persist != 0), true); hipLaunchKernelGGL((in_rows ? (stream_b ? gemm_d2l_kernel<1, 8, true, 256, true, false, true> : gemm_d2l_kernel<1, 8, true, 256, false, false, true>) : pick(gemm_d2l_kernel<1, 8, true, 256>, gemm_d2l_kernel<1, 8, true, 256, true>, gemm_d2l_kernel<1, 8, true, 256, false, true>, gemm_d2l_kernel<1, 8, true, 256, true, true>)), g, dim3(512), 163840, stream, a); }
        else if (four) hipLaunchKernelGGL(gemm_tiled4_kernel<1>, grid_for((a.F + 127) / 128), dim3(256), lds_bytes, stream, a);
        else hipLaunchKernelGGL(gemm_tiled_kernel<1>, grid_for((a.F + 127) / 128), dim3(512), lds_bytes, stream, a);
        launch_reduce();
        mark(2, 0);
        mark(3, 1);
        // The second product's workgroups walk where its tiles are short (at most 32 steps): the next tile's record, offsets and
        // first loads are on their way while the 256 KiB a tile stores leave.  The stores themselves are not hidden: the wait for
        // the record at the end of a tile covers them.  Microseconds per call without / with: 512 experts of H 2048 F 512, 200 rows each
        // 1137 / 1104, 20 of H 5120 F 1536, 1638 rows 1642 / 1615, 160 of those 512 rows 4637 / 4581, 205 rows 2127 / 2126.
        const bool walk2 = call.tiled_persist && a.ksplit == 1 && a.F <= 2048;
        if (small) { const dim3 g = d2l_grid(d2l_all((a.H + 127) / 128, a.ksplit, false, false), false); hipLaunchKernelGGL((stream_b ? gemm_d2l_kernel<2, 4, false, 128, true> : gemm_d2l_kernel<2, 4, false, 128>), g, dim3(256), 81920, stream, a); }
        else if (d2l4) { const dim3 g = d2l_grid(d2l_all((a.H + 255) / 256, a.ksplit, false, false), false); hipLaunchKernelGGL((gemm_d2l_kernel<2, 4, false, 256>), g, dim3(256), 163840, stream, a); }
        else if (d2l && walk2) { const dim3 g = d2l_grid(d2l_all((a.H + 255) / 256, 1, false, true), true); hipLaunchKernelGGL((in_rows ? (stream_b ? gemm_d2l_kernel<2, 8, true, 256, true, false, true> : gemm_d2l_kernel<2, 8, true, 256, false, false, true>) : pick(gemm_d2l_kernel<2, 8, true, 256>, gemm_d2l_kernel<2, 8, true, 256, true>, gemm_d2l_kernel<2, 8, true, 256, false, true>, gemm_d2l_kernel<2, 8, true, 256, true, true>)), g, dim3(512), 163840, stream, a); }
        else if (d2l) { const dim3 g = d2l_grid(d2l_all((a.H + 255) / 256, a.ksplit, false, false), false); hipLaunchKernelGGL((a.tail ? pick(gemm_d2l_kernel<2, 8, false, 256, false, false, false, true>, gemm_d2l_kernel<2, 8, false, 256, true, false, false, true>, gemm_d2l_kernel<2, 8, false, 256, false, true, false, true>, gemm_d2l_kernel<2, 8, false, 256, true, true, false, true>) : pick(gemm_d2l_kernel<2, 8, false, 256>, gemm_d2l_kernel<2, 8, false, 256, true>, gemm_d2l_kernel<2, 8, false, 256, false, true>, gemm_d2l_kernel<2, 8, false, 256, true, true>)), g, dim3(512), 163840, stream, a); }
        else if (four) hipLaunchKernelGGL(gemm_tiled4_kernel<2>, grid_for((a.H + 255) / 256), dim3(256), lds_bytes, stream, a);
        else hipLaunchKernelGGL(gemm_tiled_kernel<2>, grid_for((a.H + 255) / 256), dim3(512), lds_bytes, stream, a);
        if (a.tail) hipLaunchKernelGGL(last_round_kernel, dim3(16, 32, 4), dim3(256), 0, stream, a);
        mark(3, 0);
        if (a.direct) return hipGetLastError();
        const dim3 gc2((a.H / 4 + 255) / 256, a.T, 1);
        mark(4, 1);
        launch_combine(gc2);
        mark(4, 0);
        return hipGetLastError();
    }
    if (a.m_tile != 16 && a.m_tile != 32 && a.m_tile != 64 && a.m_tile != 96 && a.m_tile != 128) return hipErrorInvalidValue;
    // the strip kernels address activations and one expert matrix with 32-bit byte offsets
    if (uint64_t(a.T) * a.H * 2 >= (1ull << 32) || uint64_t(a.H) * a.F * 2 >= (1ull << 31)) return hipErrorInvalidValue;
    mark(2, 1);
    if (routes_itself && a.halves) launch_done(gemm1_swiglu_kernel<4, true, true, true>, g1, dim3(256), 0, stream, with_routing, a);
    else if (routes_itself) launch_done(gemm1_swiglu_kernel<4, true, false, true>, g1, dim3(256), 0, stream, with_routing, a);
    else if (a.halves && a.ksplit1 > 1) hipLaunchKernelGGL((gemm1_swiglu_kernel<8, false, true, true>), g1, dim3(256), 0, stream, a);
    else if (a.halves) hipLaunchKernelGGL((gemm1_swiglu_kernel<8, false, true, false>), g1, dim3(256), 0, stream, a);
    else if (a.m_tile == 16) hipLaunchKernelGGL((gemm1_swiglu_kernel<1, false, false, true>), g1, dim3(256), 0, stream, a);
    else if (a.m_tile == 32) hipLaunchKernelGGL((gemm1_swiglu_kernel<2, false, false, true>), g1, dim3(256), 0, stream, a);
    else if (a.m_tile == 64) hipLaunchKernelGGL((gemm1_swiglu_kernel<4, false, false, true>), g1, dim3(256), 0, stream, a);
    else if (a.m_tile == 96) hipLaunchKernelGGL((gemm1_swiglu_kernel<6, false, false, true>), g1, dim3(256), 0, stream, a);
    else if (a.ksplit1 > 1) hipLaunchKernelGGL((gemm1_swiglu_kernel<8, false, false, true>), g1, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((gemm1_swiglu_kernel<8, false, false, false>), g1, dim3(256), 0, stream, a);
    if (routes_itself)
        if (hipError_t e = record_routed(); e != hipSuccess) return e;
    if (!call.few_fused) launch_reduce();
    mark(2, 0);
    mark(3, 1);
    if (call.few2) {
        const dim3 grid(strips2, a.ksplit, a.tiles_cap);
        if (call.few_fused) hipLaunchKernelGGL((gemm2_few_kernel<1, true>), grid, dim3(256), std::max(32768u, 4u * 16u * (uint32_t(few_quarter(a.F, a.ksplit)) + 8u) * 2u), stream, a);
        else hipLaunchKernelGGL((gemm2_few_kernel<4, false>), grid, dim3(256), 65536, stream, a);
    } else if (a.m_tile == 16) hipLaunchKernelGGL(gemm2_kernel<1>, g2, dim3(256), 0, stream, a);
    else if (a.m_tile == 32) hipLaunchKernelGGL(gemm2_kernel<2>, g2, dim3(256), 0, stream, a);
    else if (a.m_tile == 64) hipLaunchKernelGGL(gemm2_kernel<4>, g2, dim3(256), 0, stream, a);
    else if (a.m_tile == 96) hipLaunchKernelGGL(gemm2_kernel<6>, g2, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(gemm2_kernel<8>, g2, dim3(256), 0, stream, a);
    mark(3, 0);
    const dim3 gc((a.H / 4 + 255) / 256, a.T, 1);
    mark(4, 1);
    launch_combine(gc);
    mark(4, 0);
    return hipGetLastError();
}

}  // namespace fluxmoe
