// The shared expert's products in tiles of 32, 64 or 128 rows x 128 columns with a deep ring of LDS stages (gfx950).
//
// For launches of at most a round or two of workgroups, which are bound by latencies rather than bandwidth: both operands go from global memory straight into a ring of NS stages (global_load_lds_dwordx4) and are fetched NS - 1 steps
// of 64 k ahead.  Four wavefronts, one barrier per step; B stays row-major in LDS and its fragments are formed by the
// transposing read (ds_read_b64_tr_b16), as in gemm_d2l_kernel.  K may be any multiple of 8: the pieces of the last step that
// lie past its end are fetched from a piece of zeros.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ffn_device.h"
#include "kernels.h"

namespace fluxmoe {

namespace {

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kTK = 64;                       // k of a step
constexpr int kTN = 128;                      // columns of a tile: of y, or 64 of W1 and the same 64 of W3

template <int N> using Int = std::integral_constant<int, N>;

// MODE 1: h = SwiGLU(X W1, X W3).  MODE 2: y = h W2, K split ksplit ways, or the output itself (a.direct).
// MODE 3: the first product with K split ksplit1 ways, FP32 partial sums of gate and up.
// TM 128: wavefronts 2 x 2 of 64 x 64; 64: 2 x 2 of 32 x 64; 32: 1 x 4 of 32 x 32, in the first product with 16 columns of
// W1 and the same 16 of W3.
template <int MODE, int TM, int NS>
__global__ __launch_bounds__(256, 2) void gemm_ring_kernel(FfnArgs a) {
    constexpr bool kFirst = MODE != 2;
    constexpr int kWaveRows = TM == 32 ? 1 : 2;              // wavefronts along the rows
    constexpr int kRowTiles = TM / 32 / kWaveRows;           // 32-row MFMA tiles of a wavefront: groups wm, wm + 2
    constexpr int kColTiles = TM == 32 ? 1 : 2;              // 32-column MFMA tiles of a wavefront
    constexpr int kDmaA = TM / 32, kDmaB = 4;                // 1 KiB loads per wavefront and step
    constexpr int kLoads = kDmaA + kDmaB;
    constexpr int kStageA = TM * 2 * kTK, kStage = kStageA + kTN * 2 * kTK;
    constexpr int kMfma = kRowTiles * kColTiles;             // per sub-step of 16 k
    constexpr int kFrag = kRowTiles + 2 * kColTiles;         // fragment reads per sub-step
    static_assert(NS >= 3 && (NS - 2) * kLoads < 64, "the wait counter has six bits");
    extern __shared__ __align__(16) uint8_t lds[];

    const uint32_t K = kFirst ? a.H : a.F, N = kFirst ? a.F : a.H;
    const uint32_t n_ct = (N + (kFirst ? 63u : 127u)) / (kFirst ? 64u : 128u);
    const uint32_t n_split = MODE == 1 ? 1u : (MODE == 2 ? a.ksplit : a.ksplit1);
    // Workgroups go to the 8 XCDs round robin: the row tiles of a (column tile, split) follow each other on one XCD and find
    // its weights in that XCD's L2.
    const uint32_t n_rt = (a.T + TM - 1) / TM;
    const uint32_t unit = (blockIdx.x / 8u / n_rt) * 8u + blockIdx.x % 8u;
    if (unit >= n_ct * n_split) return;
    const uint32_t split = unit % n_split, col_tile = unit / n_split;
    const uint32_t row0 = blockIdx.x / 8u % n_rt * TM;       // every token once, in order, on the one expert: no lists
    const int rows = min(TM, int(a.T - row0));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = kWaveRows == 2 ? wave >> 1 : 0, wn = kWaveRows == 2 ? wave & 1 : wave;
    const uint32_t steps_all = (K + kTK - 1) / kTK;
    const uint32_t step_lo = steps_all * split / n_split, step_hi = steps_all * (split + 1) / n_split;
    const uint32_t n_steps = step_hi - step_lo;              // >= 1: the host keeps the splits <= K / 64
    const uint32_t k_begin = step_lo * kTK, k_len = min(K, step_hi * kTK) - k_begin;
    const bool ragged = k_len % kTK != 0;                    // the last step is a partial one
    const uint32_t n_base = col_tile * (kFirst ? 64u : 128u);
    const size_t mat = size_t(a.H) * a.F;
    const uint32_t lds_base = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));

    // M0 carries the LDS destination of an LDS-direct load and is read when the instruction issues; the compiler reserves
    // it, so its value is put back.  Inline assembly, because with the builtin every later LDS read waits for all loads.
    auto dma16 = [&](const uint8_t* base, uint32_t off, uint32_t dst) __attribute__((always_inline)) {
        uint32_t saved_m0;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "v"(off), "s"(base), "s"(dst) : "memory");
    };
    // Weights: non-temporal, or behind a kernel that left the caches full of dirty lines every line waits for one to be written
    // back (8 rows, H 4096 F 14336, first product behind a 768 MB fill: 95 / 49 us; otherwise the same).
    auto dma16_nt = [&](const uint8_t* base, uint32_t off, uint32_t dst) __attribute__((always_inline)) {
        uint32_t saved_m0;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\ts_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "v"(off), "s"(base), "s"(dst) : "memory");
    };
    auto dma16_at = [&](const uint8_t* ptr, uint32_t dst) __attribute__((always_inline)) {
        uint32_t saved_m0;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                     : "=&s"(saved_m0) : "v"(ptr), "s"(dst) : "memory");
    };

    // ---- what the lane fetches.  A: rows 8 (kDmaA wave + i) + lane / 8 of 128 bytes; position p of row r holds 16-byte piece
    // p ^ ((r >> 1) & 7).  B: k rows 4 (4 wave + i) + lane / 16 of 256 bytes; position u holds unit u ^ (k & 3) of 32 columns.
    const uint8_t* b_base = reinterpret_cast<const uint8_t*>((kFirst ? a.slots13 : a.slots2) + size_t(k_begin) * N);
    uint32_t b_off[kDmaB];
#pragma unroll
    for (int i = 0; i < kDmaB; ++i) {
        const uint32_t k_lds = 4u * (kDmaB * wave + i) + (lane >> 4);
        const uint32_t pp = lane & 15u, c = 32u * ((pp >> 2) ^ (k_lds & 3u)) + 8u * (pp & 3u);
        const uint32_t elems = kFirst ? (c >= 64u ? uint32_t(mat) : 0u) + min(n_base + (c & 63u), N - 8u) : min(n_base + c, N - 8u);
        b_off[i] = 2u * (elems + k_lds * N);
    }
    auto load_b = [&](uint32_t st, uint32_t stage, int i, auto TAIL) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + stage * kStage + kStageA + uint32_t(kDmaB * wave + i) * 1024u;
        const uint8_t* base = b_base + size_t(st) * kTK * N * 2;
        if (!TAIL.value) { dma16_nt(base, b_off[i], dst); return; }
        const uint32_t k_lds = 4u * (kDmaB * wave + i) + (lane >> 4);
        dma16_at(st * kTK + k_lds < k_len ? base + b_off[i] : reinterpret_cast<const uint8_t*>(&g_zero_piece), dst);
    };
    const uint8_t* a_base = reinterpret_cast<const uint8_t*>(kFirst ? a.tokens + size_t(row0) * a.H : a.hbuf + size_t(row0) * a.F) + size_t(k_begin) * 2;
    uint32_t a_off[kDmaA];
    const bool a_live = 8 * kDmaA * wave < rows;             // a wavefront past the tile's last row fetches none of A
    auto load_a = [&](uint32_t st, uint32_t stage, int i, auto TAIL) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + stage * kStage + uint32_t(kDmaA * wave + i) * 1024u;
        const uint8_t* base = a_base + size_t(st) * kTK * 2;
        if (!TAIL.value) { dma16(base, a_off[i], dst); return; }
        const uint32_t r = 8u * (kDmaA * wave + i) + (lane >> 3), piece = (lane & 7u) ^ ((r >> 1) & 7u);
        dma16_at(st * kTK + 8u * piece < k_len ? base + a_off[i] : reinterpret_cast<const uint8_t*>(&g_zero_piece), dst);
    };
    auto load_step = [&](uint32_t st, uint32_t stage) __attribute__((always_inline)) {
        auto both = [&](auto TAIL) __attribute__((always_inline)) {
            if (a_live) {
#pragma unroll
                for (int i = 0; i < kDmaA; ++i) load_a(st, stage, i, TAIL);
            }
#pragma unroll
            for (int i = 0; i < kDmaB; ++i) load_b(st, stage, i, TAIL);
        };
        if (ragged && st + 1 == n_steps) both(Int<1>{}); else both(Int<0>{});
    };
    // loads return in order: the ones of the r newest steps may stay in flight
    auto wait_loads = [&](auto R) __attribute__((always_inline)) {
        if (a_live) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(R.value * kLoads) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(R.value * kDmaB) : "memory");
    };

#pragma unroll
    for (int i = 0; i < kDmaA; ++i) {
        const uint32_t r = 8u * (kDmaA * wave + i) + (lane >> 3), piece = (lane & 7u) ^ ((r >> 1) & 7u);
        a_off[i] = 2u * (min(r, uint32_t(rows - 1)) * K + 8u * piece);
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (uint32_t(s) < n_steps) load_step(s, s);

    // ---- fragment addresses inside a stage
    int a_fr[kRowTiles][4], b_fr[kColTiles];
    {
        const int q = lane & 31, h = lane >> 5, e = (lane & 15) >> 2, g = lane & 3, nh = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i) {
            const int R = 32 * (wm + kWaveRows * i) + q;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a_fr[i][ks] = R * 128 + 16 * ((2 * ks + h) ^ ((R >> 1) & 7));
        }
#pragma unroll
        for (int j = 0; j < kColTiles; ++j) {
            if (TM == 32 && kFirst) b_fr[j] = kStageA + (8 * h + e) * 256 + 64 * ((2 * nh + (wn >> 1)) ^ e) + 32 * (wn & 1) + 8 * g;
            else b_fr[j] = kStageA + (8 * h + e) * 256 + 64 * ((TM == 32 ? wn : (kFirst ? wn + 2 * j : 2 * wn + j)) ^ e) + 32 * nh + 8 * g;
        }
    }
    // A chain of sums is kChain steps long: then it is added to `total` and begins anew.  Fewer K splits than the kernels before
    // would make it longer, and its rounding decides how often an element of h is rounded the other way: share of tokens
    // with one, before / unbroken chains / 8 steps / 4 steps: H 5120 F 1536, 512 rows 0.071 / 0.09 / 0.055 / 0.043; H 4504 F 2776,
    // 241 rows 0.063 / - / 0.071 / 0.064; H 4096 F 14336, 100 rows 0.33 / - / 0.23 / 0.20.
    constexpr uint32_t kChain = 4;
    f32x16 acc[kRowTiles][kColTiles], total[kRowTiles][kColTiles];
#pragma unroll
    for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
        for (int j = 0; j < kColTiles; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = total[i][j][r] = 0.f;

    auto k_loop = [&](auto ACT) __attribute__((always_inline)) {
        bf16x8 fa[2][kRowTiles];
        i16x4 fb_lo[2][kColTiles], fb_hi[2][kColTiles];
        auto frag = [&](uint32_t stage_off, int ks, int set, int n) __attribute__((always_inline)) {
            if (n < kRowTiles) {
                if (n < ACT.value) fa[set][n] = *reinterpret_cast<const bf16x8*>(lds + a_fr[n][ks] + stage_off);
            } else {
                const int j = (n - kRowTiles) >> 1, tt = (n - kRowTiles) & 1;
                const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(lds + b_fr[j] + stage_off + ks * 4096 + tt * 1024));
                if (tt == 0) fb_lo[set][j] = v; else fb_hi[set][j] = v;
            }
        };
        // sub-step ks: its MFMAs, between them the fragment reads of the next one and a share of the step's loads
        auto sub = [&](int ks, uint32_t stage_off, int next_ks, auto READ, auto load_item, int load_from, int load_to) __attribute__((always_inline)) {
            const int set = ks & 1;
#pragma unroll
            for (int n = 0; n < (kMfma > kFrag ? kMfma : kFrag); ++n) {
                if (n < kColTiles * ACT.value) {
                    const int i = n / kColTiles, j = n % kColTiles;
                    const i16x8 full = __builtin_shufflevector(fb_lo[set][j], fb_hi[set][j], 0, 1, 2, 3, 4, 5, 6, 7);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], __builtin_bit_cast(bf16x8, full), acc[i][j], 0, 0, 0);
                }
                if (READ.value && ACT.value && n < kFrag) frag(stage_off, next_ks, set ^ 1, n);
                if (load_from + n < load_to) load_item(load_from + n);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // LOAD: fetch step s + NS - 1 into the stage that step s - 1 left (0 none, 1 whole step, 2 the partial last step);
        // WAIT: steps that may stay in flight when the next one is needed, -1: there is no next one
        auto step = [&](uint32_t s, uint32_t stage, auto LOAD, auto WAIT) __attribute__((always_inline)) {
            const uint32_t off = stage * kStage, next = stage + 1 == NS ? 0u : stage + 1, refill = stage == 0 ? NS - 1 : stage - 1;
            auto item = [&](int n) __attribute__((always_inline)) {
                if (LOAD.value == 0) return;
                if (n < kDmaA) { if (a_live) load_a(s + NS - 1, refill, n, Int<LOAD.value == 2>{}); }
                else load_b(s + NS - 1, refill, n - kDmaA, Int<LOAD.value == 2>{});
            };
            using Yes = Int<1>;
            sub(0, off, 1, Yes{}, item, 0, 3);
            sub(1, off, 2, Yes{}, item, 3, kLoads < 6 ? kLoads : 6);
            sub(2, off, 3, Yes{}, item, 6, kLoads);
            if constexpr (WAIT.value >= 0) {
                wait_loads(WAIT);
                __syncthreads();                             // the next step's stage is complete, and this one's fragments are read
                sub(3, next * kStage, 0, Yes{}, item, 0, 0);
            } else {
                sub(3, 0, 0, Int<0>{}, item, 0, 0);
            }
        };
        if (n_steps >= uint32_t(NS - 1)) wait_loads(Int<NS - 2>{}); else wait_loads(Int<0>{});
        __syncthreads();
        if (ACT.value) {
#pragma unroll
            for (int n = 0; n < kFrag; ++n) frag(0, 0, 0, n);
        }
        uint32_t s = 0, stage = 0;
        auto advance = [&]() __attribute__((always_inline)) {
            ++s;
            stage = stage + 1 == NS ? 0u : stage + 1;
            if (s % kChain == 0) {
#pragma unroll
                for (int i = 0; i < ACT.value; ++i)
#pragma unroll
                    for (int j = 0; j < kColTiles; ++j) {
                        total[i][j] += acc[i][j];
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
                    }
            }
        };
        const uint32_t whole = ragged ? n_steps - 1 : n_steps;
        for (; s + NS - 1 < whole; advance()) step(s, stage, Int<1>{}, Int<NS - 2>{});
        if (s + NS - 1 < n_steps) { step(s, stage, Int<2>{}, Int<NS - 2>{}); advance(); }
        while (s + 1 < n_steps) {                            // nothing left to fetch
            const uint32_t later = n_steps - 2 - s;          // steps after the next one, all of them fetched
            if (later >= 2 && NS > 4) step(s, stage, Int<0>{}, Int<2>{});
            else if (later >= 1) step(s, stage, Int<0>{}, Int<1>{});
            else step(s, stage, Int<0>{}, Int<0>{});
            advance();
        }
        step(s, stage, Int<0>{}, Int<-1>{});
    };
    if constexpr (kRowTiles == 2) {
        if (32 * (wm + 2) < rows) k_loop(Int<2>{});
        else if (32 * wm < rows) k_loop(Int<1>{});
        else k_loop(Int<0>{});
    } else {
        if (32 * wm < rows) k_loop(Int<1>{});
        else k_loop(Int<0>{});
    }

#pragma unroll
    for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
        for (int j = 0; j < kColTiles; ++j) acc[i][j] += total[i][j];

    // ---- epilogue.  D layout of the 32 x 32 MFMA: column q = lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4
    const int q = lane & 31, h = lane >> 5;
    auto row_of = [&](int i, int r) __attribute__((always_inline)) { return 32 * (wm + kWaveRows * i) + (r >> 2) * 8 + h * 4 + (r & 3); };
    if (MODE == 1) {
        // neighbouring lanes swap values (DPP), so that a lane stores two columns of one row: an even lane of row r, an odd
        // one of row r + 1.  v_perm_b32(other, own, sel): selector bytes 0..3 pick from own, 4..7 from other
        const uint32_t pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
        if constexpr (TM == 32) {
            // lanes 0..15 of a half hold gate, lanes 16..31 up of the same columns: they trade a register, after which the
            // first have gate and up of register r, the others of r + 8
            const uint32_t col = n_base + 16u * wn + (lane & 14);
            const int upper = (lane >> 4) & 1;
#pragma unroll
            for (int r = 0; r < 8; r += 2) {
                float v[2];
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const float lo = acc[0][0][r + d], hi = acc[0][0][r + d + 8];
                    const float got = __shfl_xor(upper ? lo : hi, 16);
                    v[d] = swiglu(upper ? got : lo, upper ? hi : got);
                }
                const uint32_t own = pack_bf16_rne(v[0], v[1]);
                const uint32_t other = uint32_t(__builtin_amdgcn_update_dpp(0, int(own), 0xB1, 0xF, 0xF, true));
                const uint32_t packed = __builtin_amdgcn_perm(other, own, pair_sel);
                const int32_t row = row_of(0, r) + 16 * upper + (lane & 1);
                if (row < rows && col < N) *reinterpret_cast<uint32_t*>(a.hbuf + (size_t(row0) + uint32_t(row)) * a.F + col) = packed;
            }
        } else {
            const uint32_t col = n_base + 32u * wn + (q & ~1);
#pragma unroll
            for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const uint32_t own = pack_bf16_rne(swiglu(acc[i][0][r], acc[i][kColTiles - 1][r]), swiglu(acc[i][0][r + 1], acc[i][kColTiles - 1][r + 1]));
                    const uint32_t other = uint32_t(__builtin_amdgcn_update_dpp(0, int(own), 0xB1, 0xF, 0xF, true));
                    const uint32_t packed = __builtin_amdgcn_perm(other, own, pair_sel);
                    const int32_t row = row_of(i, r) + (lane & 1);
                    if (row < rows && col < N) *reinterpret_cast<uint32_t*>(a.hbuf + (size_t(row0) + uint32_t(row)) * a.F + col) = packed;
                }
        }
    } else if (MODE == 3) {
        // partial sums: row r of split s at [s][r][gate | up][F]
        float* const plane = a.ybuf + (size_t(split) * a.pairs_cap + size_t(row0)) * 2 * a.F;
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int j = 0; j < kColTiles; ++j) {
                const uint32_t up = TM == 32 ? uint32_t(lane >> 4) & 1u : uint32_t(j);
                const uint32_t col = n_base + (TM == 32 ? 16u * wn + (lane & 15) : 32u * wn + q);
                if (col >= N) continue;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int32_t row = row_of(i, r);
                    if (row < rows) plane[size_t(uint32_t(row)) * 2 * a.F + up * a.F + col] = acc[i][j][r];
                }
            }
    } else {
        // y of the split, or (direct: one split, every row is one token with gate 1) the output
        float* const plane = a.direct ? a.out + size_t(row0) * a.H : a.ybuf + (size_t(split) * a.pairs_cap + size_t(row0)) * a.H;
        const bool add = a.direct && (a.flags & 1u);
#pragma unroll
        for (int i = 0; i < kRowTiles; ++i)
#pragma unroll
            for (int j = 0; j < kColTiles; ++j) {
                const uint32_t col = n_base + (TM == 32 ? 32u * wn : 64u * wn + 32u * j) + q;
                if (col >= N) continue;
                if (add) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int32_t row = min(row_of(i, r), rows - 1);
                        acc[i][j][r] += plane[size_t(uint32_t(row)) * a.H + col];
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int32_t row = row_of(i, r);
                    if (row < rows) plane[size_t(uint32_t(row)) * a.H + col] = acc[i][j][r];
                }
            }
    }
}

template <int TM, int NS>
hipError_t launch(const FfnArgs& a, int mode, hipStream_t stream) {
    constexpr uint32_t bytes = NS * (TM * 128 + 16384);
    auto* const kernel = mode == 1 ? gemm_ring_kernel<1, TM, NS> : (mode == 2 ? gemm_ring_kernel<2, TM, NS> : gemm_ring_kernel<3, TM, NS>);
    static bool attr_set[3] = {};
    if (!attr_set[mode - 1]) {
        if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)); e != hipSuccess) return e;
        attr_set[mode - 1] = true;
    }
    const uint32_t n_ct = mode == 2 ? (a.H + 127) / 128 : (a.F + 63) / 64, splits = mode == 2 ? a.ksplit : (mode == 3 ? a.ksplit1 : 1u);
    hipLaunchKernelGGL(kernel, dim3((n_ct * splits + 7) / 8 * 8 * ((a.T + TM - 1) / TM)), dim3(256), bytes, stream, a);
    return hipGetLastError();
}

}  // namespace

// Stages: what two workgroups (32 and 64 rows) or one (128) can have of a CU's 160 KiB.  Six and eight stages with one
// workgroup a CU were no faster where one fits (H 5120 F 1536, 64 rows of 64: 47 / 47 us) and lost where two do (512 rows: 46 / 47,
// second product 25 / 32).
hipError_t launch_ring(const FfnArgs& a, int product, hipStream_t stream) {
    const uint32_t splits = product == 2 ? a.ksplit : a.ksplit1, k = product == 2 ? a.F : a.H, rows = product == 2 ? a.ring2 : a.ring1;
    if (!a.identity || splits == 0 || splits > (k + kTK - 1) / kTK) return hipErrorInvalidValue;
    const int mode = product == 2 ? 2 : (a.ksplit1 > 1 ? 3 : 1);
    if (rows == 128) return launch<128, 5>(a, mode, stream);
    if (rows == 64) return launch<64, 3>(a, mode, stream);
    if (rows == 32) return launch<32, 4>(a, mode, stream);
    return hipErrorInvalidValue;
}

}  // namespace fluxmoe
