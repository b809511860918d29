// The offline encoder's loops over weights: exponent histogram, block plan, block encoding.  Host code without HIP, so that it can be
// tested on its own.  Each has a plain form and, on processors that look up 128 bytes with one instruction (AVX-512 VBMI), a
// vector form with the same results.  Bound by instructions: eight experts of H 2048 F 512 (50 MB) on 16 threads take 1.6 ms, 4.0 in
// the plain loops with a thread for each tensor and three sets of threads.
#pragma once

#include <cstdint>
#include <cstring>
#include <vector>

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define FLUXMOE_ENCODE_VECTOR 1
#include <immintrin.h>
#endif

namespace fluxmoe {

constexpr uint32_t kEncHeaderBytes = 136;     // u32 n, u32 e0, u16 sub_bits[64]
constexpr uint32_t kEncSubStreams = 64;
constexpr uint32_t kEncGroup = 64;

inline uint32_t exponent_of(uint16_t w) { return (w >> 7) & 0xFFu; }

// What one tensor type's code looks like to the loops: lengths, and the codes with their first bit in bit 0 (the stream is
// filled from bit 0 upwards), whole and as two byte tables.
struct Coder {
    alignas(64) uint8_t lens[256];
    alignas(64) uint8_t lo[256];
    alignas(64) uint8_t hi[256];
    uint32_t rev[256];

    Coder() = default;
    Coder(const uint8_t code_lens[256], const uint16_t codes[256]) {
        for (int s = 0; s < 256; ++s) {
            uint32_t r = 0;
            for (uint32_t b = 0; b < code_lens[s]; ++b) r |= ((codes[s] >> (code_lens[s] - 1 - b)) & 1u) << b;
            lens[s] = code_lens[s];
            rev[s] = r;
            lo[s] = uint8_t(r);
            hi[s] = uint8_t(r >> 8);
        }
    }
};

inline bool encode_vector_available() {
#ifdef FLUXMOE_ENCODE_VECTOR
    return __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512bw") && __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("avx512vbmi");
#else
    return false;
#endif
}

// hist[s] += number of elements of w[0..n) with exponent s.  Eight tables, so that equal neighbours do not wait for each other.
inline void count_exponents(const uint16_t* w, uint64_t n, uint64_t hist[256]) {
    uint32_t local[8][256];
    for (uint64_t at = 0; at < n;) {
        const uint64_t end = at + (n - at < (1ull << 30) ? n - at : (1ull << 30));
        std::memset(local, 0, sizeof local);
        uint64_t m = at;
        for (; m + 8 <= end; m += 8) {
            uint64_t a, b;
            std::memcpy(&a, w + m, 8);
            std::memcpy(&b, w + m + 4, 8);
            ++local[0][(a >> 7) & 0xFF]; ++local[1][(a >> 23) & 0xFF]; ++local[2][(a >> 39) & 0xFF]; ++local[3][(a >> 55) & 0xFF];
            ++local[4][(b >> 7) & 0xFF]; ++local[5][(b >> 23) & 0xFF]; ++local[6][(b >> 39) & 0xFF]; ++local[7][(b >> 55) & 0xFF];
        }
        for (; m < end; ++m) ++local[0][exponent_of(w[m])];
        for (int s = 0; s < 256; ++s)
            for (int t = 0; t < 8; ++t) hist[s] += local[t][s];
        at = end;
    }
}

// Greedy packing in groups of 64 elements: a block takes the largest number of whole groups whose header + raw bytes + code
// words still fit.  group_bits(pointer to 64 elements) -> their code bits.
template <typename F>
inline __attribute__((always_inline)) void plan_with(const uint16_t* w, uint64_t n_elems, uint32_t block_bytes, std::vector<uint32_t>& first_elem, F&& group_bits) {
    first_elem.clear();
    first_elem.push_back(0);
    uint64_t pos = 0;
    while (pos < n_elems) {
        uint64_t n = 0, bits = 0;
        while (pos + n < n_elems) {
            const uint64_t gbits = group_bits(w + pos + n);
            const uint64_t need = kEncHeaderBytes + (n + kEncGroup) + 4 * ((bits + gbits + 31) / 32);
            if (need > block_bytes) break;
            n += kEncGroup;
            bits += gbits;
        }
        pos += n;   // n >= 64 always: 136 + 64 + 96 bytes fit any supported block size
        first_elem.push_back(static_cast<uint32_t>(pos));
    }
}

inline void plan_plain(const uint16_t* w, uint64_t n_elems, const Coder& c, uint32_t block_bytes, std::vector<uint32_t>& first_elem) {
    plan_with(w, n_elems, block_bytes, first_elem, [&](const uint16_t* g) {
        uint64_t bits = 0;
        for (uint32_t i = 0; i < kEncGroup; ++i) bits += c.lens[exponent_of(g[i])];
        return bits;
    });
}

// Block of elements w[e0 .. e0 + n) at blk (block_bytes bytes, all written).
inline void encode_block_plain(const uint16_t* w, uint32_t e0, uint32_t n, const Coder& c, uint32_t block_bytes, uint8_t* blk) {
    std::memset(blk, 0, block_bytes);
    const uint16_t* src = w + e0;
    std::memcpy(blk, &n, 4);
    std::memcpy(blk + 4, &e0, 4);
    uint8_t* sm = blk + kEncHeaderBytes;
    for (uint32_t m = 0; m < n; ++m) sm[m] = static_cast<uint8_t>(((src[m] >> 8) & 0x80u) | (src[m] & 0x7Fu));
    // sub-streams are written one after another by a single bit writer
    uint8_t* area = blk + kEncHeaderBytes + n;
    uint64_t acc = 0;
    uint32_t fill = 0;
    size_t word = 0;
    const uint32_t n_runs = n / 8;
    for (uint32_t j = 0; j < kEncSubStreams; ++j) {
        uint32_t bits_j = 0;
        for (uint32_t r = j; r < n_runs; r += kEncSubStreams) {
            const uint16_t* run = src + 8u * r;
            for (uint32_t i = 0; i < 8; ++i) {
                const uint32_t s = exponent_of(run[i]);
                acc |= static_cast<uint64_t>(c.rev[s]) << fill;
                fill += c.lens[s];
                bits_j += c.lens[s];
                if (fill >= 32) {
                    const uint32_t out = static_cast<uint32_t>(acc);
                    std::memcpy(area + 4 * word, &out, 4);
                    ++word;
                    acc >>= 32;
                    fill -= 32;
                }
            }
        }
        const uint16_t sb = static_cast<uint16_t>(bits_j);
        std::memcpy(blk + 8 + 2 * j, &sb, 2);
    }
    if (fill) {
        const uint32_t out = static_cast<uint32_t>(acc);
        std::memcpy(area + 4 * word, &out, 4);
    }
}

#ifdef FLUXMOE_ENCODE_VECTOR
#define FLUXMOE_VBMI __attribute__((target("avx512f,avx512bw,avx512vl,avx512vbmi,bmi2")))

// table[index] for 64 byte indices
FLUXMOE_VBMI inline __m512i lookup256(const __m512i (&t)[4], __m512i index) {
    const __m512i low = _mm512_permutex2var_epi8(t[0], index, t[1]), high = _mm512_permutex2var_epi8(t[2], index, t[3]);
    return _mm512_mask_blend_epi8(_mm512_movepi8_mask(index), low, high);
}
FLUXMOE_VBMI inline void load_table(__m512i (&t)[4], const uint8_t* bytes) {
    for (int i = 0; i < 4; ++i) t[i] = _mm512_load_si512(bytes + 64 * i);
}
// the exponents of 64 elements
FLUXMOE_VBMI inline __m512i exponents64(const uint16_t* w) {
    const __m256i a = _mm512_cvtepi16_epi8(_mm512_srli_epi16(_mm512_loadu_si512(w), 7)), b = _mm512_cvtepi16_epi8(_mm512_srli_epi16(_mm512_loadu_si512(w + 32), 7));
    return _mm512_inserti64x4(_mm512_castsi256_si512(a), b, 1);
}

FLUXMOE_VBMI inline void plan_vector(const uint16_t* w, uint64_t n_elems, const Coder& c, uint32_t block_bytes, std::vector<uint32_t>& first_elem) {
    // code bits of every group first (independent of each other), then the packing
    const uint64_t groups = n_elems / kEncGroup;
    std::vector<uint16_t> bits(groups);
    __m512i lens[4];
    load_table(lens, c.lens);
    for (uint64_t g = 0; g < groups; ++g) {
        const __m512i l = lookup256(lens, exponents64(w + g * kEncGroup));
        bits[g] = uint16_t(_mm512_reduce_add_epi64(_mm512_sad_epu8(l, _mm512_setzero_si512())));
    }
    plan_with(w, n_elems, block_bytes, first_elem, [&](const uint16_t* g) { return uint64_t(bits[uint64_t(g - w) / kEncGroup]); });
}

// 64 elements at a time: codes and lengths by table look-up, four neighbours joined into one word of up to 48 bits; what is left for the
// serial bit writer is one such word for every four elements, without a branch.
FLUXMOE_VBMI inline void encode_block_vector(const uint16_t* w, uint32_t e0, uint32_t n, const Coder& c, uint32_t block_bytes, uint8_t* blk) {
    constexpr uint32_t kMost = 4096;                         // elements: one raw byte each, block_bytes is 4096
    if (n > kMost || n % 64 != 0 || block_bytes > kMost) { encode_block_plain(w, e0, n, c, block_bytes, blk); return; }
    alignas(64) uint64_t code[kMost / 4];
    alignas(64) uint64_t len[kMost / 4];
    alignas(64) uint8_t out[2 * kMost];                      // the writers store eight bytes at a time
    __m512i lens[4], lo[4], hi[4];
    load_table(lens, c.lens);
    load_table(lo, c.lo);
    load_table(hi, c.hi);
    const uint16_t* src = w + e0;
    std::memcpy(out, &n, 4);
    std::memcpy(out + 4, &e0, 4);
    uint8_t* sm = out + kEncHeaderBytes;
    const __m512i sign = _mm512_set1_epi16(0x80), mantissa = _mm512_set1_epi16(0x7F);
    // bytes 0, 64, 1, 65, .. of (low, high) give the 16-bit codes of elements 0..31, then 32..63
    alignas(64) uint8_t order[2][64];
    for (int i = 0; i < 64; ++i)
        for (int half = 0; half < 2; ++half) order[half][i] = uint8_t(32 * half + i / 2 + 64 * (i & 1));
    const __m512i order_lo = _mm512_load_si512(order[0]), order_hi = _mm512_load_si512(order[1]);
    auto join = [](__m512i codes, __m512i lengths, uint64_t* code_out, uint64_t* len_out) FLUXMOE_VBMI {
        // 16-bit codes and lengths -> pairs in 32 bits -> fours in 64
        const __m512i even = _mm512_and_si512(codes, _mm512_set1_epi32(0xFFFF)), odd = _mm512_srli_epi32(codes, 16);
        const __m512i len_even = _mm512_and_si512(lengths, _mm512_set1_epi32(0xFFFF));
        const __m512i pair = _mm512_or_si512(even, _mm512_sllv_epi32(odd, len_even));
        const __m512i pair_len = _mm512_add_epi32(len_even, _mm512_srli_epi32(lengths, 16));
        const __m512i low = _mm512_and_si512(pair, _mm512_set1_epi64(0xFFFFFFFFll)), high = _mm512_srli_epi64(pair, 32);
        const __m512i len_low = _mm512_and_si512(pair_len, _mm512_set1_epi64(0xFFFFFFFFll));
        _mm512_store_si512(code_out, _mm512_or_si512(low, _mm512_sllv_epi64(high, len_low)));
        _mm512_store_si512(len_out, _mm512_add_epi64(len_low, _mm512_srli_epi64(pair_len, 32)));
    };
    for (uint32_t m = 0; m < n; m += 64) {
        const __m512i a = _mm512_loadu_si512(src + m), b = _mm512_loadu_si512(src + m + 32);
        const __m512i raw_a = _mm512_or_si512(_mm512_and_si512(_mm512_srli_epi16(a, 8), sign), _mm512_and_si512(a, mantissa));
        const __m512i raw_b = _mm512_or_si512(_mm512_and_si512(_mm512_srli_epi16(b, 8), sign), _mm512_and_si512(b, mantissa));
        _mm256_storeu_si256(reinterpret_cast<__m256i*>(sm + m), _mm512_cvtepi16_epi8(raw_a));
        _mm256_storeu_si256(reinterpret_cast<__m256i*>(sm + m + 32), _mm512_cvtepi16_epi8(raw_b));
        const __m512i e = exponents64(src + m);
        const __m512i l = lookup256(lens, e), cl = lookup256(lo, e), ch = lookup256(hi, e);
        const __m512i zero = _mm512_setzero_si512();
        join(_mm512_permutex2var_epi8(cl, order_lo, ch), _mm512_permutex2var_epi8(l, order_lo, zero), code + m / 4, len + m / 4);
        join(_mm512_permutex2var_epi8(cl, order_hi, ch), _mm512_permutex2var_epi8(l, order_hi, zero), code + m / 4 + 8, len + m / 4 + 8);
    }
    // two writers, for sub-streams 0..31 and 32..63, so that their chains of shifts overlap; the second writes elsewhere (a
    // store of the first reaches past its end) from the bit where the first will stop
    const uint32_t n_runs = n / 8;
    uint64_t bits_first = 0;
    for (uint32_t r = 0; r < n_runs; r += kEncSubStreams)
        for (uint32_t i = 2 * r; i < 2 * (r + 32 < n_runs ? r + 32 : n_runs); ++i) bits_first += len[i];
    struct Writer {
        uint8_t* at;
        uint64_t acc, fill;
        void put(uint64_t code, uint64_t bits) {             // fill <= 7, bits <= 48
            acc |= code << fill;
            std::memcpy(at, &acc, 8);
            fill += bits;
            at += fill >> 3;
            acc >>= fill & ~7ull;
            fill &= 7;
        }
    };
    alignas(64) uint8_t out2[kMost + 64];
    Writer x{sm + n, 0, 0}, y{out2, 0, bits_first & 7};
    uint16_t sub_bits[kEncSubStreams];
    for (uint32_t j = 0; j < 32; ++j) {
        uint64_t bx = 0, by = 0;
        uint32_t r = j;
        for (; r + 32 < n_runs; r += kEncSubStreams) {
            const uint32_t i = 2 * r, k = 2 * (r + 32);
            x.put(code[i], len[i]);
            y.put(code[k], len[k]);
            x.put(code[i + 1], len[i + 1]);
            y.put(code[k + 1], len[k + 1]);
            bx += len[i] + len[i + 1];
            by += len[k] + len[k + 1];
        }
        if (r < n_runs) {
            const uint32_t i = 2 * r;
            x.put(code[i], len[i]);
            x.put(code[i + 1], len[i + 1]);
            bx += len[i] + len[i + 1];
        }
        sub_bits[j] = uint16_t(bx);
        sub_bits[j + 32] = uint16_t(by);
    }
    std::memcpy(out + 8, sub_bits, sizeof sub_bits);
    std::memcpy(y.at, &y.acc, 8);                            // the last bits, and zeros behind them
    out2[0] |= uint8_t(x.acc);                               // the byte in which the second begins
    const size_t second = size_t(y.at - out2) + 8;
    std::memcpy(x.at, out2, second);
    const size_t used = size_t(x.at - out) + second;
    std::memcpy(blk, out, used < block_bytes ? used : block_bytes);
    if (used < block_bytes) std::memset(blk + used, 0, block_bytes - used);
}
#endif

inline void plan_tensor(const uint16_t* w, uint64_t n_elems, const Coder& c, uint32_t block_bytes, std::vector<uint32_t>& first_elem, bool vector) {
#ifdef FLUXMOE_ENCODE_VECTOR
    if (vector) { plan_vector(w, n_elems, c, block_bytes, first_elem); return; }
#endif
    (void)vector;
    plan_plain(w, n_elems, c, block_bytes, first_elem);
}

// Blocks [k0, k1) of a tensor whose block 0 goes to dst (first_elem: the tensor's plan).
inline void encode_blocks(const uint16_t* w, const std::vector<uint32_t>& first_elem, size_t k0, size_t k1, const Coder& c, uint32_t block_bytes, uint8_t* dst, bool vector) {
    for (size_t k = k0; k < k1; ++k) {
        const uint32_t e0 = first_elem[k], n = first_elem[k + 1] - e0;
        uint8_t* blk = dst + k * size_t(block_bytes);
#ifdef FLUXMOE_ENCODE_VECTOR
        if (vector) { encode_block_vector(w, e0, n, c, block_bytes, blk); continue; }
#endif
        encode_block_plain(w, e0, n, c, block_bytes, blk);
    }
    (void)vector;
}

}  // namespace fluxmoe
