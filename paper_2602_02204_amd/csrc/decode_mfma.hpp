// Matrix-core split-context decode kernel, group size <= 16: bf16 and fp32 caches with head_dim 64 or 128, 8-bit (E4M3)
// caches with head_dim 128.
//
// A workgroup takes the ranges the plan gives it (see plan.hpp) for one KV head; the 32-token tiles of a range are dealt
// to its four waves in contiguous runs, a wave keeps one online-softmax state per request its run touches, and the
// states meet in LDS when the range is done.
//
// Per 32-token tile a wave computes, with v_mfma_f32_16x16x32_bf16 (A: 16 rows x 32 k, B: 32 k x 16 columns;
// a lane holds row/column lane%16 and the 8 consecutive k of group lane/16):
//   S^T = K Q^T     A = K rows (row = token), B = the group's query heads (column = head, zero beyond G)
//   O^T += V^T P^T  A = V transposed in registers (row = output dim), B = softmax weights (column = head)
// With this orientation every lane owns one head (lane%16) in S^T, in P^T and in the O^T accumulators, so the
// running max, the rescale factor and the weights never cross lanes except for two max-exchanges per tile.
// The k-slots of a lane group may be bound to any 8 tokens / any 8 dims as long as both operands agree:
//   - for K Q^T the 8 k-slots of group j in step kk are dims (4kk+j)*8 .. +8: one 16-byte load per lane;
//   - for V^T P^T the 8 k-slots of group j are tokens {4j..4j+3, 16+4j..16+4j+3}, exactly the tokens whose scores
//     the S^T accumulators of that lane group hold, so P needs no data movement; V is loaded row-wise (a 256-byte
//     row per 16 lanes) and an 8x8 in-lane transpose (v_perm_b32) turns 8 rows x 8 dims into 8 operands.
// The weights go to the matrix core as bf16 hi + bf16 lo (two MFMAs), which keeps them to ~2^-16 relative; for caches
// with head_dim 64, whose products are half as many, as three bf16 parts that hold all 24 bits.  An fp32 cache uses
// v_mfma_f32_16x16x4_f32 for both products (fp32 operands and sums): its k-slot j in step (kk, e) of K Q^T is dim
// 4 (4kk + j) + e and in step r of V^T P^T token slot_token(j, r), so it loads and stages exactly as the 16-bit caches
// do and V needs no transposing at all.
// Measured against the vector-ALU kernel (fp32 FMAs and cross-lane sums: bound by the vector ALUs from four heads per KV
// head on, by a barrier per request below), with ranges as the unit of work (whole requests: at decode_mfma_kernel): 256 requests of a speech-token stage with 64-dim bf16 heads 81.2 -> 22.2 us per
// step (76 MB), four short fp32 requests 15.4 -> 10.9 us; fp32, 64 requests of 512 .. 4096 tokens (one pool): 16/4 heads of
// 128 dims 265.7 -> 109.3 us (K staged; 606 MB, 5.5 TB/s), 32/4 heads 390.2 -> 121.9 us (K not staged), 32/4 heads of 64
// dims 184.3 -> 57.0 us (303 MB, 5.3 TB/s).
// With T query tokens per request (kernel variant MT, T * G <= 16) a column is a (query token, head) pair instead of
// a head: it has its own query row, its own causal limit (tokens 0 .. L - T + i) and its own output row; everything
// that is said of a head above holds per column.  An 8-bit cache is widened to bf16 in registers.
#pragma once
#include "common.hpp"

namespace omni {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4_t mfma_bf16(const uint4 &a, const uint4 &b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2_t x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
}

__device__ __forceinline__ uint32_t dword_of(const uint4 &v, int w) {
    return w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
}

constexpr int kAppendFlag = 1 << 30;   // in a slot's tile word: the tile holds the token to append (fused decode step)

// token of k-slot r (0..7) of lane group j inside a 32-token tile
__device__ __forceinline__ int slot_token(int j, int r) { return (r < 4) ? 4 * j + r : 16 + 4 * j + (r - 4); }

// 8 E4M3 bytes (two dwords, dims ascending) -> 8 bf16 (exact: 4 significant bits fit in 8).
__device__ __forceinline__ uint4 fp8x8_to_bf16x8(uint32_t lo, uint32_t hi) {
    uint4 r;
    r.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false));
    r.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true));
    r.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false));
    r.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true));
    return r;
}

// What a KV cache holds: element type and head_dim, and what follows from them for one lane.
enum CacheFormat { kBf16D128, kFp8D128, kBf16D64, kF32D64, kF32D128 };

template <CacheFormat F>
struct CacheTraits {
    static constexpr bool kFp8 = F == kFp8D128, kF32 = F == kF32D64 || F == kF32D128;
    static constexpr int D = (F == kBf16D64 || F == kF32D64) ? 64 : 128;
    static constexpr int ES = kFp8 ? 1 : (kF32 ? 4 : 2);         // bytes per cache element
    static constexpr int kRowBytes = D * ES;                     // 128, 256 or 512
    static constexpr int kChunks = kRowBytes / 16;               // 16-byte chunks of a row
    static constexpr int kKRegs = kRowBytes / 64;                // chunks of one K row a lane takes
    static constexpr int kVDwords = kRowBytes / 64;              // dwords of one V row a lane takes ...
    static constexpr int kVWide = kFp8 ? 4 : kVDwords;           // ... and once widened to 16 bits
    static constexpr int kQRegs = D * (kF32 ? 4 : 2) / 64;       // 16-byte chunks of the query row a lane takes
    static constexpr int kBlocks = D / 16;                       // 16-dim blocks of output rows
    static constexpr int kStageBytes = kTile * kRowBytes;        // one 32-token K tile
};

// Loads of one 32-token tile.  pg0 / pg1 are the physical pages of its first / second 16 tokens (wave-uniform; with
// 32-token pages only pg0 is used).
//   K: lane (token = lane%16, group j) takes the row's chunks 4n + j (n < kKRegs), or, of an 8-bit cache, the 32 bytes
//      of dims 32j .. 32j+31 (MFMA step kk of group j then uses dims 32j + 8kk .. +8, and the query is bound the same way).
//   V: lane (c = lane%16, group j) takes 1/16 of each of the rows 4j .. 4j+3 and 16+4j .. 16+4j+3: dims 8c .. (128-dim
//      16-bit and 8-bit caches), 4c .. (64-dim caches), 4c .. and 64 + 4c .. (128-dim fp32).  Whole rows per instruction.
// The scales of an 8-bit cache's two pages ride along.
template <int PS, CacheFormat F>
struct TileLoader {
    using C = CacheTraits<F>;
    static constexpr int RB = C::kRowBytes, CH = C::kChunks, NK = C::kKRegs;
    const char *kbase, *vbase;       // pool base + KV-head offset
    const float *k_scale, *v_scale;  // 8-bit cache only: already offset by the KV head
    size_t page_stride;              // bytes between pages
    int Hkv;
    int koff;                        // byte offset of this lane's first K chunk inside a 16-token block
    int voff;                        // byte offset of this lane's first V row piece inside a 16-token block
    int kst_goff[NK];                // per lane: byte offset of the chunk it fetches in instruction r, inside a block
    int kst_roff[NK];                // per lane: byte offset of its n-th operand chunk inside a staged block

    __device__ __forceinline__ static int k_chunk(int n, int j) { return C::kFp8 ? 2 * j + n : 4 * n + j; }

    __device__ __forceinline__ void init(const AttnParams &p, int kvh, int lane) {
        const int i = lane & 15, j = lane >> 4;
        page_stride = (size_t)p.Hkv * PS * RB;
        kbase = reinterpret_cast<const char *>(p.k_cache) + (size_t)kvh * PS * RB;
        vbase = reinterpret_cast<const char *>(p.v_cache) + (size_t)kvh * PS * RB;
        k_scale = C::kFp8 ? p.k_scale + kvh : nullptr;
        v_scale = C::kFp8 ? p.v_scale + kvh : nullptr;
        Hkv = p.Hkv;
        koff = i * RB + k_chunk(0, j) * 16;
        voff = i * (RB < 512 ? RB / 16 : 16) + (4 * j) * RB;
        // K through shared memory: the operand layout puts four lanes on a token row, so loading it directly fetches every
        // cache line in pieces by several instructions, which keeps non-temporal loads from paying off for K.  Instead a
        // wave copies the tile's rows into its own part of shared memory with loads that cover whole rows (lane l of
        // instruction r: row r * 64 / CH + l / CH of the 16-token block, chunk (l % CH) ^ (row % CH), landing at 16 l behind
        // the instruction's base: the xor spreads a column of chunks over the banks), and reads its MFMA operands back from
        // there.  No register holds the tile while it is on its way.
#pragma unroll
        for (int r = 0; r < NK; ++r) {
            const int row = r * (64 / CH) + lane / CH;
            kst_goff[r] = row * RB + (((lane % CH) ^ (row % CH)) << 4);
            kst_roff[r] = i * RB + ((k_chunk(r, j) ^ (i % CH)) << 4);
        }
    }
    __device__ __forceinline__ size_t second_half(int pg0, int pg1) const {
        return PS == 16 ? (size_t)pg1 * page_stride : (size_t)pg0 * page_stride + 16 * RB;
    }
    __device__ __forceinline__ void load_k_scales(int pg0, int pg1, float (&ks)[2]) const {
        if constexpr (C::kFp8) { ks[0] = k_scale[(size_t)pg0 * Hkv]; ks[1] = k_scale[(size_t)(PS == 16 ? pg1 : pg0) * Hkv]; }
    }
    __device__ __forceinline__ void issue_k(int pg0, int pg1, uint4 (&K)[2 * NK], float (&ks)[2]) const {
        const char *k0 = kbase + (size_t)pg0 * page_stride + koff, *k1 = kbase + second_half(pg0, pg1) + koff;
#pragma unroll
        for (int n = 0; n < NK; ++n) {
            const int off = (k_chunk(n, 0) - k_chunk(0, 0)) * 16;
            if constexpr (C::kFp8) {                             // non-temporal loads lose on this pattern
                K[n] = *reinterpret_cast<const uint4 *>(k0 + off);
                K[NK + n] = *reinterpret_cast<const uint4 *>(k1 + off);
            } else {
                K[n] = nt_load16(k0 + off);
                K[NK + n] = nt_load16(k1 + off);
            }
        }
        load_k_scales(pg0, pg1, ks);
    }
    __device__ __forceinline__ void issue_k_half(const char *rows, uint4 *K) const {     // 16-bit and fp32 caches
#pragma unroll
        for (int n = 0; n < NK; ++n) K[n] = nt_load16(rows + koff + n * 64);
    }
    __device__ __forceinline__ void issue_k_staged(int pg0, int pg1, char *stage, float (&ks)[2]) const {
        const char *k0 = kbase + (size_t)pg0 * page_stride, *k1 = kbase + second_half(pg0, pg1);
#pragma unroll
        for (int r = 0; r < NK; ++r) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(k0 + kst_goff[r]),
                                             (__attribute__((address_space(3))) void *)(stage + r * 1024), 16, 0, 2);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(k1 + kst_goff[r]),
                                             (__attribute__((address_space(3))) void *)(stage + 16 * RB + r * 1024), 16, 0, 2);
        }
        load_k_scales(pg0, pg1, ks);
    }
    __device__ __forceinline__ void read_k_staged(const char *stage, uint4 (&K)[2 * NK]) const {
#pragma unroll
        for (int n = 0; n < NK; ++n) {
            K[n] = *reinterpret_cast<const uint4 *>(stage + kst_roff[n]);
            K[NK + n] = *reinterpret_cast<const uint4 *>(stage + 16 * RB + kst_roff[n]);
        }
    }
    __device__ __forceinline__ void read_k_staged_half(const char *stage, int half, uint4 *K) const {
#pragma unroll
        for (int n = 0; n < NK; ++n) K[n] = *reinterpret_cast<const uint4 *>(stage + half * (16 * RB) + kst_roff[n]);
    }
    __device__ __forceinline__ static void load_v_piece(const char *src, uint32_t (&v)[C::kVDwords]) {
        if constexpr (C::kVDwords == 2) {
            const uint2 x = nt_load8(src);
            v[0] = x.x; v[1] = x.y;
        } else {
#pragma unroll
            for (int h = 0; h < C::kVDwords / 4; ++h) {
                const uint4 x = nt_load16(src + h * 256);
                v[4 * h] = x.x; v[4 * h + 1] = x.y; v[4 * h + 2] = x.z; v[4 * h + 3] = x.w;
            }
        }
    }
    __device__ __forceinline__ void issue_v(int pg0, int pg1, uint32_t (&V)[8][C::kVDwords], float (&vs)[2]) const {
        const char *v0 = vbase + (size_t)pg0 * page_stride + voff, *v1 = vbase + second_half(pg0, pg1) + voff;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            load_v_piece(v0 + r * RB, V[r]);
            load_v_piece(v1 + r * RB, V[4 + r]);
        }
        if constexpr (C::kFp8) { vs[0] = v_scale[(size_t)pg0 * Hkv]; vs[1] = v_scale[(size_t)(PS == 16 ? pg1 : pg0) * Hkv]; }
    }
};

__device__ __forceinline__ f32x4_t mfma_f32(uint32_t a, uint32_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a), __uint_as_float(b), c, 0, 0, 0);
}

template <CacheFormat F>
struct MfmaState {
    float m, l;
    f32x4_t acc[CacheTraits<F>::kBlocks];    // acc[e][i] = O^T[dim of output row 4j + i of block e][column lane%16]
};

__device__ __forceinline__ f32x4_t rescale_add(const f32x4_t &acc, float alpha, const f32x4_t &t) {
    f32x4_t r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = fmaf(acc[i], alpha, t[i]);
    return r;
}

// The raw scores of one 16-token half of an fp32 tile.  A matrix instruction adds its products one after the other, so a
// chain over all dims rounds 64 or 128 partial sums one upon the other.  Each instruction starts from zero instead and the
// four-product sums are added as a tree, like the lanes of the vector-ALU kernel.  With the chains of mfma_softmax_pv this
// brings the error against 64 bits from 1.6 - 3.3 times that kernel's to 0.8 - 1.06 times (64 .. 2 requests of 17 .. 17000
// tokens, scores of deviation 1 and 4), for 11 % of the time over 128-dim rows (28/4 heads, 592 MB: 109 -> 123 us; the
// vector-ALU kernel takes 354) and 1 - 4 % over 64-dim rows.
template <CacheFormat F>
__device__ __forceinline__ f32x4_t mfma_scores_f32(const uint4 *K, const uint4 (&Q)[CacheTraits<F>::kQRegs]) {
    constexpr int N = CacheTraits<F>::kQRegs;
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    f32x4_t part[4], sum = zero;                                 // sums of 1, 2, 4 chunks that wait for their sibling
#pragma unroll
    for (int n = 0; n < N; ++n) {
        f32x4_t t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = mfma_f32(dword_of(K[n], e), dword_of(Q[n], e), zero);
        sum = (t[0] + t[1]) + (t[2] + t[3]);
        int b = 0;
#pragma unroll
        for (; n >> b & 1; ++b) sum = part[b] + sum;
        // the additions stay here: moved down to where the scores are used, their 128 operands would wait in registers
        if (n & 1) asm volatile("" : "+v"(sum));
        part[b] = sum;
    }
    return sum;
}

// First half of a 32-token tile: the scores S^T = K Q^T of the tile, in the log2 domain.  Bytes of an 8-bit cache are
// widened to bf16 right before each MFMA step, and the K scale of each 16-token half (ks) joins the softmax scale.
template <CacheFormat F>
__device__ __forceinline__ void mfma_scores(const uint4 (&K)[2 * CacheTraits<F>::kKRegs], const uint4 (&Q)[CacheTraits<F>::kQRegs],
                                            float (&sv)[8], float scale_log2, const float (&ks)[2]) {
    // Scores are rounded before the running max is subtracted (no fused multiply-subtract): s - max is then exactly
    // 0 for the maximal score, and a length-1 context returns its V row bit for bit.
#pragma clang fp contract(off)
    using C = CacheTraits<F>;
    constexpr int NK = C::kKRegs;
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
    if constexpr (C::kF32) { s0 = mfma_scores_f32<F>(K, Q); s1 = mfma_scores_f32<F>(K + NK, Q); }
#pragma unroll
    for (int n = 0; n < (C::kF32 ? 0 : C::kQRegs); ++n) {
        if constexpr (C::kFp8) {
            const uint4 &a = K[n >> 1], &b = K[NK + (n >> 1)];
            const uint4 A0 = (n & 1) ? fp8x8_to_bf16x8(a.z, a.w) : fp8x8_to_bf16x8(a.x, a.y);
            const uint4 A1 = (n & 1) ? fp8x8_to_bf16x8(b.z, b.w) : fp8x8_to_bf16x8(b.x, b.y);
            s0 = mfma_bf16(A0, Q[n], s0);
            s1 = mfma_bf16(A1, Q[n], s1);
        } else if constexpr (C::D == 64) {       // each from zero, as in mfma_scores_f32: error 1.15 -> 1.03 times
            const f32x4_t none = {0.f, 0.f, 0.f, 0.f};
            s0 += mfma_bf16(K[n], Q[n], none);
            s1 += mfma_bf16(K[NK + n], Q[n], none);
        } else {
            s0 = mfma_bf16(K[n], Q[n], s0);
            s1 = mfma_bf16(K[NK + n], Q[n], s1);
        }
    }
    const float c0 = C::kFp8 ? ks[0] * scale_log2 : scale_log2, c1 = C::kFp8 ? ks[1] * scale_log2 : scale_log2;
#pragma unroll
    for (int i = 0; i < 4; ++i) { sv[i] = s0[i] * c0; sv[4 + i] = s1[i] * c1; }
}

// Two floats' upper halves as a pair of bf16 (truncated).
__device__ __forceinline__ uint32_t upper_halves(float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ float below_upper_half(float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

// Each half of `part` (bf16, not negative), or 2^-40 of the same half of `first` if that is more: never zero where `first` is
// 2^-86 or more.
__device__ __forceinline__ uint32_t at_least_a_trace(uint32_t part, uint32_t first) {
    typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
    const u16x2_t f = __builtin_bit_cast(u16x2_t, first), shift = {40 << 7, 40 << 7};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, part), __builtin_elementwise_sub_sat(f, shift)));
}

// The eight weights of a lane as bf16 MFMA operands whose sum is the weight: two parts to ~2^-16 relative (rounded), or
// three that hold all 24 bits (each the upper half of what the parts before it left, so nothing is rounded).  kTrace: a
// lower part that has nothing left is 2^-40 of the weight instead of zero, so that an infinite V element times it is
// infinite like its product with the first part and not NaN.
template <int kParts, bool kTrace = false>
__device__ __forceinline__ void split_weights(const float (&pw)[8], uint4 (&P)[kParts]) {
#pragma clang fp contract(off)
    uint32_t d[kParts][4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float a = pw[2 * w], b = pw[2 * w + 1];
        if constexpr (kParts == 2) {
            d[0][w] = pack_bf16x2(a, b);
            d[1][w] = pack_bf16x2(a - bf16_bits_to_float(d[0][w] & 0xffffu), b - __uint_as_float(d[0][w] & 0xffff0000u));
        } else {
            d[0][w] = upper_halves(a, b);
            const float a1 = below_upper_half(a), b1 = below_upper_half(b);
            d[1][w] = upper_halves(a1, b1);
            d[2][w] = upper_halves(below_upper_half(a1), below_upper_half(b1));
            if constexpr (kTrace) { d[1][w] = at_least_a_trace(d[1][w], d[0][w]); d[2][w] = at_least_a_trace(d[2][w], d[0][w]); }
        }
    }
#pragma unroll
    for (int i = 0; i < kParts; ++i) P[i] = make_uint4(d[i][0], d[i][1], d[i][2], d[i][3]);
}

// Second half: online softmax over the tile's scores and the weighted V accumulation O^T += V^T P^T.
// `vs0` / `vs1` scale the weights of the tile's first / second 16 tokens on their way into the product (the V scales of
// an 8-bit cache): the sum of weights stays unscaled.
// t1: the request's length; t1col: tokens this lane's column may see (t1 less the query tokens after its own; = t1 in
// plain decode); t1min: the smallest t1col of the wave's columns.
// kMulti (several query tokens per request): the three differ; otherwise all are t1.
// kAllBits: weights keep 24 bits whatever the format.
template <CacheFormat F, bool kMulti, bool kAllBits>
__device__ __forceinline__ void mfma_softmax_pv(float (&sv)[8], uint32_t (&V)[8][CacheTraits<F>::kVWide], MfmaState<F> &st,
                                                int tb, int t1, int t1col, int t1min, int j, float vs0, float vs1) {
#pragma clang fp contract(off)
    using C = CacheTraits<F>;
    auto drop_v = [&](int r) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < C::kVWide; ++w) V[r][w] = 0;
    };
    if (tb + 32 > (kMulti ? t1min : t1)) {               // last tiles of the request (uniform branch)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (kMulti) {
                if (tb + slot_token(j, r) >= t1col) sv[r] = -INFINITY;      // not visible to this column
                if (tb + slot_token(j, r) >= t1) drop_v(r);
            } else if (tb + slot_token(j, r) >= t1) {    // unowned slot: its K/V bits are arbitrary, possibly NaN
                sv[r] = -INFINITY;
                drop_v(r);
            }
        }
    }
    float tmax = sv[0];
#pragma unroll
    for (int r = 1; r < 8; ++r) tmax = fmaxf(tmax, sv[r]);
    tmax = across_lane_groups(tmax, [](float a, float b) { return fmaxf(a, b); });
    // finite: in plain decode every tile holds a live token; with several query tokens a column may see none of a
    // tile's, and then keeps a finite stand-in
    const float mn = kMulti ? fmaxf(fmaxf(st.m, tmax), kNoTokenReference) : fmaxf(st.m, tmax);
    const float alpha = fast_exp2(st.m - mn);
    float pw[8], psum = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) { pw[r] = fast_exp2(sv[r] - mn); psum += pw[r]; }
    st.l = st.l * alpha + psum;
    st.m = mn;
    if constexpr (C::kFp8) {
#pragma unroll
        for (int r = 0; r < 4; ++r) { pw[r] *= vs0; pw[4 + r] *= vs1; }
    }
    const f32x4_t none = {0.f, 0.f, 0.f, 0.f};
    if constexpr (C::kF32) {
        // a tile's sum in two chains (four over 64 dims), each as long as a lane group's in the vector-ALU kernel, and one
        // rounding where it joins the sum of the tiles before
        constexpr int kChains = C::D == 128 ? 2 : 4, kLength = 8 / kChains;
#pragma unroll
        for (int e = 0; e < C::kBlocks; ++e) {
            f32x4_t t[kChains];
#pragma unroll
            for (int c = 0; c < kChains; ++c) {
                t[c] = none;
#pragma unroll
                for (int r = 0; r < kLength; ++r) t[c] = mfma_f32(V[c * kLength + r][e], __float_as_uint(pw[c * kLength + r]), t[c]);
            }
            st.acc[e] = rescale_add(st.acc[e], alpha, kChains == 2 ? t[0] + t[1] : (t[0] + t[1]) + (t[kChains - 2] + t[kChains - 1]));
            if constexpr (C::D == 128) { if (e & 1) asm volatile("" : "+v"(st.acc[e]), "+v"(st.acc[e - 1])); }   // two blocks at a time
        }
    } else {
        constexpr int kParts = C::D == 64 || kAllBits ? 3 : 2;
        uint4 P[kParts];
        split_weights<kParts, true>(pw, P);
        if constexpr (kParts == 2) {
#pragma unroll
            for (int e = 0; e < C::kBlocks; ++e) st.acc[e] *= alpha;
        }
        // in-lane transpose: operand e holds dim e of the lane's chunk for the 8 tokens of its lane group
        // (dword w of V[r] holds dims 2w and 2w+1 of token slot r)
#pragma unroll
        for (int e = 0; e < C::kBlocks; ++e) {
            const int w = e >> 1;
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            uint4 A;
            A.x = __builtin_amdgcn_perm(V[1][w], V[0][w], sel);
            A.y = __builtin_amdgcn_perm(V[3][w], V[2][w], sel);
            A.z = __builtin_amdgcn_perm(V[5][w], V[4][w], sel);
            A.w = __builtin_amdgcn_perm(V[7][w], V[6][w], sel);
            if constexpr (kParts == 2) {
#pragma unroll
                for (int i = 0; i < kParts; ++i) st.acc[e] = mfma_bf16(A, P[i], st.acc[e]);
            } else {                                             // the tile's sum first, from its smallest part up
                f32x4_t t = none;
#pragma unroll
                for (int i = kParts - 1; i >= 0; --i) t = mfma_bf16(A, P[i], t);
                st.acc[e] = rescale_add(st.acc[e], alpha, t);
            }
        }
    }
}

constexpr int kMaxStates = 16;                         // states the ring holds at most
constexpr int kKStageBytes = 8192;                     // one 32-token K tile of 256-byte rows

// Shared-memory layout for a batch of B requests and G columns per KV head: as many states (up to sixteen) as fit
// while two workgroups still share the 160 KB of a compute unit.  Four is the least the kernel works with (one state
// per wave: one request at a time); where not even four fit beside the plan's arrays (thousands of requests with 16
// columns), the layout keeps four and `two_per_cu` is false: the launch is still valid, with one workgroup per
// compute unit.
constexpr int kLdsPerWorkgroup = 80 * 1024 - 512;      // half a compute unit's shared memory less the kernel's own variables
constexpr MfmaLds mfma_lds_layout(int B, int G, int D, int row_bytes, bool staged, bool query_counts = false, int max_states = kMaxStates) {
    MfmaLds L{};
    L.ring_off = (((query_counts ? 3 : 2) * B + 1) * 4 + 15) & ~15;      // E[B + 1], Lc[B] and, if asked for, Nc[B]
    L.state_floats = G * (D + 4) + 2 * kMaxGroup;
    L.static_bytes = staged ? kWaves * kTile * row_bytes : 0;          // the waves' K tiles
    const int budget = kLdsPerWorkgroup - L.ring_off - L.static_bytes;
    const int cap = budget / (L.state_floats * 4);
    L.two_per_cu = cap >= kWaves;
    L.ring_states = cap > max_states ? max_states : (cap < kWaves ? kWaves : cap);
    L.total = L.ring_off + L.ring_states * L.state_floats * 4;
    return L;
}

// A range (or a chunk of it) of `clen` tiles is dealt to the four waves in contiguous runs: wave w takes tiles
// run_start(w) .. run_start(w + 1) - 1 of the chunk.  With fewer than four tiles, waves 0 .. clen - 1 take one each.
__device__ __forceinline__ int run_start(int clen, int w) { return clen >= kWaves ? (clen * w) >> 2 : min(w, clen); }
// The wave whose run holds tile x of the chunk (0 <= x < clen).
__device__ __forceinline__ int wave_of_tile(int clen, int x) {
    return (x >= run_start(clen, 1)) + (x >= run_start(clen, 2)) + (x >= run_start(clen, 3));
}

// Combine the `cnt` consecutive states (m, l, o) that the waves left for one request's piece of a chunk and store the
// result: the normalised output if the request lies inside one range, else the unnormalised values (plus, once per
// head, the running max and sum) into the piece's partial-result slot.  Every thread owns four consecutive output
// elements.  All threads call it between barriers.
template <int D, bool MT>
__device__ __forceinline__ void mfma_combine_states(const float *first, int cnt, int state_floats, const AttnParams &p,
                                                    const Segment &seg, int kvh, int n_tokens = 1) {
    const int G = MT ? p.Gq : p.G;                       // columns: (query token, head) pairs of the KV head
    for (int idx = 4 * threadIdx.x; idx < G * D; idx += 4 * kThreads) {
        const int g = idx / D, d = idx - g * D;
        // a request's piece lies in at most four runs: all four reads are issued before any is used (a state that is
        // not part of the piece is read from the first one and dropped)
        float mu[kWaves], lu[kWaves];
        float4 ou[kWaves];
#pragma unroll
        for (int u = 0; u < kWaves; ++u) {
            const float *st = first + (u < cnt ? u : 0) * state_floats;
            mu[u] = st[G * (D + 4) + g];
            lu[u] = st[G * (D + 4) + kMaxGroup + g];
            ou[u] = *reinterpret_cast<const float4 *>(st + g * (D + 4) + d);
        }
        float M = -INFINITY;
#pragma unroll
        for (int u = 0; u < kWaves; ++u) {
            if (u >= cnt) mu[u] = -INFINITY;
            M = fmaxf(M, mu[u]);
        }
        float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
        float den = 0.f;
#pragma unroll
        for (int u = 0; u < kWaves; ++u) {
            if (mu[u] > -INFINITY) {
                const float a = fast_exp2(mu[u] - M);
                num.x += a * ou[u].x; num.y += a * ou[u].y; num.z += a * ou[u].z; num.w += a * ou[u].w;
                den += a * lu[u];
            }
        }
        if (MT && p.t_off + g / p.G >= n_tokens) {           // no query token behind this column: zeros, weight 0
            num = make_float4(0.f, 0.f, 0.f, 0.f);
            den = 0.f;
        }
        if (seg.nparts == 1) {
            const size_t o0 = (MT ? out_row(p, seg.b, kvh, g) : (size_t)seg.b * p.Hq + kvh * G + g) * D + d;
            const bool live = den > 0.f;
            store_out4(p, o0, make_float4(live ? num.x / den : 0.f, live ? num.y / den : 0.f, live ? num.z / den : 0.f,
                                          live ? num.w / den : 0.f));
        } else {
            const size_t pi = MT ? partial_row(p, seg.slot, kvh, g) : (size_t)seg.slot * p.Hq + kvh * G + g;
            *reinterpret_cast<float4 *>(p.ws.part_o + pi * D + d) = num;
            if (d == 0) p.ws.part_ml[pi] = make_float2(M, den);
        }
    }
}

// Workgroups that run on a compute unit where each takes a request whole: with four states and no plan in shared memory, and
// without the plan in registers, more of them fit than where ranges are taken.
constexpr int whole_workgroups_per_cu(CacheFormat F) { return F == kBf16D64 ? 4 : F == kFp8D128 ? 3 : 2; }

// The tiles of a range are dealt to the four waves in contiguous runs, so a wave holds one online-softmax state per
// request its run touches: four states plus one per request boundary that falls inside a run, whatever the number
// of requests (dealt round-robin, every request would leave four).  A wave leaves each finished state in shared memory
// and goes on; the workgroup meets once, when the range is done: one barrier, then every thread combines, request by
// request, the one to four consecutive states that belong to it.  A range that holds more requests than the states'
// area has room for (all but three of its states) is taken in chunks of that many requests, with the same meeting
// after each chunk.
// F: what the pools hold (an 8-bit cache has one scale per (page, KV head); its queries stay bf16).
// KST: K tiles go through the per-wave staging area in shared memory (the host chooses it where room for enough
// states is left beside it); otherwise they are loaded straight into the operand registers.
// MT: several query tokens per request (the columns are (query token, head) pairs with a causal limit each); the
// one-token kernel is compiled without any of it.
// WHOLE: a workgroup takes one request whole (request w for workgroup w of a KV head), for batches of short contexts.  Nothing
// is cut, so there is nothing to plan and no merge launch behind it, and the request's table row, its length and its query
// are asked for at once: two trips to memory before the first scores where the plan makes them three or four.
// Four fp32 requests of 17 .. 200 tokens 11.2 -> 7.5 us per step, 256 speech-token requests of 129 .. 1025 tokens, 16/2 heads,
// 34.0 -> 31.5 us (64-dim heads 22.1 -> 18.1 us).
template <int PS, CacheFormat F, bool KST, bool MT, bool WHOLE = false>
__global__ __launch_bounds__(kThreads, WHOLE ? whole_workgroups_per_cu(F) : 2) void decode_mfma_kernel(AttnParams p) {
    using C = CacheTraits<F>;
    constexpr int D = C::D, RB = C::kRowBytes;
    // A request's largest weights are exactly one in every state that holds them, so the fewer states of a whole request made
    // 16-bit weights 1.02 - 1.15 times as far from 64 bits over contexts of 17 .. 760 tokens.  All 24 bits instead: 0.08 -
    // 0.76 times as far, for 1 % (256 requests of 129 .. 1025 tokens 29.35 -> 29.72 us) to 6 % (few of 512) of the step.  Over
    // an 8-bit cache a page's scale multiplies the weights first and the distance stays what it was (0.97 - 1.01).
    constexpr bool kAllBits = WHOLE && !C::kFp8;
    constexpr int kLog2Ps = (PS == 16) ? 4 : 5;
    __shared__ PlanSmem ps;
    extern __shared__ __align__(16) int E[];                 // E[B + 1] tile offsets, then Lc[B] lengths, then the ring
    __shared__ __align__(16) char kstage_all[KST ? kWaves * C::kStageBytes : 16];  // a K tile per wave
    float *ring = reinterpret_cast<float *>(reinterpret_cast<char *>(E) + p.lds.ring_off);
    const int state_floats = p.lds.state_floats;
    const int max_seg = p.lds.ring_states - (kWaves - 1);    // requests a chunk may hold: the states then fit

    int w, kvh;
    if constexpr (WHOLE) wg_coords_whole(p, &w, &kvh); else wg_coords(p, &w, &kvh);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, j = lane >> 4;
    const int G = p.G, Gq = MT ? p.Gq : G;                       // heads per KV head; columns = query tokens x heads
    const int head0 = kvh * G;
    const int col_qi = (MT && col < Gq) ? col / G : 0;           // this lane's column: query token, head, and how many
    const int col_g = col - col_qi * G;                          // of the request's newest tokens it must not see
    const int tokens = MT ? p.Tq : 1;                            // query tokens per request, t_off .. in this launch
    const int t_off = MT ? p.t_off : 0;
    const int col_tok = t_off + col_qi;                          // which of the request's query tokens

    TileLoader<PS, F> ld;
    ld.init(p, kvh, lane);
    char *kstage = kstage_all + (KST ? wave * C::kStageBytes : 0);

    // Several query tokens per request: Nc[b] = how many request b brings (behind E[] and Lc[] in shared memory).
    const int nb_plan = WHOLE ? 1 : p.plan.B;                    // requests the arrays in shared memory describe ...
    int *Nc = E + 2 * nb_plan + 1;
    const int b0 = WHOLE ? w : 0;                                // ... from this one on
    auto load_q = [&](int b, uint4 (&Q)[C::kQRegs]) {            // B operand of K Q^T for request b
#pragma unroll
        for (int n = 0; n < C::kQRegs; ++n) Q[n] = make_uint4(0, 0, 0, 0);
        if (col < Gq && (!MT || t_off + col_qi < Nc[b])) {       // a column no query token stands behind keeps zeros
            const char *qrow = reinterpret_cast<const char *>(p.q) + (((size_t)(b0 + b) * tokens + t_off + col_qi) * p.Hq + head0 + col_g) * (D * (C::kF32 ? 4 : 2));
#pragma unroll
            for (int n = 0; n < C::kQRegs; ++n)                 // the dims that meet the lane's K chunks
                Q[n] = *reinterpret_cast<const uint4 *>(qrow + (C::kFp8 ? 4 * j + n : 4 * n + j) * 16);
        }
    };

    // Tile offsets and lengths of all requests, in shared memory.
    const int *Lc = E + nb_plan + 1;
    const bool wave_plan = WHOLE || p.plan.B <= kWavePlanMax;    // small batch: every wave plans for itself, no barrier
    WavePlan wp{0, 0, 0, 0};
    Plan pl;
    int tab0 = 0, tab1 = 0;                                      // WHOLE: the table's entries for tile `lane`
    uint4 Qw[C::kQRegs];
    if constexpr (WHOLE) {
        constexpr int kEntries = kTile / PS;
        const int32_t *bt = p.block_table + (size_t)b0 * p.MB;
        if (lane * kEntries < p.MB) tab0 = bt[lane * kEntries];
        if (kEntries == 2 && lane * kEntries + 1 < p.MB) tab1 = bt[lane * kEntries + 1];
        const int L = max(p.context_lens[b0], 0);
        const int n = MT ? (p.q_lens ? p.q_lens[b0] : tokens) : 1;
        E[0] = 0; E[1] = (L + kTile - 1) >> kLog2Tile; E[2] = L;     // every wave writes the same values: no barrier needed
        if constexpr (MT) Nc[0] = min(max(n, 0), tokens);
        pl.C = __builtin_amdgcn_readfirstlane((L + kTile - 1) >> kLog2Tile);
        pl.S = max(pl.C, 1);
        pl.nranges = pl.C > 0 ? 1 : 0;
        load_q(0, Qw);
        if (pl.C == 0 && wave == 0) wave_zero_rows<D>(p, b0, kvh);
    } else if (wave_plan) {
        unsigned long long T = 0;
        const bool first = blockIdx.x == 0 && wave == 0;
        pl = plan_build_wave(p.context_lens, p.plan, E, E + p.plan.B + 1, &wp, w == 0 && wave == 0,
                             [&](int b) { wave_zero_rows<D>(p, b, kvh); }, first, T);
        if (first && lane == 0) {
            p.ws.plan_words[0] = pl.S * kTile; p.ws.plan_words[1] = pl.nranges;
            p.ws.plan_words[2] = (int)(T & 0xffffffffULL); p.ws.plan_words[3] = (int)(T >> 32);
        }
    } else {
        pl = attn_prologue<D>(p, &ps, E, w, kvh);
    }
    if constexpr (MT && !WHOLE) {                                // every wave writes the same values: no barrier needed
        for (int b = lane; b < p.plan.B; b += 64) {
            const int n = p.q_lens ? p.q_lens[b] : tokens;
            Nc[b] = min(max(n, 0), tokens);
        }
    }

    for (int range = WHOLE ? 0 : w; range < pl.nranges; range += WHOLE ? 1 : p.plan.nw) {
        const int start = range * pl.S, end = min(pl.C, start + pl.S);
        int cs = start;                  // first tile of the chunk
        int cb = WHOLE ? 0 : wave_plan ? wave_first_request(wp, start) : plan_first_request(p.plan, &ps, E, start);   // its request
      while (cs < end) {                 // chunks of the range: normally one
        // ---- the chunk: up to max_seg requests from tile cs on; nb = the request the next chunk starts with
        int ce = end, nb = cb;
        // (with the plan in registers the common case needs no walk: the requests up to the one that holds the range's
        // last tile, empty ones included, are no more than a chunk may hold)
        if (!WHOLE && !(wave_plan && wave_first_request(wp, end - 1) - cb < max_seg)) {
            int bb = cb;
            for (int nseg = 1;; ++nseg) {
                const int e1 = __builtin_amdgcn_readfirstlane(E[bb + 1]);
                if (e1 >= end) break;                            // the request reaches the end of the range
                do { ++bb; } while (__builtin_amdgcn_readfirstlane(E[bb + 1]) == __builtin_amdgcn_readfirstlane(E[bb]));   // next request that owns tiles (one exists: e1 < C)
                if (nseg == max_seg) { ce = e1; nb = bb; break; }
            }
        }
        const int clen = ce - cs;
        const int r0 = run_start(clen, wave), nk = run_start(clen, wave + 1) - r0;     // this wave's run of the chunk's tiles
        const int first_b = cb;
        // the request that holds the chunk's last tile bounds every lane's search below: a chunk rarely spans more than
        // two or three requests, so the search takes one or two steps instead of log2(B)
        const int search_hi = WHOLE ? 1 : wave_plan ? wave_first_request(wp, ce - 1) + 1 : p.plan.B;

        // ---- this wave's tiles: tile r0 + slot of the chunk, slot = 0 .. nk-1.  Lane s of the wave looks up
        // everything about slot s (of the current group of 64 slots) once: the request, the tile's index inside the
        // request and its physical pages.  The tile loop then only picks values out with v_readlane, so neither the
        // block table nor the plan sits between two tiles, also across request boundaries.
        int4 meta = make_int4(-1, 0, 0, 0);                      // request, tile in request, page of tokens 0-15, 16-31
        auto fetch_meta = [&](int first_slot) {
            const int slot = first_slot + lane;
            meta = make_int4(-1, 0, 0, 0);
            if (slot < nk) {
                const int pos = cs + r0 + slot;
                int lo = first_b, hi = search_hi;                // E[lo] <= pos < E[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (E[mid] <= pos) lo = mid; else hi = mid;
                }
                const int t = pos - E[lo];
                const int last_page = (Lc[lo] - 1) >> kLog2Ps;
                const int32_t *bt = p.block_table + (size_t)lo * p.MB;
                const int page = (t * kTile) >> kLog2Ps;
                meta.x = lo;
                // fused step: the tiles that hold the request's newest token(s) get their rows written first
                bool newest = t == ((Lc[lo] - 1) >> kLog2Tile);
                if (MT) newest = Nc[lo] > 0 && t <= ((Lc[lo] - 1) >> kLog2Tile) && t >= (max(Lc[lo] - Nc[lo], 0) >> kLog2Tile);
                meta.y = t | ((p.k_new != nullptr && newest) ? kAppendFlag : 0);
                if (PS == 16 && page < last_page) {              // both pages exist: one 8-byte read (page is even)
                    struct alignas(4) PagePair { int first, second; };   // rows of odd length keep 4-byte alignment
                    const PagePair pp2 = *reinterpret_cast<const PagePair *>(bt + page);
                    meta.z = pp2.first; meta.w = pp2.second;
                } else {                                         // never read beyond the request's pages
                    meta.z = bt[page]; meta.w = meta.z;
                }
            }
        };
        if constexpr (!WHOLE) fetch_meta(0);
        struct SlotInfo { int req, tile, pg0, pg1; bool append; };
        auto slot_info = [&](int slot) {
            SlotInfo si{-1, 0, 0, 0, false};
            if (slot >= nk) return si;
            if constexpr (WHOLE) {
                const int L = __builtin_amdgcn_readfirstlane(Lc[0]), last_page = (L - 1) >> kLog2Ps;
                si.req = 0; si.tile = r0 + slot;
                if (si.tile < 64) {
                    si.pg0 = __builtin_amdgcn_readlane(tab0, si.tile);
                    si.pg1 = __builtin_amdgcn_readlane(tab1, si.tile);
                } else {                                         // longer than the bound the caller gave
                    const int32_t *bt = p.block_table + (size_t)b0 * p.MB + si.tile * (kTile / PS);
                    si.pg0 = bt[0];
                    si.pg1 = PS == 16 && ((si.tile * kTile) >> kLog2Ps) < last_page ? bt[1] : 0;
                }
                if (PS == 32 || ((si.tile * kTile) >> kLog2Ps) >= last_page) si.pg1 = si.pg0;       // never an entry beyond the request's pages
                bool newest = si.tile == ((L - 1) >> kLog2Tile);
                if (MT) {
                    const int n = __builtin_amdgcn_readfirstlane(Nc[0]);
                    newest = n > 0 && si.tile <= ((L - 1) >> kLog2Tile) && si.tile >= (max(L - n, 0) >> kLog2Tile);
                }
                si.append = p.k_new != nullptr && newest;
                return si;
            }
            if ((slot & 63) == 0 && slot > 0) fetch_meta(slot);  // rare: more than 64 tiles per wave in a range
            const int l = slot & 63;
            const int ty = __builtin_amdgcn_readlane(meta.y, l);
            si.req = __builtin_amdgcn_readlane(meta.x, l); si.tile = ty & ~kAppendFlag; si.append = (ty & kAppendFlag) != 0;
            si.pg0 = __builtin_amdgcn_readlane(meta.z, l); si.pg1 = __builtin_amdgcn_readlane(meta.w, l);
            return si;
        };
        // Fused decode step, with several query tokens per request or K loaded straight into registers: the tile that
        // holds the request's last token gets the new K/V row written into its page (a bit copy, the first lanes the K
        // row, the next ones the V row, 16 bytes each) before the tile is requested; the wave waits for the write to be
        // acknowledged, so the loads that follow see it.  With several query tokens per request the new rows are
        // [B, T, Hkv, D] and each tile takes those of the request's last T positions that fall into it.
        constexpr int kRowPieces = C::kChunks;                   // 16-byte pieces of a row
        auto append_row = [&](const SlotInfo &si) {
            const int L = Lc[si.req];
            const int n_new = MT ? Nc[si.req] : 1;               // rows 0 .. n_new - 1 of the request's new rows
#pragma unroll 1
            for (int qi = 0; qi < n_new; ++qi) {
                const int pos = L - n_new + qi;
                if (MT && (pos < 0 || (pos >> kLog2Tile) != si.tile)) continue;      // uniform
                const int pg = (PS == 16 && (pos & 16)) ? si.pg1 : si.pg0;
                const size_t row = (size_t)pg * ld.page_stride + (size_t)(pos & (PS - 1)) * RB;
                if (lane < 2 * kRowPieces) {
                    const bool is_v = lane >= kRowPieces;
                    const int piece = lane & (kRowPieces - 1);
                    const char *src = reinterpret_cast<const char *>(is_v ? p.v_new : p.k_new) +
                                      (((size_t)(b0 + si.req) * tokens + qi) * p.Hkv + kvh) * RB + piece * 16;
                    char *dst = const_cast<char *>(is_v ? ld.vbase : ld.kbase) + row + piece * 16;
                    *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_s_waitcnt(0);           // all counters: the row is in memory before the tile is read
        };
        // One query token per request and K staged: no wait at all.  The new rows are asked for together with the
        // tile's loads (every lane one 16-byte piece of each); when the tile has arrived the K row is written over its
        // place in the staging area, the V row over the registers of the lanes that hold that token, and both go to
        // their page with stores nobody waits for: within this launch only this wave reads that row of that KV head.
        constexpr bool kPatchAppend = KST && !MT;
        int patch_row = -1;                                      // the new token's place in the tile in flight, or none
        size_t patch_dst = 0;                                    // byte offset of its row behind kbase / vbase
        uint4 Kn = make_uint4(0, 0, 0, 0);
        uint32_t Vn[C::kVDwords] = {};
        constexpr int kVStep = RB < 512 ? RB / 16 : 16;          // a lane's V piece: 8 or 16 bytes, or two of 16, 256 apart
        auto load_v_new = [&](const char *src, uint32_t (&v)[C::kVDwords]) __attribute__((always_inline)) {
            if constexpr (C::kVDwords == 2) {
                const uint2 x = *reinterpret_cast<const uint2 *>(src);
                v[0] = x.x; v[1] = x.y;
            } else {
#pragma unroll
                for (int h = 0; h < C::kVDwords / 4; ++h) {
                    const uint4 x = *reinterpret_cast<const uint4 *>(src + h * 256);
                    v[4 * h] = x.x; v[4 * h + 1] = x.y; v[4 * h + 2] = x.z; v[4 * h + 3] = x.w;
                }
            }
        };
        auto request_new_row = [&](const SlotInfo &si) {
            const int pos = __builtin_amdgcn_readfirstlane(Lc[si.req]) - 1;
            patch_row = pos - si.tile * kTile;
            const int pg = (PS == 16 && (pos & 16)) ? si.pg1 : si.pg0;
            patch_dst = (size_t)pg * ld.page_stride + (size_t)(pos & (PS - 1)) * RB;
            const size_t src = ((size_t)(b0 + si.req) * p.Hkv + kvh) * RB;
            Kn = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(p.k_new) + src + (lane & (kRowPieces - 1)) * 16);
            const char *vsrc = reinterpret_cast<const char *>(p.v_new) + src + col * kVStep;
            load_v_new(vsrc, Vn);
        };

        // Software pipeline of one wave (single K and V buffers): the K rows of the next tile are requested as soon
        // as the scores of the current tile have consumed K, its V rows as soon as the accumulation has consumed V,
        // and the next request's query as soon as the last scores of the current request are done.  The requests
        // stay in flight across the end-of-segment exchange below.
        // 512-byte rows: with both halves' staged K operands, V and the query in registers at once the kernel spills 30 of
        // them, so the halves take turns
        constexpr bool kHalves = KST && RB == 512;
        uint4 K[kHalves ? C::kKRegs : 2 * C::kKRegs], Q[C::kQRegs];
        uint32_t Vr[8][C::kVDwords];     // V rows as they are stored
        float ks[2] = {1.f, 1.f}, vs[2] = {1.f, 1.f};            // 8-bit cache: the scales of the tile's two pages
        auto issue_k = [&](int pg0, int pg1) __attribute__((always_inline)) {
            if constexpr (KST) ld.issue_k_staged(pg0, pg1, kstage, ks); else ld.issue_k(pg0, pg1, K, ks);
        };
        auto issue_v = [&](int pg0, int pg1) __attribute__((always_inline)) { ld.issue_v(pg0, pg1, Vr, vs); };
        int s = 0;                       // slot being computed; its loads are in flight
        SlotInfo cur = slot_info(0);
        if (cur.req >= 0) {
            if (cur.append) { if constexpr (kPatchAppend) request_new_row(cur); else append_row(cur); }
            issue_k(cur.pg0, cur.pg1);
            if constexpr (WHOLE) {
#pragma unroll
                for (int n = 0; n < C::kQRegs; ++n) Q[n] = Qw[n];
            } else {
                load_q(cur.req, Q);
            }
            issue_v(cur.pg0, cur.pg1);
        }
        __builtin_amdgcn_sched_barrier(0);       // nothing below may move in front of the first tile's loads

        // where this wave's states go: behind those of the waves before it (one per wave with a run, and one more for
        // every request that begins inside a run); worked out while the first tile is on its way
        int wbase = 0;
        for (int ww = 0; ww < wave; ++ww) wbase += run_start(clen, ww + 1) > run_start(clen, ww) ? 1 : 0;
        if constexpr (WHOLE) {           // no boundaries
        } else if (wave_plan) {          // from the plan in registers: the boundaries in front of this wave's run ...
            const int mine = run_start(clen, wave);
            wbase += wave_count_ends(wp, cs, cs + mine);
            for (int ww = 1; ww < wave; ++ww)                    // ... less those a run begins with
                if (run_start(clen, ww) < mine) wbase -= wave_count_ends(wp, cs + run_start(clen, ww) - 1, cs + run_start(clen, ww) + 1);
        } else {
            int bb = cb;
            while (true) {
                const int e1 = __builtin_amdgcn_readfirstlane(E[bb + 1]) - cs;   // where the next request begins, in the chunk
                if (e1 >= clen) break;
                const int ww = wave_of_tile(clen, e1);
                if (ww < wave && e1 != run_start(clen, ww)) ++wbase;
                do { ++bb; } while (__builtin_amdgcn_readfirstlane(E[bb + 1]) == __builtin_amdgcn_readfirstlane(E[bb]));
            }
        }
        int nstate = 0;                  // states this wave has left in shared memory for this chunk
        while (cur.req >= 0) {           // one pass per request the wave's run touches
            const int b = cur.req;
            const Segment seg = plan_segment(E, Lc, pl, b, range, start, end);
            // several query tokens: query i of the request's n sits at position L - n + i; a column with no query behind
            // it runs unmasked on zero queries and is dropped when the segment is combined
            const int seg_n = MT ? __builtin_amdgcn_readfirstlane(Nc[b]) : 1;
            const int col_back = (MT && col < Gq && col_tok < seg_n) ? seg_n - 1 - col_tok : 0;
            const int t1min = MT ? seg.L - max(seg_n - 1 - t_off, 0) : seg.L;
            MfmaState<F> st;
            st.m = -INFINITY; st.l = 0.f;
#pragma unroll
            for (int e = 0; e < C::kBlocks; ++e) st.acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            while (cur.req == seg.b) {
                const SlotInfo nxt = slot_info(s + 1);
                const bool more = nxt.req >= 0;
                float sv[8];
                float ks_cur[2] = {ks[0], ks[1]};                // scales of this tile's K (8-bit cache)
                if constexpr (KST) {
                    // The copy into shared memory is complete when every load of this wave is (vmcnt = 0; the compiler
                    // does not order shared-memory reads behind such copies by itself).  This one wait also covers the V
                    // rows and the query asked for at the end of the previous tile, so nothing below waits for memory:
                    // the compiler would turn any wait for an older load into one for all loads while a copy into
                    // shared memory is in flight.
                    __builtin_amdgcn_s_waitcnt(0x0f70);
                    if constexpr (kPatchAppend) {
                        if (patch_row >= 0) {                    // this tile holds its request's new token (uniform)
                            const int blk = patch_row >> 4, row = patch_row & 15;
                            if (lane < kRowPieces) {             // piece `lane` of the K row: staging area, and its page
                                *reinterpret_cast<uint4 *>(kstage + blk * (16 * RB) + row * RB +
                                                           (((lane ^ row) & (kRowPieces - 1)) << 4)) = Kn;
                                *reinterpret_cast<uint4 *>(const_cast<char *>(ld.kbase) + patch_dst + lane * 16) = Kn;
                            }
                            if (lane < 16) {                     // piece `lane` of the V row to its page
                                char *vdst = const_cast<char *>(ld.vbase) + patch_dst;
                                vdst += lane * kVStep;
                                if constexpr (C::kVDwords == 2) {
                                    *reinterpret_cast<uint2 *>(vdst) = make_uint2(Vn[0], Vn[1]);
                                } else {
#pragma unroll
                                    for (int h = 0; h < C::kVDwords / 4; ++h)
                                        *reinterpret_cast<uint4 *>(vdst + h * 256) = make_uint4(Vn[4 * h], Vn[4 * h + 1], Vn[4 * h + 2], Vn[4 * h + 3]);
                                }
                            }
#pragma unroll
                            for (int r = 0; r < 8; ++r) {        // the lane group that holds the token takes the new V
                                if (slot_token(j, r) == patch_row) {
#pragma unroll
                                    for (int w = 0; w < C::kVDwords; ++w) Vr[r][w] = Vn[w];
                                }
                            }
                            patch_row = -1;
                        }
                    }
                    ks_cur[0] = ks[0]; ks_cur[1] = ks[1];
                    if constexpr (kHalves) {
                        ld.read_k_staged_half(kstage, 0, K);
                        const f32x4_t s0 = mfma_scores_f32<F>(K, Q);
                        __builtin_amdgcn_sched_barrier(0);       // the second half's operands take the first half's registers
                        ld.read_k_staged_half(kstage, 1, K);
#pragma unroll
                        for (int i = 0; i < 4; ++i) sv[i] = s0[i] * p.scale_log2;
                    } else {
                        ld.read_k_staged(kstage, K);
                    }
                    __builtin_amdgcn_s_waitcnt(0xc07f);          // operands are in registers (lgkmcnt = 0) ...
                    if (more) {                                  // ... so the next tile may take their place
                        if (nxt.append) { if constexpr (kPatchAppend) request_new_row(nxt); else append_row(nxt); }
                        issue_k(nxt.pg0, nxt.pg1);
                    }
                    if constexpr (kHalves) {
                        const f32x4_t s1 = mfma_scores_f32<F>(K, Q);
#pragma unroll
                        for (int i = 0; i < 4; ++i) sv[4 + i] = s1[i] * p.scale_log2;
                    } else {
                        mfma_scores<F>(K, Q, sv, p.scale_log2, ks_cur);
                    }
                } else if constexpr (C::kF32) {
                    // the halves' operands are asked for as soon as each is free: the scores take as long as a trip to memory
                    const f32x4_t s0 = mfma_scores_f32<F>(K, Q);
                    if (more) {
                        if (nxt.append) append_row(nxt);
                        ld.issue_k_half(ld.kbase + (size_t)nxt.pg0 * ld.page_stride, K);
                    }
                    const f32x4_t s1 = mfma_scores_f32<F>(K + C::kKRegs, Q);
                    if (more) {
                        ld.issue_k_half(ld.kbase + ld.second_half(nxt.pg0, nxt.pg1), K + C::kKRegs);
                        if (nxt.req != seg.b) load_q(nxt.req, Q);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) { sv[i] = s0[i] * p.scale_log2; sv[4 + i] = s1[i] * p.scale_log2; }
                } else {
                    mfma_scores<F>(K, Q, sv, p.scale_log2, ks);
                    if (more) {
                        if (nxt.append) append_row(nxt);
                        issue_k(nxt.pg0, nxt.pg1);
                        if (nxt.req != seg.b) load_q(nxt.req, Q);
                    }
                }
                auto request_next = [&]() __attribute__((always_inline)) {
                    if (!more) return;
                    if (KST && nxt.req != seg.b) load_q(nxt.req, Q);
                    issue_v(nxt.pg0, nxt.pg1);
                };
                if constexpr (C::kFp8) {
                    const float v0 = vs[0], v1 = vs[1];          // of the current tile: the next V request replaces them
                    uint32_t V[8][4];
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const uint4 x = fp8x8_to_bf16x8(Vr[r][0], Vr[r][1]);
                        V[r][0] = x.x; V[r][1] = x.y; V[r][2] = x.z; V[r][3] = x.w;
                    }
                    request_next();                              // the raw V bytes are consumed: request the next ones
                    mfma_softmax_pv<F, MT, kAllBits>(sv, V, st, cur.tile * kTile, seg.L, seg.L - col_back, t1min, j, v0, v1);
                } else {
                    mfma_softmax_pv<F, MT, kAllBits>(sv, Vr, st, cur.tile * kTile, seg.L, seg.L - col_back, t1min, j, 1.f, 1.f);
                    request_next();
                }
                ++s; cur = nxt;
            }

            // ---- end of the wave's share of this request: it leaves its state in shared memory and goes on
            st.l = across_lane_groups(st.l, [](float a, float b) { return a + b; });     // per-lane sums of the four groups; m is common
            float *state = ring + (size_t)(wbase + nstate) * state_floats;
            ++nstate;
            if (col < Gq) {
                float *orow = state + col * (D + 4);             // four dims per store: see the V loads for which block holds them
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int h = 0; h < C::kBlocks / 4; ++h) {
                        const int at = F == kF32D128 ? 64 * h + 16 * j + 4 * i : (4 * j + i) * C::kBlocks + 4 * h;
                        *reinterpret_cast<float4 *>(orow + at) = make_float4(st.acc[4 * h][i], st.acc[4 * h + 1][i], st.acc[4 * h + 2][i], st.acc[4 * h + 3][i]);
                    }
                if (j == 0) {
                    float *sm_m = state + Gq * (D + 4);
                    sm_m[col] = st.m; sm_m[kMaxGroup + col] = st.l;
                }
            }
        }

        // ---- the chunk is done: the workgroup meets and combines, request by request, the states that belong to it
        // (consecutive ones: the runs are in tile order).  Which states a request has depends on the plan alone, so the
        // first request's are worked out before the meeting and each further one's while the stores of the one before
        // are on their way.
        {
            int bb = cb, at = 0, e1, cnt;
            Segment sg;
            auto piece = [&]() {
                const int e0 = __builtin_amdgcn_readfirstlane(E[bb]);
                e1 = __builtin_amdgcn_readfirstlane(E[bb + 1]);
                const int lo = max(e0, cs) - cs, hi = min(e1, ce) - cs;              // the request's tiles in the chunk
                cnt = wave_of_tile(clen, hi - 1) - wave_of_tile(clen, lo) + 1;
                sg = plan_segment(E, Lc, pl, bb, range, start, end);
                sg.b += b0;
            };
            piece();
            lds_barrier();
            while (true) {
                mfma_combine_states<D, MT>(ring + (size_t)at * state_floats, cnt, state_floats, p, sg, kvh, MT ? Nc[bb] : 1);   // nobody waits for its stores
                at += cnt;
                if (e1 >= ce) break;
                do { ++bb; } while (__builtin_amdgcn_readfirstlane(E[bb + 1]) == __builtin_amdgcn_readfirstlane(E[bb]));
                piece();
            }
        }
        lds_barrier();
        cs = ce; cb = nb;
      }
    }
    if constexpr (WHOLE) {
        if (blockIdx.x == 0 && wave == 0) {                      // what the plan words say of such a launch
            unsigned long long T = 0;
            for (int b = lane; b < p.plan.B; b += 64) T += (unsigned)max(p.context_lens[b], 0);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) T += __shfl_xor(T, off);
            if (lane == 0) {
                p.ws.plan_words[0] = p.plan.s_force * kTile; p.ws.plan_words[1] = p.plan.B;
                p.ws.plan_words[2] = (int)(T & 0xffffffffULL); p.ws.plan_words[3] = (int)(T >> 32);
            }
        }
    } else {
        if (blockIdx.x == 0) write_merge_records(p, pl, E);
    }
}

}  // namespace omni
