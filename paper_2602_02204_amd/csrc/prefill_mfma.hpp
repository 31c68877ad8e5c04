// Matrix-core attention kernel for multi-token queries over the paged cache (chunked prefill): bf16 q/K/V,
// head_dim 128, group size <= 16.  Query i of request b's chunk sits at position p = L_b - n_b + i and attends to
// tokens 0 .. p (causal inside the chunk).
//
// The (query token, query head of the group) pairs of a request's chunk and one KV head are its "columns", in token-major
// order; a workgroup (8 waves, two per SIMD; 4 waves and two workgroups per compute unit where there are few columns) owns
// 256 (128) consecutive ones, wherever that cuts a token's heads (512 tokens of 7 heads are 14 workgroups; whole tokens only
// would make them 15), a wave 32 of them = the columns of one 32x32x16 matrix instruction.  Per 32-token tile:
//   S^T = K Q^T     (A = K rows from shared memory, B = the wave's queries, held in registers for the whole kernel)
//   O^T += V^T P^T  (A = V transposed, B = the softmax weights; both as fp16: V is converted once per workgroup on
//                    its way into shared memory, exactly for 2^-14 <= |V| <= 65504, and fp16 weights carry 11
//                    significant bits, so one product does what bf16 weights need a hi + lo pair for)
// so every lane owns one column (the two halves of a wave hold its even and odd groups of four tokens): running reference,
// sum and rescale never cross lanes on the common path.
// What differs from decode is reuse: K/V tiles are fetched once per workgroup into shared memory (double buffered,
// one barrier per 64 tokens) and feed all its columns, and V^T comes out of shared memory through transposing reads.
// That makes the path a dense contraction, not a stream.  The three pieces of a tile's work are software-pipelined
// across tiles, so that a wave has matrix-core and vector-ALU instructions to issue side by side.
// What bounds it: the clock the chip holds under this load (1.7 - 1.85 GHz of 2.4), at which the matrix cores are busy
// 56 % of the time on long contexts (1080 TFLOP/s; a library product of 8192^3 reaches 1190) and 47 % on 32 requests with
// 512-token chunks, whose workgroups spend 10 of 75 us on their start and end.  Against 16-column instructions over 36
// whole tokens with every step testing each of its tiles: 16 % fewer cycles at a clock 8 % lower,
// 590.0 -> 574.8 us for those 32 requests with their append.
// The instructions are 32 columns wide: half as many to issue for the same product.  The rows of V are padded to 320 bytes because a transposing read of 32 lanes takes 64 bytes of each of four rows
// (288: 583 -> 564 us); the steps at the ends of the context have their own code because conditions around 16-register
// operands made the compiler copy and spill the accumulators (in one loop with tests: 2400 us).
#pragma once
#include <type_traits>

#include "decode_mfma.hpp"

namespace omni {

constexpr int kPrefillRowBytes = 256 + 16;            // a 256-byte K row plus padding: conflict-free 16-byte LDS reads
constexpr int kPrefillVRowBytes = 256 + 64;           // V rows: conflict-free 8-byte transposing reads (4 rows x 64 B)
constexpr float kPrefillBias = 6.f;                   // a moved reference sits this many log2 units below the maximum
constexpr float kPrefillSumLimit = 32768.f;           // sum of a lane's 16 weights of a tile beyond which the reference moves

// Transposing 64-bit read from shared memory (see its use below for the lane arrangement).
__device__ __forceinline__ uint2 lds_read_tr16_b64(const char *p) {
    typedef short short4_t __attribute__((ext_vector_type(4)));
    const short4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (short4_t __attribute__((address_space(3))) *)(const __attribute__((address_space(3))) char *)p);
    return __builtin_bit_cast(uint2, v);
}

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// A: 32 rows x 16 k, B: 16 k x 32 columns; a lane holds row / column lane % 32 and the 8 k of half lane / 32.  The result
// leaves it with rows 8 (r / 4) + 4 (lane / 32) + r % 4 of column lane % 32 in register r.
__device__ __forceinline__ f32x16_t mfma32_bf16(const uint4 &a, const uint4 &b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mfma32_f16(const uint4 &a, const uint4 &b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));

// c + the two fp16 values packed in w, in fp32.
__device__ __forceinline__ float sum_f16x2(uint32_t w, float c) {
    const f16x2_t ones = {(_Float16)1.f, (_Float16)1.f};
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, w), ones, c, false);
}

// Two floats -> packed fp16, round to nearest even.
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}

// Eight bf16 values -> eight fp16 values.  Exact wherever the value is a normal fp16 number (2^-14 <= |V| <= 65504);
// below that the spacing is 2^-24, i.e. an absolute error of at most 2^-25; above it the value becomes infinite and
// shows in the result.
__device__ __forceinline__ uint4 bf16x8_to_f16x8(const uint4 &v) {
    uint4 r;
    r.x = pack_f16x2(bf16_bits_to_float(v.x & 0xffffu), __uint_as_float(v.x & 0xffff0000u));
    r.y = pack_f16x2(bf16_bits_to_float(v.y & 0xffffu), __uint_as_float(v.y & 0xffff0000u));
    r.z = pack_f16x2(bf16_bits_to_float(v.z & 0xffffu), __uint_as_float(v.z & 0xffff0000u));
    r.w = pack_f16x2(bf16_bits_to_float(v.w & 0xffffu), __uint_as_float(v.w & 0xffff0000u));
    return r;
}

// Eight E4M3 bytes times a scale -> eight fp16 values: widened exactly (bf16, then fp32), scaled in fp32, rounded once.
__device__ __forceinline__ uint4 fp8x8_scaled_to_f16x8(uint32_t lo, uint32_t hi, float sc) {
    const uint4 v = fp8x8_to_bf16x8(lo, hi);
    uint4 r;
    r.x = pack_f16x2(bf16_bits_to_float(v.x & 0xffffu) * sc, __uint_as_float(v.x & 0xffff0000u) * sc);
    r.y = pack_f16x2(bf16_bits_to_float(v.y & 0xffffu) * sc, __uint_as_float(v.y & 0xffff0000u) * sc);
    r.z = pack_f16x2(bf16_bits_to_float(v.z & 0xffffu) * sc, __uint_as_float(v.z & 0xffff0000u) * sc);
    r.w = pack_f16x2(bf16_bits_to_float(v.w & 0xffffu) * sc, __uint_as_float(v.w & 0xffff0000u) * sc);
    return r;
}

struct PrefillParams {
    const void *q;                    // [Tq, Hq, D] bf16
    const void *k_cache, *v_cache;
    const float *k_scale, *v_scale;   // 8-bit cache only (else null): [P, Hkv] scales of the K and V pools
    const int32_t *block_table, *context_lens, *q_lens;
    const long long *q_offsets;
    void *out;                        // [Tq, Hq, D]
    float scale_log2;
    int Hq, Hkv, G, MB;
    int out_bf16;
    // Context split (matrix-core kernel): each workgroup's 64-token steps are dealt to num_splits workgroups, which
    // leave unnormalised rows and (reference, sum) per (request, query token < max_q_len, head, split) for the merge.
    int num_splits;                   // 1: no split, results go straight to out
    int min_split_steps;              // fewest 64-token steps a split's share may have
    int max_q_len;
    int columns;                      // (query token, head) pairs per workgroup
    float *part_o;                    // [B, max_q_len, Hq, num_splits, D]
    float2 *part_ml;                  // [B, max_q_len, Hq, num_splits]
    const int32_t *order;             // null, or [B]: the requests by descending context length (blockIdx.z -> request)
    int B;
};

// A split's share of the context is at least this many 64-token steps: below that the pieces' trip through memory
// costs more than the extra workgroups bring.  Decided per query block on the device, where the lengths are known.
constexpr int kPrefillMinSplitTokens = 256;          // default; a tuning value
__device__ __forceinline__ int prefill_effective_splits(int num_splits, int n_steps, int min_split_steps) {
    return max(1, min(num_splits, n_steps / min_split_steps));
}

// The (query token, head) pairs of a chunk and one KV head, in token-major order, are cut into runs of 32 per wave of a
// workgroup.
constexpr int prefill_columns(int waves) { return 32 * waves; }
// The chunk's last query token that the workgroup with first column c0 has a column of (n_live tokens are live).
__host__ __device__ inline int prefill_last_token(int c0, int columns, int G, int n_live) {
    const int t = (c0 + columns - 1) / G;
    return t < n_live ? t : n_live - 1;
}

// What a workgroup works on: grid (blocks x splits, KV heads, requests), dispatched in linear order, requests slowest.
struct PrefillPlace {
    int b, kvh;                       // request, KV head
    int L;                            // the request's context length
    int block;                        // place among the workgroups of the (request, KV head): block x splits
};

__device__ __forceinline__ PrefillPlace prefill_place(const PrefillParams &p) {
    PrefillPlace at;
    at.b = p.order ? p.order[blockIdx.z] : (int)blockIdx.z;
    at.L = p.context_lens[at.b];
    at.kvh = blockIdx.y;
    at.block = blockIdx.x;
    // Workgroups are dealt to the eight compute dies in turn.  A request's are arranged so that a die gets workgroups of one
    // KV head of it (or every eighth of the heads, whole): they share its rows in the die's cache.  Every die still gets the
    // same number of them, so it does not matter how the lengths differ.  32 requests with 512-token chunks, 28/4 heads 548 ->
    // 535 us, 32/8 heads 641 -> 614 us; 64-dim heads, 24 requests with chunks of 1 .. 1024 tokens, 16/2 heads 114.9 -> 110.2
    // us.  With a split the workgroups of one head read different rows, and it is left as it comes.
    constexpr int kDies = 8;
    const int gx = gridDim.x, heads = gridDim.y;
    if (p.num_splits == 1 && gx * heads % kDies == 0) {
        const int u = blockIdx.x + gx * blockIdx.y, die = u % kDies, i = u / kDies;
        if (heads % kDies == 0) { at.kvh = die + kDies * (i / gx); at.block = i % gx; }
        else if (kDies % heads == 0) {                           // (short chunks lack the last blocks: not always on one die)
            const int share = kDies / heads;
            at.kvh = die % heads; at.block = (die / heads + blockIdx.z) % share + share * i;
        }
    }
    return at;
}

// KV8: the pools hold 8-bit E4M3 bytes with one scale per (page, KV head).  The staging threads widen K to bf16
// (exact) and V times its page's scale to fp16 (one rounding, 2^-12 relative: the size of the weights' own rounding) on
// the way into shared memory, so the products are the 16-bit ones; the K scale of each 16-token half of a tile joins
// the softmax scale in the exponent's multiply-add.
// W: waves per workgroup, 8 (one workgroup per compute unit) or 4 (two).
template <int PS, bool KV8, int W>
__global__ __launch_bounds__(64 * W, 2) void prefill_mfma_kernel(PrefillParams p) {
    constexpr int D = 128;
    constexpr int ES = KV8 ? 1 : 2;                              // bytes per cache element
    constexpr int kLog2Ps = (PS == 16) ? 4 : 5;
    constexpr int kStep = 2 * kTile;                             // tokens staged at a time
    constexpr int kColumns = prefill_columns(W);
    constexpr int kKRow = kPrefillRowBytes, kVRow = kPrefillVRowBytes;
    constexpr int kTokStride = 64 * W / 16;                      // a thread stages one of a row's 16 pieces of every
    constexpr int NP = kStep / kTokStride;                       // kTokStride-th token of a step
    __shared__ __align__(16) char k_lds[2][kStep * kKRow];
    __shared__ __align__(16) char v_lds[2][kStep * kVRow];
    __shared__ float kscale_lds[2][4];                           // 8-bit cache: [buffer][16 tokens] K scales

    // Workgroups are dispatched in blockIdx order, z slowest: with the requests taken longest first the long-running
    // workgroups start first and the short ones fill the end of the launch.
    const PrefillPlace at = prefill_place(p);
    const int b = at.b, kvh = at.kvh, L = at.L;
    const int G = p.G, head0 = kvh * G;
    const int n_q = min(p.q_lens[b], L);
    const int n_live = min(n_q, p.max_q_len);                    // a chunk longer than the grid's bound is cut off there
    const int NS = p.num_splits;
    const int split = NS > 1 ? at.block % NS : 0;
    const int c0 = (NS > 1 ? at.block / NS : at.block) * kColumns;     // first column of this workgroup
    if (n_live <= 0 || c0 >= n_live * G) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, h = lane >> 5;
    const long long q_row0 = p.q_offsets[b];
    const int pos0 = L - n_q;                                    // position of the chunk's first token
    const int wg_last = prefill_last_token(c0, kColumns, G, n_live);
    const int n_tiles = (pos0 + wg_last) / kTile + 1;            // tiles that hold tokens 0 .. position of wg_last

    // ---- this lane's column: query token, head, position; and the queries as MFMA B operands
    const int qi = (c0 + wave * 32 + col) / G, g = c0 + wave * 32 + col - qi * G;
    const bool live = qi < n_live;
    const int pos = live ? pos0 + qi : -1;                       // -1: padding column (never stored)
    uint4 Q[8];
    {
        const char *qrow = reinterpret_cast<const char *>(p.q) + ((size_t)(q_row0 + qi) * p.Hq + head0 + g) * (D * 2);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            Q[kk] = make_uint4(0, 0, 0, 0);
            if (live) Q[kk] = *reinterpret_cast<const uint4 *>(qrow + (2 * kk + h) * 16);
        }
    }
    int wave_max_pos = pos, wave_min_pos = live ? pos : 0x7fffffff;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
        wave_max_pos = max(wave_max_pos, __shfl_xor(wave_max_pos, off));
        wave_min_pos = min(wave_min_pos, __shfl_xor(wave_min_pos, off));
    }
    wave_max_pos = __builtin_amdgcn_readfirstlane(wave_max_pos);
    wave_min_pos = __builtin_amdgcn_readfirstlane(wave_min_pos);

    // ---- staging: thread t moves piece t % 16 of tokens t / 16, ... of a step's K rows and V rows.  The products below run
    // as a pipeline in which V of a tile is needed two tiles after its K, so V is fetched and staged one step behind K.
    const unsigned page_stride = (unsigned)(p.Hkv * PS * D * ES);   // gridDim.y bounds Hkv: fits 32 bits
    const char *kbase = reinterpret_cast<const char *>(p.k_cache) + (size_t)kvh * PS * D * ES;
    const char *vbase = reinterpret_cast<const char *>(p.v_cache) + (size_t)kvh * PS * D * ES;
    const int32_t *bt = p.block_table + (size_t)b * p.MB;
    const int st_tok = threadIdx.x >> 4, st_chunk = threadIdx.x & 15;
    const int lds_off = st_tok * kKRow + st_chunk * 16;
    const int lds_off_v = st_tok * kVRow + st_chunk * 16;
    const int n_steps = (n_tiles + 1) >> 1;
    // this workgroup's share of the steps: [s_begin, s_end), all of them without a split.  The launch provides NS
    // workgroups per run of columns; how many of them share the work depends on their context.
    const int ns_eff = prefill_effective_splits(NS, n_steps, p.min_split_steps);
    if (split >= ns_eff) return;
    const int s_begin = (int)((long long)n_steps * split / ns_eff);
    const int s_end = (int)((long long)n_steps * (split + 1) / ns_eff);
    const int last_page = (L - 1) >> kLog2Ps;
    uint4 sk[NP], sv_[NP];                                       // 8-bit cache: 8 bytes each, in .x and .y
    float sks[NP], svs[NP];                                      // 8-bit cache: the scales of the rows' pages
    // Page numbers are looked up one step before the rows they address are fetched, so that no fetch waits for its
    // own table entry: pg_k holds the pages of the step whose K rows are fetched next, pg_v (the same entries one
    // step later) those of the step whose V rows are fetched next.
    int pg_k[NP], pg_v[NP];
    auto lookup = [&](int step) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i)
            pg_k[i] = bt[(unsigned)min(step * (kStep / PS) + ((st_tok + i * kTokStride) >> kLog2Ps), last_page)];
    };
    auto fetch_rows = [&](auto fast, const char *base, const float *scale, int step, const int (&pg)[NP], uint4 (&r)[NP],
                          float (&sc)[NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int t = step * kStep + st_tok + i * kTokStride;
            const char *src = base + (unsigned long long)(unsigned)pg[i] * page_stride +
                              ((st_tok + i * kTokStride) & (PS - 1)) * (D * ES) + st_chunk * (8 * ES);
            const bool in = decltype(fast)::value || (step < s_end && t < L);
            r[i] = make_uint4(0, 0, 0, 0);                                // rows beyond the context are zero
            if constexpr (KV8) {
                if (in) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(src);
                    r[i].x = v.x; r[i].y = v.y;
                }
                sc[i] = scale[(size_t)pg[i] * p.Hkv];                   // the page is a valid one also beyond the context
            } else {
                if (in) r[i] = *reinterpret_cast<const uint4 *>(src);
            }
        }
    };
    auto stage_k = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            char *dst = &k_lds[buf][lds_off + i * (kTokStride * kKRow)];
            if constexpr (KV8) {
                *reinterpret_cast<uint4 *>(dst) = fp8x8_to_bf16x8(sk[i].x, sk[i].y);
                if (st_chunk == 0 && (st_tok & 15) == 0) kscale_lds[buf][(st_tok + i * kTokStride) >> 4] = sks[i];
            } else {
                *reinterpret_cast<uint4 *>(dst) = sk[i];
            }
        }
    };
    auto stage_v = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            char *dst = &v_lds[buf][lds_off_v + i * (kTokStride * kVRow)];
            if constexpr (KV8)
                *reinterpret_cast<uint4 *>(dst) = fp8x8_scaled_to_f16x8(sv_[i].x, sv_[i].y, svs[i]);
            else
                *reinterpret_cast<uint4 *>(dst) = bf16x8_to_f16x8(sv_[i]);
        }
    };

    // ---- the column's online-softmax state
    float m = -INFINITY, l = 0.f;
    f32x16_t acc[4] = {{}, {}, {}, {}};                          // acc[e][r] = O^T[dim 32 e + 8 (r / 4) + 4 h + r % 4][column]

    // ---- the three pieces of a tile's work
    // Raw scores q.k: S[r] holds token 8 (r / 4) + 4 h + r % 4 of the tile for column `col`.  The softmax scale is applied
    // inside the exponent (one fused multiply-add per score): scale > 0, so the order of scores is that of the raw dot
    // products.
    const int k_off = col * kKRow + h * 16;
    const int v_off = (4 * h + ((lane & 15) >> 2)) * kVRow + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    auto scores = [&](const char *ks, f32x16_t &S, const float *ksc, float (&a)[2]) __attribute__((always_inline)) {
        if constexpr (KV8) {                                     // read with the rows: both are replaced together
            a[0] = ksc[0] * p.scale_log2; a[1] = ksc[1] * p.scale_log2;
        }
        uint4 K[8];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) K[kk] = *reinterpret_cast<const uint4 *>(ks + k_off + kk * 32);
        S = f32x16_t{};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) S = mfma32_bf16(K[kk], Q[kk], S);
    };
    // Weights of tile t from its raw scores: P as two fp16 MFMA operands.  A column's reference m (log2 domain) is
    // moved only when a weight would leave the fp16 range, which shows in the sum of the tile's weights: any common
    // reference gives the same softmax.  A move puts m at the running maximum less the bias, so the largest weight of a
    // column then lies between 2^bias and the limit, and a weight loses precision as an fp16 subnormal only when it is
    // 2^-20 of the largest or less.  After a column's first tiles moves are rare, so the maximum over the tile, its
    // exchange between the two halves of a column and the rescale of what was summed under the old reference
    // leave the common path.  The sums are taken over the rounded weights, the ones the matrix cores multiply.
    // `mask`: tokens after the column's position may be among the tile's (kMaybe: the wave looks first).
    constexpr int kNone = 0, kMaybe = 1, kAlways = 2;
    constexpr std::integral_constant<int, kNone> before{};
    constexpr std::integral_constant<int, kMaybe> maybe{};
    constexpr std::integral_constant<int, kAlways> masked{};
    auto weights = [&](auto mask, int t, f32x16_t &S, uint4 (&P)[2], const float (&a)[2]) __attribute__((always_inline)) {
        const int tb = t * kTile;
        if (decltype(mask)::value == kAlways || (decltype(mask)::value == kMaybe && tb + kTile - 1 > wave_min_pos)) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (tb + 8 * (r >> 2) + 4 * h + (r & 3) > pos) S[r] = -INFINITY;
        }
        float psum;
        auto form = [&]() __attribute__((always_inline)) {
            float pw[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) pw[r] = fast_exp2(fmaf(S[r], KV8 ? a[r >> 3] : p.scale_log2, -m));
            float s2[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                P[i] = make_uint4(pack_f16x2(pw[8 * i], pw[8 * i + 1]), pack_f16x2(pw[8 * i + 2], pw[8 * i + 3]),
                                  pack_f16x2(pw[8 * i + 4], pw[8 * i + 5]), pack_f16x2(pw[8 * i + 6], pw[8 * i + 7]));
                s2[i] = sum_f16x2(P[i].w, sum_f16x2(P[i].z, sum_f16x2(P[i].y, sum_f16x2(P[i].x, i ? s2[0] : 0.f))));
            }
            psum = s2[1];
        };
        form();
        if (__any(!(psum < kPrefillSumLimit))) {                 // also for an infinite or undefined sum
            float t0 = fmaxf(S[0], S[1]), t1 = fmaxf(S[8], S[9]);
#pragma unroll
            for (int r = 2; r < 8; ++r) { t0 = fmaxf(t0, S[r]); t1 = fmaxf(t1, S[8 + r]); }
            // the largest scaled score of the tile, in log2 units (scales are positive)
            float tmax = KV8 ? fmaxf(t0 * a[0], t1 * a[1]) : fmaxf(t0, t1) * p.scale_log2;
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            // a column whose tokens are all masked so far keeps a finite stand-in: exp2 then sees -inf - finite
            const float mn = fmaxf(fmaxf(m, tmax - kPrefillBias), -1e30f);
            const float alpha = fast_exp2(m - mn);       // 0 while m is still -inf
            l *= alpha;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] *= alpha;
            m = mn;
            form();
        }
        l += psum;
    };
    // O^T += V^T P^T.  The V^T operands come transposed out of shared memory: in a transposing 8-byte read the 16 lanes of a
    // group each name four consecutive 16-bit values (lane 4k + q: dims 4q .. 4q+3 of token k of the group's four tokens) and
    // lane i receives value i of each token, i.e. one output dim for four tokens.  Two reads (tokens 4h .. 4h+3 and
    // 8+4h .. 8+4h+3 of 16, exactly the tokens whose weights this half holds) make the operand of 16 tokens and 32 dims.
    auto pv = [&](const char *vs, const uint4 (&P)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint2 a0 = lds_read_tr16_b64(vs + v_off + (16 * i) * kVRow + e * 64);
                const uint2 a1 = lds_read_tr16_b64(vs + v_off + (16 * i + 8) * kVRow + e * 64);
                acc[e] = mfma32_f16(make_uint4(a0.x, a0.y, a1.x, a1.y), P[i], acc[e]);
            }
    };
    // ---- the pipeline.  Phase t multiplies the weights of tile t-1 into the accumulators and forms the scores of
    // tile t+1 on the matrix cores while the vector ALUs turn the scores of tile t into weights; the three are
    // independent, so one wave keeps both units busy.  A step is the two phases of an (even, odd) pair of tiles and
    // ends with one barrier: during step s the workgroup reads K of step s (tiles 2s, 2s+1) and V of step s-1 from
    // shared memory and stages K of step s+1 and V of step s.
    f32x16_t Se, So;                                             // scores of the even / odd tile in flight
    uint4 Pe[2], Po[2];                                          // weights of the even / odd tile in flight
    float ae[2] = {0.f, 0.f}, ao[2] = {0.f, 0.f};                // 8-bit cache: their scores' multipliers per 16-token half
    const float *k_scale = KV8 ? p.k_scale + kvh : nullptr, *v_scale = KV8 ? p.v_scale + kvh : nullptr;
    auto fetch = [&](auto inside, int s) __attribute__((always_inline)) {        // in flight while step s is computed
        fetch_rows(inside, vbase, v_scale, s, pg_v, sv_, svs);
        fetch_rows(inside, kbase, k_scale, s + 1, pg_k, sk, sks);
#pragma unroll
        for (int i = 0; i < NP; ++i) pg_v[i] = pg_k[i];
        lookup(s + 2);
    };
    auto stage = [&](int s) __attribute__((always_inline)) { stage_k((s & 1) ^ 1); stage_v(s & 1); };
    // A step all of whose tiles 2s-2 .. 2s+1 hold tokens that the wave sees.  `mask` none: they lie wholly before all of its
    // positions, and what is fetched lies wholly inside the context.
    auto full_step = [&](auto mask, int s) __attribute__((always_inline)) {
        const int buf = s & 1;
        fetch(std::integral_constant<bool, decltype(mask)::value == kNone>{}, s);
        // phase 2s-1: P.V of tile 2s-2, weights of tile 2s-1, scores of tile 2s
        pv(v_lds[buf ^ 1], Pe);
        scores(k_lds[buf], Se, kscale_lds[buf], ae);
        weights(mask, 2 * s - 1, So, Po, ao);
        // phase 2s: P.V of tile 2s-1, weights of tile 2s, scores of tile 2s+1
        pv(v_lds[buf ^ 1] + kTile * kVRow, Po);
        scores(k_lds[buf] + kTile * kKRow, So, kscale_lds[buf] + 2, ao);
        stage(s);                                                // ahead of the weights: one block with the MFMAs above
        weights(mask, 2 * s, Se, Pe, ae);
        lds_barrier();
    };
    const int fast_last = min(min(((wave_min_pos - (kTile - 1)) / kTile - 1) / 2, L / kStep - 2), s_end - 1);
    const int last_tile = min(wave_max_pos >> kLog2Tile, 2 * s_end - 1);     // the last one the wave sees any of (-1: no live column)
    lookup(s_begin);
    fetch_rows(std::false_type{}, kbase, k_scale, s_begin, pg_k, sk, sks);
#pragma unroll
    for (int i = 0; i < NP; ++i) pg_v[i] = pg_k[i];
    lookup(s_begin + 1);
    stage_k(s_begin & 1);
    lds_barrier();
    // Every wave passes s_end - s_begin more barriers, one at the end of each step before s_end, wherever its own tiles end.
    int s = s_begin;
    if (last_tile >= 2 * s) {
        fetch(std::false_type{}, s);                             // the first step: nothing to multiply yet
        scores(k_lds[s & 1], Se, kscale_lds[s & 1], ae);
        if (last_tile > 2 * s) scores(k_lds[s & 1] + kTile * kKRow, So, kscale_lds[s & 1] + 2, ao);
        stage(s);
        weights(maybe, 2 * s, Se, Pe, ae);
        lds_barrier();
        for (++s; s <= fast_last; ++s) full_step(before, s);
        for (; last_tile > 2 * s; ++s) full_step(masked, s);
        // here the last tile is 2s-1 or 2s, or 2s-2 if the first step held it; what is left: an even tile's weights to
        // multiply, and the odd one's before them
        bool even = true;
        if (last_tile >= 2 * s - 1) {
            even = last_tile == 2 * s;
            if (s < s_end) fetch(std::false_type{}, s);
            pv(v_lds[(s & 1) ^ 1], Pe);
            if (even) scores(k_lds[s & 1], Se, kscale_lds[s & 1], ae);
            weights(masked, 2 * s - 1, So, Po, ao);
            pv(v_lds[(s & 1) ^ 1] + kTile * kVRow, Po);
            if (s < s_end) stage(s);
            if (even) weights(masked, 2 * s, Se, Pe, ae);
            if (s < s_end) lds_barrier();
            ++s;
        }
        if (even) {
            if (s < s_end) fetch(std::false_type{}, s);
            pv(v_lds[(s & 1) ^ 1], Pe);
            if (s < s_end) { stage(s); lds_barrier(); }
            ++s;
        }
    }
    for (; s < s_end; ++s) { fetch(std::false_type{}, s); stage(s); lds_barrier(); }     // for the other waves

    // ---- normalise and store
    const float lsum = l + __shfl_xor(l, 32);                    // the two halves hold disjoint tokens
    if (!live) return;
    if (ns_eff > 1) {                                            // a piece for the merge: unnormalised, with (m, l)
        const size_t pi = ((((size_t)b * p.max_q_len + qi) * p.Hq + head0 + g) * NS + split);
        float *po = p.part_o + pi * D;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<float4 *>(po + 32 * e + 8 * i + 4 * h) = make_float4(acc[e][4 * i], acc[e][4 * i + 1], acc[e][4 * i + 2], acc[e][4 * i + 3]);
        if (h == 0) p.part_ml[pi] = make_float2(m, lsum);
        return;
    }
    const size_t row = ((size_t)(q_row0 + qi) * p.Hq + head0 + g) * D;
    const float inv = 1.f / lsum;                                // every live column saw its own position: lsum > 0
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            store_out4(p, row + 32 * e + 8 * i + 4 * h, make_float4(acc[e][4 * i] * inv, acc[e][4 * i + 1] * inv, acc[e][4 * i + 2] * inv, acc[e][4 * i + 3] * inv));
}

// order[r] = the request with the r-th longest context (ties by index): one workgroup, thread t ranks request t.
constexpr int kPrefillOrderMax = 1024;
__global__ __launch_bounds__(kPrefillOrderMax) void prefill_order_kernel(const int32_t *__restrict__ context_lens, int B,
                                                                         int32_t *__restrict__ order) {
    __shared__ int lens[kPrefillOrderMax];
    const int t = threadIdx.x;
    if (t < B) lens[t] = context_lens[t];
    __syncthreads();
    if (t >= B) return;
    const int mine = lens[t];
    int rank = 0;
    for (int j = 0; j < B; ++j) rank += (lens[j] > mine) || (lens[j] == mine && j < t);
    order[rank] = t;
}

// Merge of a context split: out row = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s over the pieces with l_s != 0, in
// split order (M = the largest reference among them; any common reference gives the same quotient).  One thread per
// four output elements of one (query token, head); grid (ceil(max_q_len * Hq * D / 4 / 256), B).
template <int D>
__global__ __launch_bounds__(kThreads) void prefill_merge_kernel(PrefillParams p) {
    constexpr int kRowThreads = D / 4;
    const int b = blockIdx.y;
    const long long lin = (long long)blockIdx.x * kThreads + threadIdx.x;
    const int d4 = (int)(lin % kRowThreads);
    const long long rh = lin / kRowThreads;
    const int head = (int)(rh % p.Hq);
    const long long qi = rh / p.Hq;
    const int L = p.context_lens[b];
    const int n_q = min(p.q_lens[b], L);
    const int n_live = min(n_q, p.max_q_len);
    if (qi >= n_live) return;
    // the split count of the row's workgroup, as the attention kernel derived it
    const int c = (int)qi * p.G + head % p.G;
    const int wg_last = prefill_last_token(c - c % p.columns, p.columns, p.G, n_live);
    const int n_tiles = (L - n_q + wg_last) / kTile + 1;
    const int ns_eff = prefill_effective_splits(p.num_splits, (n_tiles + 1) >> 1, p.min_split_steps);
    if (ns_eff == 1) return;                                     // written by the attention kernel itself
    const int NS = p.num_splits;
    const size_t pi = (((size_t)b * p.max_q_len + qi) * p.Hq + head) * NS;
    float M = -INFINITY, den = 0.f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    // All loads of a round are issued before any is used: one piece after the other, each behind a test of its sum, made the
    // launch a chain of two trips to memory per piece (one request, 28/4 heads, 16 tokens of 16384, 16 pieces: 27.9 -> 21.0 us a
    // call; 8/8 heads, four requests of 2048, 8 pieces: 18.1 -> 15.1 us).
    auto round = [&](auto size, int s0) __attribute__((always_inline)) {
        constexpr int R = decltype(size)::value;
        float2 ml[R];
        float4 o[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const size_t at = pi + min(s0 + r, ns_eff - 1);
            ml[r] = p.part_ml[at];
            o[r] = *reinterpret_cast<const float4 *>(p.part_o + at * D + 4 * d4);
        }
        float Mn = M;
        bool has[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            has[r] = s0 + r < ns_eff && ml[r].y != 0.f;          // also a NaN: a piece with a NaN score must show
            if (has[r]) Mn = fmaxf(Mn, ml[r].x);
        }
        const float a = M > -INFINITY ? fast_exp2(M - Mn) : 0.f;
        num.x *= a; num.y *= a; num.z *= a; num.w *= a;
        den *= a;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (has[r]) {
                const float w = fast_exp2(ml[r].x - Mn);
                num.x += w * o[r].x; num.y += w * o[r].y; num.z += w * o[r].z; num.w += w * o[r].w;
                den += w * ml[r].y;
            }
        }
        M = Mn;
    };
    if (ns_eff <= 4) round(std::integral_constant<int, 4>{}, 0);
    else
        for (int s0 = 0; s0 < ns_eff; s0 += 8) round(std::integral_constant<int, 8>{}, s0);
    const float inv = 1.f / den;                                 // the split that holds the token's own position has l > 0
    const size_t at = ((size_t)(p.q_offsets[b] + qi) * p.Hq + head) * D + 4 * d4;
    if (p.out_bf16) {
        uint2 pk;
        pk.x = (uint32_t)float_to_bf16_rne(num.x * inv) | ((uint32_t)float_to_bf16_rne(num.y * inv) << 16);
        pk.y = (uint32_t)float_to_bf16_rne(num.z * inv) | ((uint32_t)float_to_bf16_rne(num.w * inv) << 16);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(p.out) + at) = pk;
    } else {
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.out) + at) = make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv);
    }
}

}  // namespace omni
