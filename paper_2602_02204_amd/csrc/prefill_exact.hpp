// Matrix-core attention kernel for multi-token queries (chunked prefill) over bf16 caches with head_dim 64, group size
// <= 16, whose softmax weights keep 24 bits.  Same definition, column layout, context split and order of the requests as
// prefill_mfma.hpp.
//
// A workgroup (4 waves) owns 128 (query token, head) columns of one (request, KV head); a wave owns 32 of them = the
// columns of one v_mfma_f32_32x32x16_bf16 (A: 32 rows x 16 k, B: 16 k x 32 columns; a lane holds row / column lane % 32
// and the 8 k of half lane / 32).  Per 32-token tile:
//   S^T = K Q^T      A = K rows from shared memory, B = the queries, in registers for the whole kernel
//   O^T += V^T P^T   A = V transposed by its reads from shared memory, B = the weights as three bf16 parts whose sum is
//                    the fp32 weight (split_weights<3>): products are exact, sums fp32, as in the vector-ALU kernel
// so a lane owns one column and nothing crosses lanes on the common path.  The scores leave a lane with tokens
// 8 (r / 4) + 4 (lane / 32) + r % 4 in register r, and the k-slots of the second product are bound to just these.
//
// Bound by the vector ALUs: 174 instructions per wave and tile on 512-token chunks, 196 on ragged ones (half of them split
// the weights), against 16 matrix instructions; the counters show the ALUs issuing 81 and 71 % of the time, exponentials at a
// quarter of the rate on top, and the matrix cores busy 50 and 40 %.  Therefore 32-column instructions (half as many to issue
// as 16-column ones) and three
// independent workgroups per compute unit: their barriers do not meet, so one's matrix work hides another's weights.
// Measured with the append, 24 requests of 129 .. 2049 tokens with chunks of 1 .. 1024, 16/2 heads: vector-ALU kernel
// 2010 us, this one 115 us, 111 us with the workgroups of a KV head on one die; 32 requests with 512-token chunks (137 GFLOP) 310
// -> 304 us = 450 TFLOP/s.  Taken back: 8 waves per
// workgroup (174 us, 330 us), the tiles' work software-pipelined as in prefill_mfma.hpp at two waves per SIMD (143 us, 331 us),
// four waves per SIMD (231 us: 128 registers do not hold it).  v_dot2_f32_bf16 for the split's subtractions (one instruction
// for two) gained nothing: it does not run at the full rate.  Distance from 64 bits against the vector-ALU kernel's: 1.05 - 1.17
// times where scores have deviation one and the context is not split, 0.2 - 0.8 times where it is split or scores are larger;
// the scores in two chains bring 1.12 to 1.06 on 40-token contexts and cost 2 % (taken back).
#pragma once
#include "prefill_mfma.hpp"
#include "row_walk.hpp"

namespace omni {

constexpr int kPrefillExactWaves = 4, kPrefillExactThreads = 64 * kPrefillExactWaves;
constexpr float kPrefillExactLimit = 256.f;                        // sum of a lane's 16 weights of a tile beyond which the reference moves

template <int PS>
__global__ __launch_bounds__(kPrefillExactThreads, 3) void prefill_exact_kernel(PrefillParams p) {
    constexpr int D = 64, RB = 2 * D;                            // bytes of a cache row
    constexpr int kLog2Ps = (PS == 16) ? 4 : 5;
    constexpr int kStep = 2 * kTile;                             // tokens staged at a time
    constexpr int kKRow = RB + 16, kVRow = RB + 32;              // staged rows: conflict-free 16-byte / transposing reads
    constexpr int kChunks = RB / 16;
    constexpr int NP = kStep * kChunks / kPrefillExactThreads;   // 16-byte pieces of K (and of V) a thread stages per step
    constexpr int kTokStride = kPrefillExactThreads / kChunks;   // tokens between them
    __shared__ __align__(16) char k_lds[2][kStep * kKRow];
    __shared__ __align__(16) char v_lds[2][kStep * kVRow];

    const PrefillPlace at = prefill_place(p);
    const int b = at.b, kvh = at.kvh, L = at.L;
    const int G = p.G, head0 = kvh * G;
    const int n_q = min(p.q_lens[b], L);
    const int n_live = min(n_q, p.max_q_len);                    // a chunk longer than the grid's bound is cut off there
    constexpr int kColumns = prefill_columns(kPrefillExactWaves);
    const int NS = p.num_splits;
    const int split = NS > 1 ? at.block % NS : 0;
    const int c0 = (NS > 1 ? at.block / NS : at.block) * kColumns;     // first column of this workgroup
    if (n_live <= 0 || c0 >= n_live * G) return;
    const int pos0 = L - n_q;                                    // position of the chunk's first token
    const int wg_last = prefill_last_token(c0, kColumns, G, n_live);
    const int kv_end = pos0 + wg_last + 1;                       // the workgroup's queries see tokens 0 .. kv_end - 1
    const int n_tiles = (kv_end + kTile - 1) / kTile;
    const int n_steps = (n_tiles + 1) >> 1;
    // this workgroup's share of the steps (see prefill_mfma.hpp)
    const int ns_eff = prefill_effective_splits(NS, n_steps, p.min_split_steps);
    if (split >= ns_eff) return;
    const int s_begin = (int)((long long)n_steps * split / ns_eff);
    const int s_end = (int)((long long)n_steps * (split + 1) / ns_eff);

    // ---- this lane's column: query token, head, position; and the queries as MFMA B operands
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int c = c0 + wave * 32 + col;
    const int qi = c / G, g = c - qi * G;
    const bool live = qi < n_live;
    const int pos = live ? pos0 + qi : -1;                       // -1: padding column (never stored)
    const size_t row = ((size_t)(p.q_offsets[b] + qi) * p.Hq + head0 + g) * D;
    uint4 Q[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        Q[kk] = make_uint4(0, 0, 0, 0);
        if (live) Q[kk] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(p.q) + row * 2 + (2 * kk + h) * 16);
    }
    int wave_max_pos = pos, wave_min_pos = live ? pos : 0x7fffffff;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
        wave_max_pos = max(wave_max_pos, __shfl_xor(wave_max_pos, off));
        wave_min_pos = min(wave_min_pos, __shfl_xor(wave_min_pos, off));
    }
    wave_max_pos = __builtin_amdgcn_readfirstlane(wave_max_pos);
    wave_min_pos = __builtin_amdgcn_readfirstlane(wave_min_pos);

    // ---- staging.  A step is a whole number of pages, so a piece's place in its page is the same in every step; its page
    // is looked up one step before the rows are fetched.  Rows beyond kv_end are staged as zeros (whatever their slots
    // hold, a weight of zero times it is zero).
    const unsigned page_stride = (unsigned)(p.Hkv * PS * RB);    // gridDim.y bounds Hkv: fits 32 bits
    const int32_t *bt = p.block_table + (size_t)b * p.MB;
    const int last_page = (L - 1) >> kLog2Ps;
    const int st_tok = threadIdx.x / kChunks, st_chunk = threadIdx.x % kChunks;
    const char *k_src[NP], *v_src[NP];
    int first_page[NP], pg[NP];
    uint4 sk[NP], sv[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int t = st_tok + i * kTokStride;
        const size_t off = ((size_t)kvh * PS + (t & (PS - 1))) * RB + st_chunk * 16;
        k_src[i] = reinterpret_cast<const char *>(p.k_cache) + off;
        v_src[i] = reinterpret_cast<const char *>(p.v_cache) + off;
        first_page[i] = t >> kLog2Ps;
    }
    auto lookup = [&](int step) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) pg[i] = bt[(unsigned)min(step * (kStep / PS) + first_page[i], last_page)];
    };
    auto fetch = [&](auto fast, int step) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const bool in = decltype(fast)::value || (step < s_end && step * kStep + st_tok + i * kTokStride < kv_end);
            const unsigned long long off = (unsigned long long)(unsigned)pg[i] * page_stride;
            sk[i] = sv[i] = make_uint4(0, 0, 0, 0);
            if (in) {
                sk[i] = *reinterpret_cast<const uint4 *>(k_src[i] + off);
                sv[i] = *reinterpret_cast<const uint4 *>(v_src[i] + off);
            }
        }
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int t = st_tok + i * kTokStride;
            *reinterpret_cast<uint4 *>(&k_lds[buf][t * kKRow + st_chunk * 16]) = sk[i];
            *reinterpret_cast<uint4 *>(&v_lds[buf][t * kVRow + st_chunk * 16]) = sv[i];
        }
    };

    // ---- the column's online-softmax state, and a tile's work
    float m = -INFINITY, l = 0.f;
    f32x16_t acc[2] = {{}, {}};                                  // acc[e][r] = O^T[dim 32 e + 8 (r / 4) + 4 h + r % 4][column]
    auto tile = [&](auto fast, int t, const char *ks, const char *vs) __attribute__((always_inline)) {
        const int tb = t * kTile;
        f32x16_t S = {};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            S = mfma32_bf16(*reinterpret_cast<const uint4 *>(ks + col * kKRow + (2 * kk + h) * 16), Q[kk], S);
        if constexpr (!decltype(fast)::value) {
            if (tb + kTile - 1 > wave_min_pos) {                 // tokens after the column's position
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (tb + 8 * (r >> 2) + 4 * h + (r & 3) > pos) S[r] = -INFINITY;
            }
        }
        // The reference m (log2 domain) is the running maximum at its last move, and moves when the weights outgrow it by
        // the limit: any common reference gives the same softmax, and at most 8 log2 units below the maximum it costs the
        // exponent's argument no precision that the score's own rounding leaves it.
        float pw[16], psum;
        auto form = [&]() __attribute__((always_inline)) {
            float s4[4];
#pragma unroll
            for (int r = 0; r < 16; ++r) pw[r] = fast_exp2(fmaf(S[r], p.scale_log2, -m));
#pragma unroll
            for (int i = 0; i < 4; ++i) s4[i] = (pw[4 * i] + pw[4 * i + 1]) + (pw[4 * i + 2] + pw[4 * i + 3]);
            psum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        };
        form();
        if (__any(!(psum < kPrefillExactLimit))) {               // also for an infinite or undefined sum
            float tmax = S[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, S[r]);
            tmax *= p.scale_log2;
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            // a column whose tokens are all masked so far keeps a finite stand-in
            const float mn = fmaxf(fmaxf(m, tmax), kNoTokenReference);
            const float alpha = fast_exp2(m - mn);               // 0 while m is still -inf
            l *= alpha;
            acc[0] *= alpha; acc[1] *= alpha;
            m = mn;
            form();
        }
        l += psum;
        // V^T operands by transposing reads: in a 16-lane group lane 4k + q names dims 4q .. 4q+3 of token k of the group's
        // four tokens and lane i receives dim i of each; two reads make the operand of 16 tokens and one 32-dim block.
        const char *v0 = vs + (4 * h + ((lane & 15) >> 2)) * kVRow + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
#pragma unroll
        for (int s16 = 0; s16 < 2; ++s16) {
            float part[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) part[r] = pw[8 * s16 + r];
            uint4 P[3];
            split_weights<3>(part, P);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint2 a0 = lds_read_tr16_b64(v0 + (16 * s16) * kVRow + e * 64);
                const uint2 a1 = lds_read_tr16_b64(v0 + (16 * s16 + 8) * kVRow + e * 64);
                const uint4 A = make_uint4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
                for (int i = 0; i < 3; ++i) acc[e] = mfma32_bf16(A, P[i], acc[e]);
            }
        }
    };

    // ---- a step: its two tiles, while the next step's rows are on their way; one barrier
    auto step = [&](auto fast, int s) __attribute__((always_inline)) {
        constexpr bool kFast = decltype(fast)::value;
        const int buf = s & 1;
        fetch(fast, s + 1);
        lookup(s + 2);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
            if (kFast || (2 * s + sub) * kTile <= wave_max_pos)
                tile(fast, 2 * s + sub, &k_lds[buf][sub * kTile * kKRow], &v_lds[buf][sub * kTile * kVRow]);
        if (kFast || s + 1 < s_end) {
            stage(buf ^ 1);
            lds_barrier();
        }
    };
    // last step whose tiles every live column of the wave sees wholly and whose fetch lies wholly inside the context
    const int fast_last = wave_max_pos < 0 ? -1 : min(min((wave_min_pos + 1) / kStep - 1, kv_end / kStep - 2), s_end - 2);
    lookup(s_begin);
    fetch(std::false_type{}, s_begin);
    lookup(s_begin + 1);
    stage(s_begin & 1);
    lds_barrier();
    for (int s = s_begin; s < s_end; ++s) {
        if (s <= fast_last) step(std::true_type{}, s);
        else step(std::false_type{}, s);
    }

    // ---- normalise and store.  The column's indices are worked out anew, from a lane number the compiler cannot trace
    // back to the first one: kept across the loop they cost registers and with those a spill in its fast step (24 requests
    // with chunks of 1 .. 1024 tokens 120.3 -> 124.3 us; this way 116.4 -> 116.6).
    int id;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(id));
    const int ecol = id & 31, eh = id >> 5;
    const int wc0 = c0 + wave * 32;                              // the wave's first column
    const int eqi = (wc0 + ecol) / G, eg = wc0 + ecol - eqi * G;
    const int epos = eqi < n_live ? pos0 + eqi : -1;
    const long long q_row0 = p.q_offsets[b];
    const float lsum = l + __shfl_xor(l, 32);                    // the two halves hold disjoint tokens
    // A column is sound if its sums are finite and its largest weight is about one.  Else it is walked again row by row:
    //  - an infinite or NaN V element is multiplied with the weights of all 32 columns, that is with zero for a query in
    //    front of it, and with the lower parts of a weight, which may be zero;
    //  - weights of up to the limit may overflow the sums of huge values;
    //  - with scores of 2^28 log2 units and more the rounding of the reference scales every weight, out of range in the end.
    // One test when the loop is done and nothing inside it.  A column that sees none of this workgroup's tokens is left out.
    float zero = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero = fmaf(acc[0][r], 0.f, fmaf(acc[1][r], 0.f, zero));
    const bool sound = zero == 0.f && lsum > 0x1p-32f && lsum < 0x1p64f;
    const unsigned long long halves = __ballot(epos >= s_begin * kStep && !sound);
    unsigned again = (unsigned)halves | (unsigned)(halves >> 32);            // by column
    if (epos >= 0 && !(again >> ecol & 1)) {
        const float inv = 1.f / lsum;                            // without a split the column saw its own position: lsum > 0
        const size_t row = ((size_t)(q_row0 + eqi) * p.Hq + head0 + eg) * D;
        const size_t pi = (((size_t)b * p.max_q_len + eqi) * p.Hq + head0 + eg) * NS + split;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int d = 32 * e + 8 * i + 4 * eh;
                if (ns_eff > 1)                                  // a piece for the merge: unnormalised, with (m, l)
                    *reinterpret_cast<float4 *>(p.part_o + pi * D + d) = make_float4(acc[e][4 * i], acc[e][4 * i + 1], acc[e][4 * i + 2], acc[e][4 * i + 3]);
                else
                    store_out4(p, row + d, make_float4(acc[e][4 * i] * inv, acc[e][4 * i + 1] * inv, acc[e][4 * i + 2] * inv, acc[e][4 * i + 3] * inv));
            }
        if (ns_eff > 1 && eh == 0) p.part_ml[pi] = make_float2(m, lsum);
    }
    const RowSource src = row_source<uint16_t, D>(p.k_cache, p.v_cache, bt, p.Hkv, kvh, kLog2Ps);
    while (again) {                                              // uniform
        const int c1 = __builtin_ctz(again), tok = (wc0 + c1) / G, h0 = wc0 + c1 - tok * G;
        const int nh = min(min(kWalkHeads, G - h0), 32 - c1);    // heads of one query token: consecutive columns
        const size_t row0 = (size_t)(q_row0 + tok) * p.Hq + head0 + h0;
        RowWalk<D> w;
        walk_rows<uint16_t, D, true>(src, reinterpret_cast<const char *>(p.q) + row0 * RB, nh, s_begin * kStep,
                                     min(s_end * kStep, pos0 + tok + 1), p.scale_log2, id, w);
#pragma unroll
        for (int i = 0; i < kWalkHeads; ++i)
            if (i < nh && (again >> (c1 + i) & 1) && id < 16) {            // every lane group has the sums: one stores them
                if (ns_eff > 1) {
                    const size_t pi = (((size_t)b * p.max_q_len + tok) * p.Hq + head0 + h0 + i) * NS + split;
                    *reinterpret_cast<float4 *>(p.part_o + pi * D + 4 * id) = make_float4(w.o[i][0], w.o[i][1], w.o[i][2], w.o[i][3]);
                    if (id == 0) p.part_ml[pi] = make_float2(w.m[i], w.l[i]);
                } else {
                    const float inv = 1.f / w.l[i];
                    store_out4(p, (row0 + i) * D + 4 * id, make_float4(w.o[i][0] * inv, w.o[i][1] * inv, w.o[i][2] * inv, w.o[i][3] * inv));
                }
            }
        again &= ~(((1u << nh) - 1) << c1);
    }
}

}  // namespace omni
