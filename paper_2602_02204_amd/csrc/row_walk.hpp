// A wave's walk over the rows of one request on the vector ALUs: the plain form of the attention, for any dtype and head
// size.  It is the whole of prefill_valu.hpp, and what the matrix-core kernel of prefill_exact.hpp goes back to for
// columns whose sums did not stay in range.
//
// Four tokens at a time: lane group tg = lane / 16 takes token t + tg, and the 16 lanes of a group each hold D / 16
// consecutive dims of the K / V row.  Each lane group keeps one online-softmax state (m, l, o) per head; the four are
// merged at the end, so that every lane group returns the same sums.
#pragma once
#include "common.hpp"

namespace omni {

constexpr int kWalkHeads = 4;                         // query heads per walk

template <typename T, int E>
__device__ __forceinline__ void load_row_slice(const char *row, int c, float (&x)[E]) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int v = 0; v < E / 4; ++v) {
            const float4 f = *reinterpret_cast<const float4 *>(row + (size_t)(c * E + 4 * v) * 4);
            x[4 * v] = f.x; x[4 * v + 1] = f.y; x[4 * v + 2] = f.z; x[4 * v + 3] = f.w;
        }
    } else if constexpr (E == 8) {
        const uint4 u = *reinterpret_cast<const uint4 *>(row + (size_t)c * 16);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) { x[2 * v] = bf16_bits_to_float(w[v] & 0xffffu); x[2 * v + 1] = __uint_as_float(w[v] & 0xffff0000u); }
    } else {
        const uint2 u = *reinterpret_cast<const uint2 *>(row + (size_t)c * 8);
        x[0] = bf16_bits_to_float(u.x & 0xffffu); x[1] = __uint_as_float(u.x & 0xffff0000u);
        x[2] = bf16_bits_to_float(u.y & 0xffffu); x[3] = __uint_as_float(u.y & 0xffff0000u);
    }
}

// Where the rows of one request and KV head are.
struct RowSource {
    const char *k, *v;               // pools, at the KV head
    const int32_t *block_table;      // the request's row
    size_t page_stride;              // bytes
    int log2_ps;
};

template <typename T, int D>
__device__ __forceinline__ RowSource row_source(const void *k_cache, const void *v_cache, const int32_t *block_table, int Hkv,
                                                int kvh, int log2_ps) {
    const size_t head_bytes = (sizeof(T) * D) << log2_ps;
    return RowSource{reinterpret_cast<const char *>(k_cache) + kvh * head_bytes,
                     reinterpret_cast<const char *>(v_cache) + kvh * head_bytes, block_table, Hkv * head_bytes, log2_ps};
}

template <int D>
struct RowWalk {
    float m[kWalkHeads], l[kWalkHeads], o[kWalkHeads][D / 16];   // o: dims (lane % 16) * D / 16 ..
};

__device__ __forceinline__ float subtract_rounded(float a, float b) {
#pragma clang fp contract(off)
    return a - b;
}

// Tokens t_lo .. t_hi - 1 for the nh heads whose query rows begin at `q`.  No token: m = -inf, l = 0, o = 0.
// kRoundScores: scores are rounded before the reference is subtracted, so that the largest one's weight is exactly one
// however large it is (in one multiply-subtract the reference's own rounding is left over: 2^4 log2 units at 2^28).
template <typename T, int D, bool kRoundScores>
__device__ __forceinline__ void walk_rows(const RowSource &src, const char *q, int nh, int t_lo, int t_hi, float scale_log2,
                                          int lane, RowWalk<D> &w) {
    constexpr int E = D / 16, HC = kWalkHeads;
    constexpr size_t row_bytes = sizeof(T) * D;
    const int c = lane & 15, tg = lane >> 4;
    auto other = [&](float x, int d) __attribute__((always_inline)) {        // x of lane ^ d
        return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (lane ^ d), __float_as_int(x)));
    };
    float qf[HC][E];
#pragma unroll
    for (int h = 0; h < HC; ++h) {
        w.m[h] = -INFINITY; w.l[h] = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) { qf[h][e] = 0.f; w.o[h][e] = 0.f; }
        if (h < nh) load_row_slice<T, E>(q + h * row_bytes, c, qf[h]);
    }
    for (int t0 = t_lo; t0 < t_hi; t0 += 4) {
        const int t = t0 + tg;
        if (t >= t_hi) continue;                                 // lanes of a group stay together
        const size_t off = (size_t)src.block_table[t >> src.log2_ps] * src.page_stride + (size_t)(t & ((1 << src.log2_ps) - 1)) * row_bytes;
        float k[E], v[E];
        load_row_slice<T, E>(src.k + off, c, k);
        load_row_slice<T, E>(src.v + off, c, v);
#pragma unroll
        for (int h = 0; h < HC; ++h) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) s = fmaf(qf[h][e], k[e], s);
            s += other(s, 1); s += other(s, 2); s += other(s, 4); s += other(s, 8);
            s *= scale_log2;
            const float mn = fmaxf(w.m[h], s);
            const float a = fast_exp2(w.m[h] - mn);              // exp2(-inf) = 0 on the first token
            const float p = fast_exp2(kRoundScores ? subtract_rounded(s, mn) : s - mn);
            w.l[h] = w.l[h] * a + p;
#pragma unroll
            for (int e = 0; e < E; ++e) w.o[h][e] = fmaf(p, v[e], w.o[h][e] * a);
            w.m[h] = mn;
        }
    }
    // merge the four lane groups (a group that saw no token has m = -inf, l = 0)
#pragma unroll
    for (int h = 0; h < HC; ++h) {
        if (h >= nh) continue;
#pragma unroll
        for (int d = 16; d <= 32; d <<= 1) {
            const float mo = other(w.m[h], d), lo = other(w.l[h], d);
            const float M = fmaxf(w.m[h], mo);
            const float a = w.m[h] > -INFINITY ? fast_exp2(w.m[h] - M) : 0.f;
            const float bsc = mo > -INFINITY ? fast_exp2(mo - M) : 0.f;
            w.l[h] = w.l[h] * a + lo * bsc;
#pragma unroll
            for (int e = 0; e < E; ++e) w.o[h][e] = w.o[h][e] * a + other(w.o[h][e], d) * bsc;
            w.m[h] = M;
        }
    }
}

}  // namespace omni
