// Vector-ALU kernel for multi-token queries over the paged cache: every dtype and head size the library knows
// (fp32 / bf16, head_dim 64 / 128).  It is the multi-token call's path for fp32 caches (tolerance 1e-5), for bf16 caches
// with 64-dim heads where the scale is not positive, and for any 16-bit cache on request; it is not tuned.
//
// A wave owns one query token of one (request, KV head) and walks the token's whole context (row_walk.hpp), the G query
// heads of the group in passes of up to four (the rows are read again per pass).
#pragma once
#include "prefill_mfma.hpp"
#include "row_walk.hpp"

namespace omni {

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void prefill_valu_kernel(PrefillParams p, int log2_ps) {
    constexpr int E = D / 16;                                    // dims per lane
    const int b = blockIdx.z, kvh = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, tg = lane >> 4;
    const int L = p.context_lens[b];
    const int n_q = min(p.q_lens[b], L);
    const int qi = blockIdx.x * kWaves + wave;                   // query token inside the chunk
    if (qi >= min(n_q, p.max_q_len)) return;                     // a chunk longer than the grid's bound is cut off there
    const int pos = L - n_q + qi;                                // attends to tokens 0 .. pos
    const size_t q_row = (size_t)(p.q_offsets[b] + qi);
    const size_t row_bytes = (size_t)D * sizeof(T);
    const RowSource src = row_source<T, D>(p.k_cache, p.v_cache, p.block_table + (size_t)b * p.MB, p.Hkv, kvh, log2_ps);

    for (int g0 = 0; g0 < p.G; g0 += kWalkHeads) {
        const int nh = min(kWalkHeads, p.G - g0);
        RowWalk<D> w;
        walk_rows<T, D, false>(src, reinterpret_cast<const char *>(p.q) + (q_row * p.Hq + kvh * p.G + g0) * row_bytes, nh, 0, pos + 1,
                        p.scale_log2, lane, w);
#pragma unroll
        for (int h = 0; h < kWalkHeads; ++h) {
            if (h < nh && tg == 0) {                             // pos >= 0: at least one token, l > 0
                const float inv = 1.f / w.l[h];
                const size_t at = (q_row * p.Hq + kvh * p.G + g0 + h) * D + (size_t)c * E;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float r = w.o[h][e] * inv;
                    if (p.out_bf16) reinterpret_cast<uint16_t *>(p.out)[at + e] = float_to_bf16_rne(r);
                    else reinterpret_cast<float *>(p.out)[at + e] = r;
                }
            }
        }
    }
}

}  // namespace omni
