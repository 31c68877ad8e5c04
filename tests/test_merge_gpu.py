"""Decode calls of few requests, each cut into many pieces: waves share the pieces in the merge.  Against the oracle, and against
the same pieces put together by one thread each (a handle with few workgroups).

Bars: the cache formats' own against the oracle.  Between the two merges only the order of fp32 sums differs: each holds n
products within three roundings and n - 1 additions, so numerator and denominator are each within (n + 4) 2^-24 of the sum of
their terms' sizes, and both quotients within 2 (n + 5) 2^-24 max|v| of the exact one.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import DeviceBatch, to_dev
from test_multi_token_decode_gpu import queries

pytestmark = pytest.mark.gpu

TILE = 32
FORCED = {omni.OMNI_TUNE_FORCE_PARTITION: TILE}
FEW = {**FORCED, omni.OMNI_TUNE_TARGET_WORKGROUPS: 32}
# pieces: none, one, two, rounds of eight per wave and one more, a share with empty waves, the most
PIECES = {4: [0, 1, 2, 3, 5, 31, 32, 33, 64], 8: [0, 1, 2, 9, 63, 64, 65, 129, 150]}


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("dtype,D,G,Hkv,T", [(W.BF16, 128, 7, 2, 1), (W.BF16, 128, 5, 2, 2), (W.BF16, 64, 1, 4, 1), (W.F32, 64, 8, 2, 1),
                                               (W.F32, 128, 3, 1, 1)])
def test_waves_share_the_pieces(dtype, D, G, Hkv, T, waves):
    n = PIECES[waves]
    lens = [max(0, k * TILE - (k % 3)) for k in n]
    wl = W.build("merge", 4100 + G + waves, lens, Hq=G * Hkv, Hkv=Hkv, D=D, ps=16, dtype=dtype)
    q = queries(wl, T, 4101) if T > 1 else wl.q
    rows = np.minimum(np.full(wl.B, T), wl.context_lens).astype(np.int32)
    got = {}
    for name, tuning in (("shared", FORCED), ("alone", FEW)):
        dev = DeviceBatch(wl, tuning={**tuning, omni.OMNI_TUNE_QUERY_TOKENS: T})
        shared_bytes = dev.h.omni_debug_kernel_resources(1)["static_lds_bytes"]
        assert shared_bytes == (waves * 64 * 24 if name == "shared" else 0)
        if T > 1:
            dev.h.omni_set_query_lens(torch.from_numpy(rows).cuda())
        out = torch.full((wl.B, T, wl.Hq, wl.D), float("nan"), device="cuda")
        dev.h.omni_paged_decode_attn(to_dev(q, wl.dtype), dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens,
                                     float(wl.scale), out)
        torch.cuda.synchronize()
        got[name] = out.cpu().numpy().astype(np.float64)
    ref = oracle.paged_prefill_attn(q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, rows,
                                    np.arange(wl.B, dtype=np.int64) * T, wl.scale, wl.dtype).reshape(wl.B, T, wl.Hq, wl.D)
    tol = 2e-3 if (dtype, D) == (W.BF16, 128) else 1e-5
    v = wl.v_cache if dtype == W.F32 else W.bf16_bits_to_f32(wl.v_cache)
    for b in range(wl.B):
        live = slice(0, rows[b])
        for name, x in got.items():
            assert np.max(np.abs(x[b, live] - ref[b, live]), initial=0) <= tol, (name, n[b])
        between = np.max(np.abs(got["shared"][b, live] - got["alone"][b, live]), initial=0)
        assert between <= 4 * (n[b] + 5) * 2.0**-24 * np.nanmax(np.abs(v)), n[b]            # unused rows hold NaN
