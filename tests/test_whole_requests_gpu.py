"""Decode calls over short contexts, where a workgroup takes one request whole and no merge follows: against the oracle, and
against the same handle with a tuned number of workgroups, which keeps the plan of equal ranges.

Bars: the cache formats' own (2e-3 for 16-bit softmax weights, 1e-5 for 24-bit ones).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import DeviceBatch, bits_of, to_dev
from test_fp8_gpu import Fp8Batch, ref_of
from test_multi_token_decode_gpu import queries

pytestmark = pytest.mark.gpu

# no token, one, tile and page edges, fewer tiles than waves, uneven runs, the longest (24 tiles; 8 over fp32 caches)
LENS = {W.BF16: [0, 1, 15, 16, 17, 31, 32, 33, 64, 65, 96, 127, 129, 250, 511, 513, 737, 768],
        W.F32: [0, 1, 15, 16, 17, 31, 32, 33, 64, 65, 96, 97, 128, 129, 200, 255, 256]}
PLANNED = {omni.OMNI_TUNE_TARGET_WORKGROUPS: 256}


def parts(h):
    return h.omni_debug_last_plan()["request_parts"]


@pytest.mark.parametrize("ps", [16, 32])
@pytest.mark.parametrize("G,Hkv", [(1, 3), (5, 1), (7, 4), (8, 8), (16, 2)])
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.BF16, 64), (W.F32, 64), (W.F32, 128)])
def test_edge_lengths_and_the_fused_step(dtype, D, G, Hkv, ps):
    lens = LENS[dtype]
    wl = W.build("whole", 3000 + G + D, lens, Hq=G * Hkv, Hkv=Hkv, D=D, ps=ps, dtype=dtype, pool_factor=1.4, append=True)
    tol = 2e-3 if (dtype, D) == (W.BF16, 128) else 1e-5
    fused = {}
    for name, tuning in (("whole", None), ("planned", PLANNED)):
        dev = DeviceBatch(wl, tuning=tuning)
        dev.out.fill_(float("nan"))
        dev.h.omni_decode_step(dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens,
                               float(wl.scale), dev.out)
        torch.cuda.synchronize()
        fused[name] = dev.out.cpu().numpy().astype(np.float64)
        assert np.array_equal(dev.attend(), fused[name]), name               # over the rows the step has written
        if name == "whole" and not (dtype == W.F32 and D == 128 and G > 6):  # 512-byte rows leave no room for more states
            assert parts(dev.h) == wl.B and dev.h.omni_debug_last_plan()["total_tokens"] == wl.total_tokens
        pools = dev.k_cache, dev.v_cache
    oracle.kv_append(wl.k_new, wl.v_new, wl.k_cache, wl.v_cache, wl.block_table, wl.positions, wl.dtype)
    for got, want in zip(pools, (wl.k_cache, wl.v_cache)):
        assert np.array_equal(bits_of(got).view(np.uint8), np.ascontiguousarray(want).view(np.uint8))
    ref = oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype)
    for name, got in fused.items():
        assert np.all(got[0] == 0) and np.max(np.abs(got - ref)) <= tol, name


@pytest.mark.parametrize("G,Hkv,ps", [(1, 3, 16), (7, 4, 32), (16, 2, 16)])
def test_8_bit_cache(G, Hkv, ps):
    wl = W.build("whole8", 3100 + G, LENS[W.BF16], Hq=G * Hkv, Hkv=Hkv, D=128, ps=ps, dtype=W.BF16, pool_factor=1.4)
    f8 = W.quantize_fp8(wl)
    dev = Fp8Batch(wl, f8)
    got = dev.attend()
    assert parts(dev.h) == wl.B
    assert np.all(got[0] == 0) and np.max(np.abs(got - ref_of(wl, f8))) <= 2e-3


@pytest.mark.parametrize("G,Hkv,T,ps", [(7, 4, 2, 16), (4, 2, 4, 32), (1, 3, 16, 16), (5, 1, 4, 16)])       # the last in two passes
def test_several_tokens_of_varying_number(G, Hkv, T, ps):
    wl = W.build("wholemt", 3200 + G, LENS[W.BF16], Hq=G * Hkv, Hkv=Hkv, D=128, ps=ps, dtype=W.BF16, pool_factor=1.4)
    q = queries(wl, T, 3201)
    n = np.random.default_rng(3202).integers(0, T + 1, size=wl.B).astype(np.int32)
    n = np.minimum(n, wl.context_lens).astype(np.int32)
    dev = DeviceBatch(wl, tuning={omni.OMNI_TUNE_QUERY_TOKENS: T})
    dev.h.omni_set_query_lens(torch.from_numpy(n).cuda())
    out = torch.full((wl.B, T, wl.Hq, wl.D), float("nan"), device="cuda")
    dev.h.omni_paged_decode_attn(to_dev(q, wl.dtype), dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, float(wl.scale), out)
    torch.cuda.synchronize()
    assert parts(dev.h) == wl.B
    offs = np.arange(wl.B, dtype=np.int64) * T
    ref = oracle.paged_prefill_attn(q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, n, offs, wl.scale, wl.dtype)
    ref = ref.reshape(wl.B, T, wl.Hq, wl.D)
    for b in range(wl.B):
        ref[b, n[b]:] = 0.0
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 2e-3


def test_a_context_longer_than_the_hint():
    """The hint decides the launch, not what is read: 70 tiles of a request where the hint allows 16."""
    wl = W.build("hint", 3300, [2240, 100, 0, 512], Hq=14, Hkv=2, D=128, ps=16, dtype=W.BF16)
    dev = DeviceBatch(wl, max_context_hint=512)
    got = dev.attend()
    assert parts(dev.h) == wl.B
    ref = oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype)
    assert np.max(np.abs(got - ref)) <= 2e-3


@pytest.mark.parametrize("Hkv", [1, 2, 3, 4, 6, 8, 16, 24])
def test_every_request_and_head_runs_once(Hkv):
    """However many KV heads are dealt to the compute dies: more workgroups than run at once."""
    lens = np.random.default_rng(3400).integers(0, 120, size=130)
    wl = W.build("deal", 3401, lens, Hq=2 * Hkv, Hkv=Hkv, D=64, ps=16, dtype=W.BF16)
    dev = DeviceBatch(wl)
    got = dev.attend()
    assert parts(dev.h) == wl.B
    ref = oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype)
    assert np.max(np.abs(got - ref)) <= 1e-5
