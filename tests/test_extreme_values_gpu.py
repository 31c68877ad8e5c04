"""Scores and values at the ends of their formats: what the kernels with deferred references and shared tiles make of them.

The oracle computes in fp64, so a value is compared where the oracle's is finite, and the kind of infinity (or NaN) where
it is not.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import TOL, DeviceBatch
from test_multi_token_decode_gpu import attend, expected
from test_prefill_gpu import run_chunk

pytestmark = pytest.mark.gpu

ONE_PIECE = {omni.OMNI_TUNE_PREFILL_SPLITS: 1}
FIVE_PIECES = {omni.OMNI_TUNE_PREFILL_SPLITS: 5, omni.OMNI_TUNE_PREFILL_MIN_SPLIT: 64}
SPLITS = pytest.mark.parametrize("tuning", [ONE_PIECE, FIVE_PIECES], ids=["one-piece", "five-pieces"])


def tokens_of(wl, b):
    t = np.arange(int(wl.context_lens[b]))
    return wl.block_table[b, t // wl.ps], t % wl.ps


def same_kind(got, ref, tol):
    """Finite where the reference is, to `tol` of the larger of one and its magnitude; else the same infinity, or NaN."""
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.all(np.abs(got[fin] - ref[fin]) <= tol * np.maximum(1.0, np.abs(ref[fin])))
    assert np.array_equal(got[~fin], ref[~fin], equal_nan=True)


def along_dim_0(shape):
    q = np.zeros(shape, np.float32)
    q[..., 0] = 1e17
    return W.f32_to_bf16_bits(q)


def far_below_zero(wl, rising):
    """Keys whose scores with those queries lie between -1e33 and -2e33, no two of a request alike: a softmax takes one row."""
    for b in range(wl.B):
        pages, slots = tokens_of(wl, b)
        t = np.arange(pages.size) % 128 / 128.0
        k = -(2.0 - t) if rising else -(1.0 + t)
        wl.k_cache[pages, :, slots, :] = 0
        wl.k_cache[pages, :, slots, 0] = W.f32_to_bf16_bits((1e16 * k).astype(np.float32))[:, None]


@pytest.mark.parametrize("rising", [False, True], ids=["falling", "rising"])
@pytest.mark.parametrize("part", [0, 32], ids=["planned", "one-tile-ranges"])
def test_decode_of_several_tokens_whose_scores_all_lie_far_below_zero(part, rising):
    wl = W.build("low", 9, [2, 33, 128, 5], Hq=4, Hkv=2, D=128, ps=16, dtype=W.BF16, scale=1.0)
    q = along_dim_0((wl.B * 3, wl.Hq, wl.D))
    far_below_zero(wl, rising)
    _, got = attend(wl, q, 3, {omni.OMNI_TUNE_FORCE_PARTITION: part})
    want = expected(wl, q, 3)
    assert np.max(np.abs(got - want)) <= TOL[W.BF16]


@pytest.mark.parametrize("rising", [False, True], ids=["falling", "rising"])
@SPLITS
def test_chunk_whose_scores_all_lie_far_below_zero(tuning, rising):
    """The largest visible score is the reference however low it is, and rounding it moves no weight out of range."""
    wl = W.build("low", 7, [100, 1, 128], Hq=4, Hkv=2, D=64, ps=16, dtype=W.BF16, scale=1.0)
    far_below_zero(wl, rising)
    ch = W.add_chunk(wl, [100, 1, 70], 8)
    ch.q[:] = along_dim_0(ch.q.shape)
    _, got = run_chunk(wl, ch, tuning={**tuning, omni.OMNI_TUNE_PREFILL_MIN_SPLIT: 64}, split_workspace=True)
    ref = oracle.paged_prefill_attn(ch.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets,
                                    wl.scale, wl.dtype)
    assert np.max(np.abs(got - ref)) <= 1e-5


def put(cache, wl, b, t, dim, value):
    pages, slots = tokens_of(wl, b)
    enc = (lambda x: x) if wl.dtype == W.F32 else W.f32_to_bf16_bits
    bits = W.BF16_NAN_BITS if wl.dtype == W.BF16 and np.isnan(value) else enc(np.array([value], np.float32))[0]
    cache[pages[t], :, slots[t], dim] = bits


@pytest.mark.parametrize("G,Hkv", [(1, 3), (5, 2), (16, 1)])
@SPLITS
def test_chunk_query_sees_nothing_of_values_behind_it(tuning, G, Hkv):
    """Infinities and NaN among the chunk's own V rows: the queries in front of them get what the oracle says, in every dim,
    the queries behind them the infinity or NaN in that dim alone."""
    wl = W.build("behind", 17 + G, [330, 64, 40], Hq=G * Hkv, Hkv=Hkv, D=64, ps=16, dtype=W.BF16)
    for b, t, dim, value in ((0, 299, 3, np.nan), (0, 301, 5, np.inf), (0, 321, 63, -np.inf), (1, 0, 0, np.inf),
                             (1, 63, 0, -np.inf), (2, 38, 9, np.nan)):
        put(wl.v_cache, wl, b, t, dim, value)
    ch = W.add_chunk(wl, [130, 64, 3], 18)
    _, got = run_chunk(wl, ch, tuning=tuning, split_workspace=True)
    ref = oracle.paged_prefill_attn(ch.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets,
                                    wl.scale, wl.dtype)
    assert np.isfinite(ref[:99]).all() and not np.isfinite(ref).all()
    same_kind(got, ref, 1e-5)


@SPLITS
def test_chunk_over_values_near_the_largest_finite_one(tuning):
    """A weighted mean of values of up to 2^120 is finite, whatever the sum of its unscaled weights does."""
    wl = W.build("huge", 27, [400, 333], Hq=8, Hkv=2, D=64, ps=16, dtype=W.BF16)
    big = (1 + np.abs(np.nan_to_num(W.bf16_bits_to_f32(wl.v_cache))).clip(0, 1)) * np.float32(2.0 ** 119)
    wl.v_cache[:] = W.f32_to_bf16_bits(big)
    ramp = W.f32_to_bf16_bits((6 * np.linspace(0, 1, 400)).astype(np.float32))
    for b in range(2):
        pages, slots = tokens_of(wl, b)
        wl.k_cache[pages, :, slots, 0] = ramp[:pages.size, None]
    ch = W.add_chunk(wl, [100, 333], 28)
    ch.q[..., 0] = W.f32_to_bf16_bits(np.full(1, 8.0, np.float32))[0]
    _, got = run_chunk(wl, ch, tuning=tuning, split_workspace=True)
    ref = oracle.paged_prefill_attn(ch.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets,
                                    wl.scale, wl.dtype)
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - ref)) <= 2e-5 * 2.0 ** 120


@pytest.mark.parametrize("D", [64, 128])
@SPLITS
def test_a_nan_key_shows_in_every_query_that_sees_it(D, tuning):
    """Its score is NaN and so is the softmax; a piece of a split context that holds it must not be left out of the sum."""
    wl = W.build("nan-key", 47, [400], Hq=4, Hkv=2, D=D, ps=16, dtype=W.BF16)
    put(wl.k_cache, wl, 0, 380, 11, np.nan)                      # query 50 of the chunk
    ch = W.add_chunk(wl, [70], 48)
    _, got = run_chunk(wl, ch, tuning=tuning, split_workspace=True)
    ref = oracle.paged_prefill_attn(ch.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets,
                                    wl.scale, wl.dtype)
    assert np.max(np.abs(got[:50] - ref[:50])) <= TOL[W.BF16] and np.all(np.isnan(got[50:]))


@pytest.mark.parametrize("fused", [False, True], ids=["attention", "fused-step"])
@pytest.mark.parametrize("part", [0, 64], ids=["planned", "two-tile-ranges"])
@pytest.mark.parametrize("dtype,D", [(W.F32, 64), (W.F32, 128), (W.BF16, 64)], ids=["f32-64", "f32-128", "bf16-64"])
def test_decode_over_infinite_values(dtype, D, part, fused):
    """An infinite V element makes its own output dim infinite (NaN where both signs meet) and leaves the others alone,
    whatever bits the weights have: a weight of one, the only token's, among them."""
    wl = W.build("inf", 37 + D, [1, 2, 40, 300, 129], Hq=10, Hkv=2, D=D, ps=16, dtype=dtype, append=fused)
    for b, t, dim, value in ((0, 0, 3, np.inf), (1, 0, 5, -np.inf), (2, 38, 0, np.inf), (2, 3, 0, -np.inf), (2, 20, 63, np.nan),
                             (3, 100, 7, np.inf), (4, 128, 9, -np.inf)):
        new = fused and t == int(wl.context_lens[b]) - 1
        if new:
            wl.v_new[b, :, dim] = value if dtype == W.F32 else W.f32_to_bf16_bits(np.array([value], np.float32))[0]
        else:
            put(wl.v_cache, wl, b, t, dim, value)
    dev = DeviceBatch(wl, tuning={omni.OMNI_TUNE_FORCE_PARTITION: part})
    if fused:
        dev.h.omni_decode_step(dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens,
                               float(wl.scale), dev.out)
        torch.cuda.synchronize()
        got = dev.out.cpu().numpy().astype(np.float64)
        oracle.kv_append(wl.k_new, wl.v_new, wl.k_cache, wl.v_cache, wl.block_table, wl.positions, wl.dtype)
    else:
        got = dev.attend()
    same_kind(got, oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype),
              1e-5)
