"""Scores and values at the ends of their formats: what the kernels with deferred references and shared tiles make of them.

The oracle computes in fp64, so a value is compared where the oracle's is finite, and the kind of infinity (or NaN) where
it is not.
"""
import numpy as np
import pytest

from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import TOL
from test_multi_token_decode_gpu import attend, expected

pytestmark = pytest.mark.gpu


def tokens_of(wl, b):
    t = np.arange(int(wl.context_lens[b]))
    return wl.block_table[b, t // wl.ps], t % wl.ps


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
