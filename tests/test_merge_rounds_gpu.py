"""The merge of requests cut into many pieces: every round size of the merge kernel and its edges (4, 8, 16 pieces, several
rounds), and more elements per KV head than one workgroup takes.

Bars: fp32 caches as in the exact-format tests, 1e-5.  With queries four times as large scores reach about 30 log2 units, so a
weight's argument is rounded to 2^-20 and the result to about 3e-6 at |V| <= 4: still inside it.
"""
import numpy as np
import pytest

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import TOL, DeviceBatch
from test_multi_token_decode_gpu import attend, expected, queries

pytestmark = pytest.mark.gpu

PIECES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 50]
LENS = [max(0, 32 * n - (n % 3)) for n in PIECES]                # one-tile ranges: a piece per 32 tokens
ONE_TILE = {omni.OMNI_TUNE_FORCE_PARTITION: 32}


@pytest.mark.parametrize("D,G", [(64, 1), (64, 16), (128, 7), (128, 8), (128, 9), (128, 16)])
@pytest.mark.parametrize("sharp", [1.0, 4.0])
def test_rounds(D, G, sharp):
    wl = W.build("rounds", 400 + G + D, LENS, Hq=2 * G, Hkv=2, D=D, ps=16, dtype=W.F32)
    wl.q *= sharp
    got = DeviceBatch(wl, tuning=ONE_TILE).attend()
    ref = oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype)
    assert np.all(np.isfinite(got)) and np.all(got[0] == 0.0)
    assert np.max(np.abs(got - ref)) <= 1e-5


@pytest.mark.parametrize("G,T", [(4, 3), (7, 2), (8, 2), (2, 7), (7, 3)])
def test_rounds_with_several_query_tokens(G, T):
    """Pieces that hold only tokens a query must not see have weight 0 and no reference."""
    wl = W.build("rounds-mt", 500 + G, LENS, Hq=2 * G, Hkv=2, D=128, ps=16, dtype=W.BF16)
    q = queries(wl, T, 510 + G)
    _, got = attend(wl, q, T, ONE_TILE)
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got - expected(wl, q, T))) <= TOL[W.BF16]
