"""The matrix-core decode kernel on the caches whose softmax weights stay fp32-exact: fp32, and bf16 with 64-dim heads.

Bars: fp32 sums of exact products under weights of 24 bits, as in the vector-ALU kernel, hence its bar of 1e-5 also over
bf16 caches with 64-dim heads; length-1 contexts, fused appends and unowned slots bit-exact.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import DeviceBatch, bits_of, to_dev

pytestmark = pytest.mark.gpu

EDGE_LENS = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 129, 255, 257, 513, 1000]
FORMATS = [(W.F32, 64), (W.F32, 128), (W.BF16, 64)]
IDS = ["f32-64", "f32-128", "bf16-64"]


def ref_of(wl):
    return oracle.paged_decode_attn(wl.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, wl.scale, wl.dtype)


@pytest.mark.parametrize("dtype,D", FORMATS, ids=IDS)
@pytest.mark.parametrize("ps", [16, 32])
@pytest.mark.parametrize("G,Hkv", [(1, 3), (2, 2), (5, 1), (7, 2), (16, 1)])
def test_tile_edges(dtype, D, ps, G, Hkv):
    """Tile, page and range edges for every lane-to-column filling; with 512-byte rows G = 1, 2 stage K, G = 7, 16 do not."""
    wl = W.build("edge", 77 + G + D, EDGE_LENS, Hq=G * Hkv, Hkv=Hkv, D=D, ps=ps, dtype=dtype, pool_factor=1.3)
    ref = ref_of(wl)
    for pl in (0, 32, 96):
        dev = DeviceBatch(wl, tuning={omni.OMNI_TUNE_FORCE_PARTITION: pl} if pl else None)
        assert dev.h.omni_debug_lds_layout()["k_staged"] == (D * (4 if dtype == W.F32 else 2) < 512 or G <= 5)
        got = dev.attend()
        assert np.all(np.isfinite(got)) and np.all(got[0] == 0.0)
        assert np.max(np.abs(got - ref)) <= 1e-5
        v1 = wl.v_cache[wl.block_table[1, 0], :, 0, :]
        v1 = (v1 if dtype == W.F32 else W.bf16_bits_to_f32(v1)).astype(np.float64)
        assert np.array_equal(got[1], np.repeat(v1, G, axis=0))


# every variant that appends: K staged (the new rows are patched into the tile in flight) or not (they are written first)
APPENDS = [(W.F32, 64, 3, True), (W.F32, 128, 3, True), (W.BF16, 64, 3, True), (W.BF16, 64, 16, True), (W.F32, 128, 7, False),
           (W.F32, 128, 16, False)]


@pytest.mark.parametrize("dtype,D,G,staged", APPENDS, ids=[f"{'f32' if t == W.F32 else 'bf16'}-{D}-G{G}" for t, D, G, _ in APPENDS])
@pytest.mark.parametrize("ps", [16, 32])
@pytest.mark.parametrize("batch", [40, 300], ids=["wave-plan", "workgroup-plan"])
def test_fused_step_equals_append_then_attention(dtype, D, G, staged, ps, batch):
    """Many short requests per range (more than a chunk holds) and both plans; pools and outputs bit for bit."""
    rng = np.random.default_rng(5 + batch + D)
    lens = rng.choice([0, 1, 2, 16, 17, 31, 32, 33, 48, 64, 65, 200], size=batch)
    check_fused_step(W.build("step", 9 + D, lens, Hq=2 * G, Hkv=2, D=D, ps=ps, dtype=dtype, append=True), staged)


@pytest.mark.parametrize("ps", [16, 32])
def test_fused_step_of_the_largest_batch_without_staging(ps):
    """fp32 caches with 64-dim heads leave no room for staging only with 12 columns or more and thousands of requests."""
    rng = np.random.default_rng(3)
    lens = rng.choice([0, 1, 16, 17, 31, 32, 33, 40], size=4096)
    check_fused_step(W.build("step", 11, lens, Hq=16, Hkv=1, D=64, ps=ps, dtype=W.F32, append=True), False)


def check_fused_step(wl, staged):
    res = []
    for fused in (True, False):
        dev = DeviceBatch(wl, tuning={omni.OMNI_TUNE_FORCE_PARTITION: 1024})
        assert dev.h.omni_debug_lds_layout()["k_staged"] == staged
        if fused:
            dev.h.omni_decode_step(dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens,
                                   float(wl.scale), dev.out)
            torch.cuda.synchronize()
        else:
            dev.append()
            dev.attend()
        res.append([bits_of(x).view(np.uint8) for x in (dev.out, dev.k_cache, dev.v_cache)])
    assert all(np.array_equal(a, b) for a, b in zip(*res))
    oracle.kv_append(wl.k_new, wl.v_new, wl.k_cache, wl.v_cache, wl.block_table, wl.positions, wl.dtype)
    assert np.array_equal(res[0][1], wl.k_cache.view(np.uint8)) and np.array_equal(res[0][2], wl.v_cache.view(np.uint8))
    ref = ref_of(wl)
    assert np.max(np.abs(res[0][0].view(np.float32).reshape(ref.shape) - ref)) <= 1e-5


def test_subnormal_values_pass_through():
    """A length-1 context returns its V row bit for bit also where the row holds fp32 subnormals."""
    wl = W.build("tiny-values", 3, [1, 1], Hq=2, Hkv=1, D=64, ps=16, dtype=W.F32)
    for b in range(2):
        row = wl.v_cache[wl.block_table[b, 0], 0, 0]
        row[:] = np.ldexp(np.arange(1, 65, dtype=np.float32), -149 + b)
    got = DeviceBatch(wl).attend()
    assert np.array_equal(got[:, 0], np.stack([wl.v_cache[wl.block_table[b, 0], 0, 0] for b in range(2)]).astype(np.float64))


@pytest.mark.parametrize("sharp", [1.0, 4.0])
@pytest.mark.parametrize("dtype,D", FORMATS, ids=IDS)
def test_sums_are_as_accurate_as_the_vector_alu_kernels(dtype, D, sharp):
    """Both kernels take exact products and fp32 sums; the order of the sums decides how far the result is from 64 bits.
    896 (request, head) pairs: the ratio of two such errors scatters by about sqrt(2 / 896) = 5 %, hence 10 %."""
    rng = np.random.default_rng(7)
    wl = W.build("sums", 8, rng.integers(256, 2048, size=32), Hq=28, Hkv=4, D=D, ps=16, dtype=dtype)
    wl.q = wl.q * np.float32(sharp) if dtype == W.F32 else W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.q) * np.float32(sharp))
    ref = ref_of(wl)
    err = [np.linalg.norm(DeviceBatch(wl, tuning={omni.OMNI_TUNE_KERNEL: k}).attend() - ref)
           for k in (omni.KERNEL_AUTO, omni.KERNEL_VALU)]
    assert err[0] <= 1.1 * err[1], err[0] / err[1]
