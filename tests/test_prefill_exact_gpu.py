"""The matrix-core kernel for multi-token queries over bf16 caches with 64-dim heads, whose softmax weights keep 24 bits.

Bar: the vector-ALU kernel's 1e-5 (exact products, fp32 sums of values around one).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_02204_amd import binding as omni
from paper_2602_02204_amd import workloads as W
from gpu_util import DeviceBatch, to_dev
from test_prefill_gpu import ChunkOnDevice, run_chunk

pytestmark = pytest.mark.gpu

# one token, tile / step / page edges, empty, more tokens than one workgroup's columns hold, contexts before the chunk
LENS = [1, 31, 32, 33, 63, 64, 65, 0, 127, 129, 300, 700, 96, 40]
Q_LENS = [1, 31, 1, 33, 2, 64, 65, 0, 3, 129, 17, 150, 0, 40]


def owned_rows(ch):
    return np.concatenate([np.arange(o, o + n) for o, n in zip(ch.q_offsets, ch.q_lens)])


def reference(wl, ch, scale=None):
    oracle.kv_append_chunk(ch.k_new, ch.v_new, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets)
    return oracle.paged_prefill_attn(ch.q, wl.k_cache, wl.v_cache, wl.block_table, wl.context_lens, ch.q_lens, ch.q_offsets,
                                     wl.scale if scale is None else scale, wl.dtype)


@pytest.mark.parametrize("ps", [16, 32])
@pytest.mark.parametrize("G,Hkv", [(1, 3), (3, 1), (7, 2), (8, 2), (16, 1)])
def test_tile_and_block_edges_with_and_without_a_context_split(G, Hkv, ps):
    wl = W.build("edge", 41 + G, LENS, Hq=G * Hkv, Hkv=Hkv, D=64, ps=ps, dtype=W.BF16, pool_factor=1.3)
    ch = W.add_chunk(wl, Q_LENS, 42, gap=1)
    ref, owned = None, owned_rows(ch)
    for tuning in ({omni.OMNI_TUNE_PREFILL_SPLITS: 1}, {omni.OMNI_TUNE_PREFILL_SPLITS: 5, omni.OMNI_TUNE_PREFILL_MIN_SPLIT: 64}):
        _, got = run_chunk(wl, ch, tuning=tuning, split_workspace=True)
        ref = reference(wl, ch) if ref is None else ref
        assert np.max(np.abs(got[owned] - ref[owned])) <= 1e-5
        assert np.all(np.isnan(np.delete(got, owned, axis=0)))


@pytest.mark.parametrize("gain", [0.0, 1.0, 30.0, 1000.0])
def test_peaked_and_growing_scores_move_the_reference(gain):
    """Keys grow along the context, so the reference moves again and again.  A relative error of 2^-23 of the largest score
    (at most gain * 64 * 4 log2 units; a peaked softmax compares few of them) is an error of a weight."""
    wl = W.build("grow", 51, [400, 333], Hq=8, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ramp = W.f32_to_bf16_bits((gain * np.linspace(0, 1, 25)).astype(np.float32))
    for b in range(2):
        for i, page in enumerate(wl.block_table[b][:-(-int(wl.context_lens[b]) // 16)]):
            wl.k_cache[page, :, :, 0] = ramp[i]
    ch = W.add_chunk(wl, [100, 333], 52)
    ch.q[..., 0] = W.f32_to_bf16_bits(np.full(1, 1.0, np.float32))[0]
    _, got = run_chunk(wl, ch)
    assert np.max(np.abs(got - reference(wl, ch))) <= 1e-5 + 2.0 ** -23 * gain


@pytest.mark.parametrize("scale", [0.0, -0.125])
def test_scales_the_matrix_core_kernel_does_not_take(scale):
    wl = W.build("scale", 61, [100, 65], Hq=4, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [40, 65], 62, in_cache=True)
    dev = DeviceBatch(wl)
    c = ChunkOnDevice(dev, ch)
    dev.h.omni_paged_prefill_attn(c.q, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens, c.q_offsets,
                                  ch.max_q_len, scale, c.out)
    torch.cuda.synchronize()
    assert np.max(np.abs(c.out.cpu().numpy() - reference(wl, ch, scale))) <= 1e-5


def test_rows_beyond_a_cut_off_chunk_have_no_effect():
    """Chunks longer than max_q_len: rows after the last computed token hold NaN and stay unread or weigh exactly nothing."""
    wl = W.build("cut", 71, [150, 90], Hq=16, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [100, 60], 72, in_cache=False)                          # the chunk's rows are NaN until appended
    _, got = run_chunk(wl, ch, max_q_len=37)
    ref = reference(wl, ch)
    for o, n in zip(ch.q_offsets, ch.q_lens):
        assert np.max(np.abs(got[o:o + 37] - ref[o:o + 37])) <= 1e-5
        assert np.all(np.isnan(got[o + 37:o + n]))


@pytest.mark.parametrize("splits", [1, 4])
def test_bf16_output_rounds_the_result_once(splits):
    """Stored by the attention kernel itself and by the merge of a split context.  Eight significant bits: rounding to nearest
    moves x by at most half the spacing 2^(e - 7) of its binade 2^e <= |x|, that is 2^-8 |x|, beside the fp32 bar."""
    wl = W.build("bf16", 91, [1800, 70, 333], Hq=16, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [100, 70, 1], 92, gap=1)
    _, got = run_chunk(wl, ch, out_dtype=W.BF16, split_workspace=True,
                       tuning={omni.OMNI_TUNE_PREFILL_SPLITS: splits, omni.OMNI_TUNE_PREFILL_MIN_SPLIT: 64})
    ref, rows = reference(wl, ch), owned_rows(ch)
    assert np.all(np.abs(got[rows] - ref[rows]) <= 1e-5 + np.abs(ref[rows]) * 2.0 ** -8)
    assert np.all(np.isnan(np.delete(got, rows, axis=0)))


def test_the_librarys_own_split_and_its_repeatability():
    """One long request with a short chunk leaves most of the chip idle, so its context is split; the result is the same
    from call to call, whatever the workspace holds."""
    wl = W.build("auto", 101, [5000], Hq=16, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [40], 102)
    _, unsplit = run_chunk(wl, ch, tuning={omni.OMNI_TUNE_PREFILL_SPLITS: 1})
    dev, got = run_chunk(wl, ch, split_workspace=True)
    assert not np.array_equal(got, unsplit)
    assert np.max(np.abs(got - reference(wl, ch))) <= 1e-5
    c = ChunkOnDevice(dev, ch)
    for poison in (0.0, float("inf")):
        dev.ws.fill_(poison)
        dev.h.omni_paged_prefill_attn(c.q, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens, c.q_offsets,
                                      ch.max_q_len, float(wl.scale), c.out)
        torch.cuda.synchronize()
        assert np.array_equal(c.out.cpu().numpy().astype(np.float64), got)


@pytest.mark.parametrize("out_dtype", [W.F32, W.BF16])
def test_longest_first_order_changes_nothing_but_the_schedule(out_dtype):
    """More than 256 workgroups: ranked by context length on the device (ties, empty requests and one-token chunks
    included), every output bit is as in batch order."""
    rng = np.random.default_rng(111)
    lens = np.concatenate([rng.integers(1, 700, size=70), [0, 0, 300, 300, 300, 1, 64]]).astype(np.int64)
    q_lens = np.minimum(lens, rng.integers(0, 100, size=lens.size)).astype(np.int64)
    wl = W.build("order", 112, lens, Hq=16, Hkv=2, D=64, ps=16, dtype=W.BF16, pool_factor=1.5)
    ch = W.add_chunk(wl, q_lens, 113, gap=1)
    assert ((ch.max_q_len + 15) // 16) * wl.Hkv * wl.B > 256
    _, ranked = run_chunk(wl, ch, out_dtype=out_dtype, split_workspace=True)
    _, in_order = run_chunk(wl, ch, out_dtype=out_dtype, split_workspace=True, tuning={omni.OMNI_TUNE_PREFILL_SORT: 0})
    assert np.array_equal(ranked, in_order, equal_nan=True)
    ref, rows = reference(wl, ch), owned_rows(ch)
    assert np.all(np.abs(ranked[rows] - ref[rows]) <= 1e-5 + (np.abs(ref[rows]) * 2.0 ** -8 if out_dtype == W.BF16 else 0))


def test_pieces_of_a_cut_off_chunk_stay_inside_the_workspace():
    """Chunks longer than max_q_len with a split context: the pieces of tokens beyond the bound would land in the next
    request's rows, and those of the last request behind the workspace."""
    wl = W.build("cut", 121, [1500, 900, 700], Hq=14, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [100, 90, 50], 122)
    dev = DeviceBatch(wl)
    c = ChunkOnDevice(dev, ch)
    mq = 40
    need = dev.h.omni_prefill_workspace_bytes(mq)
    assert need > dev.h.omni_workspace_bytes()
    buf = torch.full((need + (1 << 20),), 0x5a, dtype=torch.uint8, device="cuda")
    dev.h.omni_set_workspace(buf, need)
    dev.h.omni_paged_prefill_attn(c.q, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens, c.q_offsets, mq,
                                  float(wl.scale), c.out)
    torch.cuda.synchronize()
    assert bool(torch.all(buf[need:] == 0x5a))
    got, ref = c.out.cpu().numpy(), reference(wl, ch)
    for o, n in zip(ch.q_offsets, ch.q_lens):
        assert np.max(np.abs(got[o:o + mq] - ref[o:o + mq])) <= 1e-5
        assert np.all(np.isnan(got[o + mq:o + n]))


@pytest.mark.parametrize("lens,q_len", [([1200, 900], 40), ([150] * 40, 64)], ids=["split", "ranked"])
def test_replayed_graph_follows_its_inputs(lens, q_len):
    """One graph, replayed with other queries, lengths and rows, eager work and a synchronisation between the replays: each
    replay is bit for bit the eager call, for a split context and for ranked requests."""
    wl = W.build("graph", 131, lens, Hq=16, Hkv=2, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, [q_len] * wl.B, 132)
    dev = DeviceBatch(wl)
    c = ChunkOnDevice(dev, ch)
    dev.ws = dev.h.alloc_workspace(prefill_max_q_len=q_len)
    eager = torch.empty_like(c.out)
    s = torch.cuda.Stream()

    def call(out, stream):
        dev.h.omni_kv_append_chunk(c.k_new, c.v_new, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens,
                                   c.q_offsets, q_len, stream)
        dev.h.omni_paged_prefill_attn(c.q, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens, c.q_offsets,
                                      q_len, float(wl.scale), out, stream)

    torch.cuda.synchronize()
    call(eager, s)
    torch.cuda.synchronize()
    with omni.Graph(s) as g:
        call(c.out, s)
    full = dev.context_lens.clone()
    for step in range(4):
        c.q.copy_(to_dev(W.f32_to_bf16_bits(np.random.default_rng(step).standard_normal(ch.q.shape).astype(np.float32)), W.BF16))
        dev.context_lens.copy_(full - 7 * step * (torch.arange(wl.B, device="cuda") % 3).int())
        torch.cuda.synchronize()
        call(eager, None)
        torch.cuda.synchronize()
        c.out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(c.out, eager), step
    g.close()


@pytest.mark.parametrize("lens,q_lens,max_q_len", [([3000], [300], 300), ([90] * 40, [70] * 40, 70)], ids=["split", "ranked"])
@pytest.mark.parametrize("given", ["decode-calls-bytes", "chunk-calls-bytes"])
def test_the_decode_calls_part_of_the_workspace_stays_as_it_is(lens, q_lens, max_q_len, given):
    """A decode call of the same handle may be under way on another stream: nothing of its part of the workspace changes,
    and nothing beyond the registered bytes does."""
    wl = W.build("apart", 81, lens, Hq=16, Hkv=4, D=64, ps=16, dtype=W.BF16)
    ch = W.add_chunk(wl, q_lens, 82)
    ref = reference(wl, ch)
    dev = DeviceBatch(wl, tuning={omni.OMNI_TUNE_PREFILL_MIN_SPLIT: 64})
    c = ChunkOnDevice(dev, ch)
    decode, chunk = dev.h.omni_workspace_bytes(), dev.h.omni_prefill_workspace_bytes(max_q_len)
    assert chunk > 0
    n = decode if given == "decode-calls-bytes" else max(decode, chunk)
    buf = torch.full((n + (1 << 20),), 0x5a, dtype=torch.uint8, device="cuda")
    dev.h.omni_set_workspace(buf, n)
    dev.h.omni_paged_prefill_attn(c.q, dev.k_cache, dev.v_cache, dev.block_table, dev.context_lens, c.q_lens, c.q_offsets,
                                  max_q_len, float(wl.scale), c.out)
    torch.cuda.synchronize()
    assert bool(torch.all(buf[:decode] == 0x5a)) and bool(torch.all(buf[n:] == 0x5a))
    assert bool(torch.all(buf[decode:n] == 0x5a)) == (n == decode)               # the part behind it is what the call uses
    assert np.max(np.abs(c.out.cpu().numpy() - ref)) <= 1e-5
