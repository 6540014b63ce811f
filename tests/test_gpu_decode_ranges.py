"""Decode rows dealt to the waves as ranges of cache blocks (the rows laid end
to end and cut every `range` blocks) against the oracle: one-block parts (300
parts in one row: the merge's groups of 64, and its form for few rows of many
parts), ranges that cross several rows, rows that begin or end on a range's
edge, and one range over the whole launch.  The new tokens are written by the
decode kernel (one call) or before it (two calls), to the same bits."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from test_gpu_parity import check_batch, run_step, torch_gpu  # noqa: F401  (torch_gpu: the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch
from workloads.device import to_device

pytestmark = pytest.mark.gpu

DTYPE = {"bf16": mpa.MPA_BF16, "f32": mpa.MPA_F32, "fp8": mpa.MPA_FP8}
# 16 * 7 = 112 tokens: rows of 112 and 224 end on a 7-block range's edge when they begin on one
LENS = [112, 224, 1, 15, 16, 17, 63, 64, 65, 111, 113, 1000, 1025, 2049, 4800]


def info_of(b):
    h = b.heads
    sh = mpa.make_shape(num_seqs=b.num_seqs, num_q_heads=h.num_q_heads, num_kv_heads=h.num_kv_heads,
                        head_dim=h.head_dim, num_blocks=b.num_blocks, max_blocks_per_seq=b.block_tables.shape[1],
                        total_q_tokens=b.total_q, scale=b.scale, dtype=DTYPE[b.dtype], k_scale=b.k_scale,
                        v_scale=b.v_scale)
    return mpa.plan_info(sh, b.seq_lens, b.query_start_loc)


def parts(lens, r):
    blocks = [-(-n // 16) for n in lens]
    at = np.concatenate([[0], np.cumsum(blocks)])
    return sum((at[j] + n - 1) // r - at[j] // r + 1 for j, n in enumerate(blocks))


@pytest.mark.parametrize("dtype", ["bf16", "f32", "fp8"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (10, 2, 64)], ids=lambda h: f"hq{h[0]}_hkv{h[1]}_d{h[2]}")
@pytest.mark.parametrize("blocks", [1, 7, 64, 100000])
def test_ranges(torch_gpu, dtype, heads, blocks, monkeypatch):  # noqa: F811
    monkeypatch.setenv("MPA_DECODE_RANGE", str(blocks))
    lens = LENS if blocks > 1 else [4800, 17]
    b = make_batch([SeqSpec(n, 1) for n in lens], HeadSpec(*heads, 16), dtype, np.random.default_rng(800 + blocks))
    info = info_of(b)
    assert info.split_tokens == 16 * blocks and info.num_decode_items == parts(lens, blocks)
    _, out, lse = check_batch(b, f"decode ranges of {blocks} blocks", fused=True)
    out2, lse2 = run_step(to_device(b))
    assert torch_gpu.equal(out, out2) and torch_gpu.equal(lse, lse2)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_ranges_chosen_for_batches_that_fill_the_device(torch_gpu, dtype):  # noqa: F811
    rng = np.random.default_rng(810)
    lens = [int(n) for n in rng.integers(2000, 8000, size=24)]
    b = make_batch([SeqSpec(n, 1) for n in lens], HeadSpec(16, 16, 64), dtype, rng)
    info = info_of(b)
    assert info.split_tokens % 16 == 0 and info.num_decode_items == parts(lens, info.split_tokens // 16)
    check_batch(b, f"ranges of {info.split_tokens} tokens, {info.num_decode_items} parts", fused=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32", "fp8"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (10, 2, 64), (16, 1, 128)],
                         ids=lambda h: f"hq{h[0]}_hkv{h[1]}_d{h[2]}")
def test_short_rows(torch_gpu, dtype, heads):  # noqa: F811
    """Short rows take one workgroup per row and KV head, whose eight waves
    share the row's blocks: rows of fewer blocks than waves, of one block more
    or less than a whole share, and the longest that is not split."""
    longest = (512 if dtype == "f32" else 1024) * (128 // heads[2])
    lens = [1, 15, 16, 17, 64, 65, 112, 113, 128, 129, 145, 257, 400, longest - 1, longest]
    b = make_batch([SeqSpec(n, 1) for n in lens], HeadSpec(*heads, 16), dtype, np.random.default_rng(820))
    info = info_of(b)
    assert info.num_decode_items == len(lens)
    _, out, lse = check_batch(b, "short rows", fused=True)
    out2, lse2 = run_step(to_device(b))
    assert torch_gpu.equal(out, out2) and torch_gpu.equal(lse, lse2)
    # one key more: the rows are split
    b = make_batch([SeqSpec(n, 1) for n in lens[:-1] + [longest + 1]], HeadSpec(*heads, 16), dtype,
                   np.random.default_rng(821))
    assert info_of(b).num_decode_items > len(lens)
    check_batch(b, "one row past the short ones", fused=True)
