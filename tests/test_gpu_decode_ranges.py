"""Decode rows dealt to the waves as ranges of cache blocks (the rows laid end
to end and cut every `range` blocks) against the oracle: one-block parts (300
parts in one row: the merge's groups of 64, and its form for few rows of many
parts), ranges that cross several rows, rows that begin or end on a range's
edge, and one range over the whole launch.  The new tokens are written by the
decode kernel (one call) or before it (two calls), to the same bits."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from test_gpu_parity import (as_f64, assert_close, check_batch, oracle_for, run_step,  # noqa: F401  (torch_gpu: the
                             torch_gpu)                                                # module's fixture)
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
    # fp8 rows are split on their own while one round of the device's waves holds their parts
    lens = [int(n) for n in rng.integers(2000, 8000, size=80 if dtype == "fp8" else 24)]
    b = make_batch([SeqSpec(n, 1) for n in lens], HeadSpec(16, 16, 64), dtype, rng)
    info = info_of(b)
    assert info.split_tokens % 16 == 0 and info.num_decode_items == parts(lens, info.split_tokens // 16)
    check_batch(b, f"ranges of {info.split_tokens} tokens, {info.num_decode_items} parts", fused=True)


def plan_of(heads, lens, dtype):
    sl = np.asarray(lens, np.int32)
    qsl = np.arange(len(lens) + 1, dtype=np.int32)
    sh = mpa.make_shape(len(lens), *heads, 10 ** 6, 10 ** 5, len(lens), 0.1, DTYPE[dtype], k_scale=0.01, v_scale=0.01)
    return mpa.plan_info(sh, sl, qsl), mpa.workspace_size(sh, sl, qsl)


def row_parts(lens, split):
    """Parts of rows that are split on their own."""
    per = [-(-n // -(-n // split)) for n in lens]
    return sum(-(-n // max(16, -(-p // 16) * 16)) for n, p in zip(lens, per))


@pytest.mark.parametrize("dtype,heads,crowded,spread", [
    # 805 -> 994 us as ranges; 821 -> 741
    ("bf16", (32, 8, 128), [131072] * 8 + [1 + k % 64 for k in range(248)], [65536] * 16 + [300] * 240),
    # 185 -> 261; 174 -> 161
    ("bf16", (32, 8, 64), [65536] * 8 + [32] * 64, [100 + 31 * k for k in range(256)]),
    # 719 -> 953; 379 -> 342
    ("f32", (32, 8, 128), [65536] * 8 + [32] * 64, [1100] * 256),
    # 448 -> 575; 204 -> 182
    ("fp8", (32, 8, 128), [131072] * 8 + [1 + k % 64 for k in range(248)], [100 + 31 * k for k in range(256)]),
    # splits that fill one round of waves: 35.1 -> 38.8; more: 83.8 -> 81.7 (without tokens)
    ("fp8", (32, 8, 64), [1100] * 128, [100 + 31 * k for k in range(256)]),
], ids=lambda x: x if isinstance(x, str) else "")
def test_rows_that_crowd_a_range_are_split(torch_gpu, dtype, heads, crowded, spread):  # noqa: F811
    """A wave walks the rows of its range one after another: a batch whose
    fullest range holds many rows for its blocks is split row by row."""
    for lens in (crowded, crowded[::-1]):
        info, _ = plan_of(heads, lens, dtype)
        assert info.split_tokens <= 1024 and info.num_decode_items == row_parts(lens, info.split_tokens)
    info, _ = plan_of(heads, spread, dtype)
    assert info.num_decode_items == parts(spread, info.split_tokens // 16)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_crowded_batch(torch_gpu, dtype):  # noqa: F811
    lens = [9000, 11000] + [1 + k % 40 for k in range(100)] + [8000]
    b = make_batch([SeqSpec(n, 1) for n in lens], HeadSpec(16, 16, 64), dtype, np.random.default_rng(811))
    assert info_of(b).num_decode_items == row_parts(lens, info_of(b).split_tokens)
    check_batch(b, f"long rows before short ones {dtype}", fused=True)


def test_ranges_give_way_to_row_splits_past_the_fixed_array(torch_gpu):  # noqa: F811
    """Ranges cut every launch of 256 rows at 287 places, row splits cut each
    of these rows at most once: past the no-allocation call's array the step
    takes those."""
    heads = (128, 8, 128)
    few, ws = plan_of(heads, [700] * 1280, "bf16")
    r = few.split_tokens // 16
    assert few.num_decode_items == 5 * parts([700] * 256, r) > row_parts([700] * 1280, 1024)
    assert ws <= mpa.MPA_SCRATCH_BYTES
    last = -(-208 * 44 // 288)  # the last launch's range
    assert (7 * parts([700] * 256, r) + parts([700] * 208, last)) * 128 * 130 * 4 > mpa.MPA_SCRATCH_BYTES
    lens = [700] * 2000
    many, ws = plan_of(heads, lens, "bf16")
    assert many.num_decode_items == row_parts(lens, many.split_tokens) and ws <= mpa.MPA_SCRATCH_BYTES


@pytest.mark.parametrize("route,dtype,specs", [
    ("MPA_DECODE_RANGE=7", "bf16", [(100, 1), (260, 1), (40, 1), (900, 1)]),
    ("MPA_DECODE_RANGE=7", "f32", [(100, 1), (260, 1), (40, 1), (900, 1)]),
    ("MPA_DECODE_RANGE=7", "fp8", [(100, 1), (260, 1), (40, 1), (900, 1)]),
    ("MPA_SPLIT_TOKENS=128", "fp8", [(100, 1), (260, 1), (40, 1), (900, 1)]),
    ("", "bf16", [(100, 1), (260, 1), (40, 1), (900, 1)]),  # short rows
    ("", "f32", [(100, 100), (260, 60), (300, 40)]),        # keys dealt to the waves
    ("", "bf16", [(100, 100), (260, 60), (300, 40)]),       # half tiles
], ids=lambda x: x.replace("=", "") if isinstance(x, str) else "")
def test_bad_block_id(torch_gpu, route, dtype, specs, monkeypatch):  # noqa: F811
    """A block id outside the pool in the device's table makes the rows that
    read it NaN and leaves the others right, in each kernel's own walk."""
    if route:
        monkeypatch.setenv(*route.split("="))
    b = make_batch([SeqSpec(*s) for s in specs], HeadSpec(8, 2, 64), dtype, np.random.default_rng(812))
    if not route and specs[0][1] > 1:
        sh = mpa.make_shape(b.num_seqs, 8, 2, 64, b.num_blocks, b.block_tables.shape[1], b.total_q, b.scale,
                            DTYPE[dtype])
        assert mpa.prefill_rows(sh, b.seq_lens, b.query_start_loc) == {"f32": 16, "bf16": 128}[dtype]
    o_ref, _ = oracle_for(b)
    d = to_device(b)
    mpa.kv_append(d.k_new, d.v_new, d.k_cache, d.v_cache, d.block_tables, d.seq_lens, d.query_start_loc,
                  d.seq_lens_host, d.qsl_host, k_scale=d.k_scale, v_scale=d.v_scale)
    bt = d.block_tables.clone()
    bt[1, 3] = b.num_blocks + 1000  # sequence 1, keys 48-63: read by all its rows
    out = torch_gpu.zeros_like(d.q)
    ws = mpa.alloc_workspace(d.q, d.k_cache, d.block_tables, d.seq_lens_host, d.qsl_host, d.scale)
    print(f"[gpu] bad block id {route} {dtype}", flush=True)
    mpa.mixed_paged_attention(d.q, d.k_cache, d.v_cache, bt, d.seq_lens, d.query_start_loc, d.seq_lens_host,
                              d.qsl_host, out, workspace=ws, scale=d.scale, k_scale=d.k_scale, v_scale=d.v_scale)
    torch_gpu.cuda.synchronize()
    got = as_f64(out)
    t0, t1 = int(b.query_start_loc[1]), int(b.query_start_loc[2])
    assert np.isnan(got[t0:t1]).all()
    others = np.r_[0:t0, t1:b.total_q]
    assert_close(got[others], o_ref[others], dtype, "rows that do not read the bad block")


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


@pytest.fixture(scope="module")
def ranged_step(torch_gpu):  # noqa: F811
    """A step whose decode rows are dealt as ranges, beside chunks that are
    split, on the device."""
    rng = np.random.default_rng(815)
    specs = [SeqSpec(int(n), 1) for n in rng.integers(2000, 8000, size=24)]
    specs += [SeqSpec(3000 + 100, 100), SeqSpec(700, 700)]
    b = make_batch(specs, HeadSpec(16, 16, 64), "bf16", rng)
    info = info_of(b)
    assert info.num_decode_items == parts([n.ctx for n in specs[:24]], info.split_tokens // 16)
    assert info.prefill_max_splits > 1
    return to_device(b)


def test_graph_replays_of_ranges(torch_gpu, ranged_step):  # noqa: F811
    torch, d = torch_gpu, ranged_step
    out, lse = torch.full_like(d.q, float("nan")), torch.full(d.q.shape[:2], float("nan"), device=d.q.device)
    ws = mpa.alloc_workspace(d.q, d.k_cache, d.block_tables, d.seq_lens_host, d.qsl_host, d.scale)

    def step():
        mpa.append_attention(d.q, d.k_new, d.v_new, d.k_cache, d.v_cache, d.block_tables, d.seq_lens,
                             d.query_start_loc, d.seq_lens_host, d.qsl_host, out, lse=lse, workspace=ws, scale=d.scale)

    step()
    torch.cuda.synchronize()
    eager = [t.clone() for t in (out, lse, d.k_cache, d.v_cache)]
    assert torch.isfinite(eager[0]).all()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(3):
        out.fill_(float("nan"))
        lse.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, got, e in zip(("out", "lse", "K", "V"), (out, lse, d.k_cache, d.v_cache), eager):
            assert torch.equal(got.view(torch.uint8), e.view(torch.uint8)), (replay, name)


def test_coexec_modes_of_ranges(torch_gpu, ranged_step):  # noqa: F811
    torch, d = torch_gpu, ranged_step
    mpa.kv_append(d.k_new, d.v_new, d.k_cache, d.v_cache, d.block_tables, d.seq_lens, d.query_start_loc,
                  d.seq_lens_host, d.qsl_host)
    ws = mpa.alloc_workspace(d.q, d.k_cache, d.block_tables, d.seq_lens_host, d.qsl_host, d.scale)
    args = (d.q, d.k_cache, d.v_cache, d.block_tables, d.seq_lens, d.query_start_loc, d.seq_lens_host, d.qsl_host)
    o0, l0 = torch.full_like(d.q, float("nan")), torch.full(d.q.shape[:2], float("nan"), device=d.q.device)
    mpa.mixed_paged_attention(*args, o0, lse=l0, workspace=ws, scale=d.scale)
    torch.cuda.synchronize()
    assert torch.isfinite(o0).all()
    for mode in (1, 2, 3):
        o, l = torch.full_like(d.q, float("nan")), torch.full_like(l0, float("nan"))
        assert mpa.coexec_attention(*args, o, lse=l, workspace=ws, scale=d.scale, mode=mode) == mode
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), o0.view(torch.int16)) and torch.equal(l, l0), mode


@pytest.mark.parametrize("dtype, rows, ctx, waves", [("bf16", 100, 3000, 2304), ("bf16", 256, 6000, 2304),
                                                     ("fp8", 256, 6000, 3072)])
def test_ranges_are_one_round_on_three_quarters_of_the_device(torch_gpu, dtype, rows, ctx, waves):  # noqa: F811
    """12 waves of 128-wide heads to a CU: 3072 on the device, 2304 on 192 CUs.  bf16 ranges are one round there; fp8
    ranges take every slot."""
    sl = np.full(rows, ctx, np.int32)
    sh = mpa.make_shape(num_seqs=rows, num_q_heads=32, num_kv_heads=8, head_dim=128, num_blocks=1 << 20,
                        max_blocks_per_seq=512, total_q_tokens=rows, scale=0.088, dtype=DTYPE[dtype])
    info = mpa.plan_info(sh, sl, np.arange(rows + 1, dtype=np.int32))
    want = -(-rows * -(-ctx // 16) // (waves // 8))
    assert info.split_tokens == 16 * want and info.num_decode_items == parts(sl, want)


def test_planner_keeps_partitioned_steps_beside_ranges(torch_gpu):  # noqa: F811
    """The modes that measured fastest with the decode half in ranges: agentic 3.43 ms on a quarter of the CUs (3.71 on
    one stream), budget4096 1.32 on three quarters (1.37); lent and longctx on one stream."""
    from workloads.configs import config_specs

    for cfg, mode in {"agentic": 1, "budget4096": 3, "lent": 0, "longctx": 0, "decode8b": 0}.items():
        specs, h, _, _ = config_specs(cfg, 0)
        sl = np.asarray([s.ctx for s in specs], np.int32)
        qsl = np.concatenate([[0], np.cumsum([s.q_len for s in specs])]).astype(np.int32)
        sh = mpa.make_shape(num_seqs=len(sl), num_q_heads=h.num_q_heads, num_kv_heads=h.num_kv_heads,
                            head_dim=h.head_dim, num_blocks=1 << 20, max_blocks_per_seq=1 << 14,
                            total_q_tokens=int(qsl[-1]), scale=0.088, dtype=mpa.MPA_BF16)
        assert mpa.plan_coexec(sh, sl, qsl)[0] == mode, cfg
