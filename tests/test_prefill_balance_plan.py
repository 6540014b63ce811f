"""The planner's balancing of prefill launches that fill the device, on the
host: which batches it cuts, that the plan does not depend on the order of the
sequences, and that a step which fits the fixed array of
mpa_append_attention_noalloc with whole chunks still fits it."""

import itertools
import time

import numpy as np
import pytest

import paper_2609_27085_amd as mpa


def plan(heads, chunks):
    sl = np.asarray([p + c for c, p in chunks], np.int32)
    qsl = np.concatenate([[0], np.cumsum([c for c, _ in chunks])]).astype(np.int32)
    sh = mpa.make_shape(len(chunks), *heads, 10 ** 6, 10 ** 5, int(qsl[-1]), 0.1, mpa.MPA_BF16)
    return mpa.plan_info(sh, sl, qsl), mpa.workspace_size(sh, sl, qsl)


def whole_tiles(heads, chunks):
    qt = 256 // (heads[0] // heads[1])
    return sum(-(-c // qt) for c, _ in chunks) * heads[1]


def test_even_batches_stay_whole():
    # two full rounds of equal tiles on 256 CUs
    info, ws = plan((32, 8, 128), [(8192, 65536)])
    assert info.prefill_max_splits == 1 and ws == 0
    info, ws = plan((32, 8, 128), [(2048, 2130), (2048, 5559)])
    assert info.prefill_max_splits == 1 and ws == 0


@pytest.mark.parametrize("chunks", [[(3025, 613), (439, 35613)], [(2077, 0), (421, 19111), (64, 300)]])
def test_long_units_are_split_in_any_order(chunks):
    heads = (64, 8, 128)
    got = {(i.num_prefill_tiles, i.prefill_max_splits, ws)
           for i, ws in (plan(heads, list(c)) for c in itertools.permutations(chunks))}
    assert len(got) == 1
    tiles, splits, ws = got.pop()
    assert splits > 1 and tiles > whole_tiles(heads, chunks) >= 512 and ws > 0


def test_last_tiles_are_split():
    # 568 equal tiles on 256 CUs: the last of the third round in four parts
    info, ws = plan((64, 8, 128), [(2249, 3017)])
    assert info.prefill_max_splits == 4 and info.num_prefill_tiles == whole_tiles((64, 8, 128), [(2249, 3017)]) + 3 * 64
    assert ws == 4 * 256 * 64 * (128 + 2) * 4  # eight query tiles of 32 tokens, every head and split


def test_balance_stays_within_the_fixed_array():
    # a launch that fills the device needs no partial results with whole
    # chunks, so however it is balanced they fit the fixed array
    rng = np.random.default_rng(980)
    sizes = []
    while len(sizes) < 300:
        heads = [(32, 8, 128), (64, 8, 128), (128, 8, 128), (128, 8, 64)][rng.integers(4)]
        chunks = [(int(2 ** rng.uniform(8, 13.5)), int(2 ** rng.uniform(8, 17))) for _ in range(rng.integers(1, 5))]
        if whole_tiles(heads, chunks) < 512:
            continue
        info, ws = plan(heads, chunks)
        assert (ws > 0) == (info.prefill_max_splits > 1) and ws <= mpa.MPA_SCRATCH_BYTES
        sizes.append(ws)
    assert sum(n > 0 for n in sizes) > 30 and max(sizes) > mpa.MPA_SCRATCH_BYTES // 2


def test_launches_too_long_to_end_unevenly_are_not_simulated():
    # 60 chunks of 8,192 tokens on 8,192, 10 KV heads: the longest of 98,400
    # units is 0.5 % of a CU's share.  Dealing them all out took the planner
    # 3.9 ms; the pass over the units takes 0.1 ms
    chunks = [(8192, 8192)] * 60
    plan((40, 10, 128), chunks)
    best = 1.0
    for k in range(10):
        t = time.perf_counter()
        info, ws = plan((40, 10, 128), [(8192 - k, 8192)] + chunks[1:])
        best = min(best, time.perf_counter() - t)
        assert info.prefill_max_splits == 1 and ws == 0
    assert best < 1.5e-3, best
