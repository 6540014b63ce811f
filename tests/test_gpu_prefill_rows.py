"""The four-wave form of the MFMA prefill kernel (128 rows per workgroup) and
the eight-wave one against the oracle, each where the planner takes it: chunks
that end inside, at and just past a half tile, group sizes that do not divide
it, KV splits at head_dim 64, launches of 1,024 workgroups, and both sides of
the line."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from test_gpu_parity import check_batch, torch_gpu  # noqa: F401  (torch_gpu: the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch

pytestmark = pytest.mark.gpu

# heads, (tokens, prefix) of the chunks, rows per workgroup, most KV splits
CASES = [
    ((8, 2, 128), [(31, 0), (32, 0), (33, 100), (65, 15)], 128, 1),    # half tiles of 32 tokens
    ((8, 2, 128), [(1003, 0)], 128, 1),
    ((10, 2, 128), [(25, 0), (26, 39), (51, 40), (200, 300)], 128, 1),  # G 5: 25 tokens a half tile, 51 a whole one
    ((16, 1, 128), [(2, 0), (9, 7), (70, 500)], 128, 1),
    ((7, 7, 64), [(127, 0), (129, 3), (300, 250)], 128, 1),            # G 1
    ((12, 4, 64), [(43, 90), (90, 1700)], 128, 4),                     # G 3, KV-split
    ((64, 8, 128), [(1014, 0)], 128, 1),                               # 256 workgroups of 256 rows
    ((64, 8, 128), [(1270, 0)], 128, 1),                               # 320
    ((64, 8, 128), [(1494, 0)], 256, 1),                               # 376
    ((64, 8, 128), [(1790, 10)], 256, 1),
    ((64, 8, 64), [(1700, 10)], 128, 1),                               # 432
    ((64, 8, 64), [(1790, 10)], 256, 1),                               # 448
    ((128, 8, 64), [(2033, 0)], 128, 1),                               # 1,024
    ((128, 8, 64), [(500, 4000)], 256, 1),
    ((8, 2, 128), [(700, 2600)], 256, 5),
]


@pytest.mark.parametrize("heads,chunks,rows,splits", CASES, ids=lambda x: str(x).replace(" ", ""))
def test_half_tiles(torch_gpu, heads, chunks, rows, splits):  # noqa: F811
    rng = np.random.default_rng(970 + heads[0])
    specs = [SeqSpec(p + c, c) for c, p in chunks] + [SeqSpec(77, 1)]
    b = make_batch(specs, HeadSpec(*heads, 16), "bf16", rng)
    sh = mpa.make_shape(num_seqs=b.num_seqs, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2],
                        num_blocks=b.num_blocks, max_blocks_per_seq=b.block_tables.shape[1], total_q_tokens=b.total_q,
                        scale=b.scale, dtype=mpa.MPA_BF16)
    assert mpa.prefill_rows(sh, b.seq_lens, b.query_start_loc) == rows
    assert mpa.plan_info(sh, b.seq_lens, b.query_start_loc).prefill_max_splits == splits
    check_batch(b, f"{rows} rows per workgroup, {chunks}")
