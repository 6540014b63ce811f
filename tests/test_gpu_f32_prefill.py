"""The two forms of the float32 prefill kernel (whole tiles, and 16 rows with
the keys dealt to eight waves) against the oracle, each where the planner takes
it, with fewer key blocks than waves, group sizes that do not divide a tile,
rows that see keys of some waves only, and launches of about one and about two
rounds of tiles."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from test_gpu_parity import check_batch, torch_gpu  # noqa: F401  (torch_gpu: the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch

pytestmark = pytest.mark.gpu

# (Hq, Hkv, d), (tokens, prefix) of the chunks, (tile, KV head) pairs, rows per workgroup
CASES = [
    ((8, 2, 128), [(2, 0)], 2, 64),                    # one key block
    ((8, 2, 64), [(17, 0), (33, 100), (5, 111)], 12, 16),
    ((10, 2, 128), [(100, 29), (13, 500)], 22, 16),    # G 5: 12 tokens a tile
    ((7, 1, 64), [(200, 1000)], 23, 16),               # G 7: 9 tokens a tile
    ((128, 8, 64), [(112, 300)], 224, 64),
    ((8, 1, 64), [(2000, 500)], 250, 16),
    ((128, 8, 64), [(128, 15)], 256, 64),
    ((128, 8, 64), [(129, 16)], 264, 64),
    ((128, 8, 64), [(129, 900)], 264, 16),
    ((16, 1, 64), [(1984, 40)], 496, 16),
    ((128, 8, 64), [(250, 40)], 504, 64),
]


@pytest.mark.parametrize("heads,chunks,tiles,rows", CASES, ids=lambda x: str(x).replace(" ", ""))
def test_f32_prefill_forms(torch_gpu, heads, chunks, tiles, rows):  # noqa: F811
    rng = np.random.default_rng(900 + tiles)
    b = make_batch([SeqSpec(p + c, c) for c, p in chunks], HeadSpec(*heads, 16), "f32", rng)
    sh = mpa.make_shape(num_seqs=b.num_seqs, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2],
                        num_blocks=b.num_blocks, max_blocks_per_seq=b.block_tables.shape[1], total_q_tokens=b.total_q,
                        scale=b.scale, dtype=mpa.MPA_F32)
    assert mpa.plan_info(sh, b.seq_lens, b.query_start_loc).num_prefill_tiles == tiles
    assert mpa.prefill_rows(sh, b.seq_lens, b.query_start_loc) == rows
    check_batch(b, f"f32 prefill, {tiles} tiles, {rows} rows per workgroup")
