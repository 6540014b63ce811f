"""The four-wave form of the MFMA prefill kernel (128 rows per workgroup) and
the launch rule between it and the eight-wave one, against the oracle: chunks
that end inside, at and just past a half tile, group sizes that do not divide
it, KV splits at head_dim 64, and both sides of the line."""

import numpy as np
import pytest

from test_gpu_parity import check_batch, torch_gpu  # noqa: F401  (torch_gpu: the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch

pytestmark = pytest.mark.gpu

CASES = [
    ((8, 2, 128), [(31, 0), (32, 0), (33, 100), (65, 15)]),   # half tiles of 32 tokens
    ((8, 2, 128), [(1003, 0)]),
    ((10, 2, 128), [(25, 0), (26, 39), (51, 40), (200, 300)]),  # G 5: 25 tokens a half tile, 51 a whole one
    ((16, 1, 128), [(2, 0), (9, 7), (70, 500)]),
    ((7, 7, 64), [(127, 0), (129, 3), (300, 250)]),           # G 1
    ((12, 4, 64), [(43, 90), (90, 1700)]),                    # G 3, KV-split
    ((64, 8, 128), [(1790, 10)]),                             # 448 workgroups of 256 rows: whole tiles
    ((64, 8, 128), [(1760, 10)]),                             # 440: half tiles
    ((64, 8, 64), [(1790, 10)]),
]


@pytest.mark.parametrize("heads,chunks", CASES, ids=lambda x: str(x).replace(" ", ""))
def test_half_tiles(torch_gpu, heads, chunks):  # noqa: F811
    rng = np.random.default_rng(970 + heads[0])
    specs = [SeqSpec(p + c, c) for c, p in chunks] + [SeqSpec(77, 1)]
    check_batch(make_batch(specs, HeadSpec(*heads, 16), "bf16", rng), f"half tiles {chunks}")
