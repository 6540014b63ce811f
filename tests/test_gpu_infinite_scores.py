"""Keys whose score is -inf (a key element of -inf against a positive query
element) have probability 0 wherever the keys are cut into parts: a part, a
wave's share or a tile that holds only such keys adds nothing, and a row that
sees nothing else has the log-sum-exp -inf."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa  # noqa: F401
from test_gpu_parity import LSE_TOL, assert_close, as_f64, bf16_to_f32, oracle_for, run_step, torch_gpu  # noqa: F401
from workloads import HeadSpec, SeqSpec, bf16_bits_from_f32, make_batch
from workloads.device import to_device

pytestmark = pytest.mark.gpu


def masked_batch(specs, heads, dtype, seed, dead):
    """A batch whose queries are positive in dim 0 and whose sequence s has
    -inf in dim 0 of its cached or new keys at the positions dead[s]."""
    b = make_batch([SeqSpec(n, c) for n, c in specs], HeadSpec(*heads, 16), dtype, np.random.default_rng(seed))
    to_bits = bf16_bits_from_f32 if dtype == "bf16" else np.float32
    q0 = bf16_to_f32(b.q[:, :, 0]) if dtype == "bf16" else b.q[:, :, 0]
    b.q[:, :, 0] = to_bits(np.abs(q0) + np.float32(0.5))
    low = to_bits(np.array([-np.inf], np.float32))[0]
    for s, positions in enumerate(dead):
        n, c = specs[s]
        for p in positions:
            if p >= n - c:
                b.k_new[int(b.query_start_loc[s]) + p - (n - c), :, 0] = low
            else:
                b.k_cache[b.block_tables[s, p // 16], :, 0, p % 16, 0] = low
    return b


def check(b, what):
    out, lse = run_step(to_device(b))
    with np.errstate(invalid="ignore", divide="ignore"):
        o_ref, l_ref = oracle_for(b)
    got, lg = as_f64(out), lse.cpu().numpy().astype(np.float64)
    seen = np.isfinite(l_ref).all(axis=1)
    print(f"[gpu] {what}: {int(seen.sum())} rows with finite scores, {int((~seen).sum())} without", flush=True)
    assert_close(got[seen], o_ref[seen], b.dtype, what)
    assert np.abs(lg[seen] - l_ref[seen]).max() <= LSE_TOL[b.dtype]
    assert (lg[~seen] == -np.inf).all(), lg[~seen]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("override", ["MPA_SPLIT_TOKENS=128", "MPA_DECODE_RANGE=8"])
def test_split_rows(torch_gpu, dtype, override, monkeypatch):  # noqa: F811
    """40 and 80 parts: a quarter of them (a wave of the wide merge), the first
    64 (a group of the merge) or all of them without a finite score."""
    monkeypatch.setenv(*override.split("="))
    specs = [(5000, 1), (10000, 1), (3000, 1), (300, 1)]
    dead = [range(0, 1500), range(0, 8500), range(3000), range(150, 290)]
    check(masked_batch(specs, (8, 2, 128), dtype, 900, dead), f"split rows {dtype} {override}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (10, 2, 64)], ids=lambda h: f"hq{h[0]}_hkv{h[1]}_d{h[2]}")
def test_short_rows(torch_gpu, dtype, heads):  # noqa: F811
    specs = [(300, 1), (400, 1), (17, 1), (200, 1)]
    dead = [range(0, 200), range(60, 399), range(17), range(200)]
    check(masked_batch(specs, heads, dtype, 901, dead), f"short rows {dtype}")


@pytest.mark.parametrize("heads", [(8, 2, 128), (10, 2, 64)], ids=lambda h: f"hq{h[0]}_hkv{h[1]}_d{h[2]}")
def test_f32_chunk(torch_gpu, heads):  # noqa: F811
    check(masked_batch([(90, 90), (400, 100)], heads, "f32", 902, [range(20), range(0, 310)]), "f32 chunks")


@pytest.mark.parametrize("splits", ["1", "2", "3"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (10, 2, 64)], ids=lambda h: f"hq{h[0]}_hkv{h[1]}_d{h[2]}")
def test_bf16_chunk(torch_gpu, heads, splits, monkeypatch):  # noqa: F811
    """Whole 64-key tiles without a finite score: a chunk's first, those where
    its KV splits begin, and one with a finite score for some rows only."""
    monkeypatch.setenv("MPA_PREFILL_SPLITS", splits)
    specs = [(2148, 100), (1500, 200), (150, 150)]
    dead = [[*range(0, 64), *range(640, 1280)], range(0, 1200), range(20)]
    check(masked_batch(specs, heads, "bf16", 903, dead), f"bf16 chunks in {splits}")
