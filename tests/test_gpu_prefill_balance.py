"""Prefill batches of more than two workgroups per CU that the planner cuts:
chunks whose units are long beside the others are KV-split (against the
oracle), and the last query tiles to run are (against the same batch with
every chunk whole, each of the two within the bars of the exact result, so
they are within twice the bars of each other)."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from test_gpu_parity import check_batch, torch_gpu  # noqa: F401  (torch_gpu: the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch
from workloads.device import device_step

pytestmark = pytest.mark.gpu

DTYPE = {"bf16": mpa.MPA_BF16, "fp8": mpa.MPA_FP8}


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("chunks", [[(1000, 100), (40, 9000)], [(300, 0), (17, 8001), (823, 333), (200, 64)]],
                         ids=lambda c: f"{len(c)}chunks")
def test_long_units_are_split(torch_gpu, dtype, chunks):  # noqa: F811
    rng = np.random.default_rng(950 + len(chunks))
    specs = [SeqSpec(p + c, c) for c, p in chunks] + [SeqSpec(700, 1)]
    b = make_batch(specs, HeadSpec(128, 8, 64, 16), dtype, rng)
    sh = mpa.make_shape(num_seqs=b.num_seqs, num_q_heads=128, num_kv_heads=8, head_dim=64, num_blocks=b.num_blocks,
                        max_blocks_per_seq=b.block_tables.shape[1], total_q_tokens=b.total_q, scale=b.scale,
                        dtype=DTYPE[dtype], k_scale=b.k_scale, v_scale=b.v_scale)
    info = mpa.plan_info(sh, b.seq_lens, b.query_start_loc)
    assert info.prefill_max_splits > 1 and info.num_prefill_tiles > 512
    check_batch(b, f"long units split {info.prefill_max_splits} ways {dtype}")


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("heads,chunks", [((64, 8, 64), [(2207, 3311)]), ((64, 8, 128), [(2249, 3017)]),
                                          ((80, 16, 64), [(1372, 3282), (429, 4173)])],
                         ids=["d64", "d128", "g5_two_chunks"])
def test_last_tiles_are_split(torch_gpu, dtype, heads, chunks, monkeypatch):  # noqa: F811
    torch = torch_gpu
    rng = np.random.default_rng(960)
    d = device_step([SeqSpec(p + c, c) for c, p in chunks], HeadSpec(*heads, 16), dtype, rng, 960)
    mpa.kv_append(d.k_new, d.v_new, d.k_cache, d.v_cache, d.block_tables, d.seq_lens, d.query_start_loc,
                  d.seq_lens_host, d.qsl_host, k_scale=d.k_scale, v_scale=d.v_scale)

    def run():
        shape = mpa.shape_of(d.q, d.k_cache, d.block_tables, d.seq_lens_host, d.scale, d.k_scale, d.v_scale)
        info = mpa.plan_info(shape, d.seq_lens_host, d.qsl_host)
        ws = mpa.alloc_workspace(d.q, d.k_cache, d.block_tables, d.seq_lens_host, d.qsl_host, d.scale)
        out = torch.full_like(d.q, float("nan"))
        lse = torch.full(d.q.shape[:2], float("nan"), dtype=torch.float32, device=d.q.device)
        mpa.prefill_attention(d.q, d.k_cache, d.v_cache, d.block_tables, d.seq_lens, d.query_start_loc,
                              d.seq_lens_host, d.qsl_host, out, lse=lse, workspace=ws, scale=d.scale,
                              k_scale=d.k_scale, v_scale=d.v_scale)
        torch.cuda.synchronize()
        return out.double(), lse.double(), info

    out, lse, info = run()
    monkeypatch.setenv("MPA_PREFILL_SPLITS", "1")
    whole, whole_lse, whole_info = run()
    print(f"[gpu] last tiles split {heads} {dtype}: {whole_info.num_prefill_tiles} -> {info.num_prefill_tiles} units, "
          f"up to {info.prefill_max_splits} splits", flush=True)
    assert whole_info.prefill_max_splits == 1 and info.prefill_max_splits in (3, 4)
    # fewer units than if whole chunks were split
    assert whole_info.num_prefill_tiles < info.num_prefill_tiles < 2 * whole_info.num_prefill_tiles
    err = (out - whole).abs()
    assert torch.isfinite(out).all() and err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
    assert (lse - whole_lse).abs().max() <= 4e-3
