"""The fp8 append's conversion over all 65,536 bf16 values (unit scales), bit
for bit against the oracle's codes, in every kernel that stores new tokens: a
chunk's block append, the single-token append, the append inside the decode
kernels (short rows, row splits, ranges)."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa
from oracle import ref
from test_gpu_parity import torch_gpu  # noqa: F401  (the module's fixture)
from workloads import HeadSpec, SeqSpec, make_batch
from workloads.device import tensor_to_raw, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("specs,call,env", [
    ([(512, 512)], "append", None),
    ([(1 + k % 40, 1) for k in range(512)], "append", None),
    ([(1300 + k % 40, 1) for k in range(512)], "append", None),  # beside a large decode: streaming stores
    ([(1 + k % 40, 1) for k in range(512)], "step", None),
    ([(1 + k % 40, 1) for k in range(512)], "step", "MPA_SPLIT_TOKENS=16"),
    ([(1 + k % 40, 1) for k in range(512)], "step", "MPA_DECODE_RANGE=5"),
], ids=["chunk", "tokens", "tokens_streamed", "short_rows", "row_splits", "ranges"])
def test_every_bf16_value(torch_gpu, specs, call, env, monkeypatch):  # noqa: F811
    if env:
        monkeypatch.setenv(*env.split("="))
    hkv, d = 2, 64
    b = make_batch([SeqSpec(*s) for s in specs], HeadSpec(2 * hkv, hkv, d, 16), "fp8", 26)
    b.k_scale = b.v_scale = 1.0
    patterns = np.arange(1 << 16, dtype=np.uint16)
    b.k_new[:] = patterns.reshape(b.k_new.shape)
    b.v_new[:] = np.random.default_rng(27).permutation(patterns).reshape(b.v_new.shape)
    dev = to_device(b)
    args = (dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_tables, dev.seq_lens, dev.query_start_loc,
            dev.seq_lens_host, dev.qsl_host)
    print(f"[gpu] fp8 codes: {len(specs)} sequences, {call} {env}", flush=True)
    if call == "append":
        mpa.kv_append(*args, k_scale=1.0, v_scale=1.0)
    else:
        ws = mpa.alloc_workspace(dev.q, dev.k_cache, dev.block_tables, dev.seq_lens_host, dev.qsl_host, dev.scale)
        mpa.append_attention(dev.q, *args, torch_gpu.empty_like(dev.q), workspace=ws, scale=dev.scale, k_scale=1.0,
                             v_scale=1.0)
    torch_gpu.cuda.synchronize()
    kc, vc = ref.append_reference(b.k_cache, b.v_cache, b.k_new, b.v_new, b.block_tables, b.seq_lens,
                                  b.query_start_loc, 16, "fp8", k_scale=1.0, v_scale=1.0)
    assert tensor_to_raw(dev.k_cache, "fp8").tobytes() == kc.tobytes()
    assert tensor_to_raw(dev.v_cache, "fp8").tobytes() == vc.tobytes()
