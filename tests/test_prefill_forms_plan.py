"""The form the planner gives a prefill launch, on the host: half or whole
tiles of bf16 caches and whole tiles or dealt keys of f32 ones, at points
where the two forms' measured times are at least 3 % apart."""

import numpy as np
import pytest

import paper_2609_27085_amd as mpa


def rows(dtype, heads, chunks):
    sl = np.asarray([p + c for c, p in chunks], np.int32)
    qsl = np.concatenate([[0], np.cumsum([c for c, _ in chunks])]).astype(np.int32)
    sh = mpa.make_shape(len(chunks), *heads, 10 ** 6, 10 ** 5, int(qsl[-1]), 0.1, dtype)
    return mpa.prefill_rows(sh, sl, qsl)


@pytest.mark.parametrize("heads,chunks,expected", [
    # whole -> half (us): 41.4 -> 33.4, 53.5 -> 49.4, 92.0 -> 72.2, 20.3 -> 17.0, 82.7 -> 79.4
    ((32, 8, 128), [(1003, 500)], 128),
    ((32, 8, 128), [(2027, 0)], 128),
    ((8, 2, 128), [(4075, 0)], 128),
    ((32, 8, 128), [(491, 0)], 128),
    ((32, 8, 128), [(3001, 0)], 128),
    # 261 -> 272, 883 -> 942, 863 -> 924, 165.9 -> 176.6, 97.6 -> 105.8, 87.7 -> 92.2
    ((32, 8, 128), [(2027, 8000)], 256),
    ((32, 8, 128), [(2027, 32000)], 256),
    ((64, 8, 128), [(1014, 32000)], 256),
    ((32, 8, 128), [(2987, 2000)], 256),
    ((32, 8, 128), [(3499, 0)], 256),
    ((32, 8, 128), [(3201, 0)], 256),
    # d 64: 38.9 -> 29.5, 95.8 -> 85.2; KV-split 301 -> 317 and 105.4 -> 109.5
    ((16, 2, 64), [(2038, 0)], 128),
    ((32, 8, 64), [(2539, 2000)], 128),
    ((16, 2, 64), [(2038, 32000)], 256),
    ((16, 2, 64), [(2038, 8000)], 256),
    ((32, 8, 64), [(8171, 0)], 128),  # 1,024 workgroups: 0.946 of whole tiles' time
])
def test_bf16_form(heads, chunks, expected):
    assert rows(mpa.MPA_BF16, heads, chunks) == expected
    assert rows(mpa.MPA_FP8, heads, chunks) == 256


@pytest.mark.parametrize("heads,chunks,expected", [
    # tiles -> keys (us): 115.9 -> 56.7, 183.5 -> 148.9 (248 tiles), 189 -> 154 (256), 137 -> 103, 601 -> 470 (504)
    ((8, 2, 128), [(1024, 500)], 16),
    ((8, 2, 128), [(1984, 500)], 16),
    ((8, 2, 128), [(2048, 500)], 16),
    ((32, 8, 128), [(528, 500)], 16),
    ((8, 2, 128), [(4032, 500)], 16),
    ((16, 2, 64), [(512, 500)], 16),
    ((16, 2, 64), [(1984, 0)], 16),
    # 670 -> 745 (200 tiles), 79.9 -> 88.2 (256); d 64: 13.5 -> 18.6 (200), 32.3 -> 47.1 (496)
    ((8, 2, 128), [(1600, 8000)], 64),
    ((32, 8, 128), [(512, 500)], 64),
    ((64, 8, 64), [(200, 0)], 64),
    ((64, 8, 64), [(496, 0)], 64),
    # past 512 tiles
    ((8, 2, 128), [(4800, 0)], 64),
])
def test_f32_form(heads, chunks, expected):
    assert rows(mpa.MPA_F32, heads, chunks) == expected


def test_one_form_per_launch():
    # 64 segments a launch: the second launch of 66 prompts holds the two longest
    chunks = [(300, 0)] * 64 + [(301, 0)] * 2
    sl = np.asarray([c for c, _ in chunks], np.int32)
    qsl = np.concatenate([[0], np.cumsum(sl)]).astype(np.int32)
    sh = mpa.make_shape(len(chunks), 8, 2, 128, 10 ** 6, 10 ** 5, int(qsl[-1]), 0.1, mpa.MPA_BF16)
    assert [mpa.prefill_rows(sh, sl, qsl, k) for k in range(2)] == [256, 128]
    for bad in (-1, 2):
        with pytest.raises(mpa.MpaError):
            mpa.prefill_rows(sh, sl, qsl, bad)
