"""Attention at the sizes where its form changes: the last context read whole by
one workgroup and the first split one (512 keys; 1024 from 64 workgroups on),
and the prefill kernel's phases (one stage of 64 keys, a stage's first and
second half, the first stage past the three buffers, rows of the trailing waves
absent).  Against the float64 oracle, with the bound of the other attention
comparisons (bf16 probabilities and outputs)."""

import pytest

from tests.test_gpu_kernels import _attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,pos0,Hq,Hkv,hd", [
    ([6], [506], 4, 4, 64),
    ([6], [507], 4, 4, 64),
    ([3, 6], [7, 506], 8, 2, 128),
    ([6] * 8, [1018] * 7 + [100], 8, 8, 64),     # 64 workgroups, 1024 keys: whole
    ([6] * 8, [1019] * 7 + [100], 8, 8, 64),     # 1025 keys: split
    ([6] * 7, [1000] * 7, 8, 8, 64),             # 56 workgroups: split
])
def test_whole_or_split(rows, pos0, Hq, Hkv, hd):
    assert _attn_case(1, rows, pos0, Hq, Hkv, hd, seed=sum(rows) + sum(pos0)) < 1.5e-2


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,pos0", [([64], [0]), ([65], [0]), ([96], [0]), ([97], [1]), ([128], [0]), ([129], [31]),
                                       ([193], [0]), ([64, 70], [63, 250])])
def test_prefill_phases(rows, pos0, hd):
    assert _attn_case(1, rows, pos0, 8, 2, hd, seed=sum(rows) + hd) < 1.5e-2
