"""Attention at the sizes where its form changes: the last context read whole by
one workgroup and the first split one (512 keys; 1024 from 64 workgroups on),
and the prefill kernel's phases (one stage of 64 keys, a stage's first and
second half, the first stage past the three buffers, rows of the trailing waves
absent).  Against the float64 oracle, with the bound of the other attention
comparisons (bf16 probabilities and outputs)."""

import pytest

from tests.gpu_util import device, say, torch
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


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("pos0", [40, 300, 1500])
def test_probabilities_below_the_normal_range(pos0, hd):
    """A key whose probability is below 2^-126 of the largest still counts: its
    value is 2^126.  Base-2 logits of 0 and, for the 16 keys of page 0, about
    -127; bf16 probabilities there hold 7 bits, like the value below: a bound
    of 2^-6 on the sum of equal terms."""
    import numpy as np
    from paper_2607_20507_amd import binding as B
    dev, H, rows = device(), 2, 3
    n = (pos0 + rows + 15) // 16
    kp = torch.zeros(n, H, 16, hd, device=dev)
    vp = torch.zeros(n, H, hd, 16, device=dev)
    kp[0] = -88.0 / hd ** 0.5
    vp[0] = 2.0 ** 126
    kp, vp = kp.bfloat16(), vp.bfloat16()
    q = torch.ones(rows, H, hd, device=dev).bfloat16()
    out = torch.zeros(rows, H * hd, device=dev).bfloat16()
    ws = torch.empty(B.spec_op_attention_workspace_bytes(1, rows, n, H, hd) + 8192, dtype=torch.uint8, device=dev)
    say("small probabilities", pos0, hd)
    B.spec_op_attention(B.SPEC_BF16, [rows], [pos0], np.arange(n, dtype=np.int32)[None], H, H, hd, q, kp, vp, out, ws)
    torch.cuda.synchronize()
    e = np.exp(float(kp[0, 0, 0, 0]) * hd ** 0.5)
    assert 0 < e < 2.0 ** -126
    for r in range(rows):
        want = 16 * e * 2.0 ** 126 / (16 * e + pos0 + r + 1 - 16)
        got = out[r].double().cpu().numpy()
        assert np.all(np.abs(got - want) < 2.0 ** -6 * want), (got[0], want)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,pos0", [([64, 64], [0, 320]), ([300], [0]), ([384], [0]), ([385], [0]), ([64], [321]),
                                       ([100, 70, 65], [284, 1, 200])])
def test_prefill_on_both_sides_of_few_keys(rows, pos0, hd):
    assert _attn_case(1, rows, pos0, 8, 2, hd, seed=sum(rows) + hd + 1) < 1.5e-2
