"""The fp32 kernels at the ends of their tiles and steps, against float64: the
matrix-core projection (16 x 16 and 32 x 32 tiles, K down to one float4 and
not a multiple of the 16-column chunk, operands at any float address) and the
attention (contexts around its 256-key step, keys of other sequences and
stale values behind the mask).

Tolerance: fp32 sums of n terms in any order stay within n 2^-24 of the sum of
magnitudes, sqrt(n) 2^-24 of the norm in practice: 8 sqrt(n) 2^-24."""

import numpy as np
import pytest
import torch

from paper_2607_20507_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("epi", [B.SPEC_EPI_STORE_F32, B.SPEC_EPI_ADD_F32, B.SPEC_EPI_SWIGLU])
@pytest.mark.parametrize("R,N,K", [(1, 1, 4), (5, 17, 12), (16, 16, 16), (17, 15, 60), (33, 768, 256), (127, 688, 688),
                                   (500, 1376, 256), (700, 1030, 100), (3, 40, 30)])
def test_projection(R, N, K, epi, shift):
    Nw = 2 * N if epi == B.SPEC_EPI_SWIGLU else N
    x = torch.randn(R * K + shift, generator=_gen(R + N), device=DEV)[shift:]
    w = torch.randn(Nw * K + shift, generator=_gen(K), device=DEV)[shift:] * 0.1
    w = torch.cat([torch.zeros(shift, device=DEV), w])[shift:]
    y = torch.randn(R * N + 64, generator=_gen(4), device=DEV)
    want = x.double().view(R, K) @ w.double().view(Nw, K).t().contiguous()
    if epi == B.SPEC_EPI_SWIGLU:
        want = torch.nn.functional.silu(want[:, :N]) * want[:, N:]
    elif epi == B.SPEC_EPI_ADD_F32:
        want = want + y[:R * N].view(R, N).double()
    tail = y[R * N:].clone()
    B.spec_op_gemm(B.SPEC_F32, R, N, K, x, w, y, epi)
    torch.cuda.synchronize()
    assert torch.equal(y[R * N:], tail)
    # (SwiGLU: two sums and an fp32 exponential of a few units in the last place)
    tol = (8 * K ** 0.5 + (32 if epi == B.SPEC_EPI_SWIGLU else 0)) * 2 ** -24
    assert float((y[:R * N].view(R, N).double() - want).norm() / want.norm()) < tol


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,pos0", [([1], [0]), ([2, 1], [254, 255]), ([5, 3], [256, 15]), ([1, 8], [511, 900])])
def test_attention(rows, pos0, hd):
    hq, hkv = 4, 2
    need = [(p + r + 15) // 16 for p, r in zip(pos0, rows)]
    pt = np.zeros((len(rows), max(need)), dtype=np.int32)
    perm = np.random.default_rng(3).permutation(sum(need)).astype(np.int32)
    o = 0
    for i, n in enumerate(need):
        pt[i, :n] = perm[o:o + n]
        o += n
    kp = torch.randn(sum(need), hkv, 16, hd, generator=_gen(1), device=DEV)
    vp = torch.randn(sum(need), hkv, hd, 16, generator=_gen(2), device=DEV)
    q = torch.randn(sum(rows), hq, hd, generator=_gen(5), device=DEV)
    out = torch.zeros(sum(rows), hq * hd, device=DEV)
    for i, (r, p) in enumerate(zip(rows, pos0)):  # slots past a sequence's end hold anything
        end = p + r
        if end % 16:
            vp[int(pt[i, end // 16]), :, :, end % 16:] = float("nan")
    ws = torch.empty(B.spec_op_attention_workspace_bytes(len(rows), sum(rows), pt.shape[1], hkv, hd) + 8192,
                     dtype=torch.uint8, device=DEV)
    B.spec_op_attention(B.SPEC_F32, rows, pos0, pt, hq, hkv, hd, q, kp, vp, out, ws)
    torch.cuda.synchronize()
    r0 = 0
    for i, (r, p) in enumerate(zip(rows, pos0)):
        pages = torch.from_numpy(pt[i, :need[i]].astype(np.int64)).to(DEV)
        k = kp[pages].double().transpose(1, 2).reshape(-1, hkv, hd)
        v = vp[pages].double().permute(0, 3, 1, 2).reshape(-1, hkv, hd)
        for j in range(r):
            for h in range(hq):
                n = p + j + 1
                z = k[:n, h // 2] @ q[r0 + j, h].double() / hd ** 0.5
                want = torch.softmax(z, 0) @ v[:n, h // 2]
                got = out[r0 + j, h * hd:(h + 1) * hd].double()
                assert float((got - want).norm() / want.norm()) < 8 * n ** 0.5 * 2 ** -24 + 1e-6
        r0 += r
