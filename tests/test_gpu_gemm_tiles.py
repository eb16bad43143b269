"""The projections of more than 128 rows against float64, with and without the
split-K workspace: sizes where tiles, splits and loops end (one row past a
tile, one 16-feature W tile, the shortest k-loop) whatever kernel takes them,
and one for every form of the resident-workgroup MFMA GEMM (epilogue, tile, K
split, one or several tiles per workgroup) that the planner returns for the
configured models (a CPU test holds the list to that).

Tolerance: a sum of K bf16 products in fp32, in any order, is within K 2^-24
sum |x w| of the exact one; for normal inputs that is sqrt(K) 2^-24 of the
result's norm in practice, so 8 sqrt(K) 2^-24 bounds the 2-norm.  SwiGLU
results are rounded to bf16 (2^-9) after an fp32 SiLU."""

import numpy as np
import pytest
import torch

from paper_2607_20507_amd import binding as B
from paper_2607_20507_amd.session import DeviceModel, SpecSession
from workloads.configs import ModelShape

pytestmark = pytest.mark.gpu
DEV = "cuda"

STORE, ADD, SWIGLU = B.SPEC_EPI_STORE_F32, B.SPEC_EPI_ADD_F32, B.SPEC_EPI_SWIGLU
CASES = [
    # rows, outputs, K: the smallest of everything; one tile and one row more; several rounds of workgroups
    (129, 16, 256), (129, 1040, 512), (192, 2048, 2048), (193, 272, 1024), (256, 4096, 4096), (257, 1024, 2816),
    (385, 4112, 768), (500, 6144, 1024), (640, 2816, 1024), (1000, 3072, 2048), (1025, 2048, 8192), (2049, 6160, 512),
    (4111, 1024, 1024), (5000, 4096, 256),
]


# epilogue, rows, outputs, K: partial tiles on both sides, several tiles of three unrolled k-loops
FORMS = [
    (STORE, 129, 272, 256), (STORE, 193, 16448, 256), (STORE, 1706, 272, 1536), (STORE, 259, 6640, 256),
    (STORE, 271, 4160, 2816), (STORE, 259, 13072, 512), (STORE, 774, 17360, 768), (STORE, 262, 8272, 8192),
    (STORE, 526, 14528, 256), (STORE, 906, 16464, 768), (STORE, 649, 14896, 256), (STORE, 990, 16784, 768),
    (STORE, 196, 16848, 4096), (STORE, 644, 16736, 512), (STORE, 1420, 16784, 768), (STORE, 580, 8256, 6144),
    (ADD, 130, 272, 256), (ADD, 1684, 272, 1536), (ADD, 197, 464, 1024), (ADD, 323, 6096, 256),
    (ADD, 259, 3472, 2048), (ADD, 200, 2064, 2048), (ADD, 257, 912, 4096), (ADD, 257, 13120, 512),
    (ADD, 196, 5408, 6144), (ADD, 260, 1568, 10240), (ADD, 516, 14624, 256), (ADD, 907, 16448, 768),
    (ADD, 258, 12368, 4096), (ADD, 258, 6432, 4096), (ADD, 584, 1952, 8192), (ADD, 6360, 1328, 256),
    (ADD, 1924, 8208, 768), (ADD, 6646, 528, 2816), (ADD, 641, 16672, 512), (ADD, 1423, 16400, 768),
    (ADD, 596, 8352, 5120), (ADD, 193, 12480, 8192), (SWIGLU, 130, 272, 256), (SWIGLU, 130, 10960, 256),
    (SWIGLU, 264, 3296, 256), (SWIGLU, 258, 6560, 512), (SWIGLU, 263, 16432, 768), (SWIGLU, 517, 7392, 256),
    (SWIGLU, 390, 16736, 768), (SWIGLU, 395, 12992, 512), (SWIGLU, 666, 16560, 768),
]


def _inputs(R, N, K, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn(R, K, generator=g, device=DEV).bfloat16()
    w = (torch.randn(N, K, generator=g, device=DEV) * 0.05).bfloat16()
    return x, w


@pytest.mark.parametrize("workspace", [True, False])
@pytest.mark.parametrize("epi", [STORE, ADD, SWIGLU])
@pytest.mark.parametrize("R,N,K", CASES)
def test_projection(R, N, K, epi, workspace):
    Nw = 2 * N if epi == SWIGLU else N
    x, w = _inputs(R, Nw, K, R + N + K + epi)
    want = x.double() @ w.double().t().contiguous()
    packed = w.clone()
    if epi == SWIGLU:
        B.spec_pack_weight(packed[:N], N, K)
        B.spec_pack_weight(packed[N:], N, K)
        want = torch.nn.functional.silu(want[:, :N]) * want[:, N:]
    else:
        B.spec_pack_weight(packed, N, K)
    guard = 4096  # past the output: untouched
    y = torch.zeros(R * N + guard, device=DEV, dtype=torch.bfloat16 if epi == SWIGLU else torch.float32)
    y[R * N:] = 7.0
    if epi == ADD:
        y[:R * N] = torch.randn(R * N, device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
        want = want + y[:R * N].view(R, N).double()
    ws = torch.empty(B.spec_op_gemm_workspace_bytes(R, Nw), dtype=torch.uint8, device=DEV) if workspace else None
    B.spec_op_gemm(B.SPEC_BF16, R, N, K, x, packed, y, epi, ws)
    torch.cuda.synchronize()
    got = y[:R * N].view(R, N).double()
    assert torch.all(y[R * N:] == 7.0)
    tol = 8 * K ** 0.5 * 2 ** -24 + (2 ** -9 if epi == SWIGLU else 0.0)
    assert float((got - want).norm() / want.norm()) < tol
    # no single element is off by more than its own rounding and the sum's worst case over a row's scale
    scale = want.pow(2).mean().sqrt()
    lim = (2 ** -8 * want.abs() if epi == SWIGLU else 0.0) + 64 * K ** 0.5 * 2 ** -24 * scale
    assert torch.all((got - want).abs() <= lim)


@pytest.mark.parametrize("epi,R,N,K", FORMS)
def test_form(epi, R, N, K):
    test_projection(R, N, K, epi, True)


def test_unaligned_output_takes_the_general_path():
    """An output that is not 16-byte aligned is as right as an aligned one."""
    R, N, K = 300, 1024, 1024
    x, w = _inputs(R, N, K, 5)
    want = x.double() @ w.double().t().contiguous()
    B.spec_pack_weight(w, N, K)
    y = torch.zeros(R * N + 1, device=DEV)
    B.spec_op_gemm(B.SPEC_BF16, R, N, K, x, w, y[1:], STORE)
    torch.cuda.synchronize()
    assert float((y[1:].view(R, N).double() - want).norm() / want.norm()) < 8 * K ** 0.5 * 2 ** -24


def test_draft_rows_of_a_large_batch():
    """More than 128 sequences drafting at once: the LM head writes each row
    to its sequence's place (an output row map), as it does one by one."""
    sh = ModelShape("tiles", 1, 256, 4, 4, 64, 512, 1040, 1e4)
    n = 136
    target, draft = DeviceModel(sh, seed=1), DeviceModel(sh, seed=2)
    rng = np.random.default_rng(9)
    prompts = [rng.integers(0, sh.vocab, int(k), dtype=np.int32) for k in rng.integers(2, 40, n)]
    ids = list(range(1, n + 1))

    def session():
        s = SpecSession(target, draft, max_seqs=n, k_max=2, max_pages_per_seq=4, max_rows=4096)
        s.prefill(ids, prompts)
        return s

    a, b = session(), session()
    a.draft_step(ids, [0.8] * n, 3)
    for i in ids[::17]:
        b.draft_step([i], [0.8], 3)
        za, zb = a.draft_logits(i, 0).double(), b.draft_logits(i, 0).double()
        # one bf16 layer either way: roundings of 2^-9 at each of its half dozen steps
        assert float((za - zb).norm() / zb.norm()) < 2e-2
    a.close()
    b.close()
