"""CPU checks of the projection planner (plan_mfma, host C++): its tiles and
splits cover the projection inside the workspace, its choice is not slower
than the other kernels on projections measured with every form, and the GPU
tests reach every gemm_mfma4_bf16 form that it returns for the configured
models."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from workloads import configs as C

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(ROOT, "paper_2607_20507_amd", "csrc")
STORE, ADD, SWIGLU = 0, 1, 2
NONE, NORM, ROPE = 0, 1, 2  # what follows the projection


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    hipcc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if not hipcc:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("gplan") / "gemm_plan_driver")
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(HERE, "native", "gemm_plan_driver.cpp"),
                    os.path.join(CSRC, "gemm_plan.cpp"), "-o", exe], check=True, capture_output=True)

    def run(jobs):
        """(R, N, K, epi, workspace, tail) -> (kernel, tile rows, tile W rows, row tiles, W tiles, splits, k_len)."""
        text = "".join(" ".join(map(str, j)) + "\n" for j in jobs)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(jobs)
        return [None if o == "skinny" else tuple(map(int, o.split())) for o in out]

    return run


def _form(plan, epi):
    """(epilogue, tile rows, tile W rows, splits, several tiles per workgroup)"""
    _, rows, wrows, mt, nt, s, _ = plan
    return epi, rows, wrows, s, mt * nt * s > 256 * (2 if wrows == 128 else 1)


def test_plans_cover_the_projection(plans):
    rng = np.random.default_rng(3)
    jobs = []
    for _ in range(4000):
        R = int(np.exp(rng.uniform(np.log(13), np.log(9000))))
        jobs.append((R, int(rng.integers(1, 900)) * int(rng.choice([1, 16])), 128 * int(rng.integers(1, 120)),
                     int(rng.integers(0, 3)), int(rng.integers(0, 2)), NONE))
    for (R, N, K, epi, ws, _), p in zip(jobs, plans(jobs)):
        if p is None:
            assert R <= 40
            continue
        kernel, rows, wrows, mt, nt, s, k_len = p
        Nw = 2 * N if epi == SWIGLU else N
        assert (mt - 1) * rows < R <= mt * rows and (nt - 1) * wrows < Nw <= nt * wrows
        assert k_len % 128 == 0 and (s - 1) * k_len < K <= s * k_len
        assert s == 1 or (ws and s * R * Nw <= min(8 * R * Nw, 256 ** 3))
        if kernel == 4:
            assert R > 128 and N % 16 == 0 and K % 256 == 0 and (k_len % 256 == 0 or s == 1)


# us of every form near the best: (R, N, K, epilogue): the other kernels, {gemm_mfma4_bf16 (tile, tile, splits): us}.
# Weights rotated through 1.6 GB, MI355X.
MEASURED = {
    (224, 5120, 5120, STORE): (31.7, {(192, 256, 4): 36.1, (128, 256, 4): 36.4, (128, 128, 2): 37.4, (64, 128, 1): 41.6, (64, 128, 4): 40.8}),
    (256, 5120, 5120, STORE): (33.9, {(192, 256, 4): 38.1, (128, 256, 4): 38.5, (128, 128, 2): 40.4, (64, 128, 4): 44.2, (64, 128, 1): 46.2}),
    (192, 3072, 2048, STORE): (15.9, {(64, 128, 2): 16.8, (128, 128, 4): 18.0, (128, 128, 2): 18.7, (64, 128, 4): 19.6, (64, 128, 1): 20.3}),
    (129, 6144, 4096, STORE): (26.5, {(128, 128, 2): 25.7, (128, 256, 4): 25.9, (128, 128, 4): 26.5, (64, 128, 4): 30.4, (64, 128, 8): 31.7}),
    (300, 2048, 2048, ADD): (16.3, {(64, 128, 2): 16.4, (128, 128, 4): 17.4, (128, 128, 2): 18.1, (64, 128, 4): 19.2, (64, 128, 1): 19.3}),
    (640, 2048, 8192, ADD): (40.4, {(192, 256, 8): 39.8, (256, 256, 8): 44.5, (256, 192, 4): 48.0, (128, 256, 4): 48.4, (64, 128, 4): 49.8}),
    (448, 5120, 13824, ADD): (83.2, {(192, 256, 4): 85.9, (256, 192, 4): 93.9, (256, 256, 4): 100.9, (128, 256, 2): 108.0}),
    (512, 5120, 13824, ADD): (86.9, {(192, 256, 4): 98.7, (256, 192, 4): 98.9, (256, 256, 4): 106.2, (128, 256, 2): 130.1}),
    (640, 5120, 13824, ADD): (103.2, {(256, 256, 4): 108.8, (256, 192, 2): 127.8, (192, 256, 2): 129.3, (128, 256, 2): 135.5, (256, 256, 2): 144.6}),
    (400, 4096, 14336, ADD): (71.4, {(128, 256, 4): 62.2, (256, 256, 8): 67.1, (128, 128, 2): 67.7, (128, 128, 4): 71.0}),
    (4096, 6144, 4096, STORE): (257.7, {(256, 192, 1): 181.8, (256, 256, 1): 194.1, (128, 256, 1): 207.2, (192, 256, 1): 212.9}),
    (4096, 4096, 4096, ADD): (175.9, {(256, 256, 1): 115.3, (128, 256, 1): 148.1, (192, 256, 1): 164.1, (256, 192, 1): 180.3}),
    (4096, 14336, 4096, SWIGLU): (872.3, {(256, 256, 1): 681.5, (192, 256, 1): 798.0, (128, 256, 1): 902.5}),
}


def test_choice_against_every_form_measured(plans):
    """The estimates leave a few percent; a projection that gemm_mfma4_bf16
    slows down stays with the other kernels, one that it speeds up moves."""
    for (case, (other, m4)), p in zip(MEASURED.items(), plans([c + (1, NONE) for c in MEASURED])):
        t = m4[p[1], p[2], p[5]] if p[0] == 4 else other
        assert t < 1.05 * other, (case, p)
        assert t < 1.08 * min([other] + list(m4.values())), (case, p)


def test_gpu_cases_reach_every_form(plans):
    from tests import test_gpu_gemm_tiles as G
    got = {}
    cases = [(R, N, K, epi, 1, NONE) for epi, R, N, K in G.FORMS]
    for c, p in zip(cases, plans(cases)):
        assert p[0] == 4, (c, p)
        got.setdefault(_form(p, c[3]), c)
    rows = list(range(129, 520)) + list(range(520, 8193, 23)) + [8192]
    jobs = []
    for sh in (C.SMALL_TARGET, C.SMALL_DRAFT, C.L8B_TARGET, C.L1B_DRAFT):
        d = sh.d_model
        for R in rows:
            for tail in (NONE, ROPE):
                jobs.append((R, sh.qkv_rows, d, STORE, 1, tail))
            for tail in (NONE, NORM):
                jobs += [(R, d, sh.q_dim, ADD, 1, tail), (R, d, sh.ffn_dim, ADD, 1, tail)]
            jobs.append((R, sh.ffn_dim, d, SWIGLU, 1, NONE))
            if R <= 512:
                jobs.append((R, sh.vocab, d, STORE, 1, NONE))
    want = {}
    for j, p in zip(jobs, plans(jobs)):
        if p[0] == 4:
            want.setdefault(_form(p, j[3]), j)
    assert not {f: j for f, j in want.items() if f not in got}
