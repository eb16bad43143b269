"""Verify forwards on both sides of each row count where the few-row path
changes: 16 rows (12 of a model wider than 4096), one workgroup per 16 rows up
to 64 where the projections are small, the separate kernels beyond.  Two layers
of the small bf16 target and of two with grouped heads, one layer of three whose
projections set another limit; sequences of 8 rows and one of the remainder, logits against the float64 decoder.  The bound is the
2e-2 of the 12-layer comparison (bf16 roundings; 2 layers stay below it)."""

import numpy as np
import pytest

from oracle.decoder import Decoder
from tests.gpu_util import device, rel_err, say, torch
from workloads import SMALL_BF16, model_weights, uniform_prompts
from workloads.configs import ModelShape

pytestmark = pytest.mark.gpu

SEED = SMALL_BF16.seed
# 6 q / 3 kv heads of 64; 4 / 2 of 128 and a vocabulary of no whole tiles; 23M gate and up weights
GROUPED_64 = ModelShape("grouped-64", 2, 384, 6, 3, 64, 640, 1040, 1e4)
GROUPED = ModelShape("grouped", 2, 512, 4, 2, 128, 1408, 1000, 1e4)
WIDE = ModelShape("wide", 1, 2048, 16, 4, 128, 5632, 2048, 5e5)
WIDER = ModelShape("wider", 1, 4224, 2, 1, 128, 2048, 1024, 5e5)  # past 4096 columns: 12 rows
MID = ModelShape("mid", 1, 1536, 12, 12, 64, 4096, 2048, 1e4)     # 12M weights: 42 rows


@pytest.mark.parametrize("rows", [9, 15, 16, 17, 32, 33, 47, 49, 64, 65])
def test_rows(rows):
    _check(SMALL_BF16.target, 2, rows)


@pytest.mark.parametrize("shape,rows", [(GROUPED_64, 9), (GROUPED_64, 17), (GROUPED_64, 33), (GROUPED_64, 64), (GROUPED, 16),
                                        (GROUPED, 17), (GROUPED, 48), (GROUPED, 64), (WIDE, 8), (WIDE, 9), (WIDE, 16), (WIDE, 17),
                                        (WIDER, 12), (WIDER, 13), (MID, 42), (MID, 43)],
                         ids=lambda x: getattr(x, "name", x))
def test_rows_of_other_models(shape, rows):
    _check(shape, shape.n_layers, rows)


def _check(shape, layers, rows):
    from paper_2607_20507_amd.session import DeviceModel, SpecSession
    dev = device()
    tw = model_weights(shape, SEED, layers)
    n_rows = [8] * (rows // 8) + ([rows % 8] if rows % 8 else [])
    ids = [i + 1 for i in range(len(n_rows))]
    lens = [17 + 7 * i for i in range(len(n_rows))]
    rng = np.random.default_rng(rows)
    V = shape.vocab
    say("fused rows", shape.name, rows, n_rows)
    gpu = SpecSession(DeviceModel(shape, tw, dev, n_layers=layers), None, max_seqs=len(ids), k_max=7,
                      max_pages_per_seq=8, max_rows=512)
    ora = Decoder(shape, tw)
    prompts = uniform_prompts(SEED, lens, V)
    gpu.prefill(ids, prompts)
    q = torch.zeros(7, V, device=dev)
    want = []
    for sid, n, p in zip(ids, n_rows, prompts):
        drafts = rng.integers(0, V, n - 1).astype(np.int32)
        if n > 1:
            gpu.set_drafts(sid, drafts, q)
        toks = np.concatenate([p, drafts])
        want.append(ora.full_logits(toks)[-n:])
    gpu.target_forward(ids)
    got = gpu.last_logits().cpu().numpy()
    want = np.concatenate(want)
    assert got.shape == want.shape
    worst = max(rel_err(got[r], want[r]) for r in range(rows))
    assert worst < 2e-2, worst
    gpu.close()

