"""Verify forwards on both sides of each row count where the few-row path
changes: 16 rows of any model, one workgroup per 16 rows up to 64 where the
projections are small, the separate kernels beyond.  Two layers of the small
bf16 target; sequences of 8 rows and one of the remainder, logits against the
float64 decoder.  The bound is the 2e-2 of the 12-layer comparison (bf16
roundings; 2 layers stay below it)."""

import numpy as np
import pytest

from oracle.decoder import Decoder
from tests.gpu_util import device, rel_err, say, torch
from workloads import SMALL_BF16, model_weights, uniform_prompts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [9, 15, 16, 17, 32, 33, 47, 49, 64, 65])
def test_rows(rows):
    from paper_2607_20507_amd.session import DeviceModel, SpecSession
    dev = device()
    cfg = SMALL_BF16
    tw = model_weights(cfg.target, cfg.seed, 2)
    n_rows = [8] * (rows // 8) + ([rows % 8] if rows % 8 else [])
    ids = [i + 1 for i in range(len(n_rows))]
    lens = [17 + 7 * i for i in range(len(n_rows))]
    rng = np.random.default_rng(rows)
    V = cfg.target.vocab
    say("fused rows", rows, n_rows)
    gpu = SpecSession(DeviceModel(cfg.target, tw, dev, n_layers=2), None, max_seqs=len(ids), k_max=7,
                      max_pages_per_seq=8, max_rows=512)
    ora = Decoder(cfg.target, tw)
    prompts = uniform_prompts(cfg.seed, lens, V)
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

