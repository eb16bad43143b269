"""Call tables on their way to the device: kernel arguments up to 3072 bytes, a
pinned buffer above.  Draws of n rows (32 bytes of table each; up to 64 rows
in the arguments of the draw itself) around these limits, issued back to back so that the pinned slots are reused, against the
same rows drawn one by one."""

import numpy as np
import pytest

from tests.gpu_util import device, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 64, 65, 95, 96, 97, 700])
def test_draws_of_n_rows(n):
    from paper_2607_20507_amd import binding as B
    dev, V, reps = device(), 512, 12
    logits = torch.randn(n, V, device=dev)
    ws = torch.empty(B.spec_sample_workspace_bytes(n, 2 * n, V) + (1 << 20), dtype=torch.uint8, device=dev)
    ids = np.arange(n, dtype=np.int64) * 3 + 1
    temps = np.where(np.arange(n) % 4 == 0, 0.0, 0.9).astype(np.float32)
    outs = []
    for r in range(reps):
        out = torch.full((n,), -1, dtype=torch.int32, device=dev)
        B.spec_sample_draft(logits, V, temps, ids, np.arange(n, dtype=np.int32) + 10 * r, 5, out, ws)
        outs.append(out)
    one = torch.full((n,), -1, dtype=torch.int32, device=dev)
    for r in (0, reps - 1):
        for i in range(n):
            B.spec_sample_draft(logits[i], V, temps[i:i + 1], ids[i:i + 1], np.array([i + 10 * r], np.int32), 5,
                                one[i:i + 1], ws)
        assert torch.equal(outs[r], one)
