"""Budgeted commit at the edges of its workgroup sizes (blocks of up to 16, 64 and 128 rows), rounds
(256 rows), LDS tiles (2048 rows) and remembered rounds (32), with ties in conf, against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import Ragged, eb_unmask_select_topm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [0, 1, 7, 300, 100000])
@pytest.mark.parametrize("blocks", [
    [1, 0, 16, 3], [0, 0], [17, 64, 1, 0], [65, 128, 4], [129, 127],
    [1, 0, 3, 64, 65, 255, 256, 257], [1023, 1024, 1025, 2047, 2048], [2049, 4100, 5], [8192, 9001]])
def test_topm_edges(blocks, m):
    print(f"topm blocks={blocks} m={m}", flush=True)
    rng = np.random.default_rng([m, *blocks])
    T, B = sum(blocks), len(blocks)
    conf = (rng.integers(1, 200, T) / 256).astype(np.float32)        # many exact ties
    argmax = rng.integers(0, 1000, T).astype(np.int32)
    masked = (rng.random(T) < 0.6).astype(np.uint8)
    tokens = np.where(masked, -1, 7).astype(np.int32)
    tau = np.where(rng.random(B) < 0.5, 0.7, 1.5).astype(np.float32)  # 1.5: no threshold
    cu = np.concatenate([[0], np.cumsum(blocks)]).astype(np.int32)
    ref = oracle.unmask_select_topm(conf, argmax, masked, tokens, tau, cu, m)
    d = {k: torch.from_numpy(v).cuda() for k, v in dict(
        conf=conf, argmax=argmax, tau=tau, masked=masked, tokens=tokens).items()}
    unmask = torch.full((T,), 9, dtype=torch.uint8, device="cuda")
    n_commit = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    resolved = torch.full((B,), 9, dtype=torch.uint8, device="cuda")
    eb_unmask_select_topm(Ragged.from_lengths(blocks, [0] * B), d["conf"], d["argmax"], d["tau"], m,
                          d["masked"], d["tokens"], unmask, n_commit, resolved)
    for got, want in ((unmask, "unmask"), (d["tokens"], "tokens"), (d["masked"], "masked"),
                      (n_commit, "n_commit"), (resolved, "resolved")):
        np.testing.assert_array_equal(got.cpu().numpy(), ref[want], err_msg=want)
