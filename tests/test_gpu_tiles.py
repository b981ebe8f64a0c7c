"""LM-head tile kernel (more than 64 positions) at the edges of its tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import eb_lmhead_features
from workloads import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

# A head this wide has 128 vocabulary tiles of 256 rows, the last one partial.  Hidden sizes give
# one, two, three and five stages of 64 columns per tile; row counts lie at the edges of the
# position tiles and at their remainders.
VOCAB = 32700


@pytest.mark.parametrize("hidden", [64, 128, 192, 320])
@pytest.mark.parametrize("rows", [65, 96, 97, 160, 193, 256, 257, 321, 384, 385, 449, 512, 513])
def test_tile_edges(rows, hidden):
    print(f"tile rows={rows} hidden={hidden}", flush=True)
    rng = np.random.default_rng([rows, hidden])
    w = f32_to_bf16_bits(rng.standard_normal((VOCAB, hidden), dtype=np.float32) / np.sqrt(hidden))
    h = rng.standard_normal((rows, hidden), dtype=np.float32)
    # every row points at a token of its own, the first and last vocabulary rows among them, by a
    # margin that the argmax cannot lose
    t = rng.integers(0, VOCAB, rows)
    t[:2] = 0, VOCAB - 1
    u = bf16_bits_to_f32(w[t])
    h += 12.0 * u / np.linalg.norm(u, axis=1, keepdims=True)
    h = f32_to_bf16_bits(h)
    ref = oracle.lmhead_confidence(bf16_bits_to_f32(h), bf16_bits_to_f32(w))

    dev = [torch.from_numpy(x).cuda().view(torch.bfloat16) for x in (h, w)]
    conf, ent, gap, top = (torch.empty(rows, device="cuda") for _ in range(4))
    arg = torch.empty(rows, dtype=torch.int32, device="cuda")
    eb_lmhead_features(*dev, conf, ent, arg, gap, max_logit=top)
    # An fp32 sum of d products of size |w||h| <= 20 is off by at most d 2^-24 20 < 4e-4 (d = 320),
    # which is also the relative error of a probability; 1e-3 as in the other parity tests.
    np.testing.assert_array_equal(arg.cpu().numpy(), ref["argmax"])
    for got, want in ((conf, "conf"), (ent, "entropy"), (top, "max_logit"), (gap, "top2_gap")):
        np.testing.assert_allclose(got.cpu().numpy(), ref[want], rtol=0, atol=1e-3, err_msg=want)
