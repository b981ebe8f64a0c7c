"""Key-split plan and fused epilogue at the places where their rules switch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import (eb_block_attn, eb_decode_step, eb_lmhead_confidence,
                                  eb_unmask_select)
from paper_2609_16450_amd.device_case import DeviceStep
from workloads import bf16_bits_to_f32, custom_config, make_step

pytestmark = pytest.mark.gpu


# One K/V head, one row tile: the ranges go by the keys alone, from one key to 64 stages of 64
# keys.  Two heads and rows of several tiles: fewer ranges of more stages.
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("hq,hkv,blocks,prefix", [
    (1, 1, 70, 0), (1, 1, 70, 441), (1, 1, 70, 443), (1, 1, 65, 4031), (2, 2, 66, 2047),
    (56, 8, 90, 1000), (128, 64, 65, 63)])
def test_split_plan(hq, hkv, blocks, prefix, head_dim):
    print(f"split hq={hq} hkv={hkv} rows={blocks} prefix={prefix} D={head_dim}", flush=True)
    cfg = custom_config(seed=prefix + 1, batch=2, hq=hq, hkv=hkv, head_dim=head_dim, hidden=64,
                        vocab=64, block_len=("fixed", blocks), prefix_len=("uniform", prefix // 3, prefix))
    case = make_step(cfg)
    ref = oracle.block_attention(*(bf16_bits_to_f32(x) for x in (
        case.q, case.k_blk, case.v_blk, case.k_pre, case.v_pre)), case.cu_block, case.cu_prefix,
        hq, hkv)
    ds = DeviceStep(case)
    eb_block_attn(ds.ragged, ds.q, ds.k_blk, ds.v_blk, ds.k_pre, ds.v_pre, ds.attn_out)
    # as in the other attention tests: probabilities and outputs rounded to bf16
    np.testing.assert_allclose(ds.attn_out.float().cpu().numpy(), ref, rtol=2e-2, atol=2e-2)


# 118 vocabulary slices of 256 rows: a block of 69 rows has 8142 partials (fused epilogue), one of
# 70 rows 8260 (three kernels).  64 rows in one block: the attention shares the LM-head launch and
# the epilogue is fused with 64 x 256 partials.
@pytest.mark.parametrize("rows,vocab", [(69, 30000), (70, 30000), (64, 9000)])
def test_epilogue_rule(rows, vocab):
    print(f"epilogue rows={rows} vocab={vocab}", flush=True)
    cfg = custom_config(seed=rows, batch=1, hq=4, hkv=4, head_dim=128, hidden=128, vocab=vocab,
                        block_len=("fixed", rows), prefix_len=("fixed", 300))
    case = make_step(cfg)
    a, b = DeviceStep(case), DeviceStep(case)
    eb_decode_step(a.buffers)
    eb_block_attn(b.ragged, b.q, b.k_blk, b.v_blk, b.k_pre, b.v_pre, b.attn_out)
    eb_lmhead_confidence(b.h, b.w, b.conf, b.entropy, b.argmax, b.max_logit)
    eb_unmask_select(b.ragged, b.conf, b.argmax, b.tau, b.masked, b.tokens, b.unmask, b.n_commit,
                     b.resolved)
    for k in ("attn_out", "conf", "entropy", "argmax", "max_logit", "masked", "tokens", "unmask",
              "n_commit", "resolved"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
