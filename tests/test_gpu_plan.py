"""Key-split plan and fused epilogue at the places where their rules switch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import (Ragged, StepBuffers, eb_block_attn, eb_decode_step,
                                  eb_lmhead_confidence, eb_unmask_select)
from paper_2609_16450_amd.binding import eb_step_trace
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


# fp32 steps, bit for bit against the separate entry points.  The attention is in the epilogue
# launch with up to 256 workgroups (tiles of 16 query rows, K/V heads, sequences), when that is one
# launch: 70001 entries are 274 slices, so a block of 29 rows has 7946 partials (one launch) and one
# of 30 rows 8220 (three kernels).  Empty blocks, both head dimensions in the epilogue, and a step
# of four (row, key) pairs, whose attention is a launch of its own.
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lens,hq,hkv,vocab", [
    ((20, 0, 7, 33), 4, 2, 2048), ((0, 1, 5, 0), 3, 1, 300),
    ((16,) * 8, 32, 32, 999), ((16,) * 8 + (1,), 32, 32, 999),  # 256 workgroups, 288
    ((29, 3), 2, 2, 70001), ((30, 3), 2, 2, 70001), ((2,), 2, 2, 300)])
def test_fp32_step(lens, hq, hkv, vocab, head_dim):
    print(f"fp32 step blocks={lens} hq={hq} hkv={hkv} V={vocab} D={head_dim}", flush=True)
    T, B, hidden = sum(lens), len(lens), 100
    prefix = [37 * b % 150 for b in range(B)]
    g = torch.Generator(device="cuda").manual_seed(T + vocab)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    q, h, w = normal(T, hq, head_dim), normal(T, hidden), normal(vocab, hidden)
    kv = [normal(n, hkv, head_dim) for n in (T, T, sum(prefix), sum(prefix))]
    masked0 = (torch.rand(T, generator=g, device="cuda") < 0.7).to(torch.uint8)
    tau = torch.full((B,), 0.5, device="cuda")
    r = Ragged.from_lengths(list(lens), prefix)
    got = []
    for step in (True, False):
        f32 = [torch.full((T,), -1.0, device="cuda") for _ in range(3)]
        i32 = [torch.full((n,), -1, dtype=torch.int32, device="cuda") for n in (T, T, B)]
        u8 = [torch.full((n,), 9, dtype=torch.uint8, device="cuda") for n in (T, B)]
        (conf, ent, top), (arg, tokens, n_commit), (unmask, resolved) = f32, i32, u8
        out, masked = torch.full_like(q, 7.0), masked0.clone()
        if step:
            eb_decode_step(StepBuffers(r, q, *kv, out, h, w, conf, ent, arg, tau, masked, tokens,
                                       unmask, n_commit, resolved, max_logit=top))
        else:
            eb_block_attn(r, q, *kv, out)
            eb_lmhead_confidence(h, w, conf, ent, arg, top)
            eb_unmask_select(r, conf, arg, tau, masked, tokens, unmask, n_commit, resolved)
        got.append([out, masked, *f32, *i32, *u8])
    for i, (a, b) in enumerate(zip(*got)):
        assert torch.equal(a, b), i
    ref = oracle.block_attention(q.cpu().numpy(), *(x.cpu().numpy() for x in kv),
                                 r.cu_block.cpu().numpy(), r.cu_prefix.cpu().numpy(), hq, hkv)
    # scores of size |q||k| / sqrt(d) < 16 off by some 128 2^-24 16 / sqrt(128): 1e-5 in a weight
    np.testing.assert_allclose(got[0][0].cpu().numpy(), ref, rtol=2e-5, atol=2e-5)


def test_traced_fp32_step_times_its_attention():
    """The attn_* events of a traced fp32 step bracket the attention, and the step's outputs are those
    of an untraced one.  4096 keys: some 200 us of attention for an idle bracket of under 20 us."""
    case = make_step(custom_config(seed=5, hidden=64, vocab=300, head_dim=128, dtype="f32",
                                   block_len=("fixed", 32), prefix_len=("fixed", 4064)))
    a, b = DeviceStep(case), DeviceStep(case)
    eb_decode_step(a.buffers)
    begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    for e in (begin, end):
        e.record()  # creates the event
    eb_decode_step(b.buffers, trace=eb_step_trace(begin.cuda_event, end.cuda_event, 0, 0, 0, 0))
    torch.cuda.synchronize()
    assert begin.elapsed_time(end) > 0.05
    for k in ("attn_out", "conf", "entropy", "argmax", "max_logit", "masked", "tokens", "unmask"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
