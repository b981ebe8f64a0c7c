"""fp32 kernels at the edges of their tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import (Ragged, eb_block_attn, eb_block_attn_dual, eb_lmhead_confidence,
                                  eb_lmhead_features)

pytestmark = pytest.mark.gpu


def _cu(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


# Query rows per K/V head at, below and above 16; keys below one 16-key chunk, one chunk per wave
# (128), a few more, and empty segments and blocks.
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("group", [1, 3])
@pytest.mark.parametrize("blocks,prefix,suffix", [
    ([1], [0], [0]), ([16], [112], [0]), ([5, 0, 6], [3, 7, 300], [0, 1, 33]),
    ([17, 33], [0, 95], [1, 0])])
def test_attention_f32(blocks, prefix, suffix, group, head_dim):
    print(f"attn f32 {blocks} {prefix} {suffix} G={group} D={head_dim}", flush=True)
    rng = np.random.default_rng([head_dim, group, *blocks])
    hkv, T, S, U = 2, sum(blocks), sum(prefix), sum(suffix)
    def x(*s): return rng.standard_normal(s, dtype=np.float32)
    q = x(T, hkv * group, head_dim)
    kv = [x(n, hkv, head_dim) for n in (T, T, S, S, U, U)]
    ref = oracle.block_attention(q, *kv[:4], _cu(blocks), _cu(prefix), hkv * group, hkv,
                                 k_suf=kv[4], v_suf=kv[5], cu_suffix=_cu(suffix))
    out = torch.full(q.shape, 7.0, device="cuda")
    eb_block_attn_dual(Ragged.from_lengths(blocks, prefix), torch.from_numpy(_cu(suffix)).cuda(),
                       max(suffix), torch.from_numpy(q).cuda(),
                       *(torch.from_numpy(a).cuda() for a in kv), out)
    # scores of size |q||k| / sqrt(d) < 16 off by some 128 2^-24 16 / sqrt(128): 1e-5 in a weight
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=2e-5, atol=2e-5)


def _attention(blocks, prefix, x, group):
    """Output of eb_block_attn and the oracle's; x: q, k_blk, v_blk, k_pre, v_pre."""
    out = torch.full(x[0].shape, 7.0, device="cuda")
    eb_block_attn(Ragged.from_lengths(blocks, prefix), *(torch.from_numpy(a).cuda() for a in x), out)
    hkv = x[1].shape[1]
    with np.errstate(all="ignore"):
        return out.cpu().numpy(), oracle.block_attention(*x, _cu(blocks), _cu(prefix), hkv * group,
                                                         hkv)


# Both sides of the launch rules: 8 and 9 (row, key) pairs; 64 and 65 keys; 1022 and 1024 tiles of
# query rows with 128 and 129 keys.  Every fourth sequence is shorter than the largest.
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,rows,keys,group", [
    (3, 1, 8, 1), (3, 1, 9, 1), (2, 2, 4, 1), (5, 1, 2, 4), (5, 1, 2, 5),
    (4, 3, 64, 2), (4, 3, 65, 2), (511, 1, 20, 1), (512, 1, 20, 1), (512, 2, 128, 3),
    (512, 2, 129, 3)])
def test_attention_f32_launches(batch, rows, keys, group, head_dim):
    print(f"attn f32 batch={batch} rows={rows} keys={keys} G={group} D={head_dim}", flush=True)
    blocks = [rows] * batch
    prefix = [(keys - rows) // (4 if b % 4 == 3 else 1) for b in range(batch)]
    rng = np.random.default_rng([batch, rows, keys, head_dim])
    T, S = sum(blocks), sum(prefix)
    x = [rng.standard_normal((n, hh, head_dim), dtype=np.float32)
         for n, hh in ((T, 2 * group), (T, 2), (T, 2), (S, 2), (S, 2))]
    got, ref = _attention(blocks, prefix, x, group)
    # scores of size |q||k| / sqrt(d) < 16 off by some 128 2^-24 16 / sqrt(128): 1e-5 in a weight
    np.testing.assert_allclose(got, ref, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_attention_f32_infinities(head_dim):
    """Scores of -inf have a weight of zero, and an infinite value of the last key, which the tile's
    keys past the end repeat, reaches the output."""
    rng = np.random.default_rng(head_dim)
    x = [rng.standard_normal((n, 1, head_dim), dtype=np.float32) for n in (5, 5, 5, 48, 48)]
    q, k_blk, v_blk, k_pre, v_pre = x
    q[:, 0, 0], k_blk[:, 0, 0], k_pre[:, 0, 0] = 3e20, 0, 0
    k_pre[16:32, 0, 0] = -3e20          # a whole chunk of keys
    v_blk[4, 0, 7] = np.inf
    got, ref = _attention([5], [48], x, 1)
    assert np.isinf(got[:, 0, 7]).all()
    got[:, 0, 7] = ref[:, 0, 7] = 0
    np.testing.assert_allclose(got, ref, rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("rows,vocab", [(3, 300), (300, 70001)])  # slices of 64 and of 256 rows
def test_lmhead_f32_infinities(rows, vocab):
    """Logits of -inf, of the lowest finite value and NaN take no part in the statistics."""
    rng = np.random.default_rng([rows, vocab])
    h, w = (rng.standard_normal((n, 65), dtype=np.float32) for n in (rows, vocab))
    h[:, 3] = 1
    bad = rng.permutation(vocab)[:120]
    w[bad] = 0
    w[bad[:40], 3], w[bad[40:80], 3] = -np.inf, np.finfo(np.float32).min
    w[bad[80:], 3] = np.nan
    good = np.setdiff1d(np.arange(vocab), bad)
    z = h.astype(np.float64) @ w[good].astype(np.float64).T
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    conf, ent, top = (torch.empty(rows, device="cuda") for _ in range(3))
    arg = torch.empty(rows, dtype=torch.int32, device="cuda")
    eb_lmhead_confidence(torch.from_numpy(h).cuda(), torch.from_numpy(w).cuda(), conf, ent, arg, top)
    np.testing.assert_array_equal(arg.cpu().numpy(), good[z.argmax(axis=1)])
    # logits of size 65 off by some 65 2^-24 of that: 3e-4 at most, relative in conf
    np.testing.assert_allclose(conf.cpu().numpy(), p.max(axis=1), rtol=1e-3)
    np.testing.assert_allclose(ent.cpu().numpy(), -(p * np.log(np.maximum(p, 1e-300))).sum(axis=1),
                               rtol=1e-3, atol=1e-3)
    np.testing.assert_allclose(top.cpu().numpy(), z.max(axis=1), rtol=1e-5)


def test_attention_f32_many_workgroups():
    """A batch of one long block and thousands of single rows: 64 tiles x 32 heads x 4200 sequences
    of 512 threads pass 2^32 threads.  A single row without a prefix attends to itself alone."""
    lens = [1024] + [1] * 4199
    print(f"attn f32 batch={len(lens)}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(sum(lens), 32, 64, generator=g, device="cuda") for _ in range(3))
    none = torch.empty(0, 32, 64, device="cuda")
    out = torch.full(q.shape, 7.0, device="cuda")
    eb_block_attn(Ragged.from_lengths(lens, [0] * len(lens)), q, k, v, none, none, out)
    assert torch.equal(out[1024:], v[1024:])  # one weight of exactly one
    x, y, z = (t[:1024].double().transpose(0, 1).contiguous() for t in (q, k, v))
    ref = torch.softmax(x @ y.transpose(1, 2).contiguous() / 8.0, dim=-1) @ z
    # scores of size |q||k| / sqrt(d) < 16 off by some 64 2^-24 16 / 8: 1e-5 in a weight
    torch.testing.assert_close(out[:1024].double(), ref.transpose(0, 1), rtol=2e-5, atol=2e-5)


# Slices of 64 and of 256 rows (70001 x 300 positions), odd and unaligned hidden sizes with and
# without whole 64-column rounds, partial position tiles, waves without vocabulary rows.
@pytest.mark.parametrize("rows,hidden,vocab", [
    (1, 1, 1), (2, 3, 5), (31, 64, 65), (32, 16, 256), (33, 333, 300), (64, 100, 2049),
    (300, 65, 70001)])
def test_lmhead_f32(rows, hidden, vocab):
    print(f"lmhead f32 rows={rows} hidden={hidden} vocab={vocab}", flush=True)
    rng = np.random.default_rng([rows, hidden, vocab])
    w = rng.standard_normal((vocab, hidden), dtype=np.float32) / np.float32(np.sqrt(hidden))
    h = 2.0 * rng.standard_normal((rows, hidden), dtype=np.float32)
    ref = oracle.lmhead_confidence(h, w)
    conf, ent, gap, top = (torch.empty(rows, device="cuda") for _ in range(4))
    arg = torch.empty(rows, dtype=torch.int32, device="cuda")
    eb_lmhead_features(torch.from_numpy(h).cuda(), torch.from_numpy(w).cuda(), conf, ent, arg, gap,
                       max_logit=top)
    np.testing.assert_array_equal(arg.cpu().numpy(), ref["argmax"])
    # d products of |w||h| < 40 in fp32: below d 2^-24 40 = 8e-4 (d = 333) at worst, some sqrt(d)
    # of that for random signs
    for got, want in ((conf, "conf"), (ent, "entropy"), (top, "max_logit"), (gap, "top2_gap")):
        np.testing.assert_allclose(got.cpu().numpy(), ref[want], rtol=0, atol=5e-5, err_msg=want)
