"""LM-head kernels at the edges of their tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16450_amd import eb_lmhead_confidence, eb_lmhead_features
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


@pytest.mark.parametrize("hidden", [64, 192, 1088])
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("vocab", [1, 40, 30000, 40000, 70000, 100001, 152064, 190000])
def test_stream_loads(rows, hidden, vocab):
    """LM-head streaming kernel: one to six 8-row loads per wave (with whole and half 16-row tiles
    and waves without rows), one, two and four position tiles, hidden sizes of one 64-column k-step,
    of less than a chunk and of a chunk and a remainder; whole lines with one load and, at the
    largest hidden size, with five and six, half lines otherwise."""
    print(f"stream rows={rows} hidden={hidden} vocab={vocab}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + 100 * hidden + vocab)
    w = torch.randn(vocab, hidden, generator=g, device="cuda").mul_(hidden ** -0.5).bfloat16()
    h = torch.randn(rows, hidden, generator=g, device="cuda")
    t = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
    t[-1] = vocab - 1
    u = w[t].float()
    h = (h + 12.0 * u / u.norm(dim=1, keepdim=True)).bfloat16()
    conf, ent, gap, top = (torch.empty(rows, device="cuda") for _ in range(4))
    arg = torch.empty(rows, dtype=torch.int32, device="cuda")
    eb_lmhead_features(h, w, conf, ent, arg, gap, max_logit=top)
    z = h.double() @ w.double().t()
    ref = oracle.eb_oracle.confidence_stats(z.cpu().numpy())
    # fp32 sums of d products, |w||h| <= 50: d 2^-24 50 < 4e-3 at worst (d = 1088) and some
    # sqrt(d) of that, 1e-4, for sums of random signs
    two = torch.topk(z, min(2, vocab), dim=1).values
    clear = ((two[:, 0] - two[:, -1] > 1e-3) | (vocab == 1)).cpu().numpy()
    np.testing.assert_array_equal(arg.cpu().numpy()[clear], ref["argmax"][clear])
    for got, want in ((conf, "conf"), (ent, "entropy"), (top, "max_logit"), (gap, "top2_gap")):
        np.testing.assert_allclose(got.cpu().numpy(), ref[want], rtol=0, atol=1e-3, err_msg=want)


@pytest.mark.parametrize("hidden", [2048, 3584, 4096])
@pytest.mark.parametrize("rows", [16, 32, 64])
def test_stream_equal_rows(rows, hidden):
    """Equal rows of W in any vocabulary slices have bit-identical logits: the lowest id wins and
    the gap is 0.  Hidden sizes of two to sixteen chunks (3.5 at one position tile), one, two and
    four position tiles; every position's largest logit is shared by four ids anywhere in 94 slices
    of 32."""
    vocab = 3000
    print(f"equal rows rows={rows} hidden={hidden}", flush=True)
    rng = np.random.default_rng([rows, hidden])
    g = torch.Generator(device="cuda").manual_seed(rows + hidden)
    w = torch.randn(vocab, hidden, generator=g, device="cuda").mul_(hidden ** -0.5).bfloat16()
    h = torch.randn(rows, hidden, generator=g, device="cuda").bfloat16()
    ids = rng.permutation(vocab)[:4 * rows].reshape(rows, 4)
    # z = |h| (8 sigma of a noise logit) for the four, below 6 |h| / sqrt(hidden) for the others
    u = (h.float() / h.float().norm(dim=1, keepdim=True)).bfloat16()
    w[torch.from_numpy(ids).cuda().flatten()] = u.repeat_interleave(4, dim=0)
    conf, ent, gap, top = (torch.empty(rows, device="cuda") for _ in range(4))
    arg = torch.empty(rows, dtype=torch.int32, device="cuda")
    eb_lmhead_features(h, w, conf, ent, arg, gap, max_logit=top)
    np.testing.assert_array_equal(arg.cpu().numpy(), ids.min(axis=1))
    np.testing.assert_array_equal(gap.cpu().numpy(), np.zeros(rows, np.float32))


# The last two heads have three and four loads per wave and are large enough for whole lines.
@pytest.mark.parametrize("hidden,vocab", [(64, 5000), (1088, 5000), (3584, 5000), (4096, 5000),
                                          (1024, 66000), (2304, 66000), (1536, 100000)])
def test_logits_do_not_depend_on_the_row_count(hidden, vocab):
    """A logit is summed in the order of its columns by every bf16 kernel: a position's largest logit
    and its id are the same bits alone, with one, two and four position tiles of the streaming kernel
    and in the tile kernel.  The sums over the vocabulary are grouped differently."""
    print(f"row counts hidden={hidden} vocab={vocab}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(hidden)
    w = torch.randn(vocab, hidden, generator=g, device="cuda").mul_(hidden ** -0.5).bfloat16()
    h = torch.randn(300, hidden, generator=g, device="cuda").bfloat16()
    got = {}
    for rows in (300, 65, 64, 33, 17, 16, 1):
        for gap in (False, True):
            conf, ent, top, delta = (torch.empty(rows, device="cuda") for _ in range(4))
            arg = torch.empty(rows, dtype=torch.int32, device="cuda")
            if gap:
                eb_lmhead_features(h[:rows], w, conf, ent, arg, delta, max_logit=top)
            else:
                eb_lmhead_confidence(h[:rows], w, conf, ent, arg, max_logit=top)
            got[rows, gap] = top, arg, conf, ent
    for (rows, gap), x in got.items():
        for i, (a, b) in enumerate(zip(x, got[300, False])):
            if i < 2:
                assert torch.equal(a, b[:rows]), (rows, gap, i)
            else:  # fp32 sums of the same terms in some 10 levels: 1e-6, and ln of it
                torch.testing.assert_close(a, b[:rows], rtol=1e-5, atol=1e-5)
