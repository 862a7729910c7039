"""bf16 forward with the keys of a query tile shared by several waves, which small launches of windows
of more than 256 tokens take: windows that leave a wave's share of the last 256-key chunk
empty, partial or holding the pad token alone, at every head_dim, several grids, RoPE (table and per
piece) and the training forward's log-sum-exp, against the fp64 oracle.  Bounds are the bf16 bars of the
parity tests (2e-2 max, 2e-3 mean: one rounding of values of order 1 to bf16 is up to 2^-8, that of
the probabilities averages out); the log-sum-exp 4e-3, twice what rounded probabilities can move it."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2407_02109_amd import binding as fb
from paper_2407_02109_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # B, heads, H, W, head_dim, window, shift, pad_mode
    (1, 1, 1, 257, 64, 257, 0, 0), (1, 2, 17, 17, 64, 17, 0, 0),      # n = 257, 289
    (1, 1, 16, 16, 64, 17, 0, 1), (1, 1, 9, 32, 64, 32, 0, 1),       # the pad token alone in a chunk, in a tile (n = 256, 288)
    (1, 1, 13, 25, 64, 25, 0, 1), (2, 3, 16, 24, 64, 24, 0, 0),      # n = 325, 384
    (1, 3, 37, 41, 64, 24, 11, 1), (1, 2, 64, 64, 64, 64, 32, 0),    # windows of many sizes; 1024 tokens
    (1, 2, 19, 31, 32, 20, 10, 1), (1, 2, 33, 32, 32, 33, 0, 0),
    (1, 2, 19, 31, 128, 20, 10, 1), (1, 2, 33, 32, 128, 33, 0, 0),
    # two blocks of 256 queries per window and head: 64 | 66 .. 128 | 130 blocks, four, two and one wave per query tile
    (1, 32, 17, 16, 64, 17, 0, 1), (1, 33, 17, 16, 64, 17, 0, 1), (2, 32, 17, 17, 64, 17, 0, 0),
    (1, 65, 17, 16, 64, 17, 0, 1), (1, 40, 17, 17, 32, 18, 0, 1), (1, 40, 17, 17, 128, 18, 0, 1),
    (2, 9, 33, 32, 64, 33, 0, 0),
]


def _close(got, ref):
    e = np.abs(synth.to_f64_numpy(got) - ref)
    assert np.isfinite(e).all() and e.max() <= 2e-2 and e.mean() <= 2e-3, (e.max(), e.mean())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_shared_keys(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, heads, H, W, d, k, s, pm = case
    print("[case] bf16 forward split %s" % (case,), flush=True)
    wl = synth.Workload("case", B, heads, H, W, d, k, s, "bf16", seed=91, pad_mode=pm)
    q, kk, v = synth.make_inputs(wl)
    gpu = [t.to("cuda:0") for t in (q, kk, v)]
    out = fb.swin_attn(*gpu, H, W, k, s, pm)
    f64 = [synth.to_f64_numpy(t) for t in (q, kk, v)]
    _close(out, O.swin_attention_textbook(*f64, H, W, k, s, pm))
    if d != 64:
        return
    train, lse = fb.swin_attn_fwd_train(*gpu, [(H, W)], k, s, pm)
    assert torch.equal(train, out)
    assert np.abs(synth.to_f64_numpy(lse) - O.swin_attention_lse(*f64, H, W, k, s, pm)).max() <= 4e-3


def test_a_share_of_minus_infinity_logits_has_no_weight():
    """Every second key tile has logits of -inf for every query: one wave's whole share."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] bf16 forward split, logits of -inf", flush=True)
    g = torch.Generator().manual_seed(6)
    q, k, v = (torch.randn(1, 1024, 1, 64, generator=g) for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 0.1
    dead = (torch.arange(1024) // 32) % 2 == 1
    k[0, dead, 0, 0] = -float("inf")
    q, k, v = (t.bfloat16() for t in (q, k, v))
    ref = torch.nn.functional.scaled_dot_product_attention(
        *(t.transpose(1, 2).double() for t in (q, k[:, ~dead], v[:, ~dead]))).transpose(1, 2)
    out = fb.swin_attn(*(t.to("cuda:0") for t in (q, k, v)), 32, 32, 32, 0, 0)
    torch.cuda.synchronize()
    _close(out, ref.numpy())
