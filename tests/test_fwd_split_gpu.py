"""bf16 forward of windows of more than 256 tokens, by the waves that share the keys of a query tile:
four in launches of at most 64 blocks of 256 queries, two up to 128, one above (256 compute units; at
head_dim 128 fewer where a workgroup would wait for another).  Windows that leave a wave's share of the
last 256-key chunk empty, partial or holding the pad token alone, and each of the three with every
head_dim, with several grids, with RoPE (table and per piece) and with the training forward's
log-sum-exp, against the fp64 oracle.  Bounds are the bf16 bars of the parity tests (2e-2 max, 2e-3 mean:
one rounding of values of order 1 to bf16 is up to 2^-8, that of the probabilities averages out); the
log-sum-exp 4e-3, twice what rounded probabilities can move it, and with RoPE the rounding of the
rotated q and k besides (2 * 2^-9 relative per logit: a rotation keeps norms)."""
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
    # one wave per query tile, shifted ragged windows of up to 1024 tokens
    (1, 10, 61, 66, 64, 32, 11, 1), (2, 6, 61, 66, 32, 32, 11, 0), (1, 10, 61, 66, 128, 32, 11, 1),
    # head_dim 128, fewer waves than the blocks alone would give: 120 blocks, one wave; 63, two
    (1, 5, 64, 64, 128, 20, 10, 1), (1, 9, 42, 42, 128, 42, 0, 1),
]


def _waves(B, heads, grids, window, shift):
    """Waves per query tile at head_dim 32 and 64, from the blocks of 256 queries."""
    def extents(n):
        cuts = [0] + list(range(shift if shift > 0 else window, n, window)) + [n]
        return [b - a for a, b in zip(cuts[:-1], cuts[1:])]
    blocks = B * heads * sum((y * x + 255) // 256 for H, W in grids for y in extents(H) for x in extents(W))
    return 4 if blocks <= 64 else 2 if blocks <= 128 else 1


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


ROPE_CASES = [  # waves per tile, heads, H, W, window, shift, pad_mode; windows past 32 x 32 tokens: per piece
    (4, 3, 49, 50, 32, 13, 1), (2, 5, 49, 50, 32, 13, 0), (1, 12, 49, 50, 32, 13, 1),
    (4, 2, 57, 63, 40, 20, 0), (2, 6, 57, 63, 40, 20, 1), (1, 11, 57, 63, 40, 20, 0),
]


@pytest.mark.parametrize("case", ROPE_CASES, ids=lambda c: "x".join(map(str, c)))
def test_shared_keys_rope(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    waves, heads, H, W, k, s, pm = case
    assert _waves(1, heads, [(H, W)], k, s) == waves
    print("[case] bf16 forward split, RoPE %s" % (case,), flush=True)
    wl = synth.Workload("case", 1, heads, H, W, 64, k, s, "bf16", seed=92, pad_mode=pm)
    q, kk, v = synth.make_inputs(wl)
    gpu = [t.to("cuda:0") for t in (q, kk, v)]
    out = fb.swin_attn_rope(*gpu, H, W, k, s, pm)
    f64 = [synth.to_f64_numpy(t) for t in (q, kk, v)]
    _close(out, O.swin_attention_rope(*f64, H, W, k, s, pm, 10000.0, 1.0))
    train, lse = fb.swin_attn_rope_fwd_train(*gpu, H, W, k, s, pm)
    assert torch.equal(train, out)
    qn = np.linalg.norm(f64[0], axis=-1).transpose(0, 2, 1)
    kmax = np.linalg.norm(f64[1], axis=-1).max(axis=1)[:, :, None]
    e = np.abs(synth.to_f64_numpy(lse) - O.swin_attention_rope_lse(*f64, H, W, k, s, pm, 10000.0, 1.0))
    assert (e <= 4e-3 + 2.0 * 2.0 ** -9 * 0.125 * qn * kmax).all()


MS_CASES = [  # waves per tile, heads, grids, head_dim, window, shift, pad_mode
    (4, 2, [(41, 47), (20, 19)], 64, 30, 11, 1), (2, 5, [(41, 47), (20, 19)], 64, 30, 11, 0),
    (1, 10, [(41, 47), (20, 19)], 64, 30, 11, 1),
    (4, 2, [(41, 47), (20, 19)], 32, 30, 11, 0), (2, 5, [(41, 47), (20, 19)], 32, 30, 11, 1),
    (1, 10, [(41, 47), (20, 19)], 32, 30, 11, 0),
    (4, 2, [(41, 47), (20, 19)], 128, 30, 11, 1), (2, 5, [(41, 47), (20, 19)], 128, 30, 11, 0),
    (1, 10, [(41, 47), (20, 19)], 128, 30, 11, 1),
]


@pytest.mark.parametrize("case", MS_CASES, ids=lambda c: "-".join(map(str, c[:2] + c[3:])))
def test_shared_keys_several_grids(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    waves, heads, grids, d, k, s, pm = case
    assert _waves(1, heads, grids, k, s) == waves
    print("[case] bf16 forward split, grids %s" % (case,), flush=True)
    wl = synth.Workload("case", 1, heads, *grids[0], d, k, s, "bf16", seed=93, pad_mode=pm, grids=tuple(grids))
    q, kk, v = synth.make_inputs(wl)
    gpu = [t.to("cuda:0") for t in (q, kk, v)]
    out = fb.swin_attn_ms(*gpu, grids, k, s, pm)
    f64 = [synth.to_f64_numpy(t) for t in (q, kk, v)]
    _close(out, O.swin_attention_ms(*f64, grids, k, s, pm))
    if d != 64:
        return
    train, lse = fb.swin_attn_fwd_train(*gpu, grids, k, s, pm)
    assert torch.equal(train, out)
    assert np.abs(synth.to_f64_numpy(lse) - O.swin_attention_ms_lse(*f64, grids, k, s, pm)).max() <= 4e-3
