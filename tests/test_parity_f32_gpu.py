"""fp32 forward and backward kernels at the edges of their tiles (32 tokens), blocks and chunks
(64 tokens), against the fp64 oracle.

A window of n tokens is cut into query and key tiles of 32, and each query (key) tile is shared by
two waves that take its even and odd streamed tiles: n = 1, 31 .. 33 leave the second wave without
a tile or with one, 63 .. 65 end a block and a chunk, and in KV-token mode n = 64 puts the pad token
alone into a chunk.  Bounds: 1e-5 absolute for the output (values of order 1) and the log-sum-exp,
1e-5 of the largest reference gradient: sums of up to 300 products of order 1 in fp32 are off by a
few 2^-24 times their size (~1e-6 here)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2407_02109_amd import binding as fb
from paper_2407_02109_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # B, heads, H, W, window, shift, pad_mode
    (1, 2, 1, 1, 4, 0, 0),      # one token
    (1, 1, 1, 31, 33, 0, 1), (1, 1, 1, 32, 33, 0, 1), (2, 3, 3, 11, 12, 0, 0),        # n = 31, 32, 33
    (1, 1, 7, 9, 9, 0, 0), (1, 2, 8, 8, 9, 0, 1), (1, 2, 8, 8, 8, 0, 0), (1, 1, 5, 13, 13, 0, 1),   # 63, 64, 64, 65
    (1, 1, 9, 14, 14, 0, 1), (2, 1, 16, 8, 16, 0, 0), (1, 1, 3, 43, 43, 0, 0),        # 126, 128, 129
    (1, 5, 19, 23, 10, 7, 1),   # shifted, ragged: windows of many sizes, five heads
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_tile_edges(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, heads, H, W, k, s, pm = case
    print("[case] fp32 %s" % (case,), flush=True)
    wl = synth.Workload("case", B, heads, H, W, 64, k, s, "f32", seed=77, pad_mode=pm)
    q, kk, v = synth.make_inputs(wl)
    dout = synth.make_grad(wl)
    gpu = [t.to("cuda:0") for t in (q, kk, v, dout)]
    out, lse = fb.swin_attn_fwd_train(*gpu[:3], [(H, W)], k, s, pm)
    plain = fb.swin_attn(*gpu[:3], H, W, k, s, pm)
    grads = fb.swin_attn_bwd(*gpu[:3], out, gpu[3], lse, [(H, W)], k, s, pm)
    torch.cuda.synchronize()
    assert torch.equal(out, plain)
    f64 = [synth.to_f64_numpy(t) for t in (q, kk, v, dout)]
    assert np.abs(synth.to_f64_numpy(out) - O.swin_attention_textbook(*f64[:3], H, W, k, s, pm)).max() <= 1e-5
    assert np.abs(synth.to_f64_numpy(lse) - O.swin_attention_lse(*f64[:3], H, W, k, s, pm)).max() <= 1e-5
    for name, got, ref in zip(("dq", "dk", "dv"), grads, O.swin_attention_bwd(*f64, H, W, k, s, pm)):
        assert np.abs(synth.to_f64_numpy(got) - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max()), name


@pytest.mark.parametrize("d", [32, 128])
@pytest.mark.parametrize("n", [33, 64, 65])
def test_head_dim_tile_edges(d, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] fp32 head_dim %d, %d tokens" % (d, n), flush=True)
    wl = synth.Workload("case", 2, 3, 1, n, d, n + 1, 0, "f32", seed=78, pad_mode=1)
    q, k, v = synth.make_inputs(wl)
    out = fb.swin_attn(*(t.to("cuda:0") for t in (q, k, v)), 1, n, n + 1, 0, 1)
    torch.cuda.synchronize()
    ref = O.swin_attention_textbook(*(synth.to_f64_numpy(t) for t in (q, k, v)), 1, n, n + 1, 0, 1)
    assert np.abs(synth.to_f64_numpy(out) - ref).max() <= 1e-5


def test_minus_infinity_logits_have_no_weight():
    """Keys whose logits are -inf for every query have weight zero, also when they fill the whole
    first tile of one of the two waves of a query tile."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] fp32 logits of -inf", flush=True)
    g = torch.Generator().manual_seed(5)
    q, k, v = (torch.randn(1, 64, 1, 64, generator=g) for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 0.1
    k[0, :32, 0, 0] = -float("inf")       # the whole first key tile: weight zero for every query
    ref = torch.nn.functional.scaled_dot_product_attention(
        *(t.transpose(1, 2).double() for t in (q, k[:, 32:], v[:, 32:]))).transpose(1, 2)
    out = fb.swin_attn(*(t.to("cuda:0") for t in (q, k, v)), 8, 8, 8, 0, 0)
    torch.cuda.synchronize()
    assert (out.cpu().double() - ref).abs().max() <= 1e-5


@pytest.mark.parametrize("hw", [(5, 9), (4, 16)], ids=lambda c: "%dx%d" % c)
def test_key_of_minus_infinity_logits_gets_no_gradient(hw):
    """A key whose logit is -inf for every query: its dk and dv are zero, and the other keys' and dq
    (but for the channel where zero weight meets the key's -inf) are those of the window without it,
    with the last tile of queries partial (45 tokens) and whole."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] fp32 backward, a key of -inf logits, %dx%d" % hw, flush=True)
    H, W = hw
    g = torch.Generator().manual_seed(7)
    q, k, v, dout = (torch.randn(1, H * W, 2, 64, generator=g) for _ in range(4))
    q[..., 0] = q[..., 0].abs() + 0.1
    k[0, 7, :, 0] = -float("inf")
    gpu = [t.to("cuda:0") for t in (q, k, v, dout)]
    out, lse = fb.swin_attn_fwd_train(*gpu[:3], [hw], 16, 0, 0)
    dq, dk, dv = (t.cpu().double() for t in fb.swin_attn_bwd(*gpu[:3], out, gpu[3], lse, [hw], 16, 0, 0))
    rest = torch.arange(H * W) != 7
    ref = [t.transpose(1, 2).double().contiguous().requires_grad_() for t in (q, k[:, rest], v[:, rest])]
    torch.nn.functional.scaled_dot_product_attention(*ref).backward(dout.transpose(1, 2).double().contiguous())
    rq, rk, rv = (t.grad.transpose(1, 2) for t in ref)
    assert (dk[0, 7] == 0).all() and (dv[0, 7] == 0).all()
    for name, got, want in (("dq", dq[..., 1:], rq[..., 1:]), ("dk", dk[:, rest], rk), ("dv", dv[:, rest], rv)):
        assert (got - want).abs().max() <= 1e-5 * max(1.0, want.abs().max().item()), name


@pytest.mark.parametrize("pm", [0, 1])
def test_query_of_infinite_lse_has_no_weight(pm):
    """A query whose log-sum-exp the caller sets to +inf has P = 0: its dq is zero, and the other
    gradients (the pad token's too) are those of a zero dout row."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] fp32 backward, infinite log-sum-exp, pad mode %d" % pm, flush=True)
    wl = synth.Workload("case", 1, 2, 4, 11, 64, 16, 0, "f32", seed=79, pad_mode=pm)
    q, k, v = synth.make_inputs(wl)
    dout = synth.make_grad(wl)
    gpu = [t.to("cuda:0") for t in (q, k, v, dout)]
    out, lse = fb.swin_attn_fwd_train(*gpu[:3], [(4, 11)], 16, 0, pm)
    lse[:, :, 3] = float("inf")
    grads = fb.swin_attn_bwd(*gpu[:3], out, gpu[3], lse, [(4, 11)], 16, 0, pm)
    dout[:, 3] = 0
    f64 = [synth.to_f64_numpy(t) for t in (q, k, v, dout)]
    assert (synth.to_f64_numpy(grads[0])[:, 3] == 0).all()
    for name, got, ref in zip(("dq", "dk", "dv"), grads, O.swin_attention_bwd(*f64, 4, 11, 16, 0, pm)):
        assert np.abs(synth.to_f64_numpy(got) - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max()), name


def test_an_image_has_the_same_bits_alone_and_in_a_batch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] fp32 alone and in a batch", flush=True)
    wl = synth.Workload("case", 3, 2, 21, 19, 64, 18, 5, "f32", seed=80, pad_mode=1)
    q, k, v = (t.to("cuda:0") for t in synth.make_inputs(wl))
    dout = synth.make_grad(wl).to("cuda:0")
    both = []
    for b in (slice(0, 3), slice(2, 3)):
        t = [x[b].contiguous() for x in (q, k, v, dout)]
        out, lse = fb.swin_attn_fwd_train(*t[:3], [(21, 19)], 18, 5, 1)
        both.append([x[-1] for x in (out, lse, *fb.swin_attn_bwd(*t[:3], out, t[3], lse, [(21, 19)], 18, 5, 1))])
    assert all(torch.equal(x, y) for x, y in zip(*both))
