"""The generic (row-major weights, exact fp32 products) kernels at the edges of their tiles."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import decoder as od
from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth
import helpers as H

pytestmark = pytest.mark.gpu


# one and two row tiles, the last row of a tile; K of one partial chunk, of one wave's share, one chunk into the
# second turn of the waves' ring and beyond it; one and several feature tiles
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,k", [(1, 16, 8), (5, 48, 40), (16, 16, 256), (17, 32, 264), (32, 80, 776), (31, 16, 1600)])
def test_linear(dtype, m, n, k):
    g = torch.Generator().manual_seed(m * 1000 + k)
    x = torch.randn(m, k, generator=g)
    w = torch.randn(n, k, generator=g).to(dtype)
    y = B.linear(x.cuda(), w.cuda(), B.GEMM_DOT).cpu().double()
    ref = x.double() @ w.double().t()
    # products exact, k sums of fp32 at worst: k * 2^-24 times the sum of magnitudes
    bound = k * 2.0 ** -24 * (x.double().abs() @ w.double().abs().t())
    assert torch.all((y - ref).abs() <= bound)
    one = B.linear(x[m - 1:].contiguous().cuda(), w.cuda(), B.GEMM_DOT).cpu().double()
    assert torch.equal(one[0], y[m - 1])    # a row's sums do not depend on the other rows


@pytest.mark.parametrize("shape,page_tokens", [(synth.TINY, 8), (synth.TINY, 256), (synth.TINY_MQA, 16),
                                               (dataclasses.replace(synth.MID_GQA, dtype="f32"), 32)])
@pytest.mark.parametrize("cached", [0, 47, 64, 130])
def test_windows_across_tile_and_split_edges(shape, page_tokens, cached):
    w = synth.make_weights(shape, 5)
    cap = 256
    dec = od.Decoder(shape, w, cap)
    model = B.Model(shape, H.to_cuda(w), max_window=32, max_positions=cap, page_tokens=page_tokens)
    kv = B.KVCache(model, cap)
    if cached:
        H.seed_kv_both(shape, dec, kv, cached, 9)
    pos = cached
    for n in (17, 1, 16, 32):
        win = synth.random_tokens(shape.vocab, n, pos + 1)
        ref = dec.forward(win)
        dec.set_length(pos + n)
        # (an odd address: the logits go through the workspace; an even one takes them directly)
        flat = torch.empty(n * shape.vocab + 1, dtype=torch.float32, device="cuda")
        buf = flat[1:] if n == 17 else flat[:-1]
        B.verify(model, kv, win, B.APPEND, out_logits=buf)
        err = float(np.max(np.abs(buf.cpu().numpy().astype(np.float64).reshape(n, -1) - ref)))
        assert err < H.TOL["f32"], (n, err)
        pos += n


def test_prompt_windows_leave_what_one_window_at_a_time_leaves():
    shape = synth.TINY
    w = H.to_cuda(synth.make_weights(shape, 5))
    model = B.Model(shape, w, max_window=32, max_positions=256)
    a, b = B.KVCache(model, 256), B.KVCache(model, 256)
    prompt = synth.random_tokens(shape.vocab, 107, 3)
    last = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    rows = torch.empty(11, shape.vocab, dtype=torch.float32, device="cuda")
    t0 = B.prefill(model, a, prompt, out_logits=last)
    for lo in (0, 32, 64):
        B.verify(model, b, prompt[lo:lo + 32], B.APPEND)
    _, t1 = B.verify(model, b, prompt[96:], B.APPEND, out_logits=rows)
    assert t0 == t1 and a.length == b.length == 107 and torch.equal(last, rows[10])
    for layer in range(shape.n_layers):
        for x, y in zip(a.read(layer, 0, 107), b.read(layer, 0, 107)):
            assert torch.equal(x, y)
    win = synth.random_tokens(shape.vocab, 5, 77)     # the device's length followed
    assert B.verify(model, a, win, want_predicts=True) == B.verify(model, b, win, want_predicts=True)


# bf16, a few rows, two and three blocks per compute unit (of 256): K of a partial chunk and of several turns of the
# waves, the longest rows that are kept in LDS (12288 floats) and one piece more
@pytest.mark.parametrize("n,k", [(8192, 8), (8192, 776), (8192, 4096), (12288, 264), (12288, 4104), (12288, 6144), (12288, 6152), (8192, 12288)])
def test_linear_of_a_few_rows_has_the_bits_of_sixteen(n, k):
    g = torch.Generator(device="cuda").manual_seed(n + k)
    x = torch.randn(16, k, generator=g, device="cuda")
    w = torch.randn(n, k, generator=g, device="cuda").to(torch.bfloat16)
    y = B.linear(x, w, B.GEMM_DOT)
    for m in (1, 2, 3, 4, 5):
        assert torch.equal(y[:m], B.linear(x[:m].contiguous(), w, B.GEMM_DOT)), m


# bf16 weights: LM heads of two and three blocks per compute unit (of 256); O and down of just over one, K of down up to
# what one row and not two may take in LDS, and beyond it
@pytest.mark.parametrize("shape", [dataclasses.replace(synth.MID_GQA, vocab=8192), dataclasses.replace(synth.MID_GQA, vocab=12288),
                                   synth.ModelShape(1, 4224, 33, 128, 7056, 512, "bf16", n_kv_heads=3),
                                   synth.ModelShape(1, 4224, 33, 128, 14080, 512, "bf16", n_kv_heads=3),
                                   synth.ModelShape(1, 4224, 33, 128, 14096, 512, "bf16", n_kv_heads=3)], ids=lambda s: "%dx%dx%d" % (s.d_model, s.d_ffn, s.vocab))
def test_windows_of_a_few_rows_have_the_bits_of_sixteen(shape):
    model = B.Model(shape, synth.make_weights(shape, 5, device="cuda"), max_window=16, max_positions=128, gemm_path=B.GEMM_DOT)
    kv = B.KVCache(model, 128)
    win = synth.random_tokens(shape.vocab, 16, 3)
    rows = {}
    for n in (16, 5, 4, 3, 2, 1):
        kv.truncate(0)
        rows[n] = torch.empty(n, shape.vocab, dtype=torch.float32, device="cuda")
        B.verify(model, kv, win[:n], B.APPEND, out_logits=rows[n])
        assert torch.equal(rows[n], rows[16][:n]), n


# tokens whose logits are NaN: the first, one that is the first a thread reads, in it and behind it, the first of a wave, every
# fourth (the first of every thread), all but one, all
@pytest.mark.parametrize("shape,path", [(synth.TINY, B.GEMM_AUTO), (synth.MID_BF16, B.GEMM_MFMA_LAUNCHES)])
@pytest.mark.parametrize("bad", [[0], [4], [5], [256], range(0, 1024, 4), [i for i in range(2048) if i != 700], range(2048)],
                         ids=["0", "4", "5", "256", "fourths", "all_but_one", "all"])
def test_a_nan_among_the_logits_hides_no_other(shape, path, bad):
    w = synth.make_weights(shape, 4, device="cuda")
    bad = [i for i in bad if i < shape.vocab]
    w["lm_head"][bad] = float("nan")
    model = B.Model(shape, w, max_window=32, max_positions=64, gemm_path=path)
    kv = B.KVCache(model, 32)
    logits = torch.empty(32, shape.vocab, dtype=torch.float32, device="cuda")
    preds = B.verify(model, kv, synth.random_tokens(shape.vocab, 32, 9), B.APPEND, want_predicts=True, out_logits=logits)[2]
    assert torch.equal(torch.isnan(logits).any(0).nonzero().flatten().cpu(), torch.tensor(bad))
    assert preds == torch.nan_to_num(logits, nan=-float("inf")).argmax(-1).tolist()
