"""Prompt attention at the edges of pages, page pairs and the waves' turns: the prompt in one pass against the same rows
through the step, and bit for bit against the prompt in pieces cut inside pages."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu


# rows x cached: one row, a page, a pair, one row more, first groups that start inside a page, an odd number of groups,
# fewer pairs than waves, several turns of the waves, past the 64 pairs whose page numbers a wave holds at a time
@pytest.mark.parametrize("shape", [synth.MID_GQA, synth.TINY_BF16], ids=["dh128_gqa", "dh64"])
@pytest.mark.parametrize("cached,rows", [(0, 1), (0, 16), (0, 17), (0, 33), (5, 27), (15, 1), (16, 49), (31, 34), (100, 129), (250, 130), (8300, 40)])
def test_one_pass_against_windows_and_pieces(shape, cached, rows):
    w = synth.make_weights(shape, 3, device="cuda")
    cap = cached + rows + 8
    model = B.Model(shape, w, max_window=8, max_positions=cap)
    kvs = []
    for _ in range(3):
        kv = B.KVCache(model, cap)
        for layer in range(shape.n_layers):
            if cached:
                k, v = synth.kv_fill(shape, 7, layer, cached, device="cuda")
                kv.write(layer, 0, k.float().contiguous(), v.float().contiguous())
        kv.truncate(cached)
        kvs.append(kv)
    prompt = synth.random_tokens(shape.vocab, rows, 11)
    logits = [torch.empty(shape.vocab, dtype=torch.float32, device="cuda") for _ in range(3)]
    B.prefill(model, kvs[0], prompt, out_logits=logits[0])
    for lo in range(0, rows, 21):
        B.prefill(model, kvs[1], prompt[lo:lo + 21], out_logits=logits[1])
    for lo in range(0, rows, 8):
        n = len(prompt[lo:lo + 8])
        buf = torch.empty(n, shape.vocab, dtype=torch.float32, device="cuda")
        B.verify(model, kvs[2], prompt[lo:lo + 8], B.APPEND, out_logits=buf)
        logits[2] = buf[-1]
    assert torch.equal(logits[0], logits[1])
    # two orders of the same sums over bf16 keys and values: the tolerance the logits have against the oracle
    assert (logits[0] - logits[2]).abs().max().item() < 2e-2
    for layer in range(shape.n_layers):
        one, cut, step = (kv.read(layer, cached, rows) for kv in kvs)
        for x, y, z in zip(one, cut, step):
            assert torch.equal(x, y)
            # a rounding boundary apart at most: one bf16 unit in the last place of the largest value
            assert (x - z).abs().max().item() <= 2.0 ** -7 * x.abs().max().item()


# the first row of a page pair's second page, one inside it, the last row of a first page, the first of a pair
@pytest.mark.parametrize("shape", [synth.MID_GQA, synth.TINY_BF16], ids=["dh128_gqa", "dh64"])
@pytest.mark.parametrize("at", [16, 20, 47, 48, 64, 90])
def test_a_row_that_is_not_finite_leaves_the_pages_before_it_alone(shape, at):
    w = synth.make_weights(shape, 3, device="cuda")
    w["embed"][7] = float("nan")
    model = B.Model(shape, w, max_window=8, max_positions=128)
    prompt = [t if t != 7 else 8 for t in synth.random_tokens(shape.vocab, 100, 11)]
    page0 = at // 16 * 16
    whole, before = B.KVCache(model, 128), B.KVCache(model, 128)
    B.prefill(model, whole, prompt[:at] + [7] + prompt[at + 1:])
    B.prefill(model, before, prompt[:page0])
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, page0), before.read(layer, 0, page0)):
            assert torch.equal(x, y), layer   # (NaN equals nothing)


# a cached key with a NaN, or with values whose scores are far beyond what a rounded sum resolves: on a page seen in full by
# every row, on the last cached one, on the rows' own page
@pytest.mark.parametrize("shape", [synth.MID_GQA, synth.TINY_BF16], ids=["dh128_gqa", "dh64"])
@pytest.mark.parametrize("at,cached,rows", [(3, 64, 40), (63, 64, 40), (150, 200, 33), (40, 50, 3)])
@pytest.mark.parametrize("value", [float("nan"), 1e6, 1e10, 1e20, 1e30])
def test_a_key_with_a_nan_has_weight_zero_and_a_huge_one_its_weight_as_in_a_step(shape, at, cached, rows, value):
    w = synth.make_weights(shape, 3, device="cuda")
    model = B.Model(shape, w, max_window=8, max_positions=256)
    prompt = synth.random_tokens(shape.vocab, rows, 11)
    one, step = B.KVCache(model, 256), B.KVCache(model, 256)
    for kv in (one, step):
        for layer in range(shape.n_layers):
            k, v = (t.float().contiguous() for t in synth.kv_fill(shape, 7, layer, cached, device="cuda"))
            k[at, ::3] = value
            kv.write(layer, 0, k, v)
        kv.truncate(cached)
    got = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    B.prefill(model, one, prompt, out_logits=got)
    for lo in range(0, rows, 8):
        ref = torch.empty(len(prompt[lo:lo + 8]), shape.vocab, dtype=torch.float32, device="cuda")
        B.verify(model, step, prompt[lo:lo + 8], B.APPEND, out_logits=ref)
    assert torch.isfinite(ref[-1]).all()
    assert (got - ref[-1]).abs().max().item() < 2e-2   # (as in the comparison with windows above)


# query rows in LDS where the blocks (heads x pairs of row groups) are more than one per compute unit, two at head dim 64, in registers otherwise: a prompt whose
# blocks are, at a page's start and inside one, against pieces of it whose blocks are not, and one of the last size that has them in registers
@pytest.mark.parametrize("shape,rows,piece", [(synth.RING_BF16, 513, 512), (synth.RING_BF16, 600, 256), (synth.TINY_BF16, 4097, 4096), (synth.TINY_BF16, 4200, 1300)],
                         ids=["dh128_first", "dh128", "dh64_first", "dh64"])
@pytest.mark.parametrize("before", [0, 21])
def test_query_rows_in_lds_and_in_registers_give_the_same_bits(shape, rows, piece, before):
    w = synth.make_weights(shape, 3, device="cuda")
    model = B.Model(shape, w, max_window=8, max_positions=before + rows)
    prompt = synth.random_tokens(shape.vocab, before + rows, 11)
    one, cut = (B.KVCache(model, before + rows) for _ in range(2))
    logits = [torch.empty(shape.vocab, dtype=torch.float32, device="cuda") for _ in range(2)]
    for kv in (one, cut):
        if before:
            B.prefill(model, kv, prompt[:before])
    B.prefill(model, one, prompt[before:], out_logits=logits[0])
    piece -= before % 16    # (so that its groups are as many)
    for lo in range(before, before + rows, piece):
        B.prefill(model, cut, prompt[lo:min(lo + piece, before + rows)], out_logits=logits[1])
    assert torch.equal(logits[0], logits[1])
    for layer in range(shape.n_layers):
        for x, y in zip(one.read(layer, 0, before + rows), cut.read(layer, 0, before + rows)):
            assert torch.equal(x, y)
