"""Windows of 17..32 rows on shapes whose GEMMs take each of the forms for them: rows are bit for bit those of a window
of 16 rows or fewer, which the oracle tests pin, and close to the generic path's."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

# on 256 compute units: d 4096 to 8192 split O and down (8, 9, 10, 12 and 16 waves per block, the last block of d 4224 with
# three tiles for its nine waves; K of one, two and three buffers, an odd number of k-steps in a class); gate / up of one
# tile per compute unit (ffn 1360 / 2048) and of 5, 6, 7 and 11 tiles per block (one pass of T = 6, 6 and 8, two of 6), LM heads of
# one tile per compute unit or fewer, of 2, 9 and 16 per block (two passes of 5 and of 8)
SHAPES = {
    "d4096": synth.ModelShape(1, 4096, 32, 128, 11008, 4096, "bf16"),
    "d4096_narrow": synth.ModelShape(1, 4096, 32, 128, 1360, 36864, "bf16", n_kv_heads=2),
    "d4224": synth.ModelShape(1, 4224, 33, 128, 10000, 65024, "bf16", n_kv_heads=3),
    "d5120": synth.ModelShape(1, 5120, 40, 128, 13824, 8192, "bf16"),
    "d4096_wide": synth.ModelShape(1, 4096, 64, 64, 21776, 2048, "bf16"),
    "d6144": synth.ModelShape(1, 6144, 48, 128, 2048, 1024, "bf16", n_kv_heads=4),
    "d8192": synth.ModelShape(1, 8192, 64, 128, 2048, 1024, "bf16", n_kv_heads=4),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_rows_of_a_wide_window(name):
    shape = SHAPES[name]
    w = synth.make_weights(shape, 3, device="cuda")
    model = B.Model(shape, w, max_window=32, max_positions=256)
    kv = B.KVCache(model, 256)
    B.prefill(model, kv, synth.random_tokens(shape.vocab, 75, 1))
    win = synth.random_tokens(shape.vocab, 32, 2)
    rows = {}
    for n in (32, 25, 17, 16, 8):
        kv.truncate(75)
        rows[n] = torch.empty(n, shape.vocab, dtype=torch.float32, device="cuda")
        B.verify(model, kv, win[:n], B.APPEND, out_logits=rows[n])
    for n in (25, 17, 16, 8):
        assert torch.equal(rows[32][:n], rows[n]), n
    # row 31 through sixteen-row windows
    kv.truncate(75)
    B.verify(model, kv, win[:16], B.APPEND)
    last = torch.empty(16, shape.vocab, dtype=torch.float32, device="cuda")
    B.verify(model, kv, win[16:], B.APPEND, out_logits=last)
    assert torch.equal(rows[32][16:], last)


@pytest.mark.parametrize("n,k", [(4096, 11008), (16, 2048), (4096, 264), (5120, 5120), (22016, 4096), (27648, 5120), (36864, 2056), (53248, 1024), (65024, 520)])
def test_linear_of_17_to_32_rows(n, k):
    g = torch.Generator(device="cuda").manual_seed(n + k)
    x = torch.randn(32, k, generator=g, device="cuda")
    w = (torch.randn(n, k, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    packed = B.pack_weights(w)
    ref = x.double() @ w.double().t()
    y = B.linear(x, w, B.GEMM_MFMA, packed=packed)
    # operand error 2^-17 per term (hi + lo), fp32 sums
    bound = (2.0 ** -16 + k * 2.0 ** -24) * (x.double().abs() @ w.double().abs().t())
    assert torch.all((y.double() - ref).abs() <= bound)
    for m in (17, 16):
        assert torch.equal(y[:m], B.linear(x[:m].contiguous(), w, B.GEMM_MFMA, packed=packed))
