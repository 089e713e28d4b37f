"""The prompt GEMM's block widths: a prompt long enough to be cut into wider blocks gives, bit for bit, what the same
prompt gives in pieces, whose GEMMs have a tile per wave (an element's sums do not depend on the form)."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def model():
    w = synth.make_weights(synth.RING_BF16, 3, device="cuda")
    return B.Model(synth.RING_BF16, w, max_window=8, max_positions=1100)


# gate / up of this shape on 256 compute units: 2, 3, 4, 5 and 6 weight fragments per wave, ragged last row groups;
# the down projection's K = 6144 splits into 4 x 48 k-steps, an odd piece length leaves odd row counts
@pytest.mark.parametrize("rows", [129, 250, 385, 640, 767, 1001])
def test_every_block_width_gives_the_bits_of_a_tile_per_wave(model, rows):
    shape = synth.RING_BF16
    prompt = synth.random_tokens(shape.vocab, rows, 11)
    whole, parts = B.KVCache(model, 1100), B.KVCache(model, 1100)
    a = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    t0 = B.prefill(model, whole, prompt, out_logits=a)
    t1 = -1
    for lo in range(0, rows, 113):
        t1 = B.prefill(model, parts, prompt[lo:lo + 113], out_logits=b)
    assert t0 == t1 and torch.equal(a, b)
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, rows), parts.read(layer, 0, rows)):
            assert torch.equal(x, y)
