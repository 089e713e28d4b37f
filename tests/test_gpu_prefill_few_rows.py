"""The prompt GEMMs with a tile per wave: pieces of one row to 128, on either side of every row group and of the numbers of row
groups per block, leave bit for bit what the prompt in one piece does (its rows in the wide blocks; a small model's, in the same
form): an element's sums do not depend on the form.  The forms that only wide models take: test_gpu_prefill_forms.py."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

# cuts at every remainder of a row group: the pieces' first and last groups are partly other pieces' rows
PIECES = [1, 16, 15, 17, 32, 33, 31, 64, 65, 48, 113, 128, 127]


# K of 48 and 192 k-steps (whole buffers of eight) / of 8 and 22, split by four into 2 and 5 or 6 (less than one buffer)
@pytest.mark.parametrize("shape", [synth.RING_BF16, synth.TINY_BF16], ids=["ring", "tiny"])
def test_pieces_of_few_rows_give_the_bits_of_one_long_piece(shape):
    w = synth.make_weights(shape, 5, device="cuda")
    rows = sum(PIECES)
    model = B.Model(shape, w, max_window=8, max_positions=rows)
    prompt = synth.random_tokens(shape.vocab, rows, 12)
    whole, parts = B.KVCache(model, rows), B.KVCache(model, rows)
    a = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    t0 = B.prefill(model, whole, prompt, out_logits=a)
    lo = t1 = 0
    for n in PIECES:
        t1 = B.prefill(model, parts, prompt[lo:lo + n], out_logits=b)
        lo += n
    assert t0 == t1 and torch.equal(a, b)
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, rows), parts.read(layer, 0, rows)):
            assert torch.equal(x, y)
