"""Behind the last layer's keys and values a prompt goes on with its last row's group alone: bit for bit what a last piece that lies
in one row group, where there is nothing to leave out, makes of the same row, and the same cache."""
import dataclasses

import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {"bf16": dataclasses.replace(synth.TINY_BF16, n_layers=3), "f32": dataclasses.replace(synth.TINY, n_layers=3),
          "bf16_one_layer": dataclasses.replace(synth.TINY_BF16, n_layers=1), "f32_one_layer": dataclasses.replace(synth.TINY, n_layers=1)}


# rows behind `before` cached ones: one row group and two, either side of the 16 groups from which the queries are a launch of their
# own, a last group of one row and of sixteen; fp32: pieces of 256 rows, of which only the last has a row that goes on
@pytest.mark.parametrize("dtype", sorted(SHAPES))
@pytest.mark.parametrize("before,rows", [(0, 16), (0, 17), (5, 12), (0, 256), (0, 257), (11, 246), (0, 272), (3, 270), (0, 527)])
def test_a_prompt_ends_like_its_last_row_group(dtype, before, rows):
    shape, n = SHAPES[dtype], before + rows
    model = B.Model(shape, synth.make_weights(shape, 5, device="cuda"), max_window=8, max_positions=n)
    prompt = synth.random_tokens(shape.vocab, n, 13)
    whole, cut = B.KVCache(model, n), B.KVCache(model, n)
    a = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    if before:
        B.prefill(model, whole, prompt[:before])
    t0 = B.prefill(model, whole, prompt[before:], out_logits=a)
    last = (n - 1) // 16 * 16
    if last:
        B.prefill(model, cut, prompt[:last])
    t1 = B.prefill(model, cut, prompt[last:], out_logits=b)
    assert t0 == t1 and torch.equal(a, b)
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, n), cut.read(layer, 0, n)):
            assert torch.equal(x, y), layer
