"""The prompt GEMMs that only wide models take: blocks half as wide for up to 128 rows (narrow) and two widths of blocks side by
side (mixed) leave, bit for bit, what the prompt in pieces of up to 32 rows leaves, whose GEMMs have a tile per wave."""
import dataclasses

import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {f"d{d}": dataclasses.replace(synth.LLAMA_7B, n_layers=2, d_model=d, n_heads=d // 128, d_ffn=ffn, vocab=1024)
          for d, ffn in ((3072, 8192), (4096, 11008), (5120, 13824), (6144, 16384))}
# shape, rows behind 21 others (the first row group is partly theirs) -> the forms in question that 256 compute units give: QKV,
# residual (O and down) or gate / up, and weight fragments per wave, of both kinds of block in the mixed one (asserted without a GPU)
CASES = {
    ("d4096", 100): {"narrow residual 2", "narrow gate_up 3"}, ("d4096", 123): {"narrow residual 2", "narrow gate_up 3"},
    ("d5120", 92): {"narrow qkv 2", "narrow residual 3"}, ("d3072", 120): {"narrow gate_up 2"}, ("d6144", 97): {"narrow qkv 3", "narrow residual 3"},
    ("d4096", 1100): {"mixed gate_up 6 4"}, ("d4096", 1339): {"mixed qkv 6 3"}, ("d5120", 635): {"mixed gate_up 6 3"},
    ("d5120", 890): {"mixed residual 6 3"}, ("d5120", 1230): {"mixed residual 6 4"}, ("d5120", 1595): {"mixed qkv 6 4"},
}
BEFORE = 21


def pieces(n):
    """The rows from BEFORE on in two row groups at a time."""
    at = [BEFORE, *range(32, n, 32), n]
    return list(zip(at, at[1:]))


@pytest.fixture(scope="module")
def models():
    made = {}

    def get(name):
        if name not in made:
            made.clear()
            made[name] = B.Model(SHAPES[name], synth.make_weights(SHAPES[name], 5, device="cuda"), max_window=8, max_positions=1700)
        return made[name]
    yield get
    made.clear()


@pytest.mark.parametrize("name,rows", sorted(CASES), ids=lambda x: str(x))
def test_wide_models_forms_give_the_bits_of_a_tile_per_wave(models, name, rows):
    model, shape = models(name), SHAPES[name]
    n = BEFORE + rows
    prompt = synth.random_tokens(shape.vocab, n, 11)
    one, cut = B.KVCache(model, n), B.KVCache(model, n)
    a = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    for kv in (one, cut):
        B.prefill(model, kv, prompt[:BEFORE])
    t0 = B.prefill(model, one, prompt[BEFORE:], out_logits=a)
    t1 = -1
    for lo, hi in pieces(n):
        t1 = B.prefill(model, cut, prompt[lo:hi], out_logits=b)
    assert t0 == t1 and torch.equal(a, b)
    for layer in range(shape.n_layers):
        for x, y in zip(one.read(layer, 0, n), cut.read(layer, 0, n)):
            assert torch.equal(x, y), layer
