"""The one-kernel step, asked for by name (left to itself a small model takes separate launches): its forms - windows of up to 16 rows,
draft trees and several sequences of up to 8 - leave, bit for bit, what the separate launches leave; and what AUTO takes, and that it
leaves the same."""
import dataclasses

import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth
from helpers import ran_as_one_kernel

pytestmark = pytest.mark.gpu

SHAPES = {"tiny": synth.TINY_BF16, "tiny_grouped": synth.TINY_MQA_BF16, "mid": synth.MID_BF16, "mid_grouped": synth.MID_GQA,
          "d1984": dataclasses.replace(synth.TINY_BF16, d_model=1984, n_heads=31, d_ffn=2048),
          # the widths whose windows of 9 rows and more AUTO runs as one kernel, and as launches
          "d4096_grouped": synth.ModelShape(2, 4096, 32, 128, 13696, 1024, "bf16", n_kv_heads=2), "d4096": synth.ModelShape(2, 4096, 32, 128, 11008, 1024, "bf16")}
LENGTHS = [0, 21, 130, 1030]     # nothing cached, a piece of a page, two splits, one of several pages


def taken(shape, path, rows, positions):
    """Whether such a step runs as one kernel."""
    if path != B.GEMM_AUTO:
        return path == B.GEMM_MFMA
    return shape.d_model >= 2048 and (rows <= 8 or (shape.d_model > 3072 and shape.kv_heads < shape.n_heads and positions <= 1024))


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_one_kernel_and_separate_launches(name):
    shape = SHAPES[name]
    w = synth.make_weights(shape, 5, device="cuda")
    tokens = synth.random_tokens(shape.vocab, 1100, 17)
    seen = {}
    for path in (B.GEMM_MFMA, B.GEMM_MFMA_LAUNCHES, B.GEMM_AUTO):
        model = B.Model(shape, w, max_window=16, max_positions=1100, gemm_path=path)
        out = seen[path] = []
        kvs = [B.KVCache(model, 1100) for _ in range(3)]

        def step(rows, length, call):
            logits = torch.zeros(rows, shape.vocab, dtype=torch.float32, device="cuda")
            model.profile(True)      # (from zero: prompts have no part in the one kernel)
            done = call(logits)
            assert ran_as_one_kernel(model) == taken(shape, path, rows, length + rows), (path, rows, length)
            out.append((logits, done, [kv.read(layer, 0, kv.length) for kv in kvs for layer in range(shape.n_layers) if kv.length]))

        for length in LENGTHS:
            for kv in kvs:
                kv.truncate(0)
                if length:
                    B.prefill(model, kv, tokens[:length])
            for rows in (1, 7, 8, 9, 12, 16):
                kvs[0].truncate(length)
                step(rows, length, lambda logits: B.verify(model, kvs[0], tokens[length:length + rows], B.VERIFY, out_logits=logits))
            for parents in ([-1, 0, 0, 1, 2, 3], [-1, 0, 1, 2, 0, 4, 5, 0]):
                kvs[0].truncate(length)
                step(len(parents), length, lambda logits: B.verify_tree(model, kvs[0], tokens[length:length + len(parents)], parents, out_logits=logits))
            for windows in ([1, 1], [2, 5, 1]):
                for kv in kvs:
                    kv.truncate(length)
                step(sum(windows), length, lambda logits: B.verify_batch(model, kvs[:len(windows)], [tokens[length + i:length + i + n] for i, n in enumerate(windows)],
                                                                         out_logits=logits))
        del model
    for path in (B.GEMM_MFMA, B.GEMM_AUTO):
        for (la, da, ka), (lb, db, kb) in zip(seen[path], seen[B.GEMM_MFMA_LAUNCHES]):
            assert torch.equal(la, lb) and da == db
            for x, y in zip(ka, kb):
                assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])


# d 2048 and more: one kernel up to 8 rows; above, only with grouped heads at d above 3072 and up to 1024 positions
@pytest.mark.parametrize("d,heads,kv_heads,length,rows,expected", [
    (2048, 16, 0, 40, 8, True), (2048, 16, 0, 40, 9, False), (4096, 32, 2, 40, 9, True), (4096, 32, 2, 1008, 16, True), (4096, 32, 2, 1009, 16, False),
    (4096, 32, 0, 40, 16, False), (3072, 24, 2, 40, 9, False)])
def test_what_a_wide_model_takes(d, heads, kv_heads, length, rows, expected):
    shape = synth.ModelShape(1, d, heads, 128, 2048, 1024, "bf16", n_kv_heads=kv_heads)
    model = B.Model(shape, synth.make_weights(shape, 5, device="cuda"), max_window=16, max_positions=1100)
    kv = B.KVCache(model, 1100)
    tokens = synth.random_tokens(shape.vocab, length + rows, 3)
    B.prefill(model, kv, tokens[:length])
    model.profile(True)
    B.verify(model, kv, tokens[length:])
    assert ran_as_one_kernel(model) == expected
