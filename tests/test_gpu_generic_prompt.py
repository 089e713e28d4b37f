"""Prompts of models on the caller's weights: pieces of many rows leave, bit for bit, what windows of a few rows through the
step leave (a row's sums depend on nothing but the row)."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu


# one launch of attention per piece; max_positions of 20000, whose partial results of 256 rows would be more than 16 MiB: launches of
# 48 rows; a window that is no multiple of a row group; 2 and 4 heads per key / value head; prompts of one piece, of two
@pytest.mark.parametrize("shape,path,max_window,max_positions,before,rows", [
    (synth.TINY, B.GEMM_AUTO, 32, 400, 0, 128), (synth.TINY, B.GEMM_AUTO, 5, 400, 37, 300), (synth.TINY, B.GEMM_AUTO, 32, 20000, 11, 270),
    (synth.TINY_MQA, B.GEMM_AUTO, 7, 20000, 63, 65), (synth.MID_BF16, B.GEMM_DOT, 32, 600, 130, 257), (synth.MID_GQA, B.GEMM_DOT, 12, 600, 0, 17),
])
def test_pieces_give_the_bits_of_windows(shape, path, max_window, max_positions, before, rows):
    w = synth.make_weights(shape, 4, device="cuda")
    model = B.Model(shape, w, max_window=max_window, max_positions=max_positions, gemm_path=path)
    capacity = before + rows
    tokens = synth.random_tokens(shape.vocab, capacity, 9)
    whole, parts = B.KVCache(model, capacity), B.KVCache(model, capacity)
    a = torch.empty(shape.vocab, dtype=torch.float32, device="cuda")
    t0 = t1 = None
    if before:
        B.prefill(model, whole, tokens[:before])
    t0 = B.prefill(model, whole, tokens[before:], out_logits=a)
    for lo in range(0, capacity, max_window):
        window = tokens[lo:lo + max_window]
        b = torch.empty(len(window), shape.vocab, dtype=torch.float32, device="cuda")
        _, t1 = B.verify(model, parts, window, B.APPEND, out_logits=b)[:2]
    assert whole.length == parts.length == capacity and t0 == t1 and torch.equal(a, b[-1])
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, capacity), parts.read(layer, 0, capacity)):
            assert torch.equal(x, y)


# a step's first QKV takes its rows from the embedding table in 16-byte loads; a table at another address is copied by a launch
# of its own, one element at a time.  Both give the same bits, at one row group and at two
@pytest.mark.parametrize("shape,path", [(synth.TINY, B.GEMM_AUTO), (synth.MID_BF16, B.GEMM_DOT)])
@pytest.mark.parametrize("rows", [1, 16, 17, 32])
def test_embedding_table_at_any_address(shape, path, rows):
    w = synth.make_weights(shape, 4, device="cuda")
    table = w["embed"]
    moved = torch.empty(table.numel() + 1, dtype=table.dtype, device="cuda")[1:].view_as(table).copy_(table)
    assert table.data_ptr() % 16 == 0 and moved.data_ptr() % 16 == table.element_size()
    tokens = synth.random_tokens(shape.vocab, rows, 9)
    seen = []
    for embed in (table, moved):
        model = B.Model(shape, {**w, "embed": embed}, max_window=32, max_positions=64, gemm_path=path)
        kv = B.KVCache(model, rows)
        logits = torch.empty(rows, shape.vocab, dtype=torch.float32, device="cuda")
        B.verify(model, kv, tokens, B.APPEND, out_logits=logits)
        seen.append((logits, [kv.read(layer, 0, rows) for layer in range(shape.n_layers)]))
    assert torch.equal(seen[0][0], seen[1][0])
    for x, y in zip(seen[0][1], seen[1][1]):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])


# a row whose keys and values are not finite: the first of a row group, inside one, the last of a piece's keys that a wave holds;
# one window of a prompt before it or a whole one in its piece, one launch of attention per piece or several
@pytest.mark.parametrize("shape,path,max_window,max_positions", [(synth.TINY, B.GEMM_AUTO, 5, 400), (synth.TINY, B.GEMM_AUTO, 32, 20000),
                                                                 (synth.MID_GQA, B.GEMM_DOT, 8, 400)])
@pytest.mark.parametrize("at", [1, 16, 40, 47, 63, 64, 90])
def test_a_row_that_is_not_finite_leaves_the_rows_before_it_alone(shape, path, max_window, max_positions, at):
    w = synth.make_weights(shape, 3, device="cuda")
    w["embed"][7] = float("nan")
    model = B.Model(shape, w, max_window=max_window, max_positions=max_positions, gemm_path=path)
    prompt = [t if t != 7 else 8 for t in synth.random_tokens(shape.vocab, 100, 11)]
    whole, before = B.KVCache(model, 128), B.KVCache(model, 128)
    B.prefill(model, whole, prompt[:at] + [7] + prompt[at + 1:])
    B.prefill(model, before, prompt[:at])
    for layer in range(shape.n_layers):
        for x, y in zip(whole.read(layer, 0, at), before.read(layer, 0, at)):
            assert torch.equal(x, y), layer   # (NaN equals nothing)
