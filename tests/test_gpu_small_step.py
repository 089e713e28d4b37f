"""A small fp32 model's step in one launch leaves, bit for bit, what the separate launches leave: logits, results, cache."""
import dataclasses

import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

T = synth.TINY
SHAPES = {
    "tiny": T, "one_layer": dataclasses.replace(T, n_layers=1), "grouped": synth.TINY_MQA,
    # K of half a round of the eight waves, and of two and three rounds; no tile of the feed-forward layer left over, one
    "d128": dataclasses.replace(T, n_layers=3, d_model=128, n_heads=2, d_ffn=512, vocab=512),
    "d320": dataclasses.replace(T, d_model=320, n_heads=5, d_ffn=512, vocab=528),
    "head128": dataclasses.replace(T, d_model=256, n_heads=2, head_dim=128, d_ffn=528),
}


@pytest.fixture(scope="module")
def pairs():
    made = {}

    def get(name):
        if name not in made:
            made.clear()
            w = synth.make_weights(SHAPES[name], 6, device="cuda")
            made[name] = [B.Model(SHAPES[name], w, max_window=32, max_positions=600, gemm_path=p) for p in (B.GEMM_AUTO, B.GEMM_DOT)]
        return made[name]
    yield get
    made.clear()


def one_launch(model):
    p = model.profile_read()
    return p["steps"] == p["intervals"]["step"] > 0


# key splits (of 64): one, up to four, which O's blocks merge, five and eight; the window's rows on either side of a split; row
# tiles of one and two.  Repeated: flags and counters of the launch before are there.
@pytest.mark.parametrize("name", sorted(SHAPES))
@pytest.mark.parametrize("length,rows", [(0, 1), (59, 5), (60, 5), (128, 16), (128, 17), (200, 32), (239, 17), (251, 5), (252, 5), (300, 1), (496, 16)])
def test_a_step_has_the_bits_of_separate_launches(pairs, name, length, rows):
    shape = SHAPES[name]
    tokens = synth.random_tokens(shape.vocab, length + rows, 21)
    seen = []
    for model in pairs(name):
        kv = B.KVCache(model, length + rows)
        if length:
            B.prefill(model, kv, tokens[:length])
        runs = []
        model.profile(True)
        for mode in (B.VERIFY, B.APPEND, B.APPEND):
            kv.truncate(length)
            logits = torch.zeros(rows, shape.vocab, dtype=torch.float32, device="cuda")
            done = B.verify(model, kv, tokens[length:], mode, out_logits=logits)
            runs.append((logits, done, kv.length, [kv.read(layer, 0, kv.length) for layer in range(shape.n_layers)]))
        seen.append((runs, one_launch(model)))
        model.profile(False)
    assert seen[0][1] and not seen[1][1]
    for (la, da, na, ka), (lb, db, nb, kb) in zip(seen[0][0], seen[1][0]):
        assert torch.equal(la, lb) and da == db and na == nb
        for x, y in zip(ka, kb):
            assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])


# a tree whose accepted path (what the model itself says, as second child of every row) has to be moved in the cache; a short prompt
def test_trees_and_short_prompts(pairs):
    shape, length = SHAPES["tiny"], 70
    tokens = synth.random_tokens(shape.vocab, length + 1, 22)
    seen = []
    for model in pairs("tiny"):
        kv = B.KVCache(model, 200)
        first = B.prefill(model, kv, tokens[:30])
        B.prefill(model, kv, tokens[30:length])
        window, parents = [tokens[length]], [-1]
        chain = [tokens[length]]
        for _ in range(3):
            kv.truncate(length)
            chain.append(B.verify(model, kv, chain, B.APPEND)[1])
        at = 0
        for t in chain[1:]:
            window += [(t + 1) % shape.vocab, t]
            parents += [at, at]
            at = len(window) - 1
        kv.truncate(length)
        logits = torch.zeros(len(window), shape.vocab, dtype=torch.float32, device="cuda")
        done = B.verify_tree(model, kv, window, parents, out_logits=logits)
        assert done[0] == 3
        seen.append((first, done, logits, kv.length, [kv.read(layer, 0, kv.length) for layer in range(shape.n_layers)]))
    a, b = seen
    assert a[0] == b[0] and a[1] == b[1] and torch.equal(a[2], b[2]) and a[3] == b[3] == length + 4
    for x, y in zip(a[4], b[4]):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])


# logits between weights, sharing their first and last line with them (a caller that packs its buffers to 64 bytes): the predictions are
# those of the logits that are there, also where a block that looks for them has read those weights before
def test_logits_that_share_lines_with_weights(pairs):
    shape, rows = SHAPES["tiny"], 5
    w = {k: list(v) if isinstance(v, list) else v for k, v in pairs("tiny")[0].weights.items()}
    n_lm, n_out, d = w["lm_head"].numel(), rows * shape.vocab, shape.d_model
    arena = torch.zeros(n_lm + n_out + d + 64, dtype=torch.float32, device="cuda")
    base = (-arena.data_ptr() // 4) % 32 + 16       # half a line of 128 bytes
    lm, out, norm = arena[base:base + n_lm], arena[base + n_lm:base + n_lm + n_out], arena[base + n_lm + n_out:base + n_lm + n_out + d]
    lm.copy_(w["lm_head"].flatten())
    norm.copy_(w["final_norm"])
    lm, out = lm.view(shape.vocab, d), out.view(rows, shape.vocab)
    assert out.data_ptr() % 128 == 64 and norm.data_ptr() % 128 == 64
    lm[0] *= 20.0        # one of these is the largest logit of nearly every row
    lm[-1] *= 20.0
    w["lm_head"], w["final_norm"] = lm, norm
    model = B.Model(shape, w, max_window=8, max_positions=64)
    kv = B.KVCache(model, 64)
    model.profile(True)
    seen = set()
    for i in range(400):
        kv.truncate(20)
        _, _, preds = B.verify(model, kv, synth.random_tokens(shape.vocab, rows, 1000 + i), B.APPEND, want_predicts=True, out_logits=out)
        assert preds == out.argmax(1).tolist(), i
        seen |= set(preds)
    assert one_launch(model) and {0, shape.vocab - 1} <= seen


# A wait inside the launch gives up at once (its limit is set from the host; all items are still worked off, in order): the call says so, and
# the next one, in one launch again, has the bits of a fresh step.  Keys of two splits, merged by O's blocks, and of five, merged by the
# last of attention's.
@pytest.mark.parametrize("length", [70, 300])
@pytest.mark.parametrize("what", ["window", "tree", "prompt"])
def test_a_wait_that_gives_up_is_reported_and_the_next_step_is_correct(pairs, what, length):
    shape, model = SHAPES["tiny"], pairs("tiny")[0]
    rows = 16 if what == "prompt" else 7
    tokens = synth.random_tokens(shape.vocab, length + rows, 23)
    kv = B.KVCache(model, length + rows)
    B.prefill(model, kv, tokens[:length])
    logits = torch.zeros(1 if what == "prompt" else rows, shape.vocab, dtype=torch.float32, device="cuda")

    def call():
        if what == "window":
            return B.verify(model, kv, tokens[length:], B.APPEND, want_predicts=True, out_logits=logits)
        if what == "tree":
            return B.verify_tree(model, kv, tokens[length:], [-1, 0, 1, 0, 3, 4, 0], want_predicts=True, out_logits=logits)
        return B.prefill(model, kv, tokens[length:], out_logits=logits[0])

    def fresh():
        logits.zero_()
        model.profile(True)
        done = call()
        assert one_launch(model)
        kept = done, logits.clone(), kv.length, [kv.read(layer, 0, kv.length) for layer in range(shape.n_layers)]
        kv.truncate(length)
        return kept

    want = fresh()
    for _ in range(3):
        model.set_barrier_spin_limit(1)
        try:
            with pytest.raises(B.AnpdError) as e:
                call()
        finally:
            model.set_barrier_spin_limit(0)
        assert e.value.code == B.E_HIP and kv.length == length
        kv.truncate(length)
        for _ in range(2):
            got = fresh()
            assert got[0] == want[0] and torch.equal(got[1], want[1]) and got[2] == want[2]
            for x, y in zip(got[3], want[3]):
                assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])
