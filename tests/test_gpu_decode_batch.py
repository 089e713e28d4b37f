"""Plain decoding of many sequences in one step: bit for bit the sequences verified alone, at the ends of pages, of splits
and of the eight one-page splits, and where the rule for the many-sequences attention kernel does not hold."""
import pytest
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

pytestmark = pytest.mark.gpu

MHA = synth.ModelShape(2, 2048, 32, 64, 512, 1024, "bf16")
GQA = synth.ModelShape(2, 4096, 32, 128, 512, 1024, "bf16", n_kv_heads=4)
MHA128 = synth.ModelShape(1, 4096, 32, 128, 512, 1024, "bf16")

# cached tokens of batches that the rule gives to the many-sequences kernel on 256 compute units, in both steps of _run
# (test_host_path.py holds the rule to that): within the eight one-page splits, and beyond, where a wave goes through
# three pages per split, up to the last of the sixteen splits
SHORT = [0, 1, 15, 16, 17, 112, 127, 128, 129, 255, 300, 511, 512, 640, 700, 895, 896, 1000, 1022, 33, 897, 903, 1007, 1021]
LONG = [1023, 1024, 1025, 1151, 1152, 1153, 1279, 1280, 1281, 1407, 1408, 1409, 5, 1791, 1792, 2000, 2175, 2176, 2560, 3000, 3327, 3328,
        3711, 3712, 4093, 4094, 77]
DECODE = [(MHA, SHORT), (MHA128, SHORT), (GQA, SHORT), (MHA, LONG), (GQA, LONG)]


def _run(shape, lengths, max_positions, rows=1):
    w = synth.make_weights(shape, 3, device="cuda")
    model = B.Model(shape, w, max_window=32, max_positions=max_positions)
    n = len(lengths)
    joint, alone = [], []
    for i, length in enumerate(lengths):
        pair = []
        for _ in range(2):
            kv = B.KVCache(model, length + 2 * rows + 6)
            kv.set_page_order([(j * 7 + i) % kv.num_pages for j in range(kv.num_pages)] if kv.num_pages % 7 else list(range(kv.num_pages)))
            for layer in range(shape.n_layers):
                if length:
                    k, v = synth.kv_fill(shape, 100 + i, layer, length, device="cuda")
                    kv.write(layer, 0, k.float().contiguous(), v.float().contiguous())
            kv.truncate(length)
            pair.append(kv)
        joint.append(pair[0])
        alone.append(pair[1])
    for step in range(2):
        wins = [synth.random_tokens(shape.vocab, rows, 31 * step + i) for i in range(n)]
        logits = torch.empty(n * rows, shape.vocab, dtype=torch.float32, device="cuda")
        got = B.verify_batch(model, joint, wins, out_logits=logits)
        for i in range(n):
            row = torch.empty(rows, shape.vocab, dtype=torch.float32, device="cuda")
            assert B.verify(model, alone[i], wins[i], out_logits=row) == got[i], (step, i)
            assert torch.equal(row, logits[i * rows:(i + 1) * rows]), (step, i, lengths[i])


@pytest.mark.parametrize("shape,lengths", DECODE, ids=["dh64-short", "dh128-short", "dh128_gqa-short", "dh64-long", "dh128_gqa-long"])
def test_sequences_of_one_row(shape, lengths):
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256    # (or the rule may choose the other kernel)
    _run(shape, lengths, 4200)


def test_sequences_past_the_kernels_splits_too_few_and_uneven_ones():
    _run(GQA, [4100, 20, 30, 40, 50, 60, 70, 80, 90, 100, 110, 120, 130, 140, 150, 160], 4200)
    _run(MHA, [100, 200, 300, 400, 500, 600, 700, 800, 900], 1100)
    _run(GQA, [100] * 31 + [4000], 4200)    # (one long sequence outweighs the others)


# batches whose keys and values are more than 384 MiB, so that they are loaded as a stream (test_host_path.py holds the rule to that), in each
# form of the attention kernels: one block per (head, sequence), or cut into splits, of one page per wave and of more
@pytest.mark.parametrize("dh,layers,lengths,rows", [
    (64, 4, [1007 - 3 * i for i in range(32)], 1), (128, 2, [1300 + 7 * i for i in range(24)], 1),
    (64, 4, [1000 - 5 * i for i in range(16)], 2), (64, 4, [1640 + i for i in range(8)], 4),
    (128, 4, [1000 - i for i in range(8)], 4), (128, 2, [1700 + 3 * i for i in range(16)], 2),
])
def test_keys_and_values_as_a_stream(dh, layers, lengths, rows):
    shape = synth.ModelShape(layers, 32 * dh, 32, dh, 512, 1024, "bf16")
    assert 4 * layers * shape.d_model * sum(n + rows for n in lengths) > 384 << 20
    _run(shape, lengths, 2100, rows)
