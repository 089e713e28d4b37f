"""The library's host code on a stand-in for the HIP runtime (hip_stub.cpp: kernels are written down, not run): which
calls it makes, with what, and what it leaves behind when one of them fails.  Each test is a process of its own."""
import ctypes as C
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CHILD = os.environ.get("ANPD_HIP_STUB")     # set in the test's own process: the built stand-in


@pytest.fixture(scope="session")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", out], check=True)
    return out


def in_child(stub, name, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), name, *map(str, args)], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ANPD_HIP_STUB=stub, PYTHONPATH=os.path.dirname(HERE)))
    assert r.returncode == 0, r.stdout + r.stderr


# ------------------------------------------------------------------------------------------- in the child

class Host:
    """The library on the stand-in, with a one-layer model and caches in host memory."""

    def __init__(self, d=256, heads=4, dh=64, ffn=256, vocab=512, dtype="bf16", kv_heads=0, path=0, max_window=32, max_positions=256, layers=1):
        sys.modules["torch"] = None           # (it would bring a HIP runtime of its own)
        self.stub = C.CDLL(CHILD, mode=C.RTLD_GLOBAL)
        self.stub.stub_name.restype = C.c_char_p
        self.stub.stub_arg0.restype = C.c_void_p
        self.stub.stub_arg0.argtypes = [C.c_int]
        self.stub.stub_memory.argtypes = [C.c_void_p, C.c_size_t, C.c_int]
        from paper_2404_08698_amd import binding as B
        self.B, self.L, self.keep, self.length_at = B, B.lib(), [], {}
        cfg = B.ModelCfg(layers, d, heads, dh, ffn, vocab, 1e-5, 10000.0, B.BF16 if dtype == "bf16" else B.F32, 16, max_window,
                         max_positions, path, kv_heads)
        w = B.Weights()
        dummy = self.memory(4096)
        for name in ("embed", "final_norm", "lm_head"):
            setattr(w, name, dummy)
        for name in B._PER_LAYER:
            arr = (C.c_void_p * layers)(*[dummy] * layers)
            self.keep.append(arr)
            setattr(w, name, C.cast(arr, C.POINTER(C.c_void_p)))
        n = self.L.anpd_model_workspace_bytes(C.byref(cfg))
        self.ws, self.ws_bytes, self.model, self.vocab = self.memory(n), n, C.c_void_p(), vocab
        self.ok(self.L.anpd_model_create(C.byref(cfg), C.byref(w), self.ws, n, None, C.byref(self.model)))

    def memory(self, n, device=0, offset=0):
        """Address of n bytes of "device" memory, 256-byte aligned plus offset; exactly those are known as such."""
        buf = C.create_string_buffer(n + 512 + offset)
        self.keep.append(buf)
        at = (C.addressof(buf) + 255) // 256 * 256
        self.stub.stub_memory(at, n + offset, device)
        return at + offset

    def ok(self, rc):
        assert rc >= 0, (rc, self.L.anpd_last_error())

    def cache(self, max_tokens, length=0):
        n = self.L.anpd_kv_pool_bytes(self.model, max_tokens)
        kv, pool = C.c_void_p(), self.memory(n)
        self.ok(self.L.anpd_kv_create(self.model, pool, n, max_tokens, C.byref(kv)))
        self.ok(self.L.anpd_kv_truncate(kv, length, None))
        # the length lies behind the pages, which end at a multiple of 256 bytes; so does the page table behind it
        pages = self.L.anpd_kv_num_pages(kv)
        self.length_at[kv.value] = pool + n - ((pages + 1) * 4 + 255) // 256 * 256
        return kv

    def names(self):
        return [self.stub.stub_name(i).decode() for i in range(self.stub.stub_launches())]

    def logits_of_argmax(self):
        """Where the last argmax kernel reads the logits, that is, where the LM head wrote them."""
        at = [i for i, n in enumerate(self.names()) if "argmax_accept" in n][-1]
        return self.stub.stub_arg0(at)

    def verify(self, kv, n, out):
        acc, nxt = C.c_int32(), C.c_int32()
        return self.L.anpd_verify(self.model, kv, (C.c_int32 * n)(*range(n)), n, self.B.APPEND, C.byref(acc), C.byref(nxt), None, out, None)

    def verify_tree(self, kv, n, out):
        acc, nxt, row = C.c_int32(), C.c_int32(), C.c_int32 * n
        return self.L.anpd_verify_tree(self.model, kv, row(*range(n)), row(-1, *[i // 2 for i in range(n - 1)]), n, C.byref(acc), C.byref(nxt),
                                       None, None, out, None)

    def prefill(self, kv, n, out=None):
        nxt = C.c_int32()
        nb = self.L.anpd_prefill_workspace_bytes(self.model, n)
        return self.L.anpd_prefill(self.model, kv, (C.c_int32 * n)(*[i % self.vocab for i in range(n)]), n, C.byref(nxt), out,
                                   self.memory(nb) if nb else None, nb, None)


def child_logits(dtype, path):
    h = Host(dtype=dtype, path=int(path))
    kv = h.cache(256)
    own = lambda p: h.ws <= p < h.ws + h.ws_bytes
    for call, rows, size in ((lambda out: h.verify(kv, 20, out), 20, 20 * 512 * 4), (lambda out: h.prefill(kv, 33, out), 1, 512 * 4)):
        h.ok(h.L.anpd_kv_truncate(kv, 0, None))
        direct = h.memory(size)
        h.ok(call(direct))
        assert h.logits_of_argmax() == direct
        for other in (h.memory(size, offset=4), h.memory(size, device=1)):    # not for wide stores; another GPU's
            h.ok(h.L.anpd_kv_truncate(kv, 0, None))
            h.ok(call(other))
            assert own(h.logits_of_argmax())
        # memory that ends before the logits do: nothing may be written past its end, the copy says so
        h.ok(h.L.anpd_kv_truncate(kv, 0, None))
        assert call(h.memory(size - 4)) == h.B.E_HIP
        assert own(h.logits_of_argmax())
        h.stub.hipGetLastError()    # (the copy's error, which stays until it is read)


@pytest.mark.parametrize("dtype,path", [("bf16", 4), ("bf16", 1), ("f32", 0)])
def test_logits_go_straight_to_a_buffer_that_holds_them_only(stub, dtype, path):
    in_child(stub, "child_logits", dtype, path)


def child_failing_prompt(dtype, path, max_window):
    """Every launch of a prompt of three pieces fails once; the copy of its logits fails, too."""
    h = Host(dtype=dtype, path=int(path), max_window=int(max_window), max_positions=700)
    kv = h.cache(700, 20)
    d_len = C.c_int32.from_address(h.length_at[kv.value])

    def unchanged():
        h.stub.hipGetLastError()
        assert h.L.anpd_kv_length(kv) == 20 and d_len.value == 20
    h.stub.stub_forget()
    h.ok(h.prefill(kv, 600))
    launches = h.stub.stub_launches()
    # pieces of 256, 256 and 88 rows, whatever the window; 32 tokens per launch of the embedding
    assert sum("advance_length" in n for n in h.names()) == 2 and h.L.anpd_kv_length(kv) == 620
    assert sum("embed_kernel" in n for n in h.names()) == 8 + 8 + 3
    for nth in range(1, launches + 1):
        h.ok(h.L.anpd_kv_truncate(kv, 20, None))
        d_len.value = 276       # as the first piece leaves it (the stand-in runs no kernel)
        h.stub.stub_fail_launch(nth)
        assert h.prefill(kv, 600) == h.B.E_HIP
        unchanged()
    d_len.value = 620
    assert h.prefill(kv, 600, h.memory(512 * 4 - 4)) == h.B.E_HIP
    unchanged()
    h.ok(h.prefill(kv, 600))
    assert h.L.anpd_kv_length(kv) == 620


@pytest.mark.parametrize("dtype,path,max_window", [("f32", 0, 16), ("f32", 0, 1), ("bf16", 1, 16)])
def test_a_prompt_in_pieces_that_fails_half_way_leaves_the_cache_as_it_was(stub, dtype, path, max_window):
    in_child(stub, "child_failing_prompt", dtype, path, max_window)


def child_failing_launch(dtype, path):
    """Every launch of a step and of a prompt fails once while the logits go to memory that the runtime does not know (the query of
    it fails, too, and leaves an error of its own): the call says so."""
    h = Host(dtype=dtype, path=int(path))
    kv = h.cache(256)
    unknown = C.create_string_buffer(20 * 512 * 4 + 16)
    out = (C.addressof(unknown) + 15) // 16 * 16
    for call in (lambda: h.verify(kv, 20, out), lambda: h.prefill(kv, 33, out)):
        h.stub.stub_forget()
        h.ok(call())
        for nth in range(1, h.stub.stub_launches() + 1):
            h.ok(h.L.anpd_kv_truncate(kv, 0, None))
            h.stub.hipGetLastError()
            h.stub.stub_fail_launch(nth)
            assert call() == h.B.E_HIP, (nth, h.names())
        h.stub.hipGetLastError()
        h.ok(h.L.anpd_kv_truncate(kv, 0, None))


@pytest.mark.parametrize("dtype,path", [("bf16", 4), ("bf16", 1), ("f32", 0)])
def test_a_launch_that_fails_in_front_of_the_lookup_of_the_logits_buffer_is_reported(stub, dtype, path):
    in_child(stub, "child_failing_launch", dtype, path)


def child_tile_blocks():
    """A tile per wave: up to four tiles per block every compute unit gets one, as long as there are tiles (257 tiles were 129 blocks of
    two), from five on the blocks are full; a wave that is alone on its compute unit has a longer ring if K fills it."""
    h = Host()
    blocks = {1: 1, 3: 3, 255: 255, 256: 256, 257: 256, 300: 256, 512: 256, 513: 256, 960: 256, 1024: 256, 1025: 205, 1376: 230, 1791: 256, 1792: 256}
    x, w, y, ws = (h.memory(n) for n in (4096, 4096, 4096, 1 << 18))
    for rows, k in ((9, 64), (17, 64), (17, 992), (17, 1000), (32, 1024)):
        for n in blocks:
            if rows <= 16 and n <= 256:     # (another kernel's)
                continue
            h.stub.stub_forget()
            h.ok(h.L.anpd_linear(x, w, y, rows, 16 * n, k, h.B.BF16, h.B.GEMM_MFMA, ws, 1 << 18, None))
            at = [i for i, name in enumerate(h.names()) if "gemm_tile_kernel" in name]
            assert len(at) == 1 and h.stub.stub_blocks(at[0]) == blocks[n], (rows, n, h.names())
            assert ("gemm_tile_kernelILi4ELi1E" in h.names()[at[0]]) == (n <= 256 and k > 992), (rows, n, k)


def test_tiles_of_a_wide_window_are_spread_over_the_compute_units(stub):
    in_child(stub, "child_tile_blocks")


def child_prompt_attention(heads, dh, length, rows, shared):
    h = Host(d=int(heads) * int(dh), heads=int(heads), dh=int(dh), max_positions=4200, layers=2)
    kv = h.cache(4200, int(length))
    h.stub.stub_forget()
    h.ok(h.prefill(kv, int(rows)))
    first, last = [n for n in h.names() if "prefill_attn_kernel" in n]
    assert f"prefill_attn_kernelILi{dh}ELb{shared}E" in first, h.names()
    assert f"prefill_attn_kernelILi{dh}ELb0E" in last, h.names()     # (one row group)


# blocks: heads x pairs of row groups; up to one per compute unit, two at head dim 64, have their query rows in registers
@pytest.mark.parametrize("heads,dh,length,rows,shared", [
    (32, 128, 0, 1, 0), (32, 128, 0, 256, 0), (32, 128, 0, 257, 1), (32, 128, 15, 241, 0), (32, 128, 15, 242, 1), (40, 128, 777, 182, 0),
    (40, 128, 777, 205, 1), (4, 64, 0, 4096, 0), (4, 64, 0, 4097, 1),
])
def test_query_rows_of_a_prompt_lie_where_its_blocks_gain_by_it(stub, heads, dh, length, rows, shared):
    in_child(stub, "child_prompt_attention", heads, dh, length, rows, shared)


def child_last_layer(dtype, layers, rows):
    """Blocks of attention in each layer of a prompt: all row groups, in the last layer one."""
    h = Host(dtype=dtype, layers=int(layers), max_positions=400)
    kv = h.cache(400)
    h.stub.stub_forget()
    h.ok(h.prefill(kv, int(rows)))
    blocks = [h.stub.stub_blocks(i) for i, n in enumerate(h.names()) if "attn_kernel" in n]
    groups, splits = -(-int(rows) // 16), -(-int(rows) // 64)
    whole, last = (4 * -(-groups // 2), 4) if dtype == "bf16" else (4 * splits * groups, 4 * splits)
    assert blocks == [whole] * (int(layers) - 1) + [last], blocks


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layers", [1, 2, 3])
def test_a_prompt_leaves_the_last_layer_with_one_row_group(stub, dtype, layers):
    in_child(stub, "child_last_layer", dtype, layers, 200)


def child_prompt_forms(heads, ffn, before, rows, expected, cuts):
    import re
    h = Host(d=128 * int(heads), heads=int(heads), dh=128, ffn=int(ffn), vocab=1024, max_positions=1700, layers=2)
    kv = h.cache(1700)
    epilogue = {"1": "qkv", "2": "residual", "3": "gate_up"}

    def forms(lo, hi):
        h.ok(h.L.anpd_kv_truncate(kv, lo, None))
        h.stub.stub_forget()
        h.ok(h.prefill(kv, hi - lo))
        found = [m for m in (re.search(r"prefill_(gemm|narrow|mixed|few)_kernelILi(\d)E((?:Li\d+E)*)", k) for k in h.names()) if m]
        layer2 = [i for i, m in enumerate(found) if epilogue[m[2]] == "qkv"][1]      # (the last one: a row group alone behind its keys and values)
        return {" ".join((m[1], epilogue[m[2]], *re.findall(r"\d+", m[3]))) for m in found[:layer2]}
    whole = forms(int(before), int(before) + int(rows))
    assert {f for f in whole if f.startswith(("narrow", "mixed"))} == set(expected.split(",")), whole
    cuts = [int(x) for x in cuts.split(",")]
    for lo, hi in zip(cuts, cuts[1:]):
        assert all(f.startswith("few") for f in forms(lo, hi)), (lo, hi)


def test_prompts_of_wide_models_take_the_forms_they_are_tested_for(stub):
    """In one piece the forms that the GPU test of wide models lists, in its pieces none of them."""
    import test_gpu_prefill_forms as G
    for (name, rows), expected in G.CASES.items():
        shape = G.SHAPES[name]
        cuts = G.pieces(G.BEFORE + rows)
        in_child(stub, "child_prompt_forms", shape.n_heads, shape.d_ffn, G.BEFORE, rows, ",".join(sorted(expected)),
                 ",".join(str(lo) for lo, _ in cuts) + f",{cuts[-1][1]}")


def child_route(lengths, heads, kv_heads, dh, expected, rows=1, layers=1, stream=""):
    lengths, heads, dh, rows, layers = [int(x) for x in lengths.split(",")], int(heads), int(dh), int(rows), int(layers)
    h = Host(d=heads * dh, heads=heads, dh=dh, kv_heads=int(kv_heads), max_positions=4200, layers=layers)
    n = len(lengths)
    kvs = [h.cache(x + 8, x) for x in lengths]
    one = C.POINTER(C.c_int32)
    windows = [(C.c_int32 * rows)(*range(i, i + rows)) for i in range(n)]
    h.stub.stub_forget()
    h.ok(h.L.anpd_verify_batch(h.model, (C.c_void_p * n)(*kvs), n, (one * n)(*[C.cast(r, one) for r in windows]), (C.c_int32 * n)(*[rows] * n),
                               h.B.VERIFY, (C.c_int32 * n)(), (C.c_int32 * n)(), None, None))
    taken = {k for k in ("attn_decode", "attn_batch", "verify_mega") if any(k in name for name in h.names())}
    assert taken == {expected}, taken
    if stream:   # the kernels' last argument: whether keys and values are loaded as a stream
        assert all(f"Lb{stream}EEE" in name for name in h.names() if expected in name), [k for k in h.names() if expected in k]


# heads, key / value heads, cached tokens: enough blocks, too few, one long sequence among short ones, in between
@pytest.mark.parametrize("heads,kv_heads,lengths,route", [
    (32, 32, [500] * 16, "attn_decode"), (32, 32, [500] * 15, "attn_batch"), (40, 40, [500] * 13, "attn_decode"),
    (32, 32, [1023] * 32, "attn_decode"), (32, 4, [2500] * 24, "attn_decode"), (32, 4, [2500] * 23, "attn_batch"),
    (32, 4, [4095] * 24, "attn_decode"), (32, 4, [4095] * 23 + [4096], "attn_batch"), (32, 32, [500] * 8, "verify_mega"),
    (32, 32, [100] * 31 + [4000], "attn_batch"), (32, 32, [100] * 31 + [1000], "attn_batch"), (32, 4, [100] * 31 + [4000], "attn_batch"),
    (32, 32, [100] * 9 + [1000] * 9, "attn_batch"), (32, 32, [100] * 24 + [1000] * 8, "attn_decode"),
    (32, 4, [100] * 24 + [3000] * 8, "attn_decode"), (32, 32, [307 + 13 * i for i in range(32)], "attn_decode"),
])
def test_attention_kernel_of_a_batch_of_one_row_windows(stub, heads, kv_heads, lengths, route):
    in_child(stub, "child_route", ",".join(map(str, lengths)), heads, kv_heads, 64, route)


def test_the_batches_meant_for_the_many_sequences_kernel_take_it(stub):
    import test_gpu_decode_batch as G
    for shape, lengths in G.DECODE:
        for step in (0, 1):
            in_child(stub, "child_route", ",".join(str(x + step) for x in lengths), shape.n_heads, shape.kv_heads, shape.head_dim, "attn_decode")


# keys and values of a step in all its layers, bytes: up to 384 MiB (what the memory-side cache may keep until the next step) ordinary loads,
# beyond a stream; with grouped heads, where several blocks read a page, ordinary loads whatever they are
@pytest.mark.parametrize("heads,kv_heads,dh,layers,lengths,rows,route,stream", [
    (32, 32, 64, 1, [1535] * 32, 1, "attn_decode", 0), (32, 32, 64, 1, [1535] * 31 + [1536], 1, "attn_decode", 1),
    (32, 32, 64, 4, [383] * 32, 1, "attn_decode", 0), (32, 32, 64, 4, [383] * 31 + [384], 1, "attn_decode", 1),
    (16, 16, 128, 3, [1022] * 16, 2, "attn_batch", 0), (16, 16, 128, 3, [1022] * 15 + [1023], 2, "attn_batch", 1),
    (32, 32, 128, 3, [1532] * 8, 4, "attn_batch", 1), (32, 32, 128, 2, [1532] * 8, 4, "attn_batch", 0), (32, 16, 64, 8, [2000] * 32, 1, "attn_decode", 0),
    (32, 16, 64, 8, [2000] * 16, 2, "attn_batch", 0),
])
def test_keys_and_values_of_a_batch_are_a_stream_where_no_cache_keeps_them(stub, heads, kv_heads, dh, layers, lengths, rows, route, stream):
    per_position = 4 * layers * kv_heads * dh
    assert stream == (kv_heads == heads and per_position * sum(n + rows for n in lengths) > 384 << 20)
    in_child(stub, "child_route", ",".join(map(str, lengths)), heads, kv_heads, dh, route, rows, layers, stream)


def child_trace(d, heads, rows):
    """While its barriers are traced a step is the one kernel, also where AUTO takes launches; and none is refused that can be one."""
    d, rows = int(d), int(rows)
    h = Host(d=d, heads=int(heads), dh=d // int(heads), max_positions=128)
    kv, kv2 = h.cache(128, 20), h.cache(128, 30)
    one, half = C.POINTER(C.c_int32), (C.c_int32 * 2)(0, 1)

    def batch():
        return h.L.anpd_verify_batch(h.model, (C.c_void_p * 2)(kv, kv2), 2, (one * 2)(C.cast(half, one), C.cast(half, one)), (C.c_int32 * 2)(2, 2),
                                     h.B.VERIFY, (C.c_int32 * 2)(), (C.c_int32 * 2)(), None, None)
    calls = [lambda: h.verify(kv, rows, None)] + ([lambda: h.verify_tree(kv, rows, None), batch] if rows <= 8 else [])
    grid = h.L.anpd_model_trace(h.model, None, 0)
    assert grid == 256
    buffer = h.memory(grid * 1024 * 8)
    for traced in (0, 1, 0):
        h.ok(h.L.anpd_model_trace(h.model, buffer if traced else None, grid * 1024 * 8 if traced else 0))
        for call in calls:
            h.stub.stub_forget()
            h.ok(call())
            assert ["verify_mega" in n for n in h.names()].count(True) == traced, (traced, h.names())


@pytest.mark.parametrize("d,heads,rows", [(256, 4, 5), (256, 4, 16), (1920, 30, 8), (2048, 16, 9)])
def test_a_traced_step_is_the_one_kernel(stub, d, heads, rows):
    in_child(stub, "child_trace", d, heads, rows)


if __name__ == "__main__":
    globals()[sys.argv[1]](*sys.argv[2:])
