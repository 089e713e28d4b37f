"""Host side of a small fp32 model's step in one launch, on the stand-in for the HIP runtime: which calls take it, and what happens
when no block ran on the XCD that it was meant for (on the stand-in none does, unless told to): the step is separate launches, then
and later; and that no error is lost or taken for another's."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_host_path import Host, in_child, stub  # noqa: E402,F401


def run(stub, name, *args, blocks=32, env=()):
    os.environ["STUB_XCD_BLOCKS"] = str(blocks)
    try:
        import subprocess
        r = subprocess.run([sys.executable, os.path.abspath(__file__), name, *map(str, args)], capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, ANPD_HIP_STUB=stub, PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), **dict(env)))
    finally:
        del os.environ["STUB_XCD_BLOCKS"]
    assert r.returncode == 0, r.stdout + r.stderr


def child_route(d, heads, dh, ffn, vocab, path, length, rows, taken, kv_heads=0):
    h = Host(d=int(d), heads=int(heads), dh=int(dh), ffn=int(ffn), vocab=int(vocab), dtype="f32", path=int(path), layers=2, max_positions=1200,
             kv_heads=int(kv_heads))
    kv = h.cache(1200, int(length))
    h.stub.stub_forget()
    h.ok(h.verify(kv, int(rows), None))
    assert ("small_step_kernel" in h.names()[0]) == bool(int(taken)), h.names()
    # (taken: it did nothing)  the separate launches did the step, and do the next one
    assert any("attn_kernel" in n for n in h.names()) and h.L.anpd_kv_length(kv) == int(length) + 1
    h.stub.stub_forget()
    h.ok(h.verify(kv, int(rows), None))
    assert not any("small_step_kernel" in n for n in h.names()), h.names()


# the tiny decoder at either end of its range (splits of 64 keys: eight; 17 rows and more count twice), a wider one, a larger
# vocabulary, separate launches asked for, too few blocks on any XCD
@pytest.mark.parametrize("d,heads,dh,ffn,vocab,path,length,rows,taken,blocks", [
    (256, 4, 64, 688, 1024, 0, 128, 5, 1, 32), (256, 4, 64, 688, 1024, 0, 0, 1, 1, 32), (256, 4, 64, 688, 1024, 0, 507, 5, 1, 32),
    (256, 4, 64, 688, 1024, 0, 508, 5, 0, 32), (256, 4, 64, 688, 1024, 0, 128, 32, 1, 32), (256, 4, 64, 688, 1024, 0, 239, 17, 1, 32),
    (256, 4, 64, 688, 1024, 0, 240, 17, 0, 32), (512, 8, 64, 1408, 1024, 0, 128, 5, 0, 32), (256, 4, 64, 688, 32000, 0, 128, 5, 0, 32),
    (256, 4, 64, 688, 1024, 1, 128, 5, 0, 32), (256, 4, 64, 688, 1024, 0, 128, 5, 0, 15),
])
def test_which_steps_are_one_launch_and_what_a_step_that_was_not_done_becomes(stub, d, heads, dh, ffn, vocab, path, length, rows, taken, blocks):
    run(stub, "child_route", d, heads, dh, ffn, vocab, path, length, rows, taken, blocks=blocks)


# an extra round of work items in a layer: up to d 384, 320 beyond 16 rows (more keys, more features, more key / value heads than 32 blocks take)
@pytest.mark.parametrize("d,heads,dh,ffn,kv_heads,length,rows,taken", [
    (320, 5, 64, 1024, 0, 128, 32, 1), (384, 6, 64, 512, 0, 128, 16, 1), (384, 6, 64, 512, 0, 8, 17, 0), (448, 7, 64, 512, 1, 128, 5, 1),
    (448, 7, 64, 512, 0, 128, 5, 0), (512, 8, 64, 512, 2, 128, 16, 1), (512, 8, 64, 512, 2, 251, 5, 1), (512, 8, 64, 512, 2, 252, 5, 0),
    (512, 8, 64, 512, 2, 128, 17, 0), (512, 8, 64, 512, 0, 128, 5, 0), (512, 8, 64, 528, 2, 128, 5, 0), (512, 4, 128, 512, 2, 450, 16, 1),
])
def test_an_extra_round_where_rounds_are_short(stub, d, heads, dh, ffn, kv_heads, length, rows, taken):
    run(stub, "child_route", d, heads, dh, ffn, 1024, 0, length, rows, taken, kv_heads)


def child_prompt():
    """A prompt whose last piece is small: its first pieces are launches, the last one's launch does nothing, and the prompt starts over."""
    import ctypes as C
    h = Host(dtype="f32", ffn=688, vocab=1024, layers=2, max_positions=700)
    kv = h.cache(700, 20)
    h.stub.stub_forget()
    h.ok(h.prefill(kv, 261))
    names = h.names()
    assert sum("small_step_kernel" in n for n in names) == 1 and sum("advance_length" in n for n in names) == 2 and h.L.anpd_kv_length(kv) == 281
    assert C.c_int32.from_address(h.length_at[kv.value]).value == 20      # (as it was before the second run, which the stand-in does not make)


def test_a_prompt_that_was_not_done_starts_over(stub):
    run(stub, "child_prompt")


def calls_in_one_launch(h, kv, out):
    return ((lambda: h.verify(kv, 5, out)), (lambda: h.verify_tree(kv, 5, out)), (lambda: h.prefill(kv, 20, out)))


def only_small(h):
    steps = [n for n in h.names() if "upload" not in n]
    return len(steps) == 1 and "small_step_kernel" in steps[0]


def child_pending_error():
    """An error that a call elsewhere left behind is reported and nothing is launched; the next call is a step like any other."""
    h = Host(dtype="f32", ffn=688, vocab=1024, layers=2, max_positions=300)
    kv = h.cache(300, 20)
    for call in calls_in_one_launch(h, kv, None):
        for _ in range(3):
            h.stub.stub_leave_error()
            h.stub.stub_forget()
            assert call() == h.B.E_HIP and not any("small_step_kernel" in n for n in h.names()), h.names()
            h.ok(h.L.anpd_kv_truncate(kv, 20, None))
            h.stub.stub_forget()
            h.ok(call())
            assert only_small(h), h.names()
            h.ok(h.L.anpd_kv_truncate(kv, 20, None))


def test_an_error_from_elsewhere_does_not_cost_the_count_of_launches(stub):
    run(stub, "child_pending_error", env={"STUB_SMALL_RUNS": "1"})


def child_lost_launch():
    """Every launch of a call fails once, while the logits go to memory that the runtime does not know (the query of it fails, too, and
    clears what was there): the call says so, and the next one is a step like any other."""
    import ctypes as C
    h = Host(dtype="f32", ffn=688, vocab=1024, layers=2, max_positions=300)
    kv = h.cache(300, 20)
    unknown = C.create_string_buffer(20 * 1024 * 4 + 16)
    for call in calls_in_one_launch(h, kv, (C.addressof(unknown) + 15) // 16 * 16):
        h.stub.stub_forget()
        h.ok(call())
        assert only_small(h), h.names()
        for nth in range(1, h.stub.stub_launches() + 1):
            h.ok(h.L.anpd_kv_truncate(kv, 20, None))
            h.stub.stub_fail_launch(nth)
            assert call() == h.B.E_HIP, (nth, h.names())
            h.ok(h.L.anpd_kv_truncate(kv, 20, None))
            h.stub.stub_forget()
            h.ok(call())
            assert only_small(h), (nth, h.names())
        h.ok(h.L.anpd_kv_truncate(kv, 20, None))


def test_a_launch_that_fails_is_reported_by_the_call_it_belongs_to(stub):
    run(stub, "child_lost_launch", env={"STUB_SMALL_RUNS": "1"})


def child_gave_up():
    """A wait inside the launch that is given up: the call says so, once, and the calls behind it are steps in one launch like any other."""
    h = Host(dtype="f32", ffn=688, vocab=1024, layers=2, max_positions=300)
    kv = h.cache(300, 20)
    for call in calls_in_one_launch(h, kv, None):
        for _ in range(3):
            h.stub.stub_give_up()
            assert call() == h.B.E_HIP and h.L.anpd_kv_length(kv) == 20
            for _ in range(2):
                h.ok(h.L.anpd_kv_truncate(kv, 20, None))
                h.stub.stub_forget()
                h.ok(call())
                assert only_small(h), h.names()
            h.ok(h.L.anpd_kv_truncate(kv, 20, None))


def test_a_wait_that_was_given_up_is_reported_once(stub):
    run(stub, "child_gave_up", env={"STUB_SMALL_RUNS": "1"})


if __name__ == "__main__":
    globals()[sys.argv[1]](*sys.argv[2:])
