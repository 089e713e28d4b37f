"""The built gfx950 code of the kernels that read LDS through assembly statements.  The compiler does not know that such
a read's registers are still being written, so its own code must leave them alone until the wait behind them: checked
here on what it made of the sources (no GPU needed; the persistent kernel, whose paths are too many to be walked, is left
out).  For the kernel whose wait counts rely on the order of its first
loads, the order as well."""
import os
import re
import struct
import subprocess

import pytest

from paper_2404_08698_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: [(address, instruction, operands)]} of the library's device code."""
    B.lib()
    blob = open(B.LIB_PATH, "rb").read()
    at = blob.index(b"__CLANG_OFFLOAD_BUNDLE__")
    count, pos = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
    for _ in range(count):
        offset, size, length = struct.unpack_from("<QQQ", blob, pos)
        triple = blob[pos + 24:pos + 24 + length]
        pos += 24 + length
        if b"gfx950" in triple:
            code = blob[at + offset:at + offset + size]
    path = tmp_path_factory.mktemp("code") / "device.co"
    path.write_bytes(code)
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
    out, cur = {}, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(\S+)>:$", line)
        if head:
            cur = out.setdefault(head.group(1), [])
            continue
        m = re.match(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m and cur is not None:
            cur.append((int(m.group(3), 16), m.group(1), m.group(2)))
    return out


def _registers(operands):
    """Vector registers named in an operand text."""
    found = set()
    for bank, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", operands):
        found |= {(bank, r) for r in range(int(lo), int(hi) + 1)}
    return found | {(bank, int(r)) for bank, r in re.findall(r"\b([va])(\d+)\b", operands)}


def _faults(code):
    """Instructions that touch a register an LDS read is still writing, over every path through the kernel."""
    index = {address: i for i, (address, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, ())], []
    while todo:
        i, flight = todo.pop()      # flight: registers written by each outstanding LDS / scalar memory operation, oldest first
        while i < len(code) and (i, flight) not in seen:
            seen.add((i, flight))
            address, name, operands = code[i]
            waits = re.search(r"lgkmcnt\((\d+)\)", operands) if name == "s_waitcnt" else None
            if waits:
                keep = int(waits.group(1))
                flight = flight[len(flight) - keep:] if keep else ()
            elif name.startswith(("ds_", "s_load", "s_buffer_load")):
                busy = frozenset().union(*flight)
                dst = operands.split(",")[0] if name.startswith(("ds_read", "ds_bpermute", "ds_swizzle")) else ""
                if _registers(operands) & busy:
                    bad.append((hex(address), name, operands))
                flight += (frozenset(_registers(dst)),)
            elif flight and _registers(operands) & frozenset().union(*flight):
                bad.append((hex(address), name, operands))
            if name == "s_endpgm":
                break
            if name.startswith(("s_cbranch", "s_branch")):
                jump = operands.split()[0]
                target = address + 4 + 4 * (int(jump) - (0x10000 if int(jump) >= 0x8000 else 0))
                todo.append((index[target], flight))
                if name == "s_branch":
                    break
            i += 1
    return bad


@pytest.mark.parametrize("name,count", [("prefill_gemm_kernel", 15), ("prefill_narrow_kernel", 6), ("prefill_mixed_kernel", 6),
                                        ("gemm_split_kernel", 1)])
def test_registers_of_reads_in_flight_are_left_alone(kernels, name, count):
    mine = {k: v for k, v in kernels.items() if name in k}
    assert len(mine) == count
    for k, code in mine.items():
        assert sum(n == "ds_read_b128" for _, n, _ in code) >= 4, k
        assert not _faults(code), k
        assert not [c for c in code if c[1].startswith("scratch_")], k    # no register was parked in memory


def test_a_register_that_is_used_too_early_is_seen():
    read, wait, end = (0, "ds_read_b128", "v[4:7], v1"), (8, "s_waitcnt", "lgkmcnt(0)"), (16, "s_endpgm", "")
    assert not _faults([read, wait, (12, "v_mov_b32_e32", "v9, v5"), end])
    assert _faults([read, (8, "v_mov_b32_e32", "v9, v5"), (12, "s_waitcnt", "lgkmcnt(0)"), end])
    assert _faults([read, (8, "v_mov_b32_e32", "v7, 0"), (12, "s_waitcnt", "lgkmcnt(0)"), end])
    assert _faults([read, (8, "ds_read_b128", "v[8:11], v1"), (12, "s_waitcnt", "lgkmcnt(1)"), (14, "v_mov_b32_e32", "v0, v8"), end])


def test_split_gemm_requests_its_operand_around_the_first_weights(kernels):
    """Its waits leave 16 weight loads and the other buffer's 8 operand loads outstanding: the first buffer's operand
    loads have to be the oldest, the second's the youngest."""
    code = next(v for k, v in kernels.items() if "gemm_split_kernel" in k)
    barrier = next(i for i, c in enumerate(code) if c[1] == "s_barrier")
    loads = ["x" if c[2].endswith("lds") else "w" for c in code[:barrier] if c[1].startswith("buffer_load")]
    assert "".join(loads) == "x" * 8 + "w" * 16 + "x" * 8


def _unordered(code):
    """Pairs (store, barrier): the second half of a row's eight columns of the residual stream is stored and the block meets behind its
    sums (16 bytes at a time, to LDS), on some path through the kernel, without a wait for all stores behind the products.  (One in front
    of them is the compiler's, for the operands it is about to use, and may leave out what came later.)"""
    index = {address: i for i, (address, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, None, False, False)], set()
    while todo:
        i, store, sums, waited = todo.pop()
        while i < len(code) and (i, store, sums, waited) not in seen:
            seen.add((i, store, sums, waited))
            address, name, operands = code[i]
            if name == "global_store_dwordx4" and operands.endswith("off offset:16"):
                store, sums, waited = hex(address), False, False
            elif name == "ds_write_b128":
                sums = True
            elif name == "s_waitcnt" and "vmcnt(0)" in operands:
                waited = True
            elif name.startswith("v_mfma"):
                waited = False
            elif name == "s_barrier" and sums:
                if store and not waited:
                    bad.add((store, hex(address)))
                store = None
            if name == "s_endpgm":
                break
            if name.startswith(("s_cbranch", "s_branch")):
                jump = int(operands.split()[0])
                todo.append((index[address + 4 + 4 * (jump - (0x10000 if jump >= 0x8000 else 0))], store, sums, waited))
                if name == "s_branch":
                    break
            i += 1
    return sorted(bad)


def test_small_step_meets_behind_the_rows_that_it_stores(kernels):
    """The flag of the first QKV item, set by one or two of its waves, stands for the residual stream that all eight have stored."""
    mine = {k: v for k, v in kernels.items() if "small_step_kernel" in k}
    assert len(mine) == 4
    for k, code in mine.items():
        assert sum(n == "global_store_dwordx4" and o.endswith("off offset:16") for _, n, o in code) >= 1, k
        assert not _unordered(code), k


def test_small_step_reads_the_windows_keys_and_values_past_the_vector_cache(kernels):
    """Other blocks of the launch have stored them, so none may come from a line that the compute unit holds: per 16 dimensions a lane has
    four numbers of one key, in pieces of 8 bytes, and one of four values each."""
    mine = {k: v for k, v in kernels.items() if "small_step_kernel" in k}
    assert len(mine) == 4
    for k, code in mine.items():
        chunks = int(re.search(r"small_step_kernelILi(\d+)E", k).group(1)) // 16
        past = [n for _, n, o in code if n.startswith("global_load") and "sc1" in o]
        assert past.count("global_load_dwordx2") >= 2 * chunks and past.count("global_load_dword") >= 4 * chunks, (k, len(past))


def test_a_store_that_a_barrier_does_not_wait_for_is_seen():
    store, sums, wait, meet = (0, "global_store_dwordx4", "v[8:9], v[4:7], off offset:16"), (8, "ds_write_b128", "v2, v[4:7]"), (16, "s_waitcnt", "vmcnt(0)"), (20, "s_barrier", "")
    assert not _unordered([store, sums, wait, meet, (24, "s_endpgm", "")])
    assert not _unordered([store, wait, sums, meet, (24, "s_endpgm", "")])
    assert _unordered([store, sums, (16, "s_waitcnt", "lgkmcnt(0)"), meet, (24, "s_endpgm", "")])
    assert _unordered([store, wait, (18, "v_mfma_f32_16x16x4_f32", "v[0:3], v1, v2, v[0:3]"), sums, meet, (24, "s_endpgm", "")])
    assert _unordered([store, sums, (12, "s_cbranch_execz", "1"), wait, meet, (24, "s_endpgm", "")])


def test_generic_attention_waits_once_in_front_of_its_keys_and_values(kernels):
    """The pages of a wave's keys come together; the loads behind them are all on their way before the first product waits."""
    mine = {k: v for k, v in kernels.items() if re.search(r"\d+attn_kernelIf", k)}
    assert len(mine) == 2
    for k, code in mine.items():
        first = next(i for i, c in enumerate(code) if c[1].startswith("global_load"))
        product = next(i for i, c in enumerate(code) if c[1].startswith("v_mfma"))
        last = max(i for i, c in enumerate(code[:product]) if c[1].startswith("global_load"))
        assert sum(n == "s_waitcnt" and "vmcnt" in o for _, n, o in code[first:last]) == 1, k


@pytest.mark.parametrize("name,count", [("prefill_few_kernel", 9), ("prefill_gemm_kernel", 15), ("prefill_narrow_kernel", 6)])
def test_prompt_gemms_request_their_arguments_together(kernels, name, count):
    """One round trip for the grid's size and the arguments that a block finds its tiles and rows with."""
    mine = {k: v for k, v in kernels.items() if name in k}
    assert len(mine) == count
    for k, code in mine.items():
        division = next(i for i, c in enumerate(code) if c[1].startswith("v_rcp_iflag"))
        assert sum(n == "s_waitcnt" for _, n, _ in code[:division]) == 1, k
