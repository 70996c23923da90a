"""What the compiler made of the kernels, read from the disassembly of the library built here (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_05965_amd", "libhap.so")


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """Instructions of every kernel symbol of the library."""
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "libhap.so")
    subprocess.run([OBJDUMP, "--offloading", "libhap.so"], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found, name = {}, None
    for f in sorted(d.glob("libhap.so.*gfx950")):
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, stdout=subprocess.PIPE, text=True).stdout.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
                found.setdefault(name, [])
            elif name and line.startswith("\t"):
                found[name].append(line.split("//")[0].strip())
    return found


@pytest.fixture(scope="module")
def chunk_accesses(code):
    """Per kernel symbol: 16-byte global (non-temporal stores, plain stores, loads)."""
    found = {}
    for name, lines in code.items():
        stores = [l for l in lines if l.startswith("global_store_dwordx4")]
        nt = sum(l.split()[-1] == "nt" for l in stores)
        found[name] = (nt, len(stores) - nt, sum(l.startswith("global_load_dwordx4") for l in lines))
    return found


def kernels(found, pattern):
    hits = {k: v for k, v in found.items() if re.search(pattern, k)}
    assert hits, pattern
    return hits


BF16, F32 = "IDF16b", "If"      # how the first template argument, the output type, shows in a symbol


def test_only_the_bf16_preactivation_copy_is_stored_non_temporally(chunk_accesses):
    """One of the epilogue's three modes has a second store, the copy: fewer non-temporal stores than plain ones.  (A non-temporal and a
    plain store in two branches of one condition would show here as plain ones only: the compiler folds them.)"""
    for what in ("gemm_pp_kernel", "gemm_dma_kernel", "gemm_kpair_kernel"):
        for name, (nt, plain, _) in kernels(chunk_accesses, what + BF16).items():
            assert plain > nt > 0, (name, nt, plain)
        for name, (nt, plain, _) in kernels(chunk_accesses, what + F32).items():
            assert plain > nt == 0, (name, nt, plain)
    for name, (nt, _, _) in kernels(chunk_accesses, "splitk_reduce_kernel").items():
        assert nt == 0, (name, nt)


def test_paired_tiles_request_each_preactivation_chunk_once(chunk_accesses):
    """A wave of the K-pair kernel stores 32 x 64 bf16: 4 chunks of 16 bytes per lane, 5 where the tile is shifted onto the output's chunks.
    The activation backward reads as many, and the two other modes of the epilogue read the old chunk when they accumulate."""
    for name, (_, _, loads) in kernels(chunk_accesses, "gemm_kpair_kernel" + BF16).items():
        assert loads == 3 * (4 + 5), (name, loads)


def registers(text):
    """The vector registers that an operand string names."""
    return {f"{k}{i}" for k, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text) for i in range(int(lo), int(hi) + 1)} | set(re.findall(r"\b[va]\d+\b", text))


def test_fragments_are_left_alone_until_their_wait(code):
    """The fragment reads of the two kernels that order their phases by hand are inline assembly, and the wait for them is a statement of its
    own: to the compiler a fragment is there at once.  From a read to the wait that covers it no instruction may name its registers - no
    copy, no address put there.  (LDS operations return in order: a wait for n leaves the last n outstanding.)"""
    for pattern in ("gemm_pp_kernel", "gemm_kpair_kernel"):
        for name, lines in kernels(code, pattern).items():
            pending, reads = [], 0      # per outstanding LDS operation: the registers it will write
            for line in lines:
                op, _, operands = line.partition(" ")
                if op == "s_waitcnt" and "lgkmcnt" in operands:
                    n = int(re.search(r"lgkmcnt\((\d+)\)", operands).group(1))
                    pending = pending[len(pending) - n:] if 0 < n < len(pending) else (pending if n else [])
                    continue
                used = registers(operands)
                assert not any(p & used for p in pending), (name, line)
                if op.startswith("ds_"):
                    read = op.startswith("ds_read")
                    reads += read
                    pending.append(registers(operands.split(",")[0]) if read else set())
            assert reads >= 32, (name, reads)


def test_fragments_of_the_other_hand_ordered_kernels_are_left_alone(code):
    """The same for the two kernels that read their fragments whole before a tile's MFMAs."""
    for pattern in ("gemm_trio_kernel", "gemm_small_kernel"):
        for name, lines in kernels(code, pattern).items():
            pending, reads = [], 0
            for line in lines:
                op, _, operands = line.partition(" ")
                if op == "s_waitcnt" and "lgkmcnt" in operands:
                    n = int(re.search(r"lgkmcnt\((\d+)\)", operands).group(1))
                    pending = pending[len(pending) - n:] if 0 < n < len(pending) else (pending if n else [])
                    continue
                used = registers(operands)
                assert not any(p & used for p in pending), (name, line)
                if op.startswith("ds_"):
                    read = op.startswith("ds_read")
                    reads += read
                    pending.append(registers(operands.split(",")[0]) if read else set())
            assert reads >= 12, (name, reads)
