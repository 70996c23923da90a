"""What the compiler made of the kernels, read from the disassembly of the library built here (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_05965_amd", "libhap.so")


@pytest.fixture(scope="module")
def chunk_accesses(tmp_path_factory):
    """Per kernel symbol: 16-byte global (non-temporal stores, plain stores, loads)."""
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "libhap.so")
    subprocess.run([OBJDUMP, "--offloading", "libhap.so"], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found, name = {}, None
    for f in sorted(d.glob("libhap.so.*gfx950")):
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, stdout=subprocess.PIPE, text=True).stdout.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
                found.setdefault(name, [0, 0, 0])
            elif "global_store_dwordx4" in line:
                found[name][0 if re.search(r"\bnt\b", line.split("//")[0]) else 1] += 1
            elif "global_load_dwordx4" in line:
                found[name][2] += 1
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
