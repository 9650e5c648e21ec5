"""The kernels as they are built: registers of the GEMMs, and that no two variants are the same code.

Every ordinary GEMM instance is launched for all projections; what an epilogue that only one of them needs would cost it shows here: the
256 x 256 tile fills the register file, and 16 spilled vector registers are what its own residual epilogue takes."""
import os
import re
import struct
import subprocess

import pytest

from paper_2506_10470_amd import build as B

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects inside the library: files"""
    if not os.path.exists(B.LIB):
        B.build()
    data = open(B.LIB, "rb").read()
    folder = tmp_path_factory.mktemp("code")
    files = []
    for at in (m.start() for m in re.finditer(MAGIC, data)):
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in target and size:
                files.append(folder / ("%d.co" % len(files)))
                files[-1].write_bytes(data[at + offset:at + offset + size])
    assert files
    return files


def readelf(what, path):
    tool = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
    return subprocess.run([tool, what, "--wide", str(path)], capture_output=True, text=True, check=True).stdout


@pytest.fixture(scope="module")
def kernels(code_objects):
    """(rows / 32, weight rows / 32, parameters) -> the worst of (spilled vector registers, bytes of scratch) over its instances"""
    found = {}
    for path in code_objects:
        for kernel in readelf("--notes", path).split("  - .agpr_count:")[1:]:
            field = dict(re.findall(r"^    \.(\w+): +(\S+)$", kernel, re.M))
            m = re.search(r"gemm_mi16_kernelILi(\d)ELi(\d)ELi\d+ELb\dE\w*?(Gemm[A-Za-z]*Params)E", field["name"])
            if m:
                key = int(m.group(1)), int(m.group(2)), m.group(3)
                use = int(field["vgpr_spill_count"]), int(field["private_segment_fixed_size"])
                found[key] = max(found.get(key, (0, 0)), use)
    return found


def test_ordinary_projections_pay_for_no_other_epilogue(kernels):
    ordinary = {k[:2]: v for k, v in kernels.items() if k[2] == "GemmParams"}
    assert len(ordinary) == 12                      # (128 x 128 has two forms)
    spills, scratch = ordinary.pop((8, 8))
    assert spills <= 16 and scratch <= 68, (spills, scratch)
    assert set(ordinary.values()) == {(0, 0)}, ordinary


def test_the_rotating_epilogue_keeps_to_registers(kernels):
    rotating = {k[:2]: v for k, v in kernels.items() if k[2] == "GemmRotateParams"}
    assert sorted(rotating) == [(n, 8) for n in (4, 5, 6, 7, 8)]
    assert set(rotating.values()) == {(0, 0)}, rotating


def test_the_maximum_epilogue_keeps_to_registers(kernels):
    maximum = {k[:2]: v for k, v in kernels.items() if k[2] == "GemmMaxParams"}
    assert len(maximum) == 12
    assert set(maximum.values()) == {(0, 0)}, maximum


def test_no_two_cache_moves_are_the_same_code(code_objects):
    """A variant that is dispatched to and does what another does is a rule without effect."""
    code = {}
    for path in code_objects:
        data = path.read_bytes()
        text = re.search(r"\.text +PROGBITS +(\w+) (\w+)", readelf("--sections", path))
        address, offset = (int(x, 16) for x in text.groups())
        for m in re.finditer(r"^ +\d+: (\w+) +(\d+) FUNC .* (\S*kv_move_kernel\S*)$", readelf("--symbols", path), re.M):
            at = int(m.group(1), 16) - address + offset
            code[m.group(3)] = data[at:at + int(m.group(2))]
    assert len(code) >= 8
    assert len(set(code.values())) == len(code), sorted(code)


def test_prefill_attention_does_not_wait_for_the_next_block_early(code_objects):
    """16-bit pools: a block is requested straight into LDS while the one before it is computed.  The only wait for memory between the
    requests and the barrier behind that block is the one in front of the barrier; any other drains the same counter."""
    tool = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    seen = 0
    for path in code_objects:
        if b"attn_prefill_kernel" not in path.read_bytes():
            continue
        text = subprocess.run([tool, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for m in re.finditer(r"^\w+ <\S*attn_prefill_kernel\S*ELb0E\S*>:\n(.*?)(?=^\w+ <|\Z)", text, re.M | re.S):
            lines = m.group(1).splitlines()
            last = max(i for i, l in enumerate(lines) if "global_load_lds" in l)
            barrier = next(i for i in range(last, len(lines)) if "s_barrier" in lines[i])
            waits = [l.strip() for l in lines[last:barrier] if "s_waitcnt" in l and "vmcnt" in l]
            assert len(waits) == 1 and "vmcnt(0)" in waits[0], waits
            seen += 1
    assert seen == 2
