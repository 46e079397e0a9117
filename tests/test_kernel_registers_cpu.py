"""Registers and spills of the kernels as they are built, from the metadata of the library's own gfx950 code objects (no GPU needed).

Only instances whose speed hangs on the figure, which the compiler changes without a word when code beside it changes."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    raw = open(lib, "rb").read()
    at = raw.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", raw, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", raw, pos)
            name = raw[pos + 24:pos + 24 + name_len].decode()
            pos += 24 + name_len
            if "gfx950" in name and size:
                yield raw[at + off:at + off + size]
        at = raw.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (registers, registers spilled)}"""
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("no llvm-readelf")
    from paper_2502_07861_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2502_07861_amd.build import build
        build()
    tmp = tmp_path_factory.mktemp("code")
    out = {}
    for i, obj in enumerate(_code_objects(binding.LIB_PATH)):
        path = tmp / ("%d.elf" % i)
        path.write_bytes(obj)
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for part in notes.split(".agpr_count:")[1:]:
            name = re.search(r"\.symbol:\s+(\S+?)(\.kd)?\s", part).group(1)
            out[name] = tuple(int(re.search(r"\.%s:\s+(\d+)" % k, part).group(1)) for k in ("vgpr_count", "vgpr_spill_count"))
    shutil.rmtree(tmp)
    assert len(out) > 60
    return out


def _compress(kernels, dtype, d, multi, vg, carry):
    """The instances of compress_kernel for these arguments, without the weight dump."""
    tag = "compress_kernelI%sLi%dELb0ELb%dELi%dELb%d" % (dict(bf16="DF16b", f32="f")[dtype], d, multi, vg, carry)
    found = {k: v for k, v in kernels.items() if tag in k}
    assert found, tag
    return found


@pytest.mark.parametrize("carry", [0, 1])
def test_blocks_of_narrow_rows_let_the_next_block_start(kernels, carry):
    """bf16 rows, d = 64: three wavefronts per SIMD (512 registers), so that a block of eight finds room before the last one has ended."""
    for name, (registers, spilled) in _compress(kernels, "bf16", 64, 0, 0, carry).items():
        assert registers <= 168 and spilled == 0, (name, registers, spilled)


def test_blocks_with_values_in_memory(kernels):
    """Blocks of several chunks with the value factor, bf16, d = 128: every tile needs 192 registers for operands and sums, what else is
    kept across it is spilled and comes back tile by tile.  182 spilled registers were 302 us for 256 blocks of 1024, 204 were 318."""
    for name, (_, spilled) in _compress(kernels, "bf16", 128, 1, 2, 0).items():
        assert spilled <= 182, (name, spilled)


@pytest.mark.parametrize("dtype,d,most", [("bf16", 128, 52), ("f32", 128, 71), ("f32", 64, 48)])
def test_carries_do_not_pay_for_the_token(kernels, dtype, d, most):
    """Resident carries with values in memory: taking a streamed token in is an instance of its own (last argument), which costs the others
    nothing (as a run-time choice 66, 87 and 62 spilled registers)."""
    plain = [v for k, v in _compress(kernels, dtype, d, 0, 2, 1).items() if "ELb0ELb0EE" in k[k.index("compress_kernel"):]]
    assert len(plain) == 1 and plain[0][1] <= most, plain
