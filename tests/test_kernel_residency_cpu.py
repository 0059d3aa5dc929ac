"""The z chunks of the 3D walking kernels are sized for the blocks that a compute
unit holds at a time.  Each launch states that number; here it is compared with what
the registers and the LDS of the built kernels allow, read from the code object's
own metadata in libes.so (no GPU)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2202_07989_amd", "libes.so")
SOURCE = os.path.join(ROOT, "paper_2202_07989_amd", "csrc", "es_kernels.hip")
LDS, REGISTERS, SIMDS, WAVES = 160 * 1024, 512, 4, 8    # of a compute unit / a SIMD's lane


def code_objects(blob):
    """The gfx950 ELF images of the offload bundles in a library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        q = at + len(magic) + 8
        if count < 16:
            for _ in range(count):
                off, size, n = struct.unpack_from("<QQQ", blob, q)
                if b"gfx950" in blob[q + 24:q + 24 + n]:
                    yield blob[at + off:at + off + size]
                q += 24 + n
        at += len(magic)


def kernels(elf):
    """Metadata of an image's kernels (the note of type 32)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for s in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + s * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + s * size + 0x18)
        while kind == 7 and length > 0:
            n, d, t = struct.unpack_from("<III", elf, off)
            body = off + 12 + (n + 3) // 4 * 4
            if t == 32:
                yield from msgpack.unpackb(elf[body:body + d])["amdhsa.kernels"]
            step = body + (d + 3) // 4 * 4 - off
            off, length = off + step, length - step


@pytest.fixture(scope="module")
def resident():
    """Blocks of each kernel a compute unit holds, by demangled name."""
    with open(LIB, "rb") as f:
        ks = [k for e in code_objects(f.read()) for k in kernels(e)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in ks), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    out = {}
    for k, name in zip(ks, names):
        waves = (k[".max_flat_workgroup_size"] + 63) // 64
        per_simd = min(WAVES, REGISTERS // ((k[".vgpr_count"] + 7) // 8 * 8))
        lds = k[".group_segment_fixed_size"]
        blocks = min(SIMDS * per_simd // waves, LDS // lds if lds else 99)
        m = re.search(r"es::(k_\w+(<[^>]*>)?)", name)
        if m:
            out[m.group(1).replace(" ", "")] = blocks
    return out


def test_walks_of_the_mesh_step(resident):
    """(a launch that states no number of its own is sized for two)"""
    with open(SOURCE) as f:
        calls = re.findall(r"march\((k_\w+<[^>]*>), \d+, \d+, \d+, \d+(?:, (\d+))?,", f.read())
    assert len(calls) == 7
    for name, blocks in calls:
        assert resident[name.replace(" ", "")] == int(blocks or 2), name


@pytest.mark.parametrize("name,blocks", [("k_metric3<32,16,true>", 1), ("k_metric3<32,16,false>", 1)] +
                         [(f"k_monitor_grad3<{n},{sig}>", 3 if sig == 0 else 2) for n in (1, 2) for sig in (0, 1, 2)])
def test_metrics_and_monitor(resident, name, blocks):
    assert resident[name] == blocks
