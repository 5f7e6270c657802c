"""What the compiled kernels ask for, as the library's own code objects state it (CPU only): registers that decide what runs beside
what, and no private memory where a chain of dependent steps or a ring of counted loads would wait for it."""
import os
import struct
import subprocess

import msgpack
import pytest


def _notes(elf):
    phoff, = struct.unpack_from("<Q", elf, 0x20)
    size, count = struct.unpack_from("<HH", elf, 0x36)
    for i in range(count):
        kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * size)
        at, end = off, off + length
        while kind == 4 and at < end:  # PT_NOTE
            n_name, n_desc, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (n_name + 3 & ~3)
            if note == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[desc:desc + n_desc], strict_map_key=False)
            at = desc + (n_desc + 3 & ~3)


@pytest.fixture(scope="module")
def kernels():
    """Demangled kernel name -> its metadata."""
    import paper_2401_14361_amd as m
    if not os.path.exists(m.lib_path()):          # build only if nothing is built
        from paper_2401_14361_amd.build import build
        build()
    lib = open(m.lib_path(), "rb").read()
    found, magic, at = {}, b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := lib.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", lib, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, n_triple = struct.unpack_from("<QQQ", lib, p)
            if size and b"gfx950" in lib[p + 24:p + 24 + n_triple]:
                for meta in _notes(lib[at + off:at + off + size]):
                    found.update((k[".name"], k) for k in meta["amdhsa.kernels"])
            p += 24 + n_triple
        at += len(magic)
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.splitlines()
    return {name.replace("(anonymous namespace)::", "").split("moei::", 1)[-1]: k for name, k in zip(names, found.values())}


def _named(kernels, *starts):
    got = {n: k for n, k in kernels.items() if n.startswith(starts)}
    assert got, (starts, sorted(kernels)[:5])
    return got


@pytest.mark.parametrize("name", ["ffn_fused_kernel<", "ffn_grouped_mm_kernel<", "ffn_grouped_kernel<", "eamc_pick_kernel", "eamc_pick_score_kernel<", "eamc_topm_kernel", "eamc_topm_score_kernel<"])
def test_no_private_memory(kernels, name):
    for n, k in _named(kernels, name).items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, (n, k[".private_segment_fixed_size"])


def test_a_scan_fits_beside_the_streaming_ffn(kernels):
    # a compute unit holds a workgroup of the FFN that streams (4, 3 or 2 wavefronts a SIMD, by the chunks of its rows) and one of a
    # scan of 48 registers; the code that steps with a match beside their experts need is in instances of their own, which fill a compute
    # unit by themselves: their registers are for the wavefronts that the launch counts on, one that routes among them
    checked = {"true": 0, "false": 0}
    for n, k in _named(kernels, "ffn_fused_kernel<").items():
        _, chunks, _, match = n[len("ffn_fused_kernel<"):n.index(">")].split(", ")
        waves = 4 if int(chunks) <= 4 else 3 if int(chunks) <= 10 else 2
        beside = 48 if match == "false" else 0
        assert waves * (k[".vgpr_count"] + 7 & ~7) + beside <= 512, (n, k[".vgpr_count"])
        checked[match] += 1
    assert checked == {"true": 52, "false": 52}
