"""What the compiler reports of the kernels in libminf.so (metadata of the library's own code objects)."""
import os
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2407_02490_amd", "libminf.so")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernel_metadata(elf):
    """Kernel entries of the metadata note of one device ELF."""
    import msgpack
    table, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3a)
    for i in range(count):
        _, kind, _, _, at, _ = struct.unpack_from("<IIQQQQ", elf, table + i * size)
        if kind == 7:                                                      # SHT_NOTE
            name, desc, _ = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            return msgpack.unpackb(elf[at:at + desc])["amdhsa.kernels"]
    return []


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        import __graft_entry__ as g
        g.build()
    data, found, pos = open(LIB, "rb").read(), {}, 0
    while (pos := data.find(BUNDLE, pos)) >= 0:
        n, = struct.unpack_from("<Q", data, pos + len(BUNDLE))
        at = pos + len(BUNDLE) + 8
        for _ in range(n):
            ofs, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in target and size:
                for k in kernel_metadata(data[pos + ofs:pos + ofs + size]):
                    found[k[".name"]] = k
        pos += 1
    return found


def test_attention_kernels_use_no_scratch_memory(kernels):
    """No vector register is spilled and no argument is copied to a stack: the one-launch kernels of two
    kinds once wrote both launch orders, 568 bytes a lane, to scratch memory at the start of every block."""
    names = [n for n in kernels if any(s in n for s in ("ashape_kernel", "ashape_split_kernel", "bs_kernel",
                                                        "bs_split_kernel", "vs_kernel", "vs_split_kernel",
                                                        "vs_share_kernel", "vs_bs_wide_kernel", "vs_ring_kernel"))]
    assert len(names) == 10
    for n in names:
        assert kernels[n][".private_segment_fixed_size"] == 0 and kernels[n][".vgpr_spill_count"] == 0, n


def test_score_kernels_are_those_that_are_launched(kernels):
    """Chunks of 64 keys belong to pass 2 only."""
    score = sorted(n[n.index("ILi") + 3:].split("EEEv")[0] for n in kernels if "vs_score_kernel" in n)
    assert score == sorted(f"{p}ELi{c}" for p, c in ((1, 128), (1, 256), (1, 1024), (2, 64), (2, 128), (2, 256), (2, 1024)))
