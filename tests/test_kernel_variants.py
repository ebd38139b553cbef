"""The generic line kernels of the built library, from its symbol table: every
one comes as two variants, and the one that serves lengths without a direct
sum holds none of its code (its presence alone slowed these lengths by 5-15%;
fft_lds_mixed in pc_solve.hip)."""
import os
import re
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2304_14690_amd", "libpcorr.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def device_elfs(blob):
    """The gfx950 code objects of the offload bundles in a shared library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + ln].decode()
            p += 24 + ln
            if name.endswith("gfx950") and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def kernel_sizes(elf):
    """{symbol: code bytes} of the functions in an ELF64 image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    sec = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    out = {}
    for s in sec:
        if s[1] != 2:  # SHT_SYMTAB
            continue
        strs = sec[s[6]]
        for q in range(s[4], s[4] + s[5], 24):
            name, info, _, _, _, size = struct.unpack_from("<IBBHQQ", elf, q)
            if info & 15 == 2:  # STT_FUNC
                a = strs[4] + name
                out[elf[a:elf.index(b"\0", a)].decode()] = size
    return out


def test_smooth_lengths_run_kernels_without_direct_sums():
    if not os.path.exists(LIB):
        pytest.skip("libpcorr.so is not built")
    with open(LIB, "rb") as f:
        blob = f.read()
    sizes = {}
    for elf in device_elfs(blob):
        sizes.update(kernel_sizes(elf))
    lines = {k: v for k, v in sizes.items()
             if re.search(r"GLOBAL__N_1\d+(dct_lines|rdft_lines|dct1_lines)I", k)}
    plain = [k for k in lines if "Lb0EEEv" in k]
    assert len(plain) == len(lines) / 2 == 50  # 30 dct_lines, 10 rdft_lines, 10 dct1_lines
    for k in plain:
        assert lines[k] < lines[k.replace("Lb0EEEv", "Lb1EEEv")], k
