"""Registers and private memory of the relaxed path's kernels, from the
metadata of the built library's own code objects (CPU): what the occupancy
that their launch plans count on needs."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2406_01821_amd", "libaerl.so")
EM_AMDGPU, NT_AMDGPU_METADATA, SHT_NOTE = 224, 32, 7


def kernels():
    """name -> metadata of every kernel: the device ELF images embedded in the
    library, their notes' msgpack."""
    blob = open(LIB, "rb").read()
    out = {}
    for m in re.finditer(rb"\x7fELF\x02\x01\x01", blob):
        b = m.start()
        if struct.unpack_from("<H", blob, b + 18)[0] != EM_AMDGPU:
            continue
        shoff, = struct.unpack_from("<Q", blob, b + 40)
        shentsize, shnum = struct.unpack_from("<HH", blob, b + 58)
        for i in range(shnum):
            h = b + shoff + i * shentsize
            if struct.unpack_from("<I", blob, h + 4)[0] != SHT_NOTE:
                continue
            at, size = (b + struct.unpack_from("<Q", blob, h + 24)[0],
                        struct.unpack_from("<Q", blob, h + 32)[0])
            end = at + size
            while at < end:
                namesz, descsz, kind = struct.unpack_from("<III", blob, at)
                desc = at + 12 + (namesz + 3) // 4 * 4
                if kind == NT_AMDGPU_METADATA:
                    meta = msgpack.unpackb(blob[desc:desc + descsz])
                    out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
                at = desc + (descsz + 3) // 4 * 4
    return out


@pytest.fixture(scope="module")
def found():
    from paper_2406_01821_amd import aerl  # noqa: F401  (builds the library if there is none)
    k = kernels()
    assert any("k_soft_fwd" in n for n in k)
    return k


def named(found, *parts):
    hits = {n: k for n, k in found.items() if any(p in n for p in parts)}
    assert hits
    return hits


def test_classifying_forwards_leave_eight_waves_per_simd(found):
    for n, k in named(found, "k_soft_fwd_cls", "k_smax_fwd_cls").items():
        assert k[".vgpr_count"] <= 64, n
        assert k[".sgpr_count"] <= 80, n


def test_private_memory_follows_the_longest_rule_set(found):
    """Up to 32 rules the adjoints and the fine-tuning kernel ask for the
    private memory of 32 rules (two or, under the softmax head, three floats
    per rule and sample, and a few spilled registers), not of 64."""
    few = {n: k for n, k in named(found, "k_soft_bwd_reg", "k_smax_bwd_reg", "k_tune_sets").items()
           if "Li32EEE" in n}
    assert few
    for n, k in few.items():
        floats = 3 if "smax" in n else 2
        samples = int(re.search(r"ILi(\d)E", n).group(1))
        assert k[".private_segment_fixed_size"] <= 4 * floats * samples * 32 + 128, n
