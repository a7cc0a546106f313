"""What the compiler made of the library's kernels: the occupancy targets of the
pair passes are chosen so that no variant spills vector registers to memory, so
the built library must hold no kernel that does."""
import os
import re

import pytest


def spills(lib_bytes):
    """{kernel: spilled vector registers} from the metadata notes of the code objects
    (MessagePack maps with sorted keys: .name precedes .vgpr_spill_count)."""
    out = {}
    for m in re.finditer(rb"\.vgpr_spill_count(?:([\x00-\x7f])|\xcc(.)|\xcd(..))", lib_bytes, re.S):
        head = lib_bytes[max(0, m.start() - 4096):m.start()]
        name = re.findall(rb"\.name(?:\xd9.|\xda..|[\xa0-\xbf])(\w+)", head, re.S)[-1].decode()
        out[name] = int.from_bytes(m.group(1) or m.group(2) or m.group(3), "big")
    return out


def test_no_kernel_spills_vector_registers():
    import paper_2108_08919_amd as P
    if not os.path.exists(P.LIB_PATH):
        pytest.skip("library not built")
    with open(P.LIB_PATH, "rb") as f:
        s = spills(f.read())
    assert sum("k_pass_" in k for k in s) > 100 and sum("k_learn_" in k for k in s) > 100
    assert any("k_mlp_backward" in k for k in s)
    assert {k: v for k, v in s.items() if v} == {}
