"""Registers of the built kernels, from the metadata that the compiler leaves in the library (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2305_04359_amd import build as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(name, template arguments): {"vgpr_count": ..., "vgpr_spill_count": ...}}"""
    data = open(B.library_path(), "rb").read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", {}
    path = str(tmp_path_factory.mktemp("co") / "code.o")
    for m in re.finditer(magic, data):
        at = m.start()
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" not in target or size == 0:
                continue
            with open(path, "wb") as f:
                f.write(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
            for block in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
                field = dict(re.findall(r"\.(name|vgpr_count|vgpr_spill_count):\s+(\S+)", block))
                name = re.match(r"_ZN5annmi\d+(\w+?)I((?:L[ijb]\d+E)+)E", field.pop("name"))
                if name:
                    args = tuple(int(x) for x in re.findall(r"L[ijb](\d+)E", name[2]))
                    out[name[1], args] = {k: int(v) for k, v in field.items()}
    return out


def _named(kernels, name):
    found = {a: f for (n, a), f in kernels.items() if n == name}
    assert found, name
    return found


def test_shared_searches_all_fit(kernels):
    """search_wide_kernel<KIND, VEC, NCH, NSLOT>: 128 registers, so that a compute unit holds two
    workgroups of eight waves and the largest launch is on the chip at once."""
    assert all(f["vgpr_count"] <= 128 for f in _named(kernels, "search_wide_kernel").values())


def test_own_start_searches_keep_eight_waves(kernels):
    """search_kernel<KIND, VEC, NCH, NSLOT, EPS, TAG16, OWN, NETWORK> of float rows of up to 64 elements with
    start vertices of their own: one-slot beams leave room for eight waves per SIMD."""
    found = {a: f for a, f in _named(kernels, "search_kernel").items() if a[:4] in ((2, 16, 2, 1), (3, 16, 2, 1)) and a[6]}
    assert found and all(f["vgpr_count"] <= 64 for f in found.values())


def test_filter_sizes_match_the_registers(kernels):
    """The visited filter takes the LDS that the waves of search_kernel<KIND, VEC, NCH, NSLOT, EPS, TAG16, OWN, NETWORK>
    leave to each other: the waves per SIMD that search.hip assumes are those of the registers, give or take one
    where variants differ."""
    def assumed(nch, nslot, own):
        if nslot <= 2:
            return 8 if nch == 1 else 7 if nch == 2 else (6 if own else 5) if nch == 4 else 5 if nch == 6 or (nch == 7 and (own or nslot == 1)) else 4
        return 5 if nch <= 2 else (5 if own else 4) if nch == 4 else 4

    for a, f in _named(kernels, "search_kernel").items():
        if a[3] <= 4 and a[5]:
            waves = min(8, 512 // (-(-f["vgpr_count"] // 8) * 8))
            assert abs(waves - assumed(a[2], a[3], a[6])) <= (2 if a[3] == 4 and a[4] else 1), (a, f)
