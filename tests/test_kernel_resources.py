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


def test_sketched_searches_keep_their_waves(kernels):
    """search_sketch_kernel<KIND, NCH, NSLOT, EPS, TAG16, OWN, NETWORK, SK>: six waves per SIMD at four pieces per lane,
    five at six and seven, four at eight."""
    waves = {4: 6, 6: 5, 7: 5, 8: 4}
    for a, f in _named(kernels, "search_sketch_kernel").items():
        assert 512 // (-(-f["vgpr_count"] // 8) * 8) >= waves[a[1]], a


def test_spills(kernels):
    """No kernel keeps registers in memory, but for the one whose third wave is worth it (PruneWaves)."""
    spills = {k: f["vgpr_spill_count"] for k, f in kernels.items() if f["vgpr_spill_count"]}
    assert set(spills) <= {("prune_kernel", (2, 16, 7))} and all(n <= 8 for n in spills.values()), spills


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,metric,d,nch", [
    ("uint8", 0, 128, 1), ("uint8", 0, 200, 2), ("uint8", 0, 400, 4), ("int8", 0, 100, 1), ("int8", 0, 256, 2), ("int8", 0, 512, 4),
    ("float32", 0, 48, 2), ("float32", 0, 100, 4), ("float32", 0, 144, 6), ("float32", 0, 200, 7), ("float32", 0, 256, 8),
    ("float32", 1, 64, 2), ("float32", 1, 128, 4), ("float32", 1, 192, 6), ("float32", 1, 224, 7), ("float32", 1, 240, 8)])
def test_filter_sizes_match_the_registers(kernels, env, dtype, metric, d, nch):
    """The visited filter takes the LDS that the waves of search_kernel<KIND, VEC, NCH, NSLOT, EPS, TAG16, OWN, NETWORK>
    leave to each other: what the library's rule gives for every instance, against the registers of its
    metadata.  A compute unit has 160 KB, handed out in units of 1,280 bytes, and four SIMDs."""
    import numpy as np
    _, A, _ = env
    found = _named(kernels, "search_kernel")
    code = {"uint8": A.U8, "int8": A.I8, "float32": A.F32}[dtype]
    kind = {"uint8": 0, "int8": 1, "float32": 2 + metric}[dtype]
    seen = set()
    for n, Rs in ((100, (32, 48, 64)), ((1 << 20) + 1, (1,)), ((1 << 22) + 1, (1,)), ((1 << 23) + 1, (1,))):
        if n > 100 and (dtype, d) not in (("uint8", 128), ("uint8", 200), ("float32", 200)):
            continue
        for R in Rs:
            g = A.ann_graph_from_host(np.full((n, R), 0xFFFFFFFF, np.uint32), d, code, metric, 0)
            for L in (7, 8, 20, 60, 64, 65, 100, 128, 129, 200, 256):
                for eps in (-1.0, 0.1):
                    for own in (0, 1):
                        for nq in (200, 20000):
                            waves, words, bits = g.search_filter(nq, L, eps, own)
                            nslot = 1 if L <= 64 else 2 if L <= 128 else 4
                            net = nslot == 1 and (R >= 64 or R > 32 and (L <= 24 or eps >= 0) or nq <= 256)
                            net = net and not (own and kind >= 2 and nch <= 2)
                            a = (kind, 16, nch, nslot, int(eps >= 0), int(bits == 16), own, int(net))
                            seen.add(a)
                            # (where 16-bit tags do not fit the first instance's table, the other instance's decides)
                            either = [a] + ([a[:5] + (0,) + a[6:]] if n > 100 else [])
                            assert waves in [min(8, 512 // (-(-found[x]["vgpr_count"] // 8) * 8)) for x in either], (a, waves)
                            if nslot == 4 or (nslot == 2 and n > 1 << 22):
                                waves = min(waves, 6)
                            share = 160 * 1024 // (4 * waves) // 1280 * 1280
                            assert words == (512 if L < 8 else min(2048, (share - 512 * nslot - 512) // 16 * 4)), (a, n, words)
                            assert bits == 16 or n > 100
    assert {a[3:] for a in seen if a[5]} >= {a[3:] for a in found if a[0] == kind and a[2] == nch and a[3] <= 4 and a[5]}
