"""Registers that the kernels of the built library leave to other workgroups on their compute units (read from its code objects, no
GPU): what include/pk.h promises the communicator beside an all-gather GEMM, and what the reduce beside a GEMM needs."""
import re
import struct
import subprocess

import pytest

from paper_2511_13940_amd import pk

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
REGS = 512                   # registers per lane of one SIMD, shared by the waves on it


def _code_objects():
    lib = open(pk.LIB_PATH, "rb").read()
    for at in (m.start() for m in re.finditer(MAGIC, lib)):
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", lib, pos - 8)[0]):
            offset, size, n = struct.unpack_from("<QQQ", lib, pos)
            triple = lib[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in triple:
                yield lib[at + offset:at + offset + size]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(name, template arguments) -> (registers per lane of one wave, of all waves of a workgroup on one SIMD)"""
    found = {}
    path = tmp_path_factory.mktemp("co") / "co.elf"
    for co in _code_objects():
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.name:\s+_ZN2pk\d+(\w+_kernel)I(.*)E+v", k)
            if not name:
                continue
            args = tuple(int(x) for x in re.findall(r"L[ib](\d+)E", name[2] + "E"))
            vgprs, threads = (int(re.search(r"\.%s:\s+(\d+)" % f, k)[1]) for f in ("vgpr_count", "max_flat_workgroup_size"))
            held = (vgprs + 7) // 8 * 8
            found[name[1], args] = held, held * ((threads + 255) // 256)
    return found


def _gemm(kernels, epilogues, fp8):
    """256-row and smaller GEMM kernels of these epilogues, without the stream-K tail: registers left beside a workgroup."""
    return {a: REGS - used for (name, a), (_, used) in kernels.items()
            if name == "gemm_kernel" and a[8] in epilogues and a[7] == fp8 and not a[10]}


@pytest.mark.parametrize("fp8,left", [(0, 80), (1, 48)])
def test_communicator_beside_an_all_gather_gemm(kernels, fp8, left):
    found = _gemm(kernels, (1, 3), fp8)                     # EPI_AG in both layouts of the second operand, EPI_AGK
    assert len(found) == 22 and min(found.values()) >= left, found


def test_reduce_beside_a_gemm(kernels):
    """Two launches (PK_PHASE_OVERLAP) are of tiles larger than 128x64; a reduce workgroup has one wave per SIMD."""
    reduce = {a: held for (name, a), (held, _) in kernels.items() if name == "reduce_kernel" and not a[2]}
    assert len(reduce) == 13
    for fp8 in (0, 1):
        for a, left in _gemm(kernels, (0, 2), fp8).items():
            if a[0] * a[1] < 128 * 128:
                continue
            for r, held in reduce.items():
                if r[1] == (a[8] == 2) and (not fp8 or r[3] or r[1] or r[0] == 0):
                    assert held <= left, (a, r, held, left)
