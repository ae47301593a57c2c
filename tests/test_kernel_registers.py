"""Register allocation of the GEMM kernels, from the metadata of the library as built here.  Their MFMAs are assembler
statements on ACC registers, whose wait states the compiler does not know: it must never put anything else there (a fragment
that finds no VGPR, moved through an ACC register in front of an MFMA, gave wrong bits), nor spill."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_12526_amd", "libmom.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def forms(name):
    """The argument tuples of a list of forms in the header, in its order."""
    text = open(os.path.join(ROOT, "paper_2504_12526_amd", "csrc", "mom_gemm_forms.h")).read()
    listed = re.search(r"#define " + name + r"\(X\)((?:.*\\\n)*.*\n)", text)[1]
    return [tuple(int(v) for v in f.split(",")) for f in re.findall(r"X\(([\d, ]+)\)", listed)]


def _code_object():
    """The gfx950 code object in the library: a bundle is a magic, the number of entries, and for each its offset from
    the magic, size and target."""
    data = open(LIB, "rb").read()
    at = data.index(MAGIC)
    n, = struct.unpack_from("<Q", data, at + 24)
    p = at + 32
    for _ in range(n):
        offset, size, length = struct.unpack_from("<QQQ", data, p)
        target = data[p + 24:p + 24 + length]
        p += 24 + length
        if b"gfx950" in target:
            return data[at + offset:at + offset + size]
    raise AssertionError("no gfx950 code object")


def _kernels(tmp_path):
    co = os.path.join(str(tmp_path), "mom.co")
    with open(co, "wb") as f:
        f.write(_code_object())
    notes = subprocess.run([READELF, "--notes", co], capture_output=True, text=True, check=True).stdout
    found = {}
    for block in notes.split("  - .agpr_count:")[1:]:
        v = {k: int(x) for k, x in re.findall(r"\.(vgpr_count|vgpr_spill_count|sgpr_spill_count|private_segment_fixed_size):\s+(\d+)", block)}
        v["agpr"] = int(block.split()[0])
        found[re.search(r"\.name:\s+(\S+)", block)[1]] = v
    return found


def accumulators(name):
    """ACC registers of the accumulator blocks of a GEMM kernel, by its template arguments; None: another kernel."""
    m = re.search(r"17gemm_short_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
    if m:
        _, tm, tn, wm, wn = map(int, m.groups())
        return 4 * (tm // 16 // wm) * (tn // 16 // wn)
    m = re.search(r"12gemm4_kernelILi\d+ELi(\d+)ELi(\d+)E", name)
    if m:
        return 4 * (int(m[1]) // 32) * (int(m[2]) // 32)
    return 4 * 8 * 8 if "gemm4_two_width_kernel" in name else None


def unsound(kernels):
    return [(n, v) for n, v in kernels.items() if accumulators(n) is not None and
            (v["agpr"] != accumulators(n) or v["vgpr_spill_count"] or v["sgpr_spill_count"] or v["private_segment_fixed_size"])]


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
def test_acc_registers_hold_the_accumulators_and_nothing_else(tmp_path):
    if not os.path.exists(LIB):
        from paper_2504_12526_amd import build
        build.build()
    kernels = _kernels(tmp_path)
    gemms = [n for n in kernels if accumulators(n) is not None]
    short = [tuple(int(x) for x in m.groups()) for n in gemms
             if (m := re.search(r"17gemm_short_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", n))]
    # (projection, form, non-temporal weights): every form of the lists, and no other
    want = [(0, *f, 0) for f in forms("MOM_SHORT_FORMS_DOWN")] + [(1, *f, nt) for f in forms("MOM_SHORT_FORMS_GATEUP") for nt in (0, 1)]
    assert sorted(short) == sorted(want)
    # 256-row tiles: five widths down, two of gate/up with and without; 128-row gate/up tiles; the two widths in one launch
    assert len(gemms) - len(short) == 5 + 2 * 2 + 1 + 2, gemms
    assert not unsound(kernels), unsound(kernels)
    # the check sees one register too many, and a spill
    for key in ("agpr", "vgpr_spill_count"):
        planted = {gemms[0]: dict(kernels[gemms[0]], **{key: kernels[gemms[0]][key] + 4})}
        assert unsound(planted)


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
def test_a_reload_finds_registers_beside_every_gemm_workgroup(tmp_path):
    """A SIMD has 512 registers per lane, allocated in eights, and a GEMM workgroup one wavefront on each; the reload kernel needs no LDS."""
    allocated = {n: -(-v["vgpr_count"] // 8) * 8 for n, v in _kernels(tmp_path).items()}
    reload, = [v for n, v in allocated.items() if "kv_reload_kernel" in n]
    gemms = {n: v for n, v in allocated.items() if re.search(r"gemm_short_kernel|gemm_rect_kernel|gemm4_", n)}
    assert len(gemms) > 100
    crowded = {n: v for n, v in gemms.items() if v + reload > 512}
    assert not crowded, (reload, crowded)
