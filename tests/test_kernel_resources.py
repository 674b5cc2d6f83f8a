"""Registers that the built kernels take, from the metadata of the code object in
libqo_hip.so: the forms of a kernel family that differ in a template argument are not all
timed, and a change that suits one can push another into spills or cost it workgroups per CU.

A CU's SIMD holds 512 registers per lane, so a kernel of up to 128 has four wavefronts per
SIMD (two 8-wave workgroups per CU), of up to 80 six.
"""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_25149_amd", "libqo_hip.so")
LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (vector registers, spilled vector registers)}"""
    for tool in ("llvm-objcopy", "llvm-readelf"):
        if not os.path.exists(f"{LLVM}/{tool}"):
            pytest.skip(f"{tool} not found")
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fat")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", LIB, str(d / "so")],
                   check=True)
    with open(fat, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(re.escape(MAGIC), data):
        (entries,) = struct.unpack_from("<Q", data, m.end())
        o = m.end() + 8
        for _ in range(entries):
            off, size, tl = struct.unpack_from("<QQQ", data, o)
            triple = data[o + 24:o + 24 + tl].decode()
            o += 24 + tl
            if "gfx950" not in triple:
                continue
            co = d / "co"
            co.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(co)], check=True,
                                   capture_output=True, text=True).stdout
            for k in notes.split(".agpr_count:")[1:]:
                def num(key, k=k):
                    return int(re.search(rf"\.{key}:\s+(\d+)", k).group(1))

                name = re.search(r"\.name:\s+(\S+)", k).group(1)
                out[name] = (num("vgpr_count"), num("vgpr_spill_count"))
    assert out
    return out


def _plane_forms(kernels):
    """(FP64, inverse, columns, whole 16-byte rows, p-forming, above 128 rows) -> registers, spills"""
    forms = {}
    for name, v in kernels.items():
        m = re.search(r"k_dst_planeI([fd])Lb([01])ELi(\d+)ELb([01])ELb([01])ELb([01])ELb([01])EE", name)
        if m:
            t, inv, nt, vec, pf, big, _ = m.groups()
            forms.setdefault((t == "d", inv == "1", 16 * int(nt), vec == "1", pf == "1",
                              big == "1"), []).append(v)
    assert len(forms) > 50
    return forms


def test_plane_pass_spills(kernels):
    for form, regs in _plane_forms(kernels).items():
        fp64, inv, cols, vec, pf, big = form
        for _, spilled in regs:
            assert spilled <= (48 if big else 1 if vec or cols <= 128 else 10), (form, regs)


def test_plane_pass_occupancy(kernels):
    """Planes of up to 128 rows: six wavefronts per SIMD up to 128 columns in FP32, two
    workgroups per CU for the forward passes above and for inverse passes up to 192."""
    for form, regs in _plane_forms(kernels).items():
        fp64, inv, cols, vec, pf, big = form
        if big:
            continue
        limit = 128 if cols > 128 or fp64 else 80
        if inv and (cols > 192 or (pf and cols > 160)):
            limit = 256
        for total, _ in regs:
            assert total <= limit, (form, regs)


@pytest.mark.parametrize("form,limit", [("k_pcg_sweep1IdLi8ELb0EE", 256), ("k_resid_relILi3EE", 128)])
def test_stencil_occupancy(kernels, form, limit):
    """The Jacobi first sweep of eight points per thread in FP64 keeps two wavefronts per SIMD,
    the residual replacement of three points four."""
    found = [v for name, v in kernels.items() if form in name]
    assert found and all(total <= limit and spilled == 0 for total, spilled in found), found


@pytest.mark.parametrize("form,limit", [("k_gram_f64ILi1ELb1EE", 300), ("k_gram_cross_f64ILi1EE", 316)])
def test_gram_registers(kernels, form, limit):
    """One-wavefront FP64 Gram kernels of many tiles: with more registers than these (128 of them
    for accumulation) the compiler moves accumulators in and out in every iteration."""
    found = [v for name, v in kernels.items() if form in name]
    assert found and all(total <= limit and spilled == 0 for total, spilled in found), found
