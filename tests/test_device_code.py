"""What the compiler made of the kernels whose speed or safety rests on it: resources and
instructions, read from the library built here (no GPU needed)."""
import os
import struct
import subprocess

import pytest

H = pytest.importorskip("paper_2306_11987_amd", reason="libhqlss.so not built")

LLVM = "/opt/rocm/llvm/bin"


def code_objects(tmp):
    """The gfx950 code objects of the library: one in each of its offload bundles."""
    data = open(H._binding.LIB_PATH, "rb").read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := data.find(magic, at)) >= 0:
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, ids = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + ids]
            p += 24 + ids
            if b"gfx950" in name and size:
                out.append(os.path.join(tmp, f"{len(out)}.co"))
                with open(out[-1], "wb") as f:
                    f.write(data[at + off:at + off + size])
        at += 24
    assert out, "no gfx950 code object found"
    return out


def llvm(tool, *args):
    return subprocess.run([os.path.join(LLVM, tool), *args], check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    return code_objects(str(tmp_path_factory.mktemp("co")))


@pytest.fixture(scope="module")
def resources(objects):
    """(mangled name, registers, bytes of private memory) of every kernel."""
    out, cur = [], {}
    for o in objects:
        for line in llvm("llvm-readelf", "--notes", o).splitlines():
            key, _, val = line.strip().lstrip("- ").partition(":")
            if key in ("private_segment_fixed_size", "symbol", "vgpr_count"):
                raise AssertionError("unexpected note layout")
            if key in (".private_segment_fixed_size", ".symbol", ".vgpr_count"):
                cur[key] = val.strip().strip("'")
            if len(cur) == 3:
                out.append((cur[".symbol"], int(cur[".vgpr_count"]), int(cur[".private_segment_fixed_size"])))
                cur = {}
    assert len(out) > 100 and not cur
    return out


def kernels(resources, name):
    got = [r for r in resources if name in r[0]]
    assert got, name
    return got


def test_sampler_state_stays_in_registers(resources):
    """One wave's chain of dependent rounds bounds the sampler: a state in private memory puts a
    store and a load into every round of it."""
    for sym, _, private in kernels(resources, "lss_plan_kernel"):
        assert private == 0, sym


def test_bit_split_runs_three_workgroups_a_cu(resources):
    """Its workgroups put two waves on each SIMD; six waves of at most 80 registers fit."""
    for sym, vgprs, private in kernels(resources, "bit_split_kernel"):
        assert vgprs <= 80 and private == 0, (sym, vgprs)


def test_quantiser_runs_three_workgroups_a_cu(resources):
    """The 16-bit types; fp32 holds two (its raw data takes twice the registers)."""
    for sym, vgprs, private in kernels(resources, "fwht_quant_kernel"):
        assert private == 0, sym
        if "ILi0E" not in sym:  # the first template argument: fp32
            assert vgprs <= 80, (sym, vgprs)
