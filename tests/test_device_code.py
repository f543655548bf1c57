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


def instructions(obj):
    for line in subprocess.Popen([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--no-leading-addr",
                                  obj], stdout=subprocess.PIPE, text=True).stdout:
        line = line.split("//")[0].strip()
        if line and not line.endswith(":"):
            yield line


def registers(operand):
    """Scalar register numbers of s5 or s[4:5]."""
    if operand.startswith("s["):
        lo, _, hi = operand[2:-1].partition(":")
        return set(range(int(lo), int(hi or lo) + 1))
    return {int(operand[1:])} if operand[1:].isdigit() and operand[0] == "s" else set()


def test_lds_dma_loads_wait_for_their_scalars(objects):
    """The loads are inline assembly, around which the compiler adds no wait states: one between a
    scalar write of M0 (the LDS address) and the load, five between a vector instruction's write of
    a scalar register and a load that reads it as its address."""
    loads = 0
    for obj in objects:
        last = []  # (instruction, wait states it gives by itself)
        for ins in instructions(obj):
            op, _, rest = ins.partition(" ")
            args = [a.strip() for a in rest.split(",")]
            if op.startswith("global_load_lds"):
                loads += 1
                reads = set().union(*(registers(a) for a in args))
                states = 0
                for p_op, p_args, given in reversed(last):
                    if p_op.startswith("s_") and p_args[0] == "m0":
                        assert states >= 1, f"{p_op} {p_args} directly before {ins}"
                    if p_op.startswith("v_") and reads & registers(p_args[0]):
                        assert states >= 5, f"{p_op} {p_args} before {ins}"
                    states += given
            given = 1 + int(args[0], 0) if op == "s_nop" else 1
            last = (last + [(op, args, given)])[-6:]
    assert loads > 10000
