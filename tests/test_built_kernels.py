"""Properties of the built kernels that results do not show, read from the library's own gfx950 code: wait states between
a vector write and a DPP read of it in the sweep of narrow networks, whose multiply-adds are assembly that the
compiler does not look into; and how many workgroups of the matrix-core sweeps a compute unit holds."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_1906_08879_amd as pl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_08879_amd", "csrc")
LLVM = "/opt/rocm/llvm/bin"
needs_llvm = pytest.mark.skipif(shutil.which("llvm-objdump", path=LLVM) is None, reason="needs ROCm's llvm tools")


def _tool(name, *args):
    return subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of libplaceto.so, one file per source."""
    if not os.path.exists(pl.library_path()):
        from paper_1906_08879_amd.build import build
        build()
    tmp = tmp_path_factory.mktemp("code")
    fat = str(tmp / "fat")
    _tool("llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", pl.library_path(), str(tmp / "copy.so"))
    data, out, magic = open(fat, "rb").read(), [], b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            offset, size, name_len = struct.unpack_from("<QQQ", data, p)
            if size and b"gfx950" in data[p + 24:p + 24 + name_len]:
                out.append(str(tmp / f"{len(out)}.elf"))
                with open(out[-1], "wb") as f:
                    f.write(data[at + offset:at + offset + size])
            p += 24 + name_len
        at = data.find(magic, at + len(magic))
    assert out, "the library holds no gfx950 code"
    return out


def _vector_registers(operand):
    m = re.fullmatch(r"v(\d+)|v\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    lo = int(m[1] or m[2])
    return set(range(lo, int(m[3] or lo) + 1))


def _instructions(code_object, kernel):
    """(function, mnemonic, operands) of every instruction of the functions whose name holds `kernel`."""
    name = None
    for line in _tool("llvm-objdump", "-d", "--no-show-raw-insn", code_object).splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            name = m[1]
            continue
        if name is None or kernel not in name:
            continue
        text = line.split("//")[0].strip()
        if text:
            mnemonic, _, rest = text.partition(" ")
            yield name, mnemonic, [x.strip() for x in rest.split(",")]


@needs_llvm
def test_dpp_reads_have_their_wait_states(code_objects):
    """A DPP operand that the vector unit wrote needs two wait states (instructions count one, s_nop N counts N + 1)."""
    reads = 0
    for obj in code_objects:
        if "k_sweep_lanes" not in _tool("llvm-readelf", "--symbols", "--wide", obj):
            continue
        last, recent = None, []                    # recent: (registers written, wait states since)
        for name, mnemonic, ops in _instructions(obj, "k_sweep_lanes"):
            if name != last:
                last, recent = name, []
            if mnemonic.endswith("_dpp"):
                reads += 1
                source = _vector_registers(ops[1].split()[0])
                assert source and not any(source & w for w, age in recent if age < 2), (name, mnemonic, ops)
            states = int(ops[0], 0) + 1 if mnemonic == "s_nop" else 1
            recent = [(w, age + states) for w, age in recent if age + states < 2]
            if mnemonic.startswith("v_") and not mnemonic.startswith("v_cmp"):
                written = _vector_registers(ops[0])
                if "swap" in mnemonic:
                    written |= _vector_registers(ops[1])
                recent.append((written, 0))
    assert reads > 1000, "no DPP instructions found: the kernels or the listing changed"


def test_no_dpp_sum_leans_on_the_statement_before_it():
    """Every statement of DPP multiply-adds begins with its own wait states: nothing keeps the compiler from writing an
    input between two statements."""
    text = open(os.path.join(CSRC, "kernels_lanes.hip")).read()
    statements = [re.sub(r"\s+", " ", t).strip() for t in re.findall(r"\basm volatile\((.*?)\);", text, flags=re.S)]
    sums = [t for t in statements if "PL_MAC" in t or "_dpp" in t]
    assert len(sums) >= 4
    for t in sums:
        assert t.startswith('"s_nop 1\\n"'), t[:80]


def _kernels(code_object, kernel):
    """(template arguments, vector registers, bytes of scratch) of the code object's kernels of that name."""
    for entry in _tool("llvm-readelf", "--notes", code_object).split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", entry)[1]
        args = re.search(kernel + r"I((?:L[ib]\d+E)+)E", name)
        if args:
            yield ([int(x) for x in re.findall(r"L[ib](\d+)E", args[1])], int(re.search(r"\.vgpr_count:\s+(\d+)", entry)[1]),
                   int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry)[1]))


# (H, parts per weight, layers) -> waves per SIMD of a first sweep, a later sweep and the reverse pass
WAVES = {(64, 3, 2): (2, 2, 2), (64, 1, 2): (3, 3, 3), (64, 3, 1): (2, 3, 3), (64, 1, 1): (3, 4, 4),
         (32, 3, 2): (2, 3, 3), (32, 1, 2): (3, 4, 3), (32, 3, 1): (3, 3, 3), (32, 1, 1): (3, 4, 4)}


@needs_llvm
def test_sweeps_on_matrix_cores_keep_their_residency(code_objects):
    """A SIMD's 512 registers, handed out in eights, hold as many waves of every variant as a batch is dispatched for,
    and nothing is spilled."""
    seen = set()
    for obj in code_objects:
        for (H, WS, L, first, _, reverse, _), registers, scratch in _kernels(obj, "k_sweep_tiles"):
            want = WAVES[(H, WS, L)][0 if first else (2 if reverse else 1)]
            waves = 512 // (-(-registers // 8) * 8)
            assert waves >= want and scratch == 0, (H, WS, L, first, reverse, registers, scratch)
            seen.add((H, WS, L))
    assert seen == set(WAVES)


@needs_llvm
def test_wide_sweep_fits_a_compute_unit(code_objects):
    """Eight waves of every variant of the sweep of 128 columns, two to a SIMD, without spills."""
    seen = 0
    for obj in code_objects:
        for args, registers, scratch in _kernels(obj, "k_sweep_wide"):
            assert registers <= 256 and scratch == 0, (args, registers, scratch)
            seen += 1
    assert seen == 12
