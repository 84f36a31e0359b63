"""Host checks of the compiled kernels: the gfx950 code of the built library,
disassembled.

  * No 64-bit vector shift takes its amount from a vector register: one with its amount
    in the last register of the wave's allocation returned wrong words (csrc/modarith.hpp,
    shr128), and which register the compiler picks cannot be chosen in the source.
  * The kernels of the external product load, rotate and decompose their operands
    without divergent branches: a branch per element puts each load's latency after
    the one before (a CMux step of 1000 ciphertexts of 2^8, 50-bit: 9.6 us so, 11.8
    with branches).
  * The matrix-core basis conversions keep their constants in registers.
"""
import os
import re
import shutil
import subprocess

import pytest

import paper_2410_05934_amd as ntt

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """Paths of the library's gfx950 code objects."""
    tool = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(tool) or not os.path.exists(ntt.library_path()):
        pytest.skip("needs the built library and llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(ntt.library_path(), d / "libntt.so")
    subprocess.run([tool, "--offloading", lib], check=True, capture_output=True, cwd=d)
    return [str(d / p) for p in sorted(os.listdir(d)) if "gfx950" in p]


@pytest.fixture(scope="module")
def kernels(objects):
    """[(symbol, [instruction, ...]), ...] of every device function."""
    out = []
    for path in objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn",
                               "--no-leading-addr", path], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"^(?=<\S+>:$)", text, flags=re.M)[1:]:
            head, *body = part.splitlines()
            out.append((head.strip("<>:"), [ln.split("//")[0].strip() for ln in body]))
    assert len(out) > 500
    return out


def test_no_64_bit_shift_by_a_vector_register(kernels):
    shift = re.compile(r"v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S* v\[\d+:\d+\], (v\d+),")
    seen = 0
    for name, body in kernels:
        for ln in body:
            seen += "rev_b64" in ln
            assert not shift.match(ln), (name, ln)
    assert seen > 1000  # shifts by constants and scalars: the pattern's mnemonics are the compiler's


def test_external_product_operands_load_without_branches(kernels):
    found = [(n, sum(ln.startswith(("s_and_saveexec", "s_andn2_saveexec")) for ln in body))
             for n, body in kernels if "xprod_kernel" in n]
    assert len(found) >= 81  # 9 lengths, 3 operand kinds, 3 classes
    # a few per kernel (the store of the slots that hold a column), none per element
    # of a thread's 8 or 16
    assert [f for f in found if f[1] >= 8] == []


def test_matrix_basis_conversion_keeps_its_constants_in_registers(objects):
    """The weights-stationary kernels hold every constant operand in registers; with 24
    k-steps ModDown has a few words of scratch (20 bytes over 64-bit words: 109 us on 48 + 48 limbs of
    4 x 2^16; at 36 bytes 128)."""
    seen = 0
    for path in objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True,
                               capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S*bconv_ws_kernel\S*)\s.*?\.private_segment_fixed_size:\s+(\d+)",
                                     notes, flags=re.S):
            seen += 1
            assert int(size) <= (28 if "Li24E" in name else 0), (name, size)
    assert seen == 48  # 2 word widths, 4 sizes, 2 pairs per helper thread, 3 modes
