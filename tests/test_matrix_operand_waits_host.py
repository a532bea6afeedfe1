"""Matrix instructions written as asm, in the gfx950 assembly of the sources that have them: the compiler pads its own matrix instructions with the
wait states that their operands need and cannot see into asm, so every such source says its waits itself."""
import re
import subprocess

import pytest

from paper_2512_07710_amd.build import CSRC, FLAGS, HIPCC

WAIT_STATES = 2                    # between a vector-ALU write of a register and a matrix instruction that reads it
REGISTERS = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _registers(text):
    return {(bank, i) for bank, one, lo, hi in REGISTERS.findall(text) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)])}


def short_waits(assembly):
    """(kernel, writer, matrix instruction) wherever fewer than WAIT_STATES lie between the two, in the order of the text."""
    found, kernel, recent, products = [], None, [], 0          # recent: (wait states, registers written, text) of the last instructions
    for line in assembly.splitlines():
        text = line.split(";")[0].split("//")[0].strip()
        if text.endswith(":") and not text.startswith("."):
            kernel, recent = text[:-1], []
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        name, _, operands = text.partition(" ")
        if name.startswith("v_mfma"):
            products += 1
            reads, between = _registers(operands.split(",", 1)[1]), 0
            for states, written, writer in reversed(recent):
                if between >= WAIT_STATES:
                    break
                if written & reads:
                    found.append((kernel, writer, text))
                between += states
        vector = name.startswith("v_") and not name.startswith("v_mfma")
        recent.append((int(operands, 0) + 1 if name == "s_nop" else 1, _registers(operands.split(",")[0]) if vector else set(), text))
        del recent[:-4]
    return found, products


def test_the_search_finds_what_it_is_for():
    mfma = "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[96:99], v[4:7], a[0:15]\n"
    write = "\tv_cvt_pk_bf16_f32 v99, v1, v2\n"
    waits = [short_waits("k:\n" + write + between + mfma)[0] != [] for between in
             ("", "\ts_cmp_ge_i32 s0, s1\n", "\ts_nop 0\n", "\ts_nop 1\n", "\tv_mov_b32_e32 v1, v2\n\ts_cmp_ge_i32 s0, s1\n",
              "\tds_read_b128 v[8:11], v3\n\ts_nop 0\n")]
    assert waits == [True, True, True, False, False, False]
    assert short_waits("k:\n\tv_accvgpr_write_b32 a3, 0\n" + mfma)[0]
    assert not short_waits("k:\n\tglobal_load_dwordx4 v[96:99], v[0:1], off\n" + mfma)[0]


@pytest.mark.parametrize("source", ["route.hip", "ffn.hip", "probe.hip"])
def test_operands_from_the_vector_alu_have_their_wait_states(source, tmp_path):
    subprocess.run([HIPCC, *FLAGS, "--cuda-device-only", "-S", f"{CSRC}/{source}", "-o", str(tmp_path / "a.s")], check=True, capture_output=True)
    found, products = short_waits((tmp_path / "a.s").read_text())
    assert products > 0 and found == []
