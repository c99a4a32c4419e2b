"""Memory instructions in inline assembly.  The compiler knows neither the registers that assembly changes without naming
them nor the distances that an instruction inside it wants: a vector memory instruction may read an SGPR five wait states
after a vector instruction wrote it.  The sources have to name M0; the distances are read from the machine code that the
build made of them, for every load into LDS."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1802_04799_amd")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 5


def asm_statements():
    """(file, instructions, operands) of every asm statement."""
    for path in sorted(glob.glob(os.path.join(ROOT, "csrc", "*"))):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"asm\s+volatile\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)+)(.*?)\)\s*;", text, re.S):
            template = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            yield os.path.basename(path), [l.strip() for l in template.replace("\\t", "").split("\\n")], m.group(2)


def test_assembly_that_changes_m0_names_it():
    found = 0
    for name, lines, operands in asm_statements():
        if any(re.match(r"s_\w+ m0\b", l) for l in lines):
            found += 1
            assert '"={m0}"' in operands, (name, lines)
    assert found >= 2


def scalar_registers(operand):
    """The SGPRs of one operand: s7, s[4:7], vcc."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


class Function:
    """Instructions of one kernel in order: (address, mnemonic, operands), and the branches to an instruction."""

    def __init__(self):
        self.code, self.jumps = [], {}

    def add(self, address, mnemonic, operands, target):
        if target is not None:
            self.jumps.setdefault(target, []).append(len(self.code))
        self.code.append((address, mnemonic, operands))

    def near_writes(self, i, wanted, left=WAIT_STATES, seen=None):
        """Vector instructions that write a wanted SGPR less than `left` wait states before instruction i, on every path."""
        found, seen = [], set() if seen is None else seen
        if (i, left) in seen:
            return found
        seen.add((i, left))
        before = [] if i == 0 or self.code[i - 1][1] in ("s_branch", "s_endpgm") else [i - 1]
        for j in before + self.jumps.get(self.code[i][0], []):
            _, mnemonic, operands = self.code[j]
            if mnemonic.startswith("v_") and operands and scalar_registers(operands[0]) & wanted:
                found.append(self.code[j])
            states = 1 + int(operands[0]) if mnemonic == "s_nop" else 1
            if states < left:
                found += self.near_writes(j, wanted, left - states, seen)
        return found


def functions(text):
    """Kernels of a listing with addresses in a comment behind each instruction and branch targets as <symbol+0xoffset>."""
    result, start, name = {}, 0, None
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(.+)>:", line)
        if m:
            start, name = int(m.group(1), 16), m.group(2)
            result[name] = Function()
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<([^>+]+)(?:\+0x([0-9a-f]+))?>)?$", line)
        if name and m:
            target = start + int(m.group(5) or "0", 16) if m.group(4) == name else None
            result[name].add(int(m.group(3), 16), m.group(1), [o for o in re.split(r",\s*|\s+", m.group(2)) if o], target)
    return result


def test_distances_are_found_on_every_path():
    text = """0000000000000100 <kernel>:
	v_readlane_b32 s5, v1, 3                                   // 000000000100: D2890005
	s_nop 4                                                    // 000000000104: BF800004
	buffer_load_dword v2, s[4:7], 0 offen lds                  // 000000000108: E0511000
	v_cmp_gt_u32_e64 s[2:3], s4, v0                            // 000000000110: D0CC0002
	s_cbranch_vccnz 2                                          // 000000000118: BF870002 <kernel+0x24>
	v_readfirstlane_b32 s9, v0                                 // 00000000011C: 7E120500
	v_mov_b32_e32 v3, 0                                        // 000000000120: 7E060280
	s_nop 0                                                    // 000000000124: BF800000
	s_mov_b32 m0, s8                                           // 000000000128: BEFC0008
	buffer_load_dwordx4 v2, v4, s[4:7], s9 offen lds           // 00000000012C: E05D1000
"""
    f = functions(text)["kernel"]
    assert not f.near_writes(2, {4, 5, 6, 7})                      # five states between: far enough
    assert [c[1] for c in f.near_writes(9, {9})] == ["v_readfirstlane_b32"]
    assert [c[1] for c in f.near_writes(9, {2})] == ["v_cmp_gt_u32_e64"]      # by the branch; falling through there are five


def test_sgprs_of_loads_into_lds_are_old_enough(tmp_path):
    """In the machine code of the built library."""
    library = os.path.join(ROOT, "libtvg.so")
    if not os.path.exists(OBJDUMP) or not os.path.exists(library):
        pytest.skip("needs the built library and its disassembler")
    shutil.copy(library, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    loads = 0
    for path in sorted(tmp_path.glob("lib.so.*gfx950*")):
        symbols = subprocess.run([OBJDUMP, "--syms", str(path)], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"\sF \.text\s+\S+\s+(?:\.\w+\s+)?(\S*conv3x3_strips_kernel\S*)$", symbols, re.M)
        if not names:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f"--disassemble-symbols={','.join(names)}", str(path)],
                              check=True, capture_output=True, text=True).stdout
        for name, f in functions(text).items():
            for i, (_, mnemonic, operands) in enumerate(f.code):
                if mnemonic.startswith("buffer_load") and operands[-1] == "lds":
                    loads += 1
                    wanted = set().union(*(scalar_registers(o) for o in operands))
                    assert wanted and not f.near_writes(i, wanted), (name, f.code[max(0, i - 6):i + 1])
    assert loads >= 25 * 18                                        # 25 instances, two times nine loads and more
