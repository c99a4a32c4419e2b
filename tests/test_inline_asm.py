"""Memory instructions in inline assembly, read from the sources.  The compiler knows neither the registers that assembly
changes without naming them nor the distances that an instruction inside it wants: a vector memory instruction may read an
SGPR five wait states after a vector instruction wrote it, and takes its LDS address from M0."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1802_04799_amd", "csrc")
WAIT_STATES = 5


def asm_statements():
    """(file, instructions, operands) of every asm statement."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"asm\s+volatile\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)+)(.*?)\)\s*;", text, re.S):
            template = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            yield os.path.basename(path), [l.strip() for l in template.replace("\\t", "").split("\\n")], m.group(2)


def wait_states(lines):
    """Of the lines before an instruction: one each, and n more for s_nop n."""
    return sum(1 + (int(l.split()[1]) if l.startswith("s_nop") else 0) for l in lines if l)


def test_memory_instructions_in_assembly_keep_their_distance_and_name_m0():
    found = 0
    for name, lines, operands in asm_statements():
        for i, line in enumerate(lines):
            if not re.match(r"(buffer|global|flat|scratch)_(load|store|atomic)", line):
                continue
            found += 1
            assert wait_states(lines[:i]) >= WAIT_STATES, (name, lines)
            assert not line.endswith(" lds") or '"{m0}"' in operands, (name, lines)
        assert not any(re.match(r"s_\w+ m0\b", l) for l in lines), (name, "M0 changed behind the compiler's back", lines)
    assert found >= 2
