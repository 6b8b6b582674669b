"""What the compiler does not see inside inline assembly.  m0 (LDS-direct loads take their address from it) is left as it was:
the register is reserved to the compiler, which neither saves it nor heeds a clobber.  A scalar operand that a vector
instruction has just written may be read by a memory instruction five wait states later only; the compiler counts them
for its own instructions."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_02199_amd", "csrc")


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(\s*\"(.*?)\"\s*:", open(path).read(), re.S):
            yield os.path.basename(path), [i.strip() for i in m.group(1).split("\\n\\t")]


def test_writes_of_m0_are_taken_back():
    found = 0
    for name, lines in statements():
        writes = [i for i in lines if re.match(r"s_\w+\s+m0\s*,", i)]
        if not writes:
            continue
        found += 1
        saved = re.fullmatch(r"s_mov_b32 (%\d), m0", lines[0])
        assert saved and lines[-1] == f"s_mov_b32 m0, {saved.group(1)}", f"{name}: {lines}"
    assert found


def test_loads_wait_for_scalars_from_vector_instructions():
    found = 0
    for name, lines in statements():
        for at, line in enumerate(lines):
            if not re.match(r"(buffer|global|flat|scratch)_", line):
                continue
            found += 1
            waits = sum(1 + (int(i.split()[1]) if i.startswith("s_nop") else 0) for i in lines[:at])
            assert waits >= 5, f"{name}: {lines}"
    assert found
