"""Rules of the hardware that the compiler cannot keep inside inline assembly, checked in the kernels' sources."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _assembly_blocks():
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2308_09723_amd", "csrc", "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)+)", text):
            lines = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            yield os.path.basename(path), [s.strip() for s in re.split(r"\\n(?:\\t)?|;", lines) if s.strip()]


def test_loads_into_lds_wait_for_m0():
    """A load that takes its LDS address from M0 needs one wait state after the scalar write of M0: the instruction
    between them may be anything that is neither."""
    seen = 0
    for name, ins in _assembly_blocks():
        for i, s in enumerate(ins):
            if "_load_lds_" in s:
                seen += 1
                assert i > 0, f"{name}: M0 is written outside the block of '{s}'"
                assert not re.match(r"s_\w+\s+m0\b", ins[i - 1]), f"{name}: no wait state between '{ins[i - 1]}' and '{s}'"
    assert seen
