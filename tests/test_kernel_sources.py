"""Properties of the kernels' sources that a run cannot show reliably (CPU)."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_28670_amd", "csrc")


def test_lds_loads_wait_after_m0():
    """A direct-to-LDS load takes its LDS address from M0, and one wait state
    must lie between a scalar write of M0 and the load (the compiler puts an
    s_nop there when it writes both; inside inline assembly nobody does)."""
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        with open(path) as f:
            src = f.read()
        for text in re.findall(r'asm\s+volatile\s*\(\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', src):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', text))
            ops = [line.strip() for line in code.replace("\\t", " ").split("\\n")]
            for i, op in enumerate(ops):
                if re.match(r"(global|buffer)_load_lds", op):
                    found += 1
                    assert i > 0 and ops[i - 1].startswith("s_nop"), f"{os.path.basename(path)}: {code}"
    assert found >= 2      # the loads with per-lane addresses and with a uniform base
