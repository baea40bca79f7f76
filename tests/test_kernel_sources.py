"""Properties of the kernels' sources, and of the gfx950 assembly they compile
to, that a run cannot show reliably (CPU)."""
import glob
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2608_28670_amd import build

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


class Kernel:
    """One kernel of a listing: its instructions (labels included) and resources."""

    def __init__(self):
        self.code, self.vgprs, self.spills, self.lds = [], None, None, None


def _listing(source, tmp):
    """{mangled name: Kernel} of one HIP source, compiled as the library is."""
    out = os.path.join(str(tmp), source + ".s")
    build._run([build._hipcc(), *build.HIP_FLAGS, "-I", CSRC, "-I", build.INCLUDE, "--cuda-device-only", "-S",
                os.path.join(CSRC, source), "-o", out])
    with open(out) as f:
        text = f.read()
    kernels, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = kernels.setdefault(m.group(1), Kernel())
        if line.startswith(".Lfunc_end"):
            cur = None
        t = line.split(";")[0].strip()
        if cur is not None and t and not (t.startswith(".") and not t.endswith(":")):
            cur.code.append(t)
    for m in re.finditer(r"\.group_segment_fixed_size: (\d+)(?:(?!\.group_segment).)*?\.name:\s+(\S+)(?:(?!\.group_segment).)*?"
                         r"\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count: (\d+)", text, re.S):
        k = kernels[m.group(2)]
        k.lds, k.vgprs, k.spills = int(m.group(1)), int(m.group(3)), int(m.group(4))
    return kernels


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """The sources with direct-to-LDS loads, compiled side by side."""
    tmp = tmp_path_factory.mktemp("listings")
    names = ("gemm.hip", "attention.hip", "ops.hip")
    with ThreadPoolExecutor(len(names)) as ex:
        return dict(zip(names, ex.map(lambda n: _listing(n, tmp), names)))


@pytest.fixture(scope="module")
def ops_listing(listings):
    return listings["ops.hip"]


@pytest.fixture(scope="module")
def attention_listing(listings):
    return listings["attention.hip"]


def _template_args(name, kernel):
    """The integer template arguments of an instantiation, or None for another kernel."""
    if kernel + "I" not in name:
        return None
    return [int(v) for v in re.findall(r"L[ib](\d+)E", name.split(kernel, 1)[1].split("EEv")[0] + "E")]


def test_weight_stream_keeps_its_ring_filled(ops_listing):
    """The conditioning linear's weight stream has S stages of two loads; its
    steady state waits for the oldest only: S - 1 stages stay on their way."""
    found = 0
    for name, k in ops_listing.items():
        t = _template_args(name, "skinny_stream_kernel")
        if not t:
            continue
        found += 1
        waits = {int(m.group(1)) for c in k.code for m in [re.match(r"s_waitcnt.*vmcnt\((\d+)\)", c)] if m}
        assert 2 * (t[1] - 1) in waits, (name, sorted(waits))
    assert found == 3


def test_weight_stream_workgroups_are_resident(ops_listing):
    """The weight stream's grid is one round of the workgroups that the
    launcher takes a CU to hold (the third template argument): registers (512
    a SIMD, in eights) and LDS (160 KB) must allow them."""
    found = 0
    for name, k in ops_listing.items():
        t = _template_args(name, "skinny_stream_kernel")
        if not t:
            continue
        found += 1
        assert len(t) == 3 and k.spills == 0, (name, k.spills)
        waves_per_simd = 512 // (-(-k.vgprs // 8) * 8)
        assert min(4 * waves_per_simd // 8, 160 * 1024 // k.lds) == t[2], (name, k.vgprs, k.lds)
    assert found == 3


def test_resident_attention_sets_up_before_its_wait(attention_listing):
    """Between the wait for the resident key tiles and the key loop lies no
    load of an argument, and (d = 72 apart) none of the set-up that needs no
    keys: accumulators, operand addresses."""
    found = 0
    for name, k in attention_listing.items():
        t = _template_args(name, "attention_dma_kernel")      # d, QG, waves, buffers, STREAM, QS, QKV
        if not t or t[4] or t[6] or t[0] == 72:
            continue
        found += 1
        at = max(i for i, c in enumerate(k.code) if c == "s_barrier")
        setup = []
        for c in k.code[at + 1:]:
            if c.endswith(":"):
                break
            setup.append(c)
        assert not any(c.startswith("s_load") for c in setup), (name, setup)
        assert len(setup) <= 16, (name, len(setup))
    assert found == 9


def test_resident_attention_stores_its_rows_without_branches(attention_listing):
    """One 8-byte store per query group and 16-row block of the output, with no second form of it."""
    found = 0
    for name, k in attention_listing.items():
        t = _template_args(name, "attention_dma_kernel")
        if not t or t[4]:
            continue
        found += 1
        stores = [c.split()[0] for c in k.code if c.startswith("global_store")]
        assert stores == ["global_store_dwordx2"] * (t[1] * -(-t[0] // 16)), (name, stores)
    assert found == 15


def _sgprs(text):
    out = set()
    for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out |= {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))
    return out


def test_lds_loads_wait_for_their_base(listings):
    """A vector memory instruction may read a scalar register that a vector
    instruction wrote (a base made uniform by v_readfirstlane) five wait states
    later at the earliest.  The compiler sees to it for its own instructions,
    not inside inline assembly, so the compiled code is looked at."""
    loads = 0
    for kernels in listings.values():
        for name, k in kernels.items():
            state, written = 0, {}          # wait states passed, scalar register -> state after its vector write
            for c in k.code:
                op, _, args = c.partition(" ")
                if c.endswith(":"):
                    continue
                if op.startswith("global_load_lds"):
                    loads += 1
                    for r in _sgprs(args):
                        assert state - written.get(r, -5) >= 5, (name, c)
                state += 1 + (int(args, 0) if op == "s_nop" else 0)
                if op.startswith("v_"):
                    for r in _sgprs(args.split(",")[0]):
                        written[r] = state
                elif op.startswith("s_"):
                    for r in _sgprs(args.split(",")[0]):
                        written.pop(r, None)
    assert loads > 1000
