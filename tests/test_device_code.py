"""Properties of the gfx950 code of the library's own kernels that no numeric test shows reliably, read from the assembly
that the compiler prints for them (no GPU needed)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2301_12017_amd import build

# wait states between a matrix instruction and a vector instruction that reads its result: eight passes, and sixteen for
# the largest format of the scaled ones
WAIT, WAIT_F8F6F4 = 12, 19
_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """{source: lines} of every source with a matrix instruction."""
    out = tmp_path_factory.mktemp("asm")

    def compile_(src):
        dst = os.path.join(out, src + ".s")
        subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", dst],
                       check=True, stderr=subprocess.DEVNULL)
        with open(dst) as f:
            return src, f.read().splitlines()

    with ThreadPoolExecutor(max_workers=4) as ex:
        return dict(ex.map(compile_, [s for s in build.SOURCES if s.startswith("gemm_") or s == "attention.hip"]))


def _regs(text):
    out = set()
    for m in _REG.finditer(text):
        lo, hi = (int(m[2]), int(m[3])) if m[2] else (int(m[4]),) * 2
        out |= {(m[1], i) for i in range(lo, hi + 1)}
    return frozenset(out)


def _early_reads(lines):
    """Instructions of inline assembly that touch a matrix instruction's result before its wait states are over, on any
    path (each label takes over the state of every branch to it).  The compiler keeps them for its own instructions only."""
    bad, at = set(), {}
    for _ in range(3):                                            # branches backwards: again with what the last walk found
        pending, in_asm = {}, False                               # {(registers, line, wait states needed): passed}
        for number, line in enumerate(lines, 1):
            if "#ASMSTART" in line or "#ASMEND" in line:
                in_asm = "#ASMSTART" in line
                continue
            text = line.split(";")[0].strip()
            if text.endswith(":"):
                if text.startswith("_Z"):
                    pending = {}
                for key, age in at.get(text[:-1], {}).items():
                    pending[key] = min(age, pending.get(key, age))
                continue
            if not line.startswith("\t") or not text or text.startswith("."):
                continue
            op, _, rest = text.partition(" ")
            if in_asm and op.startswith("v_"):
                touched = _regs(rest)
                bad |= {(number, text) for (dst, _, _) in pending if dst & touched}
            step = int(rest) + 1 if op == "s_nop" else 1
            pending = {key: age + step for key, age in pending.items() if age + step < key[2]}
            if op.startswith("v_mfma"):
                pending[_regs(rest.split(",")[0]), number, WAIT_F8F6F4 if "f8f6f4" in op else WAIT] = 0
            if op.startswith("s_cbranch") or op == "s_branch":
                d = at.setdefault(rest.strip(), {})
                for key, age in pending.items():
                    d[key] = min(age, d.get(key, age))
                if op == "s_branch":
                    pending = {}
    return sorted(bad)


def test_inline_assembly_reads_no_matrix_result_too_early(assembly):
    found = {src: _early_reads(lines) for src, lines in assembly.items()}
    assert not any(found.values()), {src: f[:4] for src, f in found.items() if f}
    assert sum("v_mfma" in line for lines in assembly.values() for line in lines) > 1000


def _loose_barriers(lines):
    """(line, allowed, requested) of each barrier behind a wait that lets more memory requests stay in flight than were issued
    since the barrier before it, on the path with the fewest."""
    found, at = {}, {}
    for _ in range(4):
        issued, allowed = 0, None
        for number, line in enumerate(lines, 1):
            text = line.split(";")[0].strip()
            if text.endswith(":"):
                if text.startswith("_Z"):
                    issued = 0
                issued = min(issued, at.get(text[:-1], issued))
                continue
            if not line.startswith("\t") or not text or text.startswith("."):
                continue
            op, _, rest = text.partition(" ")
            if op.startswith(("buffer_", "global_", "scratch_")):
                issued += 1
            wait = re.search(r"vmcnt\((\d+)\)", rest) if op == "s_waitcnt" else None
            if wait and int(wait[1]) < 63:                        # (63: no wait)
                allowed = int(wait[1])
            if op == "s_barrier":
                if allowed is not None and allowed > issued:
                    found[number] = (number, allowed, issued)
                issued, allowed = 0, None
            if op.startswith("s_cbranch") or op == "s_branch":
                at[rest.strip()] = min(issued, at.get(rest.strip(), issued))
                if op == "s_branch":
                    issued = 1 << 30                              # nothing falls through to what follows
    return sorted(found.values())


def test_barriers_of_the_group_kernel_publish_what_has_landed(assembly):
    """Its K step requests the tiles of the step after next and reads, behind the barrier, those requested a step earlier: the
    wait in front of the barrier must not leave more in flight than this step has requested."""
    lines = assembly["gemm_group.hip"]
    assert not _loose_barriers(lines)
    assert sum(line.strip() == "s_barrier" for line in lines) > 100


def test_the_search_for_loose_barriers_finds_one():
    code = ["_Zkernel:", "\ts_barrier", ".L1:", "\tbuffer_load_dwordx4 v1, s[0:3], 0 offen lds", "\tbuffer_load_dword v2, v1, s[0:3], 0",
            "\ts_waitcnt vmcnt(2)", "\ts_barrier", "\ts_cbranch_scc1 .L1", "\ts_branch .L3", ".L3:"]
    assert not _loose_barriers(code)
    assert _loose_barriers([line.replace("vmcnt(2)", "vmcnt(3)") for line in code]) == [(7, 3, 2)]


def test_the_search_for_early_reads_finds_one():
    code = ["_Zkernel:", "\tv_mfma_f32_32x32x16_f16 v[34:49], v[82:85], v[66:69], 0", "\ts_cbranch_scc1 .L1",
            "\ts_nop 11", ".L1:", "\t;;#ASMSTART", "\tv_max3_f32 v82, v34, v35, v36", "\t;;#ASMEND"]
    assert _early_reads(code) == [(7, "v_max3_f32 v82, v34, v35, v36")]
    assert not _early_reads([line for line in code if "cbranch" not in line])
