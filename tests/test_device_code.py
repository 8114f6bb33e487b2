"""Properties of the gfx950 code of the library's own kernels that no numeric test shows reliably, read from the assembly
that the compiler prints for them (no GPU needed)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2301_12017_amd import build

# Wait states that the compiler keeps between an instruction and a vector instruction that reads its result, and does not keep
# where one of the two stands in inline assembly: behind a matrix instruction (eight passes, and sixteen for the largest format of
# the scaled ones), behind a transcendental, and from a vector instruction to a matrix, cross-lane or swap instruction.
WAIT, WAIT_F8F6F4, WAIT_TRANS, WAIT_ASM = 12, 19, 1, 2
_TRANS = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")
_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """{source: lines} of every source with kernels that compute."""
    out = tmp_path_factory.mktemp("asm")

    def compile_(src):
        dst = os.path.join(out, src + ".s")
        subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", dst],
                       check=True, stderr=subprocess.DEVNULL)
        with open(dst) as f:
            return src, f.read().splitlines()

    with ThreadPoolExecutor(max_workers=4) as ex:
        return dict(ex.map(compile_, [s for s in build.SOURCES if s not in ("api.hip", "gemm.hip", "strategy.hip", "probe.hip")]))


def _regs(text):
    out = set()
    for m in _REG.finditer(text):
        lo, hi = (int(m[2]), int(m[3])) if m[2] else (int(m[4]),) * 2
        out |= {(m[1], i) for i in range(lo, hi + 1)}
    return frozenset(out)


def _early_reads(lines):
    """Instructions that read a register before the wait states behind its writer are over, where the reader or the writer is
    inline assembly, on any path (each label takes over the state of every branch to it)."""
    bad, at = set(), {}
    for _ in range(3):                                            # branches backwards: again with what the last walk found
        pending, in_asm = {}, False                               # {(registers, line, wait states needed, by assembly): passed}
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
            dst, _, src = rest.partition(",")
            if op.startswith("v_"):
                slow = op.startswith(("v_mfma", "v_permlane")) or "dpp" in op or "row_" in rest or "quad_perm" in rest
                touched, read = _regs(rest), _regs(src if op.startswith("v_mfma") else rest)
                bad |= {(number, text) for (reg, _, _, by_asm) in pending
                        if (not by_asm and in_asm and reg & touched) or (by_asm and slow and reg & read)}
            step = int(rest) + 1 if op == "s_nop" else 1
            pending = {key: age + step for key, age in pending.items() if age + step < key[2]}
            if op.startswith("v_mfma"):
                pending[_regs(dst), number, WAIT_F8F6F4 if "f8f6f4" in op else WAIT, False] = 0
            elif op.startswith(_TRANS):
                pending[_regs(dst), number, WAIT_TRANS, False] = 0
            elif in_asm and op.startswith("v_"):
                pending[_regs(dst), number, WAIT_ASM, True] = 0
            if op.startswith("s_cbranch") or op == "s_branch":
                d = at.setdefault(rest.strip(), {})
                for key, age in pending.items():
                    d[key] = min(age, d.get(key, age))
                if op == "s_branch":
                    pending = {}
    return sorted(bad)


def test_inline_assembly_keeps_wait_states(assembly):
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


def test_fp16_stores_of_the_operand_layout_round_once(assembly):
    """Its epilogue ends in a fused multiply-add whose result goes to fp16.  Left to the compiler, most pairs become instructions that
    round once and some (which ones depends on the tile) a fp32 instruction and a conversion, which rounds twice."""
    lines = assembly["gemm_olay.hip"]
    assert not [line.strip() for line in lines if re.search(r"v_cvt_(pk_)?f16_f32", line)]
    assert sum("v_fma_mixhi_f16" in line for line in lines) > 500


def test_the_search_for_loose_barriers_finds_one():
    code = ["_Zkernel:", "\ts_barrier", ".L1:", "\tbuffer_load_dwordx4 v1, s[0:3], 0 offen lds", "\tbuffer_load_dword v2, v1, s[0:3], 0",
            "\ts_waitcnt vmcnt(2)", "\ts_barrier", "\ts_cbranch_scc1 .L1", "\ts_branch .L3", ".L3:"]
    assert not _loose_barriers(code)
    assert _loose_barriers([line.replace("vmcnt(2)", "vmcnt(3)") for line in code]) == [(7, 3, 2)]


def test_the_search_for_early_reads_finds_them():
    asm = ["\t;;#ASMSTART", "\tv_max3_f32 v82, v34, v35, v36", "\t;;#ASMEND"]
    code = ["_Zkernel:", "\tv_mfma_f32_32x32x16_f16 v[34:49], v[82:85], v[66:69], 0", "\ts_cbranch_scc1 .L1", "\ts_nop 11", ".L1:", *asm]
    assert _early_reads(code) == [(7, "v_max3_f32 v82, v34, v35, v36")]
    assert not _early_reads([line for line in code if "cbranch" not in line])
    assert _early_reads(["\tv_exp_f32_e32 v36, v1", *asm]) and not _early_reads(["\tv_exp_f32_e32 v36, v1", "\tv_mov_b32_e32 v2, v3", *asm])
    for reader in ("v_mfma_f32_32x32x16_f16 v[0:15], v[80:83], v[66:69], 0", "v_permlane32_swap_b32_e32 v1, v82",
                   "v_mov_b32_dpp v1, v82 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"):
        assert _early_reads([*asm, "\ts_nop 0", "\t" + reader]) and not _early_reads([*asm, "\ts_nop 1", "\t" + reader])
    assert not _early_reads([*asm, "\tv_mul_f32_e32 v1, v82, v82"])


def test_packed_code_sums_are_unsigned(tmp_path):
    """A row's two code sums ride in one word, the sum of all codes above bit 16: with 4096 codes it passes 2^15, and the word would
    overflow as a signed one.  No addition of lanes' values in those kernels may promise the compiler that it does not (nsw)."""
    ir = tmp_path / "quantize.ll"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", os.path.join(build.CSRC, "quantize.hip"), "-o", str(ir)],
                   check=True, stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^define [^\n]*quantize_tok_rows_kernelILi1E[^\n]*\{\n(.*?)^\}", ir.read_text(), re.S | re.M)
    assert len(kernels) >= 20
    added = 0
    for body in kernels:
        moved = set(re.findall(r"(%\S+) = (?:tail )?call [^\n]*@llvm\.amdgcn\.update\.dpp\.i32", body))
        adds = re.findall(r"= add (nuw |nsw |nuw nsw )?i32 (%[^,\s]+), (%[^,\s]+)", body)
        crossed = [flags for flags, a, b in adds if a in moved or b in moved]
        assert not any("nsw" in f for f in crossed), crossed
        added += len(crossed)
    assert added >= 4 * len(kernels)
