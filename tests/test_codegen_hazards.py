"""Device-code checks of the grouped GEMM kernels (CPU only: hipcc cross-compiles gfx950).

The large-tile kernel issues its MFMAs through inline assembly (to pin the accumulators to
AGPRs), and the compiler's hazard recognizer does not look inside inline assembly. Two
rules therefore have to hold by construction of the code, and this test reads the
generated assembly to check them:

* a VALU write of a VGPR is at least two wait states ahead of an inline-assembly MFMA that
  reads it as its A or B operand (the compiler puts ``s_nop 1`` there for its own MFMAs;
  a missing gap made the projection read stale fragments);
* an inline-assembly MFMA's accumulator is not read by ``v_accvgpr_read`` within 18 wait
  states (more than the 16-pass MFMA latency).

Wait states are counted as issued instructions, ``s_nop N`` counting N + 1, along the
listing and along every branch into its target (a loop's back edge).
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_01024_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

VALU_TO_MFMA = 2
MFMA_TO_ACC_READ = 18


def _regs(tok, prefix):
    m = re.match(prefix + r"\[(\d+):(\d+)\]$", tok)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(prefix + r"(\d+)$", tok)
    return {int(m.group(1))} if m else set()


def parse(asm_text):
    """The kernels of an assembly listing: {name: [entry]}, each entry ("label", name) or
    ("ins", op, operands, inside_inline_asm, text)."""
    kernels, cur, in_asm = {}, None, False
    for line in asm_text.splitlines():
        s = line.strip()
        m = re.match(r"^(_Z\S+):", s)
        if m:
            cur, in_asm = [], False
            kernels[m.group(1)] = cur
            continue
        if cur is None:
            continue
        if s.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if s.startswith(";;#ASMEND"):
            in_asm = False
            continue
        m = re.match(r"^(\.?L\w+):", s)
        if m:
            cur.append(("label", m.group(1)))
            continue
        if not s or s.startswith(";") or s.startswith("."):
            continue
        parts = s.replace(",", " ").split()
        cur.append(("ins", parts[0], parts, in_asm, s))
    return kernels


class Window:
    """The last MFMA_TO_ACC_READ issue slots: VGPRs written by VALU and AGPRs written by an
    inline-assembly MFMA in each."""

    def __init__(self, valu=None, mfma=None):
        self.valu, self.mfma = list(valu or []), list(mfma or [])

    def copy(self):
        return Window(self.valu, self.mfma)

    def push(self, vw, md, n=1):
        for _ in range(n):
            self.valu.append(vw)
            self.mfma.append(md)
        del self.valu[:-MFMA_TO_ACC_READ]
        del self.mfma[:-MFMA_TO_ACC_READ]


def step(win, op, parts, in_asm):
    """Issue one instruction after the slots in `win`; returns the rule it breaks, or None,
    and the number of issue slots it took."""
    if op.startswith("s_nop"):
        n = int(parts[1], 0) + 1 if len(parts) > 1 else 1
        win.push(set(), set(), n)
        return None, n
    if op.startswith("v_mfma"):
        rule = None
        if in_asm:
            srcs = _regs(parts[2], "v") | _regs(parts[3], "v")
            recent = set().union(*win.valu[-VALU_TO_MFMA:]) if win.valu else set()
            if srcs & recent:
                rule = "VALU write -> MFMA read"
            win.push(set(), _regs(parts[1], "a"))
        else:
            win.push(set(), set())
        return rule, 1
    if op.startswith("v_accvgpr_read"):
        rule = "MFMA write -> accvgpr read" if _regs(parts[2], "a") & set().union(*win.mfma) else None
        win.push(_regs(parts[1], "v"), set())
        return rule, 1
    if op.startswith("v_") and not op.startswith("v_cmp") and len(parts) > 1:
        win.push(_regs(parts[1], "v"), set())
        return None, 1
    win.push(set(), set())
    return None, 1


def scan(asm_text):
    """Return a list of (kernel, rule, instruction) violations: along the listing, and along
    every branch into its target (a loop's back edge carries the end of the loop body to the
    instructions after the loop head)."""
    bad = set()
    for kernel, entries in parse(asm_text).items():
        labels = {e[1]: i for i, e in enumerate(entries) if e[0] == "label"}
        win, edges = Window(), []
        for e in entries:
            if e[0] != "ins":
                continue
            _, op, parts, in_asm, text = e
            rule, _ = step(win, op, parts, in_asm)
            if rule:
                bad.add((kernel, rule, text))
            if op.startswith(("s_branch", "s_cbranch")) and len(parts) > 1 and parts[1] in labels:
                edges.append((labels[parts[1]], win.copy()))
        for start, w in edges:   # the slots right after each branch target, entered by the branch
            used = 0
            for e in entries[start:]:
                if used >= MFMA_TO_ACC_READ:
                    break
                if e[0] != "ins":
                    continue
                _, op, parts, in_asm, text = e
                rule, n = step(w, op, parts, in_asm)
                used += n
                if rule:
                    bad.add((kernel, rule, text))
    return sorted(bad)


@pytest.fixture(scope="module")
def gemm_asm(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "gemm_bf16.s"
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S",
           "--cuda-device-only", os.path.join(CSRC, "gemm_bf16.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def test_scanner_flags_planted_hazards():
    """The scanner itself: a VALU write right before an inline MFMA, and an early
    accumulator read, are reported; the same code with enough wait states is not."""
    bad = """_Zk:
\tv_cvt_pk_f16_f32 v2, v6, v7
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_f16 a[0:3], v[2:5], v[8:11], a[0:3]
\t;;#ASMEND
\tv_accvgpr_read_b32 v20, a1
"""
    good = """_Zk:
\tv_cvt_pk_f16_f32 v2, v6, v7
\ts_nop 1
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_f16 a[0:3], v[2:5], v[8:11], a[0:3]
\t;;#ASMEND
\ts_nop 7
\ts_nop 7
\ts_nop 7
\tv_accvgpr_read_b32 v20, a1
"""
    rules = sorted(r for _, r, _ in scan(bad))
    assert rules == ["MFMA write -> accvgpr read", "VALU write -> MFMA read"]
    assert scan(good) == []
    # a loop whose last VALU write feeds the inline MFMA at its head: only the back edge
    # shows it (the listing runs the write last and falls out of the loop)
    loop = """_Zk:
.LBB0_1:
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_f16 a[0:3], v[2:5], v[8:11], a[0:3]
\t;;#ASMEND
\ts_nop 7
\ts_nop 7
\ts_nop 7
\tv_cvt_pk_f16_f32 v2, v6, v7
{gap}\ts_cbranch_scc1 .LBB0_1
\ts_endpgm
"""
    assert [r for _, r, _ in scan(loop.format(gap=""))] == ["VALU write -> MFMA read"]
    assert scan(loop.format(gap="\ts_nop 0\n")) == []


def test_inline_mfma_hazards_absent(gemm_asm):
    kernels = set(re.findall(r"^(_Z\S*gemm_il_kernel\S*):", gemm_asm, re.M))
    # expand; projection store and accumulate, each with bf16 weights widened per fragment
    # and with float16 weights used as read; each on four and on eight waves
    assert len(kernels) == 10, kernels
    bad = scan(gemm_asm)
    assert bad == [], "\n".join(f"{k[:60]}: {r}: {i}" for k, r, i in bad[:10])


# ------------------------------------------------ results of the compiler's own MFMAs
# Wait states between a 4-pass MFMA (v_mfma_f32_16x16x32) and another instruction's read of its result.
# The compiler sees to it, but where the accumulators are copied at the merge of two branches it has put
# the copies of their first registers in front of the wait (an accumulator chain ended by an if / else of
# MFMAs: every fourth column was stale).
RESULT_READ = 7


def _all_regs(tok):
    return {(p, r) for p in "va" for r in _regs(tok, p)}


def scan_results(asm_text):
    """(kernel, instruction) for every read of the result of a v_mfma_f32_16x16x32 fewer than RESULT_READ
    wait states after it (another MFMA's accumulator operand is forwarded), along the listing and along
    every branch into its target."""
    bad = set()
    for kernel, entries in parse(asm_text).items():
        labels = {e[1]: i for i, e in enumerate(entries) if e[0] == "label"}

        def walk(start, recent, follow):
            recent = list(recent)   # (wait states ago, registers)
            spent = 0
            for e in entries[start:]:
                if e[0] != "ins":
                    continue
                _, op, parts, in_asm, text = e
                mfma = op.startswith("v_mfma")
                store = "store" in op or op.startswith("ds_write")
                reads = set().union(*[_all_regs(t) for t in (parts[1:] if store else parts[2:4 if mfma else None])])
                if any(reads & regs for _, regs in recent):
                    bad.add((kernel, text))
                n = int(parts[1], 0) + 1 if op == "s_nop" else 1
                recent = [(age + n, regs) for age, regs in recent if age + n < RESULT_READ]
                if op.startswith("v_mfma_f32_16x16x32") and not in_asm:
                    recent.append((0, _all_regs(parts[1])))
                spent += n
                if op.startswith(("s_branch", "s_cbranch")) and len(parts) > 1 and parts[1] in labels and recent:
                    if follow:
                        walk(labels[parts[1]], recent, follow - 1)
                    if op == "s_branch":
                        if follow < 4:
                            return
                        recent = []
                if op == "s_endpgm" or (follow < 4 and not recent):
                    if follow < 4:
                        return
                    recent = []
        walk(0, [], 4)
    return sorted(bad)


def test_result_scanner():
    """A result copied behind a branch too early is reported, one read after the wait is not."""
    listing = """_Zk:
\ts_cbranch_scc1 .LBB0_2
\tv_mfma_f32_16x16x32_f16 a[8:11], v[2:5], v[8:11], a[4:7]
\tv_mfma_f32_16x16x32_f16 a[12:15], v[2:5], v[8:11], a[12:15]
\ts_branch .LBB0_3
.LBB0_2:
\tv_accvgpr_mov_b32 a8, a4
.LBB0_3:
{gap}\tv_accvgpr_mov_b32 a0, a12
\ts_nop 7
\tglobal_store_dwordx4 v[0:1], a[8:11], off
\ts_endpgm
"""
    assert scan_results(listing.format(gap="")) == [("_Zk", "v_accvgpr_mov_b32 a0, a12")]
    assert scan_results(listing.format(gap="\ts_nop 6\n")) == []


def test_mfma_results_waited_for(gemm_asm):
    bad = scan_results(gemm_asm)
    assert bad == [], "\n".join(f"{k[:90]}: {i}" for k, i in bad[:10])


# ------------------------------------------------ lane reads of the mix kernels
def lanes_read_narrowed(asm_text, name):
    """(kernel, instruction) for every v_readlane in a kernel whose name has `name` in it that runs between
    a narrowing of exec and its restoration: a register read from another lane has to hold that lane's value,
    which a copy or a reload made under the narrower exec does not give it. (Registers written by v_writelane
    hold spilled scalars: lane writes and reads do not depend on exec.)"""
    bad = []
    for kernel, entries in parse(asm_text).items():
        if name not in kernel:
            continue
        spilled = {e[2][1] for e in entries if e[0] == "ins" and e[1].startswith("v_writelane")}
        saved = set()   # registers that hold an exec to restore
        for e in entries:
            if e[0] != "ins":
                continue
            _, op, parts, _, text = e
            if op.endswith("saveexec_b64"):
                saved.add(parts[1])
            elif op in ("s_or_b64", "s_mov_b64") and parts[1] == "exec":
                saved.discard(parts[-1])
            elif op.startswith("v_readlane") and saved and parts[2] not in spilled:
                bad.append((kernel, text))
    return bad


def test_mix_reads_lanes_with_every_lane_active(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "mix.s"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
                    os.path.join(CSRC, "mix_combine.hip"), "-o", str(out)], check=True, capture_output=True)
    asm = out.read_text()
    assert len(re.findall(r"^_Z\S*mix_\S*kernel\S*:", asm, re.M)) >= 8 and "v_readlane" in asm
    bad = lanes_read_narrowed(asm, "mix_")
    assert bad == [], "\n".join(f"{k[:80]}: {i}" for k, i in bad[:10])
