"""The generated-code checks of the prepared-path kernel (test_kernel_asm.py)
on the key-split kernel, whose score MFMAs are the same inline assembly: MFMA
latencies, no spills; that the loop's waits leave the next tile's reads in
flight; and that no VALU instruction writes a register right before an inline
MFMA reads it (CPU only)."""
import re

import test_kernel_asm as checks
from test_kernel_asm import asm_text  # noqa: F401  (the fixture)

N_INSTANCES = 10  # (rope, sparse) and records, each with and without output records
WRITE_WAIT_STATES = 2  # a VALU write of an MFMA's A, B or C operand


def test_latencies_and_spills(asm_text):  # noqa: F811
    kernels = checks.functions(asm_text, "attn_keysplit_kernel")
    assert len(kernels) == N_INSTANCES
    checks.check_mfma_latency(kernels, past_branches=False)
    checks.check_no_spills(kernels)


def test_loop_waits(asm_text):  # noqa: F811
    """In the main loop (the block with 32 exponentials and its neighbours)
    every fragment is waited for with the 15 younger loads left in flight: no
    wait there drains the reads of the next iteration."""
    for name, body in checks.functions(asm_text, "attn_keysplit_kernel"):
        blocks, cur = [], []
        for ln in body:
            if re.match(r"\.LBB", ln):
                blocks.append(cur)
                cur = []
            cur.append(ln)
        blocks.append(cur)
        loop = [b for b in blocks if sum("v_exp_f32" in ln for ln in b) >= 16
                and sum("buffer_load" in ln for ln in b) >= 8 and not any("v_accvgpr" in ln for ln in b)]
        assert sum(sum("v_mfma" in ln for ln in b) for b in loop) == 64, name
        waits = [ln for b in loop for ln in b if "vmcnt" in ln]
        assert waits and all("vmcnt(15)" in ln for ln in waits), name


def test_operands_settled_before_inline_mfmas(asm_text):  # noqa: F811
    """The compiler keeps a VALU write of an MFMA's operand (a copy of Q' into
    an AGPR, say) two wait states clear of the MFMAs it can see, not of the
    inline ones: a build with such copies in the loop returned garbage scores."""
    for name, body in checks.functions(asm_text, "attn_keysplit_kernel"):
        ins = checks.instructions(body)
        for i, (t, in_asm) in enumerate(ins):
            if not (in_asm and t.startswith("v_mfma")):
                continue
            used = set().union(*(checks.regs(o) for o in checks.operands(t)[1:]))
            ws = 0
            for t2, _ in reversed(ins[max(0, i - 20):i]):
                m = re.match(r"s_nop (\d+)", t2)
                if ws >= WRITE_WAIT_STATES:
                    break
                if t2.startswith("v_") and not t2.startswith("v_mfma") and checks.operands(t2):
                    assert not (checks.regs(checks.operands(t2)[0]) & used), "%s: %r then %r" % (name, t2, t)
                ws += int(m.group(1)) + 1 if m else 1
