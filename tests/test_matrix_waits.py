"""Matrix instructions written as inline assembly: the compiler adds no wait states around what it does not see, so the
device code that it makes of attn_fp8.hip is looked at (AMD assembly, compiled here; no GPU)."""
import os
import re
import subprocess

from paper_2506_19651_amd import build as B


def _registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    return range(int(m.group(1)), int(m.group(2)) + 1) if m else range(0)


def _touches(line, regs):
    code = line.split(";")[0]
    named = {int(x) for x in re.findall(r"\bv(\d+)\b", code)}
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", code):
        named.update(range(int(a), int(b) + 1))
    return bool(named & regs)


def _states(lines):
    return sum(int(m.group(1)) + 1 for m in (re.match(r"\s*s_nop (\d+)", x) for x in lines) if m)


def test_score_instructions_carry_their_wait_states(tmp_path):
    out = tmp_path / "attn_fp8.s"
    cmd = [B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, "attn_fp8.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    lines = out.read_text().split("\n")
    starts = [i for i, x in enumerate(lines) if "#ASMSTART" in x]
    blocks = []
    for i in starts:
        end = next(j for j in range(i, len(lines)) if "#ASMEND" in lines[j])
        body = [x for x in lines[i + 1:end] if x.strip()]
        if any("v_mfma" in x for x in body):
            blocks.append((body, end))
    assert len(blocks) == 12  # Q quantised here or before; first tile and the others; one k-step (head_dim 64) or two
    for body, end in blocks:
        first = next(i for i, x in enumerate(body) if "v_mfma" in x)
        last = max(i for i, x in enumerate(body) if "v_mfma" in x)
        assert _states(body[:first]) >= 2  # a vector instruction may have written an operand right before
        results = {r for x in body if "v_mfma" in x for r in _registers(x.split()[1].rstrip(","))}
        if _states(body[last + 1:]) >= 20:  # 16 passes and 4 states: anything may read them
            continue
        for x in lines[end + 1:]:  # otherwise nothing touches them but the accumulation that goes on from them
            if _touches(x, results):
                assert "v_mfma" in x, x
                m = re.findall(r"v\[\d+:\d+\]", x)
                assert m[0] == m[3], x
                results -= set(_registers(m[0]))
            if not results:
                break
        assert not results
