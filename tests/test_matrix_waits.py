"""Instructions written as inline assembly beside matrix instructions: the compiler adds no wait states around what it does
not see, so the device code that it makes is looked at (AMD assembly, compiled here; no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2506_19651_amd import build as B


def _assembly(name, tmp_path):
    out = tmp_path / (name + ".s")
    cmd = [B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, name + ".hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def _registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    return range(int(m.group(1)), int(m.group(2)) + 1) if m else range(0)


def _named(code):
    named = {int(x) for x in re.findall(r"\bv(\d+)\b", code)}
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", code):
        named.update(range(int(a), int(b) + 1))
    return named


def _touches(line, regs):
    return bool(_named(line.split(";")[0]) & regs)


def _states(lines):
    return sum(int(m.group(1)) + 1 for m in (re.match(r"\s*s_nop (\d+)", x) for x in lines) if m)


def test_score_instructions_carry_their_wait_states(tmp_path):
    lines = _assembly("attn_fp8", tmp_path).split("\n")
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


def _kernels(text):
    """(name, [(opcode, operands, inline assembly?)], indexes of the instructions that may run before each) per kernel."""
    for m in re.finditer(r"^(_ZN5pevlm\w*kernel\w*):(.*?)\n\.Lfunc_end", text, re.S | re.M):
        code, labels, inline = [], {}, False
        for line in m.group(2).split("\n"):
            if "#ASMSTART" in line or "#ASMEND" in line:
                inline = "#ASMSTART" in line
                continue
            line = line.split(";")[0].strip()
            label = re.match(r"(\.LBB\w+):", line)
            if label:
                labels[label.group(1)] = len(code)
            elif line and not line.startswith(".") and not line.endswith(":"):
                op, _, args = line.partition(" ")
                code.append((op, args, inline))
        before = [[] for _ in code]
        for i, (op, args, _) in enumerate(code):
            if op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
                before[i + 1].append(i)
            if "branch" in op and labels.get(args.strip(), len(code)) < len(code):
                before[labels[args.strip()]].append(i)
        yield m.group(1), code, before


# wait states between a matrix instruction and another vector instruction that reads its result: passes and 4, or 5
WAITS = {"4x4x4": 5, "16x16": 12, "32x32x64": 20, "32x32x2": 20, "32x32x16": 12}


@pytest.mark.parametrize("name", ["attn_bf16", "attn_bf16_stream", "attn_fp8", "attn_f32", "probe"])
def test_inline_instructions_wait_for_matrix_results(name, tmp_path):
    found, seen_inline = [], 0
    for kernel, code, before in _kernels(_assembly(name, tmp_path)):
        for i, (op, args, inline) in enumerate(code):
            if not inline or not op.startswith("v_") or "mfma" in op:
                continue
            seen_inline += 1
            work = [(j, 0, frozenset(_named(args.split(",", 1)[1]))) for j in before[i]]
            best = {}
            while work:
                j, states, regs = work.pop()
                if states >= 20 or best.get((j, regs), 99) <= states:
                    continue
                best[(j, regs)] = states
                jop, jargs, _ = code[j]
                written = set()
                if jop.startswith(("v_", "ds_read", "global_load", "buffer_load")) and not jargs.endswith("lds"):
                    written = _named(jargs.split(",")[0])
                if "mfma" in jop and written & regs:
                    need = next(v for k, v in sorted(WAITS.items(), key=lambda kv: -len(kv[0])) if k in jop)
                    if states < need:
                        found.append(f"{kernel}: {states} of {need} states from {jop} {jargs} to {op} {args}")
                if regs - written:
                    cost = int(jargs) + 1 if jop == "s_nop" else 1
                    work += [(b, states + cost, regs - written) for b in before[j]]
    assert not found, found[:3]
    assert seen_inline or name in ("attn_f32", "probe")
