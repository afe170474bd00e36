"""Inline assembly in the kernels names every fixed register it writes as clobbered: the compiler keeps values in m0, vcc
and the scalar registers across a statement that does not say so."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WRITTEN = re.compile(r"^\s*[a-z]\w+\s+(m0|vcc\w*|exec\w*|[sv]\d+|[sv]\[\d+:\d+\])\s*,")


def statements(text):
    """(instructions, clobbers) of every asm statement."""
    for m in re.finditer(r"\basm\b[\s\w]*\(", text):
        depth, end = 1, m.end()
        quoted = False
        while depth:
            c = text[end]
            if c == '"' and text[end - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            end += 1
        body = re.sub(r'"\s*\n\s*"', "", text[m.end():end - 1])
        code = re.match(r'\s*"((?:[^"\\]|\\.)*)"', body).group(1)
        parts = re.sub(r'"(?:[^"\\]|\\.)*"', lambda q: q.group(0).replace(":", ";"), body).split(":")
        yield re.split(r"\\n\\t|\\n|;", code), set(re.findall(r'"(\w+)"', parts[3])) if len(parts) > 3 else set()


def test_written_registers_are_clobbered():
    seen = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2605_13907_amd", "csrc", "*"))):
        with open(path) as f:
            text = f.read()
        for code, clobbers in statements(text):
            for line in code:
                m = WRITTEN.match(line)
                if m:
                    seen += 1
                    assert m.group(1) in clobbers, f"{os.path.basename(path)}: {line}"
    assert seen > 0


def test_the_reader_of_statements():
    found = list(statements('asm volatile("s_mov_b32 m0, %0\\n\\tv_nop" : : "s"(f(x)), "v"(y) : "memory");\n'
                            'asm("" : "+v"(q)); asm volatile("s_waitcnt vmcnt(0)" ::: "memory", "m0");'))
    assert [c for _, c in found] == [{"memory"}, set(), {"memory", "m0"}]
    assert WRITTEN.match(found[0][0][0]).group(1) == "m0" and not WRITTEN.match(found[2][0][0])
