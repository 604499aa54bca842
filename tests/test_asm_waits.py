"""Assembly that reads a register across lanes brings its own wait states: a vector instruction's result may be
read that way two wait states later at the earliest, the compiler does not look into assembly, and only inside one
statement can it put no copy between the wait and the read."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")


def _statements(text):
    """The text of every asm(...) statement, macros of the same file put in."""
    text = re.sub(r"//[^\n]*", "", text)
    macros = {m.group(1): m.group(2) for m in re.finditer(r"#define (\w+)(?:\([^)]*\))?((?:[^\n]*\\\n)*[^\n]*)", text)}
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        depth, i = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[i], 0)
            i += 1
        body = text[m.end():i - 1]
        yield re.sub(r"\b(\w+)(\(\w+\))?", lambda w: macros.get(w.group(1), w.group(0)), body)


def test_lane_reads_wait_in_their_own_statement():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        for body in _statements(open(path).read()):
            if not re.search(r"_dpp\b|row_newbcast|quad_perm|row_ror", body):
                continue
            seen += 1
            assert re.match(r'\s*"s_nop [1-9]', body), (os.path.basename(path), body[:200])
    assert seen


def test_warnings_about_assembly_are_on():
    from paper_2509_23472_amd import build
    assert not {f for f in build.HIPCC_FLAGS if f in ("-w", "-Wno-inline-asm", "-Wno-everything", "-Wno-all")}
