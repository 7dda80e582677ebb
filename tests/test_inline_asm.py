"""No kernel writes an instruction in inline assembly: the compiler inserts the
wait states between a matrix instruction and the vector instructions that reuse
its registers only for instructions that it selects itself. (Empty statements
that hide a value from the optimiser emit nothing and are fine.)"""
import pathlib
import re

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2112_01579_amd" / "csrc"


def test_no_instructions_in_inline_assembly():
    seen = 0
    for f in sorted(CSRC.iterdir()):
        for m in re.finditer(r'\basm\s*(?:volatile\s*)?\(\s*"([^"]*)"', f.read_text()):
            seen += 1
            assert m.group(1) == "", "%s: %s" % (f.name, m.group(0))
    assert seen > 0
