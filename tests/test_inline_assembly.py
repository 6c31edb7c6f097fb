"""Inline assembly of the kernels, by reading the sources."""

import re

from paper_2510_18413_amd import build as B


def test_no_instruction_in_inline_assembly_reads_a_scalar_register():
    """A vector instruction that writes a scalar register (a comparison, a lane read) needs two wait states before another vector
    instruction reads that register.  The compiler keeps them between its own instructions, and does not look inside inline
    assembly: an instruction there must have vector operands only (or be one of the compiler's builtins instead)."""
    seen = 0
    for src in B.sources():
        for text, operands in re.findall(r'\basm\s*(?:volatile\s*)?\(\s*"([^"]*)"([^;]*);', src.read_text()):
            if text:
                seen += 1
                assert not re.search(r'"[^"]*s[^"]*"\s*\(', operands), "%s: %s" % (src.name, text)
    assert seen > 0
