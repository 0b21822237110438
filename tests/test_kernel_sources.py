"""What the compiler has to be able to see in the kernels' sources."""
import glob
import os
import re

import pytest

import paper_2405_04416_amd as pkg

SOURCES = sorted(glob.glob(os.path.join(os.path.dirname(pkg.__file__), "csrc", "*")))


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_no_instruction_in_inline_assembly(path):
    """A matrix instruction must not follow the vector instruction that wrote one of its operands within two wait states.  The compiler
    sees to that for the instructions that it emits itself, not for those of an inline assembly block: such blocks hold no instruction."""
    text = re.sub(r"//.*", "", open(path).read())
    for body in re.findall(r"\basm\b\s*(?:volatile\s*)?\(\s*\"([^\"]*)\"", text):
        assert body.strip() == "", body
