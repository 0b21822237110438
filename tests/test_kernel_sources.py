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


@pytest.mark.parametrize("path", [p for p in SOURCES if os.path.basename(p).startswith("encode")], ids=os.path.basename)
def test_table_gradients_are_only_added_to(path):
    """dtable "+=": other streams may add to the same gradient, so every add of a kernel is atomic.  A plain store is a NaN that marks
    the gradient."""
    for function in re.sub(r"//.*", "", open(path).read()).split("\n}\n"):
        names = "|".join(["dtable"] + re.findall(r"\*\s*(\w+)\s*=\s*dtable\b", function))
        for store in re.findall(r"\b(?:%s)\s*\[[^;=]*\]\s*[-+]?=[^=][^;]*;" % names, function):
            assert "__uint_as_float(0x7fc00000u)" in store, store


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_transposing_reads_are_fenced(path):
    """A transposing LDS read returns what other lanes stored, which the compiler cannot see: a function that reads so keeps it behind
    the stores before and ahead of those that follow."""
    text = re.sub(r"//.*", "", open(path).read())
    fences = [name for name, body in re.findall(r"\bvoid (\w+)\(\)\s*\{(.*?)\n\}", text, re.S)
              if "__builtin_amdgcn_fence" in body and "__builtin_amdgcn_wave_barrier" in body]
    for function in text.split("\n}\n"):
        reads = [m.start() for m in re.finditer(r"__builtin_amdgcn_ds_read_tr", function)]
        if reads:
            calls = [m.start() for name in fences for m in re.finditer(r"\b%s\(\);" % name, function)]
            assert calls and min(calls) < reads[0] and max(calls) > reads[-1], function
