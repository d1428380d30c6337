"""Every function that a kernel source defines is called by something (the sources are built with
-Wno-unused-function, so the compiler does not say)."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FILES = sorted(glob.glob(os.path.join(ROOT, "paper_2509_12138_amd", "csrc", "*")))


def _code(path):
    return re.sub(r"//[^\n]*", "", open(path).read())


@pytest.mark.parametrize("path", FILES, ids=os.path.basename)
def test_functions_are_used(path):
    whole = "\n".join(_code(f) for f in FILES)
    defined = re.findall(r"^(?:static|__device__|__global__)[^;{}=]*?\b(\w+)\s*\((?!.*;$)",
                         _code(path), flags=re.M)
    dead = [n for n in defined if not n.startswith("__") and
            len(re.findall(r"\b%s\b" % n, whole)) < 2]
    assert not dead, dead
