"""Entry points may be called by several threads at once: what a function of the library keeps between calls is constant, atomic or
behind a lock, never a plain variable."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1908_00213_amd", "csrc")


def test_no_function_keeps_a_plain_variable():
    found = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for n, line in enumerate(open(path), 1):
            if re.match(r"\s+static (bool|int|unsigned|size_t|int64_t|void \*|char \*)\s*\w+\s*(=|;|\{)", line):
                found.append("%s:%d: %s" % (os.path.basename(path), n, line.strip()))
    assert not found, found
