"""Rules for the kernels' source that no run can show to be kept: what breaks them fails rarely, or hangs."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04450_amd", "csrc")


def sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(path) as f:
            yield os.path.basename(path), re.sub(r"//[^\n]*|/\*.*?\*/", "", f.read(), flags=re.S)


def test_no_block_waits_for_another_one():
    # blocks of an ordinary launch need not all be resident: a loop on a word that other blocks set may never end
    for name, code in sources():
        assert "s_sleep" not in code, name
        assert not re.search(r"\b(while|for)\s*\([^{};]*atomic", code), name
        assert not re.search(r"cooperative|grid\.sync", code), name
