"""What the library's sources may not hold (CPU)."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_environment_switches():
    """A call's result and its launch depend on its arguments only: no source
    of the library reads an environment variable."""
    files = glob.glob(os.path.join(ROOT, "paper_2205_11852_amd", "csrc", "*"))
    assert len(files) >= 9
    for f in files:
        with open(f) as fh:
            assert not re.search(r"\b(secure_)?getenv\b|\benviron\b", fh.read()), f
