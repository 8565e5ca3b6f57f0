"""The environment variables the library reads are the ones its header names (host only)."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_08313_amd", "csrc")


def test_header_names_what_is_read():
    read = set()
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".h")):
            read |= set(re.findall(r'getenv\("(\w+)"\)', open(os.path.join(CSRC, f)).read()))
    named = set(re.findall(r"\bLC_[A-Z_]+\b", open(os.path.join(ROOT, "include", "localcomm.h")).read()))
    assert read
    assert read <= named, f"read but not in the header: {sorted(read - named)}"
