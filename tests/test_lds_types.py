"""Every LDS array of the kernels is accessed as the type it is declared with: the
compiler may reorder accesses to the same words through pointers of two types."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = glob.glob(os.path.join(ROOT, "paper_2607_05804_amd", "csrc", "*"))


def test_no_lds_array_is_accessed_as_another_type():
    arrays, bad = 0, []
    for path in SOURCES:
        text = re.sub(r"//[^\n]*", "", open(path).read())
        names = re.findall(r"__shared__\s+[\w ]+?(\w+)\s*(?:\[|;)", text)
        arrays += len(names)
        for m in re.finditer(r"(?:reinterpret_cast<[^>]*>|\(\s*\w+\s*\*\s*\))\s*\(?\s*&?(\w+)", text):
            if m.group(1) in names:
                bad.append((os.path.basename(path), m.group(0)))
    assert arrays >= 10
    assert not bad, bad
