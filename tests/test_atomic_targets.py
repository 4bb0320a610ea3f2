"""Atomic operations of the kernels touch the workspace and LDS only: a caller's
buffer is stored to and read, so that it needs no alignment and no kind of
memory beyond what plain accesses need."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_05804_amd", "csrc")
CALL = re.compile(r"\b(__hip_atomic_\w+|atomic(?:Add|Min|Max|Or|Exch|CAS)|__builtin_amdgcn_atomic_\w+"
                  r"|add_here|take_ticket)\(\s*([^,()]*(?:\([^()]*\))?[^,()]*)")
# the header, the workspace's arrays (SegTable t: in LDS or there), exchange
# slots, the scaled weights' array (a workspace array, below), LDS
ALLOWED = re.compile(r"^(&p\.hdr->|&ws\.|&t\.|&s_|slot\b|mine\b|reinterpret_cast<unsigned\*>\(p\.wsc \+ row\)|reinterpret_cast<unsigned\*>\(&hdr->)")


def targets():
    found = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in CALL.finditer(text):
            before = text[:m.start()].rstrip()
            if before.endswith(("void", "unsigned")):  # a wrapper's own definition
                continue
            found.append((os.path.basename(path), m.group(1), m.group(2).strip()))
    return found


def test_atomics_touch_no_caller_buffer():
    wrapped = {("segment.hip", "x"), ("row_ops.h", "counter")}  # the bodies of add_here, take_ticket
    found = targets()
    assert len(found) > 20
    bad = [t for t in found if not ALLOWED.match(t[2]) and (t[0], t[2]) not in wrapped]
    assert not bad, bad


def test_those_arrays_are_the_workspaces():
    api = open(os.path.join(CSRC, "turnkl_api.hip")).read()
    assert "rp.wsc = ws.wsc;" in api
    assert "rp.slots = ws.slots;" in api and "rp.hdr = ws.hdr;" in api
    internal = open(os.path.join(CSRC, "turnkl_internal.h")).read()
    assert "w.wsc = reinterpret_cast<float*>(b + L.wsc);" in internal
