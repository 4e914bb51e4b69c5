"""CPU test of the device descriptor: every field that the library writes is
read somewhere.  (A field that nothing reads can hold anything, as one did that
two workgroups of a launch stored different values to.)"""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2112_12271_amd", "csrc")


def _sources():
    txt = ""
    for f in sorted(os.listdir(CSRC)):
        txt += re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read()) + "\n"
    return txt


def _fields(src):
    body = re.search(r"struct SysDev \{(.*?)\n\};", src, re.S).group(1)
    names = []
    for decl in re.findall(r"[^;]+;", body):
        first, *rest = decl.strip(" \n;").split(",")
        for part in [first.split()[-1]] + rest:
            names.append(re.sub(r"[*\s]|\[.*", "", part))
    return names


def test_every_descriptor_field_is_read():
    src = _sources()
    fields = [f for f in _fields(src) if not re.fullmatch(r"pad\d*", f)]
    assert len(fields) > 60 and {"npad", "x", "ends", "rb", "ticket", "differ"} <= set(fields)
    dead = []
    for f in fields:
        # an access of the field that is neither the target of an assignment
        # nor of a maximum taken into it
        uses = re.findall(r"(atomicMax\(&)?\b\w+(?:->|\.)%s\b(\[[^\]]*\])?\s*(=(?!=))?" % f, src)
        if not any(not mx and not asg for mx, _, asg in uses):
            dead.append(f)
    assert dead == []
