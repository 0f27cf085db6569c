"""A kernel parameter declared __restrict__ must be the only way to its memory.  k_select is also handed some of its arrays inside a
struct (the small form writes the column means and reads the list it has just stored through it), which no run can be relied
on to show: the declaration itself is checked."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04569_amd", "csrc")


def _read(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def _pointers(struct, text):
    body = re.search(r"struct %s \{(.*?)\n?\};" % struct, text, re.S).group(1)
    return {name for decl in body.split(";") if "*" in decl for name in re.findall(r"\*\s*(\w+)", decl)}


def test_k_select_promises_no_array_that_its_struct_holds():
    small = _read("kernels_small.hip")
    params = re.search(r"void k_select\(([^)]*)\)", small).group(1)
    restricted = set(re.findall(r"\*\s*__restrict__\s+(\w+)", params))
    inside = _pointers("SelectSmall", small) | _pointers("GatherArgs", _read("gather.h"))
    assert {"kv_list", "s_ctx", "pctx", "kcn"} <= inside and {"sharp", "full_list", "flat_list"} <= restricted
    assert not restricted & inside, sorted(restricted & inside)
