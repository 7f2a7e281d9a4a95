"""What the compiler left of the loop kernel's registers, read from the library's own kernel descriptions."""
import os
import re

from paper_2310_09443_amd import build


def spilled():
    """{(ratio, clip, tight, lists, rows): vector registers spilled} of every form of k_loop."""
    if not os.path.exists(build.LIB):
        build.build()
    blob = open(build.LIB, "rb").read()
    out = {}
    # (a description is a map with its keys in order, each a length and a text: the kernel's symbol comes before the count, a small number or one of one byte)
    for m in re.finditer(rb"k_loopI((?:Lb[01]E)+)EEvPKN3g108LoopArgsE\.kd\xb8", blob):
        at = blob.index(b".vgpr_spill_count", m.end()) + len(b".vgpr_spill_count")
        n = blob[at + 1] if blob[at] == 0xcc else blob[at]
        out[tuple(int(x) for x in re.findall(rb"Lb([01])E", m.group(1)))] = n
    return out


def test_long_timelines_do_not_pay_for_the_rows():
    """Benefit key, band reading: the form for more chunks than rows of lanes take keeps no more than four registers in scratch,
    and no form without room for a list more than two."""
    s = spilled()
    assert s[(0, 0, 0, 0, 0)] <= 4, s
    assert s[(0, 0, 0, 0, 0)] < s[(0, 0, 0, 0, 1)], s
    assert all(n <= 2 for form, n in s.items() if form[0] or (form[1] and not form[3])), s
