"""The byte offsets of a wavefront of the bfloat16 weight-gradient kernel (csrc/k_wgrad_mfma.hip) are unsigned 32-bit numbers: for the
largest grids that the library accepts, in many shapes, the furthest one stays below 2^32.  On the host: nothing of that size is allocated."""
import pytest

import paper_2003_10735_amd as st

AHEAD = 7       # units that the operand ring fetches ahead


def furthest_byte(n, h, w, grouped, splits):
    """Over all wavefronts: end of the last fetch, counted from the operand's base (the unit before the wavefront's first)."""
    rows, groups = (h + 2) * (1 if grouped else n), -(-(w + 2) // 8)
    units = (rows + 1) // 2 * groups
    per_wave = -(-units // (splits * 4))
    place = lambda u: u // groups * 2 * groups + u % groups            # group of a unit's upper row
    end = 0
    for wave in range(splits * 4):
        first, last = wave * per_wave, min((wave + 1) * per_wave, units) - 1 + AHEAD
        if first < units:
            before = place(first) - (1 if first % groups else groups + 1)
            end = max(end, (place(last) - before + groups + 1) * 512)  # (the second row of the pair is `groups` further)
    return end


@pytest.mark.parametrize("n,grouped", [(1, 0), (3, 0), (2, 1)])
@pytest.mark.parametrize("fixed,value", [("h", 1), ("h", 2), ("h", 3), ("h", 8), ("h", 90), ("w", 1), ("w", 6), ("w", 7), ("w", 250), ("w", 4000)])
def test_the_largest_accepted_grid(n, grouped, fixed, value):
    c = 64 if grouped else 1
    desc = lambda x: st.HeadDesc(n, c, **{fixed: value, "w" if fixed == "h" else "h": x}, c1=c, c2=c, n_classes=2, grouped=grouped)
    lo, hi = 1, 1 << 25
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if st.st_workspace_bytes(desc(mid)) else (lo, mid)
    for x in (lo, lo // 2 + 1, lo // 17 + 1):
        d = desc(x)
        assert st.st_workspace_bytes(d) > 0
        for splits in st.st_get_workspace_layout(d)["splits"][:2]:
            assert furthest_byte(n, d.h, d.w, grouped, splits) < 1 << 32, (d.h, d.w, splits)
