"""The collide-stream kernels that take the only box's description as a launch
argument exist for periodic boxes alone: with walls they are slower than the
generic ones at every size (14 % of a step of a walled 128^3 FP16 box).  The
library's kernel names say which were compiled."""
import re

from paper_2403_05443_amd import lbell


def test_single_box_kernels_are_periodic():
    blob = open(lbell.LIB_PATH, "rb").read()
    # k_collide_stream<ST, COLL, WALLS, SPT, XCD, NT, Q, ONE>, k_collide_stream_aa<..., NT, CIN, Q, ONE>
    names = set(re.findall(rb"k_collide_streamILi\dELi\dELb(\d)ELi\dELi\dELb\dELi(?:19|27)ELb(\d)E", blob))
    names_aa = set(re.findall(rb"k_collide_stream_aaILi\dELi\dELb(\d)ELi\dELi\dELb\dELi\dELi(?:19|27)ELb(\d)E", blob))
    for seen in (names, names_aa):
        assert (b"0", b"1") in seen  # periodic, one box
        assert (b"1", b"0") in seen  # walls, described in memory
        assert (b"1", b"1") not in seen
