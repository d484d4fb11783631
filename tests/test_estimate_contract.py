"""What the header says about the estimate's scratch is what the library does."""
import os
import re

import paper_1506_03265_amd as cd

HERE = os.path.dirname(os.path.abspath(cd.__file__))


def test_noalloc_scratch_as_documented():
    header = " ".join(open(os.path.join(HERE, "..", "include", "cldiam.h")).read().split())
    source = open(os.path.join(HERE, "csrc", "estimate.hip")).read()
    text = header[header.index("with no workspace argument"):header.index("#define CLDIAM_NOALLOC_MAX_K")].replace(" * ", " ")
    lds_most = int(re.search(r"kLdsMaxK = (\d+);", source).group(1))
    assert f"above {lds_most} nodes, per-workgroup distance and queue slices" in text
    assert "a bound of 8 bytes per quotient node" in text and "CLDIAM_NOALLOC_MAX_K * 8" in source
    assert int(re.search(r"CLDIAM_NOALLOC_MAX_K (\d+)", header).group(1)) == cd.CLDIAM_NOALLOC_MAX_K
