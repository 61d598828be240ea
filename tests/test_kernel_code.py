"""Properties of the generated gfx950 code that cost speed when they are lost
(compiled here from the library's sources with its own flags, no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2608_10519_amd import build as B


@pytest.fixture(scope="module")
def select_asm(tmp_path_factory):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc is not available")
    out = str(tmp_path_factory.mktemp("asm") / "select.s")
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                        os.path.join(B.CSRC, "select.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(out).read()
    return {m.group(1): m.group(2) for m in re.finditer(r"^(_ZN8sparstar\w+):.*?\n(.*?)s_endpgm", text, re.S | re.M)}


def test_list_stores_take_a_scalar_descriptor(select_asm):
    """The selectors store the list through a buffer descriptor.  Kept in vector
    registers it is read back lane by lane around every store: then there are
    several v_readfirstlane per store instead of a few per kernel."""
    kernels = {n: t for n, t in select_asm.items() if "score_select_kernel" in n or "select_reg_kernel" in n}
    assert len(kernels) == 8 + 7, sorted(kernels)  # fused: two head dims, four row lengths
    for name, text in kernels.items():
        stores, reads = text.count("buffer_store_dword"), text.count("v_readfirstlane_b32")
        assert stores > 0 and reads <= 16 + stores // 8, (name, stores, reads)
