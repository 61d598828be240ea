"""Properties of the generated gfx950 code that cost speed when they are lost
(compiled here from the library's sources with its own flags, no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2608_10519_amd import build as B


def _compile(tmp_path, source):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc is not available")
    out = str(tmp_path / "kernels.asm")
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                        os.path.join(B.CSRC, source), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return open(out).read()


def test_list_stores_take_a_scalar_descriptor(tmp_path):
    """The selectors store the list through a buffer descriptor.  Kept in vector
    registers it is read back lane by lane around every store: then there are
    several v_readfirstlane per store instead of a few per kernel."""
    text = _compile(tmp_path, "select.hip")
    bodies = {m.group(1): m.group(2) for m in re.finditer(r"^(_ZN8sparstar\w+):.*?\n(.*?)s_endpgm", text, re.S | re.M)}
    kernels = {n: t for n, t in bodies.items() if "score_select_kernel" in n or "select_reg_kernel" in n}
    assert len(kernels) == 8 + 7, sorted(kernels)  # fused: two head dims, four row lengths
    for name, text in kernels.items():
        stores, reads = text.count("buffer_store_dword"), text.count("v_readfirstlane_b32")
        assert stores > 0 and reads <= 16 + stores // 8, (name, stores, reads)


def test_short_rows_of_the_mass_kernel_share_a_cu(tmp_path):
    """The ranking kernel has instances that fit a CU (160 KB of LDS, 2,048
    threads) eight and four times, for calls with many short rows."""
    text = _compile(tmp_path, "mass.hip")
    fits = []
    for m in re.finditer(r"\.group_segment_fixed_size: (\d+)(?:(?!group_segment).)*?\.max_flat_workgroup_size: (\d+)"
                         r"\s+\.name:\s+(\S*topk_mass_kernel\S*)", text, re.S):
        fits.append(min(160 * 1024 // int(m.group(1)), 2048 // int(m.group(2))))
    assert sorted(fits) == [1, 4, 8]


def test_attention_steps_hold_sixteen_products(tmp_path):
    """Between two barriers pairs of the attention loop lie sixteen 32x32x16
    products at D = 64 as at D = 128 (the loop is written out twice, and the
    prologue and the last P V hold eight of each): the work that a step's two
    barriers, waits and address updates are spread over."""
    text = _compile(tmp_path, "attn_fwd.hip")
    bodies = {m.group(1): m.group(2) for m in re.finditer(r"^(_ZN8sparstar15attn_fwd\w+):.*?\n(.*?)s_endpgm", text, re.S | re.M)}
    assert len(bodies) == 24
    for name, body in bodies.items():
        assert body.count("v_mfma_f32_32x32x16_bf16") >= 2 * 16 + 16, name
