"""Which kernel runs a depthwise + 1x1 block and what it is called (host only: nothing is launched)."""
import os
import re

import pytest

from paper_1904_08368_amd import binding as B

CSRC = os.path.join(os.path.dirname(os.path.abspath(B.__file__)), "csrc")


def _desc(n, c, h, w, stride):
    return B.conv_desc(n, c, h, w, c, 3, 3, stride, 1, B.RELAY_F16, B.RELAY_NHWC, 0)


@pytest.mark.parametrize("stride", [1, 2])
def test_every_variant_has_the_name_of_its_kernel(stride):
    """All template arguments, as a kernel trace prints them: no two variants share a name (but the two that are one kernel at stride 2)."""
    src = open(os.path.join(CSRC, "dwpw_direct.hip")).read()
    table = re.search(r"#define RELAY_DWPW_DIRECT\(X\)(.*?)#define", src, re.S).group(1)
    rows = [tuple(int(v) for v in m.split(",")) for m in re.findall(r"X\(([^)]*)\)", table)]
    assert [r[0] for r in rows] == list(range(len(rows))) and len(rows) >= 13
    names = set()
    for v, *args, rows_per_item in rows:
        B.relay_set_conv_tile(500 + v)
        try:
            name = B.relay_dwconv_pwconv_kernel_name(_desc(1, 64, 9, 9, stride), 64)
        finally:
            B.relay_set_conv_tile(-1)
        want = [stride] + args + [rows_per_item if stride == 1 else 2]
        assert name == "dwpw_fused_direct_kernel<" + ", ".join(str(a) for a in want) + ">"
        names.add(name)
    assert len(names) == len(rows) - (stride == 2)


# where the rule has two tiles of one size: items of two and of four rows, one or two of them in registers
@pytest.mark.parametrize("n,c,h,w,k,stride,tail", [
    (16, 512, 13, 12, 512, 1, "32, 8, 8, 6, 16, 2, 4"), (32, 512, 10, 9, 512, 1, "32, 8, 8, 6, 16, 0, 2"),
    (32, 512, 14, 14, 1024, 2, "32, 8, 8, 6, 16, 2, 2"), (32, 512, 14, 14, 512, 1, "64, 8, 8, 4, 16, 2, 4"),
    (32, 256, 28, 28, 512, 2, "64, 8, 8, 4, 16, 2, 2"), (7, 128, 90, 70, 128, 2, "64, 8, 8, 4, 16, 0, 2"),
    (32, 128, 56, 56, 128, 1, "64, 4, 4, 4, 4, 3, 4"), (32, 64, 56, 56, 64, 1, "64, 4, 4, 4, 4, 3, 2"),
    (32, 64, 112, 112, 128, 2, "64, 4, 4, 4, 4, 3, 2")])
def test_the_rule_names_one_variant(n, c, h, w, k, stride, tail):
    assert B.relay_dwconv_pwconv_kernel_name(_desc(n, c, h, w, stride), k) == f"dwpw_fused_direct_kernel<{stride}, {tail}>"


@pytest.mark.parametrize("n,c,h,w,k,stride,pays", [
    (4096, 128, 1, 1, 128, 1, False), (1024, 64, 1, 1, 8, 2, False), (2048, 64, 2, 2, 64, 1, False), (2048, 128, 2, 2, 128, 2, False),
    (1024, 64, 3, 3, 128, 1, False), (1024, 128, 3, 3, 64, 1, False), (2048, 64, 9, 9, 32, 2, True), (2420, 64, 7, 7, 96, 2, False),
    # up to two workgroups to a CU, however empty
    (512, 64, 3, 3, 64, 1, True), (513, 64, 3, 3, 64, 1, False), (300, 128, 5, 5, 8, 2, True),
    # just enough rows: 13 of 128 channels (12, 13), 16 of 64 channels within one round of three to a CU, 24 beyond
    (1024, 128, 3, 4, 32, 1, False), (1024, 128, 1, 13, 32, 1, True), (768, 64, 4, 4, 32, 1, True), (769, 64, 4, 4, 32, 1, False),
    (681, 64, 4, 6, 32, 1, True), (1024, 64, 1, 15, 32, 1, False),
    # the blocks of a network, small outputs
    (32, 64, 56, 56, 64, 1, True), (32, 128, 56, 56, 128, 1, True), (32, 64, 112, 112, 128, 2, True), (32, 64, 56, 56, 8, 1, True),
    (16, 128, 33, 47, 16, 1, True)])
def test_one_launch_is_offered_only_where_its_rows_are_filled(n, c, h, w, k, stride, pays):
    d = _desc(n, c, h, w, stride)
    assert B.relay_dwconv_pwconv_few_pixels(d, k) == pays
    assert "direct_kernel" in B.relay_dwconv_pwconv_kernel_name(d, k)      # the entry point itself takes this kernel either way
