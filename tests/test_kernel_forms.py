"""Which forms of a kernel the library holds, read from the names in the
objects that its build leaves (no GPU)."""
import os
import re

import pytest

from paper_1602_04691_amd import build as ori_build


def kernels(obj):
    path = os.path.join(ori_build.BUILD, obj)
    if not os.path.exists(path):
        pytest.skip("no objects of the build here")
    return set(re.findall(rb"k_zpassI([df])Li(\d+)ELb([01])ELb([01])ELb([01])ELi(\d)E", open(path, "rb").read()))


def test_complex128_z_at_1024_takes_64_bit_addresses():
    # the per-lane form is 5 % slower there (n = 512: 6.27 vs 5.96 ms), for
    # complex64 and at the other lengths it is the faster one
    soff = {t: {k[4] for k in kernels("passes_L1024.o") if k[0] == t} for t in (b"d", b"f")}
    assert soff == {b"d": {b"0"}, b"f": {b"0", b"1"}}
    assert {k[4] for k in kernels("passes_L720.o")} == {b"0", b"1"}
