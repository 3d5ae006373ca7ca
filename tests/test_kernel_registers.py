"""No kernel of the library parks more than a few registers in scratch memory.  Every one that the compiler spills is written and
read back in every block: with 22 to 34 of them the instances for a run-time block size lost up to a quarter of their speed."""
import os
import re

import pytest


def test_no_kernel_spills_its_registers():
    from paper_2604_03298_amd import enec
    if not os.path.exists(enec.LIB_PATH):
        from paper_2604_03298_amd import build
        build.build()
    with open(enec.LIB_PATH, "rb") as f:
        data = f.read()
    # the kernels' metadata, written by the compiler: a map per kernel, keys in alphabetical order
    found = dict(re.findall(rb"\.symbol.{1,3}?(_ZN4enec\w+)\.kd.{0,200}?\.vgpr_spill_count(\xcc?.)", data, re.S))
    assert sum(b"15compress_kernel" in name for name in found) == 648          # 108 tuples of widths, 3 group lengths, 2 kinds of block size
    assert {name.decode(): count[-1] for name, count in found.items() if count[-1] > 16} == {}


def test_the_arguments_of_compression_launches_stay_short():
    """Arguments are written over the link for every launch: sixteen tensors' fit in 1704 bytes (the runtime's own among them), and
    the tensors of one block that a launch takes along have to fit in with them (1 KB more cost small calls 1 to 2 %)."""
    from paper_2604_03298_amd import enec
    with open(enec.LIB_PATH, "rb") as f:
        data = f.read()
    found = dict((name.decode(), int.from_bytes(size, "big")) for size, name in
                 re.findall(rb"\.kernarg_segment_size\xcd(..).{0,400}?\.symbol.{1,3}?(_ZN4enec\w+)\.kd", data, re.S))
    takes = {name: size for name, size in found.items() if "CompressArgs" in name and "PbCompressArgs" not in name}
    assert len(takes) == 648 + 9
    assert {name: size for name, size in takes.items() if size > 1704} == {}
