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
    """Arguments are written over the link for every launch: sixteen tensors' fit in 1448 bytes, 1704 with the runtime's own, which
    the kernel for one tuple per tensor does without (its grid is an argument among the others).  Tensors of one block that a
    launch takes along have to fit in with them (1 KB more, and a branch on their number before the grid was known, cost small
    calls 1 to 2 %)."""
    from paper_2604_03298_amd import enec
    with open(enec.LIB_PATH, "rb") as f:
        data = f.read()
    found = dict((name.decode(), int.from_bytes(size, "big")) for size, name in
                 re.findall(rb"\.kernarg_segment_size\xcd(..).{0,400}?\.symbol.{1,3}?(_ZN4enec\w+)\.kd", data, re.S))
    takes = {name: size for name, size in found.items() if "CompressArgs" in name and "PbCompressArgs" not in name}
    assert len(takes) == 648 + 9
    assert {name: size for name, size in takes.items() if size > (1448 if "15compress_kernel" in name else 1704)} == {}


def test_few_instances_hold_the_code_for_tensors_of_one_block():
    """That code is the same in every instance, a quarter of its size, and all of a unit are loaded by a process's first compression:
    only the default block's instances for the tuples that matrices get have it (by the table in LDS that it needs), and none is
    taken from three waves per SIMD to two by it."""
    from paper_2604_03298_amd import enec
    with open(enec.LIB_PATH, "rb") as f:
        data = f.read()
    number = lambda b: b[0] if b[0] < 0x80 else int.from_bytes(b[1:], "big")
    value = rb"([\x00-\x7f]|\xcc.|\xcd..)"
    name = rb"\.symbol.{1,3}?_ZN4enec15compress_kernelILi(\d+)ELi(\d+)ELi(\d)ELi(\d)ELj(\d+)E\w+\.kd"
    found = re.findall(rb"\.group_segment_fixed_size" + value + rb".{0,500}?" + name + rb".{0,200}?\.vgpr_count" + value, data, re.S)
    assert len(found) == 648
    holds = {tuple(map(int, k[1:6])) for k in found if number(k[0]) > 128}
    assert holds == {(m, a, dt, lpg, 14) for dt in (0, 1, 2) for lpg in (1, 2, 4) for a in (1, 2, 3)
                     for m in range(2, (5 if dt == 1 else 8) - a + 1)}
    assert {k[1:6] for k in found if (k[1], k[2], k[3], k[5]) == (b"5", b"0", b"2", b"14") and number(k[-1]) > 168} == set()
