"""What the compiler says about the kernels of the built library: none keeps its tiles in scratch memory.  (Every
kernel is laid out so that its tiles fit the register file; one that spills them answers correctly but pays for it
on each pass, most where its loop is short.)"""
import re

from paper_2605_24022_amd import binding as B


def _scratch_bytes(data):
    """(kernel, bytes of scratch memory per lane) from the MessagePack metadata of the library's code objects."""
    names = [(m.start(), m.group(1).decode()) for m in re.finditer(rb"\.symbol(?:[\xa0-\xbf]|\xd9.|\xda..)(_Z\w+?)\.kd", data, re.S)]
    out = []
    for m in re.finditer(rb"\.private_segment_fixed_size", data):
        tag = data[m.end()]
        size = tag if tag < 0x80 else int.from_bytes(data[m.end() + 1:m.end() + 1 + (1 << (tag - 0xcc))], "big")
        out.append((next(n for at, n in names if at > m.start()), size))     # a kernel's keys are in alphabetical order
    return out


def test_no_kernel_keeps_tiles_in_scratch_memory():
    B.load()
    with open(B.LIB_PATH, "rb") as f:
        kernels = _scratch_bytes(f.read())
    assert len(kernels) > 30 and len({n for n, _ in kernels}) == len(kernels), "kernel metadata not found"
    assert [k for k in kernels if k[1] > 0] == []
