"""The kernels of the accept pass need no scratch memory.  Their workgroups wait for one another, and the first launch with
scratch in a process is held up while it is allocated: waits ran out and every slice was computed many times over."""
import re

from paper_2502_20330_amd import binding, build


def private_bytes(image: bytes) -> dict:
    """Kernel name -> private segment size, out of the code objects' metadata (msgpack: a short name, then the size)."""
    sizes = {}
    for m in re.finditer(rb"\.name(?:\xd9.|[\xa0-\xbf])(\w+)\xbb\.private_segment_fixed_size([\x00-\x7f]|\xcc.|\xcd..|\xce....)", image, re.S):
        sizes[m.group(1).decode()] = m.group(2)[0] if len(m.group(2)) == 1 else int.from_bytes(m.group(2)[1:], "big")
    return sizes


def test_accept_kernels_need_no_scratch():
    with open(build.LIB, "rb") as f:
        sizes = {k: v for k, v in private_bytes(f.read()).items() if "accept_" in k or "greedy_" in k}
    assert binding.LIB_PATH == build.LIB and len(sizes) >= 16         # 7 + 7 of the general pass, 2 of the greedy one
    assert not any(sizes.values()), {k: v for k, v in sizes.items() if v}
