"""The library is compiled in parts; every kernel belongs to one of them.  (A
kernel that a function outside the part tables names would be compiled into
every part: its name then stands in the library once more for each.)"""
import re

from paper_2609_04910_amd import build as hip_build
from paper_2609_04910_amd import gauss_sum as gs


def test_each_kernel_is_compiled_into_one_part():
    gs.load(torch_runtime=False)
    with open(hip_build.LIB, "rb") as f:
        data = f.read()
    once = data.count(b"k_prep_max")            # a kernel of part 0: its mentions in one code object and the host part
    names = set(re.findall(rb"_ZN2gs\d+k_[a-z0-9_]+I\w*?EEv", data)) | {b"7k_fwd32ILi1EE", b"8k_fwd32cILi2ELi4EE"}
    assert once > 0 and len(names) > 100
    counts = {n: data.count(n) for n in names}
    assert max(counts.values()) <= 2 * once, max(counts.items(), key=lambda x: x[1])
