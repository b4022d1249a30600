"""LDS of the first-order cross-overlap kernel: the padded count of library
records (csrc/shape_surrogate.hip, fo_cross_padded) is stated once, and the
launch asks for as many as the kernel lays out."""
import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2607_20766_amd", "csrc", "shape_surrogate.hip")


def test_kernel_and_launch_pad_alike():
    src = open(SRC).read()
    kernel = src[src.index("void k_fo_cross("):src.index("void k_fo_cross_rows(")]
    launch = src[src.index("static hipError_t launch_fo_cross_t("):]
    launch = launch[:launch.index("\n}\n")]
    for part in (kernel, launch):
        assert re.findall(r"max_b_pad = ([^;]+);", part) == ["fo_cross_padded<NI, CH>(L.max_atoms)"]
