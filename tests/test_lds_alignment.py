"""The LDS that a census tile is made in is read and written 16 bytes at a time, so every kernel that
makes a tile has to declare it as aligned as that (a compiler may choose to align an LDS array
further than its type, but does not have to). No GPU."""
import os

from paper_2604_07980_amd import build


def test_every_kernel_that_makes_a_tile_declares_it_aligned():
    text = "".join(open(os.path.join(build.CSRC, f)).read() for f in ("census.hip", "match.hip", "fused.hip"))
    decls = [l for l in text.splitlines() if "__shared__" in l and ("CensusTile" in l or "[(kLds + 7) / 8]" in l)]
    assert len(decls) == 4
    assert all("alignas(dev::kCensusLdsAlign)" in l for l in decls)
