"""The flags of a solve as the kernels read them (source checks, no GPU): where a block takes
item after item of the Gram-Schmidt lists, another block of the group can raise the error flag
while this one reads it, so the block's waves must share one answer before they part."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_01481_amd", "csrc")


def test_gram_schmidt_items_are_left_by_whole_blocks():
    src = open(os.path.join(CSRC, "batch.hip")).read()
    at = src.index("void bmgs_kernel(")
    body = re.sub(r"//[^\n]*", "", src[at:src.index("__global__", at)])
    assert len(re.findall(r"\bblock_halted\(st, k\)", body)) == 2
    assert not re.search(r"\bhalted\(|->error|->stop", body)
    helper = open(os.path.join(CSRC, "krylov_body.h")).read()
    assert re.search(r"bool block_halted\([^)]*\) \{ return __syncthreads_or\(halted\(st, k\)\) != 0; \}", helper)
