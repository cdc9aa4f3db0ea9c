"""Addresses of the FP64 wavefront tiles' operands, on the CPU through the
function that the kernels use."""
import pytest

from paper_2309_16724_amd import binding as B


@pytest.mark.parametrize("pos,pos_stride,row,row_stride,line,line_stride", [
    (3, 83 * 70, 1, 83, 17, 1),
    (1, 65536 * 65536, 0, 65536, 0, 1),             # an operator block of 2^32 elements
    (3, 65536 * 65537, 65536, 65536, 65535, 1),
    (1431, 70001 * 70003, 70000, 70003, 70002, 1),
    (0, 0, 65535, 2 ** 31, 3, 1),                   # a stripe of 2^31 columns
    (0, 0, 0, 1, 2 ** 31 - 1, 2 ** 31 - 1),         # lines along a column
])
def test_operand_offsets_are_exact(pos, pos_stride, row, row_stride, line, line_stride):
    want = pos * pos_stride + row * row_stride + line * line_stride
    assert B.load().dmrg_debug_operand_offset(pos, pos_stride, row, row_stride, line, line_stride) == want
