"""Addresses of the FP64 tiles' operands, on the CPU through the functions that
the plans and kernels use."""
import ctypes

import numpy as np
import pytest

from oracle.hpsi import HEff
from paper_2309_16724_amd import binding as B
from paper_2309_16724_amd.synth.problem import random_problem, random_vector


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


def test_operator_arrays_may_lie_at_any_address():
    """The plan's tiles run on the CPU with operator arrays that start between
    two multiples of eight bytes: the same products, bit for bit."""
    prob = random_problem(6, 6, 0, 4, D=60)
    x = random_vector(HEff(prob).size, 5)
    want = B.debug_plan_host_apply(prob, x)[0]
    buf = []
    for data in (prob.left.data, prob.right.data):
        raw = np.zeros(8 * data.size + 16, dtype=np.uint8)
        at = -raw.ctypes.data % 8 + 4
        raw[at:at + 8 * data.size] = np.frombuffer(data.tobytes(), dtype=np.uint8)
        buf.append((raw, raw.ctypes.data + at))
    args = B.ProblemArgs(prob, buf[0][1], buf[1][1])
    y = np.zeros_like(x)
    B.check(B.load().dmrg_debug_plan_host_apply(ctypes.byref(args.s), x.ctypes.data, y.ctypes.data, None, None), B.load())
    assert np.array_equal(y, want)
