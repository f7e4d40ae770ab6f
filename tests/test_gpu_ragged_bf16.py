"""bf16 layers of ragged rows and odd kernels, whose operands are read in whole dwords and shifted (ukst_mfma_parts_kernel.h):
tensors that start in the middle of a dword, channels of odd sizes, and NaN right before and after both operands."""
import numpy as np
import pytest

import oracle
from paper_2502_20493_amd import binding as ukst
from paper_2502_20493_amd import workloads as wl
from gpu_util import TOL, check_against_oracle

# B, Cin, Cout, H, W, n, P
SHAPES = [
    (2, 17, 21, 9, 11, 3, 0),     # odd image, one channel past a stage
    (1, 47, 70, 5, 13, 3, 2),     # two tiles of output channels
    (2, 31, 33, 3, 4, 3, 1),      # rows of one piece
    (2, 35, 9, 7, 22, 5, 3),      # even image, odd kernel
    (1, 16, 33, 3, 129, 5, 4),    # one stage
    (3, 33, 64, 33, 31, 5, 2),    # a second last stage of one channel
    (2, 19, 37, 9, 31, 4, 2),     # odd image, even kernel
    (2, 19, 100, 95, 97, 3, 2),   # many tiles: two activation units per thread and one
    (2, 17, 100, 95, 97, 5, 1),
]


def _offset(bits, off):
    """The operand as a view that starts off elements into a buffer whose other elements are NaN."""
    import torch
    buf = np.full(bits.size + 64, 0x7FC0, np.uint16)
    buf[16 + off:16 + off + bits.size] = bits.ravel()
    t = torch.from_numpy(buf.view(np.int16)).view(torch.bfloat16).cuda()
    return t[16 + off:16 + off + bits.size].view(bits.shape)


@pytest.mark.gpu
@pytest.mark.parametrize("xo,wo", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("shape", SHAPES)
def test_any_start(shape, xo, wo):
    import torch
    w = wl.Workload("ragged", 9870 + sum(shape), *shape, "bf16", "normal", "normal:0.5")
    assert ukst.ukst_kernel_name(*shape, ukst.UKST_BF16_F32) == "ukst_mfma_f32_kernel_parts"
    for integer in (True, False):
        print(f"case {shape} {xo} {wo} integer={integer}", flush=True)
        data = wl.generate(w, integer=integer)
        y_ref, S = oracle.naive(data["x"], data["w"], w.P)
        y = torch.full(y_ref.shape, -777.0, device="cuda")
        ukst.ukst_conv_transpose2d(_offset(data["x_bits"], xo), _offset(data["w_bits"], wo), w.P, y=y)
        torch.cuda.synchronize()
        check_against_oracle(y.cpu().numpy(), y_ref, S, TOL["f32"], exact=integer)  # (bf16 products are exact in fp32)
