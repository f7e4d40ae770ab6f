"""Kernel gradients that walk down the rows of the images (ukst_grad_weight_rows.hip): every element against the oracle at
the edges of groups, tiles, stages and chains, operands at any alignment, infinities and NaN next to masked columns."""
import numpy as np
import pytest

import oracle
from paper_2502_20493_amd import binding as ukst
from paper_2502_20493_amd import workloads as wl

pytestmark = pytest.mark.gpu

# B, Cin, Cout, H, W, n, P, dtype: chains a block adds to its copy of dw
SHAPES = [
    ((1, 40, 33, 1, 5, 2, 1, "bf16"), 1),        # one row without rows before it
    ((9, 80, 160, 34, 48, 2, 1, "bf16"), 1),
    ((3, 40, 40, 1, 3, 3, 2, "bf16"), 1),        # rows shorter than a piece
    ((2, 130, 40, 7, 9, 3, 0, "bf16"), 1),       # two groups, seven columns masked; a second tile of input channels
    ((12, 128, 70, 32, 40, 3, 3, "bf16"), 2),    # five groups: the last step half empty
    ((1, 40, 160, 1, 8, 4, 2, "bf16"), 1),       # dy one element before whole 16 bytes
    ((3, 37, 50, 9, 8, 4, 1, "bf16"), 1),
    ((10, 90, 70, 40, 48, 4, 2, "bf16"), 2),
    ((9, 40, 300, 8, 68, 4, 0, "bf16"), 2),      # two column tiles, nine groups
    ((3, 70, 35, 11, 22, 4, 5, "bf16"), 1),      # P beyond the kernel, three groups
    ((2, 40, 32, 1, 8, 5, 3, "bf16"), 1),
    ((5, 80, 33, 37, 65, 5, 1, "bf16"), 2),
    ((2, 66, 33, 13, 14, 5, 4, "bf16"), 1),
    ((7, 90, 33, 38, 64, 2, 1, "f32"), 2),
    ((2, 90, 33, 1, 47, 2, 1, "f32"), 1),
    ((11, 90, 33, 23, 69, 3, 0, "f32"), 2),
    ((10, 80, 33, 13, 64, 4, 1, "f32"), 1),
    ((8, 100, 33, 21, 65, 4, 2, "f32"), 2),
    ((11, 100, 40, 12, 48, 5, 3, "f32"), 2),
    ((9, 100, 300, 1, 68, 5, 2, "f32"), 2),
]


def _mk(shape):
    return wl.Workload("rows", 9850 + sum(shape[:7]), *shape[:7], shape[7], "normal", "normal:0.5")


def _chains(shape):
    """Chains a block adds to its copy, 0 where another kernel takes the layer."""
    v = ukst.lib().ukst_test_plan(2, *shape[:7], 2, ukst.UKST_F32 if shape[7] == "f32" else ukst.UKST_BF16_F32)
    return v & 0xFFFF if v >> 30 & 1 else 0


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("shape,chains", SHAPES)
def test_every_element(shape, chains, integer):
    from gpu_util import TOL, check_elements, run_gpu_grad_weight
    assert min(_chains(shape), 2) == chains
    w = _mk(shape)
    print(f"case {shape} integer={integer}", flush=True)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_weight(data["x"], dyd["dy"], w.n, w.P)
    got = run_gpu_grad_weight(data, dyd, w.dtype, w.n, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)  # (sums of fp32 products, also of bf16 operands)


@pytest.mark.parametrize("dx,dy", [(1, 0), (0, 1), (3, 5)])
@pytest.mark.parametrize("shape", [SHAPES[3][0], SHAPES[5][0], SHAPES[6][0], SHAPES[11][0], SHAPES[15][0], SHAPES[19][0]])
def test_operands_at_element_alignment(shape, dx, dy):
    """The same bits wherever the operands begin, and whatever lies before and behind them."""
    import torch
    B, Cin, Cout, H, W, n, P, dtype = shape
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    OH, OW = ukst.ukst_output_shape(H, W, n, P)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)

    def at(sizes, shift):
        count = int(np.prod(sizes))
        buf = torch.full((count + 16,), float("nan"), dtype=t, device="cuda")
        buf[shift:shift + count] = torch.randn((count,), generator=g, device="cuda").to(t)
        return buf[shift:shift + count].view(*sizes)

    x, d = at((B, Cin, H, W), 0), at((B, Cout, OH, OW), 0)
    want = ukst.ukst_conv_transpose2d_grad_weight(x, d, n, P)
    x2, d2 = at((B, Cin, H, W), dx), at((B, Cout, OH, OW), dy)
    x2.copy_(x)
    d2.copy_(d)
    print(f"case {shape} {dx} {dy}", flush=True)
    assert torch.isfinite(want).all()
    assert torch.equal(ukst.ukst_conv_transpose2d_grad_weight(x2, d2, n, P), want)


@pytest.mark.parametrize("what", ["dy_inf", "dy_nan", "x_inf", "large"])
@pytest.mark.parametrize("shape", [SHAPES[3][0], SHAPES[10][0], SHAPES[17][0]])
def test_operands_that_are_not_finite(shape, what):
    """An infinite or NaN operand reaches the elements whose sums hold it, and no others."""
    import torch
    from test_gpu_small import _kernel_gradient64
    B, Cin, Cout, H, W, n, P, dtype = shape
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    OH, OW = ukst.ukst_output_shape(H, W, n, P)
    g = torch.Generator(device="cuda")
    g.manual_seed(10)
    x = torch.randn((B, Cin, H, W), generator=g, device="cuda").to(t)
    dy = torch.randn((B, Cout, OH, OW), generator=g, device="cuda").to(t)
    scale = 1.0
    if what == "large":  # beyond what the parts hold
        scale = 1e30
        x *= 1e15
        dy *= 1e15
    clean = _kernel_gradient64(x, dy, n, P)
    hit = torch.zeros_like(clean, dtype=torch.bool)
    b, i, j = B - 1, H - 1, W - 1  # the last pixel: its neighbours in memory are masked, or another image's
    if what == "x_inf":
        x[b, 7, i, j] = float("inf")
    elif what != "large":
        oy, ox = min(2 * i + P, OH - 1), min(2 * j + P, OW - 1)
        dy[b, 11, oy, ox] = float("inf") if what == "dy_inf" else float("nan")
    for a in range(n):
        for c in range(n):
            r, q = 2 * i + P - a, 2 * j + P - c
            if what == "x_inf" and 0 <= r < OH and 0 <= q < OW:
                hit[:, 7, a, c] = True
            if what in ("dy_inf", "dy_nan"):
                p, s = oy - P + a, ox - P + c  # the pixel this tap pairs it with
                if p % 2 == 0 and s % 2 == 0 and 0 <= p // 2 < H and 0 <= s // 2 < W:
                    hit[11, :, a, c] = True
    print(f"case {shape} {what}", flush=True)
    got = ukst.ukst_conv_transpose2d_grad_weight(x, dy, n, P).double()
    assert bool(hit.any()) == (what != "large")
    assert torch.equal(~torch.isfinite(got), hit)
    # at most B*H*W products of factors below 6 (times 1e30): 1e-5 of the sum of their magnitudes
    assert ((got - clean).abs()[~hit] <= 1e-5 * 36 * B * H * W * scale).all()
