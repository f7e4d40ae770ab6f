"""The matrix-core kernels on bf16 parts: edges of their tiles (channel tails, ragged columns, several images
per tile), and operands and sums at and beyond the ends of what scaled bf16 parts hold (infinite, NaN, huge, tiny)."""
import numpy as np
import pytest

import oracle
from paper_2502_20493_amd import binding as ukst
from paper_2502_20493_amd import workloads as wl
from gpu_util import TOL, check_against_oracle, run_gpu

pytestmark = pytest.mark.gpu

# B, Cin, Cout, H, W, n, P, dtype
SHAPES = [
    (2, 33, 21, 9, 11, 3, 0, "f32"),     # channel tail of 1, one partial 32-channel block
    (1, 47, 70, 5, 13, 4, 2, "f32"),     # aligned quads, two channel blocks, the second with 6 channels
    (3, 40, 37, 3, 4, 4, 1, "f32"),      # shifted quads, many images per tile
    (2, 51, 5, 7, 19, 2, 0, "f32"),      # n = 2 aligned
    (2, 51, 9, 7, 19, 2, 3, "f32"),      # n = 2 shifted, P beyond the kernel
    (1, 50, 33, 2, 129, 3, 2, "f32"),    # rows longer than a tile's quads
    (1, 36, 30, 40, 117, 3, 1, "f32"),   # 512-quad tiles of 32 channels
    (4, 17, 41, 64, 63, 5, 3, "f32"),    # n = 5: 26 stages of taps, 17 channels
    (9, 18, 35, 33, 61, 5, 0, "f32"),
    (17, 16, 64, 32, 32, 5, 2, "f32"),   # 68 tiles: just beyond one round of the fp32 pipe
    (17, 16, 64, 32, 32, 4, 2, "f32"),
    (2, 45, 33, 9, 11, 5, 3, "f32"),     # the fewest channels that leave the vector ALUs with a single tile
    (2, 17, 21, 9, 11, 3, 0, "bf16"),
    (1, 47, 70, 5, 13, 4, 2, "bf16"),    # rows of no multiple of 4: the last piece starts inside its neighbour
    (3, 24, 37, 3, 4, 4, 1, "bf16"),
    (2, 31, 2, 7, 5, 5, 2, "bf16"),      # thin output
    (2, 35, 9, 7, 19, 2, 3, "bf16"),
    (1, 16, 33, 2, 130, 5, 4, "bf16"),
    (2, 64, 100, 16, 127, 3, 1, "bf16"),
    # 256-quad tiles on eight waves: from 129 of them on
    (2, 17, 70, 95, 97, 5, 0, "f32"),
    (3, 33, 70, 79, 93, 3, 1, "f32"),
    (2, 17, 100, 95, 97, 5, 2, "bf16"),
    (2, 19, 100, 95, 97, 2, 1, "bf16"),
]


def _mk(shape):
    B, Cin, Cout, H, W, n, P, dtype = shape
    return wl.Workload("parts", 9800 + sum(shape[:7]), B, Cin, Cout, H, W, n, P, dtype, "normal", "normal:0.5")


@pytest.mark.parametrize("shape", SHAPES)
def test_tile_edges_every_element(shape):
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    assert ukst.ukst_kernel_name(w.B, w.Cin, w.Cout, w.H, w.W, w.n, w.P, dt) == "ukst_mfma_f32_kernel_parts"
    for integer in (True, False):
        print(f"case {shape} integer={integer}", flush=True)
        data = wl.generate(w, integer=integer)
        y_ref, S = oracle.naive(data["x"], data["w"], w.P)
        y = run_gpu(data, w.dtype, w.P, guard=4096)
        check_against_oracle(y, y_ref, S, TOL["f32"], exact=integer)  # (bf16 products are exact in fp32)


@pytest.mark.parametrize("shape", [SHAPES[13], SHAPES[16], (2, 33, 21, 9, 11, 3, 0, "bf16"), SHAPES[21], SHAPES[22]])
def test_bf16_output_and_epilogue(shape):
    import torch
    from gpu_util import to_device
    w = _mk(shape)
    data = wl.generate(w)
    x, k = to_device(data, w.dtype)
    bias = np.linspace(-1.0, 1.0, w.Cout).astype(np.float32)
    y_ref, S = oracle.naive(data["x"], data["w"], w.P)
    z = np.maximum(y_ref + bias.astype(np.float64)[None, :, None, None], 0.0)
    y = ukst.ukst_conv_transpose2d_bias_act(x, k, w.P, bias=torch.from_numpy(bias).cuda(), act=ukst.UKST_ACT_RELU,
                                            out_bf16=True)
    got = y.float().cpu().numpy().astype(np.float64)
    # the fp32 sum's tolerance and half a bf16 ulp (2^-9 of the value)
    assert (np.abs(got - z) <= TOL["f32"] * S + 2.0 ** -8 * np.abs(z) + 1e-30).all()


@pytest.mark.parametrize("shape", [(2, 41, 24, 9, 12, 4, 2, "f32"), (2, 33, 35, 10, 9, 3, 1, "f32")])
@pytest.mark.parametrize("what", ["inf", "nan", "huge", "tiny", "weight_inf", "all_tiny", "denormal", "zero"])
def test_operands_that_three_parts_do_not_hold(shape, what):
    """Values a bf16 part cannot carry reach the outputs they reach in fp32 arithmetic, and no others."""
    import torch
    w = _mk(shape)
    data = wl.generate(w)
    x, k = data["x"].copy(), data["w"].copy()
    if what == "inf":
        x[0, 3, 2, 4], x[1, 7, 0, 0] = np.inf, -np.inf
    elif what == "nan":
        x[1, 5, 3, 3] = np.nan
    elif what == "huge":
        x[0, 1, 4, 4], k[2, 1, 1, 1] = 3.4e38, 1e-3  # rounds up to infinity as a bf16
    elif what == "tiny":
        x[0, :, 4:6, :] *= np.float32(1e-36)
    elif what == "weight_inf":
        k[3, 2, 1, 1] = np.inf
    elif what == "all_tiny":
        x *= np.float32(1e-34)
    elif what == "denormal":
        x *= np.float32(1e-41)
    elif what == "zero":
        x[0] = 0.0
    assert ukst.ukst_kernel_name(w.B, w.Cin, w.Cout, w.H, w.W, w.n, w.P, ukst.UKST_F32) == "ukst_mfma_f32_kernel_parts"
    y = ukst.ukst_conv_transpose2d(torch.from_numpy(x).cuda(), torch.from_numpy(k).cuda(), w.P).cpu().numpy()
    fin = lambda a: np.where(np.isfinite(a), a, 0.0).astype(np.float32)
    ref, S = oracle.naive(fin(x), fin(k), w.P)
    # which outputs an infinite or NaN operand reaches, and with what
    x64, k64 = torch.from_numpy(x).double(), torch.from_numpy(k).double()
    full = torch.nn.functional.conv_transpose2d(x64, k64.flip(2, 3).transpose(0, 1), stride=2, padding=0).numpy()
    lo = w.n - 1 - w.P
    full = full[:, :, lo:full.shape[2] - lo, lo:full.shape[3] - lo]
    with np.errstate(over="ignore"):
        full = full.astype(np.float32).astype(np.float64)  # (sums beyond fp32 are infinite)
    assert np.array_equal(np.isnan(full), np.isnan(y))
    inf = np.isinf(full)
    assert np.array_equal(inf, np.isinf(y)) and np.array_equal(full[inf], y[inf])
    ok = np.isfinite(full)
    # (5e-43: half a unit of the smallest fp32 number for each of 41 x 16 products)
    assert (np.abs(y[ok].astype(np.float64) - ref[ok]) <= 1e-5 * S[ok] + 5e-43).all()


@pytest.mark.parametrize("dx,dw,dy", [(1, 0, 0), (0, 1, 0), (0, 0, 1), (3, 3, 3)])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[8], SHAPES[13], SHAPES[14], SHAPES[17]])
def test_operands_at_element_alignment(shape, dx, dw, dy):
    """x, w and y that start dx, dw and dy elements past 16 bytes: 16- and 8-byte loads at 4 and 2 bytes."""
    import torch
    from gpu_util import to_device
    w = _mk(shape)
    data = wl.generate(w, integer=True)
    x, k = to_device(data, w.dtype)

    def off(t, n):
        buf = torch.empty(t.numel() + 64, dtype=t.dtype, device="cuda")
        assert buf.data_ptr() % 16 == 0
        return buf[n:n + t.numel()].view(t.shape).copy_(t)
    OH, OW = oracle.out_shape(w.H, w.W, w.n, w.P)
    y = off(torch.full((w.B, w.Cout, OH, OW), -777.0, device="cuda"), dy)
    ukst.ukst_conv_transpose2d(off(x, dx), off(k, dw), w.P, y=y)
    y_ref, S = oracle.naive(data["x"], data["w"], w.P)
    check_against_oracle(y.cpu().numpy(), y_ref, S, TOL["f32"], exact=True)


@pytest.mark.parametrize("out_bf16", [False, True])
@pytest.mark.parametrize("what", ["weight_inf", "inf", "nan"])
@pytest.mark.parametrize("shape", [(2, 17, 21, 9, 11, 3, 0, "bf16"), (2, 31, 34, 7, 10, 5, 3, "bf16"),
                                   (1, 47, 70, 5, 13, 4, 2, "bf16")])
def test_bf16_operands_that_are_not_finite(shape, what, out_bf16):
    """They reach the outputs whose sums hold them: the halo is left out, not multiplied by zero."""
    import torch
    w = _mk(shape)
    data = wl.generate(w)
    x, k = data["x"].copy(), data["w"].copy()
    if what == "weight_inf":
        k[3, 2, 0, 1], k[4, 16, w.n - 1, w.n - 1] = np.inf, -np.inf
    else:
        x[0, 3, 2, 4], x[w.B - 1, 7, 0, 0] = (np.inf, -np.inf) if what == "inf" else (np.nan, np.nan)
    assert ukst.ukst_kernel_name(w.B, w.Cin, w.Cout, w.H, w.W, w.n, w.P, ukst.UKST_BF16_F32) == "ukst_mfma_f32_kernel_parts"
    put = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    y = ukst.ukst_conv_transpose2d(put(x), put(k), w.P, out_bf16=out_bf16).float().cpu().numpy()
    ref = torch.nn.functional.conv_transpose2d(torch.from_numpy(x).double(),
                                               torch.from_numpy(k).double().flip(2, 3).transpose(0, 1), stride=2)
    pad = w.P - (w.n - 1)
    ref = torch.nn.functional.pad(ref, (pad, pad, pad, pad)).numpy()
    assert np.array_equal(np.isnan(ref), np.isnan(y))
    inf = np.isinf(ref)
    assert np.array_equal(inf, np.isinf(y)) and np.array_equal(ref[inf], y[inf])
    ok = np.isfinite(ref)
    # (one bf16 rounding; up to 47 x 9 products of a few units in fp32)
    assert (np.abs(y[ok] - ref[ok]) <= 2.0 ** -8 * np.abs(ref[ok]) + 1e-3).all()


# scales of x and w.  Products of 2e-38 and less are denormal; 1e25 and 1e30 are beyond the range that the scaled
# parts hold; sums of 1e26 fit fp32 but not a sum that is 2^48 times as large
@pytest.mark.parametrize("sx,sw", [(1e-19, 1e-19), (1e-22, 1e-17), (1e-28, 1e-12), (1e25, 1e-20), (1e30, 1e-36),
                                   (1e13, 1e13)])
@pytest.mark.parametrize("shape", [(2, 41, 24, 9, 12, 4, 2, "f32"), (2, 33, 35, 10, 9, 3, 1, "f32")])
def test_products_at_the_ends_of_the_range(shape, sx, sw):
    import torch
    w = _mk(shape)
    data = wl.generate(w)
    x, k = data["x"] * np.float32(sx), data["w"] * np.float32(sw)
    y = ukst.ukst_conv_transpose2d(torch.from_numpy(x).cuda(), torch.from_numpy(k).cuda(), w.P).cpu().numpy()
    ref, S = oracle.naive(x, k, w.P)
    # (1.4e-45 for each of up to 41 x 16 / 4 products, were each rounded to a denormal)
    assert (np.abs(y.astype(np.float64) - ref) <= 1e-5 * S + 164 * 1.4e-45).all()


def _time(call):
    import torch
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("op", ["forward", "strided", "grad_input", "grad_weight"])
def test_tiny_operands_cost_no_time(op):
    """One weight (or gradient element) in 64 channels far below the smallest bf16 product, or all of them: the same
    kernel in the same time (2 times: the clock; a tile summed again costs ten times and more)."""
    import torch
    B, C, H, n, P = 16, 128, 40, 3, 1
    g = torch.Generator(device="cuda").manual_seed(5)
    OH, OW = ukst.ukst_output_shape(H, H, n, P)
    x, w, dy = (torch.randn(s, generator=g, device="cuda") for s in ((B, C, H, H), (C, C, n, n), (B, C, OH, OW)))
    calls = {"forward": lambda: ukst.ukst_conv_transpose2d(x, w, P),
             "strided": lambda: ukst.ukst_conv_transpose2d_strided(x, w, P, 3),
             "grad_input": lambda: ukst.ukst_conv_transpose2d_grad_input(dy, w, H, H, P),
             "grad_weight": lambda: ukst.ukst_conv_transpose2d_grad_weight(x, dy, n, P)}
    plain = _time(calls[op])
    w[::64, 3, 1, 1] = 1e-35
    dy[:, ::32, 3, 1] = 1e-41
    some = _time(calls[op])
    w *= 1e-33
    dy *= 1e-33
    every = _time(calls[op])
    print(op, plain, some, every, flush=True)
    assert some < 2 * plain and every < 2 * plain


# op, k, (B, Cin, Cout, H, W, n, P)
GENERAL_SHAPES = [
    ("strided", 3, (2, 16, 8, 9, 11, 5, 2)),     # classes of 4, 2 and 1 taps
    ("strided", 3, (2, 33, 70, 7, 13, 4, 0)),    # channel tails, input columns that start at 1
    ("strided", 4, (3, 21, 33, 5, 6, 3, 1)),     # classes without taps: zeros
    ("strided", 5, (1, 18, 9, 6, 37, 7, 8)),     # P beyond the kernel
    ("strided", 1, (2, 17, 40, 12, 20, 4, 3)),   # one class
    ("strided", 3, (1, 32, 33, 2, 130, 3, 2)),   # rows longer than half a tile
    ("dilated", 2, (2, 33, 37, 15, 19, 3, 2)),
    ("dilated", 4, (3, 20, 8, 11, 11, 5, 8)),    # several images per tile, mostly halo
    ("dilated", 3, (1, 17, 65, 21, 13, 4, 13)),  # windows that meet no input
    ("dilated", 1, (2, 32, 9, 8, 70, 1, 0)),     # a single tap
    # few channels and at most a tap per class: the vector ALUs, beside the first layers that leave them
    ("strided", 8, (2, 17, 8, 9, 11, 3, 1)),
    ("strided", 8, (2, 20, 8, 9, 11, 3, 1)),
    ("strided", 2, (2, 19, 40, 12, 13, 2, 0)),
    ("dilated", 3, (2, 19, 9, 8, 70, 1, 0)),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", GENERAL_SHAPES)
def test_general_operations_on_the_matrix_cores(case, dtype):
    from test_gpu_general import _run
    op, k, shape = case
    w = wl.Workload("general_parts", 9900 + sum(shape) + k, *shape, dtype, "normal", "normal:0.5")
    _run(op, w, k, integer=True)
    _run(op, w, k, integer=False)


@pytest.mark.parametrize("what", ["inf", "nan", "all_tiny", "large", "bf16_weight_inf"])
def test_general_operations_with_operands_that_three_parts_do_not_hold(what):
    import torch
    rng = np.random.default_rng(31)
    x = rng.normal(size=(2, 17, 9, 10)).astype(np.float32)
    w = rng.normal(size=(9, 17, 3, 3)).astype(np.float32)
    if what == "bf16_weight_inf":  # the padding is left out, not multiplied
        x, w = (wl.bf16_bits_to_f32(wl.round_to_bf16_bits(a)) for a in (x, w))
        w[4, 3, 0, 1] = np.inf
        put = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
        y = ukst.ukst_dilated_conv2d(put(x), put(w), 2, 2).cpu().numpy()
        assert np.isfinite(y[:, [0, 1, 2, 3, 5, 6, 7, 8]]).all() and not np.isnan(y).any()
        assert np.isfinite(y[:, 4, :2]).all() and np.isinf(y[:, 4, 2:]).all()
        return
    if what == "all_tiny":
        x *= np.float32(1e-34)
    elif what == "large":  # sums beyond 2^80
        x *= np.float32(1e15)
        w *= np.float32(1e15)
    else:
        x[1, 4, 3, 5] = np.inf if what == "inf" else np.nan
    x64, w64 = torch.from_numpy(x).double(), torch.from_numpy(w).double()
    for got, ref in (
            (ukst.ukst_conv_transpose2d_strided(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 2, 3),
             torch.nn.functional.conv_transpose2d(x64, w64.flip(2, 3).transpose(0, 1), stride=3)),
            (ukst.ukst_dilated_conv2d(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 0, 2),
             torch.nn.functional.conv2d(x64, w64, dilation=2))):
        got, ref = got.cpu().numpy(), ref.numpy()
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.isinf(got), np.isinf(ref))
        ok = np.isfinite(ref)
        # 153 products of at most |x| |w| < 25 units of x's scale: 1e-5 of their sum
        scale = {"all_tiny": 1e-34, "large": 1e30}.get(what, 1.0)
        assert (np.abs(got[ok] - ref[ok]) <= 1e-5 * 153 * 25 * scale + 1e-44).all()


@pytest.mark.parametrize("shape", [
    (1, 512, 40, 3, 4, 4, 2),    # small tiles of the fp32 pipe in slices of one stage, ragged channel block
    (60, 512, 24, 4, 4, 4, 2),   # slices of two stages
    (60, 376, 72, 8, 8, 4, 2),   # bf16 parts, slices of 16 channels, a half stage at the end
])
def test_slices_of_the_input_channels(shape):
    """Layers of few tiles with a workspace: partial sums per slice of the input channels, with the epilogue on
    their sum; without one, or with one that is too small for the slices, the unsliced kernel."""
    import torch
    B, Cin, Cout, H, W, n, P = shape
    w = wl.Workload("slices", 9700 + sum(shape), *shape, "f32", "normal", "normal:0.5")
    need = ukst.ukst_workspace_bytes(ukst.UKST_OP_FORWARD, *shape, ukst.UKST_F32)
    assert need > 0
    data = wl.generate(w)
    y_ref, S = oracle.naive(data["x"], data["w"], P)
    bias = np.linspace(-1.0, 1.0, Cout).astype(np.float32)
    z = np.maximum(y_ref + bias.astype(np.float64)[None, :, None, None], 0.0)
    x, k, b = (torch.from_numpy(a).cuda() for a in (data["x"], data["w"], bias))
    for space in (None, False, torch.empty(256, dtype=torch.uint8, device="cuda")):
        y = ukst.ukst_conv_transpose2d_ws(x, k, P, bias=b, act=ukst.UKST_ACT_RELU, workspace=space)
        print(shape, space is None, flush=True)
        err = np.abs(y.cpu().numpy().astype(np.float64) - z)
        assert (err <= 1e-5 * S + 1.2e-7 * np.abs(y_ref)).all()
    one, two = (ukst.ukst_conv_transpose2d_ws(x, k, P) for _ in range(2))
    assert torch.equal(one, two)


# B, Cin, Cout, H, W, n, P, dtype
GRAD_WEIGHT_SHAPES = [
    (3, 33, 34, 65, 63, 3, 0, "f32"),     # channel tails, odd rows, a second column tile of 31
    (1, 40, 70, 96, 90, 4, 1, "f32"),     # tap rows in two halves, third column tile of 26
    (40, 32, 33, 13, 20, 3, 2, "f32"),    # 20 of 32 columns, several images per slice
    (33, 65, 32, 16, 16, 4, 2, "f32"),    # 16-column tiles, two rows per stage
    (3, 33, 34, 65, 63, 4, 2, "bf16"),
    (3, 40, 36, 64, 49, 3, 1, "bf16"),
]
# from 100 tiles of 256 pixels on
GRAD_INPUT_SHAPES = [
    (3, 66, 17, 100, 90, 3, 1),           # eight waves, two channels of the second group, one channel past a stage
    (7, 33, 20, 61, 61, 4, 0),            # four waves
    (2, 72, 16, 128, 101, 5, 2),          # classes of 9, 6, 6 and 4 taps
    (26, 40, 16, 32, 32, 5, 2),           # the same on four waves
    (2, 35, 18, 120, 110, 2, 1),          # one tap per class
    (26, 33, 16, 31, 33, 7, 9),           # P beyond the kernel
    (420, 34, 16, 8, 8, 3, 0),            # four images per tile
]


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("shape", GRAD_WEIGHT_SHAPES)
def test_kernel_gradient_from_parts(shape, integer):
    from gpu_util import check_elements, run_gpu_grad_weight
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    assert ukst.ukst_grad_kernel_name(1, *shape[:7], dt) == "ukst_grad_weight_mfma_kernel_parts"
    print(f"case {shape} integer={integer}", flush=True)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_weight(data["x"], dyd["dy"], w.n, w.P)
    got = run_gpu_grad_weight(data, dyd, w.dtype, w.n, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)


@pytest.mark.parametrize("shape", [(2, 530, 256, 4, 16, 4, 2, "bf16"), (2, 530, 256, 5, 7, 3, 1, "f32")])
def test_sum_of_the_copies_of_many_channel_pairs(shape):
    """From 2048 runs of 64 input channels on the copies are turned through LDS; the last run here has 18."""
    from gpu_util import check_elements, run_gpu_grad_weight
    w = _mk(shape)
    data = wl.generate(w, integer=True)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=True)
    ref, S = oracle.grad_weight(data["x"], dyd["dy"], w.n, w.P)
    check_elements(run_gpu_grad_weight(data, dyd, w.dtype, w.n, w.P, guard=4096), ref, S, TOL["f32"], exact=True)


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("shape", GRAD_INPUT_SHAPES)
def test_input_gradient_from_parts(shape, integer):
    from gpu_util import check_elements, run_gpu_grad_input
    w = _mk(shape + ("f32",))
    assert ukst.ukst_grad_kernel_name(0, *shape, ukst.UKST_F32) == "ukst_grad_input_mfma_kernel_parts"
    print(f"case {shape} integer={integer}", flush=True)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_input(dyd["dy"], data["w"], w.H, w.W, w.P)
    got = run_gpu_grad_input(data, dyd, w.dtype, w.H, w.W, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)


@pytest.mark.parametrize("what,dtype", [("inf", "f32"), ("nan", "f32"), ("tiny", "f32"), ("large", "f32"),
                                        ("inf", "bf16"), ("nan", "bf16"), ("x_inf", "bf16")])
def test_gradients_with_operands_that_three_parts_do_not_hold(what, dtype):
    """An infinite or NaN gradient reaches the elements whose sums hold it, and no others; tiny ones keep their bits."""
    import torch
    import torch.nn.functional as F
    B, Cin, Cout, H, W, n, P = 7, 33, 34, 61, 61, 3, 1
    rng = np.random.default_rng(77)
    x = rng.normal(size=(B, Cin, H, W)).astype(np.float32)
    w = rng.normal(size=(Cout, Cin, n, n)).astype(np.float32)
    OH, OW = oracle.out_shape(H, W, n, P)
    dy = rng.normal(size=(B, Cout, OH, OW)).astype(np.float32)
    scale = 1.0
    if what == "tiny":
        scale = 1e-33
        dy *= np.float32(scale)
    elif what == "large":  # sums beyond 2^80
        scale = 1e30
        for t in (x, w, dy):
            t *= np.float32(1e15)
    elif what == "x_inf":
        x[4, 9, 30, 20] = np.inf
    else:
        dy[2, 5, 40, 7] = np.inf if what == "inf" else np.nan
    if dtype == "bf16":
        x, w, dy = (np.where(np.isfinite(a), wl.bf16_bits_to_f32(wl.round_to_bf16_bits(a)), a) for a in (x, w, dy))
    code = ukst.UKST_F32 if dtype == "f32" else ukst.UKST_BF16_F32
    shape = (B, Cin, Cout, H, W, n, P)
    assert ukst.ukst_grad_kernel_name(1, *shape, code) == "ukst_grad_weight_mfma_kernel_parts"
    if dtype == "f32":
        assert ukst.ukst_grad_kernel_name(0, *shape, code) == "ukst_grad_input_mfma_kernel_parts"
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    xg, wg, dg = (torch.from_numpy(a).to(tt).cuda() for a in (x, w, dy))
    dx = ukst.ukst_conv_transpose2d_grad_input(dg, wg, H, W, P).cpu().double()
    dw = ukst.ukst_conv_transpose2d_grad_weight(xg, dg, n, P).cpu().double()
    x64, w64, d64 = (torch.from_numpy(a).double() for a in (x, w, dy))
    rx = F.conv2d(d64, w64.flip(2, 3).transpose(0, 1).contiguous(), stride=2, padding=n - 1 - P)
    padded = F.pad(d64, (n - 1, n - 1, n - 1, n - 1))
    rw = torch.zeros(Cout, Cin, n, n, dtype=torch.float64)
    for a in range(n):
        for c in range(n):
            d = padded[:, :, n - 1 + P - a:, n - 1 + P - c:][:, :, :2 * H:2, :2 * W:2][:, :, :H, :W]
            # (finite factors first: an infinite one meets every input channel of its output channel)
            rw[:, :, a, c] = d.transpose(0, 1).reshape(Cout, -1) @ x64.transpose(0, 1).reshape(Cin, -1).t()
    # sums of up to 26047 products of factors below 6 (and dy's scale): 1e-5 of the sum of their magnitudes
    # (the bf16 input gradient is another kernel)
    for got, ref, terms in ((dx, rx, Cout * n * n), (dw, rw, B * H * W))[0 if dtype == "f32" else 1:]:
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
        ok = torch.isfinite(ref)
        assert (~ok).any() == (what in ("inf", "nan", "x_inf"))
        assert ((got - ref).abs()[ok] <= 1e-5 * terms * scale).all()
