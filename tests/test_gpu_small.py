"""The small tiles of the fp32 matrix pipe (layers of few tiles and a long sum): tails of the channels and of the tiles,
several images per tile, every quad alignment, the last stage that repeats channels, and operands that are not finite."""
import numpy as np
import pytest

import oracle
from paper_2502_20493_amd import binding as ukst
from paper_2502_20493_amd import workloads as wl
from gpu_util import TOL, check_against_oracle, run_gpu

pytestmark = pytest.mark.gpu

# B, Cin, Cout, H, W, n, P, dtype; in tiles of 16 x 16 but for one
FORWARD_SHAPES = [
    (1, 52, 8, 4, 4, 4, 2, "f32"),       # one tile of 16 x 16, half of it empty
    (3, 53, 33, 5, 7, 4, 2, "f32"),      # a last stage of one new channel, a second channel tile of one
    (5, 61, 40, 5, 5, 3, 0, "f32"),      # several images per tile, odd output
    (2, 70, 65, 9, 17, 2, 0, "f32"),     # columns in three tiles of six
    (2, 66, 17, 6, 9, 2, 3, "f32"),      # P beyond the kernel
    (1, 101, 35, 33, 11, 5, 4, "f32"),   # n = 5, seven and a half windows of P
    (64, 128, 64, 6, 6, 4, 2, "f32"),    # 32 x 32, blocks of eight waves
    (3, 97, 4, 8, 8, 5, 1, "f32"),       # a thin output
    (3, 60, 33, 5, 7, 4, 1, "bf16"),
    (2, 77, 35, 7, 5, 5, 3, "bf16"),
    (9, 64, 40, 3, 3, 3, 2, "bf16"),
]

# ... on every instance of 32 x 32 tiles: output-aligned and shifted quads, every kernel side, eight and four waves
FORWARD_SHAPES_32 = [(s, 8) for s in [
    (15, 73, 33, 4, 16, 2, 2, "f32"), (9, 63, 37, 4, 3, 4, 0, "f32"),
    (5, 61, 34, 7, 40, 2, 1, "f32"), (15, 53, 55, 3, 13, 3, 3, "f32"), (14, 53, 49, 16, 4, 4, 3, "f32"), (11, 56, 48, 3, 6, 5, 0, "f32"),
    (11, 55, 34, 8, 12, 2, 2, "bf16"), (13, 82, 35, 3, 3, 4, 0, "bf16"),
    (4, 53, 37, 9, 37, 2, 1, "bf16"), (7, 53, 49, 11, 9, 3, 3, "bf16"), (13, 59, 65, 17, 3, 4, 3, "bf16"), (4, 78, 52, 6, 3, 5, 0, "bf16"),
]] + [(s, 4) for s in [
    (14, 56, 34, 7, 35, 2, 2, "f32"), (14, 59, 34, 55, 4, 4, 4, "f32"),
    (4, 64, 36, 39, 26, 2, 1, "f32"), (10, 66, 34, 13, 7, 3, 3, "f32"), (9, 55, 34, 8, 49, 4, 3, "f32"), (14, 53, 34, 51, 3, 5, 5, "f32"),
    (6, 57, 71, 22, 19, 4, 2, "bf16"), (9, 66, 34, 24, 4, 3, 3, "bf16"), (8, 78, 37, 22, 17, 5, 5, "bf16"),
]]


def _plan(op, shape, dtype="f32", k=2):
    """What the dispatch of ukst_internal.h says: tile rows, waves, slices on the small tiles (zeros elsewhere); of a kernel
    gradient, the stages after which its sums are added to memory, and the stages of a slice."""
    v = ukst.lib().ukst_test_plan(("forward", "grad_input", "grad_weight", "strided", "dilated").index(op), *shape[:7], k,
                                  ukst.UKST_F32 if dtype == "f32" else ukst.UKST_BF16_F32)
    assert v >= 0
    return (v & 0xFFFF, v >> 16) if op == "grad_weight" else (v & 255, v >> 8 & 255, v >> 16)


def _mk(shape):
    B, Cin, Cout, H, W, n, P, dtype = shape
    return wl.Workload("small", 9500 + sum(shape[:7]), B, Cin, Cout, H, W, n, P, dtype, "normal", "normal:0.5")


@pytest.mark.parametrize("shape,tile", [(s, (32, 8) if s[0] == 64 else (16, 8)) for s in FORWARD_SHAPES] +
                         [(s, (32, waves)) for s, waves in FORWARD_SHAPES_32])
def test_forward_every_element(shape, tile):
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    assert ukst.ukst_kernel_name(*shape[:7], dt) == "ukst_mfma_f32_kernel"
    assert _plan("forward", shape, w.dtype) == tile + (1,)
    for integer in (True, False):
        print(f"case {shape} integer={integer}", flush=True)
        data = wl.generate(w, integer=integer)
        y_ref, S = oracle.naive(data["x"], data["w"], w.P)
        y = run_gpu(data, w.dtype, w.P, guard=4096)
        check_against_oracle(y, y_ref, S, TOL["f32"], exact=integer)  # (bf16 products are exact in fp32)


@pytest.mark.parametrize("out_bf16", [False, True])
@pytest.mark.parametrize("act", [ukst.UKST_ACT_RELU, ukst.UKST_ACT_TANH])
def test_epilogue_and_bf16_output(act, out_bf16):
    import torch
    from gpu_util import to_device
    w = _mk(FORWARD_SHAPES[8] if out_bf16 else FORWARD_SHAPES[2])
    data = wl.generate(w)
    x, k = to_device(data, w.dtype)
    bias = np.linspace(-1.0, 1.0, w.Cout).astype(np.float32)
    y_ref, S = oracle.naive(data["x"], data["w"], w.P)
    z = y_ref + bias.astype(np.float64)[None, :, None, None]
    z = np.maximum(z, 0.0) if act == ukst.UKST_ACT_RELU else np.tanh(z)
    y = ukst.ukst_conv_transpose2d_bias_act(x, k, w.P, bias=torch.from_numpy(bias).cuda(), act=act, out_bf16=out_bf16)
    got = y.float().cpu().numpy().astype(np.float64)
    # the fp32 sum, half an ulp of the biased value, the activation's own error, half a bf16 ulp
    slack = TOL["f32"] * S + 1.2e-7 * np.abs(y_ref) + (2e-6 if act == ukst.UKST_ACT_TANH else 0.0)
    assert (np.abs(got - z) <= slack + (2.0 ** -8 * np.abs(z) if out_bf16 else 0.0)).all()


@pytest.mark.parametrize("what", ["weight_inf", "inf", "nan", "huge"])
@pytest.mark.parametrize("shape", [FORWARD_SHAPES[1], FORWARD_SHAPES[2], FORWARD_SHAPES[9], FORWARD_SHAPES_32[1][0],
                                   FORWARD_SHAPES_32[15][0], FORWARD_SHAPES_32[11][0]])
def test_forward_operands_that_are_not_finite(shape, what):
    """They reach the outputs whose sums hold them: the halo is left out, not multiplied by zero, and neither are the
    channels that a last stage repeats."""
    import torch
    w = _mk(shape)
    data = wl.generate(w)
    x, k = data["x"].copy(), data["w"].copy()
    if what == "weight_inf":
        k[3, 2, 0, 1], k[4, w.Cin - 3, w.n - 1, w.n - 1] = np.inf, -np.inf
    elif what == "huge":
        x[0, 5, 2, w.W // 2] = 3e38
        k[:, 5] *= 100.0
    else:
        x[0, 3, 2, w.W - 1], x[w.B - 1, w.Cin - 4, 0, 0] = (np.inf, -np.inf) if what == "inf" else (np.nan, np.nan)
    dt = torch.float32 if w.dtype == "f32" else torch.bfloat16
    x, k = torch.from_numpy(x).to(dt), torch.from_numpy(k).to(dt)
    y = ukst.ukst_conv_transpose2d(x.cuda(), k.cuda(), w.P).cpu().numpy()
    # (products that overflow do so in any order of the sums: 3e38 against weights of 100 and more)
    ref = torch.nn.functional.conv_transpose2d(x.double(), k.double().flip(2, 3).transpose(0, 1), stride=2)
    pad = w.P - (w.n - 1)
    ref = torch.nn.functional.pad(ref, (pad, pad, pad, pad)).numpy()
    with np.errstate(over="ignore"):
        ref32 = ref.astype(np.float32)
    assert np.array_equal(np.isnan(ref32), np.isnan(y))
    inf = np.isinf(ref32)
    assert np.array_equal(inf, np.isinf(y)) and np.array_equal(ref32[inf], y[inf])
    ok = np.isfinite(ref32)
    scale = 3e38 * 1e2 * 1e-7 if what == "huge" else 1.0
    assert (np.abs(y[ok] - ref32[ok]) <= 1e-5 * np.abs(ref32[ok]) + 1e-3 * scale).all()


def test_element_alignment_and_repeat_runs():
    import torch
    from gpu_util import to_device
    for shape in (FORWARD_SHAPES[2], FORWARD_SHAPES[9]):
        w = _mk(shape)
        data = wl.generate(w, integer=True)
        x, k = to_device(data, w.dtype)

        def off(t, n):
            buf = torch.empty(t.numel() + 64, dtype=t.dtype, device="cuda")
            return buf[n:n + t.numel()].view(t.shape).copy_(t)
        y = ukst.ukst_conv_transpose2d(off(x, 1), off(k, 3), w.P)
        y_ref, S = oracle.naive(data["x"], data["w"], w.P)
        check_against_oracle(y.cpu().numpy(), y_ref, S, TOL["f32"], exact=True)
        a, b = (ukst.ukst_conv_transpose2d(x, k, w.P) for _ in range(2))
        assert torch.equal(a, b)


# B, Cin, Cout, H, W, n, P, dtype
GRAD_INPUT_SHAPES = [
    (3, 17, 9, 5, 5, 4, 2, "f32"),       # several images per tile, two channel tiles of 16, a stage of nine channels
    (2, 33, 40, 7, 19, 3, 0, "f32"),     # odd rows of dy
    (1, 70, 53, 11, 6, 5, 4, "f32"),     # a last stage of one new channel
    (5, 40, 24, 3, 4, 2, 1, "f32"),
    (2, 16, 30, 9, 9, 4, 6, "f32"),      # P beyond the kernel
    (9, 130, 72, 6, 7, 4, 1, "bf16"),
    (2, 24, 37, 9, 10, 3, 2, "bf16"),
    (2, 19, 16, 6, 5, 5, 0, "bf16"),     # an odd number of channels of 25 taps
    (1, 35, 38, 4, 5, 2, 1, "f32"), (2, 17, 34, 4, 5, 2, 0, "bf16"),
]
# in 32 x 32 tiles: every kernel side, eight and four waves
GRAD_INPUT_SHAPES_32 = [(s, 8) for s in [
    (9, 35, 33, 19, 11, 2, 2, "f32"), (3, 33, 19, 39, 11, 3, 2, "f32"), (1, 34, 18, 43, 35, 4, 2, "f32"), (16, 66, 17, 3, 17, 5, 1, "f32"),
    (9, 17, 34, 11, 20, 2, 0, "bf16"), (10, 34, 83, 14, 9, 3, 1, "bf16"), (6, 33, 75, 20, 12, 4, 0, "bf16"), (13, 178, 19, 7, 4, 5, 0, "bf16"),
]] + [(s, 4) for s in [
    (5, 40, 17, 35, 22, 2, 1, "f32"), GRAD_INPUT_SHAPES[3], (5, 39, 19, 41, 19, 3, 1, "f32"), (12, 34, 34, 11, 11, 4, 4, "f32"), (1, 34, 34, 50, 27, 5, 4, "f32"),
    (12, 34, 72, 16, 23, 2, 1, "bf16"), (15, 38, 80, 24, 11, 3, 0, "bf16"), (15, 37, 75, 23, 11, 4, 1, "bf16"), (15, 134, 35, 4, 7, 5, 4, "bf16"),
]]


@pytest.mark.parametrize("integer", [True, False])
@pytest.mark.parametrize("shape,tile", [(s, (16, 8)) for s in GRAD_INPUT_SHAPES if s != GRAD_INPUT_SHAPES[3]] +
                         [(s, (32, waves)) for s, waves in GRAD_INPUT_SHAPES_32])
def test_input_gradient_every_element(shape, tile, integer):
    from gpu_util import check_elements, run_gpu_grad_input
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    if shape[:2] != (2, 19):  # (the vector ALUs keep that one)
        assert ukst.ukst_grad_kernel_name(0, *shape[:7], dt) == "ukst_grad_input_mfma_kernel"
        assert _plan("grad_input", shape, w.dtype) == tile + (1,)
    print(f"case {shape} integer={integer}", flush=True)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_input(dyd["dy"], data["w"], w.H, w.W, w.P)
    got = run_gpu_grad_input(data, dyd, w.dtype, w.H, w.W, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)


# op, step, B, Cin, Cout, H, W, n, P; the last two of each beyond the line, on the kernel for larger layers
GENERAL_SHAPES = [
    ("strided", 3, (2, 17, 9, 7, 9, 4, 2)), ("strided", 4, (1, 53, 33, 6, 11, 5, 3)), ("strided", 4, (3, 20, 16, 5, 5, 3, 7)),
    ("strided", 3, (1, 21, 35, 64, 70, 5, 2)), ("strided", 4, (2, 33, 40, 61, 63, 3, 1)),
    ("dilated", 2, (3, 33, 17, 9, 9, 5, 4)), ("dilated", 3, (2, 61, 40, 10, 17, 3, 4)), ("dilated", 4, (7, 20, 9, 5, 6, 4, 6)),
    ("dilated", 1, (2, 19, 33, 8, 9, 2, 1)), ("dilated", 8, (1, 16, 8, 20, 20, 3, 9)),
    ("dilated", 2, (3, 17, 70, 90, 95, 3, 2)), ("dilated", 3, (2, 20, 100, 101, 97, 4, 5)),
]


# the kernel for larger layers on blocks of 32 channels (no more of them than compute units, fp32 two to one; of 64, they do not fit LDS), the
# small tiles where neither fits, and blocks of 64 on either side
GENERAL_SHAPES += [
    ("dilated", 2, (10, 17, 125, 38, 38, 5, 4)), ("dilated", 2, (10, 17, 70, 38, 38, 5, 4)), ("dilated", 2, (10, 17, 170, 38, 38, 2, 1)),
    ("dilated", 4, (9, 16, 50, 60, 84, 3, 4)), ("dilated", 4, (13, 17, 40, 56, 56, 5, 8)), ("strided", 3, (1, 33, 61, 37, 39, 5, 2)),
    ("dilated", 2, (11, 17, 61, 64, 64, 3, 2)),
    ("strided", 3, (14, 130, 37, 31, 33, 5, 2)),  # classes in order of their taps, two tiles left over
    ("strided", 2, (9, 66, 37, 63, 65, 3, 1)), ("strided", 4, (9, 65, 50, 33, 31, 5, 3)),  # ... of four and of sixteen classes
]

# dilated layers in 32 x 32 tiles: every kernel side, both operand types, eight and four waves (strided ones take 16 x 16)
DILATED_SHAPES_32 = [
    (2, (10, 18, 78, 11, 3, 2, 2), "f32", 8), (3, (5, 45, 41, 11, 3, 3, 2), "f32", 8), (2, (7, 22, 38, 7, 4, 4, 2), "f32", 8),
    (2, (8, 28, 23, 5, 16, 5, 2), "f32", 8), (3, (15, 20, 57, 3, 13, 2, 2), "bf16", 8), (2, (10, 55, 21, 6, 5, 3, 0), "bf16", 8),
    (3, (8, 28, 32, 9, 3, 4, 4), "bf16", 8), (2, (5, 17, 19, 11, 27, 5, 5), "bf16", 8),
    (2, (6, 17, 35, 12, 43, 2, 2), "f32", 4), (2, (8, 19, 33, 3, 13, 3, 1), "f32", 4), (4, (7, 35, 19, 5, 25, 4, 4), "f32", 4),
    (3, (7, 34, 24, 11, 5, 5, 5), "f32", 4), (2, (11, 19, 34, 21, 13, 2, 2), "bf16", 4), (3, (10, 25, 20, 5, 8, 3, 1), "bf16", 4),
    (2, (12, 48, 41, 3, 7, 4, 2), "bf16", 4), (2, (8, 47, 33, 4, 5, 5, 3), "bf16", 4),
]


@pytest.mark.parametrize("case", DILATED_SHAPES_32)
def test_dilated_32_x_32_every_element(case):
    from test_gpu_general import _run
    k, shape, dtype, waves = case
    assert _plan("dilated", shape, dtype, k) == (32, waves, 1)
    w = wl.Workload("small_dilated", 9800 + sum(shape) + k, *shape, dtype, "normal", "normal:0.5")
    _run("dilated", w, k, integer=True)
    _run("dilated", w, k, integer=False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", GENERAL_SHAPES)
def test_strided_and_dilated_every_element(case, dtype):
    from test_gpu_general import _run
    op, k, shape = case
    w = wl.Workload("small_general", 9600 + sum(shape) + k, *shape, dtype, "normal", "normal:0.5")
    _run(op, w, k, integer=True)
    _run(op, w, k, integer=False)


@pytest.mark.parametrize("what", ["inf", "nan", "weight_inf"])
@pytest.mark.parametrize("op,shape,tile", [  # images, summed channels, channels of the result, H, W, n, P, step
    ("grad_input", (2, 53, 20, 6, 7, 3, 1, 3), (16, 8)), ("grad_input", (3, 19, 33, 39, 11, 3, 2, 2), (32, 8)),
    ("strided", (2, 53, 20, 6, 7, 3, 1, 3), (16, 8)),
    ("dilated", (2, 53, 20, 6, 7, 3, 1, 3), (16, 8)), ("dilated", (7, 22, 38, 7, 4, 4, 2, 2), (32, 8)),
    ("dilated", (10, 25, 20, 5, 8, 3, 1, 3), (32, 4)),
])
def test_other_operations_with_operands_that_are_not_finite(op, shape, tile, what):
    """As for the forward layers; against the definitions in 64 bits, products with the padding left out."""
    import torch
    B, K, M, H, W, n, P, k = shape
    cin, cout = (M, K) if op == "grad_input" else (K, M)
    assert _plan(op, (B, cin, cout, H, W, n, P), "f32", k) == tile + (1,)
    rng = np.random.default_rng(7)
    wshape = (K, M, n, n) if op == "grad_input" else (M, K, n, n)
    OH, OW = ukst.ukst_output_shape(H, W, n, P) if op == "grad_input" else (0, 0)
    x = rng.normal(size=(B, K, OH, OW) if op == "grad_input" else (B, K, H, W)).astype(np.float32)
    w = rng.normal(size=wshape).astype(np.float32)
    if what == "weight_inf":
        w[1, 2, 0, 1], w[3, 9, 2, 2] = np.inf, -np.inf
    else:
        x[0, 5, 2, 3], x[1, K - 2, 0, 0] = (np.inf, -np.inf) if what == "inf" else (np.nan, np.nan)
    xt, wt = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    call = {"grad_input": lambda: ukst.ukst_conv_transpose2d_grad_input(xt, wt, H, W, P),
            "strided": lambda: ukst.ukst_conv_transpose2d_strided(xt, wt, P, k),
            "dilated": lambda: ukst.ukst_dilated_conv2d(xt, wt, P, k)}[op]
    y = call().cpu().numpy()
    ref = np.zeros(y.shape)
    with np.errstate(invalid="ignore"):
        for a in range(n):
            for c in range(n):
                for i in range(y.shape[2]):
                    for j in range(y.shape[3]):
                        if op == "grad_input":
                            r, q = 2 * i + P - a, 2 * j + P - c
                        elif op == "dilated":
                            r, q = i - P + k * a, j - P + k * c
                        else:
                            r, q = i - P + a, j - P + c
                            if r % k or q % k:
                                continue
                            r, q = r // k, q // k
                        if 0 <= r < x.shape[2] and 0 <= q < x.shape[3]:
                            t = w[:, :, a, c].astype(np.float64)
                            t = t.T if op == "grad_input" else t
                            ref[:, :, i, j] += (x[:, None, :, r, q].astype(np.float64) * t[None]).sum(-1)
    assert np.array_equal(np.isnan(ref), np.isnan(y))
    inf = np.isinf(ref)
    assert np.array_equal(inf, np.isinf(y)) and np.array_equal(ref[inf], y[inf])
    ok = np.isfinite(ref)
    assert ok.any() and (np.abs(y[ok] - ref[ok]) <= 1e-5 * K * n * n * 16).all()


# B, Cin, Cout, H, W, n, P, dtype
@pytest.mark.parametrize("shape", [
    (2, 17, 40, 33, 35, 5, 2, "bf16"),   # fp32 pipe, widened
    (3, 40, 19, 26, 32, 3, 1, "bf16"),   # bf16 pipe, a channel tile of 8
    (2, 21, 18, 65, 63, 4, 0, "bf16"),   # one part
    (5, 16, 33, 30, 31, 2, 1, "bf16"),
    (4, 18, 37, 33, 35, 5, 2, "f32"),
    (9, 70, 16, 20, 25, 5, 4, "f32"),
])
@pytest.mark.parametrize("integer", [True, False])
def test_kernel_gradient_of_16_to_31_channels(shape, integer):
    from gpu_util import check_elements, run_gpu_grad_weight
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    assert "mfma" in ukst.ukst_grad_kernel_name(1, *shape[:7], dt)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_weight(data["x"], dyd["dy"], w.n, w.P)
    got = run_gpu_grad_weight(data, dyd, w.dtype, w.n, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)


# B, Cin, Cout, H, W, n, P, dtype: stages after which the sums go to memory, stages of a slice
@pytest.mark.parametrize("shape,plan", [
    ((3, 17, 300, 35, 45, 5, 2, "f32"), (2, 5)),     # twice, and a remainder of one
    ((4, 17, 78, 90, 90, 5, 4, "f32"), (1, 4)),      # after every stage
    ((6, 17, 590, 35, 45, 5, 2, "bf16"), (8, 9)),
    ((6, 17, 1200, 35, 45, 2, 1, "bf16"), (8, 17)),  # two sets of accumulators
    ((12, 590, 17, 35, 45, 2, 0, "bf16"), (8, 9)),
    ((3, 17, 1200, 35, 45, 3, 0, "bf16"), (8, 9)),
    ((3, 17, 1200, 35, 45, 4, 3, "bf16"), (8, 9)),
])
@pytest.mark.parametrize("integer", [True, False])
def test_kernel_gradient_sums_added_to_memory_on_the_way(shape, plan, integer):
    from gpu_util import check_elements, run_gpu_grad_weight
    w = _mk(shape)
    assert _plan("grad_weight", shape, w.dtype) == plan
    print(f"case {shape} integer={integer}", flush=True)
    data = wl.generate(w, integer=integer)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P), integer=integer)
    ref, S = oracle.grad_weight(data["x"], dyd["dy"], w.n, w.P)
    got = run_gpu_grad_weight(data, dyd, w.dtype, w.n, w.P, guard=4096)
    check_elements(got, ref, S, TOL["f32"], exact=integer)


def _kernel_gradient64(x, dy, n, P):
    """dw of the definition in 64 bits, from the operands as they are."""
    import torch
    B, Cin, H, W = x.shape
    Cout, OH, OW = dy.shape[1:]
    dw = torch.zeros((Cout, Cin, n, n), dtype=torch.float64, device=x.device)
    # rows of dy from -(n - 1) + P on: the lattice of tap a starts at row P - a
    lo, hi = max(0, n - 1 - P), max(0, 2 * (H - 1) + P - (OH - 1))
    wi = max(0, 2 * (W - 1) + P - (OW - 1))
    for b in range(B):
        xb = x[b].double().reshape(Cin, H * W).t().contiguous()
        d = torch.nn.functional.pad(dy[b].double(), (lo, wi, lo, hi))
        for a in range(n):
            for c in range(n):
                r, q = P - a + lo, P - c + lo
                t = d[:, r:r + 2 * H - 1:2, q:q + 2 * W - 1:2]
                dw[:, :, a, c] += t.reshape(Cout, H * W) @ xb
    return dw


# B, Cin, Cout, H, W, n, P, dtype, the error of the vector ALUs' kernel (2-norm, against 64 bits) on operands of this law
@pytest.mark.parametrize("shape,before", [
    ((8, 20, 512, 90, 90, 5, 2, "bf16"), 1.96e-7),   # fp32 pipe, sums added to memory on the way
    ((8, 20, 512, 90, 90, 2, 1, "bf16"), 1.57e-7),   # ... on two sets of accumulators
    ((8, 20, 512, 88, 88, 2, 1, "bf16"), 1.55e-7),   # bf16 pipe
    ((8, 20, 512, 88, 88, 3, 1, "bf16"), 1.85e-7),
    ((8, 20, 512, 88, 88, 4, 1, "bf16"), 1.94e-7),
    ((8, 20, 512, 90, 90, 3, 1, "bf16"), 1.86e-7),   # one part
    ((8, 20, 512, 90, 90, 4, 1, "bf16"), 1.95e-7),
    ((2, 24, 24, 48, 48, 3, 1, "bf16"), 8.11e-8),    # few pixels
    ((7, 20, 24, 34, 34, 2, 1, "bf16"), 8.01e-8),
    ((4, 16, 25, 33, 33, 3, 2, "bf16"), 7.71e-8),
    ((2, 24, 24, 48, 48, 4, 1, "bf16"), 8.30e-8),
    ((5, 24, 100, 31, 33, 5, 2, "f32"), 1.44e-7),
])
def test_kernel_gradient_of_16_to_31_channels_is_as_exact_as_the_vector_alus(shape, before):
    import torch
    B, Cin, Cout, H, W, n, P, dtype = shape
    print(f"case {shape}", flush=True)
    dt = ukst.UKST_F32 if dtype == "f32" else ukst.UKST_BF16_F32
    assert "mfma" in ukst.ukst_grad_kernel_name(1, *shape[:7], dt)
    OH, OW = ukst.ukst_output_shape(H, W, n, P)
    g = torch.Generator(device="cuda")
    g.manual_seed(9700 + sum(shape[:7]))
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.randn((B, Cin, H, W), generator=g, device="cuda").to(t)
    dy = torch.randn((B, Cout, OH, OW), generator=g, device="cuda").to(t)
    dw = ukst.ukst_conv_transpose2d_grad_weight(x, dy, n, P)
    ref = _kernel_gradient64(x, dy, n, P)
    err = float((dw - ref).norm() / ref.norm())
    assert err <= 1.02 * before, err  # (other operands of the same law: 2 %)


# odd P, kernels of odd side, channel counts that are no whole stages
@pytest.mark.parametrize("shape,slices", [
    ((1, 500, 256, 4, 4, 4, 2), 8), ((1, 333, 37, 5, 4, 5, 1), 6), ((2, 430, 8, 7, 10, 3, 1), 7), ((2, 704, 4, 17, 17, 2, 0), 6),
    ((3, 397, 35, 5, 7, 4, 3), 7)])
def test_forward_layers_in_slices(shape, slices):
    """Whatever layer the plan cuts, with what ukst_workspace_bytes asks for; with less, or none, the whole sum in one block."""
    import torch
    from gpu_util import to_device
    B, Cin, Cout, H, W, n, P = shape
    assert _plan("forward", shape)[2] == slices
    OH, OW = ukst.ukst_output_shape(H, W, n, P)
    need = ukst.ukst_workspace_bytes(ukst.UKST_OP_FORWARD, *shape, ukst.UKST_F32)
    copy = -(-B * Cout * OH * OW * 4 // 256) * 256  # (copies start at whole 256 bytes)
    assert need == slices * copy
    w = _mk(shape + ("f32",))
    data = wl.generate(w)
    x, k = to_device(data, w.dtype)
    y_ref, S = oracle.naive(data["x"], data["w"], P)
    bias = np.linspace(-1.0, 1.0, Cout).astype(np.float32)
    z = np.tanh(y_ref + bias.astype(np.float64)[None, :, None, None])
    whole = ukst.ukst_conv_transpose2d(x, k, P)
    space = torch.empty(need, dtype=torch.uint8, device="cuda")
    for ws in (None, space, space[:need - 256], False):
        y = ukst.ukst_conv_transpose2d(x, k, P, workspace=ws)
        check_against_oracle(y.cpu().numpy(), y_ref, S, TOL["f32"])
        assert torch.equal(y, whole) == (ws is False or (ws is not None and ws.numel() < need))
        y = ukst.ukst_conv_transpose2d_ws(x, k, P, bias=torch.from_numpy(bias).cuda(), act=ukst.UKST_ACT_TANH, workspace=ws)
        assert (np.abs(y.cpu().numpy() - z) <= TOL["f32"] * S + 1.2e-7 * np.abs(y_ref) + 2e-6).all()


@pytest.mark.parametrize("shape", [GRAD_INPUT_SHAPES[1], GRAD_INPUT_SHAPES[5], GRAD_INPUT_SHAPES_32[2][0]])
def test_input_gradients_on_the_small_tiles_ask_for_no_workspace(shape):
    import torch
    from gpu_util import check_elements
    w = _mk(shape)
    dt = ukst.UKST_F32 if w.dtype == "f32" else ukst.UKST_BF16_F32
    assert ukst.ukst_workspace_bytes(ukst.UKST_OP_GRAD_INPUT, *shape[:7], dt) == 0
    data = wl.generate(w)
    dyd = wl.generate_dy(w, oracle.out_shape(w.H, w.W, w.n, w.P))
    ref, S = oracle.grad_input(dyd["dy"], data["w"], w.H, w.W, w.P)

    def dev(a, bits):
        return (torch.from_numpy(a) if w.dtype == "f32" else torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16)).cuda()
    dy, k = dev(dyd["dy"], dyd.get("dy_bits")), dev(data["w"], data.get("w_bits"))
    dx = torch.full((w.B, w.Cin, w.H, w.W), -777.0, device="cuda")
    status = ukst.lib().ukst_conv_transpose2d_grad_input(dy.data_ptr(), k.data_ptr(), dx.data_ptr(), *shape[:7], dt, None, 0,
                                                         torch.cuda.current_stream().cuda_stream)
    assert status == ukst.UKST_OK
    check_elements(dx.cpu().numpy(), ref, S, TOL["f32"])
    # a workspace that an earlier version asked for is accepted
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    assert torch.equal(ukst.ukst_conv_transpose2d_grad_input(dy, k, w.H, w.W, w.P, workspace=ws), dx)
