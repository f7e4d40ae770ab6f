"""Host-side checks of the C-ABI library (no GPU): it loads, exports what include/ukst.h declares,
validates arguments before touching the GPU, and its host arithmetic is right."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2502_20493_amd import binding as ukst
from paper_2502_20493_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "ukst.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ukst_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = ctypes.CDLL(ukst.LIB_PATH)
    declared = _declared_symbols()
    assert len(declared) >= 8
    for name in declared:
        assert hasattr(lib, name), name
    assert sorted(ukst.EXPORTS) == declared


def test_bench_library_exports_every_declared_symbol():
    # the measured ceilings live in a library of their own: the product ABI has no benchmark kernel
    text = open(os.path.join(ROOT, "include", "ukst_bench.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = sorted(set(re.findall(r"\b(ukst_[a-z0-9_]+)\s*\(", text)))
    lib = ctypes.CDLL(ukst.BENCH_LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert sorted(ukst.BENCH_EXPORTS) == declared
    product = ctypes.CDLL(ukst.LIB_PATH)
    for name in declared:
        assert not hasattr(product, name), name


def test_version_and_status_strings():
    assert ukst.ukst_version() >= 100
    seen = {ukst.ukst_status_string(s) for s in range(7)}
    assert len(seen) == 7 and ukst.ukst_status_string(0) == "ok"
    assert ukst.ukst_status_string(99) == "unknown status"


def test_output_shape():
    assert ukst.ukst_output_shape(4, 4, 3, 0) == (5, 5)      # Sec. 1
    assert ukst.ukst_output_shape(4, 4, 3, 2) == (9, 9)      # Fig. 2
    assert ukst.ukst_output_shape(4, 4, 5, 2) == (7, 7)      # Figs. 5-6
    assert ukst.ukst_output_shape(224, 200, 3, 0) == (445, 397)
    for bad in [(1, 4, 3, 0), (4, 1, 3, 0), (0, 4, 3, 2), (4, 4, 0, 0), (4, 4, 3, -1)]:
        with pytest.raises(ukst.UkstError) as e:
            ukst.ukst_output_shape(*bad)
        assert e.value.status == ukst.UKST_ERR_SHAPE
    oh = ctypes.c_int(0)
    assert ukst.lib().ukst_output_shape(4, 4, 3, 0, None, ctypes.byref(oh)) == ukst.UKST_ERR_NULL


def test_validation_happens_on_the_host():
    # fake non-null addresses: validation must reject before any launch
    X = W = Y = 0x1000
    call = ukst.ukst_conv_transpose2d_raw
    ok_shape = (1, 1, 1, 4, 4, 3, 0)
    assert call(None, W, Y, *ok_shape, 0) == ukst.UKST_ERR_NULL
    assert call(X, None, Y, *ok_shape, 0) == ukst.UKST_ERR_NULL
    assert call(X, W, None, *ok_shape, 0) == ukst.UKST_ERR_NULL
    for bad in [(0, 1, 1, 4, 4, 3, 0), (1, 0, 1, 4, 4, 3, 0), (1, 1, 0, 4, 4, 3, 0),
                (1, 1, 1, 0, 4, 3, 0), (1, 1, 1, 4, 0, 3, 0), (1, 1, 1, 4, 4, 0, 0),
                (1, 1, 1, 4, 4, 3, -1), (1, 1, 1, 1, 4, 3, 0), (1, 1, 1, 4, 1, 3, 0)]:
        assert call(X, W, Y, *bad, 0) == ukst.UKST_ERR_SHAPE, bad
    assert call(X, W, Y, *ok_shape, 3) == ukst.UKST_ERR_DTYPE
    assert call(X, W, Y, *ok_shape, -1) == ukst.UKST_ERR_DTYPE
    assert call(X, W, Y, 1, 1, 1, 8, 8, ukst.UKST_MAX_N + 1, 0, 0) == ukst.UKST_ERR_UNSUPPORTED
    assert call(X, W, Y, *ok_shape, 0, path=7) == ukst.UKST_ERR_UNSUPPORTED
    # MFMA path cannot run a 1-channel problem
    assert call(X, W, Y, *ok_shape, 0, path=ukst.UKST_PATH_MFMA) == ukst.UKST_ERR_UNSUPPORTED
    # element alignment: fp32 buffers at 4 bytes, a bf16 output at 2
    assert call(X + 2, W, Y, *ok_shape, 0) == ukst.UKST_ERR_UNSUPPORTED
    assert call(X, W, Y + 2, *ok_shape, ukst.UKST_BF16_F32) == ukst.UKST_ERR_UNSUPPORTED
    assert call(X, W, Y + 1, *ok_shape, ukst.UKST_BF16_BF16) == ukst.UKST_ERR_UNSUPPORTED
    # the fused entry point validates the same way, plus the activation code
    fused = ukst.lib().ukst_conv_transpose2d_bias_act
    assert fused(X, W, None, None, *ok_shape, 0, 0, 0, None) == ukst.UKST_ERR_NULL
    assert fused(X, W, None, Y, 1, 1, 1, 0, 4, 3, 0, 0, 0, 0, None) == ukst.UKST_ERR_SHAPE
    assert fused(X, W, None, Y, *ok_shape, 0, 9, 0, None) == ukst.UKST_ERR_UNSUPPORTED
    assert fused(X, W, X + 2, Y, *ok_shape, 0, 1, 0, None) == ukst.UKST_ERR_UNSUPPORTED
    # the backward entry points validate the same way; gradients are fp32 only
    for back in (ukst.lib().ukst_conv_transpose2d_grad_input, ukst.lib().ukst_conv_transpose2d_grad_weight):
        assert back(None, W, Y, *ok_shape, 0, None, 0, None) == ukst.UKST_ERR_NULL
        assert back(X, None, Y, *ok_shape, 0, None, 0, None) == ukst.UKST_ERR_NULL
        assert back(X, W, None, *ok_shape, 0, None, 0, None) == ukst.UKST_ERR_NULL
        assert back(X, W, Y, 1, 1, 1, 4, 1, 3, 0, 0, None, 0, None) == ukst.UKST_ERR_SHAPE
        assert back(X, W, Y, *ok_shape, 5, None, 0, None) == ukst.UKST_ERR_DTYPE
        assert back(X, W, Y, *ok_shape, ukst.UKST_BF16_BF16, None, 0, None) == ukst.UKST_ERR_UNSUPPORTED
        assert back(X, W, Y, 1, 1, 1, 8, 8, ukst.UKST_MAX_N + 1, 0, 0, None, 0, None) == ukst.UKST_ERR_UNSUPPORTED
        assert back(X + 2, W, Y, *ok_shape, 0, None, 0, None) == ukst.UKST_ERR_UNSUPPORTED
        assert back(X, W, Y + 2, *ok_shape, ukst.UKST_BF16_F32, None, 0, None) == ukst.UKST_ERR_UNSUPPORTED
        # workspace: NULL with a size, or misaligned, is refused before anything else happens
        assert back(X, W, Y, *ok_shape, 0, None, 64, None) == ukst.UKST_ERR_WORKSPACE
        assert back(X, W, Y, *ok_shape, 0, 0x1010, 1 << 20, None) == ukst.UKST_ERR_WORKSPACE


def test_workspace_sizes_are_host_arithmetic():
    """ukst_workspace_bytes needs no GPU, and a call whose workspace is too small is refused on the
    host (fake addresses: nothing may be launched)."""
    wsb = ukst.ukst_workspace_bytes
    F, GI, GW = ukst.UKST_OP_FORWARD, ukst.UKST_OP_GRAD_INPUT, ukst.UKST_OP_GRAD_WEIGHT
    w = wl.WORKLOADS

    def shape(k):
        return (w[k].B, w[k].Cin, w[k].Cout, w[k].H, w[k].W, w[k].n, w[k].P)

    # forward: only layers whose K loop is split want one (a whole number of copies of y)
    for k in ("cfg1", "cfg2a", "cfg2b", "cfg3_L4", "cfg4a", "cfg4b"):
        assert wsb(F, *shape(k), ukst.UKST_F32) == 0, k
    for k in ("cfg5a", "cfg5b"):
        assert wsb(F, *shape(k), ukst.UKST_BF16_F32) == 0, k
    # kernel gradient: always a whole number of copies of dw, at least one
    for k in ("cfg2a", "cfg3_L1", "cfg3_L4", "cfg4a"):
        n_dw = w[k].Cout * w[k].Cin * w[k].n ** 2 * 4
        got = wsb(GW, *shape(k), ukst.UKST_F32)
        assert got >= n_dw and got % n_dw == 0, k
    # input gradient: the vector-ALU kernels need none, the matrix-core kernels at least the
    # packed weights
    assert wsb(GI, *shape("cfg2a"), ukst.UKST_F32) == 0
    assert wsb(GI, *shape("cfg4a"), ukst.UKST_F32) >= 128 * 128 * 25 * 4
    assert wsb(GI, *shape("cfg5a"), ukst.UKST_BF16_F32) >= 128 * 256 * 16 * 2
    # invalid arguments give 0
    assert wsb(7, *shape("cfg4a"), ukst.UKST_F32) == 0
    assert wsb(GW, 1, 1, 1, 1, 4, 3, 0, ukst.UKST_F32) == 0
    assert wsb(GW, *shape("cfg4a"), ukst.UKST_BF16_BF16) == 0
    # too small a workspace is a host-side error
    X = W = Y = 0x1000
    WS = 0x10000
    need = wsb(GW, *shape("cfg4a"), ukst.UKST_F32)
    gw = ukst.lib().ukst_conv_transpose2d_grad_weight
    assert gw(X, W, Y, *shape("cfg4a"), ukst.UKST_F32, WS, need - 1, None) == ukst.UKST_ERR_WORKSPACE
    assert gw(X, W, Y, *shape("cfg4a"), ukst.UKST_F32, None, 0, None) == ukst.UKST_ERR_WORKSPACE
    gi = ukst.lib().ukst_conv_transpose2d_grad_input
    need = wsb(GI, *shape("cfg4a"), ukst.UKST_F32)
    assert gi(X, W, Y, *shape("cfg4a"), ukst.UKST_F32, WS, need - 1, None) == ukst.UKST_ERR_WORKSPACE
    fw = ukst.lib().ukst_conv_transpose2d_ws
    ok_shape = (1, 1, 1, 4, 4, 3, 0)
    assert fw(X, W, None, Y, *ok_shape, 0, 0, 0, None, 16, None) == ukst.UKST_ERR_WORKSPACE
    assert fw(X, W, None, Y, *ok_shape, 0, 0, 0, WS + 8, 1 << 20, None) == ukst.UKST_ERR_WORKSPACE
    assert fw(None, W, None, Y, *ok_shape, 0, 0, 0, None, 0, None) == ukst.UKST_ERR_NULL


def _brute_macs(H, W, n, P):
    """Count products by walking the padded upsampled map of Algorithm 1."""
    OH, OW = 2 * H + 2 * P - n, 2 * W + 2 * P - n
    U = np.zeros((2 * H - 1 + 2 * P, 2 * W - 1 + 2 * P), dtype=np.int64)
    U[P:P + 2 * H - 1:2, P:P + 2 * W - 1:2] = 1
    exact = sum(int(U[oy:oy + n, ox:ox + n].sum()) for oy in range(OH) for ox in range(OW))
    hi, lo = (n + 1) // 2, n // 2
    nominal = sum((hi if (oy + P) % 2 == 0 else lo) * (hi if (ox + P) % 2 == 0 else lo)
                  for oy in range(OH) for ox in range(OW))
    return exact, nominal, OH * OW * n * n


def test_mac_counts():
    for (H, W, n, P) in [(4, 4, 3, 0), (4, 4, 4, 2), (5, 3, 5, 0), (5, 3, 5, 3), (3, 6, 2, 1),
                         (4, 4, 7, 6), (2, 2, 1, 0), (2, 3, 2, 4)]:
        e, nom, nv = _brute_macs(H, W, n, P)
        for kind, want in ((0, e), (1, nom), (2, nv)):
            assert ukst.ukst_mac_count(2, 3, 5, H, W, n, P, kind) == 2 * 3 * 5 * want
        assert e <= nom <= nv
    # Sec. 3.1: 25 multiplications per four outputs for n = 5 instead of 100
    assert ukst.ukst_mac_count(1, 1, 1, 8, 8, 5, 0, 1) * 4 < ukst.ukst_mac_count(1, 1, 1, 8, 8, 5, 0, 2) * 1.1
    assert ukst.ukst_mac_count(1, 1, 1, 1, 8, 5, 0, 0) == 0  # invalid shape
    # figures used by the benchmark (GFLOP = 2 * MAC / 1e9)
    assert ukst.ukst_mac_count(16, 3, 3, 224, 224, 3, 0, 0) == 16 * 9 * 668 * 668  # rows: 223 even outputs x 2 taps + 222 odd x 1
    assert abs(2 * ukst.ukst_mac_count(32, 128, 128, 64, 64, 5, 0, 0) / 1e9 - 99.47) < 0.01


def test_layers_of_few_channels_stay_on_the_vector_alus():
    """Where the kernel on bf16 parts is the slower one: a few channels and little work (fp32, n = 2 to 4, bf16, n = 2),
    at most 8 output channels of 17 to 19 (n = 2: up to 21) input channels whatever the work."""
    direct, parts = "ukst_direct_kernel", "ukst_mfma_f32_kernel_parts"
    for B, ci, co, n, dtype, kernel in (
            (8, 17, 31, 2, 0, direct), (64, 17, 31, 2, 0, parts), (4, 17, 63, 2, 0, direct), (16, 17, 63, 2, 0, parts),
            (8, 35, 17, 2, 0, direct), (8, 35, 31, 2, 0, parts), (4, 35, 63, 2, 0, parts), (4, 51, 9, 2, 0, parts),
            (8, 17, 31, 3, 0, direct), (64, 17, 31, 4, 0, parts), (8, 21, 31, 4, 0, direct), (8, 25, 31, 4, 0, parts),
            (256, 19, 7, 3, 0, direct), (256, 19, 7, 5, 0, direct), (256, 21, 7, 2, 0, direct), (64, 21, 7, 3, 0, parts), (64, 25, 7, 3, 0, parts), (32, 17, 31, 5, 0, parts),
            (1, 17, 80, 2, 1, direct), (2, 17, 80, 2, 1, parts), (1, 19, 80, 2, 1, parts), (1, 23, 17, 2, 1, parts), (1, 17, 17, 3, 1, parts)):
        assert ukst.ukst_kernel_name(B, ci, co, 40, 41, n, 1, dtype) == kernel, (B, ci, co, n, dtype)


def test_output_size_in_place_is_ukst_output_shape():
    """The binding works the output size out by itself for sizes in range; what the library refuses it refuses with
    the same error, whatever the sign of the result."""
    for H in (-1, 0, 1, 2, 7, 1 << 28, (1 << 28) + 1):
        for W in (0, 1, 5):
            for n in (0, 1, 3, 7):
                for P in (-1, 0, 2, 40, 1 << 28, (1 << 28) + 1):
                    want, got = [], []
                    for f, out in ((ukst.ukst_output_shape, want), (ukst._output_size, got)):
                        try:
                            out.append(f(H, W, n, P))
                        except ukst.UkstError as e:
                            out.append(e.status)
                    assert want == got, (H, W, n, P)


def test_select_path():
    assert ukst.ukst_select_path(16, 3, 3, 224, 224, 3, 0, ukst.UKST_F32) == ukst.UKST_PATH_DIRECT
    # few output channels: the parity classes fill the MFMA columns when Cin % 16 == 0, W % 4 == 0
    assert ukst.ukst_select_path(64, 64, 3, 32, 32, 4, 2, ukst.UKST_F32) == ukst.UKST_PATH_MFMA
    assert ukst.ukst_kernel_name(64, 64, 3, 32, 32, 4, 2, 0) == "ukst_thin_mfma_kernel"
    assert ukst.ukst_select_path(64, 24, 3, 32, 31, 4, 2, ukst.UKST_F32) == ukst.UKST_PATH_DIRECT
    assert ukst.ukst_kernel_name(64, 24, 3, 32, 31, 4, 2, 0) == "ukst_thin_kernel"
    assert ukst.ukst_select_path(32, 256, 128, 128, 128, 4, 2, ukst.UKST_BF16_F32) == ukst.UKST_PATH_MFMA
    with pytest.raises(ukst.UkstError):
        ukst.ukst_select_path(16, 3, 3, 1, 224, 3, 0, ukst.UKST_F32)
    assert "narrow" in ukst.ukst_kernel_name(16, 3, 3, 224, 224, 3, 0, 0)
    assert "direct" in ukst.ukst_kernel_name(16, 8, 8, 224, 224, 3, 0, 0)
    assert ukst.ukst_kernel_name(16, 3, 3, 1, 224, 3, 0, 0) == ""


@pytest.mark.parametrize("dtype", [ukst.UKST_F32, ukst.UKST_BF16_F32, ukst.UKST_BF16_BF16])
def test_a_selected_path_can_be_forced(dtype):
    """The path that ukst_select_path names is one that a call accepts (a kernel name for it), also for the layers
    that only automatic selection takes to the matrix cores (odd channel counts, any row length)."""
    rng = np.random.default_rng(11)
    for _ in range(1500):
        B, Cin, Cout, H, W, n = (int(v) for v in rng.integers([1, 1, 1, 4, 4, 1], [40, 200, 150, 90, 90, 8]))
        shape = (B, Cin, Cout, H, W, n, int(rng.integers(0, n)))
        path = ukst.ukst_select_path(*shape, dtype)
        assert ukst.ukst_kernel_name(*shape, dtype, path) != "", (shape, path)
    assert ukst.ukst_kernel_name(8, 77, 40, 33, 35, 3, 0, ukst.UKST_F32) == "ukst_mfma_f32_kernel_parts"
    assert ukst.ukst_select_path(8, 77, 40, 33, 35, 3, 0, ukst.UKST_F32) == ukst.UKST_PATH_DIRECT


def test_workloads_are_seeded_and_shaped():
    from paper_2502_20493_amd import workloads as wl
    a = wl.generate(wl.WORKLOADS["cfg1"])
    b = wl.generate(wl.WORKLOADS["cfg1"])
    assert a["x"].shape == (1, 1, 32, 32) and a["w"].shape == (1, 1, 3, 3)
    assert np.array_equal(a["x"], b["x"]) and np.array_equal(a["w"], b["w"])
    i = wl.generate(wl.WORKLOADS["cfg1_int"])
    assert set(np.unique(i["x"])).issubset(set(range(-3, 4)))
    small = wl.WORKLOADS["cfg5b"].with_(B=1, Cin=8, Cout=4)
    d = wl.generate(small)
    assert d["x_bits"].dtype == np.uint16
    # bf16 values survive a second rounding unchanged, and rounding is to nearest even
    assert np.array_equal(wl.round_to_bf16_bits(d["x"]), d["x_bits"])
    t = np.array([1.0, 1.0 + 2 ** -8, 1.0 + 3 * 2 ** -8, 1.0 + 2 ** -7], dtype=np.float32)
    assert wl.bf16_bits_to_f32(wl.round_to_bf16_bits(t)).tolist() == [1.0, 1.0, 1.0 + 2 ** -6, 1.0 + 2 ** -7]


def test_backward_kernel_selection_is_host_arithmetic():
    """ukst_grad_kernel_name needs no GPU: wide layers go to the matrix cores (bf16 operands to the
    bf16 pipe for the input gradient), narrow ones to the vector ALUs."""
    name = ukst.ukst_grad_kernel_name
    w = wl.WORKLOADS
    def shape(k):
        return (w[k].B, w[k].Cin, w[k].Cout, w[k].H, w[k].W, w[k].n, w[k].P)
    for k in ("cfg2a", "cfg2b"):  # narrow fp32 image layers: register-blocked strips
        assert name(0, *shape(k), ukst.UKST_F32) == "ukst_grad_input_narrow_kernel"
        assert name(1, *shape(k), ukst.UKST_F32) == "ukst_grad_weight_narrow_kernel"
    # narrow layers those kernels do not take: bf16 operands, maps narrower than 32, n = 1 or n > 5
    assert name(0, *shape("cfg2a"), ukst.UKST_BF16_F32) == "ukst_grad_input_kernel"
    assert name(1, *shape("cfg2a"), ukst.UKST_BF16_F32) == "ukst_grad_weight_kernel"
    assert name(0, 2, 3, 3, 40, 24, 3, 0, ukst.UKST_F32) == "ukst_grad_input_kernel"
    assert name(1, 2, 3, 3, 40, 40, 6, 0, ukst.UKST_F32) == "ukst_grad_weight_kernel"
    assert name(1, 2, 3, 3, 40, 40, 1, 0, ukst.UKST_F32) == "ukst_grad_weight_kernel"
    assert name(0, *shape("cfg3_L4"), ukst.UKST_F32) == "ukst_grad_input_kernel"      # Cout = 3
    assert name(1, *shape("cfg3_L4"), ukst.UKST_F32) == "ukst_grad_weight_thin_mfma_kernel"  # 3 x 16 rows
    assert name(1, 2, 16, 5, 16, 16, 4, 2, ukst.UKST_F32) == "ukst_grad_weight_kernel"   # 5 x 16 rows: too many
    assert name(1, 2, 16, 3, 16, 2, 3, 0, ukst.UKST_F32) == "ukst_grad_weight_kernel"    # rows of two pixels
    assert name(1, 2, 16, 3, 16, 16, 3, 0, ukst.UKST_F32) == "ukst_grad_weight_thin_mfma_kernel"
    # wide fp32 layers: the fp32 pipe, or bf16 parts from 100 tiles of 256 pixels (input gradient) and from 8192 pixels
    # in rows of at least 16 on, n = 3, 4 (kernel gradient)
    for k, dx, dw in (("cfg3_L1", "", ""), ("cfg3_L2", "", ""), ("cfg3_L3", "", "_parts"), ("cfg4a", "_parts", ""),
                      ("cfg4b", "_parts", "_parts")):
        assert name(0, *shape(k), ukst.UKST_F32) == "ukst_grad_input_mfma_kernel" + dx, k
        assert name(1, *shape(k), ukst.UKST_F32) == "ukst_grad_weight_mfma_kernel" + dw, k
    assert name(1, 9, 64, 64, 31, 30, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_weight_mfma_kernel_parts"
    # four-wave blocks (up to 64 input channels) gain later for n = 2 and n >= 5, unless there are few output channels
    for images, co, n, tail in ((10, 160, 5, ""), (13, 160, 5, "_parts"), (10, 160, 7, ""), (10, 16, 7, "_parts"),
                                (10, 160, 3, "_parts"), (10, 96, 2, ""), (13, 96, 2, "_parts"), (10, 64, 2, "_parts")):
        assert name(0, images, 33, co, 51, 51, n, n // 2, ukst.UKST_F32) == "ukst_grad_input_mfma_kernel" + tail, (co, n)
    assert name(0, 10, 72, 160, 51, 51, 5, 2, ukst.UKST_F32) == "ukst_grad_input_mfma_kernel_parts"
    for k in ("cfg5a", "cfg5b"):
        assert name(0, *shape(k), ukst.UKST_BF16_F32) == "ukst_grad_input_window_mfma_bf16_kernel", k
        assert name(1, *shape(k), ukst.UKST_BF16_F32) == "ukst_grad_weight_mfma_bf16_kernel", k
    # bf16 layers the bf16-pipe kernel gradient does not take (n = 5, rows that are no multiple of 8)
    assert name(1, 2, 64, 64, 16, 16, 5, 2, ukst.UKST_BF16_F32) == "ukst_grad_weight_mfma_kernel"
    assert name(1, 2, 64, 64, 16, 20, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_weight_mfma_kernel"
    # bf16 layers the window kernel does not take: n other than 2, 3 or 4, at most 64 input channels or no multiple of
    # 8, output channels that are no multiple of 8, maps narrower than 16
    assert name(0, 2, 132, 32, 16, 16, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 16, 2, 0, ukst.UKST_BF16_F32) == "ukst_grad_input_window_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 16, 1, 0, ukst.UKST_BF16_F32) != "ukst_grad_input_window_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 16, 5, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 16, 3, 1, ukst.UKST_BF16_F32) == "ukst_grad_input_window_mfma_bf16_kernel"
    assert name(0, 2, 64, 32, 16, 16, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_bf16_kernel"
    assert name(0, 2, 128, 36, 16, 16, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_bf16_kernel"
    assert name(0, 2, 128, 40, 16, 16, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_window_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 8, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_bf16_kernel"
    assert name(0, 2, 128, 32, 16, 16, 4, 2, ukst.UKST_BF16_F32) == "ukst_grad_input_window_mfma_bf16_kernel"
    # kernel sides whose tile does not fit the bf16 kernel's LDS budget fall back to the fp32 pipe
    assert name(0, 2, 64, 32, 40, 40, 7, 3, ukst.UKST_BF16_F32) == "ukst_grad_input_mfma_kernel"
    assert name(0, 1, 1, 1, 4, 4, 3, 0, ukst.UKST_BF16_BF16) == ""
    assert name(2, 1, 1, 1, 4, 4, 3, 0, ukst.UKST_F32) == ""
    assert name(0, 1, 1, 1, 1, 4, 3, 0, ukst.UKST_F32) == ""


@pytest.mark.parametrize("what", ["missing", "not a library", "another torch"])
def test_an_extension_that_cannot_be_used_leaves_the_calls_to_ctypes(what, monkeypatch, tmp_path):
    """Queries and raw calls never need it; calls with tensors warn once and are marshalled in Python."""
    import torch
    if what == "another torch":
        import types
        other = types.SimpleNamespace(built_for="1.0", bind=lambda *a: pytest.fail("bound"))
        monkeypatch.setattr(ukst.importlib.util, "module_from_spec", lambda spec: other)
        monkeypatch.setattr(ukst.importlib.util, "spec_from_file_location", lambda *a: types.SimpleNamespace(
            loader=types.SimpleNamespace(exec_module=lambda m: None)))
    else:
        path = tmp_path / "_ukst_marshal.so"
        if what == "not a library":
            path.write_bytes(b"nothing")
        monkeypatch.setattr(ukst, "MARSHAL_PATH", str(path))
    monkeypatch.setattr(ukst, "_native", None)
    monkeypatch.setattr(ukst, "_lib", None)
    assert ukst.ukst_workspace_bytes(ukst.UKST_OP_GRAD_WEIGHT, 1, 3, 3, 8, 8, 3, 0, ukst.UKST_F32) > 0
    assert ukst._native is None
    x, w = torch.zeros(1, 2, 4, 4), torch.zeros(5, 2, 3, 3)
    with pytest.warns(RuntimeWarning, match="marshalled with ctypes"):
        with pytest.raises(ValueError, match="device tensors"):  # (x is on the CPU: as far as it gets here)
            ukst.ukst_conv_transpose2d(x, w, 1)
    assert ukst._native is ukst._Ctypes
    for call in (lambda: ukst.ukst_conv_transpose2d_grad_input(x, w, 4, 4, 1), lambda: ukst.ukst_dilated_conv2d(x, w, 1, 1),
                 lambda: ukst.ukst_conv_transpose2d_grad_weight(x, x, 3, 1)):
        with pytest.raises(ValueError):
            call()


def test_the_extension_is_built_for_this_torch():
    import torch
    assert ukst._load_native().built_for == torch.__version__


@pytest.mark.parametrize("call", [ukst.ukst_conv_transpose2d_ws, ukst.ukst_conv_transpose2d_bias_act])
@pytest.mark.parametrize("workspace", [None, False])
def test_a_bias_without_an_activation_is_never_left_out(call, workspace, monkeypatch):
    """act=None is no activation, with the bias or without; a call that the native marshalling turns down does not come
    back to it without its bias."""
    import types
    import torch
    ukst.lib()
    seen = []

    class Native:
        @staticmethod
        def forward(x, w, P, bias, act, out_bf16, with_workspace):
            seen.append((bias, act, with_workspace))  # (None: turned down)

    monkeypatch.setattr(ukst, "_native", Native)
    bias = types.SimpleNamespace(is_cuda=True, dtype=torch.float32, is_contiguous=lambda: True, shape=(5,))
    x, w = torch.zeros(1, 2, 4, 4), torch.zeros(5, 2, 3, 3)
    with pytest.raises(ValueError, match="device tensors"):  # (x is on the CPU: as far as it gets here)
        call(x, w, 1, bias=bias, act=None, workspace=workspace)
    assert seen == [(bias, ukst.UKST_ACT_NONE, workspace is None)]


def _small_tile(op, shape, dtype=ukst.UKST_F32):
    """(rows, waves) of the small tile a layer runs on, (0, 0) of layers that run elsewhere; op 0 forward, 1 input gradient."""
    v = ukst.lib().ukst_test_plan(op, *shape, 2, dtype)
    return v & 255, v >> 8 & 255


def test_input_gradients_of_small_kernels_count_their_staging():
    """Two and three taps a side: 16 x 16 tiles stage more for each product than 32 x 32 ones, and are only for fewer tiles."""
    for n in (2, 3):
        assert _small_tile(1, (1, 398, 344, 16, 16, n, 1)) == (32, 8), n   # n = 2: 15.0 us, in 16 x 16 tiles 24.1
        assert _small_tile(1, (1, 398, 344, 4, 5, n, 1)) == (16, 8), n


def test_bf16_input_gradients_go_where_they_are_estimated_the_faster():
    """The small tiles against the bf16 pipe, which multiplies 16 times as fast (us, the pipe / the small tiles)."""
    for shape, small in (((11, 72, 248, 10, 22, 4, 1), True),      # 99 / 27
                         ((12, 216, 176, 9, 9, 4, 1), True),       # 33.0 / 20.7
                         ((1, 272, 200, 14, 14, 5, 4), True),      # 33.0 / 16.8
                         ((55, 32, 248, 8, 19, 3, 1), True),       # 50.1 / 35.4, tiles beyond one round
                         ((4, 112, 112, 26, 26, 5, 2), False),     # 36.2 / 39.6
                         ((5, 96, 571, 24, 24, 5, 2), False),      # 68 / 157
                         ((4, 224, 504, 31, 7, 5, 2), False)):     # 45 / 80
        name = "ukst_grad_input_mfma_kernel" if small else "ukst_grad_input_mfma_bf16_kernel"
        assert ukst.ukst_grad_kernel_name(0, *shape, ukst.UKST_BF16_F32) == name, shape
        assert (_small_tile(1, shape, ukst.UKST_BF16_F32) != (0, 0)) == small, shape


def test_few_output_channels_go_to_the_small_tiles_for_one_round():
    """Up to four output channels: the kernels made for them against the small tiles (us, the former / the latter)."""
    for shape, kernel in (((45, 336, 3, 4, 4, 4, 3), "ukst_mfma_f32_kernel"),       # 14.4 / 10.4
                          ((2, 160, 2, 48, 48, 4, 1), "ukst_thin_mfma_kernel"),     # 8.5 / 15.1, more than a round
                          ((22, 112, 2, 24, 4, 4, 4), "ukst_thin_mfma_kernel"),     # 6.2 / 7.0, a short sum
                          ((3, 152, 3, 45, 32, 2, 0), "ukst_mfma_f32_kernel"),      # 10.1 / 9.5
                          ((2, 112, 1, 40, 40, 5, 5), "ukst_thin_kernel"),          # 11.8 / 18.8
                          ((3, 113, 2, 37, 37, 2, 0), "ukst_thin_kernel")):         # 7.1 / 8.8
        assert ukst.ukst_kernel_name(*shape, ukst.UKST_F32) == kernel, shape
        assert (_small_tile(0, shape) != (0, 0)) == (kernel == "ukst_mfma_f32_kernel"), shape


def test_long_sums_with_a_workspace_keep_the_slices_of_the_kernel_on_parts():
    """Given a workspace, slices on bf16 parts against the small tiles in slices (us, the latter / the former)."""
    for shape, small in (((6, 920, 336, 5, 16, 5, 2), False),      # 103 / 77
                         ((20, 896, 40, 8, 34, 4, 0), False),      # 66 / 50
                         ((12, 608, 112, 11, 11, 4, 2), False),    # 45.7 / 40.6
                         ((10, 832, 32, 12, 12, 4, 4), True),      # 38.9 / 47.5, few products
                         ((18, 432, 360, 4, 4, 5, 4), True),       # 51 / 57, fewer channels
                         ((2, 800, 312, 9, 28, 5, 2), True)):      # 87 / 111, four slices
        assert (_small_tile(0, shape) != (0, 0)) == small, shape
        assert ukst.ukst_kernel_name(*shape, ukst.UKST_F32) == "ukst_mfma_f32_kernel"  # (the choice without one)
        assert small or ukst.ukst_workspace_bytes(ukst.UKST_OP_FORWARD, *shape, ukst.UKST_F32) > 0


def test_generalised_operations_host_side():
    """Stride-s transpose convolution and dilated convolution: shapes, multiply-add counts and
    argument validation are host arithmetic (fake addresses: nothing may be launched)."""
    assert ukst.ukst_output_shape_strided(4, 4, 3, 0, 2) == ukst.ukst_output_shape(4, 4, 3, 0)
    assert ukst.ukst_output_shape_strided(2, 2, 2, 1, 3) == (5, 5)     # tests/golden/worked_stride3_2x2_k2.txt
    assert ukst.ukst_output_shape_dilated(4, 4, 2, 0, 2) == (2, 2)     # tests/golden/worked_dilated2_4x4_k2.txt
    assert ukst.ukst_output_shape_dilated(9, 7, 3, 2, 3) == (7, 5)
    for bad in [(0, 4, 3, 0, 2), (4, 4, 0, 0, 2), (4, 4, 3, -1, 2), (4, 4, 3, 0, 0), (1, 1, 3, 0, 2)]:
        with pytest.raises(ukst.UkstError) as e:
            ukst.ukst_output_shape_strided(*bad)
        assert e.value.status == ukst.UKST_ERR_SHAPE
    with pytest.raises(ukst.UkstError):
        ukst.ukst_output_shape_dilated(4, 4, 3, 0, 2)  # 4 - 2*2 = 0: empty output

    def brute_strided(H, W, n, P, s):
        OH, OW = s * (H - 1) + 2 * P - n + 2, s * (W - 1) + 2 * P - n + 2
        U = np.zeros((s * (H - 1) + 1 + 2 * P, s * (W - 1) + 1 + 2 * P), dtype=np.int64)
        U[P:P + s * (H - 1) + 1:s, P:P + s * (W - 1) + 1:s] = 1
        return sum(int(U[oy:oy + n, ox:ox + n].sum()) for oy in range(OH) for ox in range(OW)), OH * OW * n * n

    def brute_dilated(H, W, n, P, d):
        OH, OW = H + 2 * P - d * (n - 1), W + 2 * P - d * (n - 1)
        X = np.pad(np.ones((H, W), dtype=np.int64), P)
        nd = d * (n - 1) + 1
        return sum(int(X[oy:oy + nd:d, ox:ox + nd:d].sum()) for oy in range(OH) for ox in range(OW)), OH * OW * nd * nd

    for (H, W, n, P, k) in [(4, 4, 3, 0, 2), (3, 5, 4, 2, 3), (5, 3, 5, 3, 4), (2, 2, 2, 1, 3), (6, 4, 3, 2, 1)]:
        e, nv = brute_strided(H, W, n, P, k)
        assert ukst.ukst_mac_count_strided(2, 3, 5, H, W, n, P, k, 0) == 30 * e
        assert ukst.ukst_mac_count_strided(2, 3, 5, H, W, n, P, k, 2) == 30 * nv
        assert e <= ukst.ukst_mac_count_strided(1, 1, 1, H, W, n, P, k, 1) <= nv
    assert ukst.ukst_mac_count_strided(2, 3, 5, 4, 4, 3, 1, 2, 0) == ukst.ukst_mac_count(2, 3, 5, 4, 4, 3, 1, 0)
    assert ukst.ukst_mac_count_strided(2, 3, 5, 4, 4, 3, 1, 2, 1) == ukst.ukst_mac_count(2, 3, 5, 4, 4, 3, 1, 1)
    for (H, W, n, P, k) in [(9, 8, 3, 0, 2), (7, 7, 3, 3, 3), (6, 9, 2, 2, 4), (5, 5, 4, 1, 1)]:
        e, nv = brute_dilated(H, W, n, P, k)
        assert ukst.ukst_mac_count_dilated(2, 3, 5, H, W, n, P, k, 0) == 30 * e
        assert ukst.ukst_mac_count_dilated(2, 3, 5, H, W, n, P, k, 2) == 30 * nv
    X = W_ = Y = 0x1000
    for f in (ukst.lib().ukst_conv_transpose2d_strided, ukst.lib().ukst_dilated_conv2d):
        ok = (1, 1, 1, 8, 8, 3, 1, 2)
        assert f(None, W_, Y, *ok, 0, None) == ukst.UKST_ERR_NULL
        assert f(X, W_, None, *ok, 0, None) == ukst.UKST_ERR_NULL
        assert f(X, W_, Y, 1, 1, 1, 8, 8, 3, 1, 0, 0, None) == ukst.UKST_ERR_SHAPE
        assert f(X, W_, Y, 0, 1, 1, 8, 8, 3, 1, 2, 0, None) == ukst.UKST_ERR_SHAPE
        assert f(X, W_, Y, *ok, 7, None) == ukst.UKST_ERR_DTYPE
        assert f(X, W_, Y, *ok, ukst.UKST_BF16_BF16, None) == ukst.UKST_ERR_UNSUPPORTED
        assert f(X, W_, Y, 1, 1, 1, 8, 8, 3, 1, 9, 0, None) == ukst.UKST_ERR_UNSUPPORTED
        assert f(X + 2, W_, Y, *ok, 0, None) == ukst.UKST_ERR_UNSUPPORTED
    assert ukst.lib().ukst_dilated_conv2d(X, W_, Y, 1, 1, 1, 4, 4, 3, 0, 2, 0, None) == ukst.UKST_ERR_SHAPE
