"""GPU parity at the edges of the fused call's dispatch: every way conv_fused_pos cuts a layer (one,
two and four groups of 16 filters, 8 and 16 waves, the form in two kernels, one and four channels
per lane, caller-supplied ranges of narrow codes), and the other plans on layers large
enough to be theirs with ragged sizes.  Same bars as test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import test_gpu_parity as parity
from paper_2003_08646_amd import workloads as Wk
from test_gpu_parity import _assert_codes, _check_layer, O

pytestmark = pytest.mark.gpu


def _range_of_another_batch(L):
    """Ranges calibrated on other inputs: some values of this batch fall outside and are clamped."""
    X, Wt = Wk.make_inputs(L.with_(seed=L.seed + 1000))
    return 0.7 * O.lance_conv(X, Wt, L.pad, L.m, L.bits, bits_w=L.bits_w).v_range


# N, C, K, H, W, pad, m, bits, nhwc
_SPLITS = [
    (40, 20, 70, 14, 14, 1, 2, 8, False),    # four groups of filters, 16 waves
    (20, 33, 60, 14, 14, 1, 2, 8, False),    # two groups, 16 waves
    (90, 40, 70, 14, 15, 1, 2, 6, False),    # 8 waves, odd width
    (60, 130, 40, 12, 12, 0, 2, 8, False),   # four channels per lane
    (3, 600, 20, 9, 8, 1, 2, 8, False),      # more channel blocks than LDS holds: two kernels
    (4, 580, 20, 7, 7, 2, 2, 5, True),       # the same with 16-byte NHWC loads
    (3, 601, 17, 6, 6, 1, 2, 8, True),       # and with 4-byte ones
    (20, 530, 150, 13, 12, 1, 2, 8, False),  # two groups of filters and of tiles
    (33, 18, 70, 15, 16, 1, 4, 8, False),    # F(4x4): two groups
    (90, 30, 70, 16, 13, 1, 4, 5, False),    # four groups, odd width
    (20, 150, 24, 9, 11, 0, 4, 8, False),    # four channels per lane
    (2, 330, 20, 9, 10, 1, 4, 6, False),     # F(4x4) in two kernels
    (2, 200, 20, 9, 10, 1, 4, 8, True),
    (30, 210, 150, 14, 13, 1, 4, 7, False),  # two groups of filters
    (40, 200, 150, 15, 16, 0, 4, 8, True),   # and of tiles
    (30, 7, 70, 33, 31, 1, 4, 8, False),     # at most 16 channels
    (8, 16, 40, 33, 31, 3, 4, 4, True),
    (2, 5, 300, 20, 18, 1, 2, 7, True),
    (1, 6, 5, 3, 2, 5, 2, 8, False),         # more padding than image
    (3, 21, 10, 9, 8, 5, 4, 8, False),       # rows of F(4x4) that start five pixels before the image
    (2, 6, 20, 4, 5, 13, 4, 8, False),       # tiles far outside the image
    (3, 9, 20, 1, 1, 2, 2, 8, False),        # images smaller than a load
    (2, 70, 5, 1, 3, 2, 4, 8, False),
    (2, 4, 20, 3, 1, 5, 4, 6, False),
    (2, 9, 6, 1, 2, 3, 2, 8, True),
]


@pytest.mark.parametrize("shape", _SPLITS, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d_b%d%s" % (s[:8] + ("_nhwc" if s[8] else "",)))
@pytest.mark.parametrize("static", [False, True], ids=["dynamic", "static"])
def test_position_parallel_splits(shape, static):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, m, bits, nhwc = shape
    L = Wk.Layer("split", N, C, K, H, W, pad=pad, m=m, bits=bits, seed=500 + C)
    flags = (B.LANCE_LAYOUT_NHWC if nhwc else 0) | (B.LANCE_INPUT_RANGE_STATIC if static else 0)
    _check_layer(L, flags=flags, static_v_range=_range_of_another_batch(L) if static else None, staged=False)


def _kernels(conv, x):
    """Names of the kernels of one fused call, by slot of the timing twin."""
    from paper_2003_08646_amd import binding as B
    B.lance_conv3x3_winograd_q8_profile(conv.desc, x, conv.uq, conv.u_range, conv.u_rowsum, conv.v_range,
                                        torch.empty_like(conv.y), conv.workspace)
    return [B.lance_profile_kernel_name(i) for i in range(len(B.PROFILE_KERNELS))]


def _zeros(conv, nhwc):
    d = conv.desc
    return torch.zeros((d.N, d.H, d.W, d.C) if nhwc else (d.N, d.C, d.H, d.W), device="cuda")


# layers whose workgroups run in many rounds: the ranges are reduced in front of them
_ROUNDS = [(40, 3, 70, 65, 63, 1, 4, 8, False), (64, 12, 150, 65, 63, 0, 4, 6, True), (11, 3, 500, 65, 63, 1, 2, 8, False)]


@pytest.mark.parametrize("shape", _ROUNDS, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d_b%d%s" % (s[:8] + ("_nhwc" if s[8] else "",)))
@pytest.mark.parametrize("per_tensor", [False, True], ids=["per_position", "per_tensor"])
def test_position_parallel_reduction_kernel(shape, per_tensor):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, m, bits, nhwc = shape
    L = Wk.Layer("rounds", N, C, K, H, W, pad=pad, m=m, bits=bits, seed=650 + C)
    flags = (B.LANCE_LAYOUT_NHWC if nhwc else 0) | (B.LANCE_RANGE_PER_TENSOR if per_tensor else 0)
    conv, ref = _check_layer(L, flags=flags, staged=False)
    names = _kernels(conv, _zeros(conv, nhwc))
    assert names[1:] == ["range_finalize_kernel", "", "conv_fused_pos_kernel"], names


@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("nhwc", [False, True], ids=["nchw", "nhwc"])
def test_position_parallel_packed(m, nhwc):
    from paper_2003_08646_amd import binding as B
    L = Wk.Layer("packed", 20, 70, 50, 13, 12, m=m, bits=4, bits_w=3, seed=520)
    _check_layer(L, flags=B.LANCE_CODES_PACKED4 | (B.LANCE_LAYOUT_NHWC if nhwc else 0), staged=False)


@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("C,bits", [(40, 6), (40, 8), (12, 5), (600, 4)])
def test_undefined_value_takes_the_code_of_the_other_plans(C, bits, m):
    """Ranges skip a NaN; its code decides finite outputs: those of the few-tile plans against those
    of the plans that LANCE_PLAN_WIDE_TILES selects.  Codes and integer sums are equal, so what is
    left is the binary32 rounding of the epilogue (at most 1e-5 of the largest output)."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    X, Wt = Wk.make_inputs(Wk.Layer("nan", 2, C, 20, 12, 13, m=m, bits=bits, seed=580 + C))
    X[1, C // 2, 5, 6] = np.nan
    x, w = torch.from_numpy(X).cuda(), torch.from_numpy(Wt).cuda()
    ys = []
    for flags in (0, B.LANCE_PLAN_WIDE_TILES):
        conv = LanceConv(2, C, 12, 13, 20, 1, m, bits, flags)
        conv.prepare_filters(w)
        ys.append((conv.forward(x).cpu().numpy().astype(np.float64), conv.v_range.cpu().numpy()))
    np.testing.assert_array_equal(ys[0][1], ys[1][1])
    assert np.isfinite(ys[0][0]).all()
    assert np.abs(ys[0][0] - ys[1][0]).max() <= 1e-5 * np.abs(ys[1][0]).max()


# layers of more tiles than conv_fused_pos takes: the other plans with partial blocks and odd sizes
_LARGE = [
    (460, 60, 40, 9, 11, 0, 2, 8, False),
    (200, 50, 70, 13, 14, 1, 2, 5, False),
    (60, 64, 130, 24, 24, 1, 2, 8, False),
    (330, 60, 40, 10, 9, 1, 2, 8, True),
    (120, 100, 130, 13, 15, 1, 2, 8, False),
    (100, 96, 70, 16, 16, 1, 2, 6, False),
    (110, 72, 130, 14, 13, 0, 2, 8, True),
    (80, 150, 130, 13, 15, 1, 2, 8, False),
    (60, 192, 300, 14, 14, 1, 2, 8, False),
    (70, 140, 130, 14, 15, 0, 2, 7, True),
    (100, 40, 130, 20, 21, 1, 4, 8, False),
    (60, 100, 130, 24, 24, 1, 4, 6, False),
    (60, 150, 300, 15, 17, 1, 4, 8, False),
    (120, 70, 130, 17, 16, 0, 4, 8, True),
    (60, 12, 40, 33, 31, 1, 2, 8, False),
    (60, 3, 70, 32, 32, 1, 2, 8, True),
]


@pytest.mark.parametrize("shape", _LARGE, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d_b%d%s" % (s[:8] + ("_nhwc" if s[8] else "",)))
def test_other_plans_on_many_tiles(shape):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, m, bits, nhwc = shape
    L = Wk.Layer("many_tiles", N, C, K, H, W, pad=pad, m=m, bits=bits, seed=540 + C)
    conv, _ = _check_layer(L, flags=B.LANCE_LAYOUT_NHWC if nhwc else 0, staged=False)
    assert not _kernels(conv, _zeros(conv, nhwc))[3].endswith("_pos_kernel")


@pytest.mark.parametrize("m", [2, 4])
def test_packed_on_many_tiles(m):
    from paper_2003_08646_amd import binding as B
    L = Wk.Layer("packed_many", 80, 130, 200, 14, 16, m=m, bits=4, seed=560)
    _check_layer(L, flags=B.LANCE_CODES_PACKED4, staged=False)


# Every kernel that multiplies outside the few-tile plans, with a layer that reaches it: where a small one
# does only with LANCE_PLAN_WIDE_TILES (last item), a layer large enough to be its own.
_PLANS = [
    ("conv_fused_c64_kernel", 200, 50, 70, 13, 14, 1, 2, 5, ""),
    ("conv_fused_pairs_nhwc_c64_kernel", 330, 60, 40, 10, 9, 1, 2, 8, "nhwc"),
    ("conv_fused_c128_kernel", 100, 96, 70, 16, 18, 1, 2, 6, ""),
    ("conv_fused_pairs_c64_kernel", 200, 50, 70, 13, 16, 1, 2, 5, ""),
    ("conv_fused_pairs_c128_kernel", 100, 96, 70, 16, 16, 1, 2, 6, ""),
    ("conv_fused_pairs_nhwc_c128_kernel", 110, 72, 130, 14, 13, 0, 2, 8, "nhwc"),
    ("conv_fused_c16_shared_kernel", 60, 12, 40, 33, 31, 1, 2, 8, ""),
    ("conv_fused_c16_shared_kernel", 60, 3, 70, 32, 32, 1, 2, 4, "nhwc"),
    ("conv_fused_c16_kernel", 250, 12, 40, 33, 31, 1, 2, 8, ""),
    ("conv_fused_c16_kernel", 250, 3, 20, 32, 32, 1, 2, 4, "nhwc"),
    ("conv_fused_c16_kernel", 200, 7, 20, 33, 31, 1, 2, 6, "nhwc"),
    ("conv_fused_m4_kernel", 100, 40, 130, 20, 21, 1, 4, 8, ""),
    ("gemm_fused_rows_kernel", 90, 150, 40, 14, 14, 1, 2, 8, ""),
    ("gemm_fused_rows_kernel", 70, 140, 130, 14, 15, 0, 2, 7, "nhwc"),
    ("gemm_fused_m2_stream_kernel", 80, 150, 130, 13, 15, 1, 2, 8, ""),
    ("gemm_fused_m4_stream_kernel", 60, 150, 200, 15, 17, 1, 4, 8, ""),
    ("gemm_fused_m4_stream_kernel", 120, 70, 130, 17, 16, 0, 4, 8, "nhwc"),
    ("gemm_fused_tiled_m4_kernel", 120, 40, 130, 17, 16, 0, 4, 8, "nhwc"),
    ("gemm_fused_tiled_m4_kernel", 2, 600, 70, 12, 13, 1, 4, 8, "wide"),
    ("gemm_fused_kernel", 3, 12, 70, 13, 11, 1, 4, 8, "wide"),
    ("gemm_fused_kernel", 2, 3, 1030, 13, 11, 1, 2, 6, "wide"),
    ("gemm_fused_m2_packed_kernel", 80, 130, 200, 14, 16, 1, 2, 4, "packed"),
    ("gemm_fused_m4_packed_kernel", 80, 130, 200, 14, 16, 1, 4, 4, "packed"),
]


def _plan_id(p):
    return "%s_c%d_m%d_%s" % (p[0][:-7], p[2], p[7], p[9] or "nchw")


@pytest.mark.parametrize("option", ["static", "per_tensor", "widths", "ties"])
@pytest.mark.parametrize("plan", _PLANS, ids=_plan_id)
def test_options_of_every_plan(plan, option):
    """Ranges narrower than the data, one range for the whole tensor, filter codes of another width, and
    rounding ties with both clamps (as in test_rounding_ties_and_both_clamps)."""
    from paper_2003_08646_amd import binding as B
    kernel, N, C, K, H, W, pad, m, bits, form = plan
    bits_w = {8: 5, 7: 8, 6: 8, 5: 8, 4: 3}[bits] if option == "widths" else None
    L = Wk.Layer("plan", N, C, K, H, W, pad=pad, m=m, bits=bits, bits_w=bits_w, seed=660 + C)
    flags = {"": 0, "nhwc": B.LANCE_LAYOUT_NHWC, "wide": B.LANCE_PLAN_WIDE_TILES, "packed": B.LANCE_CODES_PACKED4}[form]
    X, Wt = Wk.make_inputs(L)
    static = None
    if option == "per_tensor":
        flags |= B.LANCE_RANGE_PER_TENSOR
    elif option == "static":
        static = (O.ranges(O.input_transform_f32(X, pad, m)) * np.float32(0.5)).astype(np.float32)
    elif option == "ties":
        X = np.random.default_rng(661).integers(0, 2 ** bits, size=X.shape).astype(np.float32)
        static = np.tile(np.array([0.0, 2.0 * (2 ** bits - 1)], np.float32), ((m + 2) ** 2, 1))
    if static is not None:
        flags |= B.LANCE_INPUT_RANGE_STATIC
    conv, _ = _check_layer(L, X, Wt, flags=flags, static_v_range=static, staged=False)
    assert _kernels(conv, _zeros(conv, form == "nhwc"))[3] == kernel


@pytest.mark.parametrize("plan", [p for p in _PLANS if p[9] in ("", "nhwc")], ids=_plan_id)
def test_twin_and_graph_of_every_plan(plan):
    """The timing twin and graph replays (test_gpu_parity.py) on layers that are the plans' own."""
    _, N, C, K, H, W, pad, m, bits, form = plan
    L = Wk.Layer("plan_" + form, N, C, K, H, W, pad=pad, m=m, bits=bits, seed=670 + C)
    parity.test_timing_twin_runs_the_same_kernels(L)
    parity.test_fused_call_replays_from_a_hip_graph(L)


@pytest.mark.parametrize("L", [
    Wk.Layer("pos", 4, 64, 48, 16, 16, m=2, seed=680),
    Wk.Layer("pos_nhwc", 4, 130, 48, 16, 16, m=4, seed=681),
    Wk.Layer("split", 2, 600, 48, 12, 12, m=2, seed=682),
    Wk.Layer("split_nhwc", 2, 330, 48, 12, 12, m=4, seed=683),
    Wk.Layer("reduction_kernel", 40, 3, 70, 65, 63, m=4, seed=684),
], ids=lambda l: l.name)
def test_twin_and_graph_of_few_tile_plans(L):
    parity.test_timing_twin_runs_the_same_kernels(L)
    parity.test_fused_call_replays_from_a_hip_graph(L)


# N, C, K, H, W, pad, m, bits_w: one and two tile groups, one, two and four filter groups, partial
# rows of 32 channels; the last ones in the vector-ALU form (few channels and filters, many tiles)
_WEIGHT_ONLY = [
    (1, 100, 20, 9, 11, 1, 2, 8),
    (20, 40, 30, 14, 13, 0, 2, 6),
    (40, 20, 70, 20, 19, 1, 2, 4),
    (3, 33, 64, 40, 41, 2, 2, 8),
    (90, 16, 33, 12, 12, 1, 2, 3),
    (4, 140, 20, 15, 17, 1, 4, 8),
    (60, 5, 40, 14, 16, 1, 4, 4),
    (70, 3, 5, 57, 55, 1, 2, 8),
    (40, 1, 40, 56, 56, 0, 2, 4),
    (70, 20, 9, 56, 54, 2, 2, 6),
    (70, 2, 3, 60, 57, 1, 4, 8),
    (3, 40, 20, 9, 8, 5, 4, 8),
    (3, 41, 20, 1, 3, 2, 2, 8),
    (2, 37, 5, 1, 1, 5, 4, 8),
]


@pytest.mark.parametrize("nhwc", [False, True], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("shape", _WEIGHT_ONLY, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d_w%d" % s)
def test_weight_only_shapes(shape, nhwc):
    """Relative error (2-norm) below that of binary32 sums: sqrt(C) * 2^-24 per sum of C terms, times
    the growth of A^T M A (at most about 8 for F(4x4)): 4e-6 at 140 channels."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    N, C, K, H, W, pad, m, bits_w = shape
    L = Wk.Layer("wo", N, C, K, H, W, pad=pad, m=m, bits_w=bits_w, seed=570 + C)
    X, Wt = Wk.make_inputs(L)
    ref = O.weight_only_conv_f64(X, Wt, pad, m, bits_w, filters=O.prepare_filters(Wt, m, bits_w))
    conv = LanceConv(N, C, H, W, K, pad, m, 8, B.LANCE_LAYOUT_NHWC if nhwc else 0, bits_w=bits_w)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    x = torch.from_numpy(np.ascontiguousarray(X.transpose(0, 2, 3, 1)) if nhwc else X).cuda()
    conv.y.fill_(float("nan"))
    B.lance_conv3x3_winograd_wq_f32(conv.desc, x, conv.uq, conv.u_range, conv.y)
    torch.cuda.synchronize()
    got = conv.y.cpu().numpy().astype(np.float64)
    got = got.transpose(0, 3, 1, 2) if nhwc else got
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"[case] {shape} nhwc={nhwc}: rel {rel:.2g}", flush=True)
    assert rel <= 4e-6


@pytest.mark.parametrize("nhwc", [False, True], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("m", [2, 4])
def test_weight_only_inputs_of_2gib(m, nhwc):
    """Beyond the matrix-core kernel's 32-bit offsets: images from both ends and the middle of a
    2047 MiB tensor, each as if it stood alone."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    N, C, K, H = 2047, 16, 4, 128
    _, Wt = Wk.make_inputs(Wk.Layer("wo_2gib", 1, C, K, 8, 8, m=m, seed=630))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(630)
    x = torch.randn((N, H, H, C) if nhwc else (N, C, H, H), generator=gen, device="cuda")
    conv = LanceConv(N, C, H, H, K, 1, m, 8, B.LANCE_LAYOUT_NHWC if nhwc else 0)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    B.lance_conv3x3_winograd_wq_f32(conv.desc, x, conv.uq, conv.u_range, conv.y)
    filters = O.prepare_filters(Wt, m, 8)
    for n in (0, 1, 1023, N - 2, N - 1):
        X, got = x[n:n + 1].cpu().numpy(), conv.y[n:n + 1].cpu().numpy().astype(np.float64)
        X, got = (X.transpose(0, 3, 1, 2), got.transpose(0, 3, 1, 2)) if nhwc else (X, got)
        ref = O.weight_only_conv_f64(np.ascontiguousarray(X), Wt, 1, m, 8, filters=filters)
        assert np.linalg.norm(got - ref) <= 4e-6 * np.linalg.norm(ref), n


@pytest.mark.parametrize("kind", ["one_sided_filter", "outlying_weight", "positive_range"])
@pytest.mark.parametrize("C,m,bits_w", [(64, 2, 8), (512, 2, 8), (512, 2, 4), (100, 4, 8)])
def test_weight_only_ranges_away_from_zero(kind, C, m, bits_w):
    """Filter ranges that are not centred at zero: one filter far larger than the others and of one
    sign (a folded batch norm), one outlying weight, and a range without zero.  The error of the other
    filters stays that of the C rounded additions of their own terms, about sqrt(C) * 2^-24 / 2 (6.7e-7
    at 512 channels; measured at most 3.8e-7), times 4 for the growth of A^T M A with F(4x4)."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    K, H = 40, 14
    L = Wk.Layer("wo_asym", 1, C, K, H, H, m=m, bits_w=bits_w, seed=600 + C)
    X, Wt = Wk.make_inputs(L)
    if kind == "one_sided_filter":
        Wt[0] = -10 * np.abs(Wt[0])
    elif kind == "outlying_weight":
        Wt[0, C // 2, 1, 1] = -3.0
    else:
        Wt = np.abs(Wt) + np.float32(0.5)
    ref = O.weight_only_conv_f64(X, Wt, 1, m, bits_w, filters=O.prepare_filters(Wt, m, bits_w))
    conv = LanceConv(1, C, H, H, K, 1, m, 8, 0, bits_w=bits_w)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    B.lance_conv3x3_winograd_wq_f32(conv.desc, torch.from_numpy(X).cuda(), conv.uq, conv.u_range, conv.y)
    got = conv.y.cpu().numpy().astype(np.float64)
    rel = float(np.linalg.norm((got - ref)[:, 1:]) / np.linalg.norm(ref[:, 1:]))
    print(f"[case] {kind} C{C} m{m} w{bits_w}: rel {rel:.2g}", flush=True)
    assert rel <= 0.5 * np.sqrt(C) * 2.0 ** -24 * (4 if m == 4 else 1)


@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("exponent", [-110, -125, -140])
def test_weight_only_tiny_inputs(exponent, m):
    """Inputs near and below the smallest normal binary32 number: the split of the inputs stays exact,
    so the bound is that of test_weight_only_shapes.  (Filters times 2^60: normal outputs.)"""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    N, C, K, H = 1, 64, 40, 14
    X, Wt = Wk.make_inputs(Wk.Layer("wo_tiny", N, C, K, H, H, m=m, seed=620))
    X, Wt = np.ldexp(X, exponent).astype(np.float32), np.ldexp(Wt, 60).astype(np.float32)
    ref = O.weight_only_conv_f64(X, Wt, 1, m, 8, filters=O.prepare_filters(Wt, m, 8))
    conv = LanceConv(N, C, H, H, K, 1, m, 8)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    B.lance_conv3x3_winograd_wq_f32(conv.desc, torch.from_numpy(X).cuda(), conv.uq, conv.u_range, conv.y)
    got = conv.y.cpu().numpy().astype(np.float64)
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"[case] 2^{exponent} m{m}: rel {rel:.2g}", flush=True)
    assert rel <= 4e-6


_BT = {2: [[1, 0, -1, 0], [0, 1, 1, 0], [0, -1, 1, 0], [0, 1, 0, -1]],
       4: [[4, 0, -5, 0, 1, 0], [0, -4, -4, 1, 1, 0], [0, 4, -4, -1, 1, 0], [0, -2, -1, 2, 1, 0],
           [0, 2, -1, -2, 1, 0], [0, 4, 0, -5, 0, 1]]}
_AT = {2: [[1, 1, 1, 0], [0, 1, -1, -1]],
       4: [[1, 1, 1, 1, 1, 0], [0, 1, -1, 2, -2, 0], [0, 1, 1, 4, 4, 0], [0, 1, -1, 8, -8, 1]]}


def _two_sided(rows, t):
    """rows t rows^T over the last two axes, terms with coefficient 0 left out (0 * inf is no term)."""
    for _ in range(2):
        t = np.stack([sum(c * t[..., i, :] for i, c in enumerate(row) if c) for row in rows], -1)
    return t


@pytest.mark.parametrize("nhwc", [False, True], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("N,K,C", [(2, 20, 3), (2, 20, 40), (72, 125, 43)])
def test_weight_only_infinities(N, K, C, m, nhwc):
    """Infinities, a NaN and values whose sums of codes overflow: infinite and undefined results are
    those of the plain sums, the others within 4e-6 of the largest term's scale."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    H, W = 12, 13
    X, Wt = Wk.make_inputs(Wk.Layer("wo", N, C, K, H, W, pad=0, m=m, seed=590 + C))
    X[0, 1, 0, 0] = np.inf
    X[0, 2, 6, 7] = -np.inf
    X[N // 2, C - 1, 5, 5] = np.inf
    X[1, 0, 11, 12] = np.nan
    X[1, 1, 0, 0] = 1e37
    f = O.prepare_filters(Wt, m, 8)
    lo, hi = (f.u_range[:, i, None, None].astype(np.float64) for i in range(2))
    u = (f.Uq[:, :, :C].astype(np.float64) + 128) * ((hi - lo) / 255) + lo  # [E][K][C]
    th, tw, a = -(-(H - 2) // m), -(-(W - 2) // m), m + 2
    xp = np.zeros((N, C, th * m + 2, tw * m + 2))
    xp[:, :, :H, :W] = X
    ref = np.zeros((N, K, th * m, tw * m))
    with np.errstate(invalid="ignore"):
        for ty in range(th):
            for tx in range(tw):
                v = _two_sided(_BT[m], xp[:, :, ty * m:ty * m + a, tx * m:tx * m + a])
                mm = np.matmul(u, v.reshape(N, C, a * a).transpose(2, 1, 0))  # [E][K][N]
                ref[:, :, ty * m:ty * m + m, tx * m:tx * m + m] = _two_sided(_AT[m], mm.transpose(2, 1, 0).reshape(N, K, a, a))
    ref = ref[:, :, :H - 2, :W - 2]
    conv = LanceConv(N, C, H, W, K, 0, m, 8, B.LANCE_LAYOUT_NHWC if nhwc else 0)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    x = torch.from_numpy(np.ascontiguousarray(X.transpose(0, 2, 3, 1)) if nhwc else X).cuda()
    B.lance_conv3x3_winograd_wq_f32(conv.desc, x, conv.uq, conv.u_range, conv.y)
    got = conv.y.cpu().numpy().astype(np.float64)
    got = got.transpose(0, 3, 1, 2) if nhwc else got
    assert np.isinf(ref).any() and np.isnan(ref).any()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    np.testing.assert_array_equal(np.where(np.isinf(got), got, 0), np.where(np.isinf(ref), ref, 0))
    fin, big = np.isfinite(ref), np.abs(ref) > 1e30
    assert (fin & big).any()
    for part in (fin & big, fin & ~big & (np.arange(H - 2) >= m)[:, None]):  # (row 0's tiles hold the 1e37)
        assert np.linalg.norm(got[part] - ref[part]) <= 4e-6 * np.linalg.norm(ref[part])


# K, C, m, bits_w: one kernel / two kernels, 256- and 512-thread workgroups, workgroups with unequal
# numbers of filters, few records per workgroup, rows of 16, 32 and 64 bytes
_FILTERS = [
    (1, 1, 2, 8), (65, 64, 2, 8), (64, 64, 4, 8), (400, 16, 2, 5), (67, 130, 2, 8), (9, 700, 4, 8),
    (333, 250, 2, 8), (333, 250, 4, 3), (700, 7, 4, 8), (5000, 3, 2, 8),
]


@pytest.mark.parametrize("K,C,m,bits_w", _FILTERS)
@pytest.mark.parametrize("flags", ["nchw", "nhwc", "packed", "per_tensor"])
def test_filter_transform_shapes(K, C, m, bits_w, flags):
    """Codes, ranges and row sums bit for bit, twice in a row on one set of buffers."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    if flags == "packed":
        if C <= 16:
            pytest.skip("packed codes need more than 16 channels")
        bits_w = min(bits_w, 4)
    f = {"nchw": 0, "nhwc": B.LANCE_LAYOUT_NHWC, "packed": B.LANCE_CODES_PACKED4, "per_tensor": B.LANCE_RANGE_PER_TENSOR}[flags]
    conv = LanceConv(1, C, 8, 8, K, 1, m, min(bits_w, 4) if flags == "packed" else 8, f, bits_w=bits_w)
    rng = np.random.default_rng(580 + K + C)
    for _ in range(2):
        Wt = rng.standard_normal((K, C, 3, 3), dtype=np.float32)
        ref = O.prepare_filters(Wt, m, bits_w, per_tensor=flags == "per_tensor")
        conv.prepare_filters(torch.from_numpy(Wt).cuda())
        torch.cuda.synchronize()
        np.testing.assert_array_equal(conv.u_range.cpu().numpy(), ref.u_range)
        _assert_codes(conv.codes_to_logical(conv.uq, K), ref.Uq, "filter codes")
        np.testing.assert_array_equal(conv.u_rowsum.cpu().numpy(), ref.u_rowsum)


@pytest.mark.parametrize("kind", ["overflow", "nan", "inf"])
@pytest.mark.parametrize("bits_w,packed", [(8, False), (4, False), (4, True), (2, False)])
@pytest.mark.parametrize("m", [2, 4])
def test_filter_codes_at_the_end_of_binary32(m, bits_w, packed, kind):
    """Ranges whose width overflows, undefined and infinite weights: codes stay within their width, and
    an undefined product takes code 0."""
    from paper_2003_08646_amd import binding as B
    from paper_2003_08646_amd.layer import LanceConv
    K, C = 20, 70
    Wt = np.random.default_rng(640).standard_normal((K, C, 3, 3)).astype(np.float32)
    if kind == "overflow":
        Wt[3, 5], Wt[7, 60] = 0, 0
        Wt[3, 5, 0, 0], Wt[7, 60, 0, 0] = 2e38, -2e38
    else:
        Wt[3, 5, 1, 1] = float(kind)
    with np.errstate(invalid="ignore", over="ignore"):
        U = O.filter_transform_f32(Wt, m)  # [E][K][C]
        lo, hi = np.fmin.reduce(U, (1, 2)), np.fmax.reduce(U, (1, 2))
        inv = ((2 ** bits_w - 1) / (hi.astype(np.float64) - lo)).astype(np.float32)
        t = (U - lo[:, None, None]) * inv[:, None, None]
        ref = np.where(np.isnan(t), 0, np.clip(np.rint(t), 0, 2 ** bits_w - 1)).astype(np.int32) - 2 ** (bits_w - 1)
    conv = LanceConv(1, C, 8, 8, K, 1, m, 4, B.LANCE_CODES_PACKED4 if packed else 0, bits_w=bits_w)
    conv.prepare_filters(torch.from_numpy(Wt).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(conv.u_range.cpu().numpy(), np.stack([lo, hi], 1))
    _assert_codes(conv.codes_to_logical(conv.uq, K), ref, "filter codes")
    np.testing.assert_array_equal(conv.u_rowsum.cpu().numpy(), ref.sum(2))


# N, C, K, H, W, bits: layers whose tiles pair up (pad 1, width a multiple of 4)
_PAIRS = [
    (1200, 20, 30, 7, 4, 8),      # one pair per row; blocks of several images; odd height
    (500, 64, 64, 9, 8, 8),       # two pairs per row, whole channel block
    (150, 61, 70, 12, 20, 5),     # rows that end inside a group of lanes
    (60, 64, 384, 16, 32, 8),
    (60, 64, 385, 16, 32, 8),     # a last block of one filter
    (60, 64, 704, 16, 16, 8),     # the most filters of one channel block
    (3, 48, 33, 111, 224, 8),     # rows of several groups of lanes
    (90, 128, 130, 14, 28, 8),    # two channel blocks, whole; two blocks of filters
    (1400, 65, 17, 6, 4, 6),
    (100, 100, 72, 15, 36, 8),
    (30, 127, 640, 20, 24, 8),
    (30, 127, 641, 20, 24, 8),
    (30, 127, 768, 20, 24, 6),    # the most filters of two channel blocks
    (33, 70, 20, 33, 64, 8),      # non-temporal stores
]


@pytest.mark.parametrize("shape", _PAIRS, ids=lambda s: "n%d_c%d_k%d_%dx%d_b%d" % s)
@pytest.mark.parametrize("option", ["dynamic", "static", "per_tensor"])
def test_layers_whose_tiles_pair_up(shape, option):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, bits = shape
    L = Wk.Layer("pairs", N, C, K, H, W, m=2, bits=bits, seed=700 + C)
    flags = {"dynamic": 0, "static": B.LANCE_INPUT_RANGE_STATIC, "per_tensor": B.LANCE_RANGE_PER_TENSOR}[option]
    static = _range_of_another_batch(L) if option == "static" else None
    conv, _ = _check_layer(L, flags=flags, static_v_range=static, staged=False)
    names = _kernels(conv, _zeros(conv, False))
    assert names[3] == ("conv_fused_pairs_c64_kernel" if C <= 64 else "conv_fused_pairs_c128_kernel"), names


# layers of 257 to 512 few-tile workgroups whose tiles pair up: (N, C, K, H, W) and the kernel that takes them
@pytest.mark.parametrize("shape,kernel", [
    ((200, 20, 16, 7, 16), "conv_fused_pos_kernel"),            # at most 16 filters on one channel block
    ((70, 64, 5, 15, 24), "conv_fused_pos_kernel"),
    ((200, 20, 17, 7, 16), "conv_fused_pairs_c64_kernel"),
    ((200, 20, 64, 7, 16), "conv_fused_pairs_c64_kernel"),
    ((200, 70, 5, 7, 16), "conv_fused_pairs_c128_kernel"),      # two channel blocks: whatever the filters
], ids=lambda v: v if isinstance(v, str) else "n%d_c%d_k%d_%dx%d" % v)
def test_where_the_pair_kernel_takes_over(shape, kernel):
    N, C, K, H, W = shape
    conv, _ = _check_layer(Wk.Layer("meet", N, C, K, H, W, m=2, seed=900 + C), staged=False)
    names = _kernels(conv, _zeros(conv, False))
    assert names[3] == kernel, names


# one filter more than the pair kernel's LDS holds: one tile per lane
@pytest.mark.parametrize("shape", [(60, 64, 705, 16, 16, 8), (30, 127, 769, 20, 24, 6)],
                         ids=lambda s: "n%d_c%d_k%d_%dx%d_b%d" % s)
def test_more_filters_than_the_pair_kernel_takes(shape):
    N, C, K, H, W, bits = shape
    conv, _ = _check_layer(Wk.Layer("pairs", N, C, K, H, W, m=2, bits=bits, seed=700 + C), staged=False)
    names = _kernels(conv, _zeros(conv, False))
    assert names[3] == ("conv_fused_c64_kernel" if C <= 64 else "conv_fused_c128_kernel"), names


# N, C, K, H, W, pad, m: patches by rows with any column outside the image, the smallest images that are
# loaded so; first and last plane of the tensor pixel by pixel
_ROWS_ANY = [
    (3, 20, 12, 2, 5, 1, 2), (1, 64, 20, 5, 7, 1, 2), (2, 33, 9, 4, 4, 0, 2), (1, 17, 5, 3, 4, 0, 2),
    (2, 130, 17, 3, 5, 1, 2), (1, 150, 8, 7, 9, 0, 2), (70, 192, 20, 7, 9, 1, 2),
    (2, 20, 12, 3, 7, 1, 4), (1, 64, 9, 6, 9, 1, 4), (2, 70, 17, 5, 6, 0, 4), (1, 17, 5, 3, 6, 0, 4),
    (2, 130, 8, 7, 11, 1, 4), (1, 150, 20, 9, 6, 0, 4), (40, 192, 20, 13, 10, 1, 4),
]


@pytest.mark.parametrize("shape", _ROWS_ANY, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d" % s)
def test_rows_of_any_width(shape):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, m = shape
    L = Wk.Layer("rows", N, C, K, H, W, pad=pad, m=m, seed=740 + C)
    _check_layer(L, flags=B.LANCE_PLAN_WIDE_TILES)


# the two-block kernel by rows with shifted ends: widths whose last patch sticks out by one and by two columns,
# few images (first and last image in many workgroups), whole and partial blocks
@pytest.mark.parametrize("shape", [(1, 128, 20, 190, 175, 1, 8), (2, 96, 130, 130, 133, 0, 8), (3, 65, 17, 106, 105, 1, 5),
                                   (1, 100, 40, 190, 182, 0, 8), (2, 127, 20, 130, 131, 1, 6), (900, 72, 20, 5, 7, 1, 8),
                                   (1500, 128, 9, 4, 5, 1, 8)],
                         ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d" % s)
def test_two_block_kernel_on_rows_of_any_width(shape):
    N, C, K, H, W, pad, bits = shape
    conv, _ = _check_layer(Wk.Layer("rows128", N, C, K, H, W, pad=pad, m=2, bits=bits, seed=920 + C), staged=False)
    names = _kernels(conv, _zeros(conv, False))
    assert names[3] == "conv_fused_c128_kernel", names


def test_fused_m4_reduction_kernel_on_many_tiles():
    """F(4x4): enough workgroups and range records that the reduction kernel runs between the passes."""
    L = Wk.Layer("m4_many_tiles", 36, 20, 8, 224, 224, m=4, seed=760)
    conv, _ = _check_layer(L, staged=False)
    assert _kernels(conv, _zeros(conv, False))[1:] == ["range_finalize_kernel", "", "conv_fused_m4_kernel"]


# N, C, K, H, W, pad, bits: quantize pass with all channel blocks in one workgroup (four to eight blocks, 1521
# to 4096 tiles; with a partial block only where two of three things favour it: the caller's ranges, unpacked
# codes, 192 workgroups of 64 tiles); the last two: one tile less and one block of tiles more
_WHOLE = [
    (32, 256, 20, 14, 13, 1, 8), (20, 300, 17, 18, 18, 1, 8), (33, 512, 9, 14, 14, 1, 8), (30, 449, 8, 16, 17, 0, 6),
    (2, 270, 5, 78, 80, 1, 8), (32, 260, 20, 14, 14, 1, 4), (33, 512, 9, 15, 15, 0, 3),
    (1, 256, 5, 80, 76, 1, 8), (1, 256, 5, 128, 130, 1, 8),
]


@pytest.mark.parametrize("shape", _WHOLE, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d" % s)
@pytest.mark.parametrize("static", [False, True], ids=["dynamic", "static"])
def test_quantize_pass_with_all_channel_blocks(shape, static):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, bits = shape
    L = Wk.Layer("whole", N, C, K, H, W, pad=pad, m=2, bits=bits, seed=800 + C)
    flags = B.LANCE_PLAN_WIDE_TILES | (B.LANCE_INPUT_RANGE_STATIC if static else 0)
    for packed in ([0, B.LANCE_CODES_PACKED4] if bits <= 4 else [0]):
        conv, _ = _check_layer(L, flags=flags | packed,
                               static_v_range=_range_of_another_batch(L) if static else None)
        P, blocks = conv.sz.P, conv.sz.NB
        whole = 1520 < P <= 4096 and (C % 64 == 0 or static + (not packed) + (blocks * -(-P // 64) >= 192) >= 2)
        assert (_kernels(conv, _zeros(conv, False))[2] == "input_quant_m2_whole_kernel") == whole


# N, C, K, H, W, pad, bits: NHWC, tile rows of whole pairs (a multiple of four tiles): a row of two pairs, padding of 0
# to 2, ragged heights, a last workgroup of two pairs, whole and partial blocks
_WHOLE_PAIRS = [
    (330, 20, 17, 13, 8, 1, 8), (421, 64, 32, 9, 7, 1, 5), (141, 44, 20, 11, 26, 0, 8), (150, 64, 48, 13, 14, 2, 8),
    (330, 68, 17, 13, 8, 1, 8), (421, 128, 32, 9, 7, 1, 5), (141, 100, 20, 11, 26, 0, 8), (150, 128, 48, 13, 14, 2, 8),
    (91, 128, 130, 16, 24, 1, 8), (70, 64, 65, 16, 32, 1, 8),
]


@pytest.mark.parametrize("shape", _WHOLE_PAIRS, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d" % s)
@pytest.mark.parametrize("static", [False, True], ids=["dynamic", "static"])
def test_nhwc_rows_of_whole_pairs(shape, static):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, bits = shape
    L = Wk.Layer("whole_pairs", N, C, K, H, W, pad=pad, m=2, bits=bits, seed=860 + C)
    conv, _ = _check_layer(L, flags=B.LANCE_LAYOUT_NHWC | (B.LANCE_INPUT_RANGE_STATIC if static else 0), staged=False,
                           static_v_range=_range_of_another_batch(L) if static else None)
    assert -(-(W + 2 * pad - 2) // 2) % 4 == 0
    names = _kernels(conv, _zeros(conv, True))
    assert names[3] == "conv_fused_pairs_nhwc_%s_kernel" % ("c64" if C <= 64 else "c128"), names


# N, C, K, H, W, pad, bits: NHWC pairs of tiles: one, two and three tile columns, odd numbers of them, widths that
# are no multiple of anything, filters that are no multiple of four and of sixteen (streamed stores; bound by them), padding lanes,
# one share of the filters, one more filter, three shares; rows of so many pairs that multiplying does not divide them
_NHWC_PAIRS = [
    (500, 20, 130, 13, 2, 1, 8), (900, 64, 20, 9, 3, 1, 8), (700, 40, 32, 9, 5, 1, 5), (420, 60, 21, 10, 11, 0, 8),
    (300, 64, 16, 8, 9, 2, 8), (300, 64, 704, 8, 9, 1, 8), (100, 44, 705, 9, 13, 1, 6), (40, 24, 1500, 9, 13, 1, 8),
    (500, 68, 260, 9, 2, 1, 8), (900, 128, 37, 9, 5, 0, 4), (260, 100, 130, 10, 11, 1, 8), (200, 128, 48, 8, 9, 2, 8),
    (60, 124, 768, 9, 13, 1, 8), (50, 72, 769, 9, 13, 1, 8), (1, 20, 17, 2, 262147, 1, 8), (8200, 20, 130, 2, 2, 1, 8),
]


# The same with pairs of any two tiles, where that takes fewer rounds of workgroups (one per compute unit): one tile column,
# three, five and nine (pairs across tile rows and images), half a pair at the end, no and wide padding, two shares of the
# filters, a row of so many tiles that multiplying does not divide them
_NHWC_ANY_PAIRS = [
    (1801, 20, 18, 13, 1, 1, 8), (1801, 64, 17, 13, 2, 1, 5), (1801, 68, 18, 9, 2, 1, 8), (985, 40, 32, 9, 5, 1, 8),
    (683, 60, 21, 10, 11, 0, 8), (277, 128, 130, 18, 18, 1, 8), (1601, 100, 64, 5, 6, 1, 6), (501, 44, 720, 9, 9, 1, 8),
    (2801, 128, 36, 5, 3, 0, 8), (650, 68, 130, 5, 3, 2, 4), (1, 20, 17, 10, 58981, 1, 8), (700, 68, 518, 5, 6, 1, 8),
    (401, 68, 830, 5, 6, 1, 8), (8200, 20, 127, 2, 2, 1, 8),
]


@pytest.mark.parametrize("shape", _NHWC_PAIRS + _NHWC_ANY_PAIRS, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d" % s)
@pytest.mark.parametrize("option", ["dynamic", "static", "per_tensor"])
def test_nhwc_pairs_of_tiles(shape, option):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, bits = shape
    L = Wk.Layer("nhwc_pairs", N, C, K, H, W, pad=pad, m=2, bits=bits, seed=880 + C)
    flags = {"dynamic": 0, "static": B.LANCE_INPUT_RANGE_STATIC, "per_tensor": B.LANCE_RANGE_PER_TENSOR}[option]
    conv, _ = _check_layer(L, flags=B.LANCE_LAYOUT_NHWC | flags, staged=False,
                           static_v_range=_range_of_another_batch(L) if option == "static" else None)
    names = _kernels(conv, _zeros(conv, True))
    kernel = "conv_fused_any_pairs_nhwc_%s_kernel" if shape in _NHWC_ANY_PAIRS else "conv_fused_pairs_nhwc_%s_kernel"
    assert names[3] == kernel % ("c64" if C <= 64 else "c128"), names


# N, C, H, W, pad: NHWC range pass in strips of one and of two tile columns (at least 4096 strips): one, two and three
# columns, an odd number of them, strips of the whole height and of a part of it
@pytest.mark.parametrize("shape", [(2100, 20, 3, 4, 1), (1400, 68, 9, 5, 1), (300, 64, 30, 9, 0), (16, 130, 70, 75, 2),
                                   (400, 256, 7, 13, 1), (1301, 20, 31, 2, 1), (2100, 64, 14, 1, 1), (2200, 36, 9, 1, 1),
                                   (1801, 128, 5, 6, 1), (900, 40, 13, 11, 0), (221, 100, 11, 11, 1)],
                         ids=lambda s: "n%d_c%d_%dx%d_p%d" % s)
def test_nhwc_ranges_from_strips(shape):
    from paper_2003_08646_amd import binding as B
    N, C, H, W, pad = shape
    C = C - C % 4
    conv, _ = _check_layer(Wk.Layer("nhwc_range", N, C, 24, H, W, pad=pad, m=2, seed=890 + C), flags=B.LANCE_LAYOUT_NHWC,
                           staged=False)
    assert _kernels(conv, _zeros(conv, True))[0] == "input_nhwc_range_roll_kernel"


def test_nhwc_of_four_byte_alignment_keeps_the_few_tile_plan():
    """Between one and two workgroups per compute unit the pair kernel takes NHWC layers whose X is 16-byte aligned."""
    from paper_2003_08646_amd import binding as B
    L = Wk.Layer("nhwc_align", 64, 128, 128, 14, 14, m=2, seed=895)
    conv, _ = _check_layer(L, flags=B.LANCE_LAYOUT_NHWC, staged=False)
    assert _kernels(conv, _zeros(conv, True))[3] == "conv_fused_pairs_nhwc_c128_kernel"
    buf = torch.zeros(64 * 14 * 14 * 128 + 1, device="cuda")
    x = torch.from_numpy(np.ascontiguousarray(Wk.make_inputs(L)[0].transpose(0, 2, 3, 1))).cuda()
    y = conv.forward(x).clone()
    shifted = buf[1:].view(x.shape)
    shifted.copy_(x)
    y2 = conv.forward(shifted)
    assert (y - y2).abs().max() <= 1e-5 * y.abs().max()
    assert _kernels(conv, shifted)[3] == "conv_fused_pos_kernel"


# Between one and two workgroups of the few-tile plan per compute unit: (N, C, K, H, W), caller's ranges, whether the pair
# kernel takes the layer
@pytest.mark.parametrize("shape,static,pairs", [
    ((2, 64, 704, 28, 28), False, False), ((2, 64, 704, 28, 28), True, False),     # several blocks of filters
    ((1, 100, 1025, 38, 38), False, False), ((4, 68, 174, 47, 55), True, False), ((12, 88, 130, 40, 20), False, False),
    ((16, 64, 65, 30, 30), False, False),
    ((20, 64, 64, 37, 35), True, True), ((20, 64, 61, 37, 35), True, False), ((20, 64, 61, 37, 35), False, False),
    ((20, 64, 32, 37, 35), True, False), ((20, 64, 20, 37, 35), False, True), ((20, 64, 16, 37, 35), False, False),
    ((64, 128, 128, 14, 14), True, True), ((64, 128, 125, 14, 14), True, False), ((64, 128, 70, 14, 14), True, True), ((64, 128, 74, 14, 14), True, False),
    ((64, 128, 125, 14, 14), False, True), ((20, 128, 33, 37, 35), True, True), ((20, 128, 62, 37, 35), True, True), ((20, 128, 31, 37, 35), True, False),
    ((896, 84, 53, 6, 6), True, False), ((896, 84, 12, 6, 6), False, False),      # pairs of any two tiles
    ((20, 128, 20, 37, 35), True, True), ((20, 128, 16, 37, 35), True, False), ((20, 128, 5, 37, 35), False, True),
], ids=lambda v: str(v) if isinstance(v, bool) else "n%d_c%d_k%d_%dx%d" % v)
def test_where_the_nhwc_pair_kernel_takes_over(shape, static, pairs):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W = shape
    groups = -(-N * -(-H // 2) * -(-W // 2) // 16) * -(-K // 64)
    assert 256 < groups <= 512
    L = Wk.Layer("meet_nhwc", N, C, K, H, W, m=2, seed=900 + C)
    conv, _ = _check_layer(L, flags=B.LANCE_LAYOUT_NHWC | (B.LANCE_INPUT_RANGE_STATIC if static else 0), staged=False,
                           static_v_range=_range_of_another_batch(L) if static else None)
    names = _kernels(conv, _zeros(conv, True))
    assert names[3] == ("conv_fused_pairs_nhwc_%s_kernel" % ("c64" if C <= 64 else "c128") if pairs else "conv_fused_pos_kernel"), names


# K, C, m, bits_w: filters of a last unit of four that is not whole, padding lanes, one, several and many units of 64 codes
# per wave on workgroups of 256, 512 and 1024 threads, equal and unequal shares, one filter to a workgroup, few filters of
# many channels, 64, 128 and 256 copies of the records
@pytest.mark.parametrize("K,C,m,bits_w", [(6, 16, 2, 8), (3, 17, 4, 2), (63, 65, 2, 4), (64, 64, 2, 3), (17, 63, 4, 8),
                                          (1, 512, 2, 8), (260, 100, 2, 6), (90, 513, 4, 8), (600, 129, 2, 8),
                                          (1025, 420, 2, 8), (4097, 1, 4, 4), (2, 2100, 2, 8), (3, 2113, 4, 4),
                                          (60, 80, 2, 8), (100, 100, 4, 3), (3100, 70, 2, 8)])
@pytest.mark.parametrize("flags", ["nchw", "nhwc", "packed", "per_tensor"])
def test_filter_transform_units(K, C, m, bits_w, flags):
    test_filter_transform_shapes(K, C, m, bits_w, flags)


# N, C, K, H, W, pad, m, bits, nhwc: few-tile plans with one range for the whole tensor, reduced by every workgroup: one,
# two and four groups of filters on 16 and 8 waves, F(4x4), two kernels
@pytest.mark.parametrize("shape", [(2, 20, 10, 9, 8, 1, 2, 8, False), (20, 33, 60, 14, 14, 1, 2, 6, False),
                                   (45, 40, 70, 14, 15, 1, 2, 8, False), (33, 18, 70, 15, 16, 1, 4, 5, False),
                                   (40, 30, 40, 16, 13, 1, 4, 8, True), (2, 330, 20, 9, 10, 1, 4, 8, False),
                                   (3, 16, 40, 120, 120, 1, 4, 8, False), (2, 48, 20, 62, 60, 1, 2, 8, False)],
                         ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_m%d_b%d%s" % (s[:8] + ("_nhwc" if s[8] else "",)))
def test_position_parallel_per_tensor(shape):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, m, bits, nhwc = shape
    L = Wk.Layer("per_tensor", N, C, K, H, W, pad=pad, m=m, bits=bits, seed=940 + C)
    conv, _ = _check_layer(L, flags=B.LANCE_RANGE_PER_TENSOR | (B.LANCE_LAYOUT_NHWC if nhwc else 0), staged=False)
    names = _kernels(conv, _zeros(conv, nhwc))
    assert names[1] == "" and names[3] in ("conv_fused_pos_kernel", "gemm_pos_kernel"), names


# N, C, K, H, W, m, batch: the same plans with more records of the range pass than the threads of a workgroup request at
# once (batch): 8 waves, F(4x4), the quantize pass of the plans in two kernels; whole turns and a part of one
_MANY_RECORDS = [(10, 128, 200, 27, 27, 2, 128), (9, 128, 200, 27, 29, 2, 128), (80, 128, 40, 15, 15, 4, 80),
                 (60, 120, 40, 15, 13, 4, 80), (9, 600, 20, 9, 7, 2, 64), (10, 330, 20, 9, 10, 4, 24)]


@pytest.mark.parametrize("shape", _MANY_RECORDS, ids=lambda s: "n%d_c%d_k%d_%dx%d_m%d_%d" % s)
@pytest.mark.parametrize("per_tensor", [False, True], ids=["per_position", "per_tensor"])
def test_position_parallel_with_many_records(shape, per_tensor):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, m, batch = shape
    blocks = -(-N * -(-H // m) * -(-W // m) // 64)                     # of the lane-per-tile range pass:
    chunk = -(-C // min(512 // blocks, -(-C // 8)))                    # channels of a work unit,
    records = -(-blocks * -(-C // (-(-chunk // 4) * 4)) // 2)          # two units to a workgroup and record
    assert records > batch
    L = Wk.Layer("records", N, C, K, H, W, m=m, seed=950 + C)
    conv, _ = _check_layer(L, flags=B.LANCE_RANGE_PER_TENSOR if per_tensor else 0, staged=False)
    names = _kernels(conv, _zeros(conv, False))
    assert names[:2] == ["input_range_kernel", ""] and names[3] in ("conv_fused_pos_kernel", "gemm_pos_kernel"), names


# N, C, K, H, W, pad, bits, nhwc, waves: the small-channel kernel with two and four waves to 64 tiles (test_share_rule.py checks
# that each shape is divided so): one, two, three and many tiles of 32 filters, odd numbers of them, a last block of one
# tile and of whole ones, odd sizes; below 12800 tiles where it takes over from the few-tile plan
_C16_SHARED = [
    (48, 5, 17, 10, 134, 1, 8, False, 2), (53, 3, 33, 19, 57, 1, 8, False, 4), (128, 16, 16, 32, 32, 1, 8, False, 2),
    (16, 4, 65, 57, 55, 1, 5, False, 4), (11, 3, 103, 75, 75, 0, 8, False, 4), (1, 16, 200, 225, 229, 1, 8, False, 4),
    (1, 3, 64, 224, 224, 1, 8, False, 4), (9, 2, 100, 65, 65, 1, 4, False, 4), (8, 1, 272, 83, 81, 1, 8, True, 4),
    (12, 2, 92, 79, 75, 1, 6, True, 2), (3, 7, 66, 131, 133, 1, 8, True, 4), (13, 1, 40, 63, 64, 1, 8, False, 4),
    (43, 16, 16, 37, 33, 1, 8, False, 2), (89, 4, 65, 25, 25, 1, 8, False, 4), (43, 2, 40, 37, 33, 1, 8, True, 4),
]


@pytest.mark.parametrize("shape", _C16_SHARED, ids=lambda s: "n%d_c%d_k%d_%dx%d_p%d_b%d%s" % (s[:7] + ("_nhwc" if s[7] else "",)))
@pytest.mark.parametrize("static", [False, True], ids=["dynamic", "static"])
def test_small_channel_waves_that_share_tiles(shape, static):
    from paper_2003_08646_amd import binding as B
    N, C, K, H, W, pad, bits, nhwc, _ = shape
    L = Wk.Layer("c16_shared", N, C, K, H, W, pad=pad, m=2, bits=bits, seed=960 + C)
    flags = (B.LANCE_LAYOUT_NHWC if nhwc else 0) | (B.LANCE_INPUT_RANGE_STATIC if static else 0)
    conv, _ = _check_layer(L, flags=flags, static_v_range=_range_of_another_batch(L) if static else None, staged=False)
    names = _kernels(conv, _zeros(conv, nhwc))
    if static or conv.sz.P > 12800:  # (with dynamic ranges the few-tile plan keeps more of the others)
        assert names[3] == "conv_fused_c16_shared_kernel", names


# N, C, H, W: F(4x4) range pass in strips of an even and of an odd number of tile rows, several strips to a plane, one
# segment to a row and as many as a wave has lanes
@pytest.mark.parametrize("shape", [(40, 20, 13, 20), (40, 20, 17, 20), (90, 33, 27, 4), (2, 24, 36, 256), (3, 20, 150, 12)],
                         ids=lambda s: "n%d_c%d_%dx%d" % s)
def test_m4_ranges_from_strips(shape):
    N, C, H, W = shape
    conv, _ = _check_layer(Wk.Layer("strip_m4", N, C, 24, H, W, pad=1, m=4, seed=900 + H), staged=False)
    assert _kernels(conv, _zeros(conv, False))[0] == "input_range_strip_m4_kernel"
