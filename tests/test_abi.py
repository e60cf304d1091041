"""CPU-only checks of the C ABI: every symbol the header declares is exported, descriptor
validation and size queries work with no GPU present, the documented code layout holds."""
import os
import re

import numpy as np
import pytest

from paper_2003_08646_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "lance.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(lance_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared()
    assert set(B.EXPORTS) == set(names), (names, B.EXPORTS)
    lib = B.lib()
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_status_strings():
    assert B.lance_version() >= 100
    assert B.status_string(0) == "ok"
    for code in (-1, -2, -3, -4, -99):
        assert B.status_string(code)


def test_query_sizes_cfg2():
    s = B.lance_query_sizes(B.make_desc(128, 64, 32, 32, 64, pad=1, m=2, bits=8))
    assert (s.Ho, s.Wo, s.tiles_h, s.tiles_w, s.P, s.E) == (32, 32, 16, 16, 32768, 16)
    assert (s.Cp, s.CB, s.NB) == (64, 64, 1)
    assert s.uq_bytes == 16 * 64 * 64 and s.vq_bytes == 16 * 32768 * 64
    assert s.acc_bytes == 16 * 64 * 32768 * 4 and s.y_bytes == 128 * 64 * 32 * 32 * 4
    assert s.u_range_bytes == 16 * 2 * 4 and s.v_colsum_bytes == 16 * 32768 * 4
    assert s.conv_workspace_bytes >= s.vq_bytes + s.v_colsum_bytes
    assert s.input_workspace_bytes < s.conv_workspace_bytes


@pytest.mark.parametrize("C,Cp,CB,NB", [(3, 16, 16, 1), (16, 16, 16, 1), (17, 64, 64, 1),
                                        (48, 64, 64, 1), (64, 64, 64, 1), (65, 128, 64, 2),
                                        (130, 192, 64, 3), (512, 512, 64, 8)])
def test_channel_padding_rule(C, Cp, CB, NB):
    s = B.lance_query_sizes(B.make_desc(1, C, 8, 8, 4))
    assert (s.Cp, s.CB, s.NB) == (Cp, CB, NB)


def test_ragged_and_m4_geometry():
    s = B.lance_query_sizes(B.make_desc(2, 3, 7, 9, 5, pad=1, m=4))
    assert (s.Ho, s.Wo, s.tiles_h, s.tiles_w, s.P, s.E) == (7, 9, 2, 3, 12, 36)
    s = B.lance_query_sizes(B.make_desc(2, 3, 7, 9, 5, pad=0, m=2))
    assert (s.Ho, s.Wo, s.tiles_h, s.tiles_w, s.P) == (5, 7, 3, 4, 24)


@pytest.mark.parametrize("kw,code", [
    (dict(N=0), B.LANCE_ERR_INVALID_ARG), (dict(C=-1), B.LANCE_ERR_INVALID_ARG),
    (dict(K=0), B.LANCE_ERR_INVALID_ARG), (dict(pad=-1), B.LANCE_ERR_INVALID_ARG),
    (dict(H=2, pad=0), B.LANCE_ERR_INVALID_ARG),      # empty output
    (dict(m=3), B.LANCE_ERR_UNSUPPORTED), (dict(m=6), B.LANCE_ERR_UNSUPPORTED),
    (dict(bits=1), B.LANCE_ERR_UNSUPPORTED), (dict(bits=9), B.LANCE_ERR_UNSUPPORTED),
    (dict(flags=32), B.LANCE_ERR_UNSUPPORTED),
    (dict(flags=16, C=64, bits=8), B.LANCE_ERR_UNSUPPORTED),          # packed codes need <= 4 bits
    (dict(flags=16 | (5 << 8), C=64, bits=4), B.LANCE_ERR_UNSUPPORTED),   # ... of the filters too
    (dict(flags=16, C=16, bits=4), B.LANCE_ERR_UNSUPPORTED),          # ... and 64-channel blocks
    (dict(flags=1 << 8), B.LANCE_ERR_UNSUPPORTED),    # filter code width 1
    (dict(flags=9 << 8), B.LANCE_ERR_UNSUPPORTED),    # filter code width 9
    (dict(flags=1 << 12), B.LANCE_ERR_UNSUPPORTED),   # unknown flag above the width field
    (dict(flags=16 << 8), B.LANCE_ERR_UNSUPPORTED),   # LANCE_FILTER_BITS(16): not dropped silently
    (dict(K=65536), B.LANCE_ERR_UNSUPPORTED),         # K is a grid's y extent in some kernels
    (dict(N=65536, H=4, W=4), B.LANCE_ERR_UNSUPPORTED),
    (dict(N=340, C=64, H=224, W=224), B.LANCE_ERR_UNSUPPORTED),    # x beyond 4 GiB
    (dict(N=300, C=8, H=224, W=224, K=72), B.LANCE_ERR_UNSUPPORTED),   # y beyond 4 GiB
    (dict(N=1, C=70, H=2900, W=2900), B.LANCE_ERR_UNSUPPORTED),    # one image beyond 2 GiB
    (dict(N=4, C=512, H=724, W=724, K=4), B.LANCE_ERR_UNSUPPORTED),   # codes of V beyond 4 GiB
])
def test_descriptor_validation_needs_no_gpu(kw, code):
    base = dict(N=1, C=4, H=8, W=8, K=4, pad=1, m=2, bits=8, flags=0)
    base.update(kw)
    d = B.make_desc(**base)
    with pytest.raises(B.LanceError) as ei:
        B.lance_query_sizes(d)
    assert ei.value.status == code
    # the compute entry points reject the same descriptor before touching HIP
    with pytest.raises(B.LanceError) as ei:
        B.lance_winograd_gemm_i8(d, 16, 16, 16, stream=0)
    assert ei.value.status == code


def test_largest_supported_tensors_pass_validation():
    """Just inside the size limits: x and y a little below 4 GiB."""
    s = B.lance_query_sizes(B.make_desc(300, 64, 220, 224, 8))
    assert s.y_bytes < 2 ** 32 and 300 * 64 * 220 * 224 * 4 < 2 ** 32 - 16
    assert B.LANCE_FILTER_BITS(16) == 16 << 8


def test_staged_calls_reject_accumulators_beyond_4gib_before_hip():
    d = B.make_desc(64, 64, 224, 224, 96)      # acc = 16 * 96 * 802816 * 4 bytes > 4 GiB
    s = B.lance_query_sizes(d)
    assert s.acc_bytes >= 2 ** 32
    with pytest.raises(B.LanceError) as ei:
        B.lance_winograd_gemm_i8(d, 16, 16, 16, stream=0)
    assert ei.value.status == B.LANCE_ERR_UNSUPPORTED
    with pytest.raises(B.LanceError) as ei:
        B.lance_output_transform_dq(d, 16, 16, 16, 16, 16, 16, stream=0)
    assert ei.value.status == B.LANCE_ERR_UNSUPPORTED


def test_filter_bits_field_is_accepted_and_leaves_sizes_unchanged():
    base = B.lance_query_sizes(B.make_desc(2, 70, 9, 11, 20, bits=5))
    for bw in range(2, 9):
        s = B.lance_query_sizes(B.make_desc(2, 70, 9, 11, 20, bits=5, flags=B.LANCE_FILTER_BITS(bw)))
        assert (s.uq_bytes, s.vq_bytes, s.acc_bytes, s.conv_workspace_bytes) == \
            (base.uq_bytes, base.vq_bytes, base.acc_bytes, base.conv_workspace_bytes)
    assert B.LANCE_FILTER_BITS(6) == 6 << 8


def test_null_pointers_and_workspace_errors_need_no_gpu():
    d = B.make_desc(1, 4, 8, 8, 4)
    s = B.lance_query_sizes(d)
    calls = [
        lambda: B.lance_filter_transform_q8(d, None, 16, 16, 16, stream=0),
        lambda: B.lance_input_transform_q8(d, 16, None, 16, 16, 256, 1 << 30, stream=0),
        lambda: B.lance_winograd_gemm_i8(d, 16, 16, None, stream=0),
        lambda: B.lance_output_transform_dq(d, 16, 16, 16, 16, 16, None, stream=0),
        lambda: B.lance_conv3x3_winograd_q8(d, None, 16, 16, 16, None, 16, 256, 1 << 30, stream=0),
        lambda: B.lance_direct_conv3x3_f32(d, 16, None, 16, stream=0),
        lambda: B.lance_alg1_literal_f32(d, 16, None, 16, stream=0),
        lambda: B.lance_conv3x3_winograd_wq_f32(d, 16, 16, None, 16, stream=0),
    ]
    for c in calls:
        with pytest.raises(B.LanceError) as ei:
            c()
        assert ei.value.status == B.LANCE_ERR_INVALID_ARG
    ws_calls = [
        lambda: B.lance_input_transform_q8(d, 16, 16, 16, 16, None, 0, stream=0),
        lambda: B.lance_input_transform_q8(d, 16, 16, 16, 16, 256, s.input_workspace_bytes - 1, stream=0),
        lambda: B.lance_input_transform_q8(d, 16, 16, 16, 16, 257, 1 << 30, stream=0),   # misaligned
        lambda: B.lance_conv3x3_winograd_q8(d, 16, 16, 16, 16, None, 16, 256,
                                            s.conv_workspace_bytes - 1, stream=0),
    ]
    for c in ws_calls:
        with pytest.raises(B.LanceError) as ei:
            c()
        assert ei.value.status == B.LANCE_ERR_WORKSPACE
    # the timing twin of the fused call checks the same things, and its repeat count, first
    prof = lambda repeats=1, x=16, ws=256, nbytes=1 << 30: B.lance_conv3x3_winograd_q8_profile(
        d, x, 16, 16, 16, None, 16, ws, nbytes, stream=0, repeats=repeats)
    for bad in (lambda: prof(0), lambda: prof(-3), lambda: prof(B.LANCE_PROFILE_MAX_REPEATS + 1),
                lambda: prof(x=None)):
        with pytest.raises(B.LanceError) as ei:
            bad()
        assert ei.value.status == B.LANCE_ERR_INVALID_ARG
    with pytest.raises(B.LanceError) as ei:
        prof(nbytes=s.conv_workspace_bytes - 1)
    assert ei.value.status == B.LANCE_ERR_WORKSPACE
    # static ranges demanded but not supplied
    ds = B.make_desc(1, 4, 8, 8, 4, flags=B.LANCE_INPUT_RANGE_STATIC)
    with pytest.raises(B.LanceError) as ei:
        B.lance_conv3x3_winograd_q8(ds, 16, 16, 16, 16, None, 16, 256, 1 << 30, stream=0)
    assert ei.value.status == B.LANCE_ERR_INVALID_ARG


@pytest.mark.parametrize("C", [3, 16, 48, 64, 130])
def test_code_offset_is_a_bijection_and_matches_documented_layout(C):
    d = B.make_desc(1, C, 8, 8, 4)
    s = B.lance_query_sizes(d)
    rows = 5
    seen = set()
    Q = s.CB // 4
    for e in (0, s.E - 1):
        for row in (0, rows - 1):
            for c in range(s.Cp):
                off = B.lance_code_offset(d, rows, e, row, c)
                b, r = divmod(c, s.CB)
                assert off == ((e * s.NB + b) * rows + row) * s.CB + 4 * (r % Q) + r // Q
                seen.add(off)
    assert len(seen) == 2 * 2 * s.Cp
    assert B.lance_code_offset(d, rows, s.E, 0, 0) == 2 ** 64 - 1
    assert B.lance_code_offset(d, rows, 0, rows, 0) == 2 ** 64 - 1


def test_alg1_literal_rejects_range_and_plan_flags():
    for flag in (B.LANCE_RANGE_PER_TENSOR, B.LANCE_INPUT_RANGE_STATIC, B.LANCE_PLAN_WIDE_TILES):
        d = B.make_desc(1, 4, 8, 8, 4, flags=flag)
        with pytest.raises(B.LanceError) as ei:
            B.lance_alg1_literal_f32(d, 16, 16, 16, stream=0)
        assert ei.value.status == B.LANCE_ERR_UNSUPPORTED


@pytest.mark.parametrize("C", [3, 48, 64, 130])
def test_code_offset_with_nhwc_keeps_the_channels_in_order(C):
    """LANCE_LAYOUT_NHWC: channel r of a block at byte r (documented in lance.h); sizes unchanged."""
    d = B.make_desc(1, C, 8, 8, 4, flags=B.LANCE_LAYOUT_NHWC)
    s, s0 = B.lance_query_sizes(d), B.lance_query_sizes(B.make_desc(1, C, 8, 8, 4))
    assert (s.Cp, s.CB, s.NB, s.uq_bytes, s.vq_bytes, s.y_bytes, s.conv_workspace_bytes) == \
           (s0.Cp, s0.CB, s0.NB, s0.uq_bytes, s0.vq_bytes, s0.y_bytes, s0.conv_workspace_bytes)
    rows = 3
    for e in (0, s.E - 1):
        for row in (0, rows - 1):
            for c in range(s.Cp):
                b, r = divmod(c, s.CB)
                assert B.lance_code_offset(d, rows, e, row, c) == ((e * s.NB + b) * rows + row) * s.CB + r


def test_codes_to_logical_follows_code_offset():
    """The numpy un-permutation used by the parity tests agrees with lance_code_offset."""
    C, rows = 130, 3
    d = B.make_desc(1, C, 8, 8, rows)
    s = B.lance_query_sizes(d)
    flat = np.arange(s.E * s.NB * rows * s.CB, dtype=np.int64)
    a = flat.reshape(s.E, s.NB, rows, s.CB)
    Q = s.CB // 4
    r = np.arange(s.CB)
    logical = a[:, :, :, 4 * (r % Q) + r // Q].transpose(0, 2, 1, 3).reshape(s.E, rows, s.Cp)
    for e, row, c in [(0, 0, 0), (3, 2, 129), (15, 1, 77), (7, 0, 191)]:
        assert logical[e, row, c] == B.lance_code_offset(d, rows, e, row, c)


def test_packed_code_layout_is_a_bijection_onto_nibbles():
    """LANCE_CODES_PACKED4: half the bytes, every (row, channel) owns one nibble of its own."""
    d8 = B.make_desc(1, 130, 8, 8, 5, bits=4)
    dp = B.make_desc(1, 130, 8, 8, 5, bits=4, flags=B.LANCE_CODES_PACKED4)
    s8, sp = B.lance_query_sizes(d8), B.lance_query_sizes(dp)
    assert (sp.Cp, sp.CB, sp.NB) == (s8.Cp, s8.CB, s8.NB) == (192, 64, 3)
    assert sp.uq_bytes * 2 == s8.uq_bytes and sp.vq_bytes * 2 == s8.vq_bytes
    assert sp.conv_workspace_bytes < s8.conv_workspace_bytes
    seen = set()
    rows = 5
    for e in (0, 7, 15):
        for row in range(rows):
            for c in range(sp.Cp):
                off, sh = B.lance_code_offset(dp, rows, e, row, c), B.lance_code_shift(dp, c)
                assert sh in (0, 4) and off < sp.uq_bytes
                # the byte is the unpacked byte position modulo 32 inside the same (e, block, row)
                off8 = B.lance_code_offset(d8, rows, e, row, c)
                assert off // 32 == off8 // 64 and off % 32 == off8 % 32 and sh == 4 * ((off8 % 64) // 32)
                seen.add((off, sh))
    assert len(seen) == 3 * rows * sp.Cp
    assert B.lance_code_shift(d8, 3) == 0 and B.lance_code_shift(dp, sp.Cp) == -1


def test_addresses_of_int_subclasses_pass_through():
    class Address(int):
        pass
    assert B._ptr(Address(4096)) == 4096 and B._stream(Address(4096)) == 4096
    assert B._ptr(None) is None and B._ptr(4096) == 4096 and B._stream(0) == 0
