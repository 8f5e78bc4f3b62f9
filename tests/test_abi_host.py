"""Host-only checks of the C-ABI library: it loads, exports every declared symbol, and
rejects bad arguments before anything is launched (so these run without a GPU)."""
import ctypes as C
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
B = pytest.importorskip("paper_1805_08691_amd.binding")


def test_every_declared_symbol_is_exported():
    hdr = open(os.path.join(ROOT, "include", "q8conv.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(q8_[a-z0-9_]+)\s*\(", hdr))
    assert len(declared) >= 16
    assert declared == set(B.EXPORTS)
    for name in declared:
        assert hasattr(B.lib, name), name


def test_strerror():
    assert B.lib.q8_strerror(0) == b"ok"
    for code in (-1, -2, -3, -4, -99):
        assert len(B.lib.q8_strerror(code)) > 3


def test_qfactor_and_extents():
    assert B.qfactor(0.0, 7) == 1.0
    assert B.qfactor(127.0, 7) == 1.0
    assert B.ConvDesc(1, 224, 224, 3, 64, 7, 7, 2, 2, 3, 3).Ho == 112
    assert B.ConvDesc(1, 19, 19, 512, 1024, 3, 3, 1, 1, 6, 6, 6, 6).Wo == 19
    assert B.ConvDesc(1, 2, 2, 16, 16, 3, 3).Ho == 0


def test_bad_arguments_are_rejected_on_the_host():
    fake = C.c_void_p(0x1000)      # never dereferenced: every call below fails validation first
    L = B.lib
    assert L.q8_calibrate_maxabs(fake, 10, None, None) == -1
    assert L.q8_calibrate_maxabs(None, 10, fake, None) == -1
    assert L.q8_calibrate_maxabs(C.c_void_p(0x1002), 10, fake, None) == -3
    assert L.q8_calibrate_maxabs(None, 0, fake, None) == 0            # empty tensor: no-op
    assert L.q8_quantize(fake, 10, 0.0, 7, fake, None) == -1          # q <= 0
    assert L.q8_quantize_image(fake, 1, 8, 8, 3, 0.5, 7, fake, 8, 9, 1, 0, None) == -1   # frame too low
    assert L.q8_quantize_image(fake, 1, 8, 8, 5, 0.5, 7, fake, 8, 8, 0, 0, None) == -1   # C > 4
    assert L.q8_quantize_image(fake, 1, 8, 8, 3, 0.5, 7, C.c_void_p(0x1002), 8, 8, 0, 0, None) == -3
    assert L.q8_quantize_image(fake, 0, 8, 8, 3, 0.5, 7, fake, 8, 8, 0, 0, None) == 0    # empty batch
    assert L.q8_quantize(fake, 10, float("nan"), 7, fake, None) == -1
    assert L.q8_quantize(fake, 10, float("inf"), 7, fake, None) == -1
    assert L.q8_quantize(fake, 10, 1.0, 8, fake, None) == -1          # p outside 1..7
    assert L.q8_quantize(fake, 10, 1.0, 0, fake, None) == -1
    assert L.q8_quantize(None, 10, 1.0, 7, fake, None) == -1
    assert L.q8_quantize(None, 0, 1.0, 7, None, None) == 0
    assert L.q8_quantize_pad_channels(fake, 10, 5, 4, 1.0, 7, fake, None) == -1
    assert L.q8_quantize_bias(fake, 4, -1.0, 1.0, fake, None) == -1
    assert L.q8_dequantize(fake, 4, 0.0, fake, None) == -1
    assert L.q8_dequantize(None, 4, 1.0, fake, None) == -1
    assert L.q8_fold_bn(fake, None, fake, fake, fake, fake, 1e-5, -1, 4, fake, fake, None) == -1
    assert L.q8_fold_bn(fake, None, None, fake, fake, fake, 1e-5, 2, 4, fake, fake, None) == -1
    assert L.q8_fold_bn(fake, None, fake, fake, fake, fake, 1e-5, 0, 4, fake, fake, None) == 0

    d = B.ConvDesc(1, 8, 8, 16, 16, 3, 3, pad_h=1, pad_w=1)
    ok = (fake, fake, None, 1.0, 1.0, 1.0, None, 0.0, fake, None, None, 0, None)   # no workspace
    assert L.q8_conv_int8(None, *ok) == -1
    bad = B.ConvDesc(1, 8, 8, 16, 16, 3, 3, stride_h=0)
    assert L.q8_conv_int8(C.byref(bad), *ok) == -1
    odd = B.ConvDesc(1, 8, 8, 24, 16, 3, 3)          # C neither <= 4 nor a multiple of 16
    assert L.q8_conv_int8(C.byref(odd), *ok) == -2
    assert B.packed_weight_bytes(odd) == 0
    assert L.q8_conv_int8(C.byref(d), fake, fake, None, 0.0, 1.0, 1.0, None, 0.0, fake, None,
                          None, 0, None) == -1
    assert L.q8_conv_int8(C.byref(d), None, fake, None, 1.0, 1.0, 1.0, None, 0.0, fake, None,
                          None, 0, None) == -1
    assert L.q8_conv_int8(C.byref(d), C.c_void_p(0x1004), fake, None, 1.0, 1.0, 1.0, None, 0.0,
                          fake, None, None, 0, None) == -3     # activations not 16-byte aligned
    narrow = B.ConvDesc(1, 8, 8, 16, 16, 3, 3, out_c_stride=8)
    assert L.q8_conv_int8(C.byref(narrow), *ok) == -1  # K does not fit the output stride
    resq = (fake, fake, None, 1.0, 1.0, 1.0, fake, 0.0, fake, None, None, 0, None)
    assert L.q8_conv_int8(C.byref(d), *resq) == -1     # residual with q_res <= 0
    empty = B.ConvDesc(0, 8, 8, 16, 16, 3, 3)
    assert L.q8_conv_int8(C.byref(empty), None, None, None, 1.0, 1.0, 1.0, None, 0.0, None, None,
                          None, 0, None) == 0          # empty batch: nothing to do
    # split reduction: the workspace is checked on the host
    deep = B.ConvDesc(2, 7, 7, 512, 512, 3, 3, pad_h=1, pad_w=1)
    names = [L.q8_conv_variant_name(v).decode() for v in range(L.q8_conv_num_variants())]
    sv = next(v for v, nm in enumerate(names) if "split" in nm)
    need = L.q8_conv_workspace_bytes_variant(C.byref(deep), sv, 4)
    assert need > 4 * 98 * 49 // 128 * 4            # counters plus four partial tiles per tile
    assert L.q8_conv_workspace_bytes_variant(C.byref(deep), sv, 1) == 0     # nothing to share
    assert L.q8_conv_workspace_bytes_variant(C.byref(deep), 0, 4) == 0      # not a split build
    assert L.q8_conv_workspace_bytes_variant(C.byref(odd), sv, 4) == 0
    assert L.q8_conv_workspace_bytes(C.byref(deep)) <= need
    sp = (fake, fake, None, 1.0, 1.0, 1.0, None, 0.0, fake, None, sv, 4)
    assert L.q8_conv_int8_variant(C.byref(deep), *sp, None, 0, None) == -1             # none given
    assert L.q8_conv_int8_variant(C.byref(deep), *sp, C.c_void_p(0x1010), need, None) == -3
    assert L.q8_conv_int8_variant(C.byref(deep), *sp, fake, need - 1, None) == -5      # too small
    assert L.q8_conv_int8_variant(C.byref(deep), *sp[:-1], 65, fake, need, None) == -1 # factor
    assert L.q8_conv_int8_variant(C.byref(deep), *sp[:-2], len(names), 2, fake, need, None) == -1
    # sizes beyond the kernels' 32-bit offsets are refused on the host, nothing is launched
    big_x = B.ConvDesc(4096, 512, 512, 64, 64, 3, 3, pad_h=1, pad_w=1)        # activations > 2 GiB
    assert L.q8_conv_int8(C.byref(big_x), *ok) == -2
    big_m = B.ConvDesc(40000, 256, 256, 16, 64, 1, 1)                          # N*Ho*Wo > 2^31
    assert L.q8_conv_int8(C.byref(big_m), *ok) == -2
    big_w = B.ConvDesc(1, 8, 8, 16384, 16384, 3, 3, pad_h=1, pad_w=1)          # filters > 2 GiB
    assert L.q8_conv_int8(C.byref(big_w), *ok) == -2
    # layer pairs: what the pair build cannot take is reported, not attempted
    p1 = B.ConvDesc(2, 14, 14, 64, 128, 3, 3, pad_h=1, pad_w=1, relu=1)
    p2_ok = B.ConvDesc(2, 14, 14, 128, 512, 1, 1)
    assert L.q8_conv_pair_supported(C.byref(p1), C.byref(p2_ok)) == 1
    for bad2 in (B.ConvDesc(2, 14, 14, 128, 4096, 1, 1),          # its filters do not fit in LDS
                 B.ConvDesc(2, 14, 14, 128, 192, 1, 1),           # K2 not a multiple of K1
                 B.ConvDesc(2, 14, 14, 128, 512, 3, 3, pad_h=1, pad_w=1),
                 B.ConvDesc(2, 7, 7, 128, 512, 1, 1),             # not the first layer's output
                 B.ConvDesc(2, 14, 14, 128, 512, 1, 1, stride_h=2, stride_w=2)):
        assert L.q8_conv_pair_supported(C.byref(p1), C.byref(bad2)) == 0
    assert L.q8_conv_pair_supported(C.byref(B.ConvDesc(2, 14, 14, 64, 96, 3, 3)), C.byref(p2_ok)) == 0
    pair_args = (fake, fake, None, 1.0, 1.0, 1.0)
    assert L.q8_conv_pair_int8(C.byref(p1), *pair_args, C.byref(B.ConvDesc(2, 14, 14, 128, 4096, 1, 1)),
                               fake, None, 1.0, 1.0, None, 0.0, fake, None) == -2
    assert L.q8_conv_pair_int8(C.byref(p1), *pair_args, C.byref(p2_ok), None, None, 1.0, 1.0, None, 0.0,
                               fake, None) == -1                     # no second filters
    assert L.q8_conv_pair_int8(C.byref(p1), *pair_args, C.byref(p2_ok), fake, None, 1.0, 0.0, None, 0.0,
                               fake, None) == -1                     # q_out <= 0
    # unsigned activation codes
    wide = B.ConvDesc(1, 8, 8, 16, 64, 3, 3, pad_h=1, pad_w=1, relu=1)
    u8 = (fake, fake, fake, fake, 1.0, 1.0, 1.0, None, 0.0, fake, None, None)
    assert L.q8_conv_u8(C.byref(d), 1, 1, 0, *u8) == -2          # K <= 32: not in the extended build
    norelu = B.ConvDesc(1, 8, 8, 16, 64, 3, 3, pad_h=1, pad_w=1, relu=0)
    assert L.q8_conv_u8(C.byref(norelu), 1, 1, 0, *u8) == -1     # unsigned output without ReLU
    assert L.q8_conv_u8(C.byref(wide), 1, 1, 1, *u8) == -1       # unsigned residual, none given
    assert L.q8_conv_u8(C.byref(wide), 1, 1, 0, fake, fake, None, fake, 1.0, 1.0, 1.0, None, 0.0,
                        fake, None, None) == -1                  # unsigned input needs bias_eff
    assert L.q8_conv_u8(C.byref(wide), 1, 1, 0, fake, fake, fake, None, 1.0, 1.0, 1.0, None, 0.0,
                        fake, None, None) == -1                  # padding needs the tap sums
    assert L.q8_u8_prepare(C.byref(wide), None, None, fake, fake, None) == -1
    assert L.q8_u8_prepare(C.byref(B.ConvDesc(1, 8, 8, 3, 64, 3, 3)), fake, None, fake, fake,
                           None) == -2
    assert L.q8_quantize_u8(fake, 4, 0.0, fake, None) == -1
    assert L.q8_dequantize_u8(None, 4, 1.0, fake, None) == -1
    assert L.q8_dequantize_u8(None, 0, 1.0, None, None) == 0
    # per-channel weight factors
    pc = (fake, fake, None, fake, 1.0, None, 0.0, fake, None, None)
    assert L.q8_conv_int8_per_channel(C.byref(wide), fake, fake, None, None, 1.0, None, 0.0, fake,
                                      None, None) == -1          # no scale vector
    assert L.q8_conv_int8_per_channel(C.byref(d), *pc) == -2     # K <= 32: not in the extended build
    assert L.q8_conv_int8_per_channel(C.byref(wide), fake, fake, None, C.c_void_p(0x1004), 1.0,
                                      None, 0.0, fake, None, None) == -3
    # real-valued (fp32) output
    ro = (fake, fake, None, 1.0, 1.0, None, 0.0)
    assert L.q8_conv_int8_real_output(C.byref(d), *ro, None, None) == -1        # no output
    assert L.q8_conv_int8_real_output(C.byref(d), *ro, C.c_void_p(0x1002), None) == -3
    assert L.q8_conv_int8_real_output(C.byref(d), fake, fake, None, 1.0, 0.0, None, 0.0, fake,
                                      None) == -1                              # q_w <= 0
    assert L.q8_conv_int8_real_output(C.byref(d), fake, fake, None, 1.0, 1.0, fake, 0.0, fake,
                                      None) == -1                              # residual, q_res <= 0
    assert L.q8_conv_int8_real_output(C.byref(empty), None, None, None, 1.0, 1.0, None, 0.0, None,
                                      None) == 0
    assert L.q8_probe_mfma_i8(0, 10, fake, None) == -1
    assert L.q8_probe_mfma_i8(4, 10, None, None) == -1
    assert L.q8_quantize_weights_per_channel(fake, 4, 16, 9, fake, fake, None) == -1   # p
    assert L.q8_quantize_weights_per_channel(None, 4, 16, 7, fake, fake, None) == -1
    assert L.q8_quantize_weights_per_channel(None, 0, 16, 7, None, None, None) == 0
    assert L.q8_quantize_bias_per_channel(fake, 4, 0.0, fake, fake, None) == -1
    assert L.q8_requant_scales(1.0, fake, 4, 0.0, fake, None) == -1
    assert B.packed_weight_bytes(d) == 16 * 3 * 3 * 16
    assert B.packed_weight_bytes(B.ConvDesc(1, 8, 8, 3, 64, 7, 7)) == 64 * 7 * 2 * 16
    assert L.q8_maxpool_i8(fake, 1, 8, 8, 4, 3, 3, 2, 3, 4, 4, fake, None) == -1   # pad >= window


# ------------------------------------------------------------------ layer lists (host side)
def _chain_layers(n_img=16, bad=None):
    """A bottleneck block (1x1 256->64, 3x3 64->64, 1x1 64->256 + residual) as a layer list on
    made-up, distinct, aligned device addresses (nothing is dereferenced on the host)."""
    base = 0x7F0000000000
    t = {"x": base, "a": base + (1 << 28), "b": base + (2 << 28), "y": base + (3 << 28)}
    geo = [(256, 64, 1, "x", "a", None), (64, 64, 3, "a", "b", None), (64, 256, 1, "b", "y", "x")]
    arr = (B.ChainLayer * 3)()
    for i, (Cc, K, R, src, dst, res) in enumerate(geo):
        a = arr[i]
        a.d = B.ConvDesc(n_img, 28, 28, Cc, K, R, R, 1, 1, R // 2, R // 2, relu=1)
        a.z_x, a.z_y = t[src], t[dst]
        a.z_w_packed, a.bias_i32 = 0x100000 + i * 0x100000, 0x10000 + i * 0x1000
        a.q_x = a.q_w = a.q_out = a.q_res = 0.5
        a.residual = t[res] if res else None
        a.src_layer = i - 1 if i else -1
        a.res_layer = -1
        a.variant = -1
    if bad:
        bad(arr)
    return arr


def test_fused_head_and_dequantized_output_host_checks():
    """q8_conv_image_f32_supported and the argument checks of q8_conv_image_f32_int8 /
    q8_conv_int8_dequantized run on the host: nothing is launched here."""
    L = B.lib
    fake = C.c_void_p(0x1000)
    # ResNet-50's first layer over its zero frame, with and without the max-pool
    d = B.ConvDesc(32, 230, 230, 3, 64, 7, 7, 2, 2, 0, 0, 1, 1, relu=1, in_c_stride=4)
    assert B.conv_image_f32_supported(d, 224, 224, 3, 3, 3, 0)
    assert B.conv_image_f32_supported(d, 224, 224, 3, 3, 3, 1)
    assert not B.conv_image_f32_supported(d, 228, 224, 3, 3, 3, 1)      # does not fit the frame
    assert not B.conv_image_f32_supported(d, 224, 224, 4, 3, 3, 1)      # C != d.C
    # outside the family: 3 filter columns; rows of more than 128 output pixels; K > 64;
    # the pool needs a vertical stride of 2
    assert not B.conv_image_f32_supported(
        B.ConvDesc(1, 301, 301, 3, 32, 3, 3, 2, 2, 0, 0, 1, 1, in_c_stride=4), 299, 299, 3, 1, 1, 0)
    assert not B.conv_image_f32_supported(
        B.ConvDesc(1, 200, 240, 3, 64, 7, 7, 1, 1, 0, 0, 1, 1, in_c_stride=4), 194, 234, 3, 3, 3, 0)
    assert not B.conv_image_f32_supported(
        B.ConvDesc(1, 70, 70, 3, 96, 7, 7, 2, 2, 0, 0, 1, 1, in_c_stride=4), 64, 64, 3, 3, 3, 0)
    d1 = B.ConvDesc(1, 70, 70, 3, 64, 7, 7, 1, 2, 0, 0, 1, 1, in_c_stride=4)
    assert B.conv_image_f32_supported(d1, 64, 64, 3, 3, 3, 0)
    assert not B.conv_image_f32_supported(d1, 64, 64, 3, 3, 3, 1)
    args = lambda dd, r, H, W, Cc, top, left, q, p, pool, y: L.q8_conv_image_f32_int8(
        C.byref(dd), r, H, W, Cc, top, left, q, p, fake, None, 0.01, 0.5, pool, y, None)
    assert args(d, fake, 224, 224, 3, 3, 3, 0.02, 7, 2, fake) == -1       # pool flag
    assert args(d, fake, 224, 224, 3, 3, 3, 0.02, 8, 1, fake) == -1       # p out of range
    assert args(d, fake, 230, 224, 3, 3, 3, 0.02, 7, 1, fake) == -1       # image beyond the frame
    assert args(d, None, 224, 224, 3, 3, 3, 0.02, 7, 1, fake) == -1       # no image
    assert args(d, C.c_void_p(0x1002), 224, 224, 3, 3, 3, 0.02, 7, 1, fake) == -3   # misaligned
    assert args(d, fake, 224, 224, 3, 3, 3, -1.0, 7, 1, fake) == -1       # factor
    d3 = B.ConvDesc(1, 30, 30, 3, 64, 3, 3, 1, 1, 0, 0, 1, 1, in_c_stride=4)
    assert args(d3, fake, 28, 28, 3, 1, 1, 0.02, 7, 0, fake) == -2        # not in the family
    dd = B.ConvDesc(2, 7, 7, 512, 2048, 1, 1)
    deq = lambda r_y: L.q8_conv_int8_dequantized(C.byref(dd), fake, fake, None, 0.02, 0.01, 0.5, None,
                                                 0.0, fake, r_y, None)
    assert deq(None) == -1
    assert deq(C.c_void_p(0x1002)) == -3


def test_chain_plan_accepts_a_block_and_sizes_its_workspace():
    arr = _chain_layers()
    n = B.lib.q8_conv_chain_plan_bytes(arr, 3)
    assert n > 0 and n % 256 == 0
    buf = C.create_string_buffer(n)
    assert B.lib.q8_conv_chain_plan(arr, 3, buf, n) == 0
    assert B.lib.q8_conv_chain_plan(arr, 3, buf, n - 1) == -1          # plan buffer too small
    ws = B.lib.q8_conv_chain_workspace_bytes(buf)
    # status line + per XCD a queue head line and one counter per pixel tile of every layer
    assert ws >= 4 * (32 + 8 * 32) and ws % 128 == 0
    fake = C.c_void_p(0x7F1000000000)
    assert B.lib.q8_conv_chain_int8(buf, fake, fake, ws - 4, None) == -5    # workspace too small
    assert B.lib.q8_conv_chain_int8(buf, C.c_void_p(0x7F1000000010), fake, ws, None) == -3
    assert B.lib.q8_conv_chain_int8(buf, None, fake, ws, None) == -1
    assert B.lib.q8_conv_chain_workspace_bytes(C.create_string_buffer(256)) == 0   # not a plan
    assert B.lib.q8_conv_chain_int8(C.create_string_buffer(256), fake, fake, 1 << 20, None) == -1
    assert B.lib.q8_conv_chain_int8_static(C.create_string_buffer(256), fake, None) == -1
    assert B.lib.q8_conv_chain_static_workspace_limit() == 1 << 20
    assert B.lib.q8_strerror(-5) != B.lib.q8_strerror(-99)


def test_chain_plan_rejects_inconsistent_lists():
    def plan_rc(bad):
        arr = _chain_layers(bad=bad)
        return B.lib.q8_conv_chain_plan_bytes(arr, 3)

    def forward_ref(arr): arr[1].src_layer = 2                     # reads a later layer
    def wrong_src(arr): arr[2].src_layer = 0                       # z_x is not that layer's z_y
    def alias(arr): arr[1].z_y = arr[0].z_y                        # a tensor written twice
    def clobber_input(arr): arr[2].z_y = arr[0].z_x                # writes what the list reads
    def odd_c(arr): arr[0].d.C = 48                                # not a chain geometry
    def sliced(arr): arr[2].d.out_c_off = 16
    def batches(arr): arr[1].d.N = 3
    def res_without_tensor(arr): arr[1].res_layer = 0
    for bad in (forward_ref, wrong_src, alias, clobber_input, odd_c, sliced, batches,
                res_without_tensor):
        assert plan_rc(bad) == 0, bad.__name__
    assert B.lib.q8_conv_chain_plan_bytes(None, 3) == 0
    assert B.lib.q8_conv_chain_plan_bytes(_chain_layers(), 0) == 0
    assert B.lib.q8_conv_chain_supported(C.byref(B.ConvDesc(8, 14, 14, 256, 256, 3, 3, 1, 1, 1, 1))) == 1
    assert B.lib.q8_conv_chain_supported(C.byref(B.ConvDesc(8, 14, 14, 48, 256, 3, 3, 1, 1, 1, 1))) == 0
    assert B.lib.q8_conv_chain_supported(C.byref(B.ConvDesc(8, 14, 14, 64, 16, 1, 1))) == 0


def test_chain_plan_splits_the_batch_over_eight_queues():
    import struct
    for n_img, want in ((16, [2] * 8), (13, [2, 2, 2, 2, 2, 1, 1, 1]), (3, [1, 1, 1, 0, 0, 0, 0, 0])):
        arr = _chain_layers(n_img)
        n = B.lib.q8_conv_chain_plan_bytes(arr, 3)
        buf = C.create_string_buffer(n)
        assert B.lib.q8_conv_chain_plan(arr, 3, buf, n) == 0
        hd = struct.unpack_from("<I7i8i", bytes(buf), 0)
        assert hd[1] == 3
        n_items = hd[8:16]
        # queue entries of an XCD are proportional to its images (28x28 = 784 pixels each)
        per_image = [i // w if w else 0 for i, w in zip(n_items, want)]
        assert [bool(i) for i in n_items] == [bool(w) for w in want]
        assert len({p for p, w in zip(per_image, want) if w == want[0]}) == 1


def test_run_ops_takes_empty_batches_as_the_single_calls_do():
    d = B.ConvDesc(0, 9, 9, 64, 64, 1, 1)
    fake, L = C.c_void_p(0x1000), B.lib
    assert L.q8_conv_int8_dequantized(C.byref(d), None, fake, None, 0.5, 0.5, 0.5, None, 0.0, None, None, None) == 0
    ops = (B.Op * 1)()
    o = ops[0]
    o.kind, o.flags, o.d, o.w, o.q_x, o.q_w, o.q_out = B.OP_CONV, B.OPF_DEQUANT, d, 0x1000, 0.5, 0.5, 0.5
    streams = (C.c_void_p * 1)(None)
    assert L.q8_run_ops(ops, 1, streams, 1) == 0
    o.d.N = 1                                  # not empty: the output is needed
    assert L.q8_run_ops(ops, 1, streams, 1) == -1


def test_layer_calls_check_their_arguments():
    """The extension module's checks are the binding's: device tensors, a descriptor, real factors."""
    import torch
    d = B.ConvDesc(1, 4, 4, 16, 16, 1, 1)
    x = torch.zeros((1, 4, 4, 16), dtype=torch.int8)
    calls = [lambda t, desc=d, q=1.0: B.conv_int8(desc, t, t, t, q, 1.0, 1.0, out=x),
             lambda t, desc=d, q=1.0: B.conv_u8(desc, 1, 1, 0, t, t, t, None, q, 1.0, 1.0, out=x),
             lambda t, desc=d, q=1.0: B.conv_int8_per_channel(desc, t, t, t, t, q, out=x),
             lambda t, desc=d, q=1.0: B.conv_int8_real_output(desc, t, t, t, q, 1.0, out=x)]
    for call in calls:
        for t in (x, torch.nn.Parameter(x, requires_grad=False)):
            with pytest.raises(AssertionError):
                call(t)                                   # not on the device
        with pytest.raises(TypeError):
            call(None, desc="no descriptor")
        with pytest.raises(TypeError):
            call(None, q="no factor")
    with pytest.raises(AssertionError):
        B.conv_f32_observed(d, x.float(), None, None, None, None, None, None)
    for f in (B._q8call.conv_int8, B._q8call.conv_u8, B._q8call.conv_per_channel, B._q8call.conv_real, B._q8call.conv_f32):
        with pytest.raises(TypeError):
            f(d)


def test_layer_calls_raise_for_tensors_without_storage():
    """Under vmap a tensor is of exactly torch.Tensor's type, on the device and contiguous, and has no
    address: an exception, as from the binding's own check, and the process goes on."""
    import torch
    from torch._subclasses.fake_tensor import FakeTensorMode
    d = B.ConvDesc(1, 4, 4, 16, 16, 1, 1)
    calls = [lambda t: B.conv_int8(d, t, t, None, 1.0, 1.0, 1.0),
             lambda t: B.conv_u8(d, 1, 1, 0, t, t, None, None, 1.0, 1.0, 1.0),
             lambda t: B.conv_int8_per_channel(d, t, t, None, None, 1.0),
             lambda t: B.conv_int8_real_output(d, t, t, None, 1.0, 1.0),
             lambda t: B.conv_f32_observed(d, t.float(), None, None, None, None, None, None)]
    seen = []

    def body(t, call):
        assert type(t) is torch.Tensor and t.is_cuda and t.is_contiguous()
        with pytest.raises(RuntimeError, match="storage"):
            call(t)
        seen.append(call)
        return t
    with FakeTensorMode():                      # (device tensors without a device)
        batch = torch.empty((3, 1, 4, 4, 16), dtype=torch.int8, device="cuda")
        for call in calls:
            torch.vmap(lambda t: body(t, call))(batch)
    assert len(seen) == 5


@pytest.fixture
def passes():
    """Max-abs, Eq. Q and Eq. D of the binding on host memory; the list of what reaches the library."""
    import torch
    seen = []

    def ptr(t, dtype=None):                     # the checks of the binding, without a device
        if t is None:
            return None
        assert t.is_contiguous() and t.dtype is dtype
        return t.data_ptr()
    vp, sz = C.c_void_p, C.c_size_t
    recorders = [C.CFUNCTYPE(C.c_int, *types)(lambda *a: seen.append(a) or 0) for types in (
        (vp, sz, vp, vp), (vp, sz, C.c_float, C.c_int, vp, vp), (vp, sz, C.c_float, vp, vp))]
    types = (B.ConvDesc, torch.int8, torch.int32, torch.float32, torch.uint8)
    layers = [C.cast(f, vp).value for f in (B.lib.q8_conv_int8, B.lib.q8_conv_u8, B.lib.q8_conv_int8_per_channel,
                                            B.lib.q8_conv_int8_real_output, B.lib.q8_conv_f32_observed_spread)]
    bind = lambda *f: B._q8call.bind(*f[:3], *types, *layers, *(C.cast(p, vp).value for p in f[3:]))
    bind(ptr, lambda: 0, lambda device: 0, *recorders)
    yield seen
    bind(B._ptr, B._device, B._raw_stream, B.lib.q8_calibrate_maxabs, B.lib.q8_quantize, B.lib.q8_dequantize)


def test_passes_need_the_tensor_that_they_read(passes):
    """None has no elements to count: refused, and not taken for a tensor of length 0."""
    import torch
    z, r, slot = torch.zeros(6, dtype=torch.int8), torch.zeros(6), torch.zeros(1)
    for call in (lambda t: B.calibrate_maxabs(t, slot), lambda t: B.quantize(t, 0.5, 7, out=z),
                 lambda t: B.dequantize(t, 0.5, out=r)):
        with pytest.raises(AttributeError):
            call(None)
    assert not passes
    B.calibrate_maxabs(r, slot), B.quantize(r, 0.5, 7, out=z), B.dequantize(z, 0.25, out=r)
    a, b, c = r.data_ptr(), z.data_ptr(), slot.data_ptr()
    assert passes == [(a, 6, c, None), (a, 6, 0.5, 7, b, None), (b, 6, 0.25, a, None)]
    with pytest.raises(AssertionError):
        B.quantize(z, 0.5, 7, out=z)
    B.calibrate_maxabs(r[:0], slot)                # empty: the library's own answer
    assert passes[3][1:3] == (0, c)


def test_passes_take_numbers_as_ctypes_does(passes):
    import numpy as np
    import torch
    r, z = torch.zeros(4), torch.zeros(4, dtype=torch.int8)
    for p in (7, True, np.int64(7), np.uint8(3), torch.tensor(5), 2**32 + 6, C.c_int(4)):
        B.quantize(r, 0.5, p, out=z)
    assert [a[3] for a in passes] == [7, 1, 7, 3, 5, 6, 4]
    for p in (7.0, np.float32(7), None, "7", C.c_float(7)):
        with pytest.raises(TypeError):
            B.quantize(r, 0.5, p, out=z)
    passes.clear()
    for q in (0.5, 2, np.float32(0.5), np.int64(3), torch.tensor(0.25), C.c_float(0.125)):
        B.quantize(r, q, 7, out=z), B.dequantize(z, q, out=r)
    assert [a[2] for a in passes] == [0.5, 0.5, 2, 2, 0.5, 0.5, 3, 3, 0.25, 0.25, 0.125, 0.125]
    for q in (None, "0.5", 1j):
        with pytest.raises(TypeError):
            B.dequantize(z, q, out=r)


def test_layer_calls_take_flags_as_int_does():
    d = B.ConvDesc(1, 4, 4, 16, 16, 1, 1)
    for bad in (None, "no number", []):
        with pytest.raises((TypeError, ValueError)):
            B._q8call.conv_u8(d, bad, 0, 0, *[None] * 4, 1.0, 1.0, 1.0, None, 0.0, None, None)


def test_a_long_slot_is_one_maximum_unless_copies_are_asked_for(monkeypatch):
    import torch
    seen = []
    monkeypatch.setattr(B._q8call, "conv_f32", lambda *a: seen.append(a[-1]) or 0)
    slot = lambda n: torch.empty(n, device="meta")
    for a, b in ((1, 1), (33, 1), (None, 512), (40, 40), (0, 1)):
        B.conv_f32_observed(*[None] * 6, *(None if n is None else slot(n) for n in (a, b)))
    assert seen == [1] * 5
    B.conv_f32_observed(*[None] * 6, slot(33), slot(64), 2)
    assert seen[5:] == [2]
    with pytest.raises(AssertionError):
        B.conv_f32_observed(*[None] * 6, slot(33), slot(32), 2)


def test_fp32_builds_on_lds_leave_wide_paddings_alone():
    """Their descriptor starts pad_h rows and pad_w pixels in front of the image: a padding that 32 bits
    do not hold goes to the register-fed builds, by the columns as by the rows."""
    name = lambda **kw: B.conv_f32_variant(B.ConvDesc(1, 1, 8, 1024, 16, 1, 1, **kw))
    assert name().startswith("conv_f32_lds_kernel")
    assert name(pad_w=1000).startswith("conv_f32_lds_kernel")
    span = 2 * 8 * 4096 + 2 * 9 * 4096      # two images, and two rows of the map and a tap
    fits = (2**31 - 1 - span) // (2 * 4096)
    assert name(pad_w=fits).startswith("conv_f32_lds_kernel")
    for pad in (fits + 1, 2**19 - 1, 2**19, 600000, 2**20):      # 2^19 pixels of 4 KB: the shift's sign
        assert name(pad_w=pad).startswith("conv_f32_mfma_kernel"), pad
    assert name(pad_h=2**15).startswith(("conv_f32_mfma_kernel", "conv_f32_any_kernel"))


def _group_variant(d, n=2, flags=0, residual=False, out_cs=0):
    """Name of the launch that n such layers of a group get (addresses stand in, nothing is launched)."""
    ops = (B.Op * n)()
    for i, o in enumerate(ops):
        o.kind, o.group, o.d, o.flags, o.q_x, o.q_w, o.q_out, o.q_res = B.OP_CONV, 1, d, flags, 1.0, 1.0, 1.0, 1.0
        o.d.out_c_stride = out_cs
        o.x, o.w, o.y, o.y_f32 = (1 << 20) * (4 * i + 1), (1 << 20) * (4 * i + 2), (1 << 20) * (4 * i + 3), 1 << 30
        o.residual = (1 << 20) * (4 * i + 4) if residual else None
    return B.lib.q8_group_variant(ops, n).decode()


@pytest.mark.parametrize("C_, K, pad", [(32, 16, 1), (32, 32, 0), (64, 16, 0)])
def test_layers_that_the_3x3_blocks_do_not_take_keep_the_latency_family(C_, K, pad):
    """The sizes choose the block-tiled kernel, the residual, the real output or the odd output stride does
    not go there: such a layer gets what it would get if there were no such kernel."""
    d = B.ConvDesc(43, 28, 28, C_, K, 3, 3, pad_h=pad, pad_w=pad)
    assert B.conv_variant(d) == "conv_i8_p3b_kernel"
    for kw in (dict(residual=True), dict(flags=B.OPF_REAL), dict(flags=B.OPF_DEQUANT), dict(out_cs=K + 4)):
        assert _group_variant(d, **kw).startswith("conv_i8_direct_kernel"), kw


@pytest.mark.parametrize("N, H, W, C_, K, pad, blocks", [
    # maps that leave the blocks empty: the general kernel or the latency family
    (8000, 5, 5, 64, 64, 0, False), (1320, 5, 5, 32, 16, 0, False), (4082, 7, 7, 32, 32, 0, False),
    (2470, 9, 9, 64, 64, 0, False), (2470, 9, 9, 64, 48, 1, False), (1184, 13, 13, 32, 64, 0, False),
    (8, 5000, 1, 32, 64, 1, False),
    # maps that fill them (1 row of 16 columns more than a block, too), and below the first size
    (693, 17, 17, 32, 64, 0, True), (1184, 13, 13, 32, 32, 1, True), (256, 28, 28, 64, 64, 1, True),
    (9, 150, 150, 64, 64, 0, True), (2, 8192, 16, 64, 64, 1, True), (32767, 1, 1, 64, 64, 1, False)])
def test_3x3_blocks_are_chosen_by_how_full_they_are(N, H, W, C_, K, pad, blocks):
    d = B.ConvDesc(N, H, W, C_, K, 3, 3, pad_h=pad, pad_w=pad)
    assert (B.conv_variant(d) == "conv_i8_p3b_kernel") == blocks


@pytest.mark.parametrize("pixels, C_, K, persistent", [
    # more channel tiles than places, and few pixel tiles to share: the general kernel
    (196, 128, 16384, False), (196, 64, 16384, False), (640, 128, 8192, False), (1140, 64, 16384, False),
    # channel tiles that leave a quarter or more of the places free
    (40900, 256, 2304, False), (40900, 256, 5120, False), (3140, 128, 2304, False),
    # full sets, at the first sizes and the largest
    (40833, 64, 64, True), (2560, 128, 1024, True), (1988, 128, 2304, True), (16324, 128, 16384, True),
    (61441, 128, 272, True), (128129, 256, 256, True), (40900, 256, 4096, True), (200704, 64, 256, True)])
def test_pointwise_family_is_chosen_by_its_places(pixels, C_, K, persistent):
    name = B.conv_variant(B.ConvDesc(1, 1, pixels, C_, K, 1, 1))
    assert name.startswith("conv_i8_pw_kernel") == persistent, name


def _block(mid=64, C=256, H=56, N=4, K2=256, **change):
    """Three ops of a bottleneck block at made-up addresses (nothing is launched)."""
    d = [B.ConvDesc(N, H, H, C, mid, 1, 1, relu=1), B.ConvDesc(N, H, H, mid, mid, 3, 3, 1, 1, 1, 1, relu=1),
         B.ConvDesc(N, H, H, mid, K2, 1, 1, relu=1)]
    at, ops = 1 << 40, (B.Op * 3)()
    for i, o in enumerate(ops):
        o.kind, o.d, o.q_x, o.q_w, o.q_out = B.OP_CONV, d[i], 0.1, 0.1, 0.1
        o.x = ops[i - 1].y if i else at
        o.w, o.bias, o.y = at + (1 << 33) * (i + 1), at + (1 << 33) * (i + 4), at + (1 << 33) * (i + 8)
    ops[2].residual, ops[2].q_res = at, 0.1
    for name, value in change.items():
        i, field = int(name[1]), name[3:]
        setattr(ops[i].d if hasattr(ops[i].d, field) else ops[i], field, value)
    return ops


def test_bottleneck_blocks_that_one_launch_takes():
    name = lambda ops: B.lib.q8_block_variant(ops).decode()
    taken = _block()
    assert name(taken).startswith("conv_i8_bneck_kernel<64,")
    assert name(_block(mid=128, C=512, H=28, K2=512)).startswith("conv_i8_bneck_kernel<128,")
    assert name(_block(mid=256, C=1024, H=14, N=32, K2=1024)).startswith("conv_i8_bneck_kernel<256,")
    assert name(_block(o2_residual=None)) == name(taken)
    single = [dict(o1_x=taken[0].x), dict(o2_x=taken[0].y), dict(o2_y=taken[0].x),           # other tensors, in place
              dict(o1_y=taken[0].y), dict(o2_y=taken[1].y + 64), dict(o0_y=taken[0].w), dict(o2_residual=taken[0].y),
              dict(o1_dil_h=2, o1_pad_h=2), dict(o1_pad_w=0), dict(o1_stride_h=2), dict(o2_pad_h=1), dict(o0_R=3, o0_pad_h=1),
              dict(o0_residual=taken[0].x, o0_q_res=0.1), dict(o2_out_c_stride=260), dict(o2_out_c_stride=264, o2_out_c_off=8),
              dict(o2_flags=B.OPF_DEQUANT, o2_y_f32=None), dict(o2_flags=B.OPF_DEQUANT, o2_y_f32=1 << 46),
              dict(o0_flags=B.OPF_REAL, o0_y_f32=1 << 46), dict(o0_flags=B.OPF_OUT_U8), dict(o1_kind=B.OP_POOL),
              dict(mid=32, C=64, K2=64), dict(mid=64, K2=96), dict(C=48), dict(H=86), dict(mid=256, C=1024, H=14, N=1, K2=1024)]
    for change in single:
        assert name(_block(**change)) == "single launches", change
    assert B.lib.q8_run_bottleneck(_block(o2_y=taken[0].x), 4, None) == -2
    assert B.lib.q8_run_bottleneck(taken, 0, None) == -2 and B.lib.q8_run_bottleneck(taken, 99, None) == -1
    assert B.lib.q8_run_bottleneck(None, 0, None) == -1 and name(None) == "single launches"


def test_blocks_that_pay_inside_a_network():
    """What a program asks before it marks a block: three layers by themselves as the library would launch them,
    but for wide blocks of few tiles, and the first one's share of a launch with others counted."""
    def pays(ops, *beside):
        return B.lib.q8_block_pays(ops, (B.Op * len(beside))(*beside), len(beside))

    def projection(ops, K, **fields):
        o = B.Op.from_buffer_copy(ops[0])
        d = ops[0].d
        o.d, o.w, o.bias, o.y = B.ConvDesc(d.N, d.H, d.W, d.C, K, 1, 1), 1 << 50, 1 << 51, 1 << 52
        for name, value in fields.items():
            setattr(o, name, value)
        return o
    one = lambda ops: B.lib.q8_block_variant(ops) != b"single launches"
    for kw, alone, beside in ((dict(), 1, 1), (dict(N=1), 1, 1), (dict(mid=128, C=256, H=20, K2=256, N=2), 1, 0),
                              (dict(mid=128, C=256, H=20, K2=256, N=1), 1, 0), (dict(mid=128, C=256, H=20, K2=256, N=12), 1, 1),
                              (dict(mid=256, C=256, H=14, K2=256, N=5), 1, 0), (dict(mid=256, C=512, H=14, K2=512, N=23), 1, 1)):
        ops = _block(**kw)
        assert one(ops) and pays(ops) == alone and pays(ops, projection(ops, ops[2].d.K)) == beside, kw
        # a layer that shares nothing with the first one's launch, and one that is none
        assert pays(ops, projection(ops, 64, kind=B.OP_POOL)) == alone
        assert pays(ops, projection(ops, ops[2].d.K, flags=B.OPF_REAL, y_f32=None)) == alone
    for N, wide in ((8, 0), (9, 0), (11, 1), (16, 1)):     # two tiles of 64 x 64 a CU in the last layer end at 2048 pixels
        ops = _block(mid=256, C=1024, H=14, K2=1024, N=N)
        assert one(ops) and pays(ops) == wide
    assert not pays(_block(o1_x=1 << 39)) and not pays(_block(mid=256, C=1024, H=14, N=1, K2=1024))
    ops = _block()
    assert B.lib.q8_block_pays(None, None, 0) == B.lib.q8_block_pays(ops, None, 1) == B.lib.q8_block_pays(ops, ops, 8) == 0
    assert B.lib.q8_block_pays(ops, None, -1) == 0


def _layer_and_maximum(n=1, kind=B.OP_MAXPOOL, **change):
    """n layers of the block-tiled 3x3 kernel, then the 2x2 maxima over their outputs, the last one's first, each pair
    on a stream index of its own, at made-up addresses (nothing is launched)."""
    ops, at = (B.Op * (2 * n))(), 1 << 40
    for i in range(n):
        o, m = ops[i], ops[2 * n - 1 - i]
        o.kind, o.d, o.stream, o.q_x, o.q_w, o.q_out = B.OP_CONV, B.ConvDesc(2, 149, 163, 64, 64, 3, 3, 1, 1, 1, 1, relu=1), i, 0.1, 0.1, 0.1
        o.x, o.w, o.bias, o.y = (at + (1 << 33) * (5 * i + j) for j in range(4))
        m.kind, m.stream, m.x, m.y, m.q_x, m.q_out = kind, i, o.y, at + (1 << 33) * (5 * i + 4), 0.1, 0.1
        m.d.N, m.H, m.W, m.C, m.R, m.S, m.stride, m.Ho, m.Wo, m.d.out_c_stride = 2, 149, 163, 64, 2, 2, 2, 75, 82, 64
    for name, value in change.items():
        o, field = ops[int(name[1])], name[3:]
        setattr(o if hasattr(o, field) else o.d, field, value)
    return ops


def test_maxima_that_join_their_layer():
    def joined(ops, *handles, first=0):
        return B.lib.q8_joined_op(ops, len(ops), (C.c_void_p * len(handles))(*handles), len(handles), first)
    assert B.conv_variant(_layer_and_maximum()[0].d) == "conv_i8_p3b_kernel"
    for kind in (B.OP_MAXPOOL, B.OP_POOL):
        assert joined(_layer_and_maximum(kind=kind), 64) == 1
        assert joined(_layer_and_maximum(kind=kind, o1_Ho=74, o1_Wo=81), 64) == 1
        for change in (dict(o1_R=3), dict(o1_S=1), dict(o1_stride=1), dict(o1_pad=1), dict(o1_Ho=76), dict(o1_C=48), dict(o1_H=148),
                       dict(o1_x=1 << 40), dict(o1_y=1 << 40), dict(o1_y=(1 << 40) + (1 << 33)), dict(o1_y=None),
                       dict(o1_y=(1 << 40) + (3 << 33) + 1024), dict(o1_y=(1 << 45) + 8), dict(o0_out_c_stride=128),
                       dict(o0_out_c_stride=128, o0_out_c_off=64), dict(o0_flags=B.OPF_OUT_U8),
                       dict(o0_flags=B.OPF_DEQUANT, o0_y_f32=1 << 46), dict(o0_flags=B.OPF_REAL, o0_y_f32=1 << 46),
                       dict(o0_residual=1 << 46, o0_q_res=0.1), dict(o0_flags=B.OPF_PER_CHANNEL, o0_aux=1 << 46),
                       dict(o0_q_out=-1.0), dict(o1_kind=B.OP_QUANTIZE)):
            assert joined(_layer_and_maximum(kind=kind, **change), 64) == -1, change
    for change in (dict(o1_mode=1), dict(o1_q_x=0.2), dict(o1_q_x=float("nan"), o1_q_out=float("nan")),
                   dict(o1_out_c_stride=72), dict(o1_out_c_stride=80, o1_out_c_off=8), dict(o1_out_c_stride=48)):
        assert joined(_layer_and_maximum(kind=B.OP_POOL, **change), 64) == -1, change
    assert joined(_layer_and_maximum(kind=B.OP_POOL, o1_out_c_stride=96, o1_out_c_off=32), 64) == 1
    # ops of other streams between the two: up to seven places on, each pair on its own
    two = _layer_and_maximum(2)
    assert joined(two, 64, 128) == 3 and joined(two, 64, 128, first=1) == 2 and joined(two, 64, 128, first=2) == -1
    assert joined(_layer_and_maximum(4), 64, 128, 192, 256) == 7
    assert joined(_layer_and_maximum(5), *range(64, 69)) == -1 and joined(_layer_and_maximum(5), *range(64, 69), first=1) == 8
    # ... unless they are ordered with it: the same stream under another index, the legacy default stream's two names
    assert joined(two, 64, 64) == -1 and joined(two, 64, 64, first=1) == 2 and joined(two, None, 1) == -1
    assert joined(two, 64) == -1 and joined(two, 64, 128, first=4) == -1


@pytest.mark.parametrize("C", range(32, 144, 16))
def test_block_tiles_take_any_channels_in_sixteens(C):
    assert B.conv_variant(B.ConvDesc(8, 150, 150, C, 64, 3, 3, 1, 1, 1, 1)) == "conv_i8_p3b_kernel"


def _kernels():
    """Metadata of every kernel in the library: the note of each code object of its offload bundles."""
    msgpack = pytest.importorskip("msgpack")
    data, magic = open(B.lib._name, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    for bundle in (m.start() for m in re.finditer(magic, data)):
        at = bundle + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, at - 8)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, at)
            triple, at, elf = data[at + 24:at + 24 + n], at + 24 + n, data[bundle + offset:bundle + offset + size]
            if b"gfx950" not in triple:
                continue
            headers, = struct.unpack_from("<Q", elf, 32)
            each, count = struct.unpack_from("<HH", elf, 54)
            for h in range(headers, headers + each * count, each):
                if struct.unpack_from("<I", elf, h)[0] == 4:                       # PT_NOTE
                    note, = struct.unpack_from("<Q", elf, h + 8)
                    name, length = struct.unpack_from("<II", elf, note)
                    text = note + 12 + (name + 3) // 4 * 4
                    yield from msgpack.unpackb(elf[text:text + length])["amdhsa.kernels"]


def test_tiles_of_the_3x3_family_stay_in_registers():
    """A register reloaded from scratch waits for every load in flight, the filters requested ahead among them."""
    found = {k[".name"]: k[".private_segment_fixed_size"] for k in _kernels() if "conv_i8_halo3_kernel" in k[".name"]}
    assert len(found) >= 18 and not {n: size for n, size in found.items() if size}


# calls of their own, us in the planned step's tile and in the larger one that the estimates name: 103 and 126, 73 and 85,
# 51 and 62, 13 and 14; and the same where the larger tile pays: 75 and 64, 138 and 96
@pytest.mark.parametrize("geom, larger", [
    ((55, 133, 130, 48, 80, 4, 4, 1, 1, 1, 1), False), ((58, 41, 101, 64, 480, 2, 2, 1, 1, 0, 0), False),
    ((35, 94, 97, 736, 80, 1, 1, 1, 1, 0, 0), False), ((57, 34, 34, 640, 400, 1, 1, 2, 2, 0, 0), False),
    ((64, 71, 71, 80, 180, 3, 3, 1, 1, 0, 0), True), ((6, 86, 85, 640, 128, 5, 5, 1, 1, 2, 2), True)])
def test_calls_take_larger_tiles_where_they_pay(geom, larger):
    d = B.ConvDesc(*geom, relu=1)
    assert (B.conv_call_variant(d) != B.conv_variant(d)) == larger


# us register-fed or on the fp32 instruction through LDS, and on the bf16 ones
@pytest.mark.parametrize("geom, split", [
    ((9, 86, 89, 320, 4, 5, 5, 1, 1, 0, 0, 2, 2), False),          # 279 and 336
    ((7, 94, 93, 448, 1, 3, 3, 1, 1, 1, 1), False),                # 150 and 171
    ((6, 140, 137, 160, 384, 1, 1), False),                        # 142 and 179
    ((19, 124, 125, 48, 128, 1, 1), False),                        # 117 and 122
    ((8, 38, 38, 512, 84, 3, 3, 1, 1, 1, 1), True),                # 146 and 94
    ((8, 38, 38, 512, 512, 3, 3, 1, 1, 1, 1), True)])              # 413 and 330
def test_fp32_layers_go_to_the_bf16_instructions_where_those_pay(geom, split):
    assert ("split" in B.conv_f32_variant(B.ConvDesc(*geom))) == split
