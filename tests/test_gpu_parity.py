"""GPU parity: every C-ABI call against the CPU oracle on the same seeded inputs.

Bar: bit-exact for int8 codes, int32 accumulators, int32 bias, max-abs and the folded fp32
weights (each is a fixed sequence of IEEE operations); dequantised values within 1e-5
relative (they are in fact bit-equal: one fp32 multiply).
"""
import numpy as np
import pytest
import torch

import oracle as orc
from oracle import net as onet
from paper_1805_08691_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import paper_1805_08691_amd.binding as b
    assert torch.cuda.is_available()
    return b


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# ------------------------------------------------------------------ calibration / Q / D
@pytest.mark.parametrize("n", [0, 1, 3, 5, 63, 1024, 4099, 1_000_003, 8_388_608 + 7])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_maxabs(B, n, offset):
    rng = np.random.default_rng(n + offset)
    x = rng.standard_normal(n + offset).astype(np.float32)
    if n > 10:
        x[offset + int(rng.integers(0, n))] = -7.25     # a single extreme, negative
    xd = dev(x)[offset:]
    slot = torch.zeros(1, device="cuda")
    B.calibrate_maxabs(xd, slot)
    assert host(slot)[0] == orc.maxabs(x[offset:])
    # running maximum over a second batch
    x2 = (x * np.float32(0.5)).astype(np.float32)
    x2[-1:] = 9.5
    B.calibrate_maxabs(dev(x2)[offset:], slot)
    assert host(slot)[0] == max(orc.maxabs(x[offset:]), orc.maxabs(x2[offset:]))


@pytest.mark.parametrize("n", [0, 1, 2, 7, 1023, 65536 + 5, 3_000_001])
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("p", [7, 4])
def test_quantize(B, n, offset, p):
    rng = np.random.default_rng(100 + n + offset)
    x = (rng.standard_normal(n + offset) * 2).astype(np.float32)
    q = np.float32(0.0371)
    if n > 64:      # exact ties and saturating values
        k = np.arange(-40, 24)
        x[offset:offset + 64] = (k.astype(np.float32) + np.float32(0.5)) * q
        x[offset + 64 - 4:offset + 64] = [1e6, -1e6, 127.5 * q, -128.5 * q]
    z = B.quantize(dev(x)[offset:], float(q), p)
    assert np.array_equal(host(z), orc.Q(x[offset:], q, p))


def test_quantize_pad_channels(B):
    rng = np.random.default_rng(7)
    x = rng.standard_normal((2, 9, 11, 3)).astype(np.float32)
    q = orc.qfactor(orc.maxabs(x), 7)
    z = host(B.quantize_pad_channels(dev(x), 4, float(q), 7))
    assert z.shape == (2, 9, 11, 4)
    assert np.array_equal(z[..., :3], orc.Q(x, q, 7)) and np.all(z[..., 3] == 0)
    z = host(B.quantize_pad_channels(dev(x), 16, float(q), 7))
    assert np.array_equal(z[..., :3], orc.Q(x, q, 7)) and np.all(z[..., 3:] == 0)


@pytest.mark.parametrize("n", [0, 1, 5, 1024, 1_000_003])
@pytest.mark.parametrize("offset", [0, 1])
def test_dequantize(B, n, offset):
    rng = np.random.default_rng(200 + n)
    z = rng.integers(-128, 128, n + offset).astype(np.int8)
    q = np.float32(0.0123)
    r = host(B.dequantize(dev(z)[offset:], float(q)))
    want = orc.D(z[offset:], q)
    assert np.array_equal(r, want)
    assert np.all(np.abs(r - want) <= 1e-5 * np.abs(want))


def test_elementwise_passes_beyond_2_31_elements(B):
    """Max-abs, Eq. Q and Eq. D on a tensor of more than 2^31 elements (64-bit indexing): a
    constant with a few planted values, checked on those and on sums over the whole tensor."""
    n = 2**31 + 1029
    x = torch.full((n,), 0.25, dtype=torch.float32, device="cuda")
    planted = {0: 3.0, 12345: -0.75, 2**31 - 1: 1.25, 2**31: -1.75, 2**31 + 3: 12.75, n - 1: -77.5}
    for i, v in planted.items():
        x[i] = v
    slot = torch.zeros(1, dtype=torch.float32, device="cuda")
    B.calibrate_maxabs(x, slot)
    assert float(host(slot)[0]) == 77.5                     # the extreme is the very last element
    q = np.float32(0.5)
    z = B.quantize(x, float(q), 7)
    idx = sorted(planted)
    want = orc.Q(np.array([planted[i] for i in idx], np.float32), q, 7)
    assert [int(z[i]) for i in idx] == want.tolist()        # incl. the tie 25.5 -> 26, clamp at -128
    assert int(orc.Q(np.array([0.25], np.float32), q, 7)[0]) == 0
    assert int(z.sum(dtype=torch.int64)) == int(want.astype(np.int64).sum())   # every other code is 0
    del x
    r = B.dequantize(z, float(q))
    assert [float(r[i]) for i in idx] == orc.D(want, q).tolist()
    assert int(torch.count_nonzero(r)) == int(np.count_nonzero(want))


def test_quantize_bias(B):
    rng = np.random.default_rng(9)
    b = (rng.standard_normal(1000) * 0.1).astype(np.float32)
    b[:4] = [1e9, -1e9, 0.0, 1e-12]
    for q_x, q_w in [(0.0137, 0.00091), (1.0, 1.0), (3e-3, 2.5e-4)]:
        z = host(B.quantize_bias(dev(b), q_x, q_w))
        assert np.array_equal(z, orc.Q31_bias(b, q_x, q_w))


@pytest.mark.parametrize("K,RSC", [(1, 1), (3, 7), (64, 576), (130, 1030)])
def test_fold_bn(B, K, RSC):
    rng = np.random.default_rng(K * 1000 + RSC)
    W = rng.standard_normal((K, RSC)).astype(np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    gamma = rng.uniform(.5, 1.5, K).astype(np.float32)
    beta = (rng.standard_normal(K) * .1).astype(np.float32)
    mu = (rng.standard_normal(K) * .1).astype(np.float32)
    var = rng.uniform(.5, 1.5, K).astype(np.float32)
    Wf, bf = B.fold_bn(dev(W), dev(b), dev(gamma), dev(beta), dev(mu), dev(var), 1e-5)
    Wo, bo = orc.fold_bn(W, b, gamma, beta, mu, var, 1e-5)
    assert np.array_equal(host(Wf), Wo) and np.array_equal(host(bf), bo)
    Wf, bf = B.fold_bn(dev(W), None, dev(gamma), dev(beta), dev(mu), dev(var), 1e-5)
    Wo, bo = orc.fold_bn(W, None, gamma, beta, mu, var, 1e-5)
    assert np.array_equal(host(Wf), Wo) and np.array_equal(host(bf), bo)


# ------------------------------------------------------------------ convolution
CONV_CASES = [
    # several tiles and ragged tails in pixels, channels and reduction
    dict(N=2, H=14, W=14, C=32, K=48, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=3, H=13, W=11, C=64, K=64, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=1, H=56, W=56, C=64, K=64, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=2, H=28, W=28, C=128, K=160, R=1, S=1),
    dict(N=2, H=28, W=28, C=256, K=128, R=1, S=1, stride_h=2, stride_w=2),
    dict(N=1, H=17, W=17, C=128, K=192, R=1, S=7, pad_w=3),
    dict(N=1, H=17, W=17, C=128, K=192, R=7, S=1, pad_h=3),
    dict(N=1, H=19, W=19, C=64, K=96, R=3, S=3, dil_h=6, dil_w=6, pad_h=6, pad_w=6),
    dict(N=2, H=12, W=12, C=48, K=64, R=5, S=5, pad_h=2, pad_w=2),
    dict(N=1, H=35, W=35, C=80, K=24, R=3, S=3, stride_h=2, stride_w=2),
    dict(N=1, H=10, W=10, C=16, K=126, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=2, H=9, W=9, C=16, K=17, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=1, H=3, W=3, C=256, K=16, R=3, S=3),
    dict(N=4, H=1, W=1, C=256, K=84, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=2, H=37, W=41, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),
    dict(N=2, H=37, W=40, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),  # rows of
    dict(N=3, H=9, W=12, C=3, K=64, R=3, S=3, pad_h=1, pad_w=1),     # whole 4-pixel groups
    dict(N=1, H=20, W=20, C=3, K=32, R=3, S=3, stride_h=2, stride_w=2),
    dict(N=1, H=16, W=16, C=4, K=8, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=1, H=7, W=7, C=512, K=2048 // 8, R=1, S=1),
    # more than 32 taps over 16-channel chunks: the register-staged kernel
    dict(N=1, H=15, W=15, C=16, K=40, R=7, S=7, pad_h=3, pad_w=3),
    dict(N=2, H=13, W=9, C=32, K=72, R=6, S=6, stride_h=2, stride_w=1, pad_h=2, pad_w=3),
    # a fully connected layer (Eq. A covers it): 1x1 convolution on a 1x1 map, M = batch
    dict(N=64, H=1, W=1, C=2048, K=1000, R=1, S=1),
]


def _run_conv_case(B, geom, relu, with_res, with_bias, seed, out_pad=0, out_off=0, variant=-1,
                   dump_acc=True, n_split=0, workspace=None):
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(seed)
    Cs = 4 if g.C < 4 else g.C                      # stored channels of the input
    x = rng.integers(-128, 128, (g.N, g.H, g.W, Cs)).astype(np.int8)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32) if with_bias else None
    Ho, Wo = g.Ho, g.Wo
    q_x, q_w = np.float32(0.021), np.float32(0.0017)
    fan = g.R * g.S * g.C
    # accumulators have std ~ 74^2 sqrt(fan): aim at ~40 output codes std, a few saturate
    q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(fan) / 40.0)
    q_res = np.float32(0.3) * q_out
    res = rng.integers(-128, 128, (g.N, Ho, Wo, g.K)).astype(np.int8) if with_res else None

    go = orc.ConvGeom(**{**geom, "in_c_stride": Cs})
    acc_o = orc.conv_i8(go, x, w, b)
    m = orc.requant_scale(q_x, q_w, q_out)
    m_r = orc.residual_scale(q_res, q_out) if with_res else 0.0
    out_cs = g.K + out_pad
    want = np.full((g.N, Ho, Wo, out_cs), 77, np.int8)
    orc.requant(acc_o, m, relu, res, m_r, out=want, out_c_stride=out_cs, out_c_off=out_off)

    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w, relu=relu, in_c_stride=Cs, out_c_stride=out_cs,
                   out_c_off=out_off)
    packed = B.pack_weights(d, dev(w))
    out = torch.full((g.N, Ho, Wo, out_cs), 77, dtype=torch.int8, device="cuda")
    dump = torch.zeros((g.N, Ho, Wo, g.K), dtype=torch.int32, device="cuda")
    B.conv_int8(d, dev(x), packed, None if b is None else dev(b), float(q_x), float(q_w),
                float(q_out), None if res is None else dev(res), float(q_res), out=out,
                acc_dump=dump if dump_acc else None, variant=variant, n_split=n_split,
                workspace=workspace)
    if dump_acc:
        assert np.array_equal(host(dump), acc_o), "int32 accumulators differ"
    got = host(out)
    assert np.array_equal(got, want), "int8 outputs differ"
    frac_sat = np.mean(np.abs(want[..., out_off:out_off + g.K].astype(int)) >= 127)
    assert frac_sat < 0.5


@pytest.mark.parametrize("idx", range(len(CONV_CASES)))
def test_conv_shapes(B, idx):
    geom = CONV_CASES[idx]
    _run_conv_case(B, geom, relu=True, with_res=False, with_bias=True, seed=idx)
    _run_conv_case(B, geom, relu=(idx % 2 == 0), with_res=True, with_bias=(idx % 3 != 0),
                   seed=1000 + idx)


VARIANT_CASES = [
    dict(N=2, H=14, W=14, C=64, K=160, R=3, S=3, pad_h=1, pad_w=1),      # uniform taps, tails
    dict(N=1, H=17, W=17, C=48, K=272, R=1, S=7, pad_w=3),               # per-lane taps, tails
    dict(N=3, H=28, W=28, C=128, K=64, R=1, S=1, stride_h=2, stride_w=2),
    dict(N=1, H=33, W=31, C=256, K=384, R=1, S=1),                       # complete + ragged tiles
    dict(N=2, H=43, W=47, C=3, K=96, R=7, S=7, stride_h=2, stride_w=2),  # unpadded 4-channel image
]


def test_conv_every_kernel_variant(B):
    """Every tile / ring variant of the main kernel gives the same bits (integer sums are
    order-independent; the epilogue is one fixed fp32 sequence)."""
    n = B.conv_num_variants()
    assert n >= 10
    for v in range(n):
        for k, geom in enumerate(VARIANT_CASES):
            _run_conv_case(B, geom, relu=bool(k % 2), with_res=bool((k + v) % 2),
                           with_bias=True, seed=100 * v + k, variant=v)


HALO_CASES = [   # 3x3, stride 1, padding 1, C % 64 == 0: the shapes the 3x3 tile family takes
    dict(N=3, H=7, W=7, C=64, K=64),          # several images inside one pixel tile
    dict(N=5, H=7, W=7, C=512, K=128),        # eight channel chunks, ragged last pixel tile
    dict(N=2, H=14, W=14, C=128, K=128),
    dict(N=1, H=28, W=28, C=64, K=256),
    dict(N=2, H=9, W=31, C=192, K=96),        # three chunks, K ends inside a channel tile
    dict(N=1, H=5, W=63, C=64, K=64),         # the widest map of the narrow patch buffers
    dict(N=1, H=3, W=100, C=64, K=128),       # only the wide patch buffers take it
    dict(N=1, H=2, W=300, C=64, K=64),        # only the widest one
    dict(N=1, H=1, W=1, C=64, K=64),          # one pixel: only the centre tap is inside
    dict(N=2, H=1, W=17, C=64, K=64),         # one row: no tap above or below
]


@pytest.mark.parametrize("idx", range(len(HALO_CASES)))
def test_conv_3x3_tile_family(B, idx):
    """Every build of the 3x3 tile family (activation patch with halo staged once per channel
    chunk, nine taps as nine row offsets) against the oracle; a build whose patch buffer is too
    narrow for the map hands the layer to the generic kernel, which must give the same bits."""
    geom = dict(R=3, S=3, pad_h=1, pad_w=1, **HALO_CASES[idx])
    n = B.conv_num_variants()
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(n)]
    halo = [v for v in range(n) if "halo3" in names[v]]
    assert len(halo) >= 4
    for k, v in enumerate(halo):
        _run_conv_case(B, geom, relu=bool(k % 2), with_res=bool((k + idx) % 2), with_bias=True,
                       seed=1000 * idx + v, variant=v)


P3_CASES = [     # 3x3, stride 1, padding 1, C = 64, K <= 64: what the persistent 3x3 family takes
    dict(N=2, H=56, W=56, C=64, K=64),        # several tiles per workgroup? no: one pass, ragged end
    dict(N=40, H=28, W=28, C=64, K=64),       # more tiles than resident workgroups: two passes
    dict(N=3, H=7, W=7, C=64, K=64),          # several images inside one pixel tile
    dict(N=1, H=5, W=63, C=64, K=48),         # the widest map of the narrow patch, K short of the tile
    dict(N=1, H=3, W=100, C=64, K=64),        # only the wide patch takes it
    dict(N=1, H=1, W=1, C=64, K=16),          # one pixel
    dict(N=2, H=1, W=17, C=64, K=32),         # one row: no tap above or below
    dict(N=2, H=19, W=301, C=64, K=64),       # a wide map: only the block-tiled build takes it
    dict(N=3, H=9, W=16, C=64, K=16),         # blocks: a ragged last block row, exact columns
]


@pytest.mark.parametrize("idx", range(len(P3_CASES)))
def test_conv_persistent_3x3_family(B, idx):
    """Every build of the persistent 3x3 family (all filters resident in LDS, workgroups walk
    over pixel tiles with the next tile's activation patch in flight) against the oracle; a
    build whose patch is too narrow for the map hands the layer to the generic kernel."""
    geom = dict(R=3, S=3, pad_h=1, pad_w=1, **P3_CASES[idx])
    n = B.conv_num_variants()
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(n)]
    p3 = [v for v in range(n) if "p3_kernel" in names[v] or "p3b_kernel" in names[v]]
    assert len(p3) >= 3
    for k, v in enumerate(p3):
        _run_conv_case(B, geom, relu=bool(k % 2), with_res=False, with_bias=True,
                       seed=5000 * idx + v, variant=v, out_pad=16 * (k % 2), out_off=16 * (k % 2),
                       dump_acc=False)


STEM_CASES = [   # unpadded 4-channel images, 5..8 taps per filter row: the image-row family
    dict(N=2, H=43, W=47, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2),
    dict(N=3, H=230, W=230, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2),   # ResNet-50's first layer
    dict(N=3, H=20, W=240, C=4, K=48, R=5, S=8, stride_h=1, stride_w=2),    # the widest image, K short
    dict(N=1, H=12, W=100, C=3, K=16, R=3, S=5),                            # stride 1
    dict(N=2, H=40, W=60, C=2, K=32, R=8, S=6, stride_h=4, stride_w=2),     # 8 + 4 rows in the ring
    dict(N=37, H=19, W=33, C=1, K=64, R=7, S=7, stride_h=2, stride_w=2),    # many images, short strips
    dict(N=1, H=9, W=200, C=3, K=64, R=3, S=5),                             # rows too long: generic kernel
]


@pytest.mark.parametrize("idx", range(len(STEM_CASES)))
def test_conv_image_row_family(B, idx):
    """The image-row family (filters resident, a ring of image rows in LDS as the activation
    operand, workgroups walking down strips of output rows) against the oracle, with and
    without ReLU and with a strided output; ResNet-50's first layer also picks it by itself."""
    geom = STEM_CASES[idx]
    n = B.conv_num_variants()
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(n)]
    stem = [v for v in range(n) if "stem_kernel" in names[v]]
    assert len(stem) == 1
    for k in range(2):
        _run_conv_case(B, geom, relu=bool(k), with_res=False, with_bias=bool(k), seed=7000 + 10 * idx + k,
                       variant=stem[0], out_pad=16 * k, out_off=16 * k, dump_acc=False)
    if idx == 1:
        g = orc.ConvGeom(**geom)
        d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, 0, 0, 1, 1,
                       relu=1, in_c_stride=4)
        assert "stem_kernel" in B.conv_variant(d)
        _run_conv_case(B, geom, relu=True, with_res=False, with_bias=True, seed=7777, dump_acc=False)


# 4-channel images with up to four rows and taps: runs of 32 pixels that end inside a row, an image, the
# tensor; fewer rows, taps and channels than the operand has; more runs than wavefronts; any stride
@pytest.mark.parametrize("geom", [
    (3, 15, 17, 3, 64, 3, 3, 1, 1), (1, 4, 5, 1, 16, 4, 4, 1, 1), (5, 33, 31, 4, 48, 2, 4, 2, 3),
    (2, 29, 27, 2, 32, 3, 1, 2, 2), (1, 3, 3, 3, 64, 3, 3, 1, 1), (7, 152, 151, 3, 64, 3, 3, 1, 1),
    (2, 23, 301, 3, 32, 1, 2, 1, 5)])
def test_conv_few_taps(B, geom):
    geom = dict(zip(("N", "H", "W", "C", "K", "R", "S", "stride_h", "stride_w"), geom))
    d = B.ConvDesc(**geom, relu=1, in_c_stride=4)
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(B.conv_num_variants())]
    v = names.index("conv_i8_taps4_kernel")
    if d.N * d.Ho * d.Wo >= 4096:
        assert B.conv_variant(d) == names[v]
    for k in range(2):
        _run_conv_case(B, geom, relu=bool(k), with_res=False, with_bias=bool(k), seed=7500 + k, variant=v,
                       out_pad=32 * k, out_off=16 * k, dump_acc=False)
    # what it does not take: a residual, accumulators as well, output rows of no 16 bytes
    _run_conv_case(B, geom, relu=True, with_res=True, with_bias=True, seed=7510, variant=v, out_pad=7, out_off=3)


HEAD_CASES = [   # image (N, H, W, C), filter, strides, padding = the zero frame around the image
    dict(N=2, H=37, W=41, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),
    dict(N=3, H=224, W=224, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),  # ResNet-50
    dict(N=1, H=24, W=20, C=1, K=48, R=5, S=5, stride_h=2, stride_w=2, pad_h=2, pad_w=2),
    dict(N=2, H=33, W=232, C=4, K=32, R=8, S=8, stride_h=2, stride_w=2, pad_h=4, pad_w=4),   # widest frame
    dict(N=35, H=19, W=33, C=2, K=16, R=3, S=6, stride_h=2, stride_w=1, pad_h=1, pad_w=2),
    dict(N=1, H=3, W=9, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),       # one or two rows
    dict(N=2, H=18, W=30, C=3, K=64, R=5, S=7, stride_h=1, stride_w=1, pad_h=2, pad_w=3),     # stride 1: no pool
]


@pytest.mark.parametrize("idx", range(len(HEAD_CASES)))
def test_conv_image_f32_head(B, idx):
    """Eq. Q on the real-valued image, the first layer and the 3x3 / 2 max-pool as one launch
    against the oracle's three steps (quantise, padded convolution + requantisation, max-pool
    of the codes); values next to rounding ties and beyond the code range are in the image."""
    geom = HEAD_CASES[idx]
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(900 + idx)
    r = rng.standard_normal((g.N, g.H, g.W, g.C)).astype(np.float32)
    q_x = orc.qfactor(np.float32(2.9), 7)                       # |r| > 2.9 saturates
    flat = r.reshape(-1)
    where = rng.choice(flat.size, flat.size // 7, replace=False)
    ties = ((rng.integers(-130, 130, where.size).astype(np.float32) + np.float32(0.5)) * q_x).astype(np.float32)
    toward = np.float32([-np.inf, 0.0, np.inf])[rng.integers(0, 3, where.size)]
    flat[where] = np.nextafter(ties, toward)                    # a tie or an fp32 neighbour of it
    z_x = orc.Q(r, q_x, 7)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-2000, 2000, g.K).astype(np.int32)
    q_w = np.float32(0.004)
    q_out = np.float32(q_x * q_w * 74 * 40 * np.sqrt(g.R * g.S * g.C) / 40.0)
    Hs, Ws = g.H + 2 * g.pad_h, g.W + 2 * g.pad_w
    d = B.ConvDesc(g.N, Hs, Ws, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, 0, 0, 1, 1,
                   relu=1, in_c_stride=4)
    packed = B.pack_weights(d, dev(w))
    for relu in (1, 0):
        d.relu = relu
        conv = orc.requant(orc.conv_i8(g, z_x, w, b), orc.requant_scale(q_x, q_w, q_out), bool(relu))
        for pool in (0, 1):
            ok = B.conv_image_f32_supported(d, g.H, g.W, g.C, g.pad_h, g.pad_w, pool)
            assert ok == (not (pool and g.stride_h != 2))
            if not ok:
                continue
            want = orc.maxpool_i8(conv, 3, 3, 2, 1, (g.Ho - 1) // 2 + 1, (g.Wo - 1) // 2 + 1) if pool else conv
            out = torch.full(want.shape, 77, dtype=torch.int8, device="cuda")
            B.conv_image_f32(d, dev(r), g.pad_h, g.pad_w, float(q_x), 7, packed, dev(b), float(q_w),
                             float(q_out), pool=pool, out=out)
            assert np.array_equal(host(out), want), f"relu={relu} pool={pool}"


@pytest.mark.parametrize("geom", [
    dict(N=2, H=7, W=7, C=512, K=2048, R=1, S=1),                          # ResNet-50's last layer
    dict(N=1, H=9, W=11, C=64, K=40, R=3, S=3, pad_h=1, pad_w=1),          # K ends inside a group
    dict(N=3, H=5, W=5, C=3, K=24, R=3, S=3, pad_h=1, pad_w=1),            # the small-channel kernel
])
def test_conv_with_dequantized_output(B, geom):
    """Eq. A' and Eq. D in one launch: the codes equal the oracle's, and the fp32 tensor is
    Eq. D of those codes (one fp32 multiplication, bit for bit); channels outside the
    layer's slice of a wider tensor are left alone."""
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(4242 + g.K)
    Cs = 4 if g.C < 4 else g.C
    x = rng.integers(-128, 128, (g.N, g.H, g.W, Cs)).astype(np.int8)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32)
    res = rng.integers(-128, 128, (g.N, g.Ho, g.Wo, g.K)).astype(np.int8)
    q_x, q_w = np.float32(0.021), np.float32(0.0017)
    q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(g.R * g.S * g.C) / 40.0)
    q_res = np.float32(0.3) * q_out
    go = orc.ConvGeom(**{**geom, "in_c_stride": Cs})
    acc = orc.conv_i8(go, x, w, b)
    for with_res, pad in ((True, 0), (False, 8)):
        ocs = g.K + pad
        want = np.full((g.N, g.Ho, g.Wo, ocs), 77, np.int8)
        orc.requant(acc, orc.requant_scale(q_x, q_w, q_out), True, res if with_res else None,
                    orc.residual_scale(q_res, q_out) if with_res else 0.0, out=want,
                    out_c_stride=ocs, out_c_off=pad)
        d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                       g.dil_h, g.dil_w, relu=1, in_c_stride=Cs, out_c_stride=ocs, out_c_off=pad)
        out = torch.full(want.shape, 77, dtype=torch.int8, device="cuda")
        out_f = torch.full(want.shape, -5.0, dtype=torch.float32, device="cuda")
        B.conv_int8_dequantized(d, dev(x), B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w),
                                float(q_out), dev(res) if with_res else None, float(q_res),
                                out=out, out_f32=out_f)
        assert np.array_equal(host(out), want)
        want_f = np.full(want.shape, -5.0, np.float32)
        want_f[..., pad:] = orc.D(want[..., pad:], q_out)
        assert np.array_equal(host(out_f), want_f)


def test_conv_image_f32_head_rejects(B):
    """Host checks of the fused head: a layer outside the family is unsupported, an image that
    does not fit its frame is invalid."""
    d = B.ConvDesc(1, 30, 30, 3, 64, 3, 3, 1, 1, 0, 0, 1, 1, relu=1, in_c_stride=4)   # 3 columns
    assert not B.conv_image_f32_supported(d, 28, 28, 3, 1, 1, 0)
    d = B.ConvDesc(1, 30, 30, 3, 64, 7, 7, 2, 2, 0, 0, 1, 1, relu=1, in_c_stride=4)
    assert B.conv_image_f32_supported(d, 24, 24, 3, 3, 3, 1)
    assert not B.conv_image_f32_supported(d, 28, 24, 3, 3, 3, 1)                     # 3 + 28 > 30
    assert not B.conv_image_f32_supported(d, 24, 24, 4, 3, 3, 1)                     # C != d.C
    r = torch.zeros((1, 28, 24, 3), dtype=torch.float32, device="cuda")
    w = torch.zeros((64, 7, 7, 3), dtype=torch.int8, device="cuda")
    with pytest.raises(B.Q8Error):
        B.conv_image_f32(d, r, 3, 3, 0.02, 7, B.pack_weights(d, w), None, 0.01, 0.5)


SPLIT_CASES = [   # long reductions over few output tiles: what a split reduction is for
    dict(N=5, H=7, W=7, C=512, K=512, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=3, H=14, W=14, C=1024, K=256, R=1, S=1),
    dict(N=2, H=9, W=11, C=192, K=96, R=3, S=3, pad_h=1, pad_w=1),        # ragged tiles
    dict(N=1, H=14, W=14, C=1024, K=512, R=1, S=1, stride_h=2, stride_w=2),
    dict(N=2, H=8, W=8, C=128, K=128, R=3, S=3, pad_h=2, pad_w=2, dil_h=2, dil_w=2),
    dict(N=1, H=6, W=6, C=64, K=64, R=1, S=1),                             # one step: never split
]


@pytest.mark.parametrize("idx", range(len(SPLIT_CASES)))
def test_conv_split_reduction(B, idx):
    """Eq. x: the accumulator is an integer sum, so splitting the reduction over 2, 3, 5 or 7
    workgroups per tile (partial tiles through the caller's workspace, the last workgroup to
    arrive adds them up) gives the oracle's accumulators and codes bit for bit, with every
    split build.  One workspace, zeroed once, serves all calls: each leaves its counters zero."""
    geom = SPLIT_CASES[idx]
    g = orc.ConvGeom(**geom)
    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w)
    n = B.conv_num_variants()
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(n)]
    split = [v for v in range(n) if "split" in names[v]]
    assert len(split) >= 4
    factors = (2, 3, 5, 7)
    need = max(B.conv_workspace_bytes(d, v, f) for v in split for f in factors)
    ws = torch.zeros(max(need, 256), dtype=torch.uint8, device="cuda")
    for k, v in enumerate(split):
        for f in factors:
            _run_conv_case(B, geom, relu=bool((k + f) % 2), with_res=bool(k % 2), with_bias=True,
                           seed=7000 + 100 * idx + 10 * k + f, variant=v, n_split=f, workspace=ws)
    if need:
        words = B.conv_workspace_bytes(d, split[0], 2)      # (an upper bound on the counters)
        assert not host(ws[:min(words, 4096)]).view(np.int32)[:16].any()


PW_CASES = [     # 1x1, stride 1, no padding, C in {64, 128, 256}: what the pointwise family takes
    dict(N=2, H=56, W=56, C=64, K=256),       # many pixel tiles per workgroup, ragged last tile
    dict(N=1, H=28, W=28, C=128, K=512),
    dict(N=3, H=19, W=23, C=256, K=64),
    dict(N=1, H=9, W=9, C=64, K=64),          # fewer pixel tiles than workgroups
    dict(N=2, H=31, W=17, C=128, K=96),       # K ends inside a channel tile
    dict(N=40, H=28, W=28, C=64, K=128),      # more pixel tiles than one round of workgroups
    dict(N=1, H=1, W=1, C=256, K=320),
]


@pytest.mark.parametrize("idx", range(len(PW_CASES)))
def test_conv_pointwise_tile_family(B, idx):
    """Every build of the pointwise tile family (persistent workgroups, filters resident in LDS,
    the next pixel tile's operands in flight while the current one is computed) against the
    oracle; a build made for another channel count hands the layer to the generic kernel."""
    geom = dict(R=1, S=1, **PW_CASES[idx])
    n = B.conv_num_variants()
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(n)]
    pw = [v for v in range(n) if "pw_kernel" in names[v]]
    assert len(pw) >= 4
    for k, v in enumerate(pw):
        for with_res in (False, True):
            _run_conv_case(B, geom, relu=bool((k + with_res) % 2), with_res=with_res,
                           with_bias=True, seed=3000 * idx + 2 * v + with_res, variant=v,
                           out_pad=16 * (k % 2), out_off=16 * (k % 2), dump_acc=False)


@pytest.mark.parametrize("q", [0.03, 0.0078125, 1.0 / 3.0, 0.0123456789, 5.5e-3])
def test_quantize_image_next_to_ties(B, q):
    """Eq. Q on values whose quotient r/q lies on, and within a few ulps of, every tie k + 1/2
    and every integer k of the code range (and beyond its ends): the image kernel, which only
    divides where a product with 1/q cannot decide the rounding, must give the oracle's codes."""
    q = np.float32(q)
    ks = np.arange(-131, 131, dtype=np.float64)
    centres = np.concatenate([ks + 0.5, ks]) * np.float64(q)
    vals = []
    for c in centres.astype(np.float32):
        v = c
        for _ in range(6):
            v = np.nextafter(v, np.float32(-np.inf), dtype=np.float32)
        for _ in range(13):
            vals.append(v)
            v = np.nextafter(v, np.float32(np.inf), dtype=np.float32)
    vals = np.array(vals, dtype=np.float32)
    n_pix = -(-vals.size // 3)
    W = 8
    Hh = -(-n_pix // W)
    r = np.zeros((1, Hh, W, 3), np.float32)
    r.reshape(-1)[:vals.size] = vals
    want = orc.Q(r, q, 7)
    ties = np.abs(np.abs(vals.astype(np.float64) / np.float64(q)) % 1.0 - 0.5) < 1e-4
    assert ties.sum() > 2000                                 # the cases are what they claim to be
    frame = torch.zeros((1, Hh, W, 4), dtype=torch.int8, device="cuda")
    B.quantize_image(dev(r), float(q), 7, frame, 0, 0)
    got = host(frame)
    assert np.array_equal(got[..., :3], want)
    assert not got[..., 3].any()


# (the last two as the kernel that holds whole image rows)
@pytest.mark.parametrize("N, H, W, K, S, stride", [
    (2, 28, 36, 128, 7, 1), (3, 9, 11, 40, 4, 1), (1, 5, 33, 70, 13, 1), (2, 9, 20, 64, 1, 1), (2, 9, 21, 64, 5, 2),
    (2, 6, 9, 16, 2, 1), (8, 70, 76, 64, 7, 1), (8, 131, 139, 48, 7, 2)])
def test_conv_image_filters_of_one_row(B, N, H, W, K, S, stride):
    """A 1 x S filter over an unpadded image of three channels, in every precision."""
    d = B.ConvDesc(N, H, W, 3, K, 1, S, stride, stride, in_c_stride=4, relu=1)
    rng = np.random.default_rng(S)
    x = rng.integers(-128, 128, (N, H, W, 4)).astype(np.int8)
    w, b = rng.integers(-128, 128, (K, 1, S, 3)).astype(np.int8), rng.integers(-20000, 20000, K).astype(np.int32)
    acc = torch.nn.functional.conv2d(torch.from_numpy(x[..., :3].astype(np.float64)).permute(0, 3, 1, 2),
                                     torch.from_numpy(w.astype(np.float64)).permute(0, 3, 1, 2),
                                     torch.from_numpy(b.astype(np.float64)), stride)
    acc = acc.permute(0, 2, 3, 1).contiguous().numpy().astype(np.int32)
    scale = np.float32(60.0 / (74.0 * 74.0 * np.sqrt(3 * S)))
    packed, dump = B.pack_weights(d, dev(w)), torch.zeros(acc.shape, dtype=torch.int32, device="cuda")
    got = B.conv_int8(d, dev(x), packed, dev(b), 1.0, float(scale), 1.0, acc_dump=dump)
    want = orc.requant(acc, orc.requant_scale(1.0, scale, 1.0), True)
    assert np.array_equal(host(dump), acc) and np.array_equal(host(got), want)
    got = B.conv_int8(d, dev(x), packed, dev(b), 1.0, float(scale), 1.0)
    assert np.array_equal(host(got), want) and len(np.unique(want)) > 16
    if K > 32:
        m = (scale * rng.uniform(0.3, 3.0, K)).astype(np.float32)
        got = B.conv_int8_per_channel(d, dev(x), packed, dev(b), dev(m), 1.0)
        assert np.array_equal(host(got), orc.requant_pc(acc, m, True, None, np.float32(0)))
        got = B.conv_u8(d, 0, 1, 0, dev(x), packed, dev(b), None, 1.0, float(scale), 1.0)
        assert np.array_equal(host(got), _stored(orc.requant_mixed(
            acc, orc.requant_scale(1.0, scale, 1.0), True, None, np.float32(0), out_unsigned=True)))


@pytest.mark.parametrize("geom", [
    dict(N=2, H=37, W=41, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, pad_h=3, pad_w=3),
    dict(N=1, H=39, W=39, C=3, K=64, R=3, S=3, stride_h=2, stride_w=2),
    dict(N=2, H=30, W=31, C=3, K=64, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=1, H=24, W=20, C=1, K=40, R=5, S=5, pad_h=2, pad_w=2),
    dict(N=1, H=12, W=12, C=4, K=48, R=3, S=9, pad_h=1, pad_w=4),
])
def test_conv_image_in_zero_frame(B, geom):
    """A C <= 4 image quantised into a zero frame that holds the layer's padding, the layer
    then run without padding, equals the oracle's padded convolution of the bare image."""
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(g.H * 100 + g.W)
    r = rng.standard_normal((g.N, g.H, g.W, g.C)).astype(np.float32)
    q_x = orc.qfactor(orc.maxabs(r), 7)
    z_x = orc.Q(r, q_x, 7)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-2000, 2000, g.K).astype(np.int32)
    q_w = np.float32(0.004)
    q_out = np.float32(q_x * q_w * 74 * 40 * np.sqrt(g.R * g.S * g.C) / 40.0)
    acc_o = orc.conv_i8(g, z_x, w, b)
    want = orc.requant(acc_o, orc.requant_scale(q_x, q_w, q_out), True)

    Hs, Ws = g.H + 2 * g.pad_h, g.W + 2 * g.pad_w
    frame = torch.zeros((g.N, Hs, Ws, 4), dtype=torch.int8, device="cuda")
    B.quantize_image(dev(r), float(q_x), 7, frame, g.pad_h, g.pad_w)
    f = host(frame)
    assert np.array_equal(f[:, g.pad_h:g.pad_h + g.H, g.pad_w:g.pad_w + g.W, :g.C], z_x)
    f[:, g.pad_h:g.pad_h + g.H, g.pad_w:g.pad_w + g.W, :g.C] = 0
    assert not f.any()
    d = B.ConvDesc(g.N, Hs, Ws, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, 0, 0, 1, 1,
                   relu=1, in_c_stride=4)
    assert (d.Ho, d.Wo) == (g.Ho, g.Wo)
    assert "ring" in B.conv_variant(d)
    dump = torch.zeros((g.N, g.Ho, g.Wo, g.K), dtype=torch.int32, device="cuda")
    got = B.conv_int8(d, frame, B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w),
                      float(q_out), acc_dump=dump)
    assert np.array_equal(host(dump), acc_o)
    assert np.array_equal(host(got), want)


# rows whose last four pixels are not a group of their own, and rows of fewer
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 7, 9, 75, 299])
def test_quantize_image_rows(B, W):
    rng = np.random.default_rng(W)
    r = (rng.standard_normal((3, 5, W, 3)) * 2).astype(np.float32)
    want = np.full((3, 8, W + 3, 4), 77, np.int8)
    want[:, 2:7, 1:1 + W, :3], want[:, 2:7, 1:1 + W, 3] = orc.Q(r, np.float32(0.021), 7), 0
    frame = torch.full(want.shape, 77, dtype=torch.int8, device="cuda")
    B.quantize_image(dev(r), 0.021, 7, frame, 2, 1)
    assert np.array_equal(host(frame), want)


# ------------------------------------------------------------------ unsigned activations
def _stored(u8):
    """unsigned codes -> the stored form (code - 128 in an int8 byte)."""
    return (u8.astype(np.int16) - 128).astype(np.int8)


def test_quantize_dequantize_u8(B):
    rng = np.random.default_rng(81)
    r = np.abs(rng.standard_normal(100_003)).astype(np.float32) * 3
    r[:4] = [0.0, 1e-9, 1e9, 2.5]
    q = orc.qfactor(np.float32(9.0), 8)              # some values saturate at 255
    want = orc.Q_u8(r, q)
    got = host(B.quantize_u8(dev(r), float(q)))
    assert np.array_equal(got, _stored(want))
    back = host(B.dequantize_u8(dev(got), float(q)))
    assert np.array_equal(back, orc.D_u8(want, q))


@pytest.mark.parametrize("q", [0.0371, 1.0, 3.3e-5, 1e-37])   # (of the last no reciprocal is taken)
@pytest.mark.parametrize("unsigned", [True, False])
def test_quantize_alignments_and_ties(B, q, unsigned):
    """Eq. Q where the vector body does not start at the first value, does not fit both buffers or
    is empty, on values on and within three ulps of every tie, and outside the code range."""
    q = np.float32(q)
    call = B.quantize_u8 if unsigned else lambda r, q, out: B.quantize(r, q, 7, out)
    ties = ((np.arange(-131, 260) + 0.5) * np.float64(q)).astype(np.float32)
    vals = [ties]
    for direction in (np.float32(-np.inf), np.float32(np.inf)):
        v = ties
        for _ in range(3):
            v = np.nextafter(v, direction, dtype=np.float32)
            vals.append(v)
    vals = np.concatenate(vals + [np.array([0, np.inf, -np.inf, 1e30, -1e30], np.float32)])
    want = _stored(orc.Q_u8(np.maximum(vals, 0), q)) if unsigned else orc.Q(vals, q, 7)
    n_max = vals.size
    r_buf, z_buf = torch.zeros(n_max + 4, device="cuda"), torch.empty(n_max + 8, dtype=torch.int8, device="cuda")
    for r_off in range(4):
        r_buf[r_off:r_off + n_max] = dev(vals)
        for z_off in range(4):
            for n in (*range(1, 34), 64, n_max):
                z_buf.fill_(55)
                call(r_buf[r_off:r_off + n], float(q), z_buf[z_off:z_off + n])
                got = host(z_buf)
                assert np.array_equal(got[z_off:z_off + n], want[:n]), (r_off, z_off, n)
                assert np.all(got[:z_off] == 55) and np.all(got[z_off + n:] == 55)


@pytest.mark.parametrize("z_off, r_off", [(0, 0), (4, 0), (1, 0), (0, 1), (3, 2)])
def test_dequantize_u8_alignments(B, z_off, r_off):
    z = np.random.default_rng(2).integers(-128, 128, 9000 + z_off).astype(np.int8)
    zd, r = dev(z), torch.empty(9000 + r_off, device="cuda")
    for n in (1, 2, 3, 4, 5, 63, 4095, 4096, 4097, 9000):
        r.fill_(-7)
        B.dequantize_u8(zd[z_off:z_off + n], 0.0123, r[r_off:r_off + n])
        want = orc.D_u8((z[z_off:z_off + n].astype(np.int16) + 128).astype(np.uint8), np.float32(0.0123))
        got = host(r)
        assert np.array_equal(got[r_off:r_off + n], want) and np.all(got[r_off + n:] == -7)


U8_CASES = [
    # geometry, in_u8, out_u8, res ("u8", "s8" or None), relu
    (dict(N=2, H=14, W=14, C=64, K=160, R=3, S=3, pad_h=1, pad_w=1), 1, 1, "u8", 1),
    (dict(N=2, H=14, W=14, C=64, K=160, R=3, S=3, pad_h=1, pad_w=1), 1, 0, "s8", 0),
    (dict(N=1, H=15, W=13, C=32, K=64, R=3, S=3, pad_h=1, pad_w=1, stride_h=2, stride_w=2), 1, 1, None, 1),
    (dict(N=3, H=9, W=9, C=128, K=256, R=1, S=1), 1, 1, "s8", 1),
    (dict(N=3, H=9, W=9, C=128, K=256, R=1, S=1), 0, 1, "u8", 1),
    (dict(N=1, H=17, W=17, C=48, K=96, R=1, S=7, pad_w=3), 1, 0, None, 1),
    (dict(N=1, H=12, W=12, C=16, K=72, R=3, S=3, dil_h=2, dil_w=2, pad_h=2, pad_w=2), 1, 1, "u8", 1),
    (dict(N=1, H=7, W=7, C=64, K=64, R=5, S=5, pad_h=2, pad_w=2), 1, 1, None, 1),   # mostly border
    (dict(N=2, H=28, W=28, C=64, K=128, R=3, S=3, pad_h=1, pad_w=1), 1, 1, "u8", 1),  # complete tiles
]


@pytest.mark.parametrize("idx", range(len(U8_CASES)))
def test_conv_unsigned_activations(B, idx):
    """Eq. A' on unsigned p = 8 codes (the paper's form for non-negative tensors) through
    the signed matrix instruction: accumulators and outputs equal the oracle's, which
    works on the codes 0..255 themselves."""
    geom, in_u8, out_u8, res_kind, relu = U8_CASES[idx]
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(500 + idx)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32)
    if in_u8:
        x = rng.integers(0, 256, (g.N, g.H, g.W, g.C)).astype(np.uint8)
        acc_o = orc.conv_u8(g, x, w, b)
        x_st = _stored(x)
    else:
        x = rng.integers(-128, 128, (g.N, g.H, g.W, g.C)).astype(np.int8)
        acc_o = orc.conv_i8(g, x, w, b)
        x_st = x
    Ho, Wo = g.Ho, g.Wo
    q_x, q_w = np.float32(0.011), np.float32(0.0017)
    fan = g.R * g.S * g.C
    q_out = np.float32(q_x * q_w * 74.0 * (147.0 if in_u8 else 74.0) * np.sqrt(fan) / 60.0)
    q_res = np.float32(0.4) * q_out
    res = res_st = None
    if res_kind == "u8":
        res = rng.integers(0, 256, (g.N, Ho, Wo, g.K)).astype(np.uint8)
        res_st = _stored(res)
    elif res_kind == "s8":
        res = res_st = rng.integers(-128, 128, (g.N, Ho, Wo, g.K)).astype(np.int8)
    m = orc.requant_scale(q_x, q_w, q_out)
    m_r = orc.residual_scale(q_res, q_out) if res is not None else 0.0
    want = orc.requant_mixed(acc_o, m, relu, res, m_r, out_unsigned=bool(out_u8))

    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w, relu=relu)
    packed = B.pack_weights(d, dev(w))
    if in_u8:
        taps, bias = B.u8_prepare(d, dev(w), dev(b))
        tw = w.astype(np.int64).sum(axis=3)                               # [K, R, S]
        # one row per rectangle [r_lo, r_hi) x [s_lo, s_hi) of taps inside the image
        tab = host(taps).reshape(g.R + 1, g.R + 1, g.S + 1, g.S + 1, g.K)
        for r_lo, r_hi, s_lo, s_hi in [(0, g.R, 0, g.S), (1, g.R, 0, g.S), (0, g.R - 1, 0, g.S - 1),
                                       (0, 1, 0, 1), (g.R, 0, 0, g.S), (0, 0, 0, 0)]:
            inside = tw[:, r_lo:r_hi, s_lo:s_hi].sum(axis=(1, 2)) if r_hi > r_lo and s_hi > s_lo else 0
            assert np.array_equal(tab[r_lo, r_hi, s_lo, s_hi], b + 128 * inside)
        assert np.array_equal(host(bias), b + 128 * tw.sum(axis=(1, 2)))
    else:
        taps, bias = None, dev(b)
    dump = torch.zeros((g.N, Ho, Wo, g.K), dtype=torch.int32, device="cuda")
    for use_dump in (True, False):             # general epilogue, then the fast one
        got = B.conv_u8(d, in_u8, out_u8, res_kind == "u8", dev(x_st), packed, bias, taps,
                        float(q_x), float(q_w), float(q_out),
                        None if res_st is None else dev(res_st), float(q_res),
                        acc_dump=dump if use_dump else None)
        if use_dump:
            assert np.array_equal(host(dump), acc_o), "int32 accumulators differ"
        got = host(got)
        if out_u8:
            assert np.array_equal(got.astype(np.int16) + 128, want.astype(np.int16))
        else:
            assert np.array_equal(got, want)
    sat = np.mean((want == (255 if out_u8 else 127)))
    assert sat < 0.5


# ------------------------------------------------------------------ per-channel weights
def test_per_channel_weight_preparation(B):
    rng = np.random.default_rng(91)
    K = 70
    W = (rng.standard_normal((K, 3, 3, 16)) * rng.uniform(0.01, 3.0, K)[:, None, None, None])
    W = W.astype(np.float32)
    W[5] = 0                                            # an all-zero filter
    b = rng.standard_normal(K).astype(np.float32)
    z_o, q_o = orc.quantize_weights_pc(W)
    q_g, z_g = B.quantize_weights_per_channel(dev(W))
    assert np.array_equal(host(q_g), q_o) and np.array_equal(host(z_g), z_o)
    q_x, q_out = np.float32(0.0231), np.float32(0.177)
    assert np.array_equal(host(B.quantize_bias_per_channel(dev(b), float(q_x), q_g)),
                          orc.Q31_bias_pc(b, q_x, q_o))
    assert np.array_equal(host(B.requant_scales(float(q_x), q_g, float(q_out))),
                          orc.requant_scales_pc(q_x, q_o, q_out))


@pytest.mark.parametrize("geom,with_res", [
    (dict(N=2, H=14, W=14, C=64, K=160, R=3, S=3, pad_h=1, pad_w=1), True),
    (dict(N=2, H=28, W=28, C=64, K=128, R=1, S=1), False),
    (dict(N=1, H=17, W=17, C=48, K=72, R=1, S=7, pad_w=3), True),
    (dict(N=2, H=30, W=30, C=3, K=64, R=3, S=3, in_c_stride=4), False),     # unpadded image
])
def test_conv_per_channel_scales(B, geom, with_res):
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(g.K + g.C)
    Cs = g.in_c_stride or g.C
    x = rng.integers(-128, 128, (g.N, g.H, g.W, Cs)).astype(np.int8)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32)
    acc_o = orc.conv_i8(g, x, w, b)
    base = 40.0 / (5476.0 * np.sqrt(g.R * g.S * g.C))
    m = (base * rng.uniform(0.3, 3.0, g.K)).astype(np.float32)
    res = rng.integers(-128, 128, acc_o.shape).astype(np.int8) if with_res else None
    m_r = np.float32(0.3)
    want = orc.requant_pc(acc_o, m, True, res, m_r)
    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w, relu=1, in_c_stride=Cs)
    packed = B.pack_weights(d, dev(w))
    dump = torch.zeros(acc_o.shape, dtype=torch.int32, device="cuda")
    for use_dump in (True, False):             # general epilogue, then the fast one
        got = B.conv_int8_per_channel(d, dev(x), packed, dev(b), dev(m), 1.0,
                                      None if res is None else dev(res), float(m_r),
                                      acc_dump=dump if use_dump else None)
        if use_dump:
            assert np.array_equal(host(dump), acc_o)
        assert np.array_equal(host(got), want)


def _random_geometries(seed, count):
    """Seeded small geometries with everything unequal: strides, pads, dilations, odd extents,
    K and C off the tile sizes."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        R, S = int(rng.integers(1, 6)), int(rng.integers(1, 6))
        g = dict(N=int(rng.integers(1, 4)), H=int(rng.integers(5, 24)), W=int(rng.integers(5, 24)),
                 C=16 * int(rng.integers(1, 7)), K=int(rng.integers(1, 200)), R=R, S=S,
                 stride_h=int(rng.integers(1, 4)), stride_w=int(rng.integers(1, 4)),
                 pad_h=int(rng.integers(0, R)), pad_w=int(rng.integers(0, S)),
                 dil_h=int(rng.integers(1, 3)), dil_w=int(rng.integers(1, 3)))
        geom = orc.ConvGeom(**g)
        if geom.Ho >= 1 and geom.Wo >= 1:
            out.append(g)
    return out


@pytest.mark.parametrize("geom", _random_geometries(1805, 24))
def test_conv_random_geometries(B, geom):
    """int32 accumulators and int8 outputs for seeded random geometries, signed and (where
    the extended build takes the shape) with unsigned input codes."""
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(g.K * 31 + g.C + g.H)
    x = rng.integers(-128, 128, (g.N, g.H, g.W, g.C)).astype(np.int8)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32)
    res = rng.integers(-128, 128, (g.N, g.Ho, g.Wo, g.K)).astype(np.int8)
    q_x, q_w = np.float32(0.021), np.float32(0.0017)
    q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(g.R * g.S * g.C) / 40.0)
    q_res = np.float32(0.3) * q_out
    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w, relu=1)
    packed = B.pack_weights(d, dev(w))
    m, m_r = orc.requant_scale(q_x, q_w, q_out), orc.residual_scale(q_res, q_out)
    acc_o = orc.conv_i8(g, x, w, b)
    want = orc.requant(acc_o, m, True, res, m_r)
    dump = torch.zeros((g.N, g.Ho, g.Wo, g.K), dtype=torch.int32, device="cuda")
    for use_dump in (True, False):
        got = B.conv_int8(d, dev(x), packed, dev(b), float(q_x), float(q_w), float(q_out), dev(res),
                          float(q_res), acc_dump=dump if use_dump else None)
        if use_dump:
            assert np.array_equal(host(dump), acc_o)
        assert np.array_equal(host(got), want)
    if g.K > 32 and g.R * g.S <= 32:          # unsigned input codes, border start table
        xu = rng.integers(0, 256, (g.N, g.H, g.W, g.C)).astype(np.uint8)
        acc_u = orc.conv_u8(g, xu, w, b)
        want_u = orc.requant_mixed(acc_u, m, True, res, m_r, out_unsigned=True)
        taps, bias = B.u8_prepare(d, dev(w), dev(b))
        got = B.conv_u8(d, 1, 1, 0, dev(_stored(xu)), packed, bias, taps, float(q_x), float(q_w),
                        float(q_out), dev(res), float(q_res), acc_dump=dump)
        assert np.array_equal(host(dump), acc_u)
        assert np.array_equal(host(got).astype(np.int16) + 128, want_u.astype(np.int16))


PAIR_CASES = [
    # first layer, K2, residual, ReLU of the second layer
    (dict(N=2, H=14, W=14, C=64, K=64, R=3, S=3, pad_h=1, pad_w=1), 256, True, True),
    (dict(N=3, H=13, W=11, C=64, K=64, R=3, S=3, pad_h=1, pad_w=1), 128, False, True),   # ragged pixels
    (dict(N=2, H=28, W=28, C=128, K=128, R=3, S=3, pad_h=1, pad_w=1), 512, True, True),
    (dict(N=1, H=9, W=7, C=128, K=128, R=3, S=3, pad_h=1, pad_w=1), 128, True, False),
    (dict(N=2, H=20, W=20, C=64, K=64, R=1, S=1), 64, False, False),                      # 1x1 -> 1x1
    (dict(N=1, H=31, W=31, C=192, K=128, R=3, S=3, stride_h=2, stride_w=2), 384, False, True),
]


@pytest.mark.parametrize("geom,K2,with_res,relu2", PAIR_CASES)
def test_conv_pair_equals_two_layers(B, geom, K2, with_res, relu2):
    """The fused 3x3 -> 1x1 launch gives the bits of the oracle's two layers."""
    g1 = orc.ConvGeom(**geom)
    rng = np.random.default_rng(g1.K + K2 + g1.H)
    x = rng.integers(-128, 128, (g1.N, g1.H, g1.W, g1.C)).astype(np.int8)
    w1 = rng.integers(-128, 128, (g1.K, g1.R, g1.S, g1.C)).astype(np.int8)
    b1 = rng.integers(-20000, 20000, g1.K).astype(np.int32)
    Ho, Wo = g1.Ho, g1.Wo
    g2 = orc.ConvGeom(N=g1.N, H=Ho, W=Wo, C=g1.K, K=K2, R=1, S=1)
    w2 = rng.integers(-128, 128, (K2, 1, 1, g1.K)).astype(np.int8)
    b2 = rng.integers(-20000, 20000, K2).astype(np.int32)
    q_x, q_w1, q_w2 = np.float32(0.021), np.float32(0.0017), np.float32(0.0023)
    q_mid = np.float32(q_x * q_w1 * 5476.0 * np.sqrt(g1.R * g1.S * g1.C) / 40.0)
    q_out = np.float32(q_mid * q_w2 * 3000.0 * np.sqrt(g1.K) / 40.0)
    q_res = np.float32(0.4) * q_out
    res = rng.integers(-128, 128, (g1.N, Ho, Wo, K2)).astype(np.int8) if with_res else None
    mid = orc.requant(orc.conv_i8(g1, x, w1, b1), orc.requant_scale(q_x, q_w1, q_mid), True)
    want = orc.requant(orc.conv_i8(g2, mid, w2, b2), orc.requant_scale(q_mid, q_w2, q_out), relu2,
                       res, orc.residual_scale(q_res, q_out) if with_res else 0.0)
    assert 0.02 < np.mean(mid != 0) and np.mean(np.abs(want.astype(int)) >= 127) < 0.5

    d1 = B.ConvDesc(g1.N, g1.H, g1.W, g1.C, g1.K, g1.R, g1.S, g1.stride_h, g1.stride_w, g1.pad_h,
                    g1.pad_w, relu=1)
    d2 = B.ConvDesc(g1.N, Ho, Wo, g1.K, K2, 1, 1, relu=int(relu2))
    assert B.conv_pair_supported(d1, d2)
    got = B.conv_pair_int8(d1, dev(x), B.pack_weights(d1, dev(w1)), dev(b1), float(q_x), float(q_w1),
                           float(q_mid), d2, B.pack_weights(d2, dev(w2)), dev(b2), float(q_w2),
                           float(q_out), None if res is None else dev(res), float(q_res))
    assert np.array_equal(host(got), want)
    # and the two launches it replaces give the same
    mid_g = B.conv_int8(d1, dev(x), B.pack_weights(d1, dev(w1)), dev(b1), float(q_x), float(q_w1),
                        float(q_mid))
    two = B.conv_int8(d2, mid_g, B.pack_weights(d2, dev(w2)), dev(b2), float(q_mid), float(q_w2),
                      float(q_out), None if res is None else dev(res), float(q_res))
    assert np.array_equal(host(two), want)


REAL_OUTPUT_CASES = [
    # geometry, residual, ReLU, extra channels of the output tensor, channel offset
    (dict(N=2, H=14, W=14, C=64, K=160, R=3, S=3, pad_h=1, pad_w=1), True, True, 0, 0),
    (dict(N=2, H=7, W=7, C=512, K=256, R=1, S=1), True, True, 0, 0),          # complete tiles
    (dict(N=1, H=19, W=19, C=64, K=84, R=3, S=3, pad_h=1, pad_w=1), False, False, 0, 0),  # SSD head
    (dict(N=1, H=17, W=17, C=48, K=72, R=1, S=7, pad_w=3), False, True, 12, 4),
    (dict(N=2, H=9, W=9, C=16, K=17, R=3, S=3, pad_h=1, pad_w=1), True, False, 5, 3),  # K <= 32: a channel tile mostly beyond K
    (dict(N=64, H=1, W=1, C=2048, K=1000, R=1, S=1), False, False, 0, 0),     # classifier logits
    (dict(N=0, H=5, W=5, C=16, K=16, R=1, S=1), False, False, 0, 0),
]


@pytest.mark.parametrize("geom,with_res,relu,out_pad,out_off", REAL_OUTPUT_CASES)
def test_conv_real_valued_output(B, geom, with_res, relu, out_pad, out_off):
    """A layer that leaves the quantised domain writes fp32 directly: the same bits as the
    oracle's fixed fp32 sequence (well inside the 1e-5 relative bound)."""
    g = orc.ConvGeom(**geom)
    rng = np.random.default_rng(g.K * 7 + g.C)
    x = rng.integers(-128, 128, (g.N, g.H, g.W, g.C)).astype(np.int8)
    w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, g.K).astype(np.int32)
    q_x, q_w, q_res = np.float32(0.021), np.float32(0.0017), np.float32(0.083)
    Ho, Wo = g.Ho, g.Wo
    res = rng.integers(-128, 128, (g.N, Ho, Wo, g.K)).astype(np.int8) if with_res else None
    out_cs = g.K + out_pad
    want = np.full((g.N, Ho, Wo, out_cs), np.float32(-7.5))
    if g.N:
        acc_o = orc.conv_i8(g, x, w, b)
        orc.real_output(acc_o, q_x, q_w, relu, res, q_res, out=want, out_c_stride=out_cs,
                        out_c_off=out_off)
    d = B.ConvDesc(g.N, g.H, g.W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w,
                   g.dil_h, g.dil_w, relu=int(relu), out_c_stride=out_cs, out_c_off=out_off)
    out = torch.full((g.N, Ho, Wo, out_cs), -7.5, dtype=torch.float32, device="cuda")
    B.conv_int8_real_output(d, dev(x), B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w),
                            None if res is None else dev(res), float(q_res), out=out)
    got = host(out)
    assert np.array_equal(got, want)
    if g.N:
        # and it is the value the int8 tail would have quantised: D(Q(y')) is within q/2 of it
        q_out = np.float32(np.abs(want[..., out_off:out_off + g.K]).max() / 127)
        z = orc.requant(acc_o, orc.requant_scale(q_x, q_w, q_out), relu, res,
                        orc.residual_scale(q_res, q_out) if with_res else 0.0)
        err = np.abs(orc.D(z, q_out) - want[..., out_off:out_off + g.K])
        assert err.max() <= 0.5001 * q_out


@pytest.mark.parametrize("xv,wv", [(-128, -128), (127, -128), (-128, 127), (0, 0)])
def test_conv_extreme_and_degenerate_values(B, xv, wv):
    """Constant tensors at the ends of the int8 range with the longest reduction of the
    benchmark networks (R*S*C = 4608): accumulators of +-7.5e7, beyond 2^24, so the int32 ->
    fp32 conversion of the epilogue rounds; and all-zero operands (the output is the bias)."""
    g = orc.ConvGeom(N=1, H=9, W=9, C=512, K=80, R=3, S=3, pad_h=1, pad_w=1)
    x = np.full((1, 9, 9, 512), xv, np.int8)
    w = np.full((80, 3, 3, 512), wv, np.int8)
    b = (np.arange(80, dtype=np.int32) - 40) * 1001
    acc_o = orc.conv_i8(g, x, w, b)
    if xv and wv:
        assert np.abs(acc_o).max() > 2**24
    q_x, q_w = np.float32(0.013), np.float32(0.0021)
    q_out = np.float32(float(q_x) * float(q_w) * max(float(np.abs(acc_o).max()), 1.0) / 100.0)
    want = orc.requant(acc_o, orc.requant_scale(q_x, q_w, q_out), False)
    d = B.ConvDesc(1, 9, 9, 512, 80, 3, 3, pad_h=1, pad_w=1)
    dump = torch.zeros(acc_o.shape, dtype=torch.int32, device="cuda")
    got = B.conv_int8(d, dev(x), B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w),
                      float(q_out), acc_dump=dump)
    assert np.array_equal(host(dump), acc_o)
    assert np.array_equal(host(got), want)
    got = B.conv_int8(d, dev(x), B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w),
                      float(q_out))                      # the fast epilogue
    assert np.array_equal(host(got), want)


def test_conv_near_the_32_bit_offset_limit(B):
    """An activation tensor of just under 2 GiB (the kernels' 32-bit offsets end there): a
    3x3 layer over it, checked on sampled output pixels (first, last, image borders, random)
    whose 3x3 neighbourhoods the oracle convolves one by one."""
    N, H, W, C, K = 8, 2044, 2044, 64, 64
    assert 2**31 - 2**24 < N * H * W * C < 2**31
    gen = torch.Generator(device="cuda").manual_seed(1805)
    x = torch.randint(-128, 128, (N, H, W, C), dtype=torch.int8, device="cuda", generator=gen)
    rng = np.random.default_rng(8691)
    w = rng.integers(-128, 128, (K, 3, 3, C)).astype(np.int8)
    b = rng.integers(-20000, 20000, K).astype(np.int32)
    q_x, q_w = np.float32(0.021), np.float32(0.0017)
    q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(9 * C) / 40.0)
    d = B.ConvDesc(N, H, W, C, K, 3, 3, pad_h=1, pad_w=1, relu=1)
    y = B.conv_int8(d, x, B.pack_weights(d, dev(w)), dev(b), float(q_x), float(q_w), float(q_out))
    picks = [(0, 0, 0), (N - 1, H - 1, W - 1), (N - 1, H - 1, 0), (N - 1, 0, W - 1), (3, 1000, 0),
             (7, 2043, 1022)]
    picks += [tuple(int(v) for v in (rng.integers(0, N), rng.integers(0, H), rng.integers(0, W)))
              for _ in range(58)]
    # the 3x3 neighbourhood of each picked pixel, zeros outside the image
    nb = np.zeros((len(picks), 3, 3, C), np.int8)
    for i, (n, h, ww) in enumerate(picks):
        for r in range(3):
            for s2 in range(3):
                hi, wi = h - 1 + r, ww - 1 + s2
                if 0 <= hi < H and 0 <= wi < W:
                    nb[i, r, s2] = host(x[n, hi, wi])
    g1 = orc.ConvGeom(N=len(picks), H=3, W=3, C=C, K=K, R=3, S=3)
    want = orc.requant(orc.conv_i8(g1, nb, w, b), orc.requant_scale(q_x, q_w, q_out), True)
    got = np.stack([host(y[n, h, ww]) for n, h, ww in picks])
    assert np.array_equal(got, want.reshape(len(picks), K))
    assert len(np.unique(want)) > 32


@pytest.mark.parametrize("out_pad,out_off", [(16, 0), (16, 16), (36, 4), (7, 3)])
def test_conv_channel_slice_of_concat(B, out_pad, out_off):
    geom = dict(N=2, H=9, W=9, C=32, K=40, R=3, S=3, pad_h=1, pad_w=1)
    _run_conv_case(B, geom, relu=True, with_res=False, with_bias=True, seed=5,
                   out_pad=out_pad, out_off=out_off)


def test_conv_input_channel_stride(B):
    # a conv that reads the first 32 channels of a 48-channel tensor
    rng = np.random.default_rng(3)
    g = orc.ConvGeom(N=2, H=10, W=10, C=32, K=32, R=3, S=3, pad_h=1, pad_w=1, in_c_stride=48)
    x = rng.integers(-128, 128, (2, 10, 10, 48)).astype(np.int8)
    w = rng.integers(-128, 128, (32, 3, 3, 32)).astype(np.int8)
    acc_o = orc.conv_i8(g, x, w)
    d = B.ConvDesc(2, 10, 10, 32, 32, 3, 3, pad_h=1, pad_w=1, in_c_stride=48)
    dump = torch.zeros((2, 10, 10, 32), dtype=torch.int32, device="cuda")
    B.conv_int8(d, dev(x), B.pack_weights(d, dev(w)), None, 1.0, 1.0, 1000.0, acc_dump=dump)
    assert np.array_equal(host(dump), acc_o)


def test_conv_batch_elements_are_independent(B):
    rng = np.random.default_rng(4)
    x = rng.integers(-128, 128, (5, 14, 14, 64)).astype(np.int8)
    w = rng.integers(-128, 128, (64, 3, 3, 64)).astype(np.int8)
    d5 = B.ConvDesc(5, 14, 14, 64, 64, 3, 3, pad_h=1, pad_w=1, relu=1)
    d1 = B.ConvDesc(1, 14, 14, 64, 64, 3, 3, pad_h=1, pad_w=1, relu=1)
    wp = B.pack_weights(d5, dev(w))
    full = host(B.conv_int8(d5, dev(x), wp, None, 0.02, 0.002, 0.08))
    for i in (0, 2, 4):
        one = host(B.conv_int8(d1, dev(x[i:i + 1]), wp, None, 0.02, 0.002, 0.08))
        assert np.array_equal(one[0], full[i])


@pytest.mark.parametrize("shape,win", [((2, 23, 23, 64), (3, 2, 1)), ((1, 10, 9, 48), (2, 2, 0)),
                                       ((2, 11, 11, 6), (3, 2, 1)), ((1, 19, 19, 32), (3, 1, 1))])
def test_maxpool_helper(B, shape, win):
    R, stride, pad = win
    rng = np.random.default_rng(sum(shape))
    x = rng.integers(-128, 128, shape).astype(np.int8)
    Ho = (shape[1] + 2 * pad - R) // stride + 1
    Wo = (shape[2] + 2 * pad - R) // stride + 1
    got = host(B.maxpool_i8(dev(x), R, R, stride, pad, Ho, Wo))
    assert np.array_equal(got, orc.maxpool_i8(x, R, R, stride, pad, Ho, Wo))


# ------------------------------------------------------------------ whole configurations
@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("shape,win,m,slice_", [
    ((2, 35, 35, 192), (3, 1, 1), 1.0, (0, 0)),        # Inception pooled branch
    ((1, 17, 17, 768), (3, 2, 0), 0.73, (1280, 512)),  # into a concatenation, rescaled
    ((2, 9, 10, 20), (2, 2, 0), 1.9, (23, 3)),         # odd widths, saturating scale
    ((1, 8, 8, 3), (8, 8, 0), 1.0, (0, 0)),            # whole-image window
    ((1, 19, 19, 64), (3, 1, 1), 0.5, (64, 0)),        # ties of .5 after the scale
])
def test_pool_i8(B, mode, shape, win, m, slice_):
    rng = np.random.default_rng(sum(shape) + win[0])
    x = rng.integers(-128, 128, size=shape, dtype=np.int8)
    R, stride, pad = win
    Ho = (shape[1] + 2 * pad - R) // stride + 1
    Wo = (shape[2] + 2 * pad - R) // stride + 1
    Cd, off = slice_
    Cd = Cd or shape[3]
    base = rng.integers(-128, 128, size=(shape[0], Ho, Wo, Cd), dtype=np.int8)
    # the library forms the rescale itself from the two factors, one fp32 division
    q_out = np.float32(0.0071)
    q_in = np.float32(m) * q_out
    m_used = orc.residual_scale(q_in, q_out)
    assert abs(float(m_used) - m) <= 1e-6 * m
    want = orc.pool_i8(x, mode, R, R, stride, pad, Ho, Wo, m_used, out=base.copy(), out_c_off=off)
    got = B.pool_i8(dev(x), mode, R, R, stride, pad, Ho, Wo, float(q_in), float(q_out),
                    out=dev(base), out_c_off=off)
    assert np.array_equal(host(got), want)


@pytest.mark.parametrize("shape,C,K,pad,ceil,slice_", [
    ((1, 299, 301), 64, 64, 1, False, (64, 0)),    # odd maps, rests of blocks in both directions
    ((1, 299, 301), 64, 48, 1, True, (80, 16)),    # the last windows hold one row and column; into a slice
    ((5, 149, 163), 32, 64, 1, True, (64, 0)),
    ((2, 149, 151), 32, 32, 0, False, (32, 0)),    # 16 x 16 blocks
    ((3, 149, 151), 64, 144, 1, True, (176, 16)),  # several channel tiles, the last with 16 of 64
    ((5, 149, 163), 32, 96, 1, False, (96, 0)),
    ((1, 299, 301), 128, 80, 1, False, (80, 0)),
    ((1, 299, 301), 128, 80, 0, True, (112, 16)),
    ((3, 149, 167), 80, 144, 0, False, (144, 0)),  # filters and patches of less than their rows
    ((2, 149, 167), 96, 80, 1, True, (80, 0)),
])
def test_maximum_behind_a_layer(B, shape, C, K, pad, ceil, slice_):
    """The block-tiled 3x3 kernel with the 2x2 maximum in its launch: both tensors as by two calls, nothing
    beside them; a maximum that writes over the layer's input goes behind it."""
    import ctypes
    N, H, W = shape
    rng = np.random.default_rng(H * W + C + K)
    Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
    Hp, Wp = (Ho + ceil) // 2, (Wo + ceil) // 2
    cs, off = slice_
    x = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8)
    z_w = rng.integers(-128, 128, (K, 3, 3, C)).astype(np.int8)
    bias = rng.integers(-2000, 2000, K).astype(np.int32)
    g = orc.ConvGeom(N=N, H=H, W=W, C=C, K=K, R=3, S=3, pad_h=pad, pad_w=pad)
    q_x, q_w, q_out = 0.02, 0.01 / np.sqrt(9.0 * C), 0.011
    d = B.ConvDesc(N, H, W, C, K, 3, 3, 1, 1, pad, pad, 1, 1)
    assert B.conv_variant(d) == "conv_i8_p3b_kernel"
    want = orc.conv_layer_i8(g, x, q_x, z_w, q_w, bias, q_out, 0)[0]
    pooled = np.full((N, Hp, Wp, cs), 77, np.int8)
    pooled = orc.pool_i8(want, "max", 2, 2, 2, 0, Hp, Wp, np.float32(1), out=pooled, out_c_off=off)
    wp, b = B.pack_weights(d, dev(z_w)), dev(bias)
    streams = (ctypes.c_void_p * 1)(torch.cuda.current_stream().cuda_stream)
    for apart in (True, False):
        xd = dev(x)
        if not apart and xd.numel() < pooled.size:
            continue
        y = torch.full((N, Ho, Wo, K), 77, dtype=torch.int8, device="cuda")
        z = torch.full(pooled.shape, 77, dtype=torch.int8, device="cuda")
        ops = (B.Op * 2)()
        o = ops[0]
        o.kind, o.d, o.x, o.w, o.bias, o.y = B.OP_CONV, d, xd.data_ptr(), wp.data_ptr(), b.data_ptr(), y.data_ptr()
        o.q_x, o.q_w, o.q_out, o.group = q_x, q_w, q_out, 1
        o = ops[1]
        o.kind = B.OP_POOL
        o.x, o.y = y.data_ptr(), (z if apart else xd).data_ptr()
        o.d.N, o.H, o.W, o.C = N, Ho, Wo, K
        o.R = o.S = o.stride = 2
        o.Ho, o.Wo, o.q_x, o.q_out, o.group = Hp, Wp, q_out, q_out, 2
        o.d.out_c_stride, o.d.out_c_off = cs, off
        assert B.lib.q8_joined_op(ops, 2, streams, 1, 0) == (1 if apart else -1)
        assert B.lib.q8_run_ops(ops, 2, streams, 1) == 0
        assert np.array_equal(host(y), want)
        if apart and cs == K:              # the same as a call without a factor
            o.kind, o.y = B.OP_MAXPOOL, z.fill_(77).data_ptr()
            y.fill_(77)
            assert B.lib.q8_joined_op(ops, 2, streams, 1, 0) == 1
            assert B.lib.q8_run_ops(ops, 2, streams, 1) == 0
            assert np.array_equal(host(y), want)
        got = host(z if apart else xd.flatten()[:pooled.size].view(pooled.shape))
        assert np.array_equal(got[..., off:off + K], pooled[..., off:off + K])
        if apart:
            assert np.array_equal(got, pooled)


@pytest.mark.parametrize("case", ["one stream, two indices", "default stream", "refused", "two streams",
                                  "leads a group"])
def test_maximum_and_ops_of_other_streams(B, case):
    """Layers and the maxima over their outputs with ops of other streams between the two: what the list's order
    says where that binds the streams, nothing behind a refused op, and every tensor as by single calls."""
    import ctypes
    N, H, W, C, pairs = 2, 149, 163, 64, 10 if case == "two streams" else 1
    d = B.ConvDesc(N, H, W, C, C, 3, 3, 1, 1, 1, 1, relu=1)
    assert B.conv_variant(d) == "conv_i8_p3b_kernel"
    def codes(*shape):
        return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda")
    w = B.pack_weights(d, codes(C, 3, 3, C))
    x = [codes(N, H, W, C) for _ in range(pairs)]
    other = codes(N, H, W, C)
    y = [torch.full((N, H, W, C), 77, dtype=torch.int8, device="cuda") for _ in x]
    z = [torch.full((N, H // 2, W // 2, C), 77, dtype=torch.int8, device="cuda") for _ in x]
    want = [B.conv_int8(d, t, w, None, 0.02, 0.0004, 0.011) for t in x]

    def conv(i, stream):
        o = B.Op()
        o.kind, o.d, o.stream, o.x, o.w, o.y = B.OP_CONV, d, stream, x[i].data_ptr(), w.data_ptr(), y[i].data_ptr()
        o.q_x, o.q_w, o.q_out = 0.02, 0.0004, 0.011
        return o

    def maximum(src, dst, win, stream):
        o = B.Op()
        o.kind, o.stream, o.x, o.y = B.OP_MAXPOOL, stream, src.data_ptr(), dst.data_ptr()
        o.d.N, o.H, o.W, o.C, o.R, o.S, o.stride, o.Ho, o.Wo = N, H, W, C, win, win, win, H // max(win, 1), W // max(win, 1)
        return o
    torch.cuda.synchronize()
    if case == "two streams":
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        handles, ops = [s.cuda_stream for s in streams], []
        for i in range(pairs):             # conv 0, conv 1, maximum 1, maximum 0, conv 3, ...
            ops += [conv(i, 0)] if i % 2 == 0 else [conv(i, 1), maximum(y[i], z[i], 2, 1), maximum(y[i - 1], z[i - 1], 2, 0)]
        joined = 3
    elif case == "leads a group":          # of two maxima, the other of which stays behind
        handles, more = [torch.cuda.Stream().cuda_stream] * 2, torch.empty_like(z[0])
        ops, joined = [conv(0, 0), maximum(y[0], z[0], 2, 0), maximum(other, more, 2, 0)], 1
        ops[1].group = ops[2].group = 3
    elif case == "refused":
        handles = [torch.cuda.Stream().cuda_stream, torch.cuda.Stream().cuda_stream]
        ops, joined = [conv(0, 0), maximum(other, other, 0, 1), maximum(y[0], z[0], 2, 0)], 2
    else:                                  # a copy over the layer's output between the layer and its maximum
        handles = [torch.cuda.Stream().cuda_stream] * 2
        if case == "default stream":       # ordered with every stream that does not say otherwise
            hip, made = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
            assert hip.hipStreamCreate(ctypes.byref(made)) == 0
            handles = [made.value, None]
        ops, joined = [conv(0, 0), maximum(other, y[0], 1, 1), maximum(y[0], z[0], 2, 0)], -1
    array, streams = (B.Op * len(ops))(*ops), (ctypes.c_void_p * 2)(*handles)
    code = B.lib.q8_run_ops(array, len(ops), streams, 2)
    torch.cuda.synchronize()
    if case == "refused":
        assert code == -1 and np.array_equal(host(y[0]), host(want[0])) and (host(z[0]) == 77).all()
    elif case in ("two streams", "leads a group"):
        assert code == 0
        if case == "leads a group":
            assert np.array_equal(host(more), host(B.maxpool_i8(other, 2, 2, 2, 0, H // 2, W // 2)))
        for a, b, c in zip(y, want, z):
            assert np.array_equal(host(a), host(b))
            assert np.array_equal(host(c), host(B.maxpool_i8(b, 2, 2, 2, 0, H // 2, W // 2)))
    else:
        assert code == 0 and np.array_equal(host(y[0]), host(other))
        assert np.array_equal(host(z[0]), host(B.maxpool_i8(other, 2, 2, 2, 0, H // 2, W // 2)))
    assert B.lib.q8_joined_op(array, len(ops), streams, 2, 0) == joined


@pytest.mark.parametrize("m", [1.0, 0.37])
@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("shape,win,extra", [
    ((1, 1, 1, 16), (3, 1, 1), 0), ((2, 2, 1, 48), (3, 1, 2), 0), ((1, 5, 6, 16), (3, 1, 0), 0),
    ((3, 7, 4, 32), (3, 1, 1), 16), ((1, 3, 3, 16), (3, 2, 2), 0), ((2, 6, 9, 48), (3, 2, 1), 0),
    ((2, 9, 8, 16), (2, 2, 0), 16), ((1, 5, 7, 32), (2, 2, 0), 1), ((1, 5, 5, 16), (3, 3, 0), 0),
    ((2, 7, 8, 32), (3, 3, 1), 16), ((1, 11, 6, 16), (3, 5, 2), 0), ((1, 6, 7, 48), (2, 1, 1), 0), ((3, 8, 9, 16), (2, 3, 1), 0),
    # two outputs a lane: many maps of one, two, an odd and an even number of columns
    ((66000, 3, 1, 16), (3, 1, 1), 0), ((35000, 3, 2, 16), (3, 1, 1), 16), ((14000, 3, 5, 16), (3, 1, 1), 0),
    ((9000, 3, 4, 16), (3, 1, 2), 0), ((40000, 4, 5, 16), (3, 1, 0), 0),
    # any other window
    ((1, 9, 7, 32), (1, 2, 0), 0), ((2, 8, 9, 16), (5, 2, 2), 16), ((1, 12, 12, 16), (11, 1, 5), 0),
])
def test_pool_i8_strips(B, shape, win, extra, mode, m):
    """Windows at every edge of the image, odd rests of a strip, a slice of a wider tensor, and one output row
    and column beyond the last whole window (extra = 1); codes at their bounds among them."""
    rng = np.random.default_rng(sum(shape) + 10 * win[0] + win[1])
    x = rng.integers(-128, 128, size=shape, dtype=np.int8)
    x[rng.random(shape) < 0.3] = -128
    x[rng.random(shape) < 0.2] = 127
    R, stride, pad = win
    Ho = (shape[1] + 2 * pad - R) // stride + 1 + extra % 2
    Wo = (shape[2] + 2 * pad - R) // stride + 1 + extra % 2
    off = extra & ~1
    base = rng.integers(-128, 128, size=(shape[0], Ho, Wo, shape[3] + off), dtype=np.int8)
    q_out = np.float32(0.013)
    q_in = np.float32(m) * q_out
    want = orc.pool_i8(x, mode, R, R, stride, pad, Ho, Wo, orc.residual_scale(q_in, q_out), out=base.copy(),
                       out_c_off=off)
    got = B.pool_i8(dev(x), mode, R, R, stride, pad, Ho, Wo, float(q_in), float(q_out), out=dev(base),
                    out_c_off=off)
    assert np.array_equal(host(got), want)
    if mode == "max" and m == 1.0:
        got = host(B.maxpool_i8(dev(x), R, R, stride, pad, Ho, Wo))
        assert np.array_equal(got, orc.maxpool_i8(x, R, R, stride, pad, Ho, Wo))


@pytest.mark.parametrize("mode,stride,shape", [("avg", 1, (3, 20, 16384, 2048)), ("avg", 2, (1, 40, 16384, 2048)),
                                               ("max", 3, (1, 70, 16384, 2048))])
def test_pool_i8_beyond_the_reach_of_a_launch(B, mode, stride, shape):
    """Tensors of more bytes than a launch's offsets reach: image by image or in bands of rows, the same as
    pieces of the padded tensor."""
    N, H, W, C = shape
    x = torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda")
    Ho, Wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    got = B.pool_i8(x, mode, 3, 3, stride, 1, Ho, Wo)
    padded = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1), value=-128 if mode == "max" else 0)
    step = 1024
    for n in range(N):
        for a in range(0, Wo, step):
            some = min(step, Wo - a)
            piece = padded[n:n + 1, :, a * stride:(a + some - 1) * stride + 3].contiguous()
            assert torch.equal(B.pool_i8(piece, mode, 3, 3, stride, 0, Ho, some), got[n:n + 1, :, a:a + some]), (n, a)


def test_pool_f32(B):
    import torch
    rng = np.random.default_rng(7)
    x = rng.standard_normal((2, 17, 15, 24)).astype(np.float32)
    xt = torch.from_numpy(x).permute(0, 3, 1, 2)
    for mode, ref in (("max", torch.nn.functional.max_pool2d(xt, 3, 2, 1)),
                      ("avg", torch.nn.functional.avg_pool2d(xt, 3, 2, 1, count_include_pad=True))):
        got = host(B.pool_f32(dev(x), mode, 3, 3, 2, 1, 9, 8))
        want = ref.permute(0, 2, 3, 1).numpy()
        assert np.allclose(got, want, rtol=1e-6, atol=1e-6), mode


# four channels a lane: slices, one pixel, a window that leaves the image, rows and images that end inside a block;
# channels and places that are no multiples of four take a value per lane
@pytest.mark.parametrize("shape,C,R,stride,pad,cs,off", [
    ((1, 1, 1), 4, 3, 1, 1, 0, 0), ((3, 17, 15), 20, 3, 2, 1, 48, 28), ((5, 9, 11), 64, 2, 2, 0, 0, 0),
    ((2, 7, 9), 12, 5, 3, 2, 24, 12), ((2, 17, 15), 6, 3, 1, 1, 0, 0), ((2, 17, 15), 8, 3, 1, 1, 19, 3)])
def test_pool_f32_builds(B, shape, C, R, stride, pad, cs, off):
    (N, H, W), g = shape, torch.Generator(device="cuda").manual_seed(C)
    Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    x = torch.randn((N, H, W, C), device="cuda", generator=g)
    for mode in ("max", "avg"):
        p = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad), value=-torch.inf if mode == "max" else 0.0)
        want = torch.full((N, Ho, Wo, C), -3.402823466e38 if mode == "max" else 0.0, device="cuda")
        for r in range(R):                      # in the kernel's order: the same sums
            for s in range(R):
                v = p[:, r:r + (Ho - 1) * stride + 1:stride, s:s + (Wo - 1) * stride + 1:stride]
                want = torch.maximum(want, v) if mode == "max" else want + v
        want = want if mode == "max" else want / torch.full((1,), float(R * R), device="cuda")
        out = torch.full((N, Ho, Wo, cs or C), -7.0, device="cuda")
        B.pool_f32(x, mode, R, R, stride, pad, Ho, Wo, out=out, out_c_off=off)
        assert torch.equal(out[..., off:off + C], want)
        assert bool((out[..., :off] == -7).all()) and bool((out[..., off + C:] == -7).all())


def _oracle_pipeline(cfg_id, batch, calib_library):
    cfg = wl.CONFIGS[cfg_id]
    net = cfg["make"]()
    params = {op.name: wl.conv_params(cfg_id, i, op) for i, op in enumerate(net.convs())}
    x = wl.input_batch(cfg_id, net, batch, 0, relu=cfg["relu_input"])
    folded = onet.fold_all(net, params)
    q = onet.calibrate(net, folded, [x], use_library=calib_library)
    qparams = onet.quantize_params(net, folded, q)
    z_in = orc.Q(x, q[net.input], 7)
    acts, accs = onet.forward_i8(net, qparams, q, z_in, keep_acc=True)
    return net, params, x, folded, q, qparams, z_in, acts, accs


def _gpu_pipeline_checks(B, cfg_id, batch, calib_library):
    from paper_1805_08691_amd.engine import Engine
    net, params, x, folded, q, qparams, z_in, acts, accs = _oracle_pipeline(
        cfg_id, batch, calib_library)
    eng = Engine(net, batch)
    eng.load_params(params)
    eng.fold()
    for name, (Wf, bf) in folded.items():          # Eq. BN: bit-exact
        assert np.array_equal(host(eng.folded[name][0]), Wf)
        assert np.array_equal(host(eng.folded[name][1]), bf)
    eng.set_factors(q)                             # frozen factor table from the oracle side
    eng.quantize_weights()
    for name, qp in qparams.items():               # q_w, int8 filters, int32 bias: bit-exact
        assert np.float32(eng.qw[name]) == qp["q_w"]
        assert np.array_equal(host(eng.zw_dense[name]), qp["z_w"])
        assert np.array_equal(host(eng.wq[name][1]), qp["z_b"])
    eng.allocate()
    xd = dev(x)
    slot = torch.zeros(1, device="cuda")           # the input factor from the GPU's own max-abs
    B.calibrate_maxabs(xd, slot)
    assert np.float32(B.qfactor(float(host(slot)[0]), 7)) == q[net.input]
    eng.quantize_input(xd)
    assert np.array_equal(host(eng.act[net.input]), z_in)
    dumps = {op.name: torch.zeros((batch, net.tensors[op.dst].H, net.tensors[op.dst].W, op.K),
                                  dtype=torch.int32, device="cuda") for op in net.convs()}
    eng.run_layers(acc_dump=dumps)
    for op in net.convs():
        assert np.array_equal(host(dumps[op.name]), accs[op.name]), op.name
        assert np.array_equal(host(eng.act[op.dst]), acts[op.dst]), op.name
    for o in net.outputs:                          # Eq. D on what leaves the int8 domain
        r = host(B.dequantize(eng.act[o], float(q[o])))
        want = orc.D(acts[o], q[o])
        assert np.all(np.abs(r - want) <= 1e-5 * np.abs(want))
        assert len(np.unique(acts[o])) > 32        # not degenerate
    return eng, net, xd, acts


def test_config1_single_conv(B):
    _gpu_pipeline_checks(B, 1, 1, calib_library=False)


def test_config2_bottleneck_block(B):
    eng, net, xd, acts = _gpu_pipeline_checks(B, 2, 32, calib_library=True)
    # the same through a captured HIP graph, replayed with eager work in between
    eng.capture(xd)
    for _ in range(3):
        for t in eng.act.values():
            if t is not eng.act[net.input]:
                t.fill_(55)
        torch.cuda.synchronize()
        eng.graph.replay()
        for o in net.outputs:
            assert np.array_equal(host(eng.act[o]), acts[o])


def test_run_step_one_and_two_pipelines_and_serial(B):
    """The step the benchmark times (quantise, layers, dequantise) gives the oracle's values
    whether the batch runs whole, as two concurrent half-batch pipelines, or as the same
    launches one pipeline after the other; an odd batch splits unevenly."""
    from paper_1805_08691_amd.engine import Engine
    cfg_id, batch = 2, 7
    net, params, x, folded, q, qparams, z_in, acts, accs = _oracle_pipeline(cfg_id, batch, True)
    o = net.outputs[0]
    want = orc.D(acts[o], q[o])
    # (left to itself a step this short runs as one pipeline)
    for n_streams, forced, serial, fuse_deq in (
            (1, False, False, False), (2, False, False, False), (2, True, False, False), (2, True, True, False),
            (3, True, False, False), (2, True, False, True), (3, True, False, True), (1, False, False, True)):
        eng = Engine(net, batch, n_streams=n_streams, fuse_dequant=fuse_deq)
        if forced:
            eng._pipelines_pay = lambda ops: True
        eng.load_params(params)
        eng.fold()
        eng.set_factors(q)
        eng.quantize_weights()
        eng.allocate()
        if n_streams == 2:
            assert eng.parts == [(0, 4), (4, 3)]
        if n_streams == 3:
            assert eng.parts == [(0, 3), (3, 2), (5, 2)]
        assert eng._plan(True, (o,))[3] == (n_streams if forced else 1)
        out = torch.full(eng.act[o].shape, -1.0, dtype=torch.float32, device="cuda")
        eng.run_step(dev(x), {o: out}, serial=serial)
        torch.cuda.synchronize()
        assert np.array_equal(host(eng.act[o]), acts[o]), (n_streams, serial)
        assert bool(eng._dequant_writer(o)) == fuse_deq
        got = host(out)
        assert np.all(np.abs(got - want) <= 1e-5 * np.abs(want)), (n_streams, serial, fuse_deq)
        assert np.array_equal(got, host(eng.dequantize(o)))       # fused or not: the same bits


@pytest.mark.parametrize("batch, pipelines", [(21, 1), (22, 1), (43, 2)])
def test_run_step_values_in_the_last_layers_launch(B, batch, pipelines):
    """A bottleneck block whose output has 2^24 values or more: Eq. D leaves with the last layer's codes, and the
    block is three launches.  One image less: the block in one launch, and Eq. D behind it."""
    from paper_1805_08691_amd.engine import Engine
    net, params, x, _, q, *_ = _oracle_pipeline(2, 2, True)
    o = net.outputs[0]
    eng = Engine(net, batch, n_streams=2)
    eng._pipelines_pay = lambda ops: pipelines == 2
    eng.load_params(params)
    eng.fold()
    eng.set_factors(q)
    eng.quantize_weights()
    eng.allocate()
    long = eng.act[o].numel() >= 1 << 24
    assert long == (batch > 20)
    segments = eng._plan(True, (o,))[0]
    assert [op.kind for op in segments[2]] == ([] if long else [B.OP_DEQUANTIZE])
    flags = [op.flags for op in segments[1]]
    assert len(flags) == 3 * pipelines
    assert sum(bool(f & B.OPF_DEQUANT) for f in flags) == (pipelines if long else 0)
    assert sum(bool(f & B.OPF_BLOCK) for f in flags) == (0 if long else pipelines)
    batches = dev(np.concatenate([x] * (batch // 2 + 1))[:batch])
    batches *= torch.linspace(0.2, 1.0, batch, device="cuda").view(-1, 1, 1, 1)
    got = []
    for serial in (True, False):
        eng.act[o].fill_(55)
        out = torch.full(eng.act[o].shape, -7.0, device="cuda")
        eng.run_step(batches, {o: out}, serial=serial)
        torch.cuda.synchronize()
        got.append((eng.act[o].clone(), out))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[1][1], got[1][0].float() * torch.full((1,), q[o], device="cuda"))
    assert len(torch.unique(got[1][0])) > 16


def test_run_step_values_of_a_layer_in_no_block(B):
    """A 1x1 layer that ends no block writes its values beside the codes at any size of its family."""
    from paper_1805_08691_amd.engine import Engine
    net = wl.Network("wide", "x")
    net.tensor("x", 40, 40, 64)
    net.tensor("y", 40, 40, 256)
    wl._conv(net, "a", "x", 256, 1, 1, dst="y")
    net.outputs = ["y"]
    eng = Engine(net, 8)
    eng.load_params({op.name: wl.conv_params(2, i, op) for i, op in enumerate(net.convs())})
    eng.fold()
    x = torch.randn((8, 40, 40, 64), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    eng.calibrate([x])
    eng.quantize_weights()
    eng.allocate()
    segments = eng._plan(True, ("y",))[0]
    assert [op.flags for op in segments[1]] == [B.OPF_DEQUANT] and not segments[2]
    out = torch.empty(eng.act["y"].shape, device="cuda")
    eng.run_step(x, {"y": out})
    values, codes = out.clone(), eng.act["y"].clone()
    eng.run_step(x, {"y": out}, serial=True)
    assert torch.equal(values, out) and torch.equal(codes, eng.act["y"]) and len(torch.unique(codes)) > 16


def test_planned_step_follows_the_engine(B):
    """The planned step equals the layer-by-layer one (``serial``) with the pipelines forced, after
    a factor was set between two steps, and for a batch longer than the engine's."""
    from paper_1805_08691_amd.engine import Engine
    net, params, x, folded, q, *_ = _oracle_pipeline(2, 7, True)
    o = net.outputs[0]
    for n_streams in (1, 2, 3):
        eng = Engine(net, 7, n_streams=n_streams)
        eng._pipelines_pay = lambda ops: True
        eng.load_params(params)
        eng.fold()
        eng.set_factors(q)
        eng.quantize_weights()
        eng.allocate()
        out = torch.empty(eng.act[o].shape, dtype=torch.float32, device="cuda")
        longer = torch.cat([dev(x), dev(x[:1])])
        for factor, batch in ((1.0, dev(x)), (2.0, dev(x)), (1.0, longer)):
            eng.q[o] = q[o] * factor
            got = []
            for serial in (True, False):
                eng.act[o].fill_(55)
                eng.run_step(batch, {o: out}, serial=serial)
                torch.cuda.synchronize()
                got.append((host(eng.act[o]).copy(), host(out).copy()))
            assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
            assert len(np.unique(got[1][0])) > 16


@pytest.mark.parametrize("fuse_dequant", [False, True])
def test_planned_step_and_other_output_buffers(B, fuse_dequant):
    """Buffers longer than the batch, flattened ones and ones whose images lie apart take the
    dequantised batch as they do layer by layer (``serial``); shorter ones are refused."""
    from paper_1805_08691_amd.engine import Engine
    net, params, x, folded, q, *_ = _oracle_pipeline(2, 2, True)
    o = net.outputs[0]
    for batch, n_streams in ((2, 1), (2, 2), (1, 1)):
        eng = Engine(net, batch, n_streams=n_streams, fuse_dequant=fuse_dequant)
        eng._pipelines_pay = lambda ops: True
        eng.load_params(params)
        eng.fold()
        eng.set_factors(q)
        eng.quantize_weights()
        eng.allocate()
        N, H, W, K = eng.act[o].shape
        want = torch.empty((N, H, W, K), device="cuda")
        eng.run_step(dev(x[:N]), {o: want}, serial=True)
        buffers = [torch.full((N + 3, H, W, K), -7.0, device="cuda")]
        if not fuse_dequant:
            buffers.append(torch.full((N * H * W * K,), -7.0, device="cuda"))
        if N == 1:
            buffers.append(torch.full((3, 2, H, W, K), -7.0, device="cuda")[:, 0])
        for out in buffers:
            eng.run_step(dev(x[:N]), {o: out})
            torch.cuda.synchronize()
            got = out if out.dim() == 1 else out[:N]
            assert torch.equal(got.reshape(want.shape), want)
            assert out.dim() == 1 or bool((out[N:] == -7).all())
        with pytest.raises(ValueError):
            eng.run_step(dev(x[:N]), {o: torch.empty((N, H, W, K - 1), device="cuda")})
        if N > 1 and n_streams == 1:            # images that lie apart are refused, as before
            with pytest.raises(AssertionError):
                eng.run_step(dev(x[:N]), {o: torch.empty((N, 2, H, W, K), device="cuda")[:, 0]})


def test_fused_head_takes_images_that_lie_apart(B):
    """Each pipeline's part of the batch has to be contiguous, the batch has not."""
    from paper_1805_08691_amd.engine import Engine
    net = wl.resnet50(image=160)
    eng = Engine(net, 2, n_streams=2, fuse_head=True)
    assert eng.head
    eng.load_params({op.name: wl.conv_params(3, i, op) for i, op in enumerate(net.convs())})
    eng.fold()
    x = dev(wl.input_batch(3, net, 2))
    eng.calibrate([x])
    eng.quantize_weights()
    eng.allocate()
    o = net.outputs[0]
    eng.run_step(x)
    want = eng.act[o].clone()
    eng.act[o].fill_(55)
    apart = torch.stack([x, x + 1], 1)[:, 0]
    assert not apart.is_contiguous()
    eng.run_step(apart)
    assert torch.equal(eng.act[o], want) and len(torch.unique(want)) > 16


def test_planned_step_follows_other_buffers(B):
    """A program may put other filters, factors of them and buffers in the place of the engine's:
    the planned step takes them, as the layer-by-layer one (``serial``) does."""
    from paper_1805_08691_amd.engine import Engine
    net, params, x, folded, q, *_ = _oracle_pipeline(2, 7, True)
    o, name = net.outputs[0], net.convs()[-1].name
    eng = Engine(net, 7)
    eng.load_params(params)
    eng.fold()
    eng.set_factors(q)
    eng.quantize_weights()
    eng.allocate()
    out, codes = torch.empty(eng.act[o].shape, dtype=torch.float32, device="cuda"), []
    (packed, bias), q_w = eng.wq[name], eng.qw[name]
    for filters, factor in ((packed, q_w), (torch.flip(packed, (0,)), q_w), (packed, 2 * q_w)):
        eng.wq[name], eng.qw[name] = (filters, bias), factor
        eng.act[o] = torch.full_like(eng.act[o], 55)
        got = []
        for serial in (False, True):
            eng.run_step(dev(x), {o: out}, serial=serial)
            torch.cuda.synchronize()
            got.append((host(eng.act[o]).copy(), host(out).copy()))
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
        codes.append(got[0][0])
    assert not np.array_equal(codes[0], codes[1]) and not np.array_equal(codes[0], codes[2])


def _sampled_images_check(B, cfg_id, batch, picks, n_cal, cal_batch, n_streams=2, unsigned=False,
                          per_channel=False, real_outputs=False, own_sum_factor=False,
                          fuse_pairs=False, chain=False, chain_variants=None, fuse_duals=False,
                          fuse_head=False):
    """Whole network at ``batch`` in the launch configuration the benchmark times; the
    oracle evaluates the images in ``picks`` (batch elements are independent once the
    factor table is frozen) and every tensor of the chain is compared bit for bit."""
    from paper_1805_08691_amd.engine import Engine
    net = wl.CONFIGS[cfg_id]["make"]()
    params = {op.name: wl.conv_params(cfg_id, i, op) for i, op in enumerate(net.convs())}
    folded = onet.fold_all(net, params)
    U = onet.unsigned_tensors(net) if unsigned else set()
    q = onet.calibrate(net, folded, (wl.input_batch(cfg_id, net, cal_batch, 100 + i)
                                     for i in range(n_cal)), unsigned=U,
                       own_sum_factor=own_sum_factor)
    qparams = onet.quantize_params(net, folded, q, per_channel=per_channel)
    x = wl.input_batch(cfg_id, net, batch, 0)
    z_in = orc.Q(x[picks], q[net.input], 7)
    plain = not (unsigned or per_channel or real_outputs or own_sum_factor)
    if plain:
        acts, accs = onet.forward_i8(net, qparams, q, z_in, keep_acc=True)
    else:
        acts = onet.forward_i8(net, qparams, q, z_in, unsigned=U)

    def codes(name, a):       # the GPU's bytes as the oracle's codes
        return (a.astype(np.int16) + 128).astype(np.uint8) if name in U else a

    eng = Engine(net, batch, n_streams=n_streams, unsigned_activations=unsigned,
                 per_channel_weights=per_channel, real_outputs=real_outputs,
                 fuse_pairs=fuse_pairs, chain=chain, fuse_duals=fuse_duals, fuse_head=fuse_head)
    assert bool(eng.head) == fuse_head
    assert bool(eng.duals) == fuse_duals
    assert eng.unsigned == U
    assert bool(eng.pairs) == fuse_pairs
    unwritten = {op.dst for op in net.convs() if op.name in eng.pairs}   # stay on chip
    if eng.head and eng.head[1]:
        unwritten.add(eng.head[0].dst)       # pooled inside the first layer's launch
    # outputs that leave the quantised domain as fp32 straight from their convolution
    real_want = {}
    if real_outputs:
        assert eng.real, "this network has no output a convolution writes whole"
        for op in net.convs():
            if op.dst in eng.real:
                qp = qparams[op.name]
                acc = orc.conv_i8(onet.geom(op, net.tensors, len(picks)), acts[op.src], qp["z_w"],
                                  qp["z_b"])
                real_want[op.dst] = orc.real_output(
                    acc, q[op.src], qp["q_w"], op.relu, acts[op.res] if op.res else None,
                    q[op.res] if op.res else 0.0)
    eng.load_params(params)
    eng.fold()
    eng.set_factors(q)
    eng.quantize_weights()
    for name, qp in qparams.items():
        if per_channel:
            assert np.array_equal(host(eng.qw[name]), qp["q_w"]), name
        else:
            assert np.float32(eng.qw[name]) == qp["q_w"], name
        bias = host(eng.wq[name][1])
        if name in eng.taps:       # reads unsigned codes: 128 * (filter sum) is folded in
            bias = bias - 128 * qp["z_w"].astype(np.int64).reshape(bias.size, -1).sum(axis=1)
        assert np.array_equal(bias, qp["z_b"]), name
    xd = dev(x)
    if chain:
        eng.allocate()
        chains = eng.build_chains(chain_variants)
        assert chains, "no run of chainable layers in this network"
    outs = eng.forward(xd)
    if chain:
        torch.cuda.synchronize()
        assert [c.status() for _, _, c in eng.chains] == [0] * len(eng.chains)
    if eng.head:
        # the head's launches quantised the image on the way in; the stand-alone Eq. Q (which
        # the small-batch check below starts from) is checked here all the same
        assert not host(eng.act[net.input]).any()
        eng.quantize_input(xd)
    zi = host(eng.input_codes())
    if z_in.shape[-1] == 3:              # an image: stored with a zero fourth channel
        assert np.array_equal(zi[picks][..., :3], z_in) and np.all(zi[..., 3] == 0)
    else:
        assert np.array_equal(zi[picks], z_in)
    if eng.in_frame:                     # the frame around the image holds zeros
        top, left = eng.in_frame[:2]
        full = host(eng.act[net.input])
        assert not full[:, :top].any() and not full[:, top + z_in.shape[1]:].any()
        assert not full[:, :, :left].any() and not full[:, :, left + z_in.shape[2]:].any()
    for op in net.ops:
        if op.dst in eng.real or op.dst in unwritten:
            continue
        got = codes(op.dst, host(eng.act[op.dst])[picks])
        assert got.dtype == acts[op.dst].dtype and np.array_equal(got, acts[op.dst]), op.name
    for o, out in zip(net.outputs, outs):
        r = host(eng.dequantize(o))[picks]
        if o in eng.real:
            assert np.array_equal(r, real_want[o]), o
            # the int8 path's D(Q(.)) of the same value is within half a step of it
            # (where the int8 range holds it)
            inside = np.abs(r) <= 127 * q[o]
            assert np.all(np.abs(orc.D(acts[o], q[o]) - r)[inside] <= 0.5001 * q[o]), o
            continue
        want = orc.D_u8(acts[o], q[o]) if o in U else orc.D(acts[o], q[o])
        assert np.all(np.abs(r - want) <= 1e-5 * np.abs(want)), o
    if plain and not chain:
        # the int32 accumulators of every layer on the sampled images (run as a small batch of
        # their own from the same int8 input codes), against the oracle's
        small = Engine(net, len(picks), fuse_pairs=fuse_pairs)
        small.load_params(params)
        small.fold()
        small.set_factors(q)
        small.quantize_weights()
        small.allocate()
        small.input_codes().copy_(eng.input_codes()[picks])
        dumps = {op.name: torch.zeros((len(picks), net.tensors[op.dst].H, net.tensors[op.dst].W,
                                       op.K), dtype=torch.int32, device="cuda")
                 for op in net.convs()}
        some = {k: v for i, (k, v) in enumerate(dumps.items()) if i % 2 == 0} if fuse_pairs else dumps
        small.run_layers(acc_dump=some)
        for name in some:
            assert np.array_equal(host(dumps[name]), accs[name]), name
        for op in net.ops:
            assert np.array_equal(host(small.act[op.dst]), acts[op.dst]), op.name
        del small, dumps
    # replays of the captured HIP graph, with eager work between them: same bits each time
    eng.capture(xd)
    for rep in range(3):
        for o in net.outputs:
            eng.act[o].fill_(3 + rep)
        torch.cuda.synchronize()
        for o in eng.real:
            eng.act_f32[o].fill_(3 + rep)
        eng.graph.replay()
        for o in net.outputs:
            if o in eng.real:
                assert np.array_equal(host(eng.act_f32[o])[picks], real_want[o]), (o, rep)
            else:
                assert np.array_equal(codes(o, host(eng.act[o])[picks]), acts[o]), (o, rep)


@pytest.mark.parametrize("n_streams", [2, 1])
def test_config3_resnet50_batch64_sampled_images(B, n_streams):
    # n_streams = 2 is the launch configuration the benchmark times (two half-batch
    # pipelines); images 31 and 32 sit on either side of the split
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=8, cal_batch=8, n_streams=n_streams)


def test_resnet50_unsigned_activations(B):
    # ResNet-50 with unsigned p = 8 codes on every ReLU output (the paper's precision for
    # non-negative activations), batch 64 in the benchmark's launch configuration
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=4, cal_batch=8, unsigned=True)


def test_resnet50_per_channel_weights(B):
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=4, cal_batch=8, per_channel=True)


def test_resnet50_after_sparsity_removal(B):
    # the paper's graph transformation of the stride-2 stage entries (config 6): strided
    # 1x1 layers with a residual that a 1x1 stride-2 pooling subsampled
    _sampled_images_check(B, 6, 16, [0, 7, 8, 15], n_cal=2, cal_batch=8)


def test_config4_inception_v3_batch64_sampled_images(B):
    # odd extents (299 -> 149 -> 147 -> 73 -> 71 -> 35 -> 17 -> 8), 1x7 / 7x1 filters,
    # pooled branches, channel-slice writes into concatenations
    _sampled_images_check(B, 4, 64, [0, 21, 63], n_cal=4, cal_batch=8)


@pytest.mark.parametrize("batch,picks", [(1, [0]), (64, [0, 32, 63])])
def test_config5_ssd300_vgg16_sampled_images(B, batch, picks):
    # 3x3 stack at 300x300, ceil-mode pooling, dilation 6, head convolutions with
    # K in {16, 24, 84, 126}, twelve int8 outputs
    _sampled_images_check(B, 5, batch, picks, n_cal=2, cal_batch=4)


def test_resnet50_with_fused_layer_pairs(B):
    # every bottleneck's 3x3 -> 1x1 whose 3x3 has 64 or 128 filters runs as one launch, in
    # the benchmark's launch configuration
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=4, cal_batch=8, fuse_pairs=True)


def test_resnet50_with_fused_head(B):
    # Eq. Q on the image, the 7x7 / 2 layer and the 3x3 / 2 max-pool as one launch per half
    # batch: the launch configuration the benchmark times
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=4, cal_batch=8, fuse_head=True)
    _sampled_images_check(B, 3, 5, [0, 2, 4], n_cal=2, cal_batch=8, fuse_head=True, n_streams=1)


def test_resnet50_with_dual_launches(B):
    # the projection branch and the first 1x1 of each of the four stages as one launch, in the
    # benchmark's launch configuration (two half-batch pipelines), also together with the fused
    # 3x3 -> 1x1 pairs
    _sampled_images_check(B, 3, 64, [0, 31, 32, 63], n_cal=4, cal_batch=8, fuse_duals=True)
    _sampled_images_check(B, 3, 16, [0, 7, 8, 15], n_cal=2, cal_batch=8, fuse_duals=True,
                          fuse_pairs=True)


def test_resnet50_as_one_chained_launch(B):
    # the 52 convolutions behind the first pooling as ONE persistent launch (the batch split
    # over the eight XCDs, tiles started by completion counters); images on both sides of
    # every boundary between two XCDs' shares are among the picks
    _sampled_images_check(B, 3, 64, [0, 7, 8, 31, 32, 55, 56, 63], n_cal=4, cal_batch=8,
                          n_streams=1, chain=True)


@pytest.mark.parametrize("batch", [13, 3])
def test_chained_launch_with_uneven_and_empty_shares(B, batch):
    # 13 images: shares of 2 and 1; 3 images: five XCDs have no work at all
    _sampled_images_check(B, 3, batch, list(range(batch)), n_cal=2, cal_batch=8, n_streams=1,
                          chain=True)


@pytest.mark.parametrize("variant", [0, 1, 2, 3])
def test_chained_launch_with_every_tile_variant(B, variant):
    # the bottleneck block of config 2 with one tile shape forced on all three layers:
    # ragged pixel tiles (25 images: shares of 4 and 3) and the residual dependency
    net = wl.CONFIGS[2]["make"]()
    _sampled_images_check(B, 2, 25, [0, 3, 4, 12, 24], n_cal=1, cal_batch=4, n_streams=1,
                          chain=True, chain_variants={op.name: variant for op in net.convs()})


def test_resnet50_sums_at_their_own_calibrated_factor(B):
    # the variant of the sum rule: q of a fused sum from its own max-abs, not max(q1, q2)
    _sampled_images_check(B, 3, 8, [0, 3, 4, 7], n_cal=2, cal_batch=8, own_sum_factor=True)


def test_networks_with_real_valued_outputs(B):
    # the last convolution (ResNet-50: fused sum + ReLU) and the twelve SSD head
    # convolutions write fp32 directly instead of int8 codes plus a dequantise pass
    _sampled_images_check(B, 3, 8, [0, 3, 4, 7], n_cal=2, cal_batch=8, real_outputs=True)
    _sampled_images_check(B, 5, 1, [0], n_cal=2, cal_batch=4, real_outputs=True)


def test_gpu_calibration_matches_oracle_closely(B):
    # the GPU's own calibration (fp32 forward in a different summation order) gives
    # factors equal to the oracle's up to fp32 rounding of the activations
    from paper_1805_08691_amd.engine import Engine
    cfg_id, batch = 2, 4
    cfg = wl.CONFIGS[cfg_id]
    net = cfg["make"]()
    params = {op.name: wl.conv_params(cfg_id, i, op) for i, op in enumerate(net.convs())}
    xs = [wl.input_batch(cfg_id, net, batch, i, relu=True) for i in range(2)]
    folded = onet.fold_all(net, params)
    q_o = onet.calibrate(net, folded, xs, use_library=False)
    eng = Engine(net, batch)
    eng.load_params(params)
    eng.fold()
    q_g = eng.calibrate([dev(x) for x in xs])
    assert set(q_g) == set(q_o)
    for k in q_o:
        assert abs(q_g[k] - float(q_o[k])) <= 1e-5 * float(q_o[k]), k


def _padded_concat_net():
    """Two branches and a pooling of the image's map side by side in a tensor that is padded to 48
    channels, read by another layer."""
    net = wl.Network("padded_concat", "x")
    net.tensor("x", 9, 11, 16)
    net.tensor("cat", 9, 11, 48)
    wl._conv(net, "a", "x", 8, 1, 1, dst="cat", dst_c_off=0)
    wl._conv(net, "b", "x", 12, 3, 3, dst="cat", dst_c_off=12)
    wl._pool(net, "p", "x", 3, 1, 1, dst="cat", dst_c_off=24)
    net.outputs = [wl._conv(net, "c", "cat", 32, 3, 3, relu=False)]
    return net


def test_gpu_calibration_of_partly_written_tensors(B):
    """Channels of a tensor that no op writes are zeros in the fp32 forward, whatever the memory
    held before."""
    from paper_1805_08691_amd.engine import Engine
    net = _padded_concat_net()
    params = {op.name: wl.conv_params(2, i, op) for i, op in enumerate(net.convs())}
    rng = np.random.default_rng(3)
    xs = [rng.standard_normal((4, 9, 11, 16)).astype(np.float32) for _ in range(2)]
    q_o = onet.calibrate(net, onet.fold_all(net, params), xs)
    eng = Engine(net, 4)
    eng.load_params(params)
    eng.fold()
    dirt = [torch.full((4, 9, 11, n), 1e6, device="cuda") for n in (16, 32, 48) for _ in range(4)]
    torch.cuda.synchronize()
    del dirt                       # what the allocator hands out next
    q_g = eng.calibrate([dev(x) for x in xs])
    assert set(q_g) == set(q_o)
    for k in q_o:
        assert abs(q_g[k] - float(q_o[k])) <= 1e-5 * float(q_o[k]), k


@pytest.mark.parametrize("scale", [100.0, 0.01])
def test_gpu_calibration_of_slices_written_over(B, scale):
    """Of a tensor's slices that one layer writes, another reads and a third writes over, the final
    values are measured, those of a pooling among them, also where nothing reads them."""
    from paper_1805_08691_amd.engine import Engine
    net = wl.Network("written_over", "x")
    net.tensor("x", 9, 11, 16)
    net.tensor("cat", 9, 11, 48)
    wl._conv(net, "a", "x", 24, 1, 1, dst="cat", dst_c_off=0)
    wl._pool(net, "p", "x", 3, 1, 1, dst="cat", dst_c_off=24)
    net.outputs = [wl._conv(net, "c", "cat", 32, 3, 3, relu=False), "cat"]
    wl._conv(net, "e", "x", 20, 1, 1, dst="cat", dst_c_off=4)
    params = {op.name: wl.conv_params(2, i, op) for i, op in enumerate(net.convs())}
    for k in ("W", "b", "beta", "mu"):             # (channels 4 and up are written over by e)
        params["a"][k][4 if scale > 1 else 0:] *= np.float32(scale)
        params["e"][k] *= np.float32(0.01)
    rng = np.random.default_rng(3)
    xs = [rng.standard_normal((4, 9, 11, 16)).astype(np.float32) for _ in range(2)]
    q_o = onet.calibrate(net, onet.fold_all(net, params), xs)
    eng = Engine(net, 4)
    eng.load_params(params)
    eng.fold()
    q_g = eng.calibrate([dev(x) for x in xs])
    assert set(q_g) == set(q_o)
    for k in q_o:
        assert abs(q_g[k] - float(q_o[k])) <= 1e-5 * float(q_o[k]), k


@pytest.mark.parametrize("make", [wl.bottleneck_block, _padded_concat_net])
def test_gpu_forward_f32_shows_what_calibration_measures(B, make):
    from paper_1805_08691_amd.engine import Engine
    net = make()
    t_in = net.tensors[net.input]
    eng = Engine(net, 2, own_sum_factor=True)
    eng.load_params({op.name: wl.conv_params(2, i, op) for i, op in enumerate(net.convs())})
    eng.fold()
    x = np.random.default_rng(3).standard_normal((2, t_in.H, t_in.W, t_in.C)).astype(np.float32)
    seen = {}
    t = eng.forward_f32(dev(x), lambda key, v: seen.update({key: v}))
    assert set(t) == set(net.tensors)
    q = eng.calibrate([dev(x)])
    assert set(seen) == set(q) - {net.input}
    for key, v in seen.items():
        assert q[key] == B.qfactor(float(v.abs().max()), 7), key
        assert key not in t or t[key] is v
    want, branches = onet.forward_f32(net, {k: (host(w), host(b)) for k, (w, b) in eng.folded.items()}, x)
    for key, v in {**want, **{k + ":branch": v for k, v in branches.items()}}.items():
        got = host(seen.get(key, t.get(key)))
        # three layers of at most 576 products and sums each in another order: 3 * 578 * 2^-24 of what
        # is summed
        assert np.abs(got - v).max() <= 1.1e-4 * np.abs(v).max(), key


# the fp32 forward of calibration: every tile build (256 x 64, 128 x 128, 64 x 64 and 32 x 32 shared by
# four wavefront groups) in every chunk mode (a stage in one tap, 16 bytes in one tap, single values),
# tails in pixels, channels and reduction, stride, dilation, a channel slice, residuals that are read
# as vectors and one by one
F32_256, F32_128, F32_64, F32_32 = "4,1,4,4,1,1,3", "2,2,4,4,1,1,3", "1,1,4,4,4,1,3", "1,1,2,2,4,2,3"


@pytest.mark.parametrize("build,geom,res,slice_", [
    (F32_32 + ",0", (1, 5, 7, 3, 20, 3, 3, 1, 1), False, (0, 0)),
    (F32_32 + ",0", (2, 17, 15, 7, 33, 5, 5, 2, 1), True, (0, 0)),
    (F32_32 + ",1", (1, 7, 7, 12, 64, 1, 1, 1, 1), True, (0, 0)),
    (F32_32 + ",1", (3, 9, 11, 20, 70, 3, 3, 1, 2), False, (90, 12)),
    (F32_32 + ",2", (1, 1, 1, 2048, 50, 1, 1, 1, 1), False, (0, 0)),
    (F32_32 + ",1", (2, 28, 28, 48, 192, 3, 3, 1, 1), True, (0, 0)),
    (F32_32 + ",2", (4, 57, 55, 32, 65, 3, 3, 2, 1), True, (0, 0)),
    (F32_128 + ",2", (8, 64, 66, 16, 130, 1, 7, 1, 1), False, (133, 1)),
    (F32_128 + ",0", (5, 57, 59, 7, 132, 3, 3, 1, 1), True, (0, 0)),
    (F32_128 + ",1", (5, 57, 59, 20, 130, 3, 3, 1, 1), True, (0, 0)),
    (F32_128 + ",2", (5, 57, 59, 48, 140, 1, 1, 1, 1), True, (0, 0)),
    (F32_64 + ",0", (5, 57, 59, 7, 40, 3, 3, 1, 2), True, (0, 0)),
    (F32_64 + ",0", (5, 113, 117, 3, 45, 7, 7, 2, 1), False, (0, 0)),
    (F32_64 + ",1", (5, 31, 33, 20, 140, 3, 3, 1, 1), True, (0, 0)),
    (F32_64 + ",1", (5, 57, 59, 12, 33, 1, 3, 1, 1), False, (41, 5)),
    (F32_64 + ",2", (5, 57, 59, 80, 50, 1, 1, 1, 1), True, (0, 0)),
    (F32_64 + ",2", (5, 31, 33, 48, 160, 3, 3, 1, 1), False, (0, 0)),
    (F32_256 + ",0", (3, 149, 151, 3, 50, 3, 3, 1, 1), False, (0, 0)),
    (F32_256 + ",0", (3, 149, 151, 5, 64, 1, 1, 1, 1), True, (0, 0)),
    (F32_256 + ",1", (3, 149, 151, 12, 36, 3, 3, 1, 1), True, (0, 0)),
    (F32_256 + ",2", (3, 149, 151, 16, 33, 3, 3, 1, 1), True, (0, 0)),
    (F32_256 + ",2", (3, 149, 151, 80, 60, 1, 1, 1, 1), False, (64, 4))])
def test_conv_f32_tiles(B, build, geom, res, slice_):
    import torch
    N, H, W, Cc, K, R, S, st, dil = geom
    rng = np.random.default_rng(11)
    ph, pw = dil * (R - 1) // 2, dil * (S - 1) // 2
    desc = B.ConvDesc(N, H, W, Cc, K, R, S, st, st, ph, pw, dil, dil, relu=1, out_c_stride=slice_[0],
                      out_c_off=slice_[1])
    assert B.conv_f32_variant(desc) == f"conv_f32_mfma_kernel<{build}>"
    x = rng.standard_normal((N, H, W, Cc)).astype(np.float32)
    w = rng.standard_normal((K, R, S, Cc)).astype(np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    r = rng.standard_normal((N, desc.Ho, desc.Wo, K)).astype(np.float32) if res else None

    def fp64(x, w, b):
        y = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2),
                                       torch.from_numpy(w).double().permute(0, 3, 1, 2),
                                       torch.from_numpy(b).double() if b is not None else None, st,
                                       (ph, pw), dil)
        return y.permute(0, 2, 3, 1).numpy()
    pre = fp64(x, w, b)
    want = np.maximum(pre + r if res else pre, 0.0)
    # any order of n fp32 products and sums: |error| <= (n + 2) 2^-24 sum |x||w| (+ |b| + |r|)
    bound = (R * S * Cc + 4) * 2.0 ** -24 * (fp64(abs(x), abs(w), abs(b)) + (abs(r) if res else 0))
    m_sum, m_out = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    out = torch.full((N, desc.Ho, desc.Wo, slice_[0] or K), -7.0, device="cuda")
    B.conv_f32_observed(desc, dev(x), dev(w), dev(b), dev(r) if res else None, out, m_sum, m_out)
    got, lo = host(out), slice_[1]
    assert np.all(abs(got[..., lo:lo + K] - want) <= bound)
    assert np.all(got[..., :lo] == -7) and np.all(got[..., lo + K:] == -7)
    assert float(m_out) == got[..., lo:lo + K].max()          # the maximum of what was written
    assert abs(float(m_sum) - abs(pre).max()) <= bound.max()
    if slice_ == (0, 0):
        ref = B.conv_f32_ref(desc, dev(x), dev(w), dev(b), dev(r) if res else None)
        assert np.array_equal(host(ref), got)                 # the same sums without the maxima


# the builds on LDS: fewer steps than groups and than the ring holds, steps that do not divide, tails in
# pixels and channels, stride, dilation, row and column filters, slices, residuals, several images a tile
@pytest.mark.parametrize("build,geom,res,slice_", [
    ("1,1,4,4", (1, 5, 7, 32, 16, 1, 1, 1, 1), True, (0, 0)),
    ("1,1,4,4", (9, 3, 3, 96, 48, 3, 3, 1, 1), False, (56, 4)),
    ("1,1,4,4", (3, 13, 11, 64, 80, 3, 3, 2, 1), True, (0, 0)),
    ("1,1,4,4", (2, 19, 19, 64, 144, 3, 3, 1, 6), True, (0, 0)),
    ("1,1,4,4", (4, 29, 31, 160, 176, 1, 7, 1, 1), False, (0, 0)),
    ("1,2,2,4", (8, 28, 28, 32, 48, 5, 5, 1, 1), True, (0, 0)),
    ("2,1,2,4", (8, 64, 66, 32, 32, 1, 7, 1, 1), False, (40, 8)),
    ("2,1,2,4", (8, 65, 67, 64, 16, 3, 3, 2, 1), True, (0, 0)),
    ("2,2,1,4", (5, 57, 59, 32, 64, 1, 1, 1, 1), False, (0, 0)),
    ("2,2,1,4", (7, 35, 37, 32, 272, 1, 1, 1, 1), True, (0, 0))])
def test_conv_f32_lds_builds(B, build, geom, res, slice_):
    N, H, W, Cc, K, R, S, st, dil = geom
    rng = np.random.default_rng(12)
    ph, pw = dil * (R - 1) // 2, dil * (S - 1) // 2
    desc = B.ConvDesc(N, H, W, Cc, K, R, S, st, st, ph, pw, dil, dil, relu=int(not res), out_c_stride=slice_[0],
                      out_c_off=slice_[1])
    assert B.conv_f32_variant(desc) == f"conv_f32_lds_kernel<{build}>"
    x = rng.standard_normal((N, H, W, Cc)).astype(np.float32)
    w = rng.standard_normal((K, R, S, Cc)).astype(np.float32)
    b = rng.standard_normal(K).astype(np.float32)
    r = rng.standard_normal((N, desc.Ho, desc.Wo, K)).astype(np.float32) if res else None

    def fp64(x, w, b):
        y = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2),
                                       torch.from_numpy(w).double().permute(0, 3, 1, 2),
                                       torch.from_numpy(b).double(), st, (ph, pw), dil)
        return y.permute(0, 2, 3, 1).numpy()
    pre = fp64(x, w, b)
    want = pre + r if res else np.maximum(pre, 0.0)
    # any order of n fp32 products and sums: |error| <= (n + 2) 2^-24 sum |x||w| (+ |b| + |r|)
    bound = (R * S * Cc + 4) * 2.0 ** -24 * (fp64(abs(x), abs(w), abs(b)) + (abs(r) if res else 0))
    spread = torch.zeros((2, 3 * B.SLOT_STRIDE), device="cuda")
    out = torch.full((N, desc.Ho, desc.Wo, slice_[0] or K), -7.0, device="cuda")
    B.conv_f32_observed(desc, dev(x), dev(w), dev(b), dev(r) if res else None, out, spread[0], spread[1], 3)
    got, lo = host(out), slice_[1]
    assert np.all(abs(got[..., lo:lo + K] - want) <= bound)
    assert np.all(got[..., :lo] == -7) and np.all(got[..., lo + K:] == -7)
    m = host(B.calibrate_fold(spread, torch.empty(2, device="cuda")))
    assert m[1] == abs(got[..., lo:lo + K]).max() and abs(m[0] - abs(pre).max()) <= bound.max()
    one = torch.zeros(2, device="cuda")                       # one copy: the same maxima
    B.conv_f32_observed(desc, dev(x), dev(w), dev(b), dev(r) if res else None, out, one[:1], one[1:])
    assert np.array_equal(host(one), m)
    # addresses the builds cannot read: the register-fed ones give as good a sum
    moved = torch.empty(w.size + 1, device="cuda")[1:]
    moved.copy_(dev(w).view(-1))
    ref = host(B.conv_f32_ref(desc, dev(x), moved.view(w.shape), dev(b), dev(r) if res else None)) \
        if slice_ == (0, 0) else want
    assert np.all(abs(ref - want) <= bound)


# the streaming passes: chunks of 8192 values per block (a ragged last one, none at all, more than the grid has
# blocks), addresses that are 4-byte aligned only, lists around a quarter of the cache, a tensor beyond it
@pytest.mark.parametrize("n,shift", [(5, 0), (8191, 1), (8192, 0), (8193, 3), (24576 + 7, 2), (2048 * 8192 + 4099, 0),
                                     (2**24 - 1, 0), (2**24 + 1, 1), (2**26 + 8195, 0)])
def test_streaming_passes(B, n, shift):
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(n + shift, device="cuda", generator=g)
    x, q = buf[shift:], 0.043
    k = torch.randint(0, n, (257,), device="cuda", generator=g)
    x[k] = (torch.randint(-140, 140, (257,), device="cuda", generator=g) + 0.5) * q       # ties and clamped codes
    x[n // 2], x[n - 1] = torch.inf, -9.25
    for unsigned in (False, True):
        # the IEEE quotient (by a tensor: torch multiplies by a number's reciprocal), half to even
        want = torch.round(x / torch.full((1,), q, device="cuda"))
        want = want.clamp(0, 255) - 128 if unsigned else want.clamp(-128, 127)
        z = B.quantize_u8(x, q) if unsigned else B.quantize(x, q, 7)
        assert torch.equal(z, want.to(torch.int8))
        r = torch.empty(n + shift, device="cuda")[shift:]
        r = B.dequantize_u8(z, q, out=r) if unsigned else B.dequantize(z, q, out=r)
        assert torch.equal(r, (z.float() + (128 if unsigned else 0)) * q)
    x[n // 2] = 8.0
    slot = torch.zeros(1, device="cuda")
    B.calibrate_maxabs(x, slot)
    assert float(slot) == 9.25


# the builds on the bf16 matrix instructions: tails in pixels, a step count that the wavefronts do not divide, stride,
# row and column filters, slices, residuals, several images a tile
@pytest.mark.parametrize("build,geom,res,slice_", [
    ("8", (3, 33, 31, 64, 192, 3, 3, 1, 1), True, (0, 0)),
    ("8", (4, 61, 67, 64, 128, 3, 3, 2, 1), False, (140, 8)),
    ("4", (6, 65, 67, 32, 64, 5, 5, 1, 1), False, (0, 0)),
    ("4", (7, 37, 35, 128, 320, 1, 3, 1, 1), True, (0, 0)),
    ("4", (3, 49, 51, 1024, 192, 1, 1, 1, 1), False, (0, 0)),
    # layers that are no multiples of the LDS builds' pieces: 16 channels, rows of 4- and of 8-byte accesses
    ("4", (5, 47, 49, 80, 180, 5, 5, 1, 1), True, (0, 0)),
    ("8", (2, 41, 43, 304, 126, 3, 3, 1, 1), True, (0, 0)),
    ("8", (2, 43, 41, 304, 84, 3, 3, 1, 1), False, (91, 6))])
def test_conv_f32_split_builds(B, build, geom, res, slice_):
    """Sums at least as near to 64 bits as the bound of n fp32 products and sums; what bf16 cannot hold, or
    holds with fewer bits, as the fp32 sum gives it."""
    N, H, W, Cc, K, R, S, st, dil = geom
    g = torch.Generator(device="cuda").manual_seed(13)
    rand = lambda *s: torch.randn(s, device="cuda", generator=g)
    ph, pw = dil * (R - 1) // 2, dil * (S - 1) // 2
    desc = B.ConvDesc(N, H, W, Cc, K, R, S, st, st, ph, pw, dil, dil, relu=int(not res), out_c_stride=slice_[0],
                      out_c_off=slice_[1])
    assert B.conv_f32_variant(desc) == f"conv_f32_split_kernel<{build}>"
    x, w, b = rand(N, H, W, Cc), rand(K, R, S, Cc), rand(K)
    r = rand(N, desc.Ho, desc.Wo, K) if res else None

    def fp64(x, w):
        x = torch.nn.functional.pad(x.double(), (0, 0, pw, pw, ph, ph))
        y = torch.zeros(N * desc.Ho * desc.Wo, K, dtype=torch.float64, device="cuda")
        for i in range(R):
            for j in range(S):
                v = x[:, i * dil:i * dil + (desc.Ho - 1) * st + 1:st, j * dil:j * dil + (desc.Wo - 1) * st + 1:st]
                y += v.reshape(-1, Cc) @ w[:, i, j].double().t().contiguous()
        return y.view(N, desc.Ho, desc.Wo, K)
    pre = fp64(x, w) + b.double()
    want = pre + r if res else pre.clamp(min=0)
    # any order of n fp32 products and sums: |error| <= (n + 2) 2^-24 sum |x||w| (+ |b| + |r|)
    bound = (R * S * Cc + 4) * 2.0 ** -24 * (fp64(x.abs(), w.abs()) + b.abs() + (r.abs() if res else 0))
    spread = torch.zeros((2, 3 * B.SLOT_STRIDE), device="cuda")
    out = torch.full((N, desc.Ho, desc.Wo, slice_[0] or K), -7.0, device="cuda")
    B.conv_f32_observed(desc, x, w, b, r, out, spread[0], spread[1], 3)
    lo = slice_[1]
    got = out[..., lo:lo + K]
    assert bool(((got - want).abs() <= bound).all())
    assert bool((out[..., :lo] == -7).all()) and bool((out[..., lo + K:] == -7).all())
    m = host(B.calibrate_fold(spread, torch.empty(2, device="cuda")))
    assert m[1] == float(got.abs().max()) and abs(m[0] - float(pre.abs().max())) <= float(bound.max())
    if slice_ != (0, 0):
        return
    # the 2-norm of the error: six rounded products of bf16 pieces and their sums stay within that of fp32's, about
    # sqrt(n) roundings of 2^-25 on values whose squares add up to the result's
    assert float((got - want).norm()) <= (R * S * Cc) ** 0.5 * 2.0 ** -25 * float(pre.norm())
    plain = desc
    plain.relu = 0
    huge = x.clone()
    huge[0, 0, 0, 1], huge[0, 5, 6, 3], huge[N - 1, H - 1, W - 1, 0] = 3.4e38, -torch.inf, torch.nan
    for xs, ws in ((huge, w * 2.0 ** -12), (x * 2.0 ** -100, w * 2.0 ** -20)):
        got = B.conv_f32_ref(plain, xs, ws)
        want = fp64(xs, ws).float()
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
        fine = want.isfinite()
        err = ((got.double() - fp64(xs, ws)).abs()[fine] <= (R * S * Cc + 4) * 2.0 ** -24 *
               fp64(xs.abs(), ws.abs())[fine] + 2.0 ** -149 * (R * S * Cc + 1))
        assert bool(err.all())


@pytest.mark.parametrize("geom", [(8, 28, 28, 128, 128), (3, 61, 59, 64, 256)])       # eight wavefronts a tile, four
@pytest.mark.parametrize("kind", ["small x, large w", "large x, small w", "denormal x", "denormal w", "few denormals",
                                  "zeros", "zeros and large"])
def test_conv_f32_split_operands_that_bf16_cannot_split(B, geom, kind):
    """Values that three bf16 pieces hold with fewer bits, or not at all, count as the fp32 sum counts them, whatever the
    size of the sum; sums of zero are zero."""
    N, H, W, Cc, K = geom
    g = torch.Generator(device="cuda").manual_seed(17)
    d = B.ConvDesc(N, H, W, Cc, K, 3, 3, pad_h=1, pad_w=1)
    assert B.conv_f32_variant(d).startswith("conv_f32_split_kernel")
    x, w = torch.randn((N, H, W, Cc), device="cuda", generator=g), torch.randn((K, 3, 3, Cc), device="cuda", generator=g)
    mantissa = lambda t, e: torch.ldexp(torch.sign(t) * (1 + t.abs().frac()), torch.tensor(e, device="cuda"))
    if kind == "small x, large w":
        x, w = mantissa(x, -124), w * 2.0 ** 100
    elif kind == "large x, small w":
        x, w = x * 2.0 ** 100, mantissa(w, -124)
    elif kind == "denormal x":
        x, w = mantissa(x, -137), w * 2.0 ** 30
    elif kind == "denormal w":
        x, w = x * 2.0 ** 30, mantissa(w, -137)
    elif kind == "few denormals":          # sums of zero in most places, of denormals' products in some
        x = torch.zeros_like(x)
        x[N - 1, H - 1, W - 1, Cc - 1] = x[0, 5, 3, 0] = 2.0 ** -138
        w = w * 2.0 ** 30
    else:
        x[:, ::2] = 0
        x[0, :8, :11] = 0
        w[:, :, :, Cc // 2:] = 0
        w[3] = 0
        if kind == "zeros and large":
            x[N - 1, H - 1, W - 1, 0] = 2.0 ** 40
    got = B.conv_f32_ref(d, x, w).double()

    def fp64(x, w):
        x = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
        return sum((x[:, i:i + H, j:j + W].reshape(-1, Cc) @ w[:, i, j].double().t().contiguous()
                    for i in range(3) for j in range(3))).view(N, H, W, K)
    want, n = fp64(x, w), 9 * Cc
    size = fp64(x.abs(), w.abs())
    assert bool(((got - want).abs() <= (n + 2) * 2.0 ** -24 * size + (n + 1) * 2.0 ** -149).all())
    if "zeros" in kind or kind == "few denormals":
        assert bool((got[size == 0] == 0).all()) and bool((size == 0).any()) and bool((got[want.abs() > 0.5 * size] != 0).all())


@pytest.mark.parametrize("geom", [(8, 28, 28, 128, 128), (4, 41, 43, 256, 192)])      # eight wavefronts a tile, four
def test_conv_f32_split_is_no_slower_than_the_fp32_instruction_where_it_sums_again(B, geom):
    """Sums that are no numbers are taken again by the whole workgroup, 16 + 5 instructions' time for 5: a layer of
    them stays within four times its time, also where only few of a tile's sums are such."""
    N, H, W, Cc, K = geom
    g = torch.Generator(device="cuda").manual_seed(5)
    d = B.ConvDesc(N, H, W, Cc, K, 3, 3, pad_h=1, pad_w=1)
    assert B.conv_f32_variant(d).startswith("conv_f32_split_kernel")
    x, w = torch.randn((N, H, W, Cc), device="cuda", generator=g), torch.randn((K, 3, 3, Cc), device="cuda", generator=g)
    few, y = x.clone(), torch.empty((N, H, W, K), device="cuda")
    few[:, ::4, ::4, 7] = torch.nan

    def us(t):
        took = []
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(4):
                B.conv_f32_observed(d, t, w, None, None, y, None, None)
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        return sorted(took)[3]
    plain = us(x)
    assert us(few) < 4 * plain and us(torch.full_like(x, torch.nan)) < 4 * plain and bool(y.isnan().all())


@pytest.mark.parametrize("channels", [(64, 64), (12, 8)])       # a build on LDS, a register-fed one
def test_conv_f32_observed_raises_the_first_value_of_a_slot(B, channels):
    """A slot of any length holds one maximum, in its first value, unless copies are asked for."""
    c, k = channels
    desc = B.ConvDesc(3, 19, 17, c, k, 3, 3, pad_h=1, pad_w=1)
    x, w = torch.randn(3, 19, 17, c, device="cuda"), torch.randn(k, 3, 3, c, device="cuda")
    out = torch.empty(3, 19, 17, k, device="cuda")
    slots = [torch.zeros(n, device="cuda") for n in (1, 33, 40, 512)]
    for a, b in zip(slots, slots[1:] + slots[:1]):            # of two lengths
        a.zero_(), b.zero_()
        B.conv_f32_observed(desc, x, w, None, None, out, a, b)
        for m in (a, b):
            assert float(m[0]) == float(out.abs().max()) and not m[1:].any()
    with pytest.raises(AssertionError):
        B.conv_f32_observed(desc, x, w, None, None, out, slots[1], None, 3)     # 33 values: two copies


@pytest.mark.parametrize("n_keys,n_slots", [(1, 1), (3, 16), (130, 70)])
def test_calibrate_fold(B, n_keys, n_slots):
    spread = torch.rand((n_keys, n_slots * B.SLOT_STRIDE), device="cuda")
    out = torch.full((n_keys,), -1.0, device="cuda")
    B.calibrate_fold(spread, out)
    assert torch.equal(out, spread.view(n_keys, n_slots, B.SLOT_STRIDE)[..., 0].amax(1))


def test_layer_calls_take_what_they_took(B):
    """Layer calls with tensors of a subclass, factors that are numpy numbers, a second stream; what is
    not contiguous, of another type or refused by the library raises."""
    rng = np.random.default_rng(3)
    d = B.ConvDesc(2, 9, 9, 64, 48, 3, 3, pad_h=1, pad_w=1, relu=1)
    x = dev(rng.integers(-128, 128, (2, 9, 9, 64)).astype(np.int8))
    w = B.pack_weights(d, dev(rng.integers(-128, 128, (48, 3, 3, 64)).astype(np.int8)))
    b = dev(rng.integers(-2000, 2000, 48).astype(np.int32))
    want = B.conv_int8(d, x, w, b, 0.01, 0.01, 0.5)
    as_param = lambda t: torch.nn.Parameter(t, requires_grad=False)
    f = np.float32
    assert torch.equal(B.conv_int8(d, as_param(x), as_param(w), as_param(b), f(0.01), f(0.01), f(0.5)), want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = B.conv_int8(d, x, w, b, 0.01, 0.01, 0.5)
    side.synchronize()
    assert torch.equal(got, want)
    assert B.conv_int8_real_output(d, x, w.view(torch.uint8), b, 0.01, 0.01).dtype is torch.float32
    for bad in (lambda: B.conv_int8(d, x.transpose(1, 2), w, b, 0.01, 0.01, 0.5),
                lambda: B.conv_int8(d, x, w, b.float(), 0.01, 0.01, 0.5),
                lambda: B.conv_int8(d, x, w, b, 0.01, 0.01, 0.5, out=want.cpu())):
        with pytest.raises(AssertionError):
            bad()
    with pytest.raises(B.Q8Error):
        B.conv_int8(d, x, w, b, 0.0, 0.01, 0.5)
    with pytest.raises(B.Q8Error):
        B.conv_int8(d, None, w, b, 0.01, 0.01, 0.5, out=want)
    empty = B.ConvDesc(0, 9, 9, 64, 48, 3, 3, pad_h=1, pad_w=1)
    assert B.conv_int8(empty, x[:0], w, None, 0.01, 0.01, 0.5).shape == (0, 9, 9, 48)


# tensors that the tiled builds' 32-bit offsets cannot reach into, by a dilation that leaves one row of
# taps inside the image, and one as tall as the dilation with all three rows in use
@pytest.mark.parametrize("H,W,C,K,S,slice_", [(9, 7, 24, 21, 3, (30, 4)), (2**20 + 37, 1, 64, 4, 1, (0, 0))])
def test_conv_f32_of_any_size(B, H, W, C, K, S, slice_):
    dil = 2**20
    d = B.ConvDesc(1, H, W, C, K, 3, S, pad_h=dil, pad_w=S // 2, dil_h=dil, relu=1, out_c_stride=slice_[0],
                   out_c_off=slice_[1])
    assert B.conv_f32_variant(d) == "conv_f32_any_kernel" and (d.Ho, d.Wo) == (H, W)
    g = torch.Generator(device="cuda").manual_seed(5)

    def rand(*shape):
        return torch.randn(shape, device="cuda", generator=g)
    x, w, b, r = rand(1, H, W, C), rand(K, 3, S, C), rand(K), rand(1, H, W, K)
    out, m = torch.full((1, H, W, slice_[0] or K), -7.0, device="cuda"), torch.zeros(2, device="cuda")
    B.conv_f32_observed(d, x, w, b, r, out, m[:1], m[1:])

    def fp64(x, w, b):
        y = torch.zeros((H, W, K), dtype=torch.float64, device="cuda") + b.double()
        for row in range(3):
            lo, hi = max(0, (1 - row) * dil), min(H, H - (row - 1) * dil)
            for s in range(S):
                w0, w1 = max(0, S // 2 - s), min(W, W - (s - S // 2))
                if lo < hi:
                    part = x[0, lo + (row - 1) * dil:hi + (row - 1) * dil, w0 + s - S // 2:w1 + s - S // 2]
                    y[lo:hi, w0:w1] += part.double() @ w[:, row, s].double().t()
        return y
    pre = fp64(x, w, b)
    bound = (3 * S * C + 4) * 2.0 ** -24 * (fp64(x.abs(), w.abs(), b.abs()) + r[0].abs())
    lo = slice_[1]
    got = out[0, :, :, lo:lo + K]
    assert bool(((got - (pre + r[0]).clamp(min=0)).abs() <= bound).all())
    assert bool((out[..., :lo] == -7).all()) and bool((out[..., lo + K:] == -7).all())
    assert float(m[1]) == float(got.max()) and abs(float(m[0]) - float(pre.abs().max())) <= float(bound.max())


@pytest.mark.parametrize("C, R, K", [(1, 1, 1), (3, 1, 1), (7, 1, 2), (5, 3, 33), (3, 7, 64)])
def test_conv_f32_filters_end_their_tensor(B, C, R, K):
    """The filters are the last values of their allocation and their reduction ends inside a 16-byte
    chunk: the same sums as with zeros behind them."""
    rng = np.random.default_rng(C)
    n = K * R * R * C
    size = -(-n // 128) * 128                 # (allocations are multiples of 512 bytes)
    d = B.ConvDesc(N=1, H=5, W=9, C=C, K=K, R=R, S=R, pad_h=R // 2, pad_w=R // 2)
    x = dev(rng.standard_normal((1, 5, 9, C)).astype(np.float32))
    last = torch.from_numpy(rng.standard_normal(size).astype(np.float32)).cuda()[size - n:]
    padded = torch.zeros(n + 64, device="cuda")
    padded[:n] = last
    got = [host(B.conv_f32_ref(d, x, w.view(K, R, R, C))) for w in (last, padded[:n])]
    assert np.array_equal(got[0], got[1]) and np.isfinite(got[0]).all() and got[0].any()


@pytest.mark.parametrize("C, R, K", [(3, 7, 8), (20, 1, 50), (5, 1, 33), (24, 3, 40)])
def test_conv_f32_keeps_filters_apart(B, C, R, K):
    """An infinity in one filter stays in its own channel, where the reduction ends inside a stage."""
    rng = np.random.default_rng(C)
    d = B.ConvDesc(N=1, H=9, W=9, C=C, K=K, R=R, S=R, pad_h=R // 2, pad_w=R // 2)
    x = dev(rng.standard_normal((1, 9, 9, C)).astype(np.float32))
    w = rng.standard_normal((K, R, R, C)).astype(np.float32)
    clean = host(B.conv_f32_ref(d, x, dev(w)))
    w[1] = np.inf
    got = host(B.conv_f32_ref(d, x, dev(w)))
    others = np.arange(K) != 1
    assert np.array_equal(got[..., others], clean[..., others]) and not np.isfinite(got[..., 1]).all()


# the latency family: one pixel, one reduction step, more steps than a wavefront keeps in flight (also
# of a single pixel and filter, which the steps behind the last one would lead out of), channel counts
# that end inside a group of four, taps per 16-byte chunk, a dilated filter
DIRECT_CASES = [
    dict(N=1, H=1, W=1, C=64, K=16, R=1, S=1), dict(N=1, H=1, W=1, C=2048, K=50, R=1, S=1),
    dict(N=3, H=5, W=3, C=16, K=126, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=1, H=17, W=17, C=160, K=48, R=1, S=7, pad_w=3), dict(N=1, H=7, W=9, C=512, K=20, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=2, H=19, W=19, C=64, K=36, R=3, S=3, pad_h=6, pad_w=6, dil_h=6, dil_w=6),
    dict(N=2, H=9, W=9, C=128, K=33, R=1, S=1, stride_h=2, stride_w=2),
    dict(N=1, H=1, W=1, C=4160, K=1, R=1, S=1), dict(N=1, H=1, W=1, C=4176, K=1, R=1, S=1),
    dict(N=1, H=1, W=1, C=512, K=1, R=3, S=3, pad_h=1, pad_w=1)]


@pytest.mark.parametrize("idx", range(len(DIRECT_CASES)))
def test_conv_latency_family(B, idx):
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(B.conv_num_variants())]
    variants = [v for v, n in enumerate(names) if "direct" in n]
    assert variants and "direct" in B.conv_variant(B.ConvDesc(**DIRECT_CASES[idx]))
    for v in variants:
        _run_conv_case(B, DIRECT_CASES[idx], relu=bool(v % 2), with_res=bool(idx % 2), with_bias=True,
                       seed=31 * v + idx, variant=v)


def test_unsigned_codes_with_a_start_table_beyond_4_gib(B):
    """A layer the latency family would take, whose table of start values (a row per rectangle of
    taps) a 32-bit offset cannot reach into."""
    d = B.ConvDesc(1, 5, 6, 16, 620000, 5, 6, pad_w=1, relu=1)
    assert (6 * 6 * 7 * 7) * d.K * 4 > 2**32 and "direct" in B.conv_variant(d)
    rng = np.random.default_rng(4)
    w = torch.from_numpy(rng.integers(-128, 128, d.K * 480).astype(np.int8)).cuda().view(d.K, 5, 6, 16)
    b = dev(rng.integers(-20000, 20000, d.K).astype(np.int32))
    x = rng.integers(0, 256, (1, 5, 6, 16)).astype(np.uint8)
    taps, bias = B.u8_prepare(d, w, b)
    scale = float(np.float32(1e-4))
    got = B.conv_u8(d, 1, 1, 0, dev(_stored(x)), B.pack_weights(d, w), bias, taps, 1.0, scale, 1.0)
    frame = torch.zeros((5, 8, 16), device="cuda")
    frame[:, 1:7] = dev(x)[0].float()
    for wo in range(3):                  # sums below 2^24: exact in fp32 in any order
        acc = (w.float() * frame[:, wo:wo + 6]).sum((1, 2, 3)) + b
        assert torch.equal(got[0, 0, wo].int() + 128, (acc * scale).round().clamp(0, 255).int())


def test_run_ops_groups_equal_single_calls(B):
    """Independent layers of one group (joined into one launch) and a list of tensors to dequantise
    give the bits of the calls one by one."""
    import ctypes
    rng = np.random.default_rng(5)
    geoms = [dict(N=1, H=17, W=17, C=64, K=48, R=1, S=1), dict(N=1, H=17, W=17, C=64, K=50, R=3, S=3, pad_h=1, pad_w=1),
             dict(N=1, H=17, W=17, C=48, K=16, R=1, S=7, pad_w=3), dict(N=1, H=9, W=5, C=256, K=33, R=1, S=1)]
    ops, keep, want = (B.Op * (2 * len(geoms)))(), [], []
    for i, geom in enumerate(geoms):
        d = B.ConvDesc(relu=i % 2, **geom)
        x = dev(rng.integers(-128, 128, (d.N, d.H, d.W, d.C)).astype(np.int8))
        w = B.pack_weights(d, dev(rng.integers(-128, 128, (d.K, d.R, d.S, d.C)).astype(np.int8)))
        b = dev(rng.integers(-2000, 2000, d.K).astype(np.int32))
        want.append(B.conv_int8(d, x, w, b, 0.01, 0.01, 0.5))
        y, r = torch.zeros_like(want[-1]), torch.zeros(want[-1].shape, device="cuda")
        o, q = ops[i], ops[len(geoms) + i]
        o.kind, o.group, o.d, o.x, o.w, o.bias, o.y = B.OP_CONV, 1, d, x.data_ptr(), w.data_ptr(), b.data_ptr(), y.data_ptr()
        o.q_x, o.q_w, o.q_out = 0.01, 0.01, 0.5
        q.kind, q.flags, q.x, q.n, q.q_x, q.y_f32 = B.OP_DEQUANTIZE, B.OPF_IN_U8 * (i % 2), y.data_ptr(), y.numel(), 0.5, r.data_ptr()
        keep.append((x, w, b, y, r))
    streams = (ctypes.c_void_p * 1)(torch.cuda.current_stream().cuda_stream)
    assert B.lib.q8_run_ops(ops, len(ops), streams, 1) == 0
    for i, (x, w, b, y, r) in enumerate(keep):
        assert np.array_equal(host(y), host(want[i]))
        assert np.array_equal(host(r), host(B.dequantize_u8(y, 0.5) if i % 2 else B.dequantize(y, 0.5)))


@pytest.mark.parametrize("scale", [0.5, 0.3, 2.0 ** -31, 1e31])
@pytest.mark.parametrize("relu", [0, 1])
@pytest.mark.parametrize("C,N", [(64, 1), (64, 13), (256, 13)])
def test_tails_on_ties_and_bounds(B, C, N, relu, scale):
    """Every tail on values at, beside and far beyond its ties and bounds: zero activations, so that the
    accumulators are the biases, -768 ... 767 and the ends of their range, at a scale of one half (ties), one without ties,
    one that only the ends reach a code with and one whose products leave the floats; one call
    in each family (few pixels: the latency family; many: persistent or general), every tile variant
    of the main kernel, and unsigned codes."""
    K, H = 1536, 28 if N > 1 else 3
    bias = np.arange(-768, 768, dtype=np.int32)
    bias[[5, 900, 1300]] = [-2**31 + 1, 2**30, 2**31 - 1]
    d = B.ConvDesc(N, H, H, C, K, 1, 1, relu=relu)
    x, w, b = (torch.zeros(s, dtype=torch.int8, device="cuda") for s in ((N, H, H, C), (K, 1, 1, C), 1))
    w, b = B.pack_weights(d, w), dev(bias)
    acc = np.broadcast_to(bias, (1, 1, 1, K))
    want = orc.requant(acc, scale, relu)
    assert len(np.unique(want)) == {0.5: 256, 0.3: 256, 2.0 ** -31: 3, 1e31: 3}[scale] // (1 + relu) + (scale not in (0.5, 0.3) and relu)
    variants = [-1] + ([v for v in range(B.conv_num_variants())] if N == 13 else [])
    for v in variants:
        got = host(B.conv_int8(d, x, w, b, scale, 1.0, 1.0, variant=v))
        assert np.array_equal(got, np.broadcast_to(want, got.shape)), v
    if relu:
        got = host(B.conv_u8(d, False, True, False, x, w, b, None, scale, 1.0, 1.0))
        want = orc.requant_mixed(acc, scale, 1, out_unsigned=True)
        assert np.array_equal(got.view(np.uint8) ^ 0x80, np.broadcast_to(want, got.shape))


# bottleneck blocks: mid channels, input channels, output rows and columns, images, output channels,
# stride of the first layer: one pixel, one row, the widest maps, ragged last strips, one to four rounds
BLOCKS = [(64, 64, 1, 1, 3, 64, 1), (64, 192, 7, 9, 2, 192, 1), (64, 256, 5, 56, 1, 256, 2), (64, 64, 3, 85, 1, 128, 1),
          (128, 128, 13, 28, 1, 384, 1), (128, 256, 9, 17, 2, 512, 2), (128, 512, 3, 64, 1, 128, 1),
          (256, 128, 14, 14, 1, 256, 1), (256, 512, 10, 13, 3, 1024, 1), (256, 256, 3, 32, 1, 512, 2), (256, 1024, 1, 7, 2, 768, 1)]


@pytest.mark.parametrize("option", ["plain", "bare", "unsigned", "per_channel"])
@pytest.mark.parametrize("idx", range(len(BLOCKS)))
def test_bottleneck_builds(B, idx, option):
    """Every build that takes the block gives the three tensors of three calls (plain: of the oracle),
    and writes nothing beside them; bare: no biases, no residual, the first two layers without ReLU."""
    import ctypes
    mid, C, H, W, N, K2, stride = BLOCKS[idx]
    rng = np.random.default_rng(40 + idx)
    Hi, Wi = (H - 1) * stride + 1, (W - 1) * stride + 1
    relu = [0, 0, 1] if option == "bare" else [1, 1, 1]
    slices = [(mid + 48, 32), (mid, 0), (K2 + 16, 16)] if idx % 2 else [(mid, 0), (mid, 0), (K2, 0)]
    shapes = [(Hi, Wi, C, mid, 1, 0, stride), (H, W, mid, mid, 3, 1, 1), (H, W, mid, K2, 1, 0, 1)]
    x = dev(rng.integers(-128, 128, (N, Hi, Wi, C)).astype(np.int8))
    res = None if option == "bare" else dev(rng.integers(-128, 128, (N, H, W, K2)).astype(np.int8))
    q = [0.02, 0.013, 0.017, 0.011]
    q_w, q_res = [0.01 / np.sqrt(s[2] * s[4] ** 2) * 1.2 for s in shapes], 0.009
    ops, keep, want = (B.Op * 3)(), [], []
    src, chain, oracle_src = x, x, host(x)     # what the launch reads, what single calls read
    for i, (h, w_, c, k, R, pad, st) in enumerate(shapes):
        z_w = rng.integers(-128, 128, (k, R, R, c)).astype(np.int8)
        bias = rng.integers(-2000, 2000, k).astype(np.int32)
        cs, off = slices[i]
        d = B.ConvDesc(N, h, w_, c, k, R, R, st, st, pad, pad, 1, 1, relu=relu[i], out_c_stride=cs, out_c_off=off,
                       in_c_stride=slices[i - 1][0] if i else 0)
        wp, b = B.pack_weights(d, dev(z_w)), None if option == "bare" else dev(bias)
        out = torch.full((N, H, W, cs), 77, dtype=torch.int8, device="cuda")
        r, qr = (res, q_res) if i == 2 and res is not None else (None, 0.0)
        o = ops[i]
        o.kind, o.d, o.w, o.bias = B.OP_CONV, d, wp.data_ptr(), b.data_ptr() if b is not None else None
        o.x = src.data_ptr() + (slices[i - 1][1] if i else 0)
        o.q_x, o.q_w, o.q_out = q[i], q_w[i], q[i + 1]
        if r is not None:
            o.residual, o.q_res = r.data_ptr(), qr
        xin = chain if not i else chain.flatten()[slices[i - 1][1]:]
        if option == "unsigned":
            o.flags = B.OPF_OUT_U8 | B.OPF_IN_U8 | (B.OPF_RES_U8 if i == 2 and idx % 2 else 0)
            taps, b = B.u8_prepare(d, dev(z_w), b)
            o.bias, o.aux = b.data_ptr(), taps.data_ptr()
            B.conv_u8(d, True, True, bool(o.flags & B.OPF_RES_U8), xin, wp, b, taps, q[i], q_w[i], q[i + 1], r, qr, out=out)
            keep.append(taps)
        elif option == "per_channel":
            m = dev((q[i] * q_w[i] / q[i + 1] * rng.uniform(0.5, 2.0, k)).astype(np.float32))
            o.flags, o.aux = B.OPF_PER_CHANNEL, m.data_ptr()
            B.conv_int8_per_channel(d, xin, wp, b, m, q[i + 1], r, qr, out=out)
            keep.append(m)
        else:
            B.conv_int8(d, xin, wp, b, q[i], q_w[i], q[i + 1], r, qr, out=out)
            g = orc.ConvGeom(N=N, H=h, W=w_, C=c, K=k, R=R, S=R, stride_h=st, stride_w=st, pad_h=pad, pad_w=pad)
            oracle_src = orc.conv_layer_i8(g, oracle_src, q[i], z_w, q_w[i], None if b is None else bias, q[i + 1],
                                           relu[i], host(r) if r is not None else None, qr or None)[0]
            assert np.array_equal(host(out)[..., off:off + k], oracle_src)
        want.append(host(out))
        assert len(np.unique(want[-1])) > (32 if out.numel() > 2000 else 8)
        keep += [wp, b, out]
        chain, src = out, torch.full_like(out, 77)
        o.y = src.data_ptr()
        keep.append(src)
    outs = [next(t for t in keep if t is not None and t.data_ptr() == ops[i].y) for i in range(3)]
    taken = 0
    for build in range(B.lib.q8_num_bottleneck_builds()):
        for t in outs:
            t.fill_(77)
        code = B.lib.q8_run_bottleneck(ops, build, torch.cuda.current_stream().cuda_stream)
        assert code in (0, -2)
        if code == 0:
            taken += 1
            for t, w_ in zip(outs, want):
                assert np.array_equal(host(t), w_), B.lib.q8_bottleneck_build_name(build)
    assert taken == (2 if 3 * W <= {64: 192, 128: 128, 256: 64}[mid] else 1)
    # as a marked triple, whatever the library makes of it
    for t in outs:
        t.fill_(77)
    ops[0].flags |= B.OPF_BLOCK
    streams = (ctypes.c_void_p * 1)(torch.cuda.current_stream().cuda_stream)
    assert B.lib.q8_run_ops(ops, 3, streams, 1) == 0
    for t, w_ in zip(outs, want):
        assert np.array_equal(host(t), w_)


@pytest.mark.parametrize("mid,K2", [(64, 320), (128, 384)])
def test_bottleneck_tables_end_in_a_part_of_a_load(B, mid, K2):
    """Biases and scales are copied 256 values at a time and the last copy is a part of one; the filters are
    requested on behind their last piece.  What lies behind the three tensors changes nothing."""
    N, H, W, C = 2, 6, 11, 128
    shapes = [(C, mid, 1), (mid, mid, 3), (mid, K2, 1)]
    stream = torch.cuda.current_stream().cuda_stream
    x = torch.randint(-128, 128, (N, H, W, C), dtype=torch.int8, device="cuda")
    z = [torch.randint(-128, 128, (k, R, R, c), dtype=torch.int8, device="cuda") for c, k, R in shapes]
    bias = [torch.randint(-2000, 2000, (k,), dtype=torch.int32, device="cuda") for _, k, _ in shapes]
    scale = [torch.rand(k, device="cuda") * 2e-3 + 1e-4 for _, k, _ in shapes]

    def ends(t, behind):                       # t as the last values of a buffer in front of others
        buffer = torch.full((t.numel() + 4096,), behind, dtype=t.dtype, device="cuda")
        buffer[:t.numel()] = t.flatten()
        return buffer
    taken = 0
    for per_channel in (False, True):
        got = {}
        for behind in (0, 99):
            ops, keep, src = (B.Op * 3)(), [], x
            for i, (c, k, R) in enumerate(shapes):
                o, d = ops[i], B.ConvDesc(N, H, W, c, k, R, R, 1, 1, R // 2, R // 2, relu=1)
                y = torch.zeros((N, H, W, k), dtype=torch.int8, device="cuda")
                keep += [ends(B.pack_weights(d, z[i]), behind), ends(bias[i], behind), ends(scale[i], behind), y]
                o.kind, o.d, o.x, o.y = B.OP_CONV, d, src.data_ptr(), y.data_ptr()
                o.w, o.bias = keep[-4].data_ptr(), keep[-3].data_ptr()
                o.q_x, o.q_w, o.q_out = 0.02, 1.0 if per_channel else 0.0005, 0.011
                if per_channel:
                    o.flags, o.aux = B.OPF_PER_CHANNEL, keep[-2].data_ptr()
                src = y
            for build in range(B.lib.q8_num_bottleneck_builds()):
                code = B.lib.q8_run_bottleneck(ops, build, stream)
                assert code in (0, -2)
                if code == 0:
                    taken += 1
                    got.setdefault(build, []).append([host(t) for t in keep[3::4]])
        for first, second in got.values():
            for a, b in zip(first, second):
                assert np.array_equal(a, b) and len(np.unique(a)) > 32
    assert taken >= 8


# layers whose reduction steps cross filter taps: several taps a step (C below the step's bytes), at
# most one further (C above), the most taps that the kernel takes, as one row and as one column
TAP_CASES = [
    dict(N=1, H=9, W=11, C=16, K=40, R=5, S=5, pad_h=2, pad_w=2),
    dict(N=2, H=12, W=13, C=32, K=64, R=3, S=3, stride_h=2, stride_w=2, pad_h=1, pad_w=1),
    dict(N=1, H=10, W=14, C=48, K=65, R=5, S=5, pad_h=2, pad_w=2),
    dict(N=1, H=13, W=12, C=80, K=48, R=3, S=3, pad_h=2, pad_w=2, dil_h=2, dil_w=2),
    dict(N=3, H=5, W=7, C=112, K=96, R=1, S=3, pad_w=1),
    dict(N=1, H=11, W=6, C=144, K=33, R=7, S=1, pad_h=3),
    dict(N=1, H=2, W=40, C=16, K=34, R=1, S=32, pad_w=4),
    dict(N=1, H=40, W=2, C=16, K=34, R=32, S=1, pad_h=4),
]


@pytest.mark.parametrize("idx", range(len(TAP_CASES)))
def test_conv_steps_across_taps(B, idx):
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(B.conv_num_variants())]
    for v, name in enumerate(names):
        if "ring_kernel" in name:
            _run_conv_case(B, TAP_CASES[idx], relu=bool(v % 2), with_res=bool((v + idx) % 2), with_bias=True,
                           seed=900 * idx + v, variant=v)


# a module's branches as one launch of the main kernel, in both group builds: 1x1 layers, steps in one
# tap, across taps (C below and above a step), a layer of the 3x3 family, stride and dilation, tails in
# pixels and channels, a residual, slices of one tensor
GROUP_LAYERS = [dict(C=320, K=72, R=1, S=1), dict(C=160, K=64, R=1, S=7, pad_w=3),
                dict(C=48, K=50, R=5, S=5, pad_h=2, pad_w=2), dict(C=192, K=130, R=3, S=3, pad_h=1, pad_w=1),
                dict(C=112, K=65, R=3, S=3, stride_h=2, stride_w=2, pad_h=1, pad_w=1),
                dict(C=128, K=64, R=3, S=3, pad_h=3, pad_w=3, dil_h=3, dil_w=3), dict(C=256, K=33, R=1, S=1)]


@pytest.mark.parametrize("N,H,W,build", [(9, 17, 17, "2,2,1,1,128,4"), (5, 17, 19, "2,2,1,1,128,4"),
                                         (16, 21, 23, "2,2,2,1,64,4")])
def test_run_ops_tiled_groups_equal_the_oracle(B, N, H, W, build):
    rng = np.random.default_rng(N)
    n = len(GROUP_LAYERS)
    ops, keep, want = (B.Op * n)(), [], []
    q_x, q_w = np.float32(0.02), np.float32(0.002)
    cat_c = sum(g["K"] for g in GROUP_LAYERS if "stride_h" not in g)
    cat, off = torch.full((N, H, W, cat_c), 77, dtype=torch.int8, device="cuda"), 0
    for i, layer in enumerate(GROUP_LAYERS):
        g = orc.ConvGeom(N=N, H=H, W=W, **layer)
        sliced = "stride_h" not in layer
        x = rng.integers(-128, 128, (N, H, W, g.C)).astype(np.int8)
        w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
        b = rng.integers(-20000, 20000, g.K).astype(np.int32)
        res = rng.integers(-128, 128, (N, g.Ho, g.Wo, g.K)).astype(np.int8) if i % 3 == 0 else None
        q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(g.R * g.S * g.C) / 40.0)
        q_res = np.float32(0.3) * q_out
        codes = orc.requant(orc.conv_i8(g, x, w, b), orc.requant_scale(q_x, q_w, q_out), bool(i % 2), res,
                            orc.residual_scale(q_res, q_out) if res is not None else 0.0)
        d = B.ConvDesc(N, H, W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w, g.dil_h, g.dil_w,
                       relu=i % 2, out_c_stride=cat_c if sliced else 0, out_c_off=off if sliced else 0)
        y = cat if sliced else torch.zeros(codes.shape, dtype=torch.int8, device="cuda")
        t = [dev(x), B.pack_weights(d, dev(w)), dev(b), y, dev(res) if res is not None else None]
        o = ops[i]
        o.kind, o.group, o.d, o.q_x, o.q_w, o.q_out, o.q_res = B.OP_CONV, 1, d, q_x, q_w, q_out, q_res
        o.x, o.w, o.bias, o.y = (v.data_ptr() for v in t[:4])
        o.residual = t[4].data_ptr() if res is not None else None
        keep.append(t)
        want.append((codes, slice(off, off + g.K) if sliced else slice(0, g.K)))
        off += g.K if sliced else 0
    assert B.lib.q8_group_variant(ops, n).decode() == f"conv_i8_ring_group_kernel<{build}>"
    _run_ops(B, ops)
    for i, (codes, part) in enumerate(want):
        assert np.array_equal(host(keep[i][3])[..., part], codes), GROUP_LAYERS[i]


# outputs that leave the codes, in one launch with layers that do not: real values with and without a
# residual, Eq. D beside the codes, slices, channel counts that end inside a group of four; steps in one tap and
# across taps.  (All of a size's layers have one kernel by themselves, so that all of them are in the launch.)
GROUP_OUTPUTS = [("codes", dict(C=320, K=72, R=1, S=1)), ("real", dict(C=160, K=84, R=1, S=7, pad_w=3)),
                 ("deq", dict(C=48, K=50, R=5, S=5, pad_h=2, pad_w=2)), ("real", dict(C=64, K=65, R=3, S=3, pad_h=1, pad_w=1)),
                 ("deq", dict(C=128, K=64, R=3, S=3, stride_h=2, stride_w=2, pad_h=1, pad_w=1))]


@pytest.mark.parametrize("N,H,W,build", [(1, 17, 17, "direct"), (11, 17, 19, "ring_group_kernel<2,2,1,1,128,4>"),
                                         (27, 23, 25, "ring_group_kernel<2,2,2,1,64,4>")])
def test_run_ops_groups_with_real_valued_outputs(B, N, H, W, build):
    rng = np.random.default_rng(40 + N)
    n = len(GROUP_OUTPUTS)
    ops, keep, want = (B.Op * n)(), [], []
    q_x, q_w = np.float32(0.021), np.float32(0.0017)
    for i, (kind, layer) in enumerate(GROUP_OUTPUTS):
        g = orc.ConvGeom(N=N, H=H, W=W, **layer)
        x = rng.integers(-128, 128, (N, H, W, g.C)).astype(np.int8)
        w = rng.integers(-128, 128, (g.K, g.R, g.S, g.C)).astype(np.int8)
        b = rng.integers(-20000, 20000, g.K).astype(np.int32)
        relu, with_res, pad = i % 2, i % 3 == 1, 4 * (i % 3)     # (slices behind 4 or 8 channels)
        res = rng.integers(-128, 128, (N, g.Ho, g.Wo, g.K)).astype(np.int8) if with_res else None
        q_out = np.float32(q_x * q_w * 5476.0 * np.sqrt(g.R * g.S * g.C) / 40.0)
        q_res = np.float32(0.3) * q_out
        ocs = g.K + pad
        codes, values = np.full((N, g.Ho, g.Wo, ocs), 77, np.int8), np.full((N, g.Ho, g.Wo, ocs), np.float32(-7.5))
        acc = orc.conv_i8(g, x, w, b)
        if kind == "real":
            orc.real_output(acc, q_x, q_w, relu, res, q_res, out=values, out_c_stride=ocs, out_c_off=pad)
        else:
            orc.requant(acc, orc.requant_scale(q_x, q_w, q_out), bool(relu), res,
                        orc.residual_scale(q_res, q_out) if with_res else 0.0, out=codes, out_c_stride=ocs, out_c_off=pad)
        if kind == "deq":
            values[..., pad:] = orc.D(codes[..., pad:], q_out)
        d = B.ConvDesc(N, H, W, g.C, g.K, g.R, g.S, g.stride_h, g.stride_w, g.pad_h, g.pad_w, relu=relu,
                       out_c_stride=ocs, out_c_off=pad)
        t = [dev(x), B.pack_weights(d, dev(w)), dev(b), torch.full(codes.shape, 77, dtype=torch.int8, device="cuda"),
             torch.full(values.shape, -7.5, device="cuda"), dev(res) if with_res else None]
        o = ops[i]
        o.kind, o.group, o.d, o.q_x, o.q_w, o.q_out, o.q_res = B.OP_CONV, 1, d, q_x, q_w, q_out, q_res
        o.flags = {"codes": 0, "real": B.OPF_REAL, "deq": B.OPF_DEQUANT}[kind]
        o.x, o.w, o.bias, o.y, o.y_f32 = (v.data_ptr() for v in t[:5])
        o.residual = t[5].data_ptr() if with_res else None
        keep.append(t)
        want.append((codes, values))
    assert B.lib.q8_group_variant(ops, n).decode().startswith("conv_i8_" + build)
    assert _run_ops(B, ops) == 0
    for i, (codes, values) in enumerate(want):
        assert np.array_equal(host(keep[i][3]), codes), GROUP_OUTPUTS[i]
        assert np.array_equal(host(keep[i][4]), values), GROUP_OUTPUTS[i]


def _dequantize_ops(B, n, lengths, offset_of=()):
    """A list of Q8_OP_DEQUANTIZE ops over int8 tensors of ``lengths``, those in ``offset_of`` one
    value behind an aligned address; (ops, tensors, outputs, factors)."""
    rng = np.random.default_rng(n)
    ops, zs, outs, factors = (B.Op * n)(), [], [], []
    for i in range(n):
        off = 1 if i in offset_of else 0
        zs.append(dev(rng.integers(-128, 128, lengths[i] + off).astype(np.int8))[off:])
        outs.append(torch.full((lengths[i] + off,), -7.0, device="cuda")[off:])
        factors.append(0.125 * (i + 1))
        o = ops[i]
        o.kind, o.flags, o.q_x = B.OP_DEQUANTIZE, B.OPF_IN_U8 * (i % 3 == 1), factors[i]
        o.x, o.n, o.y_f32 = zs[i].data_ptr(), lengths[i], outs[i].data_ptr()
    return ops, zs, outs, factors


def _run_ops(B, ops):
    import ctypes
    streams = (ctypes.c_void_p * 1)(torch.cuda.current_stream().cuda_stream)
    rc = B.lib.q8_run_ops(ops, len(ops), streams, 1)
    torch.cuda.synchronize()
    return rc


def test_run_ops_dequantises_a_long_list(B):
    """More tensors than one launch takes, unaligned and empty ones among them."""
    lengths = [4096 * (i % 3) + 5 * i for i in range(40)]
    ops, zs, outs, factors = _dequantize_ops(B, 40, lengths, offset_of=(3, 17, 39))
    assert lengths[0] == 0 and _run_ops(B, ops) == 0
    for i in range(40):
        assert torch.equal(outs[i], factors[i] * (zs[i].float() + 128 * (i % 3 == 1))), i


def test_run_ops_dequantises_what_stands_in_front_of_a_refused_op(B):
    lengths = [5000, 64, 1, 300, 77]
    ops, zs, outs, factors = _dequantize_ops(B, 5, lengths)
    ops[3].q_x = -1.0
    assert _run_ops(B, ops) == -1
    for i in range(5):
        want = factors[i] * (zs[i].float() + 128 * (i % 3 == 1)) if i < 3 else torch.full_like(outs[i], -7.0)
        assert torch.equal(outs[i], want), i


@pytest.mark.parametrize("refused", [1, 2, 3, None])
def test_run_ops_group_with_a_refused_op(B, refused):
    """Of a group of independent layers and poolings, those in front of the op that is refused for
    its arguments run and those behind it do not."""
    rng = np.random.default_rng(9)
    x = dev(rng.integers(-128, 128, (1, 9, 9, 64)).astype(np.int8))
    d = B.ConvDesc(N=1, H=9, W=9, C=64, K=32, R=1, S=1)
    w = B.pack_weights(d, dev(rng.integers(-128, 128, (32, 1, 1, 64)).astype(np.int8)))
    conv, pool = B.conv_int8(d, x, w, None, 0.01, 0.01, 0.5), B.pool_i8(x, "avg", 3, 3, 1, 1, 9, 9)
    ops, outs = (B.Op * 5)(), []
    for i, o in enumerate(ops):
        is_conv = i % 2 == 0
        outs.append(torch.full_like(conv if is_conv else pool, 55))
        o.group, o.x, o.y, o.q_x, o.q_out = 1, x.data_ptr(), outs[i].data_ptr(), 1.0, 1.0
        if is_conv:
            o.kind, o.d, o.w, o.q_x, o.q_w, o.q_out = B.OP_CONV, d, w.data_ptr(), 0.01, 0.01, 0.5
        else:
            o.kind, o.H, o.W, o.C, o.mode, o.d.N = B.OP_POOL, 9, 9, 64, 1, 1
            o.R, o.S, o.stride, o.pad, o.Ho, o.Wo, o.d.out_c_stride = 3, 3, 1, 1, 9, 9, 64
    if refused is not None:
        ops[refused].q_out = -1.0
    assert _run_ops(B, ops) == (0 if refused is None else -1)
    for i, out in enumerate(outs):
        ran = refused is None or i < refused
        assert torch.equal(out, (pool if i % 2 else conv) if ran else torch.full_like(out, 55)), i


# one layer per tiled build for unsigned codes and per-channel scales: 3x3 tiles of each split, the
# persistent 3x3 (32 and 64 channels, padding 0 and 1) and 1x1 kernels (the latter also with a residual), the rings of K = 128 rows and of
# eight wavefronts on 256 pixels, the image rows at both vertical strides; channel counts that end inside
# a tile and images that end inside one
EXT_CASES = [
    ("halo3_kernel<2,2,1,1,2,1,9>", dict(N=16, H=28, W=28, C=128, K=80, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,1,1,2,2,9>", dict(N=5, H=29, W=23, C=128, K=80, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,1,2,2,2>", dict(N=8, H=28, W=28, C=128, K=192, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,2,1,4>", dict(N=8, H=55, W=57, C=128, K=80, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,2,1,8>", dict(N=2, H=55, W=57, C=128, K=80, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,2,2,4>", dict(N=16, H=55, W=57, C=128, K=80, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<4,2,2,2,4>", dict(N=16, H=55, W=57, C=128, K=144, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<4,2,2,2,8>", dict(N=4, H=89, W=131, C=128, K=144, R=3, S=3, pad_h=1, pad_w=1)),
    ("p3b_kernel", dict(N=12, H=55, W=57, C=64, K=64, R=3, S=3, pad_h=1, pad_w=1)),
    ("pw_kernel<1,1>", dict(N=24, H=55, W=57, C=64, K=64, R=1, S=1)),
    ("pw_kernel<1,1> + residual", dict(N=24, H=55, W=57, C=64, K=80, R=1, S=1)),
    ("ring_kernel<2,2,1,1,128,4>", dict(N=24, H=37, W=35, C=128, K=128, R=1, S=1, stride_h=2, stride_w=2)),
    ("ring_kernel<2,4,2,1,64,4>", dict(N=16, H=37, W=35, C=512, K=80, R=1, S=1)),
    ("ring_kernel<4,2,2,2,64,3>", dict(N=34, H=37, W=35, C=320, K=272, R=1, S=1)),
    ("ring_kernel<2,2,2,1,64,2>", dict(N=8, H=117, W=117, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, in_c_stride=4)),
    ("stem_kernel", dict(N=8, H=135, W=137, C=3, K=64, R=7, S=7, stride_h=2, stride_w=2, in_c_stride=4)),
    ("stem_kernel", dict(N=12, H=37, W=97, C=3, K=48, R=5, S=5, in_c_stride=4)),
    ("p3b_kernel", dict(N=12, H=57, W=59, C=64, K=64, R=3, S=3)),
    ("p3b_kernel", dict(N=12, H=57, W=59, C=32, K=48, R=3, S=3)),
    ("p3b_kernel", dict(N=12, H=55, W=57, C=32, K=64, R=3, S=3, pad_h=1, pad_w=1)),
    ("pw_kernel<1,2> + residual", dict(N=2, H=91, W=113, C=128, K=80, R=1, S=1)),
    ("pw_kernel<2,2> + residual", dict(N=1, H=1, W=61441, C=128, K=272, R=1, S=1)),
    ("pw_kernel<2,4> + residual", dict(N=1, H=1, W=128129, C=256, K=368, R=1, S=1)),
    ("halo3_kernel<2,2,1,1,3,2,9>", dict(N=1, H=39, W=37, C=256, K=272, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,1,1,3,1,9>", dict(N=1, H=55, W=63, C=192, K=144, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,2,1,4,2>", dict(N=2, H=39, W=38, C=256, K=528, R=3, S=3, pad_h=1, pad_w=1)),
    ("halo3_kernel<2,2,2,1,5,2>", dict(N=1, H=66, W=95, C=256, K=272, R=3, S=3, pad_h=1, pad_w=1)),
    ("p3b_kernel", dict(N=12, H=57, W=59, C=64, K=144, R=3, S=3)),
    ("p3b_kernel", dict(N=12, H=55, W=57, C=32, K=144, R=3, S=3, pad_h=1, pad_w=1)),
    ("p3b_kernel", dict(N=1, H=183, W=181, C=64, K=528, R=3, S=3, pad_h=1, pad_w=1)),
    ("taps4_kernel", dict(N=8, H=135, W=137, C=3, K=64, R=3, S=3, in_c_stride=4)),
    ("taps4_kernel", dict(N=19, H=49, W=35, C=3, K=48, R=4, S=4, stride_h=3, stride_w=2, in_c_stride=4))]


@pytest.mark.parametrize("idx", range(len(EXT_CASES)))
def test_conv_extended_builds(B, idx):
    kernel, geom = EXT_CASES[idx]
    d = B.ConvDesc(relu=1, **geom)
    assert B.conv_variant(d) == "conv_i8_" + kernel.split()[0]
    image = d.C == 3
    rng = np.random.default_rng(900 + idx)
    w = rng.integers(-128, 128, (d.K, d.R, d.S, d.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, d.K).astype(np.int32)
    x = rng.integers(0, 128 if image else 256, (d.N, d.H, d.W, d.in_c_stride or d.C)).astype(np.uint8)
    res = None if image or kernel in ("p3b_kernel", "pw_kernel<1,1>") else rng.integers(0, 256, (d.N, d.Ho, d.Wo, d.K)).astype(np.uint8)

    def accumulate(codes):            # whole numbers below 2^53: exact in fp64
        acc = torch.nn.functional.conv2d(
            torch.from_numpy(codes[..., :d.C].astype(np.float64)).permute(0, 3, 1, 2),
            torch.from_numpy(w.astype(np.float64)).permute(0, 3, 1, 2), torch.from_numpy(b.astype(np.float64)),
            (d.stride_h, d.stride_w), (d.pad_h, d.pad_w))
        return acc.permute(0, 2, 3, 1).contiguous().numpy().astype(np.int32)

    packed = B.pack_weights(d, dev(w))
    scale = np.float32(60.0 / (74.0 * 147.0 * np.sqrt(d.R * d.S * d.C)))
    m_r, acc = np.float32(0.4), accumulate(x)
    taps, bias = (None, dev(b)) if image else B.u8_prepare(d, dev(w), dev(b))
    got = B.conv_u8(d, not image, 1, res is not None, dev(x.astype(np.int8) if image else _stored(x)), packed, bias,
                    taps, 1.0, float(scale), 1.0, None if res is None else dev(_stored(res)), float(m_r))
    assert np.array_equal(host(got), _stored(orc.requant_mixed(
        acc, orc.requant_scale(1.0, scale, 1.0), True, res, orc.residual_scale(m_r, 1.0), out_unsigned=True)))

    x_s, res_s = _stored(x) if not image else x.astype(np.int8), None if res is None else _stored(res)
    m = (scale * rng.uniform(0.3, 3.0, d.K)).astype(np.float32)
    got = B.conv_int8_per_channel(d, dev(x_s), packed, dev(b), dev(m), 1.0, None if res is None else dev(res_s), 0.4)
    acc = accumulate(x_s) if not image else acc
    assert np.array_equal(host(got), orc.requant_pc(acc, m, True, res_s, np.float32(0.4)))


# the pointwise family with Eq. D beside its codes: each build, tails in pixels and in the channel tile, slices, with and
# without a residual; values that are 4-byte aligned only, which that family does not take
@pytest.mark.parametrize("pixels,C,K,cs,off,shift", [
    (40961, 64, 80, 0, 0, 0), (40961, 64, 64, 96, 16, 0), (41999, 128, 80, 0, 0, 0), (61441, 128, 272, 0, 0, 0),
    (128129, 256, 368, 400, 32, 0), (40961, 64, 80, 0, 0, 1),
    # the last size that is written through the caches, and the first past them
    (65535, 64, 256, 0, 0, 0), (65536, 64, 256, 272, 16, 0), (52427, 128, 320, 336, 0, 0), (52429, 128, 320, 0, 0, 0)])
def test_pointwise_with_dequantized_output(B, pixels, C, K, cs, off, shift):
    d = B.ConvDesc(1, 1, pixels, C, K, 1, 1, relu=1, out_c_stride=cs, out_c_off=off)
    assert "pw_kernel" in B.conv_variant(d)
    g = torch.Generator(device="cuda").manual_seed(K)
    codes = lambda *s: torch.randint(-128, 128, s, dtype=torch.int8, device="cuda", generator=g)
    x, w, q_out = codes(1, 1, pixels, C), B.pack_weights(d, codes(K, 1, 1, C)), 0.03
    b = torch.randint(-20000, 20000, (K,), dtype=torch.int32, device="cuda", generator=g)
    for res in (None, codes(1, 1, pixels, K)):
        args = (x, w, b, 0.02, 0.0004, q_out, res, 0.02)
        want = torch.full((1, 1, pixels, cs or K), 77, dtype=torch.int8, device="cuda")
        B.conv_int8(d, *args, out=want)
        got, values = torch.full_like(want, 77), torch.full((want.numel() + shift,), -5.0, device="cuda")[shift:]
        values = values.view(want.shape)
        B.conv_int8_dequantized(d, *args, out=got, out_f32=values)
        assert torch.equal(got, want)
        expect = torch.full_like(values, -5.0)
        expect[..., off:off + K] = want[..., off:off + K].float() * q_out
        assert torch.equal(values, expect)


# layers that a call of its own takes in other tiles than a planned step: tails in pixels and channels, a residual,
# channel counts that are no multiple of 64, a column filter, a stride
RETILED = [
    ("ring_kernel<2,2,2,3,64,3>", dict(N=16, H=71, W=69, C=80, K=180, R=3, S=3), False),
    ("ring_kernel<2,2,2,1,64,4>", dict(N=5, H=61, W=67, C=320, K=176, R=1, S=7, pad_w=3), True),
    ("ring_kernel<4,2,2,2,64,3>", dict(N=1, H=119, W=117, C=272, K=400, R=5, S=5, pad_h=2, pad_w=2), False),
    ("halo3_kernel<4,2,2,4,4>", dict(N=14, H=37, W=39, C=256, K=500, R=3, S=3, pad_h=1, pad_w=1), True)]


@pytest.mark.parametrize("idx", range(len(RETILED)))
def test_conv_retiled(B, idx):
    kernel, geom, with_res = RETILED[idx]
    d = B.ConvDesc(relu=1, **geom)
    assert B.conv_call_variant(d) == "conv_i8_" + kernel != B.conv_variant(d)
    g = torch.Generator(device="cuda").manual_seed(idx)
    codes = lambda *s: torch.randint(-128, 128, s, dtype=torch.int8, device="cuda", generator=g)
    x, w = codes(d.N, d.H, d.W, d.C), B.pack_weights(d, codes(d.K, d.R, d.S, d.C))
    b = torch.randint(-20000, 20000, (d.K,), dtype=torch.int32, device="cuda", generator=g)
    args = (d, x, w, b, 0.02, 0.0004, 0.03, codes(d.N, d.Ho, d.Wo, d.K) if with_res else None, 0.02)
    got, want = B.conv_int8(*args), B.conv_int8(*args, variant=7)       # 64 x 64 tiles
    assert torch.equal(got, want) and 0 < int(want.float().std()) < 127


# the block-tiled 3x3 kernel: blocks that end inside the map in both directions, one row and one column,
# padding 0 and 1, 32 and 64 channels in, 16 to 64 out (blocks of 16 x 16 up to 32), images of several
# tiles and tiles beyond one per workgroup, slices; the last one with unsigned codes at the border, too (those
# without padding and on 64 channels: EXT_CASES)
P3B_CASES = [dict(N=1, H=1, W=1, C=32, K=16, pad_h=1, pad_w=1), dict(N=3, H=17, W=16, C=32, K=32, pad_h=1, pad_w=1),
             dict(N=2, H=19, W=35, C=32, K=32, pad_h=0, pad_w=0), dict(N=2, H=9, W=33, C=32, K=48, pad_h=1, pad_w=1),
             dict(N=2, H=10, W=18, C=32, K=64, pad_h=0, pad_w=0), dict(N=1, H=1, W=40, C=64, K=64, pad_h=1, pad_w=1),
             dict(N=2, H=23, W=17, C=64, K=16, pad_h=0, pad_w=0), dict(N=61, H=50, W=49, C=32, K=32, pad_h=1, pad_w=1),
             dict(N=40, H=47, W=50, C=32, K=64, pad_h=1, pad_w=1)]


@pytest.mark.parametrize("idx", range(len(P3B_CASES)))
def test_conv_block_tiles(B, idx):
    geom = dict(P3B_CASES[idx], R=3, S=3)
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(B.conv_num_variants())]
    v = names.index("conv_i8_p3b_kernel")
    _run_conv_case(B, geom, relu=bool(idx % 2), with_res=False, with_bias=idx % 3 != 0, seed=70 + idx, variant=v,
                   out_pad=16 * (idx % 3), out_off=16 * (idx % 3 == 2), dump_acc=False)
    d = B.ConvDesc(relu=1, **geom)
    if d.N * d.H * d.W < 32768 or d.K <= 32:
        return
    assert B.conv_variant(d) == "conv_i8_p3b_kernel"
    rng = np.random.default_rng(idx)
    x = rng.integers(0, 256, (d.N, d.H, d.W, d.C)).astype(np.uint8)
    w = rng.integers(-128, 128, (d.K, 3, 3, d.C)).astype(np.int8)
    b = rng.integers(-20000, 20000, d.K).astype(np.int32)
    taps, bias = B.u8_prepare(d, dev(w), dev(b))
    got = host(B.conv_u8(d, 1, 1, 0, dev(_stored(x)), B.pack_weights(d, dev(w)), bias, taps, 1.0, 1e-4, 1.0))
    xs = torch.nn.functional.pad(dev(x).float().permute(0, 3, 1, 2), (1, 1, 1, 1))
    acc = torch.zeros((d.N, d.H, d.W, d.K), dtype=torch.float64, device="cuda") + dev(b).double()
    for r in range(3):                 # sums of 288 products of at most 255 * 128: exact in fp64
        for s in range(3):
            part = xs[:, :, r:r + d.H, s:s + d.W].permute(0, 2, 3, 1).reshape(-1, d.C).double()
            acc += (part @ dev(w)[:, r, s].double().t().contiguous()).view(acc.shape)
    want = (acc.float() * torch.tensor(np.float32(np.float32(1.0) * np.float32(1e-4))).cuda()).round().clamp(0, 255)
    assert np.array_equal(got.astype(int) + 128, host(want.int()))


# the pointwise family by its rule, plain and extended: from the first size at which it is taken (320 tiles),
# at both tiles of 128 channels in, a last tile of one pixel, channel counts that end inside a tile
PW_RULE_CASES = [("<1,1>", (1, 1, 40833, 64, 64)), ("<1,2>", (2, 91, 113, 128, 80)), ("<2,2>", (1, 1, 61441, 128, 272)),
                 ("<2,4>", (1, 1, 128129, 256, 256))]


@pytest.mark.parametrize("build,size", PW_RULE_CASES)
@pytest.mark.parametrize("with_res", [False, True])
def test_conv_pointwise_rule(B, build, size, with_res):
    n, h, w_, c, k = size
    d = B.ConvDesc(N=n, H=h, W=w_, C=c, K=k, R=1, S=1, relu=1)
    assert B.conv_variant(d) == "conv_i8_pw_kernel" + build
    if build == "<1,1>":
        assert "pw" not in B.conv_variant(B.ConvDesc(N=1, H=1, W=319 * 128, C=c, K=k, R=1, S=1))
    rng = np.random.default_rng(c + k + with_res)
    x = rng.integers(-128, 128, (n, h, w_, c)).astype(np.int8)
    w = rng.integers(-128, 128, (k, 1, 1, c)).astype(np.int8)
    b = rng.integers(-20000, 20000, k).astype(np.int32)
    r = rng.integers(-128, 128, (n, h, w_, k)).astype(np.int8) if with_res else None
    # whole numbers below 2^24: exact in fp32
    acc = (x.reshape(-1, c).astype(np.float32) @ w.reshape(k, c).T.astype(np.float32)).astype(np.int32) + b
    acc = acc.reshape(n, h, w_, k)
    m = (np.float32(60.0 / (74.0 * 74.0 * np.sqrt(c))) * rng.uniform(0.3, 3.0, k)).astype(np.float32)
    got = B.conv_int8_per_channel(d, dev(x), B.pack_weights(d, dev(w)), dev(b), dev(m), 1.0,
                                  None if r is None else dev(r), 0.4)
    assert np.array_equal(host(got), orc.requant_pc(acc, m, True, r, np.float32(0.4)))
    got = B.conv_int8(d, dev(x), B.pack_weights(d, dev(w)), dev(b), 0.01, 0.01, 0.5,
                      None if r is None else dev(r), 0.2 if with_res else 0.0)
    one = np.full(k, orc.requant_scale(np.float32(0.01), np.float32(0.01), np.float32(0.5)), np.float32)
    m_r = orc.residual_scale(np.float32(0.2), np.float32(0.5))
    assert np.array_equal(host(got), orc.requant_pc(acc, one, True, r, m_r))


@pytest.mark.parametrize("geom", [
    dict(N=2, H=11, W=19, C=48, K=16, pad_h=1, pad_w=1), dict(N=1, H=1, W=1, C=48, K=80, pad_h=1, pad_w=1),
    dict(N=13, H=53, W=51, C=48, K=144, pad_h=0, pad_w=0), dict(N=2, H=9, W=33, C=112, K=64, pad_h=1, pad_w=1),
    dict(N=3, H=17, W=18, C=112, K=16, pad_h=0, pad_w=0), dict(N=8, H=147, W=35, C=112, K=80, pad_h=1, pad_w=1)])
def test_conv_block_tiles_of_channels_that_fill_no_patch(B, geom):
    """48 of 64 and 112 of 128: chunks of zeros in every half of the patch that is multiplied, or in its last one."""
    geom = dict(geom, R=3, S=3)
    names = [B.lib.q8_conv_variant_name(v).decode() for v in range(B.conv_num_variants())]
    _run_conv_case(B, geom, relu=geom["pad_h"] == 1, with_res=False, with_bias=True, seed=geom["C"] + geom["K"],
                   variant=names.index("conv_i8_p3b_kernel"), out_pad=16, out_off=16, dump_acc=False)
    if geom["N"] > 4:
        test_maximum_behind_a_layer(B, (3, 149, 167), geom["C"], 64 if geom["C"] < 64 else 80, geom["pad_h"], True, (96, 16))


@pytest.mark.parametrize("C,pad", [(32, 1), (64, 0)])
def test_conv_block_tiles_with_a_residual(B, C, pad):
    """A layer that the block-tiled kernel is chosen for by its sizes but cannot take: the general kernel,
    plain and with per-channel scales."""
    d = B.ConvDesc(N=3, H=131, W=97, C=C, K=48, R=3, S=3, pad_h=pad, pad_w=pad, relu=1)
    assert B.conv_variant(d) == "conv_i8_p3b_kernel"
    rng = np.random.default_rng(C + pad)
    x = rng.integers(-128, 128, (d.N, d.H, d.W, C)).astype(np.int8)
    w = rng.integers(-128, 128, (d.K, 3, 3, C)).astype(np.int8)
    b = rng.integers(-20000, 20000, d.K).astype(np.int32)
    r = rng.integers(-128, 128, (d.N, d.Ho, d.Wo, d.K)).astype(np.int8)
    acc = torch.nn.functional.conv2d(          # whole numbers below 2^24: exact in fp32
        torch.from_numpy(x.astype(np.float32)).permute(0, 3, 1, 2),
        torch.from_numpy(w.astype(np.float32)).permute(0, 3, 1, 2), padding=pad)
    acc = acc.permute(0, 2, 3, 1).contiguous().numpy().astype(np.int32) + b
    packed = B.pack_weights(d, dev(w))
    m = (np.float32(60.0 / (74.0 * 74.0 * np.sqrt(9 * C))) * rng.uniform(0.3, 3.0, d.K)).astype(np.float32)
    got = B.conv_int8_per_channel(d, dev(x), packed, dev(b), dev(m), 1.0, dev(r), 0.4)
    assert np.array_equal(host(got), orc.requant_pc(acc, m, True, r, np.float32(0.4)))
    got = B.conv_int8(d, dev(x), packed, dev(b), 0.01, 0.01, 0.5, dev(r), 0.2)
    one = np.full(d.K, orc.requant_scale(0.01, 0.01, 0.5), np.float32)
    assert np.array_equal(host(got), orc.requant_pc(acc, one, True, r, orc.residual_scale(0.2, 0.5)))
