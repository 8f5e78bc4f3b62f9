"""Host-side checks of the engine: what it refuses and how it orders layers (no GPU)."""
import pytest
import torch

B = pytest.importorskip("paper_1805_08691_amd.binding")

from paper_1805_08691_amd import workloads as wl          # noqa: E402
from paper_1805_08691_amd.engine import Engine            # noqa: E402


@pytest.mark.parametrize("batches", [[], iter(())])
def test_calibration_without_a_batch_is_refused(batches):
    eng = Engine(wl.bottleneck_block(), 1, device="cpu")
    eng.set_factors({"x": 0.5})
    with pytest.raises(ValueError):
        eng.calibrate(batches)
    assert eng.q == {"x": 0.5}


def _reused_names():
    """Networks that give a tensor's name a second time, in the three ways that orders matter."""
    def net(*layers):
        n = wl.Network("reuse", "x")
        n.tensor("x", 7, 9, 64)
        for name in ("t", "u", "v", "cat"):
            n.tensor(name, 7, 9, 64)
        for name, src, dst, K, off, res in layers:
            wl._conv(n, name, src, K, 1, 1, res=res, dst=dst, dst_c_off=off)
        n.outputs = [layers[-1][2]]
        return n
    return [
        # t is read by b, then written over by a layer that reads the image alone
        net(("a", "x", "t", 64, 0, None), ("b", "t", "u", 64, 0, None), ("c", "x", "t", 64, 0, None),
            ("d", "t", "v", 64, 0, "u")),
        # t is written twice with nothing between; a residual reads the second
        net(("a", "x", "t", 64, 0, None), ("b", "x", "u", 64, 0, None), ("c", "u", "v", 64, 0, None),
            ("d", "x", "t", 64, 0, None), ("e", "v", "u", 64, 0, "t")),
        # slices: side by side, then one written over, the last layers read by nothing
        net(("a", "x", "cat", 32, 0, None), ("b", "x", "cat", 32, 32, None), ("c", "cat", "t", 64, 0, None),
            ("d", "x", "cat", 48, 16, None), ("e", "t", "u", 64, 0, None), ("f", "u", "v", 64, 0, None)),
    ]


def _waits(net, a, b):
    """Whether op b, behind op a in the list, has to come after it."""
    def reads(o):
        return {o.src, getattr(o, "res", None)} - {None}

    def slice_(o):
        return o.dst_c_off, o.dst_c_off + (o.K if o.kind == "conv" else net.tensors[o.src].C)
    (a0, a1), (b0, b1) = slice_(a), slice_(b)
    return a.dst in reads(b) or b.dst in reads(a) or (a.dst == b.dst and a0 < b1 and b0 < a1)


@pytest.mark.parametrize("net", _reused_names() + [wl.bottleneck_block(), wl.resnet50(), wl.inception_v3(),
                                                   wl.ssd300_vgg16()], ids=lambda n: n.name)
def test_levels_keep_the_order_of_dependent_layers(net):
    eng = Engine(net, 1, device="cpu")
    members = eng._levels(net.ops, 1, lambda o: o.dst)
    level = {i: lv for lv, m in enumerate(members) for i in m}
    assert sorted(level) == list(range(len(net.ops)))
    for j, b in enumerate(net.ops):
        for i, a in enumerate(net.ops[:j]):
            assert not _waits(net, a, b) or level[i] < level[j], (a.name, b.name)
    if len(net.ops) > 10:                # independent layers do share a level
        assert len(members) < len(net.ops)


@pytest.fixture
def recorded(monkeypatch):
    """Engines on host memory, whose planned steps are recorded and not run: recorded(net, batch,
    **options) -> (engine, step), and step(x, dequant) the ops of one step."""
    def ptr(t, dtype=None):               # the checks of the binding, without a device
        if t is None:
            return None
        assert t.is_contiguous() and (dtype is None or t.dtype is dtype)
        return t.data_ptr()
    ops = []

    def run(arr, n, streams, n_streams):
        for o in arr:
            ops.append(B.Op.from_buffer_copy(o))
        return 0
    monkeypatch.setattr(B, "_ptr", ptr)
    monkeypatch.setattr(B, "_stream", lambda: 0)
    monkeypatch.setattr(B.lib, "q8_run_ops", run)

    def make(net, batch, **options):
        eng = Engine(net, batch, device="cpu", **options)
        eng.set_factors({name: 2.0 ** -i for i, name in enumerate(net.tensors)})
        for o in net.convs():
            eng.wq[o.name] = (torch.zeros(B.packed_weight_bytes(eng.desc[o.name]), dtype=torch.int8),
                              torch.zeros(o.K, dtype=torch.int32))
            eng.qw[o.name] = 0.5
        eng.allocate()

        def step(x=None, dequant=None):
            ops.clear()
            eng.run_step(x, dequant)
            assert ops
            return list(ops)
        return eng, step
    return make


def test_planned_step_follows_storage_and_names(recorded):
    """A tensor may be given other storage, and a table the same values under other names."""
    net = wl.bottleneck_block()
    eng, step = recorded(net, 2)
    conv, out = net.convs()[-1], net.outputs[0]
    first = step()[-1]
    assert first.w == eng.wq[conv.name][0].data_ptr() and first.y == eng.act[out].data_ptr()
    moved = [*eng.wq[conv.name], eng.act[out]]
    for t in moved:
        t.data = t.clone()
    o = step()[-1]
    assert [o.w, o.bias, o.y] == [t.data_ptr() for t in moved] and o.w != first.w
    names = [n for n in eng.q if n not in (conv.src, out)] + [conv.src, out]
    for order in (names, names[:-2] + [out, conv.src]):
        eng.q = dict(zip(order, (2.0 ** -i for i in range(len(names)))))
        o = step()[-1]
        assert (o.q_x, o.q_out) == (eng.q[conv.src], eng.q[out])


def test_planned_step_refuses_what_the_layer_calls_refuse(recorded):
    """Buffers of another type or with gaps are refused, layers without a bias are not."""
    net = wl.bottleneck_block()
    conv, out = net.convs()[-1], net.outputs[0]
    eng, step = recorded(net, 2)
    packed, bias = eng.wq[conv.name]
    eng.wq[conv.name] = packed, None
    assert step()[-1].bias is None
    for other in ((packed.view(torch.uint8), bias), (packed.repeat(2)[::2], bias), (packed, bias.long())):
        eng.wq[conv.name] = other
        with pytest.raises(AssertionError):
            step()
    eng.wq[conv.name] = packed, bias
    codes = eng.act[out]
    for other in (codes.float(), codes.repeat(1, 1, 1, 2)[..., ::2]):
        eng.act[out] = other
        with pytest.raises(AssertionError):
            step()


def test_planned_step_takes_buffers_longer_than_the_batch(recorded):
    net = wl.bottleneck_block()
    out = net.outputs[0]
    eng, step = recorded(net, 2)
    n = eng.act[out].numel()
    eng.act[out] = torch.cat([eng.act[out]] * 2)
    r = torch.empty(eng.act[out][:2].shape)
    deq = [o for o in step(None, {out: r}) if o.kind == B.OP_DEQUANTIZE]
    assert [o.n for o in deq] == [n] * len(deq)
    with pytest.raises(ValueError):
        step(None, {out: r[:1]})


@pytest.mark.parametrize("H, batch, pipelines, together", [(90, 4, 1, True), (90, 4, 2, False), (128, 4, 2, True),
                                                           (40, 4, 1, False)])
def test_values_beside_the_codes_are_by_the_launches_of_the_parts(recorded, H, batch, pipelines, together):
    """Eq. D joins a 1x1 layer where each part's launch is of the family that writes whole rows: 256 -> 1024 is from
    32 thousand pixels on, 90 x 90 on four images, and two of those are on the general kernel."""
    net = wl.Network("wide", "x")
    net.tensor("x", H, H, 256)
    net.tensor("y", H, H, 1024)
    wl._conv(net, "a", "x", 1024, 1, 1, dst="y")
    net.outputs = ["y"]
    eng, _ = recorded(net, batch)
    eng.parts = [(0, batch // 2), (batch // 2, batch - batch // 2)]
    eng._pipelines_pay = lambda ops: pipelines == 2
    (_, layers, behind), _, values, _ = eng._plan(False, ("y",))
    assert [o.d.N for o in layers] == [batch // pipelines] * pipelines
    assert [bool(o.flags & B.OPF_DEQUANT) for o in layers] == [together] * pipelines
    assert [o.kind for o in behind] == ([] if together else [B.OP_DEQUANTIZE])
    assert len(values) == (pipelines if together else 1)


def test_planned_step_needs_no_factor_of_a_real_valued_output(recorded):
    net = wl.bottleneck_block()
    out = net.outputs[0]
    eng, step = recorded(net, 2, real_outputs=True)
    assert eng.real == {out}
    del eng.q[out]
    o = step()[-1]
    assert o.flags == B.OPF_REAL and o.y_f32


def test_step_without_layers(recorded):
    net = wl.Network("nothing", "x")
    net.tensor("x", 5, 7, 16)
    net.outputs = ["x"]
    eng, step = recorded(net, 2)
    ops = step(torch.zeros((2, 5, 7, 16)), {"x": torch.zeros((2, 5, 7, 16))})
    assert [o.kind for o in ops] == [B.OP_QUANTIZE, B.OP_DEQUANTIZE]


@pytest.mark.parametrize("layers, late, covered", [
    ([("a", 0, 16), ("b", 16, 32)], False, True), ([("b", 16, 32), ("a", 0, 16)], False, True),
    ([("a", 0, 16), ("b", 16, 16)], False, False), ([("a", 0, 16), ("b", 32, 16)], False, False),
    ([("b", 16, 32)], False, False), ([("a", 0, 32), ("b", 16, 32)], True, True),
    ([("a", 0, 32), ("pool", 32, 16)], True, True), ([("a", 0, 16), ("read",), ("b", 16, 32)], False, False),
    ([("a", 0, 32), ("b", 32, 16), ("read",), ("c", 8, 16)], True, True)])
def test_slices_of_a_tensor(layers, late, covered):
    """What the calibration forward measures once complete and what it has to clear."""
    net = wl.Network("slices", "x")
    net.tensor("x", 5, 7, 16)
    net.tensor("cat", 5, 7, 48)
    for name, *at in layers:
        if name == "read":
            wl._conv(net, "read", "cat", 16, 1, 1)
        elif name == "pool":
            wl._pool(net, "pool", "x", 3, 1, 1, dst="cat", dst_c_off=at[0])
        else:
            wl._conv(net, name, "x", at[1], 1, 1, dst="cat", dst_c_off=at[0])
    assert Engine(net, 1, device="cpu")._slices("cat") == (late, covered)


def _two_pipelines(net, batch, **kw):
    eng = Engine(net, batch, device="cpu", **kw)
    return eng._pipelines_pay([o for o in net.ops if not eng.head or o is not eng.head[1]])


@pytest.mark.parametrize("image, batch, two", [(224, 16, False), (224, 20, False), (224, 22, True), (224, 24, True),
                                               (160, 40, False), (160, 48, True)])
def test_pipelines_of_layers_that_cannot_share_a_launch(image, batch, two):
    """Unsigned codes and per-channel scales have the same rule, for the same reason; the batches are
    those around the measured crossing."""
    net = wl.resnet50(image=image)
    assert _two_pipelines(net, batch, unsigned_activations=True) == two
    assert _two_pipelines(net, batch, per_channel_weights=True) == two


def test_pipelines_of_per_channel_layers_follow_the_unsigned_rule():
    net = wl.resnet50()
    for batch in range(4, 40):
        assert _two_pipelines(net, batch, unsigned_activations=True) == \
            _two_pipelines(net, batch, per_channel_weights=True), batch


@pytest.mark.parametrize("net, image, batch, two", [
    (wl.resnet50, 224, 16, False), (wl.resnet50, 224, 21, True), (wl.resnet50, 160, 32, False),
    (wl.resnet50, 160, 48, True), (wl.inception_v3, 299, 17, False), (wl.inception_v3, 299, 18, True),
    (wl.inception_v3, 235, 28, False), (wl.inception_v3, 235, 32, True), (wl.ssd300_vgg16, 300, 2, False),
    (wl.ssd300_vgg16, 300, 4, True), (wl.ssd300_vgg16, 270, 3, False),
    # times of one and of two, us: 377 and 349, 361 and 341, 341 and 332; 497 and 544, 583 and 546
    (wl.resnet50, 176, 28, True), (wl.resnet50, 180, 25, True), (wl.resnet50, 196, 20, True),
    (wl.inception_v3, 279, 20, False), (wl.inception_v3, 259, 26, True)])
def test_pipelines_of_layers_that_share_launches(net, image, batch, two):
    """The batches around the measured crossings (the fused head as a deployed model has it)."""
    assert _two_pipelines(net(image=image), batch, fuse_head=True) == two


def _two_blocks(*layers, H=56):
    """Layers (name, source, kernel, residual, tensor written) on 64 channels, tensors made as they come."""
    net = wl.Network("blocks", "x")
    net.tensor("x", H, H, 64)
    for name, src, R, res, dst in layers:
        if dst not in net.tensors:
            net.tensor(dst, H, H, 64)
        wl._conv(net, name, src, 64, R, R, res=res, dst=dst)
    net.outputs = [layers[-1][4]]
    return net


CHAIN = [("a", "x", 1, None, "ta"), ("b", "ta", 3, None, "tb"), ("c", "tb", 1, None, "tc")]


@pytest.mark.parametrize("layers, order, marked", [
    (CHAIN, "abc", "a"),
    # a last layer that would also begin the next block belongs to the first one only
    (CHAIN + [("d", "tc", 3, None, "td"), ("e", "td", 1, None, "te")], "abcde", "a"),
    (CHAIN + [("d", "tc", 3, None, "td"), ("e", "td", 1, None, "te"), ("f", "te", 3, None, "tf"),
              ("g", "tf", 1, None, "tg")], "abcdefg", "ae"),
    # ... where it has a sum, the next block begins with another layer
    (CHAIN[:2] + [("c", "tb", 1, "x", "tc"), ("d", "tc", 1, None, "td"), ("e", "td", 3, None, "te"),
                  ("f", "te", 1, "tc", "tf")], "abcdef", "ad"),
    # an independent layer keeps its place in front of the block's
    (CHAIN[:2] + [("p", "x", 1, None, "tp"), CHAIN[2]], "pabc", "a"),
    # another layer reads what lies between, as its input or as its residual
    (CHAIN + [("d", "ta", 1, None, "td")], None, ""), (CHAIN + [("d", "tc", 1, "tb", "td")], None, ""),
    # the block's input, a tensor inside it or its output is written over behind its first layer
    (CHAIN[:1] + [("d", "ta", 1, None, "x")] + CHAIN[1:], None, ""),
    (CHAIN[:2] + [("p", "x", 1, None, "x"), CHAIN[2]], None, ""),
    (CHAIN[:2] + [("p", "x", 1, None, "tc"), CHAIN[2]], None, ""),
    (CHAIN + [("d", "tc", 1, None, "ta")], None, ""),
    # its residual is written behind the first layer, or in front of it
    (CHAIN[:2] + [("p", "x", 1, None, "tp"), ("c", "tb", 1, "tp", "tc")], None, ""),
    ([("p", "x", 1, None, "tp")] + CHAIN[:2] + [("c", "tb", 1, "tp", "tc")], "pabc", "a"),
    # no block: its layers in another order, or two 3x3 layers
    ([("a", "x", 3, None, "ta"), ("b", "ta", 1, None, "tb"), ("c", "tb", 1, None, "tc")], "abc", ""),
    ([("a", "x", 1, None, "ta"), ("b", "ta", 3, None, "tb"), ("c", "tb", 3, None, "tc")], "abc", "")])
def test_blocks_of_a_planned_step(recorded, layers, order, marked):
    """Which triples are marked as one launch, in which place, and that every layer runs once."""
    net = _two_blocks(*layers)
    eng, step = recorded(net, 4)
    at = {eng.wq[o.name][0].data_ptr(): o.name for o in net.convs()}
    ops = step()
    names = "".join(at[o.w] for o in ops)
    assert sorted(names) == sorted(o.name for o in net.convs()) and names == (order or names)
    assert "".join(n for n, o in zip(names, ops) if o.flags & B.OPF_BLOCK) == marked
    for n, o in zip(names, ops):
        assert not (o.flags & B.OPF_BLOCK and o.group)


def test_a_block_whose_inner_values_leave_is_none(recorded):
    """Eq. D of a tensor inside a block, in the launch that writes it: the block's layers keep their places."""
    net = _two_blocks(*CHAIN)
    for name, marked in (("ta", 0), ("tb", 0), ("tc", 0), (None, 1)):
        eng, step = recorded(net, 4, fuse_dequant=True)
        ops = step(None, {name: torch.empty(eng.act[name].shape)} if name else None)
        assert sum(bool(o.flags & B.OPF_BLOCK) for o in ops) == marked
        assert all(o.group for o in ops) == (not marked)


@pytest.mark.parametrize("batch, pipelines, blocks", [
    (1, 1, "2a 2b 2c"), (8, 1, "2a 2b 2c 3a 3b 3c 3d"), (13, 1, "2a 2b 2c 3a 3b 3c 3d 4b 4c 4d 4e 4f"),
    (13, 2, "2a 2b 2c 3a 3b 3c 3d 4a 4b 4c 4d 4e 4f")])
def test_blocks_of_resnet50(recorded, batch, pipelines, blocks):
    """The blocks that are marked: a projection's launch, which a first layer would share, counts on one pipeline."""
    net = wl.resnet50()
    eng, _ = recorded(net, batch)
    levels = eng._levels(net.ops, batch, lambda o: o.dst) if pipelines == 1 else None
    found = eng._blocks(net.ops, {}, batch, levels)
    assert " ".join(net.ops[i].name[3:5] for i in sorted(found)) == blocks
