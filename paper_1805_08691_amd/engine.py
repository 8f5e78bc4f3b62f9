"""Runs a layer list on the GPU through the C-ABI calls of ``binding``.

Host-side orchestration only: which call follows which, which buffer a layer reads and
writes, which factor goes with which tensor.  All arithmetic happens inside libq8conv.so.
Offline steps (in the paper's flow, Fig. "steps to generate the optimized model"):
  fold()               Eq. BN on every conv
  calibrate(batches)   fp32 forward of the folded net + running max-abs per tensor
  quantize_weights()   per-tensor q_w, int8 filters (packed), int32 bias at q_x * q_w
Online step:
  run_step(x, dequant) Q on the input image, one fused conv launch per layer (Eq. A'), D on the
                       outputs that leave the int8 domain; forward(x) is run_step without D.
"""
import ctypes
import itertools
import operator

import numpy as np
import torch

from . import binding as B

P_ACT = 7
P_W = 7
MAX_COPIES = 16       # copies of a maximum of calibration: a launch's atomics do not queue on one address


def _pad_c(c):
    """Stored channel count of an activation tensor (3-channel images are stored as 4)."""
    return 4 if c < 4 else c


class Engine:
    """``n_streams`` = 2 (up to 4) runs every layer as that many concurrent part-batch pipelines
    (batch elements are independent once the factor table is frozen): one on the caller's
    stream, the others on side streams of the same (default) priority, forked behind the
    quantisation of the input and joined again before the outputs are dequantised.  A layer's launch latency and its
    tail then overlap the other half's work.  Results are the same bits as with one stream."""

    def __init__(self, net, batch, device="cuda", n_streams=1, unsigned_activations=False,
                 per_channel_weights=False, real_outputs=False, own_sum_factor=False,
                 fuse_pairs=False, chain=False, fuse_duals=False, fuse_head=False,
                 fuse_dequant=False):
        self.net = net
        # fuse_dequant: where run_step is asked for Eq. D of a tensor that one convolution writes
        # whole, that convolution writes the fp32 values beside its codes (same values; no
        # separate pass over the tensor)
        self.fuse_dequant = fuse_dequant
        self._deq = {}        # tensor name -> fp32 buffer of the running step (fused Eq. D)
        # fuse_head: Eq. Q on the input image, the first convolution and the max-pool behind it
        # run as one launch per pipeline where the library has a build for them (same
        # results; the image's codes and the convolution's own output are then not written
        # in a step that starts from the real-valued batch)
        self.fuse_head = fuse_head
        self.head = None      # (first conv, the pool fused into it or None)
        self._x = None        # the real-valued batch of the running step (fused head)
        # fuse_duals: two consecutive convolutions that read the same tensor and do not depend on
        # each other (a stage's projection branch and its first 1x1) run as one launch where
        # the library has a tile-shape pair for them
        self.fuse_duals = fuse_duals
        self.duals = {}       # first conv name -> second conv
        self.dualed = set()
        # chain: every run of consecutive convolutions the library can take as a list runs as
        # ONE persistent launch (q8_conv_chain_int8: the batch split over the XCDs, tiles
        # started by the completion of the tiles they read) instead of one launch per layer
        self.chain = chain
        self.chains = None    # [(first op index, one past the last, binding.ConvChain)]
        assert not (chain and (n_streams > 1 or unsigned_activations or per_channel_weights
                               or real_outputs or fuse_pairs))
        # fuse_pairs: a convolution whose output only one 1x1 layer reads runs together with
        # that layer in one launch where the library supports the pair (same results; the
        # intermediate tensor is then never written)
        self.fuse_pairs = fuse_pairs
        self.pairs = {}       # first conv name -> second conv (launched together)
        self.paired = set()   # names of the second convs
        # own_sum_factor: a fused sum's output is calibrated by its own max-abs instead of
        # the max(q1, q2) rule of Eq. + (a variant; implied by unsigned activations)
        self.own_sum_factor = own_sum_factor
        assert not (unsigned_activations and per_channel_weights)
        # real_outputs: a network output that a convolution writes whole and no layer reads
        # is produced as fp32 by that convolution (no int8 code, no separate Eq. D pass)
        self.real = set()
        if real_outputs:
            assert not (unsigned_activations or per_channel_weights)
            read = {o.src for o in net.ops} | {o.res for o in net.ops if o.kind == "conv" and o.res}
            for o in net.convs():
                if o.dst in net.outputs and o.dst not in read and net.tensors[o.dst].C == o.K:
                    self.real.add(o.dst)
        self.act_f32 = {}     # tensor name -> fp32 device buffer (real_outputs)
        self.per_channel = per_channel_weights
        self.m_vec = {}       # conv name -> per-channel scales (per_channel_weights)
        # Unsigned p = 8 codes for the outputs of ReLU layers (the calibration paragraph's
        # rule for non-negative tensors) and for max-poolings of such tensors; stored as
        # code - 128.  Everything else stays signed p = 7.
        self.unsigned = set()
        if unsigned_activations:
            for o in net.ops:
                if o.kind == "conv":
                    assert net.tensors[o.dst].C == o.K, "unsigned mode: no concatenations"
                    if o.relu:
                        self.unsigned.add(o.dst)
                else:
                    assert o.mode == "max" and net.tensors[o.dst].C == net.tensors[o.src].C
                    if o.src in self.unsigned:
                        self.unsigned.add(o.dst)
        self.taps = {}        # conv name -> table of accumulator start values (padded layers
                              # reading unsigned codes)
        self.N = batch
        self.dev = torch.device(device)
        assert 1 <= n_streams <= 4
        self.n_streams = min(n_streams, max(batch, 1))
        self.side = [torch.cuda.Stream(device=self.dev) for _ in range(self.n_streams - 1)]
        # the batch in n_streams nearly equal parts (the first ones one image larger)
        self.parts, lo = [], 0
        for i in range(self.n_streams):
            n = batch // self.n_streams + (1 if i < batch % self.n_streams else 0)
            self.parts.append((lo, n))
            lo += n
        # number of leading layers that run on the whole batch before it is split (none: the
        # pipelines start right behind the quantisation of the input)
        self.n_unsplit = 0 if self.n_streams > 1 else len(net.ops)
        self.part_desc = {}   # (conv name, images) -> ConvDesc
        # An image of fewer than 4 channels read by one convolution is stored inside a zero
        # frame that holds that layer's padding, and the layer runs without padding.
        self.in_frame = None
        t_in = net.tensors[net.input]
        readers = [o for o in net.convs() if o.src == net.input]
        if _pad_c(t_in.C) != t_in.C and len(readers) == 1 and readers[0].dil == 1:
            o = readers[0]
            self.in_frame = (o.pad_h, o.pad_w, t_in.H + 2 * o.pad_h, t_in.W + 2 * o.pad_w)
        self.params = {}      # conv name -> dict of fp32 device tensors
        self.folded = {}      # conv name -> (W', b')
        self.q = {}           # tensor name -> activation factor (host float)
        self.qw = {}          # conv name -> weight factor
        self.wq = {}          # conv name -> (packed int8 filters, int32 bias)
        self.act = {}         # tensor name -> int8 device buffer [N, H, W, C_stored]
        self.desc = {}        # conv name -> ConvDesc
        self.graph = None
        self._plans = {}      # (real-valued batch given, tensors dequantised) -> planned step
        for op in net.ops:
            if op.kind == "conv":
                self.desc[op.name] = self._desc(op, batch)
        if fuse_pairs:
            assert not (unsigned_activations or per_channel_weights)
            self._find_pairs()
        if fuse_head:
            assert not (unsigned_activations or per_channel_weights or chain)
            self._find_head()
        if fuse_duals:
            assert not (unsigned_activations or per_channel_weights or real_outputs)
            self._find_duals()

    def _find_head(self):
        ops, t_in = self.net.ops, self.net.tensors[self.net.input]
        if not self.in_frame or not ops or ops[0].kind != "conv" or ops[0].src != self.net.input:
            return
        conv = ops[0]
        if conv.res or conv.dst_c_off or conv.name in self.pairs or conv.name in self.duals \
                or conv.dst in self.real:
            return
        top, left = self.in_frame[:2]
        pool = None
        if len(ops) > 1 and ops[1].kind == "pool" and ops[1].src == conv.dst:
            o = ops[1]
            others = [u for u in ops[2:] if u.src == conv.dst or (u.kind == "conv" and u.res == conv.dst)]
            s, d = self.net.tensors[o.src], self.net.tensors[o.dst]
            if (o.mode == "max" and (o.R, o.S, o.stride, o.pad) == (3, 3, 2, 1) and not others
                    and conv.dst not in self.net.outputs and d.C == s.C and o.dst_c_off == 0
                    and (d.H, d.W) == ((s.H - 1) // 2 + 1, (s.W - 1) // 2 + 1)):
                pool = o
        for cand in ((pool,) if pool is None else (pool, None)):
            if B.conv_image_f32_supported(self.desc[conv.name], t_in.H, t_in.W, t_in.C, top, left,
                                          1 if cand else 0):
                self.head = (conv, cand)
                return

    def _find_duals(self):
        ops = self.net.ops
        n_part = self.parts[0][1]
        for a, b in zip(ops, ops[1:]):
            if a.kind != "conv" or b.kind != "conv" or a.src != b.src:
                continue
            if a.name in self.dualed or a.name in self.pairs or b.name in self.pairs or \
                    a.name in self.paired or b.name in self.paired:
                continue
            if a.dst in (b.src, b.res) or b.dst in (a.src, a.res) or a.dst == b.dst:
                continue
            if B.conv_dual_supported(self.conv_desc(a, n_part), self.conv_desc(b, n_part)):
                self.duals[a.name] = b
                self.dualed.add(b.name)

    def _find_pairs(self):
        net = self.net
        ops = net.ops
        for i, a in enumerate(ops):
            if a.kind != "conv" or a.res or a.dst in net.outputs or a.dst in self.real:
                continue
            if net.tensors[a.dst].C != a.K or a.name in self.paired:
                continue
            readers = [o for o in ops if o.src == a.dst or (o.kind == "conv" and o.res == a.dst)]
            if len(readers) != 1 or readers[0].kind != "conv" or readers[0].src != a.dst:
                continue
            b = readers[0]
            if b.dst in self.real or ops.index(b) != i + 1:
                continue
            # both launches must lie on the same side of the half-batch split
            if (i < self.n_unsplit) != (i + 1 < self.n_unsplit):
                continue
            if B.conv_pair_supported(self.desc[a.name], self.desc[b.name]):
                self.pairs[a.name] = b
                self.paired.add(b.name)

    # ------------------------------------------------------------------ descriptors
    def _desc(self, op, N, framed=True):
        s, d = self.net.tensors[op.src], self.net.tensors[op.dst]
        res_cs = _pad_c(self.net.tensors[op.res].C) if op.res else 0
        H, W, pad_h, pad_w = s.H, s.W, op.pad_h, op.pad_w
        if framed and op.src == self.net.input and self.in_frame:
            _, _, H, W = self.in_frame
            pad_h = pad_w = 0
        desc = B.ConvDesc(N, H, W, op.C, op.K, op.R, op.S, op.stride, op.stride, pad_h, pad_w,
                          op.dil, op.dil, relu=op.relu, in_c_stride=_pad_c(s.C),
                          out_c_stride=_pad_c(d.C), out_c_off=op.dst_c_off, res_c_stride=res_cs)
        assert (desc.Ho, desc.Wo) == (d.H, d.W), (op.name, desc.Ho, desc.Wo, d)
        return desc

    # ------------------------------------------------------------------ offline steps
    def load_params(self, params):
        for name, p in params.items():
            self.params[name] = {k: (torch.from_numpy(v).to(self.dev) if isinstance(v, np.ndarray)
                                     else v) for k, v in p.items()}

    def fold(self):
        for op in self.net.convs():
            p = self.params[op.name]
            self.folded[op.name] = B.fold_bn(p["W"], p["b"], p["gamma"], p["beta"], p["mu"],
                                             p["var"], p["eps"])

    def forward_f32(self, x, observe=None):
        """fp32 forward of the folded network: its tensors by name.  ``observe(key, tensor)`` sees
        every activation (tensors written in slices once they are complete) and every value in
        front of a fused sum."""
        return self._forward_f32(x, None, observe)

    def _forward_f32(self, x, slot, observe=None):
        """The fp32 forward.  With ``slot`` (device tensors of MAX_COPIES copies by key, see
        conv_f32_observed) it leaves the running max-abs of every tensor there and keeps no tensor longer
        than it is read: a convolution
        takes the maxima of its own output and of its value before a fused sum while it holds
        them; a stand-alone pooling keeps its input's factor and is not measured."""
        net, N = self.net, x.shape[0]
        t = {net.input: x}
        last_use = {}
        for i, op in enumerate(net.ops):
            last_use[op.src] = i
            if op.kind == "conv" and op.res is not None:
                last_use[op.res] = i
        last_write = {op.dst: i for i, op in enumerate(net.ops)}
        slices = {}             # tensors written in slices: see _slices
        for i, op in enumerate(net.ops):
            d = net.tensors[op.dst]
            width = op.K if op.kind == "conv" else net.tensors[op.src].C
            observed = slot[op.dst] if slot else None
            if d.C == width:        # written whole
                out = torch.empty((N, d.H, d.W, d.C), dtype=torch.float32, device=self.dev)
            else:                   # a slice: channels that are read unwritten are zeros
                if op.dst not in slices:
                    slices[op.dst] = self._slices(op.dst)
                late, covered = slices[op.dst]
                out = t.get(op.dst)
                if out is None:
                    make = torch.empty if covered else torch.zeros
                    out = make((N, d.H, d.W, d.C), dtype=torch.float32, device=self.dev)
                if late:
                    observed = None
            if op.kind == "pool":
                B.pool_f32(t[op.src], op.mode, op.R, op.S, op.stride, op.pad, d.H, d.W, out=out,
                           out_c_off=op.dst_c_off)
            else:
                Wf, bf = self.folded[op.name]
                desc = self._desc(op, N, framed=False)
                desc.in_c_stride = desc.res_c_stride = 0
                desc.out_c_stride = d.C
                branch = op.name + ":branch"       # the value before the sum
                if op.res and observe:
                    desc.relu = 0
                    observe(branch, B.conv_f32_ref(desc, t[op.src], Wf, bf))
                    desc.relu = int(op.relu)
                B.conv_f32_observed(desc, t[op.src], Wf, bf, t[op.res] if op.res else None, out,
                                    slot[branch] if op.res and slot else None, observed,
                                    MAX_COPIES if slot else 1)
            if slot and last_write[op.dst] == i and slices.get(op.dst, (False,))[0]:
                B.calibrate_maxabs(out, slot[op.dst][:1])
            t[op.dst] = out
            if observe and d.C == width:
                observe(op.dst, out)
            for name in {op.src, getattr(op, "res", None)}:
                if slot and name is not None and last_use.get(name) == i and last_write.get(name, i) <= i:
                    del t[name]
        if observe:
            for name in slices:
                observe(name, t[name])
        return t

    def _slices(self, name):
        """Of a tensor written in slices: whether it is measured once complete (a pooling takes no
        maximum, and of slices that are written over only the last values count), and whether
        all of its channels are written before any is read."""
        written, before, late, read = [], [], False, False
        for op in self.net.ops:
            read = read or name in (op.src, getattr(op, "res", None))
            if op.dst != name:
                continue
            lo = op.dst_c_off
            hi = lo + (op.K if op.kind == "conv" else self.net.tensors[op.src].C)
            if hi - lo == self.net.tensors[name].C:
                continue
            late = late or op.kind == "pool" or any(a < hi and lo < b for a, b in written)
            written.append((lo, hi))
            if not read:
                before.append((lo, hi))
        end = 0
        for lo, hi in sorted(before):
            if lo <= end:
                end = max(end, hi)
        return late, end == self.net.tensors[name].C

    def calibrate(self, batches):
        """Running max-abs over fp32 forwards of ``batches`` (device fp32 NHWC tensors, at least
        one)."""
        keys = [self.net.input]
        for op in self.net.ops:
            if op.kind == "conv" and op.res is not None:
                keys.append(op.name + ":branch")
            if op.dst not in keys:
                keys.append(op.dst)
        spread = torch.zeros((len(keys), MAX_COPIES * B.SLOT_STRIDE), dtype=torch.float32, device=self.dev)
        slot = dict(zip(keys, spread.unbind()))
        n_batches = 0
        for x in batches:
            B.calibrate_maxabs(x.contiguous(), slot[self.net.input][:1])
            self._forward_f32(x.contiguous(), slot)
            n_batches += 1
        if not n_batches:
            raise ValueError("calibrate: no batches")     # every factor would be 1
        vals = B.calibrate_fold(spread, torch.empty(len(keys), device=self.dev)).cpu().numpy()
        # qfactor of every key: one fp32 division, 1 for a maximum that is not positive
        levels = np.array([255 if k in self.unsigned else 2 ** P_ACT - 1 for k in keys], dtype=np.float32)
        q = dict(zip(keys, np.where(vals > 0, vals / levels, np.float32(1)).tolist()))
        for op in self.net.ops:
            if (op.kind == "conv" and op.res is not None and not self.unsigned
                    and not self.own_sum_factor):
                q[op.dst] = B.sum_factor(q[op.name + ":branch"], q[op.res])   # Eq. +
            if op.kind == "pool" and self.net.tensors[op.dst].C == self.net.tensors[op.src].C:
                q[op.dst] = q[op.src]       # a stand-alone pool keeps its input's factor
        self.q = q
        self._plans.clear()
        return q

    def set_factors(self, q):
        self._plans.clear()
        self.q = {k: float(v) for k, v in q.items()}

    def quantize_weights_per_channel(self):
        self._plans.clear()
        for op in self.net.convs():
            Wf, bf = self.folded[op.name]
            q_w, z_w = B.quantize_weights_per_channel(Wf, P_W)
            self.zw_dense = getattr(self, "zw_dense", {})
            self.zw_dense[op.name] = z_w
            self.qw[op.name] = q_w
            self.wq[op.name] = (B.pack_weights(self.desc[op.name], z_w),
                                B.quantize_bias_per_channel(bf, self.q[op.src], q_w))
            self.m_vec[op.name] = B.requant_scales(self.q[op.src], q_w, self.q[op.dst])

    def quantize_weights(self):
        self._plans.clear()
        if self.per_channel:
            return self.quantize_weights_per_channel()
        slots = {}
        for op in self.net.convs():
            Wf, _ = self.folded[op.name]
            slots[op.name] = torch.zeros(1, dtype=torch.float32, device=self.dev)
            B.calibrate_maxabs(Wf, slots[op.name])
        names = list(slots)
        vals = torch.cat([slots[k] for k in names]).cpu().numpy()
        self.zw_dense = {}
        for name, v in zip(names, vals):
            op = next(o for o in self.net.convs() if o.name == name)
            Wf, bf = self.folded[name]
            q_w = B.qfactor(float(v), P_W)
            z_w = B.quantize(Wf, q_w, P_W)
            self.zw_dense[name] = z_w
            self.qw[name] = q_w
            bias = B.quantize_bias(bf, self.q[op.src], q_w)
            if op.src in self.unsigned:
                self.taps[name], bias = B.u8_prepare(self.desc[name], z_w, bias)
            self.wq[name] = (B.pack_weights(self.desc[name], z_w), bias)

    # ------------------------------------------------------------------ online step
    def allocate(self):
        self._plans.clear()
        for name, t in self.net.tensors.items():
            H, W = t.H, t.W
            if name == self.net.input and self.in_frame:
                H, W = self.in_frame[2:]
            self.act[name] = torch.zeros((self.N, H, W, _pad_c(t.C)), dtype=torch.int8,
                                         device=self.dev)
            if name in self.real:
                self.act_f32[name] = torch.zeros((self.N, H, W, _pad_c(t.C)),
                                                 dtype=torch.float32, device=self.dev)

    def input_codes(self):
        """The int8 codes of the network input without the frame: [N, H, W, C_stored]."""
        a = self.act[self.net.input]
        if not self.in_frame:
            return a
        t = self.net.tensors[self.net.input]
        top, left = self.in_frame[:2]
        return a[:, top:top + t.H, left:left + t.W]

    def quantize_input(self, x, lo=0, n=None):
        """Eq. Q on images [lo, lo + n) of the fp32 batch ``x`` into the input's codes."""
        n = self.N if n is None else n
        t = self.net.tensors[self.net.input]
        x = x[lo:lo + n]
        z = self.act[self.net.input][lo:lo + n]
        if self.in_frame:
            B.quantize_image(x, self.q[self.net.input], P_ACT, z, self.in_frame[0], self.in_frame[1])
        elif _pad_c(t.C) != t.C:
            B.quantize_pad_channels(x, _pad_c(t.C), self.q[self.net.input], P_ACT, out=z)
        else:
            B.quantize(x, self.q[self.net.input], P_ACT, out=z)

    def _dequant_writer(self, name, any_engine=False):
        """The convolution that writes Eq. D of tensor ``name`` beside its codes (in an engine with
        ``fuse_dequant``; ``any_engine``: the one that could), or None."""
        if not (self.fuse_dequant or any_engine) or self.unsigned or self.per_channel or name in self.real:
            return None
        writers = [o for o in self.net.ops if o.dst == name]
        if len(writers) != 1 or writers[0].kind != "conv":
            return None
        o = writers[0]
        if o.dst_c_off or self.net.tensors[name].C != o.K or _pad_c(o.K) != o.K:
            return None
        if o.name in self.paired or o.name in self.dualed or o.name in self.pairs or o.name in self.duals:
            return None
        if self.head and o is self.head[0]:
            return None
        return o

    def set_input(self, x):
        """The real-valued batch of the next layers: with a fused head it is only remembered
        (the head's launches apply Eq. Q), otherwise Eq. Q runs on it now."""
        if self.head:
            self._x = x
        else:
            self.quantize_input(x)

    def run_head(self, lo, n):
        conv, pool = self.head
        packed, bias = self.wq[conv.name]
        dst = pool.dst if pool else conv.dst
        B.conv_image_f32(self.conv_desc(conv, n), self._x[lo:lo + n], self.in_frame[0],
                         self.in_frame[1], self.q[self.net.input], P_ACT, packed, bias,
                         self.qw[conv.name], self.q[conv.dst], pool=1 if pool else 0,
                         out=self.act[dst][lo:lo + n])

    def run_pool(self, op, lo=0, n=None):
        n = self.N if n is None else n
        s, d = self.net.tensors[op.src], self.net.tensors[op.dst]
        q_in, q_out = self.q[op.src], self.q[op.dst]
        src, dst = self.act[op.src][lo:lo + n], self.act[op.dst][lo:lo + n]
        if op.mode == "max" and q_in == q_out and _pad_c(d.C) == _pad_c(s.C):
            # exact copy of the maximum: the vectorised kernel
            B._check(B.lib.q8_maxpool_i8(src.data_ptr(), n, s.H, s.W, _pad_c(s.C), op.R, op.S,
                                         op.stride, op.pad, d.H, d.W, dst.data_ptr(),
                                         B._stream()))
        else:
            B.pool_i8(src, op.mode, op.R, op.S, op.stride, op.pad, d.H, d.W, q_in, q_out,
                      out=dst, out_c_off=op.dst_c_off)

    def conv_desc(self, op, n):
        """Descriptor of ``op`` over ``n`` images (the whole batch or one part of it)."""
        if n == self.N:
            return self.desc[op.name]
        key = (op.name, n)
        if key not in self.part_desc:
            self.part_desc[key] = self._desc(op, n)
        return self.part_desc[key]

    def run_conv(self, op, lo=0, n=None, acc_dump=None, fuse=True):
        n = self.N if n is None else n
        packed, bias = self.wq[op.name]
        res = self.act[op.res][lo:lo + n] if op.res else None
        q_res = self.q[op.res] if op.res else 0.0
        U = self.unsigned
        if (op.name in self.paired or op.name in self.dualed) and fuse:
            return                       # ran with the layer in front of it
        if op.name in self.duals and fuse:
            b = self.duals[op.name]

            def args(o):
                w, bias = self.wq[o.name]
                return (self.conv_desc(o, n), self.act[o.src][lo:lo + n], w, bias, self.q[o.src],
                        self.qw[o.name], self.q[o.dst],
                        self.act[o.res][lo:lo + n] if o.res else None,
                        self.q[o.res] if o.res else 0.0, self.act[o.dst][lo:lo + n])
            B.conv_dual_int8(args(op), args(b))
            return
        if op.name in self.pairs and fuse:
            b = self.pairs[op.name]
            packed2, bias2 = self.wq[b.name]
            res2 = self.act[b.res][lo:lo + n] if b.res else None
            B.conv_pair_int8(self.conv_desc(op, n), self.act[op.src][lo:lo + n], packed, bias,
                             self.q[op.src], self.qw[op.name], self.q[op.dst],
                             self.conv_desc(b, n), packed2, bias2, self.qw[b.name], self.q[b.dst],
                             res2, self.q[b.res] if b.res else 0.0,
                             out=self.act[b.dst][lo:lo + n])
            return
        if op.dst in self.real and acc_dump is None:
            B.conv_int8_real_output(self.conv_desc(op, n), self.act[op.src][lo:lo + n], packed,
                                    bias, self.q[op.src], self.qw[op.name], res, q_res,
                                    out=self.act_f32[op.dst][lo:lo + n])
            return
        if self.per_channel:
            B.conv_int8_per_channel(self.conv_desc(op, n), self.act[op.src][lo:lo + n], packed,
                                    bias, self.m_vec[op.name], self.q[op.dst], res, q_res,
                                    out=self.act[op.dst][lo:lo + n], acc_dump=acc_dump)
            return
        if op.src in U or op.dst in U or op.res in U:
            B.conv_u8(self.conv_desc(op, n), op.src in U, op.dst in U, op.res in U,
                      self.act[op.src][lo:lo + n], packed, bias, self.taps.get(op.name),
                      self.q[op.src], self.qw[op.name], self.q[op.dst], res, q_res,
                      out=self.act[op.dst][lo:lo + n], acc_dump=acc_dump)
            return
        if op.dst in self._deq and acc_dump is None:
            B.conv_int8_dequantized(self.conv_desc(op, n), self.act[op.src][lo:lo + n], packed, bias,
                                    self.q[op.src], self.qw[op.name], self.q[op.dst], res, q_res,
                                    out=self.act[op.dst][lo:lo + n],
                                    out_f32=self._deq[op.dst][lo:lo + n])
            return
        B.conv_int8(self.conv_desc(op, n), self.act[op.src][lo:lo + n], packed, bias,
                    self.q[op.src], self.qw[op.name], self.q[op.dst], res, q_res,
                    out=self.act[op.dst][lo:lo + n], acc_dump=acc_dump)

    def run_ops(self, ops, lo, n):
        for op in ops:
            if self._x is not None and self.head:
                if op is self.head[0]:
                    self.run_head(lo, n)
                    continue
                if op is self.head[1]:
                    continue             # ran inside the head's launch
            if op.kind == "pool":
                self.run_pool(op, lo, n)
            else:
                self.run_conv(op, lo, n)

    # ------------------------------------------------------------------ layer lists
    def _chainable(self, op):
        if op.kind != "conv" or op.dst_c_off != 0:
            return False
        s, d = self.net.tensors[op.src], self.net.tensors[op.dst]
        if d.C != op.K or s.C != op.C or (op.res and self.net.tensors[op.res].C != op.K):
            return False
        return B.conv_chain_supported(self.desc[op.name])

    def build_chains(self, variants=None):
        """Plan one q8_conv_chain_int8 launch per run of two or more chainable convolutions.
        ``variants`` ({conv name: tile variant}) forces tile shapes (tests, tuning)."""
        ops = self.net.ops
        self.chains = []
        i = 0
        while i < len(ops):
            j = i
            while j < len(ops) and self._chainable(ops[j]):
                j += 1
            if j - i >= 2:
                writer = {}
                layers = []
                for k, op in enumerate(ops[i:j]):
                    packed, bias = self.wq[op.name]
                    layers.append(dict(
                        desc=self.desc[op.name], z_x=self.act[op.src], w=packed, bias=bias,
                        q_x=self.q[op.src], q_w=self.qw[op.name], q_out=self.q[op.dst],
                        residual=self.act[op.res] if op.res else None,
                        q_res=self.q[op.res] if op.res else 0.0, out=self.act[op.dst],
                        src_layer=writer.get(op.src, -1),
                        res_layer=writer.get(op.res, -1) if op.res else -1,
                        variant=(variants or {}).get(op.name, -1)))
                    writer[op.dst] = k
                self.chains.append((i, j, B.ConvChain(layers, self.dev)))
                i = j
            else:
                i = max(j, i + 1)
        return self.chains

    def run_chained(self):
        """Every op on the whole batch: planned runs as one launch each, the rest one by one."""
        if self.chains is None:
            self.build_chains()
        ops = self.net.ops
        starts = {a: (b, c) for a, b, c in self.chains}
        i = 0
        while i < len(ops):
            if i in starts:
                end, ch = starts[i]
                ch.run()
                i = end
            else:
                self.run_ops([ops[i]], 0, self.N)
                i += 1

    # ------------------------------------------------------------------ the planned step
    # A step is described once as an array of library calls (binding.Op) and enqueued with one
    # call per stream segment; only the pointers of the real-valued batch and of the fp32
    # outputs are filled in per step.
    # (every address goes through the checks that the layer calls make)
    def _codes(self, name, lo, n):
        return B._ptr(self.act[name][lo:lo + n], torch.int8)

    def _op_conv(self, op, lo, n, deq):
        packed, bias = self.wq[op.name]
        U, o = self.unsigned, B.Op()
        o.kind, o.d = B.OP_CONV, self.conv_desc(op, n)
        o.x, o.y = self._codes(op.src, lo, n), self._codes(op.dst, lo, n)
        o.w, o.bias = B._ptr(packed, torch.int8), B._ptr(bias, torch.int32)
        o.q_x, o.q_out = self.q[op.src], 1.0 if op.dst in self.real else self.q[op.dst]
        o.q_w = 1.0 if self.per_channel else self.qw[op.name]
        if op.res:
            o.residual, o.q_res = self._codes(op.res, lo, n), self.q[op.res]
        if op.dst in self.real:
            o.flags, o.y_f32 = B.OPF_REAL, B._ptr(self.act_f32[op.dst][lo:lo + n], torch.float32)
        elif self.per_channel:
            o.flags, o.aux = B.OPF_PER_CHANNEL, B._ptr(self.m_vec[op.name], torch.float32)
        elif op.src in U or op.dst in U or op.res in U:
            o.flags = (B.OPF_IN_U8 * (op.src in U) | B.OPF_OUT_U8 * (op.dst in U) |
                       B.OPF_RES_U8 * (op.res in U))
            if op.src in U:
                o.aux = B._ptr(self.taps.get(op.name), torch.int32)
        elif deq:
            o.flags = B.OPF_DEQUANT
        return o

    def _op_pool(self, op, lo, n):
        s, d = self.net.tensors[op.src], self.net.tensors[op.dst]
        o = B.Op()
        exact = op.mode == "max" and self.q[op.src] == self.q[op.dst] and _pad_c(d.C) == _pad_c(s.C)
        o.kind = B.OP_MAXPOOL if exact else B.OP_POOL
        if exact:            # (run_pool checks nothing there either)
            o.x, o.y = self.act[op.src][lo:lo + n].data_ptr(), self.act[op.dst][lo:lo + n].data_ptr()
        else:
            o.x, o.y = self._codes(op.src, lo, n), self._codes(op.dst, lo, n)
        o.d.N, o.H, o.W, o.C = n, s.H, s.W, _pad_c(s.C)
        o.mode = 0 if op.mode == "max" else 1
        o.R, o.S, o.stride, o.pad, o.Ho, o.Wo = op.R, op.S, op.stride, op.pad, d.H, d.W
        o.q_x, o.q_out = self.q[op.src], self.q[op.dst]
        o.d.out_c_stride, o.d.out_c_off = _pad_c(d.C), op.dst_c_off
        return o

    def _op_quantize(self, n):
        t, o = self.net.tensors[self.net.input], B.Op()
        o.q_x, o.p, o.y = self.q[self.net.input], P_ACT, self._codes(self.net.input, 0, n)
        if self.in_frame:
            o.kind, o.d.N, o.H, o.W, o.C = B.OP_QUANTIZE_IMAGE, n, t.H, t.W, t.C
            o.top, o.left, o.Ho, o.Wo = self.in_frame
        elif _pad_c(t.C) != t.C:
            o.kind, o.n, o.C, o.Ho = B.OP_QUANTIZE_PAD, n * t.H * t.W, t.C, _pad_c(t.C)
        else:
            o.kind, o.n = B.OP_QUANTIZE, n * t.H * t.W * t.C
        return o

    def _op_head(self, lo, n):
        conv, pool = self.head
        packed, bias = self.wq[conv.name]
        t, o = self.net.tensors[self.net.input], B.Op()
        o.kind, o.flags, o.d = B.OP_HEAD, B.OPF_POOL if pool else 0, self.conv_desc(conv, n)
        o.H, o.W, o.C = t.H, t.W, t.C
        o.top, o.left = self.in_frame[:2]
        o.q_x, o.p, o.q_w, o.q_out = self.q[self.net.input], P_ACT, self.qw[conv.name], self.q[conv.dst]
        o.w, o.bias = B._ptr(packed, torch.int8), B._ptr(bias, torch.int32)
        o.y = self._codes(pool.dst if pool else conv.dst, lo, n)
        return o

    def _levels(self, ops, n, dst_of):
        """Level of every op: one more than the ops' it waits for (those that wrote what it reads,
        and where it writes over a tensor, those that read or wrote it before), and for an op that
        nothing waits for the level from that one on where it adds least (it then shares a launch,
        or the idle part of the chip, with the ops there)."""
        writers, readers, early, us, share = {}, {}, [], [], []
        waited_for = [False] * len(ops)
        for i, op in enumerate(ops):
            d, dst = self.net.tensors[op.dst], dst_of(op)
            reads = {op.src, getattr(op, "res", None)} - {None}
            lo = op.dst_c_off
            hi = lo + (op.K if op.kind == "conv" else _pad_c(self.net.tensors[op.src].C))
            waits = {j for name in reads for j, _, _ in writers.get(name, ())}
            waits.update(readers.get(dst, ()))
            # (slices of one tensor side by side do not wait for each other)
            waits.update(j for j, a, b in writers.get(dst, ()) if a < hi and lo < b)
            early.append(1 + max((early[j] for j in waits), default=-1))
            for j in waits:
                waited_for[j] = True
            for name in reads:
                readers.setdefault(name, []).append(i)
            writers.setdefault(dst, []).append((i, lo, hi))
            us.append(B.conv_estimate_us(self.conv_desc(op, n)) if op.kind == "conv" else 3.0)
            work = n * d.H * d.W * (op.K if op.kind == "conv" else d.C)
            share.append(min(1.0, work / 65536.0))     # tiles of 16 x 16 against 256 CUs
        depth = max(early, default=-1) + 1
        members = [[] for _ in range(depth)]
        cost = lambda m: (max([us[i] for i in m] + [2.7 + sum((us[i] - 2.7) * share[i] for i in m)])
                          if m else 0.0)
        loose = []
        for i in range(len(ops)):
            # only ops that no other op waits for: moving one never moves another
            if early[i] < depth - 1 and not waited_for[i]:
                loose.append(i)
            else:
                members[early[i]].append(i)
        for i in sorted(loose, key=lambda i: -us[i]):
            best = min(range(early[i], depth), key=lambda l: cost(members[l] + [i]) - cost(members[l]))
            members[best].append(i)
        return members

    def _plan(self, with_x, names):
        """The planned step: (ops before the pipelines fork, ops of the pipelines, ops behind the
        join, where the batch's and the outputs' pointers go)."""
        net, part_ops = self.net, []
        ops = list(net.ops)
        if with_x and self.head:
            ops = [o for o in ops if o is not self.head[1]]
        parts = self.parts
        if len(parts) > 1 and not self._pipelines_pay(ops):
            parts = [(0, self.N)]
        fused = {name: self._dequant_writer(name) for name in names}
        # Eq. D inside the launch that writes the tensor: asked for, free (a launch of the
        # latency family finishes four channels per lane whatever it writes), or a saved pass (the pointwise family
        # writes the values in whole rows from LDS: bottleneck block on 56 x 56, 32 images 69 -> 62 us, 64 images
        # 141 -> 132), here where that is worth more than the layer's block in one launch (256 channels, us with
        # the block and so: 75 thousand pixels 49.6 / 48.9, 102 thousand 67.5 / 62.0, 150 thousand 105.9 / 100.0; 48
        # thousand 36.0 / 36.7, 12.5 thousand 18.4 / 22.2), below where it ends no such block.  By the launch of every
        # part: half a batch may run on another family, whose tail writes the values four at a time
        could = {name: self._dequant_writer(name, any_engine=True) for name in names}
        writes = lambda w, family: w is not None and all(
            family in B.conv_variant(self.conv_desc(w, n)) for _, n in parts)
        fused.update({name: w for name, w in could.items() if fused[name] is None and (
            writes(w, "direct") or
            (writes(w, "pw_kernel") and self.N * self.act[name].shape[1:].numel() >= 1 << 24))})
        fused = {name: w for name, w in fused.items() if w is not None}
        x_slots, out_slots = [], []

        def add(into, o, stream=0, group=0):
            o.stream, o.group = stream, group
            into.append(o)
            return len(into) - 1

        pre, body, post = [], [], []
        t_in = net.tensors[net.input]
        image = 4 * t_in.H * t_in.W * t_in.C
        if with_x and not self.head:
            x_slots.append((0, add(pre, self._op_quantize(self.N)), 0))

        def emit(op, k, group):
            lo, n = parts[k]
            if with_x and self.head and op is self.head[0]:
                x_slots.append((1, add(body, self._op_head(lo, n), k, group), image * lo))
            elif op.kind == "pool":
                add(body, self._op_pool(op, lo, n), k, group)
            else:
                deq = fused.get(op.dst) is op
                i = add(body, self._op_conv(op, lo, n, deq), k, group)
                if deq:
                    values = self.act[op.dst].shape[1:].numel()
                    out_slots.append((1, i, op.dst, 4 * lo * values, self.N * values))
        pooled_head = with_x and self.head and self.head[1]
        dst_of = lambda o: self.head[1].dst if pooled_head and o is self.head[0] else o.dst
        # level by level, alternating between the pipelines: a captured graph hands its nodes to
        # the GPU in the order they were recorded, and a pipeline recorded whole before the next
        # one starts that much earlier and runs alone meanwhile
        levels = self._levels(ops, parts[0][1], dst_of)
        blocks = self._blocks(ops, fused, parts[0][1], levels if len(parts) == 1 else None)
        inside = {i for pair in blocks.values() for i in pair}
        fused.update({name: w for name, w in could.items() if name not in fused and writes(w, "pw_kernel") and
                      ops.index(w) not in inside | blocks.keys()})
        for level, members in enumerate(levels):
            for k in list(range(1, len(parts))) + [0]:
                for i in sorted(members):
                    if i in blocks:                  # the whole block, where its last layer has its place
                        first = len(body)
                        for j in (*blocks[i], i):
                            emit(ops[j], k, 0)
                        body[first].flags |= B.OPF_BLOCK
                    elif i not in inside:
                        emit(ops[i], k, level + 1)
        for name in names:
            if name in fused:
                continue
            o, z = B.Op(), self.act[name][:self.N]
            o.kind, o.flags = B.OP_DEQUANTIZE, B.OPF_IN_U8 if name in self.unsigned else 0
            o.x, o.n, o.q_x = B._ptr(z, torch.int8), z.numel(), self.q[name]
            out_slots.append((2, add(post, o), name, 0, z.numel()))
        segments = [(B.Op * len(s))(*s) for s in (pre, body, post)]
        return segments, x_slots, out_slots, len(parts)

    def _blocks(self, ops, fused, n, levels):
        """Bottleneck blocks that the library estimates shorter as one launch on ``n`` images: {index of the last
        layer: (1x1, 3x3)}.  ``levels``: counting what the first layer would share with its level's
        other layers; None (several pipelines, where launches of the others fill what a launch
        leaves idle): the three layers by themselves (ResNet-50 at 160 pixels, 44 images 386 us, counted 391).
        Only the block itself reads its inner tensors, and nothing behind its first layer writes over what it
        reads or writes: it can then run where its last layer has its place.  A layer belongs to one block
        (the first where one's last layer could begin another)."""
        at = {o.dst: i for i, o in enumerate(ops)}
        found, taken = {}, set()
        for i, c in enumerate(ops):
            if c.kind != "conv" or (c.R, c.S, c.stride, c.pad_h, c.pad_w) != (1, 1, 1, 0, 0):
                continue
            ib = at.get(c.src, i)
            b = ops[ib]
            if ib >= i or b.kind != "conv" or b.res or \
                    (b.R, b.S, b.stride, b.pad_h, b.pad_w, b.dil) != (3, 3, 1, 1, 1, 1):
                continue
            ia = at.get(b.src, ib)
            a = ops[ia]
            if ia >= ib or a.kind != "conv" or a.res or (a.R, a.S, a.pad_h, a.pad_w) != (1, 1, 0, 0) or \
                    taken & {ia, ib, i} or c.dst in self.real or {a.dst, b.dst, c.dst} & fused.keys() or \
                    (self.head and a is self.head[0]):
                continue
            touched = {a.src, c.res, a.dst, b.dst, c.dst}
            others = [o for j, o in enumerate(ops) if j not in (ia, ib, i)]
            if (any({a.dst, b.dst} & {o.src, getattr(o, "res", None)} for o in others) or
                    any(o.dst in touched for o in ops[ia + 1:] if o is not b and o is not c) or
                    any(o.dst in (a.dst, b.dst, c.dst) for o in others)):
                continue
            three = (B.Op * 3)(*(self._op_conv(o, 0, n, False) for o in (a, b, c)))
            if levels is None:
                pays = B.lib.q8_block_variant(three) != b"single launches"
            else:
                beside = [ops[j] for m in levels if ia in m for j in sorted(m) if j != ia and
                          ops[j].kind == "conv" and not (self.head and ops[j] is self.head[0])][:7]
                beside = (B.Op * len(beside))(*(self._op_conv(o, 0, n, fused.get(o.dst) is o) for o in beside))
                pays = B.lib.q8_block_pays(three, beside, len(beside))
            if pays:
                found[i] = (ia, ib)
                taken.update((ia, ib, i))
        return found

    def _pipelines_pay(self, ops):
        """Concurrent pipelines hide one launch's latency and tail behind the other's work, and cost
        a second set of launches (in a recorded graph also a dependency per launch): worth it
        where the layers' time on the whole batch is well above the latencies of the layers and of the
        levels they form (at least a launch each).  Fitted to both times of 285 steps around the crossing
        (ResNet-50 at 160 to 224 pixels, Inception-v3 at 235 to 299, the detector at 268 to 300): by the choice the
        steps take 1.002, 1.002 and 1.02 of the better one's time, 1.08 at worst.  A bottleneck block counts as its
        three layers though it is one launch.  us with one and with two: ResNet-50 18 images 325 / 326, 20: 358 / 354,
        22: 386 / 377, at 176 pixels 28 images 377 / 349, at 160 pixels 36 images 332 / 333; Inception-v3 17 images
        558 / 557, 18: 575 / 527, at 279 pixels 20 images 497 / 544, at 235 pixels 30 images 553 / 549, 32: 559 / 546;
        the detector 4 images 336 / 326, 5: 361 / 383, 6: 432 / 412.  Layers with unsigned codes or per-channel scales
        cannot share a launch, so a level counts as its layers: ResNet-50 16 images 341 / 361 and 344 / 361, 20:
        406 / 398 and 404 / 392, 22: 448 / 428 and 446 / 420; at 160 pixels 40 images 406 / 397 and 407 / 391,
        48: 480 / 446 and 487 / 453."""
        if self.N < 4:           # (unequal parts: the detector 3 images 291 / 330 us at 286 pixels, 336 / 326 at 300)
            return False
        us, depth = 0.0, {}
        for o in ops:
            us += B.conv_estimate_us(self.conv_desc(o, self.N)) if o.kind == "conv" else 0.0
            depth[o.dst] = max(depth.get(o.dst, 0), 1 + max(depth.get(o.src, 0),
                                                            depth.get(getattr(o, "res", None), 0)))
        levels = max(depth.values(), default=0)
        if len(ops) < 16:        # (the fork and the join count: a bottleneck block 32 images 52 / 85 us)
            return us > 8.5 * len(ops)
        if self.unsigned or self.per_channel:
            return us > 7.7 * len(ops)
        return us > 5.59 * len(ops) + 1.6 * levels

    def _plannable(self, x, dequant):
        """Not with the multi-layer kernels, and only for a batch of exactly the net's shape and
        for contiguous buffers (the plan holds one pointer to each; layer by layer takes a longer
        or flattened batch too, and buffers of which only the images it writes are contiguous)."""
        t = self.net.tensors[self.net.input]
        return not (self.chain or self.pairs or self.duals or any(
            name in self.real or (out is not None and not out.is_contiguous())
            for name, out in dequant.items())) and (
                x is None or (tuple(x.shape) == (self.N, t.H, t.W, t.C) and x.is_contiguous()))

    def _run_planned(self, x, dequant):
        names = tuple(name for name, out in dequant.items() if out is not None)
        key = (x is not None, names)
        # factors, switch, filters and buffers are attributes a program may set between steps, and a
        # tensor's storage may be another than it was: the plan holds for the same names, the same
        # objects (whose types and strides were checked) and the addresses that they have now
        given = [self.fuse_dequant, *self.q, *self.q.values(), *self.wq, *self.act, *self.taps, *self.m_vec]
        if not self.per_channel:
            given += self.qw.values()
        objects = itertools.chain(itertools.chain.from_iterable(self.wq.values()), self.act.values(),
                                  self.act_f32.values(), self.m_vec.values(), self.taps.values())
        plan, planned_for, planned_with, tensors, addresses = self._plans.get(key, (None,) * 5)
        if (planned_for != given or not all(map(operator.is_, planned_with, objects))
                or addresses != [*map(torch.Tensor.data_ptr, tensors)]):
            plan = self._plan(*key)
            objects = [*itertools.chain(*self.wq.values(), self.act.values(), self.act_f32.values(),
                                        self.m_vec.values(), self.taps.values())]
            tensors = [t for t in objects if t is not None]          # (a layer may have no bias)
            self._plans[key] = plan, given, objects, tensors, [t.data_ptr() for t in tensors]
        segments, x_slots, out_slots, n_parts = plan
        if x is not None:
            base = B._ptr(x, torch.float32)
            for s, i, off in x_slots:
                segments[s][i].x = base + off
        for s, i, name, off, length in out_slots:
            out = dequant[name]
            self._check_length(name, out, length)
            segments[s][i].y_f32 = B._ptr(out, torch.float32) + off
        run = B.lib.q8_run_ops
        streams = (ctypes.c_void_p * n_parts)(B._stream(),
                                              *(s.cuda_stream for s in self.side[:n_parts - 1]))
        if n_parts == 1:
            for ops in segments:
                if len(ops):
                    B._check(run(ops, len(ops), streams, 1))
            return
        pre, body, post = segments
        main = torch.cuda.current_stream()
        if len(pre):
            B._check(run(pre, len(pre), streams, 1))
        for side in self.side[:n_parts - 1]:
            side.wait_stream(main)
        B._check(run(body, len(body), streams, n_parts))
        for side in self.side[:n_parts - 1]:
            main.wait_stream(side)
        if len(post):
            B._check(run(post, len(post), streams, 1))

    @staticmethod
    def _check_length(name, out, length):
        if out.numel() < length:
            raise ValueError(f"run_step: the buffer of {name} is shorter than the tensor")

    def run_step(self, x=None, dequant=None, serial=False):
        """One pass over the batch: Eq. Q on ``x`` (if given), every layer, Eq. D on the
        tensors named in ``dequant`` ({name: fp32 output buffer, of the batch or longer}).  With two streams the
        layers of each half batch form a pipeline of their own between the (whole-batch)
        quantise and dequantise launches -- splitting those two as well was slower -- where
        the batch is large enough for that to pay; ``serial`` issues the launches of every
        part one pipeline after the other on the caller's stream."""
        if not serial and self._plannable(x, dequant or {}):
            self._run_planned(x, dequant or {})
            for name, out in (dequant or {}).items():
                if out is None:
                    self.dequantize(name)
            return
        for name, out in (dequant or {}).items():
            if out is not None:
                self._check_length(name, out, self.act[name][:self.N].numel())
        self._x = None
        if x is not None:
            self.set_input(x)
        # Eq. D inside the launch that writes the tensor, where there is such a launch
        self._deq = {name: out for name, out in (dequant or {}).items()
                     if out is not None and not self.chain and self._dequant_writer(name)}
        if self.chain:
            self.run_chained()
        elif self.n_streams == 1 or serial:
            for lo, n in self.parts:
                self.run_ops(self.net.ops, lo, n)
        else:
            main = torch.cuda.current_stream()
            for side in self.side:
                side.wait_stream(main)
            for op in self.net.ops:
                for side, part in zip(self.side, self.parts[1:]):
                    with torch.cuda.stream(side):
                        self.run_ops([op], *part)
                self.run_ops([op], *self.parts[0])
            for side in self.side:
                main.wait_stream(side)
        self._x = None
        done, self._deq = self._deq, {}
        for name, out in (dequant or {}).items():
            if name not in done:
                self.dequantize(name, out=out)

    def run_layers(self, acc_dump=None, serial=False):
        """Every layer on the codes already in the input buffer.  ``acc_dump``
        ({conv name: int32 buffer}): whole-batch launches that also store the accumulators."""
        if acc_dump:
            # every layer on its own in this pass (no fused pairs): a dumped layer needs its
            # input tensor written, whether or not the layer in front of it is dumped too
            for op in self.net.ops:
                if op.kind == "pool":
                    self.run_pool(op)
                else:
                    self.run_conv(op, acc_dump=acc_dump.get(op.name), fuse=False)
            return
        self.run_step(serial=serial)

    def dequantize(self, name, out=None, lo=0, n=None):
        """Eq. D on images [lo, lo + n) of tensor ``name`` (signed or unsigned codes); a
        real-valued output is already there."""
        n = self.N if n is None else n
        if out is not None:
            out = out[lo:lo + n]
        if name in self.real:
            if out is not None:
                out.copy_(self.act_f32[name][lo:lo + n])
                return out
            return self.act_f32[name][lo:lo + n]
        fn = B.dequantize_u8 if name in self.unsigned else B.dequantize
        return fn(self.act[name][lo:lo + n], self.q[name], out=out)

    def forward(self, x):
        """x: fp32 NHWC device tensor of the network input.  Returns the int8 outputs."""
        if not self.act:
            self.allocate()
        self.run_step(x)
        return [self.act[o] for o in self.net.outputs]

    def capture(self, x):
        """Record forward(x) into a HIP graph (x's storage is read at every replay)."""
        if not self.act:
            self.allocate()
        self.forward(x)                     # warm-up outside capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            self.forward(x)
        self.graph = g
        return g
