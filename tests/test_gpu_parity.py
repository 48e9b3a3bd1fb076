"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element.

int8 networks must match bit for bit (activations, logits, labels, scores, exit flags, compaction
order, and on the virtual clock the whole schedule).  bf16 networks: logits within 2e-2 of the
per-sample max-norm, confidences within 1e-3, exit decisions equal unless the oracle's confidence is
within 1e-3 of the threshold."""
import re
import sys
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    return torch


@pytest.fixture(scope="module")
def ee():
    import paper_2209_13443_amd as ee
    return ee


def dev(torch, a):
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t, like):
    a = t.cpu().numpy()
    return a.view(np.uint16) if like.dtype == np.uint16 else a


I8_NETS = ["tiny_i8", "zoo_i8", "resnet50_small_i8", "resnet18_small_i8", "mobilenetv2_small_i8", "inception_small_i8"]


@pytest.mark.parametrize("name", I8_NETS)
def test_int8_segments_and_heads_bit_exact(torch, ee, orc, name):
    blob = W.load_net(name)
    eng = ee.Engine(blob, 16)
    x = W.input_pool(blob, 13)
    for b in (1, 13, 6):                                   # ragged batches, smaller after larger
        act = x[:b]
        for s in range(blob.n_stages):
            say(f"[case] {name} segment {s} b={b}")
            ref = orc.stage_forward(blob, s, act)
            got = eng.stage_forward(s, dev(torch, act), ref.shape[1:])
            torch.cuda.synchronize()
            got = host(got, ref)
            assert np.array_equal(got, ref), f"{name} stage {s} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
            thr = float(blob.exits[s]["thr"])
            lab, conf, score, flag, logits = orc.exit_head(blob, s, ref, thr, want_logits=True)
            glab, gconf, gscore, gflag = eng.exit_head(s, dev(torch, ref), thr)
            glog = eng.last_logits(b, logits.shape[1])
            assert np.array_equal(glog, logits)
            assert np.array_equal(glab.cpu().numpy(), lab) and np.array_equal(gscore.cpu().numpy(), score)
            assert np.array_equal(gflag.cpu().numpy(), flag)
            assert np.allclose(gconf.cpu().numpy(), conf, rtol=1e-6, atol=0)
            act = ref
    eng.close()


SKINNY = [0x2211, 0x2212, 0x2213, 0x2214, 0x2314, 0x2221, 0x2222, 0x2223, 0x2224, 0x4213, 0x4214, 0x4314]


@pytest.mark.parametrize("cfg", SKINNY)
def test_few_pixel_convolution_bit_exact(torch, ee, orc, cfg):
    """The convolution kernel that splits the reduction over its wavefronts, forced on every matrix-core layer: reductions shorter than
    the wavefronts and of odd length, channel counts that fill no block, slices, residuals, strides, rectangular kernels, the folded first layer."""
    old = ee.tune_conv_tile(cfg)
    try:
        for blob in [W.load_net("zoo_i8"), W.load_net("resnet50_small_i8"), W.load_net("inception_small_i8"), W.random_net(3, W.DT_I8), W.random_net(11, W.DT_I8)]:
            eng = ee.Engine(blob, 4)
            for b in (3, 1):
                act = W.input_pool(blob, b)
                for s in range(blob.n_stages):
                    say(f"[case] cfg {cfg:#x} {len(blob.ops)} layers segment {s} b={b}")
                    ref = orc.stage_forward(blob, s, act)
                    got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
                    assert np.array_equal(got, ref), f"segment {s} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
                    act = ref
            eng.close()
    finally:
        ee.tune_conv_tile(old)


@pytest.mark.parametrize("k, stride, pad", [(1, 1, 0), (1, 2, 0), (3, 1, 1), (3, 2, 1), (5, 1, 2), (3, 1, 0)])
@pytest.mark.parametrize("c", [16, 32, 48, 64, 96, 192])
def test_few_pixel_convolution_forms_bit_exact(torch, ee, orc, c, k, stride, pad):
    """Its three forms: 1x1 without padding, taps of whole steps (32 bytes, or 64 in 16-pixel tiles), anything else; from one step to 75, so that a
    wavefront has none, one group, two, an odd and an even number of them; windows over every edge of an image of 5 x 6 pixels."""
    blob = W.single_layer_net("conv", 5, 6, c, k, stride, pad, W.DT_I8, seed=c + k, co=48)
    x = W.input_pool(blob, 2)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, 2)
    for cfg in SKINNY:
        old = ee.tune_conv_tile(cfg)
        try:
            say(f"[case] cfg {cfg:#x} {c} channels k{k} s{stride} p{pad}")
            for b in (2, 1):
                got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref[:b])
                assert np.array_equal(got, ref[:b]), f"cfg {cfg:#x} b={b}: {np.count_nonzero(got != ref[:b])} of {got.size} differ"
        finally:
            ee.tune_conv_tile(old)
    eng.close()


def test_few_pixel_convolution_past_4_gib_of_weights(torch, ee):
    """Every tile reads its own weights, those behind the first 4 GiB too: a 1x1 layer of 131,136 x 32,768 weights, of zeros but for sixteen rows, and a layer that passes their channels on."""
    from workloads import nets as N
    ci, co = 32768, 131136
    rows = np.array([0, 31, 32, 65535, 65536, 65599, 70001, 131071, 131072, 131073, 131088, 131103, 131104, 131119, 131120, 131135])
    net = N._Net(W.DT_I8, 1, 1, ci, 10)
    t = net.conv(net.begin_stage(), 128, 1, 1, 0, act="linear")
    net.end_stage(net.conv(t, 16, 1, 1, 0, act="linear"))
    small = N._assemble(net, net.dtype, 3)
    data = int(small.header[0]["data_off"])
    w1 = data
    b1 = w1 + ci * co
    w2 = b1 + 4 * co
    b2 = w2 + 16 * co
    fc = b2 + 64
    raw = np.zeros(fc + 1024, np.uint8)                      # pages of zeros are never touched on this side
    raw[:data] = small.raw[:data]
    raw[:128].view(W.HEADER_DT)["total_bytes"] = raw.size
    at = int(small.header[0]["ops_off"])
    ops = raw[at:at + 2 * W.OP_DT.itemsize].view(W.OP_DT)
    for op, cin, cout, w, b, shift in ((ops[0:1], ci, co, w1, b1, 8), (ops[1:2], co, 16, w2, b2, 0)):
        op["c_in"], op["c_out"], op["c_tot"], op["w_off"], op["b_off"], op["shift"] = cin, cout, cout, w, b, shift
    at = int(small.header[0]["exits_off"])
    exits = raw[at:at + W.EXIT_DT.itemsize].view(W.EXIT_DT)
    exits["w_off"], exits["b_off"] = fc, fc + 512
    rng = np.random.default_rng(8)
    weights = rng.integers(-2, 3, size=(16, ci), dtype=np.int8)
    for k, r in enumerate(rows):
        raw[w1 + int(r) * ci:w1 + (int(r) + 1) * ci] = weights[k].view(np.uint8)
        raw[w2 + k * co + int(r)] = 1
    x = rng.integers(-128, 128, size=(1, 1, 1, ci), dtype=np.int8)
    want = np.clip((weights.astype(np.int64) @ x.reshape(ci).astype(np.int64) + 128) >> 8, -128, 127)
    assert np.unique(want).size > 8
    eng = ee.Engine(raw, 1)
    for cfg in (0x2212, 0x2222, 0x4213):
        say(f"[case] weights past 4 GiB {cfg:#x}")
        got = forced(ee, cfg, lambda: eng.stage_forward(0, dev(torch, x), (1, 1, 16)).cpu().numpy())
        assert np.array_equal(got.reshape(16), want), (cfg, got.reshape(16), want)
    eng.close()


@pytest.mark.parametrize("seed", range(24))
def test_random_networks_bit_exact(torch, ee, orc, seed):
    """Generated networks (rectangular kernels, per-axis padding, strides, residuals, depthwise, pooling, concatenated
    slices at odd offsets, channel counts that are not multiples of 16): every segment and head against the oracle."""
    blob = W.random_net(seed, W.DT_I8)
    say(f"[case] random int8 network {seed}: {len(blob.ops)} layers")
    eng = ee.Engine(blob, 8)
    x = W.input_pool(blob, 7)
    for b in (7, 2):
        act = x[:b]
        for s in range(blob.n_stages):
            ref = orc.stage_forward(blob, s, act)
            got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"network {seed} segment {s} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
            lab, conf, score, flag = orc.exit_head(blob, s, ref, 0.5)
            glab, gconf, gscore, gflag = eng.exit_head(s, dev(torch, ref), 0.5)
            assert np.array_equal(glab.cpu().numpy(), lab) and np.array_equal(gscore.cpu().numpy(), score) and np.array_equal(gflag.cpu().numpy(), flag)
            act = ref
    assert 0 < np.count_nonzero(ref) < ref.size or blob.n_stages == 1
    eng.close()


EDGE_SHAPES = [(1, 1, 16), (2, 5, 16), (3, 3, 48), (7, 7, 32), (9, 13, 16), (4, 17, 144)]


@pytest.mark.parametrize("kind", ["maxpool", "avgpool", "dw"])
def test_int8_3x3_window_layers_edge_shapes_and_values(torch, ee, orc, kind):
    """The 3x3 pooling and depthwise kernels alone (a segment that is one layer), on shapes around their 4-pixel
    groups and borders, strides 1 and 2, paddings 0..2, with inputs of extreme values: all -128, all 127, a mix of
    -128 / 127 / 0 / -1 (negative half-way cases of the average's rounding) and uniform bytes."""
    r = np.random.default_rng(99)
    for h, w, c in EDGE_SHAPES:
        for stride in (1, 2):
            for pad in (0, 1, 2):
                if min(h, w) + 2 * pad < 3:
                    continue
                blob = W.single_layer_net(kind, h, w, c, 3, stride, pad, W.DT_I8, seed=h * 31 + w)
                say(f"[case] {kind} {h}x{w}x{c} stride {stride} pad {pad}")
                x = np.concatenate([np.full((1, h, w, c), -128, np.int8), np.full((1, h, w, c), 127, np.int8),
                                    r.choice(np.array([-128, 127, 0, -1], np.int8), size=(3, h, w, c)),
                                    r.integers(-128, 128, size=(2, h, w, c), dtype=np.int8)])
                eng = ee.Engine(blob, 8)
                for b in (7, 1):
                    ref = orc.stage_forward(blob, 0, x[:b])
                    got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
                    assert np.array_equal(got, ref), f"{kind} {h}x{w}x{c} s{stride} p{pad} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
                eng.close()


IR_CASES = [  # h, w, c_in, expanded, c_out (per block), stride, blocks, samples
    (9, 11, 16, 48, 16, 1, 2, 7), (8, 8, 24, 144, (24, 32), 1, 2, 7), (13, 8, 24, 144, 32, 2, 1, 7), (14, 14, 64, 208, 64, 1, 1, 5),
    (7, 7, 160, 320, 160, 1, 1, 3), (16, 16, 16, 96, (24, 16), 2, 2, 7), (5, 6, 8, 48, (40, 16), 1, 2, 7), (7, 7, 96, 160, 128, 1, 1, 3),
    (20, 18, 32, 64, 96, 1, 1, 3), (1, 1, 16, 32, 16, 1, 1, 2), (3, 2, 32, 96, (8, 16), 2, 2, 2), (28, 28, 32, 192, 32, 1, 1, 40),
    # without expansion (depthwise -> projection): one and several channel groups, both forms of the kernel
    (9, 11, 32, 0, 16, 1, 1, 7), (8, 8, 48, 0, (32, 16), 2, 2, 7), (14, 14, 144, 0, 64, 1, 1, 5), (7, 7, 208, 0, 96, 1, 1, 3), (12, 20, 16, 0, 16, 1, 2, 7),
    (28, 28, 32, 0, 16, 1, 1, 40),
]


@pytest.mark.parametrize("case", IR_CASES, ids=lambda c: "x".join(str(v) if isinstance(v, int) else "_".join(map(str, v)) for v in c))
def test_fused_inverted_residual_blocks_equal_separate_layers_and_oracle(torch, ee, orc, case):
    """Expansion -> depthwise -> projection (+ residual) as one launch: shapes around the kernel's pixel blocks (8, 14 and 7
    columns), channel groups (expanded channels that are and are not multiples of 32), output blocks (8 .. 160 channels, partial
    16-byte stores), strides, one- and two-block segments, extreme inputs; against the oracle and against the three
    separate layers, bit for bit."""
    h, w, ci, ce, co, stride, blocks, n = case
    blob = W.inverted_residual_net(h, w, ci, ce, co, stride, seed=h * 7 + ce, blocks=blocks)
    say(f"[case] inverted residual {h}x{w} {ci} -> {ce if ce else 'no expansion'} -> {co} stride {stride}, {blocks} block(s), {n} samples")
    r = np.random.default_rng(h * 100 + ce)
    x = np.concatenate([np.full((1, h, w, ci), -128, np.int8), np.full((1, h, w, ci), 127, np.int8),
                        r.integers(-128, 128, size=(max(n - 2, 1), h, w, ci), dtype=np.int8)])[:n]
    eng = ee.Engine(blob, max(n, 2))
    assert eng.ir_count() == blocks
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        for mode in (2, 0, 2):
            eng.ir_mode(mode)
            got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"mode {mode} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
    assert np.unique(ref).size > 8
    eng.close()


IR_SHARED_CASES = [  # h, w, c_in, expanded, c_out, stride, (samples, wavefronts that share the channel groups or 0: the pixels) at the edges of the rule
    (14, 14, 96, 576, 160, 2, [(1, 8), (5, 8)]), (28, 28, 32, 192, 32, 1, [(9, 8), (10, 8), (54, 8), (55, 0)]), (28, 28, 32, 192, 64, 2, [(36, 8), (37, 0)]),
    (14, 14, 64, 384, 64, 1, [(36, 8), (37, 8), (128, 8), (129, 0)]), (13, 14, 24, 160, 32, 2, [(3, 8)]), (13, 11, 32, 192, 32, 1, [(1, 8)]), (5, 6, 64, 128, 48, 1, [(2, 4)]),
    (15, 17, 64, 256, 144, 2, [(2, 4)]), (9, 9, 32, 128, 16, 1, [(2, 0)]), (28, 28, 32, 192, 64, 1, [(18, 8), (19, 0)]), (28, 28, 32, 192, 160, 2, [(36, 8), (37, 0)]),
    (14, 14, 64, 384, 160, 1, [(109, 8), (110, 0)]), (14, 14, 160, 0, 160, 1, [(109, 4), (110, 0)]),
]


@pytest.mark.parametrize("case", IR_SHARED_CASES, ids=lambda c: "x".join(map(str, c[:6])))
def test_wavefronts_that_share_the_channel_groups(torch, ee, orc, case):
    """Which form of the fused block a number of tiles gets, the forms' results on both sides of every edge against the separate layers, and the first and last samples against the oracle."""
    h, w, ci, ce, co, stride, edges = case
    blob = W.inverted_residual_net(h, w, ci, ce, co, stride, seed=h + co)
    n = max(b for b, _ in edges)
    x = np.random.default_rng(ce).integers(-128, 128, size=(n, h, w, ci), dtype=np.int8)
    eng = ee.Engine(blob, n)
    xd = dev(torch, x)
    for b, form in edges:
        say(f"[case] shared channel groups {case[:6]} {b} samples")
        eng.ir_mode(2)
        out, names = kernels_of(torch, lambda: eng.stage_forward(0, xd[:b], blob.stage_out_shape(0)))
        assert len(names) == 1 and names[0].startswith("ir_block_i8_kernel<") and names[0].split(",")[4].strip() == str(form), names
        eng.ir_mode(0)
        assert torch.equal(out, eng.stage_forward(0, xd[:b], blob.stage_out_shape(0))), b
        ends = sorted({0, b - 1})
        ref = orc.stage_forward(blob, 0, x[ends])
        assert np.array_equal(host(out[ends], ref), ref) and np.unique(ref).size > 8
    eng.close()


@pytest.mark.parametrize("case", [(9, 11, 16, 48), (28, 28, 32, 192), (14, 14, 96, 576), (7, 7, 160, 320), (12, 20, 16, 0), (1, 1, 16, 32)], ids=lambda c: "x".join(map(str, c)))
def test_inverted_residual_block_pools_for_the_exit_head(torch, ee, orc, case):
    """A segment that ends in a fused block with a residual, served: the block's launch carries the exit head's pooling (both forms of the kernel,
    tiles with dead pixels, several tiles per image).  Label and confidence of every request are those of the separate layers, and the oracle's."""
    h, w, ci, ce = case
    blob = W.inverted_residual_net(h, w, ci, ce, ci, 1, seed=h + ce, blocks=1)
    n, b_max = 24, 8
    x = np.random.default_rng(h).integers(-128, 128, size=(n, h, w, ci), dtype=np.int8)
    eng = ee.Engine(blob, b_max)
    assert eng.ir_count() == 1
    lut = synthetic_lut(blob.n_stages, b_max)
    want = None
    for mode in (0, 2, 2):
        say(f"[case] pooling block {case} mode {mode}")
        eng.ir_mode(mode)
        got = eng.serve_stream(np.zeros(n, np.int64), dev(torch, x), lut, refill=0)[0]
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf"):
            assert np.array_equal(got[f], want[f]), (f, mode)
    label, conf = orc.exit_head(blob, 0, orc.stage_forward(blob, 0, x), 0.5)[:2]
    assert np.array_equal(want["label"], label) and np.array_equal(want["conf"], conf) and np.unique(conf).size > 8
    eng.close()


BN_CASES = [  # h, w, c_in, blocks, samples
    (8, 8, 64, 1, 3), (9, 11, 64, 2, 7), (5, 17, 256, 1, 7), (16, 8, 256, 2, 5), (1, 1, 64, 1, 2), (28, 28, 256, 1, 40), (56, 56, 64, 2, 6), (28, 28, 64, 2, 9),
]


@pytest.mark.parametrize("case", BN_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_bottleneck_blocks_equal_separate_layers_and_oracle(torch, ee, orc, case):
    """1x1 -> 3x3 -> 1x1 + residual as one launch (64 middle channels, 256 out): images that are and are not whole tiles of
    8 x 8 pixels, a single pixel, 64 and 256 input channels (a convolution or the block's input as residual), more tiles than
    workgroups (a workgroup walks over several), extreme inputs; against the oracle and against the three separate layers,
    bit for bit."""
    h, w, ci, blocks, n = case
    blob = W.bottleneck_net(h, w, ci, seed=h * 7 + w, blocks=blocks)
    say(f"[case] bottleneck {h}x{w} {ci} -> 64 -> 64 -> 256, {blocks} block(s), {n} samples")
    r = np.random.default_rng(h * 100 + w)
    x = np.concatenate([np.full((1, h, w, ci), -128, np.int8), np.full((1, h, w, ci), 127, np.int8),
                        r.integers(-128, 128, size=(max(n - 2, 1), h, w, ci), dtype=np.int8)])[:n]
    eng = ee.Engine(blob, max(n, 2))
    heads = {i: eng.ir_layers(i) for i in range(len(blob.ops)) if eng.ir_layers(i)}
    # with 64 input channels the first block's residual is a convolution of the input: that layer heads a block of four
    assert sorted(heads.values()) == ([3] * blocks + [4] if ci == 64 else [3] * blocks) and eng.ir_count() == len(heads)
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        for mode in (2, 0, 1, 2):
            eng.ir_mode(mode)
            if mode == 1:                                                  # by table: the blocks of three fused, the block of four not
                eng.load_tables({"ir": {str(i): [0 if span == 4 else 1] for i, span in heads.items()}})
            got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"mode {mode} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
    assert np.unique(ref).size > 8
    if (h, w) == (28, 28):                                                 # the table ee_autotune writes: an entry per head, results unchanged
        eng.autotune(reps=2)
        tabs = eng.tables()["ir"]
        assert sorted(map(int, tabs)) == sorted(heads) and all(set(v) <= {0, 1} for v in tabs.values())
        eng.ir_mode(1)
        ref = orc.stage_forward(blob, 0, x)
        got = host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref)
        assert np.array_equal(got, ref)
    eng.close()


def test_fused_inverted_residual_blocks_in_a_network(torch, ee, orc):
    """The MobileNetV2-style network with every block fused, with none fused and with the table ee_autotune writes: every
    segment and head against the oracle."""
    blob = W.load_net("mobilenetv2_small_i8")
    eng = ee.Engine(blob, 8)
    assert eng.ir_count() == 16                                            # every block but the last (320 output channels)
    x = W.input_pool(blob, 7)
    for step, mode in enumerate((2, 0, 1)):
        if step == 2:
            eng.autotune(reps=2)
            tabs = eng.tables()["ir"]
            assert len(tabs) == 16 and all(set(v) <= {0, 1} for v in tabs.values())
            eng.load_tables({"ir": tabs})
        eng.ir_mode(mode)
        act = x
        for s in range(blob.n_stages):
            ref = orc.stage_forward(blob, s, act)
            got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"mode {mode} segment {s}: {np.count_nonzero(got != ref)} of {ref.size} differ"
            act = ref
    eng.close()


def test_int8_thin_1x1_layers_bit_exact(torch, ee, orc):
    """1x1 layers with 4..32 input channels (the kernel that feeds one matrix instruction per 32 x 32 outputs straight
    from global memory): every channel count, output widths that are and are not multiples of 32, pixel counts that
    end inside a strip of 32, extreme inputs, relu and linear clamps."""
    r = np.random.default_rng(7)
    for ci in (4, 8, 12, 16, 20, 24, 28, 32):
        for co, act in ((16, "linear"), (48, "relu"), (144, "relu6"), (160, "linear")):
            h, w = (4, 4) if (ci + co) % 3 else (3, 16)
            blob = W.single_layer_net("conv", h, w, ci, 1, 1, 0, W.DT_I8, seed=ci * 7 + co, co=co, act=act)
            say(f"[case] 1x1 conv {ci} -> {co} ({act}) on {h}x{w}")
            x = np.concatenate([np.full((1, h, w, ci), -128, np.int8), np.full((1, h, w, ci), 127, np.int8),
                                r.integers(-128, 128, size=(5, h, w, ci), dtype=np.int8)])
            eng = ee.Engine(blob, 8)
            for b in (7, 3, 1):
                ref = orc.stage_forward(blob, 0, x[:b])
                got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
                assert np.array_equal(got, ref), f"1x1 {ci}->{co} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
            assert 0 < np.count_nonzero(ref != ref.flat[0])
            eng.close()


STREAM_CASES = [  # (h, w, c, co, k, stride, pad): layers the streaming kernel covers, on shapes around its 32-pixel strips
    (9, 9, 32, 32, 3, 1, 1), (7, 11, 32, 64, 3, 1, 0), (12, 8, 32, 48, 3, 2, 1), (5, 5, 32, 16, 3, 2, 0), (6, 10, 32, 64, 3, 1, 2),
    (16, 16, 3, 64, 7, 2, 3), (12, 20, 3, 32, 3, 2, 1), (16, 15, 3, 32, 3, 2, 0), (8, 8, 4, 48, 7, 2, 3), (10, 6, 32, 32, (1, 3), 1, (0, 1)),
    (10, 6, 32, 64, (3, 1), 1, (1, 0)),
]


@pytest.mark.parametrize("case", STREAM_CASES)
def test_int8_streaming_kernel_bit_exact(torch, ee, orc, case):
    """The streaming convolution kernel forced on single-layer segments it covers (folded stride-2 first layers, 3 x 3 /
    1 x 3 / 3 x 1 layers over 32 channels), extreme inputs included; and the same segments with the default choice."""
    h, w, c, co, k, stride, pad = case
    r = np.random.default_rng(11)
    if (h * w * c) % 16:
        pytest.skip("a sample must be whole 16-byte chunks")
    blob = W.single_layer_net("conv", h, w, c, k, stride, pad, W.DT_I8, seed=h * 13 + co, co=co, act="relu" if co % 32 else "linear")
    x = np.concatenate([np.full((1, h, w, c), -128, np.int8), np.full((1, h, w, c), 127, np.int8), r.integers(-128, 128, size=(6, h, w, c), dtype=np.int8)])
    for tile in (7, 0):
        old = ee.tune_conv_tile(tile)
        try:
            eng = ee.Engine(blob, 8)
            for b in (8, 5, 1):
                ref = orc.stage_forward(blob, 0, x[:b])
                got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
                assert np.array_equal(got, ref), f"{case} tile {tile} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
            eng.close()
        finally:
            ee.tune_conv_tile(old)
    assert 0 < np.count_nonzero(ref != ref.flat[0])


@pytest.mark.parametrize("seed", range(8))
def test_random_networks_bf16_within_tolerance(torch, ee, orc, seed):
    blob = W.random_net(seed, W.DT_BF16)
    say(f"[case] random bf16 network {seed}: {len(blob.ops)} layers")
    eng = ee.Engine(blob, 8)
    act = W.input_pool(blob, 5)
    for s in range(blob.n_stages):
        ref = orc.stage_forward(blob, s, act)
        got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
        r, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(got).astype(np.float64)
        scale = np.abs(r).reshape(r.shape[0], -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30
        assert np.all(np.abs(g - r) <= 2e-2 * scale), f"network {seed} segment {s}: {np.max(np.abs(g - r) / scale)}"
        act = ref
    eng.close()


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("name", ["zoo_i8", "resnet50_small_i8"])
def test_int8_every_conv_tiling_bit_exact(torch, ee, orc, name, tile):
    blob = W.load_net(name)
    eng = ee.Engine(blob, 8)
    x = W.input_pool(blob, 5)
    old = ee.tune_conv_tile(tile)
    try:
        act = x
        for s in range(blob.n_stages):
            say(f"[case] {name} tile {tile} segment {s}")
            ref = orc.stage_forward(blob, s, act)
            got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"tile {tile} stage {s}"
            act = ref
    finally:
        ee.tune_conv_tile(old)
    eng.close()


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [0x0321, 0x0421, 0x0231, 0x0331, 0x0322, 0x0432, 0x0323, 0x0433, 0x0324, 0x0234,
                                 0x10321, 0x10431, 0x10222, 0x10332, 0x10323, 0x10233, 0x10324, 0x10434])
def test_int8_pipelined_steps_bit_exact(torch, ee, orc, cfg):
    """Reduction steps of 128 and 256 bytes run the pipelined form of the inner loop (fragments read two sub-steps ahead,
    barrier before the end of a step): every tiling of it with rings of 2, 3 and 4 stages, on layers with one, two and
    many steps and a ragged last tile, against the oracle.  Words with bit 16 name the slab kernel (stride-1 layers whose
    output is as large as the input; the other layers keep their default kernel): its four tiles, both weight steps."""
    for name in ("zoo_i8", "resnet50_small_i8") if cfg < 0x10000 else ("resnet50_small_i8", "resnet18_small_i8", "inception_small_i8"):
        blob = W.load_net(name)
        eng = ee.Engine(blob, 8)
        x = W.input_pool(blob, 5)
        old = ee.tune_conv_tile(cfg)
        try:
            act = x
            for s in range(blob.n_stages):
                say(f"[case] {name} cfg {cfg:#x} segment {s}")
                ref = orc.stage_forward(blob, s, act)
                got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
                assert np.array_equal(got, ref), f"cfg {cfg:#x} stage {s}"
                act = ref
        finally:
            ee.tune_conv_tile(old)
        eng.close()


def test_autotuned_configuration_table_keeps_results(torch, ee, orc):
    """The per-(layer, batch bucket) kernel configuration table only changes speed, never a byte."""
    for name in ("resnet50_small_i8", "zoo_i8"):
        blob = W.load_net(name)
        eng = ee.Engine(blob, 12)
        eng.autotune(reps=2)
        tables = [eng.config_table(k) for k in range(len(blob.ops))]
        assert any(len(t) > 0 for t in tables)
        for t in tables:
            for cfg in t:
                assert cfg == 7 or (1 <= (cfg & 15) <= 4 and 1 <= ((cfg >> 4) & 15) <= 3 and 2 <= ((cfg >> 8) & 15) <= 4 and (cfg >> 12) in (0, 2, 4))
        x = W.input_pool(blob, 11)
        for b in (11, 3, 1):
            act = x[:b]
            for s in range(blob.n_stages):
                say(f"[case] autotuned {name} segment {s} b={b}")
                ref = orc.stage_forward(blob, s, act)
                got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
                assert np.array_equal(got, ref)
                act = ref
        # the table is plain data: a second engine loads it and runs the same configurations
        stored = eng.tables()
        other = ee.Engine(blob, 12)
        other.load_tables(stored)
        assert other.tables() == stored
        ref = orc.stage_forward(blob, 0, x)
        assert np.array_equal(host(other.stage_forward(0, dev(torch, x), ref.shape[1:]), ref), ref)
        with pytest.raises(ee.EEError):
            other.load_tables({"config": {"0": [0x99]}})                    # tile 9 does not exist
        # the streaming kernel as a stored entry: accepted for the folded first layer it covers (results unchanged),
        # refused for a layer it does not cover (one with a residual)
        if name == "resnet50_small_i8":
            other.load_tables({"config": {"0": [7] * len(stored["config"]["0"])}})
            assert np.array_equal(host(other.stage_forward(0, dev(torch, x), ref.shape[1:]), ref), ref)
            with_res = next(k for k, op in enumerate(blob.ops) if int(op["res"]) >= 0 and str(k) in stored["config"])
            with pytest.raises(ee.EEError):
                other.load_tables({"config": {str(with_res): [7]}})
        other.close()
        eng.close()


HEAD_SHAPES = [(1, 1, 16, 1), (3, 5, 48, 17), (8, 8, 16, 256), (16, 16, 128, 100), (2, 2, 2048, 16), (16, 17, 128, 100), (4, 4, 128, 257)]   # the last two: past the limits


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("h, w, c, n_cls", HEAD_SHAPES)
def test_small_exit_heads(torch, ee, orc, h, w, c, n_cls, dtype):
    """Heads around the limits of the one-launch kernel: fewer classes than a group of lanes and 256 of them, one pixel, the most channels."""
    from workloads import nets as N
    net = N._Net(W.DT_I8 if dtype == "i8" else W.DT_BF16, h, w, c, n_cls)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 7)
    eng = ee.Engine(blob, 5)
    act = W.input_pool(blob, 5)
    for b in (5, 1):
        lab, conf, score, flag, logits = orc.exit_head(blob, 0, act[:b], 0.5, want_logits=True)
        glab, gconf, gscore, gflag = eng.exit_head(0, dev(torch, act[:b]), 0.5)
        glog = eng.last_logits(b, n_cls)
        if dtype == "i8":
            assert np.array_equal(glog, logits) and np.array_equal(glab.cpu().numpy(), lab) and np.array_equal(gscore.cpu().numpy(), score)
            assert np.array_equal(gflag.cpu().numpy(), flag) and np.allclose(gconf.cpu().numpy(), conf, rtol=1e-6, atol=0)
        else:
            assert np.all(np.abs(glog - logits) <= 1e-3 * np.abs(logits).max() + 1e-6) and np.all(np.abs(gconf.cpu().numpy() - conf) <= 1e-3)
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("c, n_cls", [(48, 1000), (528, 999), (2048, 257)])
def test_class_tiles_per_workgroup_of_the_fc(torch, ee, orc, c, n_cls, dtype):
    """The FC with one, two and four tiles of classes per workgroup (as many as leave a workgroup per CU), batches on both sides of each, class counts and reductions that end inside a tile and inside a
    step: logits and decisions against the oracle."""
    from workloads import nets as N
    net = N._Net(W.DT_I8 if dtype == "i8" else W.DT_BF16, 2, 1, c, n_cls)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 11)
    tiles = -(-n_cls // 16)
    edges = {1: 1, 16 * (256 // tiles): 1, 16 * (256 // tiles) + 1: 2, 16 * (256 // (-(-tiles // 2))): 2, 16 * (256 // (-(-tiles // 2))) + 1: 4}
    n = max(edges)
    eng = ee.Engine(blob, n)
    act = W.input_pool(blob, n)
    for b, tc in edges.items():
        say(f"[case] fc tiles {dtype} {c} {n_cls} b={b}")
        (glab, gconf, gscore, gflag), names = kernels_of(torch, lambda: eng.exit_head(0, dev(torch, act[:b]), 0.5))
        assert [x for x in names if x.startswith("fc_kernel")] == [f"fc_kernel<{1 if dtype == 'i8' else 2},{8 if c * (1 if dtype == 'i8' else 2) > 1024 else 4},{tc}>"], names
        glog = eng.last_logits(b, n_cls)
        ends = sorted({0, b // 2, b - 1})
        lab, conf, score, flag, logits = orc.exit_head(blob, 0, act[ends], 0.5, want_logits=True)
        if dtype == "i8":
            assert np.array_equal(glog[ends], logits) and np.array_equal(glab.cpu().numpy()[ends], lab) and np.array_equal(gscore.cpu().numpy()[ends], score)
        else:                                               # as in the test above
            assert np.all(np.abs(glog[ends] - logits) <= 1e-3 * np.abs(logits).max() + 1e-6) and np.all(np.abs(gconf.cpu().numpy()[ends] - conf) <= 1e-3)
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("c, n_cls, per", [(512, 256, 1), (512, 257, 4), (48, 1024, 4), (48, 1025, 8), (16, 2048, 8)])
def test_logits_per_lane_of_the_softmax(torch, ee, orc, c, n_cls, per, dtype):
    """The softmax with one, four and eight logits per lane, class counts on both sides of each: decisions against the oracle.  Two classes share the largest logit (the lower is the label).  bf16: the float
    denominator of up to 2048 terms in (0, 1] is within 2048 * 2^-23 of the exact one, relatively, and the logits within 1e-3 of their largest, as above."""
    from workloads import nets as N
    net = N._Net(W.DT_I8 if dtype == "i8" else W.DT_BF16, 2, 1, c, n_cls)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 23)
    act = W.input_pool(blob, 3)
    wfc, bias = blob.exit_weights(0)[:2]
    first, last = n_cls // 3, n_cls - 1
    top = int(orc.exit_head(blob, 0, act[:1], 0.5, want_logits=True)[4][0].argmax())
    wfc = wfc.reshape(n_cls, c)
    for j in (first, last):
        wfc[j], bias[j] = wfc[top], bias[top]
    eng = ee.Engine(blob, 3)
    lab, conf, score, flag, logits = orc.exit_head(blob, 0, act, 0.5, want_logits=True)
    assert logits[0, first] == logits[0, last] == logits[0].max()
    (glab, gconf, gscore, gflag), names = kernels_of(torch, lambda: eng.exit_head(0, dev(torch, act), 0.5))
    assert [x for x in names if x.startswith("softmax_kernel")] == [f"softmax_kernel<{1 if dtype == 'i8' else 2},{per}>"], names
    if dtype == "i8":
        assert np.array_equal(glab.cpu().numpy(), lab) and np.array_equal(gscore.cpu().numpy(), score) and np.array_equal(gflag.cpu().numpy(), flag)
        assert np.allclose(gconf.cpu().numpy(), conf, rtol=1e-6, atol=0)
    else:
        assert int(glab[0]) == int(lab[0]) and np.all(np.abs(gconf.cpu().numpy() - conf) <= 1e-3)
    eng.close()


def test_infinite_weights_of_the_fc(torch, ee, orc):
    """bf16: an infinite weight in the last step of a reduction that is shorter than what the wavefronts have in flight makes its class's logit infinite and no other, with every number of class tiles per
    workgroup: logits and labels are the oracle's."""
    from workloads import nets as N
    net = N._Net(W.DT_BF16, 2, 1, 64, 300)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 19)
    blob.exit_weights(0)[0].reshape(300, 64)[7, 40] = 0x7f80
    edges = {1: 1, 16 * 13 + 1: 2, 16 * 25 + 1: 4}
    eng = ee.Engine(blob, max(edges))
    act = np.empty((max(edges), 2, 1, 64), np.uint16)
    act[:, 0], act[:, 1] = 0x3f80, 0x3f81                    # means of 1 + 2^-8: 1 and a remainder above zero
    _, _, _, _, logits = orc.exit_head(blob, 0, act[:1], 0.5, want_logits=True)
    finite = np.isfinite(logits[0])
    assert logits[0, 7] == np.inf and finite.sum() == 299
    for b, tc in edges.items():
        (lab, _, _, _), names = kernels_of(torch, lambda: eng.exit_head(0, dev(torch, act[:b]), 0.5))
        assert f"fc_kernel<2,4,{tc}>" in names, names
        got = eng.last_logits(b, 300)
        assert np.all(got[:, 7] == np.inf) and np.all(np.abs(got[:, finite] - logits[:, finite]) <= 1e-3 * np.abs(logits[0, finite]).max()) and bool((lab == 7).all())
    eng.close()


@pytest.mark.parametrize("h, w, c, edges", [(7, 7, 2048, {1: 64, 9: 64}), (5, 13, 1032, {3: 64}), (14, 14, 1024, {2: 32}), (28, 28, 504, {1: 8, 33: 16}), (56, 56, 256, {2: 4, 33: 8, 65: 16}),
                                            (64, 64, 24, {3: 4}), (64, 65, 24, {3: None})], ids=str)
def test_bf16_pooling_by_slices_of_channels(torch, ee, orc, h, w, c, edges):
    """The bf16 head's pooling, one workgroup per sample and slice of channels, in every width, slices that end behind the last channel, and the images past its limit: logits against the oracle (double
    sums), which the pooled means reach within float rounding."""
    from workloads import nets as N
    net = N._Net(W.DT_BF16, h, w, c, 300)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 13)
    eng = ee.Engine(blob, max(edges))
    act = W.input_pool(blob, max(edges))
    for b, sch in edges.items():
        say(f"[case] pooling by slices {h}x{w}x{c} b={b}")
        (glab, gconf, _, _), names = kernels_of(torch, lambda: eng.exit_head(0, dev(torch, act[:b]), 0.5))
        assert names[0] == (f"gap_slice_kernel<2,{sch}>" if sch else "gap_kernel<2>"), names
        glog = eng.last_logits(b, 300)
        ends = sorted({0, b // 2, b - 1})
        _, conf, _, _, logits = orc.exit_head(blob, 0, act[ends], 0.5, want_logits=True)
        assert np.all(np.abs(glog[ends] - logits) <= 1e-3 * np.abs(logits).max() + 1e-6) and np.all(np.abs(gconf.cpu().numpy()[ends] - conf) <= 1e-3)      # as above
    eng.close()


@pytest.mark.parametrize("h, w, c, sliced", [(7, 7, 2048, 64), (1, 1, 1024, 64), (16, 16, 1040, 32), (16, 16, 1008, 0), (16, 17, 1024, 0)])
def test_int8_pooling_by_slices_of_channels(torch, ee, orc, h, w, c, sliced):
    """The int8 head's pooling by slices at the edges of its rule, slices that end behind the last channel, and heads one after the other on the same sums: everything against the oracle."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, h, w, c, 300)
    net.begin_stage()
    net.end_stage(net.maxpool(0, 3, 1, 1))
    blob = N._assemble(net, net.dtype, 17)
    eng = ee.Engine(blob, 9)
    act = W.input_pool(blob, 9)
    for b in (9, 1, 5):
        lab, _, score, flag, logits = orc.exit_head(blob, 0, act[:b], 0.5, want_logits=True)
        (glab, _, gscore, gflag), names = kernels_of(torch, lambda: eng.exit_head(0, dev(torch, act[:b]), 0.5))
        assert names[0] == (f"gap_slice_kernel<1,{sliced}>" if sliced else "gap_kernel<1>"), names
        assert np.array_equal(eng.last_logits(b, 300), logits) and np.array_equal(glab.cpu().numpy(), lab) and np.array_equal(gscore.cpu().numpy(), score) and np.array_equal(gflag.cpu().numpy(), flag)
    eng.close()


def launches_of(eng, f):
    eng.profile(True)
    eng.profile_read()
    f()
    n = sum(c["launches"] for c in eng.profile_read().values())
    eng.profile(False)
    return n


def kernels_of(torch, f):
    """What f returns, and the kernels that it launches, by name with their template arguments, spaces left out."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        out = f()
        torch.cuda.synchronize()
    return out, [m.group(1).replace(" ", "") for m in (re.search(r"\bee::(\w+_kernel(?:<[^>]*>)?)", e.name) for e in p.events()) if m]


def forced(ee, cfg, f):
    """What f returns with cfg forced for the whole process (a layer that the named kernel does not cover takes another one)."""
    old = ee.tune_conv_tile(cfg)
    try:
        return f()
    finally:
        ee.tune_conv_tile(old)


def scattering_order(exits, n_stages, b_max, n):
    """n requests out of a few that leave at the given exits: of every full batch of every level the last one goes on and the others leave.  Sample slots are
    taken in runs from the lowest one up, so what the first few batches leave behind breaks up every run of b_max of them: later full batches write through a slot table."""
    at = [np.flatnonzero(exits == e) for e in range(n_stages)]
    k = np.arange(n)
    want = sum((k % b_max ** l == b_max ** l - 1).astype(int) for l in range(1, n_stages))
    return np.array([at[e][i % len(at[e])] for i, e in zip(k, want)])


def steps_with_tables(events, exit_idx, n_stages, n_slots, by_value=0):
    """A one-lane stage-pool stream served zero-copy, from its events and the exits taken (first fit over a level's slots, inputs free when a step ends): per level the steps
    whose output slots were no run, and all steps of more than by_value samples with a table for either side."""
    waiting = [[(k, 0) for k in range(len(exit_idx))]] + [[] for _ in range(n_stages - 1)]
    taken = [np.zeros(n_slots, bool) for _ in range(n_stages)]
    outputs, either = [0] * (n_stages - 1), 0
    for ev in events:
        if ev["kind"] != 2:                                                # a step
            continue
        s, b = int(ev["stage"]), int(ev["b"])
        batch, waiting[s] = waiting[s][:b], waiting[s][b:]
        gather = s > 0 and [slot for _, slot in batch] != list(range(batch[0][1], batch[0][1] + b))
        scatter = False
        if s + 1 < n_stages:
            runs = [i for i in range(n_slots - b + 1) if not taken[s + 1][i:i + b].any()]
            slots = list(range(runs[0], runs[0] + b)) if runs else np.flatnonzero(~taken[s + 1])[:b].tolist()
            scatter = not runs
            outputs[s] += scatter
            kept = [(k, slot) for (k, _), slot in zip(batch, slots) if exit_idx[k] > s]
            waiting[s + 1] += kept
            taken[s + 1][[slot for _, slot in kept]] = True
        either += b > by_value and (gather or scatter)
        if s > 0:
            taken[s][[slot for _, slot in batch]] = False
    return outputs, either


def scattered_stream(torch, eng, pool, n, b_max):
    """n requests out of the pool in scattering_order: a function that serves them and returns results and kernels; zero-copy on one lane it checks that full batches of the
    first level, and of the deeper ones that see enough of them, wrote through slot tables."""
    n_stages = eng.n_stages
    lut = synthetic_lut(n_stages, b_max)
    exits = eng.serve_stream(np.zeros(len(pool), np.int64), dev(torch, pool), lut, refill=0, b_max=b_max)[0]["exit_idx"]
    assert all(np.count_nonzero(exits == e) for e in range(n_stages)), np.bincount(exits)
    dpool = dev(torch, pool[scattering_order(exits, n_stages, b_max, n)])

    def serve(zero_copy, lanes=1):
        (got, _, events), names = kernels_of(torch, lambda: eng.serve_stream(np.zeros(n, np.int64), dpool, lut, b_max=b_max, refill=2, lanes=lanes, zero_copy=zero_copy, max_events=5000))
        if zero_copy and lanes == 1:
            by_value = 64 if names.count("segment_small_i8_kernel") == len(events) else 0        # rows in the arguments of a small segment's launch
            outputs, either = steps_with_tables(events, got["exit_idx"], n_stages, 5 * eng.b_max, by_value)
            levels = sum(n >= 8 * b_max ** l for l in range(1, n_stages))
            assert levels >= 1 and all(outputs[:levels]), outputs
            assert names.count("upload_slots_kernel") == either            # one launch uploads a step's tables
        return got, names
    return serve


SMALL_SEGMENTS = {  # networks whose every segment runs with its exit head as one launch: the folded first layer; residuals of the segment's input and of a
    # convolution of it, 1x1 and 3x3, one pixel, channels that fill no block of 32, images that are no whole blocks of 32 pixels
    "tiny": lambda: W.load_net("tiny_i8"), "bneck_5x7": lambda: W.bottleneck_net(5, 7, 64, mid=16, stages=3, seed=1), "bneck_1x1": lambda: W.bottleneck_net(1, 1, 64, mid=32, stages=2, seed=2),
    "bneck_9x9": lambda: W.bottleneck_net(9, 9, 64, mid=32, stages=2, seed=3),
}


@pytest.mark.parametrize("name", sorted(SMALL_SEGMENTS))
def test_small_segments_in_one_launch(torch, ee, orc, name):
    """A segment and its exit head as one launch against the oracle, bit for bit: the segment alone (1, some and more than 64 samples), and served under
    the three policies, with and without zero-copy compaction, with the rows by value (up to 64 samples) and out of tables (more)."""
    blob = SMALL_SEGMENTS[name]()
    n, b_max = 260, 100
    x = W.input_pool(blob, n)
    act = x[:24]
    for s in range(blob.n_stages - 1):                                     # thresholds that split the requests
        act = orc.stage_forward(blob, s, act)
        blob.exits[s]["frac_bits"] = 12 if name != "tiny" else blob.exits[s]["frac_bits"]
        blob.exits[s]["thr"] = float(np.median(orc.exit_head(blob, s, act, 0.5)[1]))
    eng = ee.Engine(blob, b_max)
    for b in (100, 1, 13):
        act = x[:b]
        for s in range(blob.n_stages):
            say(f"[case] {name} segment {s} b={b}")
            ref = orc.stage_forward(blob, s, act)
            got = []
            assert launches_of(eng, lambda: got.append(eng.stage_forward(s, dev(torch, act), ref.shape[1:]))) == 1
            assert np.array_equal(host(got[0], ref), ref), f"{np.count_nonzero(host(got[0], ref) != ref)} of {ref.size} differ"
            act = ref
    assert eng.set_lanes(2) == 2
    dpool = dev(torch, x)
    lut = synthetic_lut(blob.n_stages, b_max)
    arrivals = np.zeros(n, np.int64)
    for refill, lanes, bm in ((0, 1, 100), (1, 1, 100), (2, 2, 100), (2, 1, 8), (1, 1, 64)):
        say(f"[case] {name} served refill={refill} lanes={lanes} b_max={bm}")
        ref, rst, rev = orc.serve_stream(blob, arrivals, x, bm, lut[:, :bm], refill=refill, lanes=lanes, max_events=5000, min_incr=max(1, bm // 2))
        for zc in (0, 1) if eng.zero_copy_supported() else (0,):
            got, gst, gev = eng.serve_stream(arrivals, dpool, lut[:, :bm], b_max=bm, clock=1, refill=refill, lanes=lanes, max_events=5000, min_incr=max(1, bm // 2), zero_copy=zc)
            for f in ("exit_idx", "label", "score", "latency_ns"):
                assert np.array_equal(got[f], ref[f]), (f, refill, lanes, bm, zc)
            assert gst == rst and np.array_equal(gev, rev)
    assert np.count_nonzero(np.bincount(ref["exit_idx"])) > 1
    if eng.zero_copy_supported():
        for bm in (72, 64):                                                # output rows that are no run: out of the device's table, by value
            say(f"[case] {name} scattered slots b_max={bm}")
            serve = scattered_stream(torch, eng, x, 12 * bm, bm)
            want, got = serve(0)[0], serve(1)[0]
            assert all(np.array_equal(got[f], want[f]) for f in ("exit_idx", "label", "conf", "score"))
    eng.close()


def test_small_segments_in_the_profile(torch, ee):
    """What the header says of the kernel timing: a small segment is booked whole under its first layer and the convolution class, exit head and admission
    included; with the fused blocks off every class and layer has launches of its own.  The operations are the same."""
    blob = W.load_net("tiny_i8")
    n = 16
    eng = ee.Engine(blob, n)
    pool, lut = dev(torch, W.input_pool(blob, n)), synthetic_lut(blob.n_stages, n)
    first = [sum(int(st["n_ops"]) for st in blob.stages[:s]) for s in range(blob.n_stages)]
    seen = {}
    for mode in (1, 0):
        eng.ir_mode(mode)
        eng.profile(True)
        eng.profile_read(len(blob.ops))
        _, stats, _ = eng.serve_stream(np.zeros(n, np.int64), pool, lut, refill=0)
        cls, lay = eng.profile_read(len(blob.ops))
        eng.profile(False)
        seen[mode] = sum(c["ops"] for c in cls.values())
        if mode:
            assert {k for k, c in cls.items() if c["launches"]} == {"conv_mfma", "compact"} and cls["conv_mfma"]["launches"] == sum(stats["seg_runs"])
            assert [x["launches"] for x in lay] == [stats["seg_runs"][first.index(k)] if k in first else 0 for k in range(len(lay))]
        else:
            assert cls["admit"]["launches"] and cls["softmax"]["launches"] == sum(stats["seg_runs"]) and all(x["launches"] for x in lay)
    assert seen[0] == seen[1] > 0
    eng.close()


def requantised(blob, lo, hi, shift, seed):
    """The network's convolutions with that shift and those bounds, weights and biases drawn so that results reach both bounds and fall between them (at 24 the bias alone decides)."""
    r = np.random.default_rng(seed)
    for op in blob.ops:
        if int(op["kind"]) not in (W.OP_CONV, W.OP_DWCONV):
            continue
        w, b = blob.op_weights(op)
        m = min(127, max(1, int(2 ** shift / np.sqrt(w.size / int(op["c_out"])))))     # results of a few hundred before the bounds
        w[:] = r.integers(-m, m + 1, size=w.shape)
        b[:] = r.integers(-2 ** min(30, shift + 7), 2 ** min(30, shift + 7), size=b.shape)
        op["shift"], op["lo"], op["hi"] = shift, lo, hi
        op["res_shift"] = min(shift, 22) if int(op["res"]) >= 0 else 0
    return blob


# the kernel that a forced configuration is there for: one of the test network's layers runs with it, the others take what covers them
FORCED_KERNELS = {0: "conv_skinny_kernel<1,32,4,1,true>", 7: "conv_stream_i8_kernel<3,3,2>", 0x221: "conv_igemm_kernel<1,128,128,128,1,true>", 0x212: "conv_igemm_kernel<1,128,64,64,1,true>",
                  0x4231: "conv_rows_kernel<1,128,4,32,true>", 0x4232: "conv_rows_kernel<1,128,4,64,true>", 0x2231: "conv_taps_kernel<1,2,4,1,4>", 0x4234: "conv_taps_kernel<1,2,2,1,4>"}


@pytest.mark.parametrize("shift", [0, 1, 2, 9, 24])
@pytest.mark.parametrize("lo, hi", [(0, 127), (-128, 127), (0, 96), (-9, 90)])
def test_requantisation_bounds_and_shifts(torch, ee, orc, lo, hi, shift):
    """The kernels of one layer that requantise whole accumulator blocks (for few pixels and staged with and without a residual, streaming and with streamed weights without, with resident
    weights with one) at the shifts and bounds where their forms part: shift 0 and 1, a shift that leaves only the bias, 0 .. 127 and others, against the oracle bit for bit."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, 9, 8, 32, 10)
    t = net.begin_stage()
    t = net.conv(t, 64, 3, 1, 1)
    t = res = net.conv(t, 128, 1, 1, 0)
    t = net.conv(t, 128, 3, 1, 1)
    net.end_stage(net.conv(t, 128, 1, 1, 0, res=res))
    blob = requantised(N._assemble(net, net.dtype, 60 + shift), lo, hi, shift, 100 * shift + hi)
    x = np.random.default_rng(shift).integers(-128, 128, size=(5, 9, 8, 32), dtype=np.int8)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, 5)
    for cfg, kernel in FORCED_KERNELS.items():
        got, names = forced(ee, cfg, lambda: kernels_of(torch, lambda: host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref)))
        assert kernel in names, (hex(cfg), names)
        assert np.array_equal(got, ref), f"cfg {cfg:#x}: {np.count_nonzero(got != ref)} of {ref.size} differ"
    assert np.unique(ref).size > 8 and (shift == 24 or (ref.min() == lo and ref.max() == hi))      # at 24 the bias alone decides, within the bounds
    eng.close()


def small_net(h, w, c):
    """One segment of convolutions small enough to run with its exit head as one launch."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, h, w, c, 10)
    t = net.conv(net.begin_stage(), 32, 3, 1, 1)
    net.end_stage(net.conv(net.conv(t, 16, 3, 1, 1), 32, 1, 1, 0, res=t))
    return N._assemble(net, net.dtype, 5)


FUSED_REQUANT = {  # network, tables, what its one launch of several layers (or of few input channels) is
    "seam": (lambda: W.bottleneck_net(9, 8, 512, blocks=2, mid=128), {"pair": {"1": [0x40001] * 4}}, "conv_seam_kernel<4,1,false>"),
    "seam with its 3x3 layer": (lambda: W.bottleneck_net(9, 8, 512, blocks=2, mid=128), {"pair": {"1": [0x40011] * 4}}, "conv_seam_kernel<4,1,true>"),
    "wide seam": (lambda: W.bottleneck_net(5, 8, 1024, blocks=2, mid=256), {"pair": {"1": [0x40012] * 4}}, "conv_seam_kernel<8,2,true>"),
    "bottleneck block": (lambda: W.bottleneck_net(9, 11, 256), {}, "bneck_block_i8_kernel<"),
    "bottleneck block with its shortcut": (lambda: W.bottleneck_net(9, 11, 64), {}, "bneck_block_i8_kernel<"),
    "inverted residual": (lambda: W.inverted_residual_net(9, 11, 32, 192, 32, 1), {}, "ir_block_i8_kernel<"),
    "first layer and pool": (lambda: W.stem_net(30, 32), {}, "stem_pool_i8_kernel<6,4>"),
    "small segment": (lambda: small_net(6, 7, 16), {}, "segment_small_i8_kernel"),
    "few input channels": (lambda: W.single_layer_net("conv", 10, 12, 24, 1, 1, 0, W.DT_I8, co=96), {}, "conv_thin_i8_kernel"),
}


@pytest.mark.parametrize("shift", [0, 1, 24])
@pytest.mark.parametrize("lo, hi", [(0, 127), (-128, 127), (0, 96)])
@pytest.mark.parametrize("kind", FUSED_REQUANT)
def test_requantisation_in_launches_of_several_layers(torch, ee, orc, kind, lo, hi, shift):
    """The same for the kernels that a forced configuration does not reach: the launch named is among those that ran, and the segment's output is the oracle's bit for bit."""
    net, tables, kernel = FUSED_REQUANT[kind]
    blob = requantised(net(), lo, hi, shift, 10 * shift + hi)
    b = 3
    x = np.random.default_rng(shift).integers(-128, 128, size=(b,) + blob.stage_in_shape(0), dtype=np.int8)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, b)
    eng.load_tables(tables)
    eng.ir_mode(2)
    got, names = kernels_of(torch, lambda: host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref))
    assert any(n.startswith(kernel) for n in names), names
    assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} differ"
    assert (np.unique(ref).size > 8 or shift == 24) and (shift == 24 or (ref.min() == lo and ref.max() == hi))
    eng.close()


@pytest.mark.parametrize("h, w, edges", [(224, 224, {1: "6,4", 2: "14,8"}), (48, 34, {2: "6,4", 42: "6,4", 43: "14,8"}), (57, 80, {16: "6,4", 17: "14,8"}), (114, 56, {11: "14,8"}),
                                         (16, 14, {256: "6,4", 257: "14,8"})], ids=str)
def test_first_layer_and_pool_in_both_tiles(torch, ee, orc, h, w, edges):
    """The fused first convolution and max-pool (int8) in small tiles and in large ones, on both sides of the rule, images that end inside a tile: against the oracle, bit for bit."""
    blob = W.stem_net(h, w, seed=h)
    n = max(edges)
    x = W.input_pool(blob, n)
    eng = ee.Engine(blob, n)
    for b, tile in edges.items():
        say(f"[case] first layer {h}x{w} b={b}")
        out, names = kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x[:b]), blob.stage_out_shape(0)))
        assert f"stem_pool_i8_kernel<{tile}>" in names, names
        ends = sorted({0, b // 2, b - 1})
        ref = orc.stage_forward(blob, 0, x[ends])
        assert np.array_equal(host(out[ends], ref), ref) and np.unique(ref).size > 8
    eng.close()


SEAM_CASES = [  # mid channels, h, w, samples: one pixel, tiles with one pixel less, none over and one over, images ending inside a tile, the widest rows that fit
    (128, 1, 1, 1), (256, 1, 2, 1), (128, 7, 9, 1), (128, 8, 8, 1), (128, 5, 13, 1), (256, 7, 9, 3), (256, 5, 13, 2), (128, 9, 11, 9), (256, 14, 14, 5), (128, 2, 300, 1), (256, 2, 144, 1),
]


@pytest.mark.parametrize("case", SEAM_CASES, ids=lambda c: "x".join(map(str, c)))
def test_seam_of_two_blocks_as_one_launch(torch, ee, orc, case):
    """The layers where two bottleneck blocks meet in one launch (both tile sizes, with and without the 3x3 layer), against the oracle and the separate layers, bit for bit; with residuals from a
    tensor of the segment and from its input, bounds that are not a ReLU's in one block, and a word where none belongs refused."""
    mid, h, w, b = case
    say(f"[case] seam {case}")
    blob = W.bottleneck_net(h, w, 4 * mid, seed=mid + h, blocks=3, mid=mid)
    for k, (lo, hi) in {1: (-20, 90), 2: (-128, 127), 3: (-7, 127)}.items():
        blob.ops[k]["lo"], blob.ops[k]["hi"] = lo, hi
    x = W.input_pool(blob, b)
    ref = orc.stage_forward(blob, 0, x)
    assert np.unique(ref).size > 8
    eng = ee.Engine(blob, b)
    xd = dev(torch, x)
    heads = [1, 4]
    taken = 0
    for form in (0x40000, 0x40010):
        for t in (1, 2):
            word = [form | t] * 3
            try:
                eng.load_tables({"pair": {str(k): word for k in heads}})
            except ee.EEError:
                assert w > 28                               # rows too wide for LDS with this tile
                continue
            taken += 1
            say(f"[case] seam {case} word {form | t:#x}")
            n, got = launches_per_layer(torch, eng, blob, xd)
            assert n == ([1, 1, 1, 0, 1, 1, 0, 1, 1] if form == 0x40000 else [1, 1, 0, 0, 1, 0, 0, 1, 1])
            got = host(got, ref)
            assert np.array_equal(got, ref), f"word {form | t:#x}: {np.count_nonzero(got != ref)} of {ref.size} differ"
    assert taken == 4 if w <= 28 else taken >= 3
    eng.pair_mode(0)
    n, got = launches_per_layer(torch, eng, blob, xd)
    assert n == [1] * 9 and np.array_equal(host(got, ref), ref)
    for layer, word in ((0, 0x40001), (2, 0x40001), (7, 0x40001), (1, 0x40000), (1, 0x40003), (1, 0x40021), (1, 0x40101), (1, 0x44001)):
        with pytest.raises(ee.EEError):
            eng.load_tables({"pair": {str(layer): [word] * 3}})
    eng.close()


@pytest.mark.parametrize("mid, hw, edges", [(128, 28, [(1, 1), (20, 1), (21, 1), (83, 1), (84, 0)]), (256, 14, [(20, 0), (21, 1), (41, 1), (42, 1), (83, 1), (84, 0)])])
def test_untuned_seams_at_the_edges_of_their_rule(torch, ee, mid, hw, edges):
    """Without a table: which numbers of samples run the seam as one launch, and the same bytes as layer by layer on both sides of every edge."""
    blob = W.bottleneck_net(hw, hw, 4 * mid, seed=3, blocks=2, mid=mid)
    eng = ee.Engine(blob, 84)
    x = dev(torch, W.input_pool(blob, 84))
    for b, fused in edges:
        say(f"[case] untuned seam {mid} {hw} {b}")
        eng.pair_mode(1)
        n, got = launches_per_layer(torch, eng, blob, x[:b])
        assert n == ([1, 1, 0, 0, 1, 1] if fused else [1] * 6), b
        eng.pair_mode(0)
        assert torch.equal(got, eng.stage_forward(0, x[:b], blob.stage_out_shape(0))), b
    eng.close()


@pytest.mark.parametrize("mid, hw, front, edges", [(128, 28, True, [(1, 0), (10, 0), (11, 1), (40, 1), (83, 1)]), (256, 14, True, [(31, 0), (32, 1), (41, 1), (42, 0), (62, 0), (63, 1)]),
                                                   (128, 28, False, [(1, 0), (20, 0)])])
def test_untuned_seams_beside_a_joint_launch(torch, ee, mid, hw, front, edges):
    """A 64-channel 1x1 layer reads the block's output too and shares a launch with the layer behind the seam: the seam runs only from the number of samples on at which it is worth more than that launch, without
    the 3x3 layer never.  The same bytes as layer by layer on both sides of every edge, and with tuned tables."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, hw, hw, 4 * mid, 10)
    t = net.begin_stage()
    for _ in range(2):
        u, sibling = net.conv(t, mid, 1, 1, 0), net.conv(t, 64, 1, 1, 0)
        t = net.conv(net.conv(u if front else sibling, mid, 3, 1, 1), 4 * mid, 1, 1, 0, res=t)
    net.end_stage(t)
    blob = N._assemble(net, net.dtype, 21)
    for op in blob.ops:
        op["shift"] = int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) * int(op["kw"])) / 127)))
        op["res_shift"] = int(op["shift"]) - 1 if int(op["res"]) >= 0 else 0
    n_max = max(b for b, _ in edges)
    eng = ee.Engine(blob, n_max)
    x = dev(torch, W.input_pool(blob, n_max))
    for tuned in (False, True):
        if tuned:
            eng.pair_mode(1)
            eng.autotune(reps=1)
        for b, fused in edges:
            say(f"[case] seam beside a joint launch {mid} {hw} {front} {b} {'tuned' if tuned else ''}")
            eng.pair_mode(1)
            n, got = launches_per_layer(torch, eng, blob, x[:b])
            assert tuned or n == ([1, 0, 1, 0, 0, 1, 1, 1] if fused else [1, 0, 1, 1, 1, 0, 1, 1]), b
            eng.pair_mode(0)
            want = eng.stage_forward(0, x[:b], blob.stage_out_shape(0))
            assert torch.equal(got, want) and torch.unique(want).numel() > 8, b
    eng.close()


ROWS_CASES = [  # h, w, input bytes per pixel, output channels, stride, samples: no whole tile, ragged last tiles, several tiles per workgroup, every channel grouping
    (1, 1, 128, 256, 1, 1), (5, 7, 128, 512, 1, 3), (9, 11, 256, 128, 2, 5), (56, 56, 128, 256, 1, 25), (13, 6, 256, 1024, 1, 4), (28, 28, 256, 256, 2, 9),
    (14, 14, 512, 512, 1, 7), (8, 8, 512, 128, 1, 3), (10, 10, 1024, 2048, 1, 20), (7, 7, 1024, 128, 1, 2),
]


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("case", ROWS_CASES, ids=lambda c: "x".join(map(str, c)))
def test_resident_weights_1x1(torch, ee, orc, case, dtype):
    """The 1x1 kernel with resident weights, both tile sizes, with and without a residual: int8 against the oracle bit for bit; bf16 against the
    staged kernel bit for bit (its sums run in the same order) and the oracle under the tolerance of the tiling tests."""
    from workloads import nets as N
    h, w, kb, co, stride, n = case
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, h, w, kb // (1 if i8 else 2), 10)
    t = net.begin_stage()
    res = net.conv(t, co, 1, stride, 0, act="linear")
    net.end_stage(net.conv(t, co, 1, stride, 0, res=res))
    blob = N._assemble(net, net.dtype, 40 + h)
    r = np.random.default_rng(co + kb)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"])) / 127))))
        op["res_shift"] = int(op["shift"]) - 2 if int(op["res"]) >= 0 else 0
        if not i8:
            blob.op_weights(op)[1][:] = r.normal(size=co) * 0.3
    x = W.input_pool(blob, n)
    eng = ee.Engine(blob, n)
    ref = orc.stage_forward(blob, 0, x)
    for cfg, px in ((0x4231, 32), (0x4232, 64)):                           # the kernel runs on both layers, but for tiles of 64 pixels of 1 KiB
        names = [k for k in forced(ee, cfg, lambda: kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x), ref.shape[1:])))[1] if k.startswith("conv_rows")]
        assert names == [f"conv_rows_kernel<{1 if i8 else 2},{kb},{4 if co == 128 else 8},{px},{residual}>" for residual in ("false", "true") if kb < 1024 or px == 32]
    staged = None
    for cfg in (0x221, 0x4231, 0x4232):
        say(f"[case] {dtype} {case} cfg {cfg:#x}")
        old = ee.tune_conv_tile(cfg)
        try:
            got = host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref)
        finally:
            ee.tune_conv_tile(old)
        if i8:
            assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
        else:
            staged = got if staged is None else staged
            assert np.array_equal(got, staged), f"{np.count_nonzero(got != staged)} of {ref.size} differ, first at {np.argwhere(got != staged)[:3].tolist()}"
            rf, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(got).astype(np.float64)
            assert np.all(np.abs(g - rf) <= 2e-2 * (np.abs(rf).reshape(n, -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30))
    assert np.unique(ref).size > 8
    eng.close()


TAPS_CASES = [  # h, w, input bytes per pixel, output channels, kernel (rows, columns), samples: one ragged tile, tiles over several samples, images smaller than the
    # window, every group of steps (pixels of whole 128, 64 and 32 bytes) and any number of them, a slab near the limit of LDS, channels that end inside a block of 32 or leave wavefronts idle
    (1, 1, 128, 32, (3, 3), 1), (2, 3, 128, 144, (3, 3), 5), (7, 7, 512, 512, (3, 3), 9), (14, 14, 256, 256, (3, 3), 5), (28, 28, 128, 128, (3, 3), 3), (17, 17, 384, 192, (1, 7), 3),
    (17, 17, 128, 80, (7, 1), 2), (9, 11, 1024, 64, (3, 3), 2), (13, 6, 256, 320, (5, 5), 4), (56, 56, 128, 64, (3, 3), 2), (1, 40, 640, 96, (1, 3), 8),
    (56, 56, 64, 64, (3, 3), 2), (35, 35, 96, 96, (3, 3), 2), (17, 17, 160, 160, (1, 7), 3), (17, 17, 192, 192, (7, 1), 3), (8, 8, 448, 384, (3, 3), 3), (6, 5, 96, 32, (5, 1), 2),
]
TAPS_CONFIGS = [0x2231, 0x2331, 0x2431, 0x4331, 0x4431, 0x2432, 0x4432, 0x4234, 0x4334, 0x4434, 0x2232, 0x2332, 0x4332]      # the last four share the reduction between wavefronts

# configuration word -> blocks of 32 pixels, blocks of 32 channels, wavefronts that share a reduction
TAPS_TILES = {0x2231: (2, 4, 1), 0x2331: (3, 4, 1), 0x2431: (4, 4, 1), 0x4331: (5, 4, 1), 0x4431: (7, 4, 1), 0x2432: (4, 8, 1), 0x4432: (7, 8, 1), 0x4234: (2, 2, 1), 0x4334: (4, 2, 1),
              0x4434: (2, 2, 2), 0x2232: (2, 4, 2), 0x2332: (4, 4, 2), 0x4332: (2, 2, 4)}


def taps_kernel(es, cfg, kb):
    return "conv_taps_kernel<%d,%d,%d,%d,%d>" % ((es,) + TAPS_TILES[cfg] + (4 if kb % 128 == 0 else 2 if kb % 64 == 0 else 1,))


def taps_runs(w, kb, kh, kw, es, cfg, residual, pooled_pixels=0):
    """Whether the kernel with streamed weights has the tile on a layer over pixels of kb bytes in rows of w: tiles of other than 2 and 4 blocks need whole runs of 128 bytes, bf16
    ones of 64; LDS holds a pixel of zeros and the slab (rows 16 bytes longer than a pixel, whole copies of the workgroup), partial sums over them, the output tile (behind
    them where a residual is staged) and, pooling for the exit head, 8 rows of sums for the samples a tile touches (pooled_pixels: of a sample)."""
    tm, nw, kp = TAPS_TILES[cfg]
    if kb % (32 * es) or (kb % 128 and tm not in (2, 4)):
        return False
    copies = 64 * nw * kp
    slab = -(-(32 * tm + (kh - 1) * w + kw - 1) * (kb // 16 + 1) // copies) * copies * 16
    parts = min(tm, kp) * (kp - 1) * nw * -(-tm // kp) * 4096 if kp > 1 else 0
    tile, front = 32 * tm * 32 * nw * es, max(kb + slab, parts)
    lds = front + tile if residual else max(front, parts + tile)
    if pooled_pixels:
        lds += 8 * 32 * nw * 4
    return lds <= 160 * 1024 and not (pooled_pixels and (32 * tm - 1) // pooled_pixels + 2 > 8)


# (height, width, bytes per pixel, output channels, kernel, images): whole and broken 32-byte steps to a pixel, rows of an even and an odd number of chunks, tiles within a row and over
# several rows and images, one pixel per image, kernels of one row and column, blocks of channels that are not there
VALID_CASES = [
    (73, 73, 80, 192, (3, 3), 2), (5, 7, 80, 32, (3, 3), 9), (3, 3, 64, 48, (3, 3), 70), (9, 4, 112, 96, (2, 3), 5), (40, 12, 128, 64, (5, 1), 3), (4, 90, 96, 256, (1, 5), 4),
    (8, 8, 176, 160, (3, 3), 6), (74, 74, 80, 192, (3, 3), 6), (11, 34, 208, 272, (2, 2), 1), (6, 5, 1040, 32, (3, 5), 4),
]

VALID_CONFIGS = {0x2431: 4, 0x4334: 2, 0x4531: 3}          # blocks of 32 channels; tiles of 128 pixels


def valid_runs(w, h, kb, kh, kw, cfg, residual):
    """Whether the kernel has the tile on a layer without padding: LDS for a pixel, the slab (an odd number of chunks to a row; what lies between the pixels of a tile that goes on to
    another row or image) and the output tile."""
    if cfg not in VALID_CONFIGS:
        return False
    ho, wo, nw = h - kh + 1, w - kw + 1, VALID_CONFIGS[cfg]
    rows = 128 + (kh - 1) * w + kw - 1 + -(-127 // wo) * (kw - 1) + -(-127 // (ho * wo)) * (kh - 1) * w
    front, tile = kb + -(-rows * (kb // 16 | 1) // (64 * nw)) * 64 * nw * 16, 128 * 32 * nw
    return (front + tile if residual else max(front, tile)) <= 160 * 1024


@pytest.mark.parametrize("case", VALID_CASES, ids=lambda c: "x".join(map(str, c)))
def test_streamed_weights_convolution_without_padding(torch, ee, orc, case):
    """The same kernel on layers whose output is smaller than their input, every tile, with and without a residual, against the oracle bit for bit."""
    from workloads import nets as N
    h, w, kb, co, (kh, kw), n = case
    net = N._Net(W.DT_I8, h, w, kb, 10)
    t = net.begin_stage()
    res = net.conv(t, co, (kh, kw), 1, (0, 0), act="linear")
    net.end_stage(net.conv(t, co, (kh, kw), 1, (0, 0), res=res))
    blob = N._assemble(net, net.dtype, 90 + h)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * kh * kw) / 127))))
        op["res_shift"] = int(op["shift"]) - 2 if int(op["res"]) >= 0 else 0
    x = W.input_pool(blob, n)
    eng = ee.Engine(blob, n)
    ref = orc.stage_forward(blob, 0, x)
    assert len(np.unique(ref)) > 20
    for cfg in [0, 0x4531] + TAPS_CONFIGS:
        say(f"[case] {case} cfg {cfg:#x}")
        got, names = forced(ee, cfg, lambda: kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x), ref.shape[1:])))
        assert np.array_equal(got.cpu().numpy(), ref), hex(cfg)
        if cfg:
            runs = sum(valid_runs(w, h, kb, kh, kw, cfg, residual) for residual in (False, True))
            assert [k for k in names if k.startswith("conv_taps")] == ["conv_taps_kernel<1,4,%d,1,0>" % VALID_CONFIGS.get(cfg, 0)] * runs, hex(cfg)


# (height, width, bytes per pixel, output channels, kernel, images from which on, 32-channel blocks of the tile): 1280 blocks of 64 x 64 outputs and 640 bytes of reduction; 96 channels where
# they leave fewer empty than 128 and the slab is small enough for four workgroups to a CU
VALID_RULE = [(74, 74, 80, 192, (3, 3), 6, 3), (38, 38, 80, 128, (3, 3), 32, 4), (35, 70, 176, 192, (3, 2), 12, 4), (38, 38, 64, 128, (3, 3), None, 0), (20, 66, 128, 48, (5, 1), 78, 4)]


@pytest.mark.parametrize("case", VALID_RULE, ids=lambda c: "x".join(map(str, c)))
def test_untuned_convolution_without_padding(torch, ee, case):
    """Which tile of the kernel an untuned layer without padding gets, on both sides of its rule: the bytes of the staged kernel."""
    h, w, kb, co, (kh, kw), edge, nw = case
    from workloads import nets as N
    net = N._Net(W.DT_I8, h, w, kb, 10)
    net.end_stage(net.conv(net.begin_stage(), co, (kh, kw), 1, (0, 0), act="linear"))
    blob = N._assemble(net, net.dtype, h)
    blob.ops[0]["shift"] = int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(kb * kh * kw) / 127)))
    n = edge or 40
    x = torch.randint(-128, 128, (n, h, w, kb), dtype=torch.int8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(h))
    eng, shape = ee.Engine(blob, n), blob.stage_out_shape(0)
    for b in (n, n - 1):
        say(f"[case] untuned without padding {case} {b}")
        got, names = kernels_of(torch, lambda: eng.stage_forward(0, x[:b], shape))
        assert [k for k in names if k.startswith("conv_taps")] == ["conv_taps_kernel<1,4,%d,1,0>" % nw] * (b == edge), names
        want, names = forced(ee, 0x221, lambda: kernels_of(torch, lambda: eng.stage_forward(0, x[:b], shape)))
        assert any(k.startswith("conv_igemm_kernel") for k in names) and torch.equal(got, want) and torch.unique(got).numel() > 20
    eng.close()


@pytest.mark.parametrize("co", [64, 96, 160, 192])
def test_convolution_without_padding_writes_slots_and_pools(torch, ee, co):
    """Segments that end in a 3x3 layer without padding and with a residual: output slots in order and scattered, the exit head's pooling in its launch.  Every request gets what the copying compaction with the
    staged kernel gives it, with every tile."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, 15, 13, 64, 10)
    for _ in range(3):
        u = net.conv(net.begin_stage(), co, 1, 1, 0)
        net.end_stage(net.conv(u, co, 3, 1, 0, res=net.maxpool(u, 3, 1, 0)))
    blob = N._assemble(net, net.dtype, co)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) * int(op["kw"])) / 127)))) if int(op["kind"]) == W.OP_CONV else 0
        op["res_shift"] = max(0, int(op["shift"]) - 2) if int(op["res"]) >= 0 else 0
    b_max = 8
    pool = W.input_pool(blob, 64)
    blob.exits["frac_bits"] = 12
    act, eng = dev(torch, pool[:8]), ee.Engine(blob, b_max)
    for s in range(3):                                                     # thresholds that split the requests
        act = eng.stage_forward(s, act, blob.stage_out_shape(s))
        blob.exits[s]["thr"] = float(np.median(eng.exit_head(s, act, 0.5)[1].cpu().numpy())) if s < 2 else 0.5
    eng.close()
    eng = ee.Engine(blob, b_max)
    assert eng.zero_copy_supported()
    serve = scattered_stream(torch, eng, pool, 512, b_max)
    want = None
    for cfg, zc in [(0x221, 0)] + [(cfg, zc) for cfg in VALID_CONFIGS for zc in (0, 1)]:
        say(f"[case] slots without padding {co} cfg {cfg:#x} zero_copy {zc}")
        got, names = forced(ee, cfg, lambda: serve(zc))
        assert cfg == 0x221 or names.count("conv_taps_kernel<1,4,%d,1,0>" % VALID_CONFIGS[cfg]) == names.count("fc_kernel<1,4,1>") + sum(k.startswith("head_small") for k in names) > 60, names[:40]
        assert not [k for k in names if k.startswith("gap_")]
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, cfg, zc)
    assert np.all(np.bincount(want["exit_idx"], minlength=3) > 0)
    eng.close()


@pytest.mark.parametrize("co", [32, 96, 144])
def test_convolution_without_padding_into_a_slice(torch, ee, orc, co):
    """The same layers where they fill channels [48, 48 + co) of a wider tensor, every tile, against the oracle."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, 13, 17, 80, 10)
    t = net.begin_stage()
    cat = net.new_concat(11, 16, 48 + co + 16)
    net.conv(t, 48, (3, 2), 1, (0, 0), into=(cat, 0))
    net.conv(t, co, (3, 2), 1, (0, 0), act="linear", into=(cat, 48))
    net.conv(t, 16, (3, 2), 1, (0, 0), into=(cat, 48 + co))
    net.end_stage(cat)
    blob = N._assemble(net, net.dtype, co)
    for op in blob.ops:
        op["shift"] = int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(480) / 127)))
    x = W.input_pool(blob, 5)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, 5)
    for cfg in VALID_CONFIGS:
        say(f"[case] slice without padding {co} cfg {cfg:#x}")
        got, names = forced(ee, cfg, lambda: kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x), ref.shape[1:])))
        assert names.count("conv_taps_kernel<1,4,%d,1,0>" % VALID_CONFIGS[cfg]) == 3 and np.array_equal(host(got, ref), ref), hex(cfg)
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("case", TAPS_CASES, ids=lambda c: "x".join(map(str, c)))
def test_streamed_weights_same_size_convolution(torch, ee, orc, case, dtype):
    """The stride-1 kernel with weights streamed into registers, every tile, with and without a residual: int8 against the oracle bit for bit; bf16
    against the staged kernel bit for bit (its sums run in the same order) and the oracle under the tolerance of the tiling tests."""
    from workloads import nets as N
    h, w, kb, co, (kh, kw), n = case
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, h, w, kb // (1 if i8 else 2), 10)
    t = net.begin_stage()
    res = net.conv(t, co, (kh, kw), 1, (kh // 2, kw // 2), act="linear")
    net.end_stage(net.conv(t, co, (kh, kw), 1, (kh // 2, kw // 2), res=res))
    blob = N._assemble(net, net.dtype, 60 + h)
    r = np.random.default_rng(co + kb)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * kh * kw) / 127))))
        op["res_shift"] = int(op["shift"]) - 2 if int(op["res"]) >= 0 else 0
        if not i8:
            blob.op_weights(op)[1][:] = r.normal(size=co) * 0.3
    x = W.input_pool(blob, n)
    eng = ee.Engine(blob, n)
    ref = orc.stage_forward(blob, 0, x)
    for cfg in TAPS_CONFIGS:                                               # the tile runs on the layers where it exists
        names = [k for k in forced(ee, cfg, lambda: kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x), ref.shape[1:])))[1] if k.startswith("conv_taps")]
        runs = [taps_runs(w, kb, kh, kw, 1 if i8 else 2, cfg, residual) for residual in (False, True)]
        assert names == [taps_kernel(1 if i8 else 2, cfg, kb) for run in runs if run], (hex(cfg), runs)
    staged = None
    for cfg in [0x221] + TAPS_CONFIGS:
        say(f"[case] {dtype} {case} cfg {cfg:#x}")
        old = ee.tune_conv_tile(cfg)
        try:
            got = host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref)
        finally:
            ee.tune_conv_tile(old)
        if i8:
            assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
        else:
            staged = got if staged is None else staged
            assert cfg in TAPS_CONFIGS[-4:] or np.array_equal(got, staged), f"{np.count_nonzero(got != staged)} of {ref.size} differ, first at {np.argwhere(got != staged)[:3].tolist()}"
            rf, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(got).astype(np.float64)
            assert np.all(np.abs(g - rf) <= 2e-2 * (np.abs(rf).reshape(n, -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30))
    assert np.unique(ref).size > 8
    eng.close()


@pytest.mark.parametrize("dtype, ci, co", [("i8", 128, 72), ("bf16", 64, 100)])
def test_untuned_slab_kernel(torch, ee, orc, dtype, ci, co):
    """What untuned launches leave to the slab kernel: 3x3 layers whose output is no whole 16-byte chunks, its three choices of tile and step (two rounds of 64 x 64 tiles,
    four rounds), against the oracle."""
    from workloads import nets as N
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, 28, 28, ci, 10)
    net.end_stage(net.conv(net.conv(net.begin_stage(), co, 3, 1, 1), 64, 1, 1, 0))
    blob = N._assemble(net, net.dtype, 29)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) ** 2) / 127))))
    x = W.input_pool(blob, 48)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, 48)
    for b, tile in ((24, "128,64,256"), (48, "128,128,128" if i8 else "128,64,128")):
        say(f"[case] untuned slab kernel {dtype} {b} samples")
        out, names = kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]))
        assert names[0] == f"conv_slab_kernel<{1 if i8 else 2},{tile}>", names
        got = host(out, ref)
        if i8:
            assert np.array_equal(got, ref[:b]), f"{np.count_nonzero(got != ref[:b])} of {got.size} differ"
        else:
            rf, g = bf16_to_f32(ref[:b]).astype(np.float64), bf16_to_f32(got).astype(np.float64)
            assert np.all(np.abs(g - rf) <= 2e-2 * (np.abs(rf).reshape(b, -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30))
    assert np.unique(ref).size > 8
    eng.close()


LOADED_WORDS = [  # h, input channels, output channels, kernel, stride, words that run on the layer, words that do not
    (14, 128, 128, 3, 1, [0x2231, 0x4431, 0x4332], [0x4231, 0x4232]),
    (14, 128, 128, 3, 2, [0x221], [0x4231, 0x4232, 0x2231, 0x4334]),              # not as large as its input
    (14, 128, 128, 1, 1, [0x4231, 0x4232], [0x2231, 0x2432]),
    (7, 1024, 256, 1, 1, [0x4231], [0x4232]),                                      # tiles of 64 pixels of 1 KiB do not exist
    (14, 96, 128, 3, 1, [0x2231, 0x2431, 0x4434], [0x2331, 0x4331, 0x4432]),      # pixels of 32-byte runs: 2 and 4 blocks only
    (28, 768, 128, 3, 1, [0x2231], [0x4431, 0x4432]),                              # 282 slab rows of 784 bytes do not fit LDS
    (14, 128, 72, 3, 1, [0x221], [0x2231, 0x4231]),                                # output pixels of no whole 16-byte chunks
]


@pytest.mark.parametrize("case", LOADED_WORDS, ids=lambda c: "x".join(map(str, c[:5])))
def test_loaded_words_are_checked_against_the_layer(torch, ee, orc, case):
    """A stored word that names the kernel with resident or with streamed weights is accepted where it runs and refused elsewhere; a refused table
    leaves the old one in place."""
    from workloads import nets as N
    h, ci, co, k, stride, good, bad = case
    net = N._Net(W.DT_I8, h, h, ci, 10)
    t = net.conv(net.begin_stage(), co, k, stride, k // 2)
    net.end_stage(net.conv(t, 64, 1, 1, 0))
    blob = N._assemble(net, W.DT_I8, 5)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) ** 2) / 127))))
    x = W.input_pool(blob, 3)
    ref = orc.stage_forward(blob, 0, x)
    eng = ee.Engine(blob, 3)
    for cfg in good:
        say(f"[case] loaded word {cfg:#x} on {case[:5]}")
        eng.load_tables({"config": {"0": [cfg, cfg, cfg]}})
        assert np.array_equal(host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref), ref)
    for cfg in bad:
        with pytest.raises(ee.EEError) as err:
            eng.load_tables({"config": {"0": [good[0], good[0], cfg]}})
        assert err.value.code == ee.EE_ERR_ARG and eng.config_table(0) == [good[-1]] * 3
    eng.close()


@pytest.mark.parametrize("case", [(7, 7, 128, 256, 1), (5, 5, 256, 512, 1), (28, 28, 128, 128, 1), (7, 7, 64, 128, 3), (6, 5, 96, 96, 3), (14, 14, 256, 256, 3), (28, 28, 128, 64, 3), (5, 5, 128, 128, 3)],
                         ids=lambda c: "x".join(map(str, c)))
def test_pooling_for_the_exit_head_rides_on_the_last_layer(torch, ee, orc, case):
    """Segments that end in a 1x1 or 3x3 layer with a residual, served with every kernel that adds up the exit head's channel sums in its own launch (blocks of
    pixels over one, two and three samples, ragged last tiles): label and confidence of every request are the oracle's."""
    from workloads import nets as N
    h, w, ci, co, k = case
    net = N._Net(W.DT_I8, h, w, ci, 10)
    t = net.begin_stage()
    res = net.conv(t, co, k, 1, k // 2, act="linear")
    net.end_stage(net.conv(t, co, k, 1, k // 2, res=res))
    blob = N._assemble(net, W.DT_I8, 90 + h)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * k * k) / 127))))
        op["res_shift"] = int(op["shift"]) - 2 if int(op["res"]) >= 0 else 0
    blob.exits[0]["frac_bits"] = 10
    n, b_max = 40, 11
    x = W.input_pool(blob, n)
    label, conf = orc.exit_head(blob, 0, orc.stage_forward(blob, 0, x), 0.5)[:2]
    eng = ee.Engine(blob, b_max)
    lut = synthetic_lut(blob.n_stages, b_max)
    for cfg in [0, 0x221] + ([0x4231, 0x4232] if k == 1 else TAPS_CONFIGS):
        say(f"[case] pooling {case} cfg {cfg:#x}")
        old = ee.tune_conv_tile(cfg)
        try:
            got = eng.serve_stream(np.zeros(n, np.int64), dev(torch, x), lut, refill=0)[0]
        finally:
            ee.tune_conv_tile(old)
        assert np.array_equal(got["label"], label) and np.array_equal(got["conf"], conf), f"{cfg:#x}"
        # no kernel pools apart, and the forced one runs in each of the four batches where it exists; that with resident weights does not pool: on the first layer
        names = forced(ee, cfg, lambda: kernels_of(torch, lambda: eng.serve_stream(np.zeros(n, np.int64), dev(torch, x), lut, refill=0)))[1]
        assert names and not [name for name in names if name.startswith("gap_")]
        if k == 1 and cfg in (0x4231, 0x4232):
            assert names.count(f"conv_rows_kernel<1,{ci},{4 if co == 128 else 8},{32 if cfg == 0x4231 else 64},false>") == 4
        elif cfg in TAPS_TILES:
            assert names.count(taps_kernel(1, cfg, ci)) == 4 * (taps_runs(w, ci, k, k, 1, cfg, False) + taps_runs(w, ci, k, k, 1, cfg, True, h * w))
    assert np.unique(conf).size > 8
    eng.close()


def test_tuned_words_of_a_pooling_layer_fit_with_the_pooling(torch, ee):
    """The layer that pools for the exit head when it serves: the tuner names no tile that covers more than 8 samples (7 blocks of 32 pixels on 5 x 5 images, the
    fastest one without the pooling at 512 samples and more) or a kernel that does not pool, since the launch that pools could not use it."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, 5, 5, 512, 10)
    t = net.begin_stage()
    res = net.conv(t, 512, 1, 1, 0, act="linear")
    net.end_stage(net.conv(t, 512, 3, 1, 1, res=res))
    eng = ee.Engine(N._assemble(net, W.DT_I8, 3), 1024)
    eng.autotune(reps=2)
    words = eng.config_table(1)
    assert len(words) == 11 and not set(words) & {0x4431, 0x4432, 0x4231, 0x4232, 7} and max(words) < 0x10000, [hex(w) for w in words]
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
def test_streamed_weights_write_slots(torch, ee, orc, dtype):
    """Zero-copy serving of segments that end in a 3x3 layer with a residual, with the kernel with streamed weights forced wherever it runs (one wavefront per
    reduction, so that bf16 results are the staged kernel's bits): what every request gets is that of the copying compaction with the staged kernel."""
    from workloads import nets as N
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, 11, 9, 64, 10)
    for _ in range(3):
        t = net.begin_stage()
        u = net.conv(t, 64, 1, 1, 0)
        res = net.conv(t, 64, 1, 1, 0, act="linear")
        net.end_stage(net.conv(u, 64, 3, 1, 1, res=res))
    blob = N._assemble(net, net.dtype, 17)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) * int(op["kw"])) / 127))))
        op["res_shift"] = max(0, int(op["shift"]) - 2) if int(op["res"]) >= 0 else 0
    n, b_max = 64, 8
    pool = W.input_pool(blob, n)
    act = pool[:24]
    for s in range(3):
        if i8:
            blob.exits[s]["frac_bits"] = 12
        act = orc.stage_forward(blob, s, act)
        blob.exits[s]["thr"] = float(np.median(orc.exit_head(blob, s, act, 0.5)[1])) if s < 2 else 0.5
    eng = ee.Engine(blob, b_max)
    assert eng.zero_copy_supported()
    lut = synthetic_lut(blob.n_stages, b_max)
    want = None
    for cfg, zc in ((0x221, 0), (0x2231, 1), (0x4334, 1), (0x2431, 0)):
        say(f"[case] slots {dtype} cfg {cfg:#x} zero_copy {zc}")
        old = ee.tune_conv_tile(cfg)
        try:
            got = eng.serve_stream(np.zeros(n, np.int64), dev(torch, pool), lut, refill=2, zero_copy=zc)[0]
        finally:
            ee.tune_conv_tile(old)
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, cfg, zc)
    assert np.count_nonzero(np.bincount(want["exit_idx"], minlength=3)) > 1
    serve = scattered_stream(torch, eng, pool, 512, b_max)                 # the same with output slots that are no run, in a kernel that ends each of 73 steps
    want = None
    for cfg, zc in ((0x221, 0), (0x2231, 1), (0x4334, 1), (0x2431, 1)):
        say(f"[case] scattered slots {dtype} cfg {cfg:#x} zero_copy {zc}")
        got, names = forced(ee, cfg, lambda: serve(zc))
        assert cfg == 0x221 or names.count(taps_kernel(1 if i8 else 2, cfg, 64 if i8 else 128)) == 73
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, cfg, zc)
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
def test_resident_weights_1x1_takes_slot_tables(torch, ee, orc, dtype):
    """Zero-copy serving with the kernel forced wherever it runs, on layers that read a segment's input through a slot table (its output slots are runs)."""
    blob = W.bottleneck_net(11, 9, 256, seed=3, blocks=2, stages=3, dtype=W.DT_I8 if dtype == "i8" else W.DT_BF16)
    n, b_max = 64, 8
    pool = W.input_pool(blob, n)
    act = pool[:24]
    for s in range(2):
        act = orc.stage_forward(blob, s, act)
        blob.exits[s]["frac_bits"] = 12 if dtype == "i8" else blob.exits[s]["frac_bits"]
        blob.exits[s]["thr"] = float(np.median(orc.exit_head(blob, s, act, 0.5)[1]))
    say(f"[case] {dtype} slots")
    eng = ee.Engine(blob, b_max)
    eng.ir_mode(0)
    assert eng.zero_copy_supported()
    lut = synthetic_lut(blob.n_stages, b_max)
    dpool = dev(torch, pool)
    want = None
    for cfg, zc in ((0x221, 0), (0x4231, 1), (0x4232, 1), (0x4232, 0)):
        old = ee.tune_conv_tile(cfg)
        try:
            got = eng.serve_stream(np.zeros(n, np.int64), dpool, lut, refill=2, zero_copy=zc)[0]
        finally:
            ee.tune_conv_tile(old)
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, cfg, zc)
    assert np.count_nonzero(np.bincount(want["exit_idx"], minlength=3)) > 1
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
def test_resident_weights_1x1_writes_slots(torch, ee, orc, dtype):
    """Zero-copy serving of segments of two 1x1 layers, of which one reads the segment's input through a slot table and the other writes its output through one (without a
    residual: int8 launches that pool for the exit head go to another kernel): what every request gets is that of the copying compaction with the staged kernel."""
    from workloads import nets as N
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, 11, 9, 256, 10)
    for _ in range(3):
        net.end_stage(net.conv(net.conv(net.begin_stage(), 128, 1, 1, 0), 256, 1, 1, 0))
    blob = N._assemble(net, net.dtype, 19)
    for op in blob.ops:
        op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"])) / 127))))
    b_max = 8
    pool = W.input_pool(blob, 64)
    act = pool[:24]
    for s in range(2):
        act = orc.stage_forward(blob, s, act)
        blob.exits[s]["frac_bits"] = 12 if i8 else blob.exits[s]["frac_bits"]
        blob.exits[s]["thr"] = float(np.median(orc.exit_head(blob, s, act, 0.5)[1]))
    eng = ee.Engine(blob, b_max)
    assert eng.zero_copy_supported()
    serve = scattered_stream(torch, eng, pool, 512, b_max)
    want = None
    for cfg, zc in ((0x221, 0), (0x4231, 1), (0x4232, 1), (0x4232, 0)):
        say(f"[case] scattered slots {dtype} cfg {cfg:#x} zero_copy {zc}")
        got, names = forced(ee, cfg, lambda: serve(zc))
        for ci, nb in ((256, 4), (128, 8)):                                # both layers of every step
            assert cfg == 0x221 or names.count("conv_rows_kernel<%d,%d,%d,%d,false>" % (((1, ci) if i8 else (2, 2 * ci)) + (nb, 32 if cfg == 0x4231 else 64))) == 73
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, cfg, zc)
    eng.close()


GROUP_CFGS = [0x211, 0x331, 0x422, 0x232, 0x313, 0x423, 0x333, 0x214, 0x324, 0x434] + [0x2213, 0x2214, 0x2223, 0x2224, 0x4213, 0x4214]


@pytest.mark.parametrize("cfg", GROUP_CFGS)
def test_sibling_layers_in_one_launch_bit_exact(torch, ee, orc, cfg):
    """Every configuration of the launch that runs a block's branches (or a first layer and its shortcut) together: branches of different
    kernels, widths and reductions, channel slices at odd offsets, tiles and eighths of the batch that do not divide."""
    for blob in [W.load_net("inception_small_i8"), W.load_net("resnet50_small_i8"), W.random_net(5, W.DT_I8), W.random_net(9, W.DT_I8)]:
        eng = ee.Engine(blob, 5)
        eng.ir_mode(0)
        heads = 0
        for layer in range(len(blob.ops)):
            try:
                eng.load_tables({"group": {str(layer): [cfg]}})
                heads += 1
            except ee.EEError:
                pass
        for b in (5, 1):
            act = W.input_pool(blob, b)
            for s in range(blob.n_stages):
                say(f"[case] cfg {cfg:#x} {len(blob.ops)} layers, {heads} joint launches, segment {s} b={b}")
                ref = orc.stage_forward(blob, s, act)
                got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
                assert np.array_equal(got, ref), f"segment {s} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ"
                act = ref
        if len(blob.ops) > 40:
            assert heads > 0
        eng.close()


@pytest.mark.parametrize("hw, ci, c1, c2, stride", [(28, 128, 64, 256, 2), (13, 64, 160, 96, 2), (9, 96, 32, 320, 3), (12, 64, 64, 64, 1)])
def test_siblings_that_read_one_input_take_turns(torch, ee, orc, hw, ci, c1, c2, stride):
    """Joint launches of 1x1 layers over one input, whose tiles go out in rounds: as many tiles of pixels to each, 2 to 9 times as many to one, ratios that do not come out even, fewer tiles than XCDs."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, hw, hw, ci, 10)
    t = net.conv(net.begin_stage(), ci, 1, 1, 0)
    u, v = net.conv(t, c1, 1, 1, 0), net.conv(t, c2, 1, stride, 0, act="linear")
    net.end_stage(net.conv(u, c2, 3, stride, 1, res=v))
    blob = N._assemble(net, net.dtype, 31)
    for op in blob.ops:
        op["shift"] = int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) ** 2) / 127)))
        op["res_shift"] = int(op["shift"]) - 1 if int(op["res"]) >= 0 else 0
    eng = ee.Engine(blob, 37)
    x = W.input_pool(blob, 37)
    ref = orc.stage_forward(blob, 0, x)
    assert len(np.unique(ref)) > 20
    for cfg in (0x211, 0x222, 0x333, 0x214):
        eng.load_tables({"group": {"1": [cfg] * 16}})
        for b in (1, 3, 37):
            say(f"[case] rounds {hw} {ci} {c1} {c2} /{stride} cfg {cfg:#x} b={b}")
            n, got = launches_per_layer(torch, eng, blob, dev(torch, x[:b]))
            assert n == [1, 1, 0, 1] and np.array_equal(host(got, ref), ref[:b]), n
    eng.close()


def sibling_net(h, c, branches):
    """One segment: a 1x1 layer, then int8 branches [(kernel, channels)] over its output that fill one tensor."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, h, h, c, 10)
    t = net.conv(net.begin_stage(), c, 1, 1, 0)
    cat, off = net.new_concat(h, h, sum(co for _, co in branches)), 0
    for (kh, kw), co in branches:
        net.conv(t, co, (kh, kw), 1, (kh // 2, kw // 2), into=(cat, off))
        off += co
    net.end_stage(cat)
    blob = N._assemble(net, W.DT_I8, 77)
    for op in blob.ops:
        op["shift"] = 6 + int(op["kh"]) // 2 + int(op["kw"]) // 2
    return blob


def launches_per_layer(torch, eng, blob, x):
    eng.profile(True)
    eng.profile_read(len(blob.ops))
    out = eng.stage_forward(0, x, blob.stage_out_shape(0))
    lay = eng.profile_read(len(blob.ops))[1]
    eng.profile(False)
    torch.cuda.synchronize()
    return [v["launches"] for v in lay], out


def test_loaded_layer_tables_without_a_joint_one_are_used(torch, ee):
    """Layers whose own table was loaded run with it, one after the other, unless a table for their joint launch says otherwise."""
    blob = sibling_net(14, 64, [((1, 1), 32), ((3, 3), 48)])
    eng = ee.Engine(blob, 4)
    x = torch.randint(-128, 128, (4, 14, 14, 64), dtype=torch.int8, device="cuda")
    n, ref = launches_per_layer(torch, eng, blob, x)
    assert n == [1, 1, 0]                                  # no table at all: together
    for tables, want in (({"config": {"2": [0x313] * 3}}, [1, 1, 1]), ({"group": {"1": [0x313] * 3}}, [1, 1, 0]), ({"group": {"1": [0] * 3}}, [1, 1, 1]),
                         ({"group": {"1": []}}, [1, 1, 1]), ({"config": {"2": []}}, [1, 1, 0])):
        eng.load_tables(tables)
        n, out = launches_per_layer(torch, eng, blob, x)
        assert n == want, tables
        assert torch.equal(out, ref)
    eng.close()


# image, channels, branches, batch, whether they go together without tables: below and from the sizes at which the streaming kernel
# (2^19 pixels), the one with streamed weights (2 million tile-bytes per launch saved) and the one with resident weights (every member, or one
# of 6144 tiles) win as launches of their own; an output of no whole 16-byte chunks (72 channels), which the slab kernel runs (1024 tiles)
SIBLING_DEFAULTS = [(112, 32, [((3, 3), 32), ((1, 3), 16)], 41, True), (112, 32, [((3, 3), 32), ((1, 3), 16)], 42, False),
                    (28, 128, [((3, 3), 128), ((1, 1), 32)], 41, True), (28, 128, [((3, 3), 128), ((1, 1), 32)], 70, True),
                    (28, 128, [((3, 3), 128), ((1, 1), 32)], 71, False),
                    (28, 64, [((3, 3), 128), ((1, 1), 32)], 64, True), (23, 256, [((3, 3), 128), ((1, 1), 32)], 62, False),
                    (24, 256, [((3, 3), 128), ((1, 1), 32)], 48, True), (24, 256, [((3, 3), 128), ((1, 1), 32)], 49, False),
                    (17, 192, [((1, 7), 192), ((7, 1), 192), ((1, 1), 192)], 109, True), (17, 192, [((1, 7), 192), ((7, 1), 192), ((1, 1), 192)], 110, False),
                    (28, 256, [((1, 1), 512), ((1, 1), 256)], 52, True), (28, 256, [((1, 1), 512), ((1, 1), 256)], 53, False),
                    (28, 128, [((1, 1), 512), ((1, 1), 64)], 62, True), (28, 128, [((1, 1), 512), ((1, 1), 64)], 63, False),
                    (28, 128, [((3, 3), 72), ((1, 1), 56)], 41, True), (28, 128, [((3, 3), 72), ((1, 1), 56)], 42, False)]


@pytest.mark.parametrize("h, c, branches, b, together", SIBLING_DEFAULTS)
def test_sibling_layers_without_tables(torch, ee, h, c, branches, b, together):
    blob = sibling_net(h, c, branches)
    eng = ee.Engine(blob, b)
    x = torch.randint(-128, 128, (b, h, h, c), dtype=torch.int8, device="cuda")
    n, out = launches_per_layer(torch, eng, blob, x)
    apart, joint = [1] * (1 + len(branches)), [1, 1] + [0] * (len(branches) - 1)
    assert n == (joint if together else apart)
    eng.load_tables({"group": {"1": [0 if together else 0x313]}})
    n, other = launches_per_layer(torch, eng, blob, x)
    assert n == (apart if together else joint)
    assert torch.equal(out, other)
    eng.close()


def test_untuned_fusion_defaults(torch, ee):
    """What the header promises of a context that was never tuned: fused blocks on, but for inverted-residual ones of more than 96 output
    channels, and no fused pairs."""
    for blob, want in ((W.bottleneck_net(8, 8, 256), [1, 0, 0]), (W.inverted_residual_net(8, 8, 16, 48, 96, 1), [1, 0, 0]),
                       (W.inverted_residual_net(8, 8, 16, 48, 112, 1), [1, 1, 1])):
        eng = ee.Engine(blob, 2)
        assert eng.ir_count() > 0
        x = dev(torch, W.input_pool(blob, 2))
        n, _ = launches_per_layer(torch, eng, blob, x)
        assert n == want
        eng.close()
    blob = W.load_net("resnet50_small_i8")
    eng = ee.Engine(blob, 2)
    assert eng.pair_count() > 0
    eng.ir_mode(0)
    eng.load_tables({"group": {str(k): [0] for k in group_heads(ee, eng, len(blob.ops))}})
    n, _ = launches_per_layer(torch, eng, blob, dev(torch, W.input_pool(blob, 2)))
    k = int(blob.stages[0]["n_ops"])
    assert n[:k] == [1] * k
    eng.close()


def group_heads(ee, eng, n_layers):
    """layers that head a joint launch of siblings"""
    heads = []
    for layer in range(n_layers):
        try:
            eng.load_tables({"group": {str(layer): []}})
            heads.append(layer)
        except ee.EEError:
            pass
    return heads


def test_thresholds_zero_and_above_one(torch, ee, orc):
    blob = W.load_net("tiny_i8")
    eng = ee.Engine(blob, 8)
    x = W.input_pool(blob, 8)
    a0 = eng.stage_forward(0, dev(torch, x), blob.stage_out_shape(0))
    assert np.all(eng.exit_head(0, a0, 0.0)[3].cpu().numpy() == 1)       # threshold 0: everyone leaves at exit 1
    assert np.all(eng.exit_head(0, a0, 1.5)[3].cpu().numpy() == 0)       # threshold > 1: nobody leaves early
    a1 = eng.stage_forward(1, a0, blob.stage_out_shape(1))
    a2 = eng.stage_forward(2, a1, blob.stage_out_shape(2))
    assert np.all(eng.exit_head(2, a2, 1.5)[3].cpu().numpy() == 1)       # ... and the last exit takes everybody
    eng.close()


def test_edge_arguments_on_device(torch, ee):
    blob = W.load_net("tiny_i8")
    eng = ee.Engine(blob, 4)
    lib = ee.raw()
    x = dev(torch, W.input_pool(blob, 4))
    out = torch.empty((4,) + blob.stage_out_shape(0), dtype=torch.int8, device="cuda")
    assert lib.ee_stage_forward(eng._h, 0, 0, None, None) == ee.EE_OK           # empty batch is a no-op
    assert lib.ee_stage_forward(eng._h, 0, 5, x.data_ptr(), out.data_ptr()) == ee.EE_ERR_ARG   # above b_max
    assert lib.ee_stage_forward(eng._h, 3, 1, x.data_ptr(), out.data_ptr()) == ee.EE_ERR_ARG   # no such segment
    assert lib.ee_stage_forward(eng._h, 0, 1, x.data_ptr() + 1, out.data_ptr()) == ee.EE_ERR_ARG  # misaligned
    assert lib.ee_stage_forward(eng._h, 0, 1, x.data_ptr(), x.data_ptr()) == ee.EE_ERR_ARG     # aliasing
    assert lib.ee_exit_head(eng._h, 0, 0, None, 0.5, None, None, None, None) == ee.EE_OK
    eng.close()


def test_compaction_and_refill(torch, ee, orc):
    blob = W.load_net("zoo_i8")
    b_max = 24
    eng = ee.Engine(blob, b_max)
    rng = np.random.default_rng(7)
    shape = blob.stage_out_shape(0)
    act = rng.integers(-128, 128, size=(16,) + shape).astype(np.int8)
    refill = rng.integers(-128, 128, size=(5,) + shape).astype(np.int8)
    ids = rng.permutation(1000)[:16].astype(np.int32)
    rids = (2000 + np.arange(5)).astype(np.int32)
    patterns = [np.zeros(16, np.uint8), np.ones(16, np.uint8)] + [rng.integers(0, 2, 16).astype(np.uint8) for _ in range(6)]
    for k, flags in enumerate(patterns):
        for with_refill in (False, True):
            say(f"[case] compaction pattern {k} refill={with_refill}")
            r_act, r_ids = (refill, rids) if with_refill else (None, None)
            ref = orc.compact_refill(flags, act, ids, r_act, r_ids)
            got = eng.compact_refill(0, dev(torch, flags), dev(torch, act), dev(torch, ids),
                                     None if r_act is None else dev(torch, r_act), None if r_ids is None else dev(torch, r_ids))
            assert got[2] == ref[2] and got[3] == ref[3]
            assert np.array_equal(got[0].cpu().numpy(), ref[0]) and np.array_equal(got[1].cpu().numpy(), ref[1])
    eng.close()


def test_steps_captured_in_a_graph(torch, ee):
    """Segment, exit head without allocations, compaction and an empty compaction captured once: every replay, with eager work and other inputs
    in between, gives what eager calls give."""
    blob = W.load_net("zoo_i8")
    lib, b, s = ee.raw(), 6, torch.cuda.Stream()
    with torch.cuda.stream(s):
        eng = ee.Engine(blob, b)
        shape, thr = blob.stage_out_shape(0), float(blob.exits[0]["thr"])
        x = dev(torch, W.input_pool(blob, b))
        act, dst = (torch.zeros((b,) + shape, dtype=torch.int8, device="cuda") for _ in range(2))
        label, conf = torch.zeros(b, dtype=torch.int32, device="cuda"), torch.zeros(b, dtype=torch.float32, device="cuda")
        score, flag = torch.zeros(b, dtype=torch.int64, device="cuda"), torch.zeros(b, dtype=torch.uint8, device="cuda")
        ids, ids_dst = torch.arange(b, dtype=torch.int32, device="cuda"), torch.zeros(b, dtype=torch.int32, device="cuda")
        counts = torch.zeros(4, dtype=torch.int32, device="cuda")

        def steps():
            assert lib.ee_stage_forward(eng._h, 0, b, x.data_ptr(), act.data_ptr()) == ee.EE_OK
            eng.exit_head_static(0, act, thr, label, conf, score, flag)
            p = counts.data_ptr()
            assert lib.ee_compact_refill(eng._h, 0, b, flag.data_ptr(), act.data_ptr(), dst.data_ptr(), ids.data_ptr(), ids_dst.data_ptr(),
                                         None, None, 0, p, p + 4) == ee.EE_OK
            assert lib.ee_compact_refill(eng._h, 0, 0, None, None, None, None, None, None, None, 0, p + 8, p + 12) == ee.EE_OK

        outs = (act, dst, label, conf, score, flag, ids_dst, counts)

        def cleared(run):
            for t in outs:
                t.fill_(3)
            run()
            s.synchronize()
            return [t.clone() for t in outs]

        cleared(steps)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            steps()
        for k in range(4):
            x.copy_(dev(torch, W.input_pool(blob, b, first=b * k)))
            want = cleared(steps)
            got = cleared(graph.replay)
            assert want[-1].tolist()[2:] == [0, 0] and 0 <= want[-1][0] <= b
            assert all(torch.equal(g, w) for g, w in zip(got, want)), f"replay {k}"
        del graph
        eng.close()


def synthetic_lut(n_stages, b_max):
    return (np.arange(1, n_stages + 1)[:, None] * 1000 + np.arange(b_max)[None, :] * 37).astype(np.int64)


SERVE_CASES = [  # name, n, b_max, arrival gap ns, slo, min_incr, refill
    ("tiny_i8", 64, 8, 0, -1, 1, 1),            # configuration 1: 64 requests, 8 slots, all at t = 0
    ("tiny_i8", 64, 8, 450, 9000, 1, 1),
    ("tiny_i8", 50, 5, 300, -1, 2, 1),
    ("tiny_i8", 40, 8, 0, -1, 1, 0),
    ("zoo_i8", 48, 8, 700, -1, 1, 1),
    ("resnet50_small_i8", 40, 8, 900, 30000, 1, 1),
    ("mobilenetv2_small_i8", 32, 8, 600, -1, 1, 1),
    ("tiny_i8", 64, 8, 0, -1, 1, 2),            # stage pools: full batches from the pools in front of the segments
    ("tiny_i8", 64, 8, 450, 9000, 1, 2),
    ("tiny_i8", 50, 5, 300, -1, 1, 2),
    ("zoo_i8", 48, 8, 700, 12000, 1, 2),
    ("resnet50_small_i8", 60, 8, 200, -1, 1, 2),
    ("mobilenetv2_small_i8", 40, 8, 100, -1, 1, 2),
    ("inception_small_i8", 40, 8, 300, -1, 1, 2),
    ("inception_small_i8", 32, 8, 0, -1, 1, 1),
]


@pytest.mark.parametrize("case", SERVE_CASES)
def test_serve_stream_virtual_clock_matches_oracle(torch, ee, orc, case):
    name, n, b_max, gap, slo, min_incr, refill = case
    say(f"[case] serve {case}")
    blob = W.load_net(name)
    pool = W.input_pool(blob, n)
    arrivals = (np.arange(n) * gap).astype(np.int64)
    lut = synthetic_lut(blob.n_stages, b_max)
    ref, rst, rev = orc.serve_stream(blob, arrivals, pool, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill, max_events=5000)
    eng = ee.Engine(blob, b_max)
    got, gst, gev = eng.serve_stream(arrivals, dev(torch, pool), lut, clock=1, t_slo_ns=slo, min_incr=min_incr, refill=refill, max_events=5000)
    for f in ("exit_idx", "label", "score", "latency_ns"):
        assert np.array_equal(got[f], ref[f]), f
    assert np.allclose(got["conf"], ref["conf"], rtol=1e-6)
    assert gst == rst
    assert np.array_equal(gev, rev)
    counts = np.bincount(got["exit_idx"], minlength=blob.n_stages)
    assert counts.sum() == n                                              # everyone leaves exactly once
    eng.close()


def test_serve_stream_wall_clock_invariants(torch, ee, orc):
    blob = W.load_net("tiny_i8")
    n, b_max = 64, 8
    pool = W.input_pool(blob, n)
    alone = orc.forward_alone(blob, pool)
    eng = ee.Engine(blob, b_max)
    lut = eng.measure_lut(reps=2)
    assert lut.shape == (3, b_max) and np.all(lut > 0)
    arrivals = (np.arange(n) * 20000).astype(np.int64)
    got, st, _ = eng.serve_stream(arrivals, dev(torch, pool), lut, clock=0)
    for f in ("exit_idx", "label", "score"):
        assert np.array_equal(got[f], alone[f]), f                       # schedule independence
    assert np.all(got["latency_ns"] > 0)
    assert st["seg_samples"][0] == n
    eng.close()


# ---- several steps in flight, and the baseline policies, on the GPU ---------------------------------------------
LANE_CASES = [  # name, n, b_max, arrival gap ns, slo, refill, lanes, t_timeout
    ("tiny_i8", 64, 8, 0, -1, 2, 2, 0),
    ("tiny_i8", 96, 8, 150, -1, 2, 3, 0),
    ("tiny_i8", 64, 8, 450, 9000, 2, 2, 0),
    ("zoo_i8", 64, 8, 100, -1, 2, 2, 0),
    ("resnet50_small_i8", 96, 8, 60, -1, 2, 2, 0),
    ("resnet50_small_i8", 96, 8, 0, -1, 2, 4, 0),
    ("mobilenetv2_small_i8", 64, 8, 50, -1, 2, 3, 0),
    ("inception_small_i8", 48, 8, 100, -1, 2, 2, 0),
    ("tiny_i8", 40, 8, 900, -1, 0, 1, 3000),       # adaptive batching <8, 3000 ns>
    ("zoo_i8", 40, 8, 400, -1, 0, 1, 100000),      # a window that always fills the batch
    ("tiny_i8", 24, 1, 500, -1, 0, 1, 0),          # SERIAL
]


@pytest.mark.parametrize("case", LANE_CASES)
def test_serve_stream_lanes_and_baselines_match_oracle(torch, ee, orc, case):
    name, n, b_max, gap, slo, refill, lanes, window = case
    say(f"[case] serve {case}")
    blob = W.load_net(name)
    pool = W.input_pool(blob, n)
    arrivals = (np.arange(n) * gap).astype(np.int64)
    lut = synthetic_lut(blob.n_stages, b_max)
    ref, rst, rev = orc.serve_stream(blob, arrivals, pool, b_max, lut, t_slo_ns=slo, refill=refill, lanes=lanes, t_timeout_ns=window, max_events=5000)
    eng = ee.Engine(blob, b_max)
    assert eng.set_lanes(lanes) == lanes
    dpool = dev(torch, pool)
    for rep in range(2):                                                   # the rings and lanes are reused by the second call
        got, gst, gev = eng.serve_stream(arrivals, dpool, lut, clock=1, t_slo_ns=slo, refill=refill, lanes=lanes, t_timeout_ns=window, max_events=5000)
        for f in ("exit_idx", "label", "score", "latency_ns"):
            assert np.array_equal(got[f], ref[f]), (f, rep)
        assert gst == rst and np.array_equal(gev, rev)
    if lanes > 1:
        assert np.any(gev["aux"][gev["kind"] == 2] > 0)                    # the other lanes did run steps
        with pytest.raises(ee.EEError):
            eng.serve_stream(arrivals, dpool, lut, clock=1, refill=2, lanes=lanes + 1)   # more lanes than ee_lanes made
    eng.close()


ZC_CASES = [  # name, n, b_max, arrival gap ns, slo, min_incr, refill, lanes
    ("tiny_i8", 64, 8, 0, -1, 1, 1, 1),              # Algorithm 1: parked survivors, catch-up batches merged behind them
    ("tiny_i8", 64, 8, 450, 9000, 1, 1, 1),
    ("tiny_i8", 50, 5, 300, -1, 2, 1, 1),
    ("tiny_i8", 40, 8, 0, -1, 1, 0, 1),              # model-level batching
    ("resnet50_small_i8", 40, 8, 900, 30000, 1, 1, 1),
    ("resnet50_small_i8", 60, 8, 200, -1, 1, 2, 1),  # stage pools, one lane
    ("resnet50_small_i8", 96, 8, 60, -1, 1, 2, 2),   # stage pools, two steps in flight
    ("resnet18_small_i8", 64, 8, 100, -1, 1, 2, 2),
    ("tiny_i8", 64, 8, 0, -1, 1, 2, 2),
]


@pytest.mark.parametrize("case", ZC_CASES)
def test_serve_stream_zero_copy_matches_oracle_and_copying(torch, ee, orc, case):
    """Zero-copy compaction (survivors stay where the segment wrote them, the next segment gathers them through a slot
    table): results, statistics and the whole event list equal the oracle's on the virtual clock, as with the copying kernel."""
    name, n, b_max, gap, slo, min_incr, refill, lanes = case
    say(f"[case] zero-copy serve {case}")
    blob = W.load_net(name)
    pool = W.input_pool(blob, n)
    arrivals = (np.arange(n) * gap).astype(np.int64)
    lut = synthetic_lut(blob.n_stages, b_max)
    ref, rst, rev = orc.serve_stream(blob, arrivals, pool, b_max, lut, t_slo_ns=slo, min_incr=min_incr, refill=refill, lanes=lanes, max_events=5000)
    eng = ee.Engine(blob, b_max)
    assert eng.zero_copy_supported()
    assert eng.set_lanes(lanes) == lanes
    dpool = dev(torch, pool)
    for zc in (1, 0, 1):                                                   # the slots are reused by later calls
        got, gst, gev = eng.serve_stream(arrivals, dpool, lut, clock=1, t_slo_ns=slo, min_incr=min_incr, refill=refill, lanes=lanes, max_events=5000, zero_copy=zc)
        for f in ("exit_idx", "label", "score", "latency_ns"):
            assert np.array_equal(got[f], ref[f]), (f, zc)
        assert gst == rst and np.array_equal(gev, rev)
    eng.close()


STEM_CASES = [(224, 224, 5), (57, 80, 7), (32, 32, 7), (17, 16, 3), (7, 16, 2), (114, 56, 9), (9, 48, 4)]      # h, w, samples (h * w a multiple of 16: whole 16-byte chunks per input sample)


@pytest.mark.parametrize("case", STEM_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_first_convolution_and_pool_equal_separate_layers_and_oracle(torch, ee, orc, case):
    """7x7 / 2 convolution and 3x3 / 2 max-pool as one launch: images whose pooled size is and is not whole tiles of 14 x 4, odd
    sizes (the last pooled row or column sees one convolution row or column only), a pooled image smaller than a tile, extreme
    inputs; against the oracle and against the two separate layers, bit for bit."""
    h, w, n = case
    blob = W.stem_net(h, w, seed=h + w)
    say(f"[case] first convolution + pool on {h}x{w}, {n} samples")
    r = np.random.default_rng(h * 100 + w)
    x = np.concatenate([np.full((1, h, w, 3), -128, np.int8), np.full((1, h, w, 3), 127, np.int8),
                        r.integers(-128, 128, size=(max(n - 2, 1), h, w, 3), dtype=np.int8)])[:n]
    eng = ee.Engine(blob, max(n, 2))
    assert eng.ir_count() == 1 and eng.ir_layers(0) == 2
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        for mode in (2, 0, 2):
            eng.ir_mode(mode)
            got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"mode {mode} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
    assert np.unique(ref).size > 8
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("h, w", [(48, 32), (33, 80), (16, 34)], ids=str)
def test_first_layer_and_pool_straight_from_the_requests(torch, ee, orc, h, w, dtype):
    """Rows of whole 16-byte chunks are read by the first layer's own launch, with no folded copy in front: requests of a stream by ids that travel as 64 and as 256 of the arguments or stay in host memory,
    steps on the caller's tensor; other rows through the folded copy.  Every request's outcome is that of a step, int8 with the layers one by one (bf16, where the launches round alike
    but may add in another order: of the same launch), and the int8 step's output is the oracle's."""
    blob = W.stem_net(h, w, seed=h, dtype=W.DT_I8 if dtype == "i8" else W.DT_BF16)
    n, kernel = 700, f"stem_pool_{dtype}_kernel"
    x = np.random.default_rng(w).integers(-128, 128, size=(n, h, w, 3), dtype=np.int8) if dtype == "i8" else W.input_pool(blob, n)
    eng = ee.Engine(blob, 300)
    assert eng.ir_count() == 1
    pool, shape = dev(torch, x), blob.stage_out_shape(0)
    eng.ir_mode(0 if dtype == "i8" else 2)
    want = [eng.exit_head(0, eng.stage_forward(0, pool[k:k + 100], shape), 0.5) for k in range(0, n, 100)]
    want_label, want_conf, want_score = (np.concatenate([v[i].cpu().numpy() for v in want]) for i in (0, 1, 2))
    assert np.unique(want_conf).size > 100
    eng.ir_mode(2)
    direct = w % 16 == 0
    for b_max in (7, 64, 65, 256, 257, 300):
        say(f"[case] first layer from the requests {h}x{w} b_max={b_max}")
        lut = synthetic_lut(blob.n_stages, b_max)
        got, names = kernels_of(torch, lambda: eng.serve_stream(np.zeros(n, np.int64), pool, lut, b_max=b_max, refill=0)[0])
        assert np.array_equal(got["label"], want_label) and np.array_equal(got["score"], want_score) and np.array_equal(got["conf"], want_conf)
        assert any(k.startswith(kernel) for k in names) and any(k.startswith("space_to_depth") for k in names) != direct, names
    ref = orc.stage_forward(blob, 0, x[:3])
    got, names = kernels_of(torch, lambda: host(eng.stage_forward(0, pool[:3], shape), ref))
    assert (dtype != "i8" or np.array_equal(got, ref)) and any(k.startswith("space_to_depth") for k in names) != direct, names
    eng.close()


@pytest.mark.parametrize("case", [(1, 16, 16, 1, 9), (33, 48, 32, 1, 40), (16, 299, 32, 0, 3), (61, 80, 48, 0, 70), (38, 160, 64, 1, 130), (224, 224, 32, 1, 19), (125, 64, 32, 0, 300)], ids=lambda c: "x".join(map(str, c)))
def test_folded_first_layer_straight_from_the_requests(torch, ee, orc, case):
    """3x3 / 2 first layers (2 x 2 taps once folded) that read the images themselves: one output row, rows of any alignment, 16 to 64 channels, padding and none, bands of one to eight output rows that end
    with the image and inside it; the step's output against the oracle and the folded copy's, requests of a stream by ids that are 64 and 256 arguments or host memory against their own steps, bit for bit."""
    from workloads import nets as N
    h, w, co, pad, n = case
    net = N._Net(W.DT_I8, h, w, 3, 10)
    t = net.begin_stage()
    t = net.conv(t, co, 3, 2, pad)
    net.end_stage(net.conv(t, 32, 1, 1, 0))
    blob = N._assemble(net, net.dtype, h + w)
    for op in blob.ops:
        op["shift"] = 9
    x = np.random.default_rng(co).integers(-128, 128, size=(n, h, w, 3), dtype=np.int8)
    eng, pool, shape = ee.Engine(blob, n), dev(torch, x), blob.stage_out_shape(0)
    say(f"[case] folded first layer {case}")
    for b in sorted({1, n // 3 + 1, n}):
        got, names = kernels_of(torch, lambda: eng.stage_forward(0, pool[:b], shape))
        ends = sorted({0, b // 2, b - 1})
        ref = orc.stage_forward(blob, 0, x[ends])
        assert np.array_equal(host(got[ends], ref), ref) and np.unique(ref).size > 8
        assert any(k.startswith("conv_stream_image_i8_kernel<") for k in names) and not any(k.startswith("space_to_depth") for k in names), names
        copied, names = forced(ee, 7, lambda: kernels_of(torch, lambda: eng.stage_forward(0, pool[:b], shape)))
        assert any(k.startswith("conv_stream_i8_kernel<2,1,") for k in names) and any(k.startswith("space_to_depth") for k in names) and bool((copied == got).all())
    label, conf, score, _ = (v.cpu().numpy() for v in eng.exit_head(0, got, 0.5))
    for b_max in sorted({min(7, n), min(65, n), n}):
        out = eng.serve_stream(np.zeros(n, np.int64), pool, synthetic_lut(blob.n_stages, b_max), b_max=b_max, refill=0)[0]
        assert np.array_equal(out["label"], label) and np.array_equal(out["score"], score) and np.array_equal(out["conf"], conf)
    eng.close()


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("h, w, k, pad", [(48, 32, 7, 0), (33, 48, 8, 3), (40, 64, 7, 5), (31, 16, 8, 1), (64, 80, 7, 2)])
def test_first_layer_and_pool_from_the_images_with_other_paddings(torch, ee, orc, h, w, k, pad, dtype):
    """The same launch for kernels of 7 and 8 and paddings of 0 to 5 pixels (every alignment of a tile's first byte): against the oracle, int8 bit for bit and with the layers one by one; requests by ids against their steps."""
    from workloads import nets as N
    i8 = dtype == "i8"
    net = N._Net(W.DT_I8 if i8 else W.DT_BF16, h, w, 3, 10)
    t = net.conv(net.begin_stage(), 64, k, 2, pad)
    net.end_stage(net.conv(net.maxpool(t, 3, 2, 1), 32, 1, 1, 0))
    blob = N._assemble(net, net.dtype, h + pad)
    for op in blob.ops:
        op["shift"] = 11 if int(op["c_in"]) == 3 else 10 if int(op["kind"]) == W.OP_CONV else 0
    n = 9
    x = W.input_pool(blob, n)
    eng, ref = ee.Engine(blob, n), orc.stage_forward(blob, 0, x)
    say(f"[case] first layer and pool from the images {dtype} {h}x{w} k{k} p{pad}")
    for b in (n, 1):
        got, names = kernels_of(torch, lambda: eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]))
        assert any(q.startswith(f"stem_pool_{dtype}_kernel") for q in names) and not any(q.startswith("space_to_depth") for q in names), names
        if i8:
            assert np.array_equal(host(got, ref), ref[:b]) and np.unique(ref).size > 8
        else:
            r, g = bf16_to_f32(ref[:b]).astype(np.float64), bf16_to_f32(host(got, ref)).astype(np.float64)
            assert np.all(np.abs(g - r) <= 2e-2 * np.abs(r).reshape(b, -1).max(axis=1).reshape(-1, 1, 1, 1))
    act = eng.stage_forward(0, dev(torch, x), ref.shape[1:])
    label, conf, score, _ = (v.cpu().numpy() for v in eng.exit_head(0, act, 0.5))
    got = eng.serve_stream(np.zeros(n, np.int64), dev(torch, x), synthetic_lut(1, 4), b_max=4, refill=0)[0]
    assert np.array_equal(got["label"], label) and np.array_equal(got["score"], score) and np.array_equal(got["conf"], conf)
    if i8:
        eng.ir_mode(0)
        assert np.array_equal(host(eng.stage_forward(0, dev(torch, x), ref.shape[1:]), ref), ref)
    eng.close()


def test_tables_of_a_first_layer_that_reads_the_images(torch, ee):
    """Without a table, with the tuner's and with stored entries of the streaming kernel it is one launch, in a segment and timed by itself; a stored entry of another kernel is that kernel, behind the folded copy, and so is the
    launch with no fused launches: the same bytes, admitted or not."""
    from workloads import nets as N
    net = N._Net(W.DT_I8, 96, 64, 3, 10)
    t = net.conv(net.begin_stage(), 32, 3, 2, 1)
    net.end_stage(net.conv(t, 64, 1, 1, 0))
    blob = N._assemble(net, net.dtype, 4)
    for op in blob.ops:
        op["shift"] = 9
    x, shape = dev(torch, W.input_pool(blob, 8)), blob.stage_out_shape(0)
    eng = ee.Engine(blob, 8)

    def first(f):
        out, names = kernels_of(torch, f)
        return out, [re.sub("_rows.*|_kernel.*", "", k) for k in names if k.startswith(("space_to_depth", "conv_stream", "conv_igemm_kernel<1,64,64,128"))]

    want = eng.stage_forward(0, x, shape)
    eng.autotune(reps=1)
    assert eng.config_table(0) == [7] * 4
    image, copy = ["conv_stream_image_i8"], ["space_to_depth"]
    for mode, word, names in ((1, 7, image), (1, 0, image), (1, 0x223, copy + ["conv_igemm"]), (0, 0x223, copy + ["conv_igemm"]), (0, 7, copy + ["conv_stream_i8"])):
        say(f"[case] first layer's table {mode} {word:#x}")
        eng.ir_mode(mode)
        eng.load_tables({"config": {"0": [word] * 4}})
        got, ran = first(lambda: eng.stage_forward(0, x, shape))
        assert ran == names and torch.equal(got, want), ran
        assert set(first(lambda: eng.time_layer(0, 8, reps=2))[1]) == set(names)
        out = eng.serve_stream(np.zeros(8, np.int64), x, synthetic_lut(1, 8), b_max=8, refill=0)[0]
        assert np.array_equal(out["score"], eng.exit_head(0, want, 0.5)[2].cpu().numpy())
    eng.ir_mode(1)
    assert set(first(lambda: eng.time_layer(0, 8, cfg=7, reps=2))[1]) == set(copy + ["conv_stream_i8"])
    eng.close()


@pytest.mark.parametrize("stem", [True, False], ids=["pool", "layer"])
def test_who_folds_is_decided_once(torch, ee, stem):
    """Admission leaves the requests to the first layer's launch or folds them for it; the segment does as admission did also when another thread forces a tile (process-wide) between the two: every request keeps its outcome."""
    from workloads import nets as N
    if stem:
        blob = W.stem_net(96, 64, seed=4)
    else:
        net = N._Net(W.DT_I8, 96, 64, 3, 10)
        t = net.conv(net.begin_stage(), 32, 3, 2, 1)
        net.end_stage(net.conv(t, 32, 1, 1, 0))
        blob = N._assemble(net, net.dtype, 4)
        for op in blob.ops:
            op["shift"] = 9
    n = 4000
    pool = dev(torch, np.random.default_rng(3).integers(-128, 128, size=(n, 96, 64, 3), dtype=np.int8))
    eng, lut = ee.Engine(blob, 2), synthetic_lut(blob.n_stages, 2)
    want = eng.serve_stream(np.zeros(n, np.int64), pool, lut, b_max=2, refill=0)[0]
    names = kernels_of(torch, lambda: eng.serve_stream(np.zeros(8, np.int64), pool, lut, b_max=2, refill=0))[1]
    assert np.unique(want["conf"]).size > 100 and any(k.startswith("stem_pool_i8" if stem else "conv_stream_image_i8") for k in names) and not any(k.startswith("space_to_depth") for k in names), names
    stop, old, turns = threading.Event(), ee.tune_conv_tile(0), [0]

    def force():
        while not stop.is_set():
            turns[0] += 1
            ee.tune_conv_tile(3 * (turns[0] & 1))

    thread = threading.Thread(target=force)
    thread.start()
    try:
        for k in range(5):
            say(f"[case] who folds {stem} pass {k}")
            got = eng.serve_stream(np.zeros(n, np.int64), pool, lut, b_max=2, refill=0)[0]
            assert all(np.array_equal(got[f], want[f]) for f in ("label", "score", "conf")), f"{np.count_nonzero(got['score'] != want['score'])} of {n} differ"
    finally:
        stop.set()
        thread.join()
        ee.tune_conv_tile(old)
        eng.close()
    assert turns[0] > 100


SB_CASES = [(224, 224, 5), (57, 80, 7), (32, 32, 9), (17, 16, 3), (7, 16, 2), (116, 60, 9)]      # pooled 56 x 56, 15 x 20, 8 x 8, 5 x 4, 2 x 4, 29 x 15: whole tiles of 7 x 8 and not


@pytest.mark.parametrize("case", SB_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_first_convolution_and_pool_bf16(torch, ee, orc, case):
    """The bf16 form of the launch above, on inputs of both signs and with whole images of zeros and of large values.  The sums run in the
    staged kernel's order and every value is rounded where the layers round it, so fused and separate layers agree exactly; the
    oracle adds in double: every value within one bf16 rounding (2^-8 of it) plus the pool's layer behind it."""
    h, w, n = case
    blob = W.stem_net(h, w, seed=h + w, dtype=W.DT_BF16)
    say(f"[case] bf16 first convolution + pool on {h}x{w}, {n} samples")
    x = W.input_pool(blob, n)
    x[0] = 0
    if n > 2:
        x[2] = np.where(x[2] >> 15, 0xC380, 0x4380)                        # -256, 256
    eng = ee.Engine(blob, n)
    assert eng.ir_count() == 1 and eng.ir_layers(0) == 2
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        out = []
        for mode in (2, 0, 2):
            eng.ir_mode(mode)
            out.append(bf16_to_f32(host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)).astype(np.float64))
        assert np.array_equal(out[0], out[2]) and np.array_equal(out[0], out[1]), f"b={b}: {np.count_nonzero(out[0] != out[1])} of {ref.size} differ"
        r = bf16_to_f32(ref).astype(np.float64)
        for k in range(b):
            assert np.abs(out[0][k] - r[k]).max() <= 2.0 ** -7 * max(np.abs(r[k]).max(), 1e-30), f"sample {k}: {np.abs(out[0][k] - r[k]).max()} of {np.abs(r[k]).max()}"
    eng.close()


CP_CASES = [(16, 14, 1, 1, 3), (17, 33, 0, 0, 5), (5, 5, 0, 0, 2), (30, 29, 1, 0, 4), (5, 47, 0, 1, 3), (149, 149, 1, 0, 9)]      # h, w, padding of the convolution, of the pool, samples


@pytest.mark.parametrize("case", CP_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_convolution_over_32_channels_and_pool(torch, ee, orc, case):
    """3x3 convolution 32 -> 64 and 3x3 / 2 max-pool as one launch: paddings of both, pooled images of whole tiles of 7 x 8, less and more,
    one pixel, extreme inputs, outputs of both signs; against the oracle and the two separate layers, bit for bit."""
    from workloads import nets as N
    h, w, pad, pool_pad, n = case
    net = N._Net(W.DT_I8, h, w, 32, 10)
    t = net.begin_stage()
    t = net.conv(t, 64, 3, 1, pad, act="linear" if h % 2 else "relu")
    t = net.maxpool(t, 3, 2, pool_pad)
    net.end_stage(net.conv(t, 32, 1, 1, 0))
    blob = N._assemble(net, W.DT_I8, 60 + h)
    for op in blob.ops:
        if int(op["kind"]) == W.OP_CONV:
            op["shift"] = max(0, int(np.ceil(np.log2(2.0 * 74 * 40 * np.sqrt(int(op["c_in"]) * int(op["kh"]) ** 2) / 127))))
    say(f"[case] 3x3 32 -> 64 on {h}x{w}, padding {pad}, pool padding {pool_pad}, {n} samples")
    r = np.random.default_rng(h * 100 + w)
    x = np.concatenate([np.full((1, h, w, 32), -128, np.int8), np.full((1, h, w, 32), 127, np.int8), r.integers(-128, 128, size=(max(n - 2, 1), h, w, 32), dtype=np.int8)])[:n]
    eng = ee.Engine(blob, max(n, 2))
    assert eng.ir_count() == 1 and eng.ir_layers(0) == 2
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        for mode in (2, 0, 1):
            eng.ir_mode(mode)
            got = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
            assert np.array_equal(got, ref), f"mode {mode} b={b}: {np.count_nonzero(got != ref)} of {ref.size} differ, first at {np.argwhere(got != ref)[:3].tolist()}"
    assert np.unique(ref).size > 8
    eng.close()


BN_SERVE_CASES = [  # h, w, c_in, seed, frac_bits, thresholds of the first two exits, lanes
    (12, 10, 64, 3, 11, (0.782, 0.955), 1), (16, 16, 256, 5, 12, (0.8371, 0.8453), 2),
]


@pytest.mark.parametrize("case", BN_SERVE_CASES, ids=lambda c: "x".join(map(str, c[:4])) + f"_lanes{c[6]}")
def test_serve_stream_with_fused_bottleneck_blocks(torch, ee, orc, case):
    """Three segments of two bottleneck blocks each, served with every block fused: the block that ends a segment also pools
    for the exit head and, with zero-copy compaction, writes its samples to their slots.  Results, statistics and events
    equal the oracle's on the virtual clock with the fused blocks, without them, with and without zero-copy compaction."""
    h, w, ci, seed, fb, thr, lanes = case
    blob = W.bottleneck_net(h, w, ci, seed=seed, blocks=2, stages=3)
    for e, t in zip(blob.exits, thr + (0.0,)):
        e["thr"], e["frac_bits"] = t, fb
    n, b_max = 96, 8
    say(f"[case] serve bottleneck net {case}")
    pool = W.input_pool(blob, n)
    arrivals = (np.arange(n) * 150).astype(np.int64)
    lut = synthetic_lut(blob.n_stages, b_max)
    ref, rst, rev = orc.serve_stream(blob, arrivals, pool, b_max, lut, refill=2, lanes=lanes, max_events=5000)
    assert np.all(np.bincount(ref["exit_idx"], minlength=3) > 0)           # every exit is taken
    eng = ee.Engine(blob, b_max)
    assert eng.ir_count() == (7 if ci == 64 else 6) and eng.zero_copy_supported()   # the first block of a later segment reads slots and stays unfused when served zero-copy
    assert eng.set_lanes(lanes) == lanes
    dpool = dev(torch, pool)
    for mode, zc in ((2, 1), (0, 1), (2, 0), (2, 1)):
        eng.ir_mode(mode)
        got, gst, gev = eng.serve_stream(arrivals, dpool, lut, clock=1, refill=2, lanes=lanes, max_events=5000, zero_copy=zc)
        for f in ("exit_idx", "label", "score", "latency_ns"):
            assert np.array_equal(got[f], ref[f]), (f, mode, zc)
        assert gst == rst and np.array_equal(gev, rev)
    serve_scattered_blocks(torch, eng, pool, b_max, lanes, "bneck_block_i8")
    eng.close()


def serve_scattered_blocks(torch, eng, pool, b_max, lanes, kernel):
    """Output slots that are no run: with the blocks fused, one of which ends each of the 73 steps, every request gets what the copying compaction and the layers give it."""
    serve = scattered_stream(torch, eng, pool, 512, b_max)
    eng.ir_mode(0)
    want = serve(0)[0]
    eng.ir_mode(2)
    for n_lanes in sorted({1, lanes}):
        got, names = serve(1, n_lanes)
        assert sum(name.startswith(kernel) for name in names) >= 73
        for f in ("exit_idx", "label", "conf", "score"):
            assert np.array_equal(got[f], want[f]), (f, n_lanes)


@pytest.mark.parametrize("case", BN_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fused_bottleneck_blocks_bf16(torch, ee, orc, case):
    """The bf16 form: every sum runs in the staged kernel's order and every layer's result is rounded where the layer stores it, so fused and
    separate layers agree bit for bit; against the oracle (double sums) under the tolerance of the tiling tests.  Biases that are not zero."""
    h, w, ci, blocks, n = case
    blob = W.bottleneck_net(h, w, ci, seed=h * 7 + w, blocks=blocks, dtype=W.DT_BF16)
    say(f"[case] bf16 bottleneck {h}x{w} {ci} -> 64 -> 64 -> 256, {blocks} block(s), {n} samples")
    r = np.random.default_rng(h * 100 + w)
    for op in blob.ops:
        blob.op_weights(op)[1][:] = r.normal(size=int(op["c_out"])) * 0.3
    x = W.input_pool(blob, n)
    eng = ee.Engine(blob, max(n, 2))
    heads = {i: eng.ir_layers(i) for i in range(len(blob.ops)) if eng.ir_layers(i)}
    assert sorted(heads.values()) == ([3] * blocks + [4] if ci == 64 else [3] * blocks) and eng.ir_count() == len(heads)
    for b in sorted({n, 1}, reverse=True):
        ref = orc.stage_forward(blob, 0, x[:b])
        out = {}
        for mode in (2, 0, 1, 2):
            eng.ir_mode(mode)
            if mode == 1:                                                  # by table: the blocks of three fused, the block of four not
                eng.load_tables({"ir": {str(i): [0 if span == 4 else 1] for i, span in heads.items()}})
            out[mode] = host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)
            assert np.array_equal(out[mode], out[2]), f"mode {mode} b={b}: {np.count_nonzero(out[mode] != out[2])} of {ref.size} differ, first at {np.argwhere(out[mode] != out[2])[:3].tolist()}"
        rf, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(out[2]).astype(np.float64)
        scale = np.abs(rf).reshape(b, -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30
        assert np.all(np.abs(g - rf) <= 2e-2 * scale), f"b={b}: {np.max(np.abs(g - rf) / scale)}"
    eng.close()


@pytest.mark.parametrize("h,w,ci", [(12, 10, 64), (16, 16, 256)])
def test_serve_stream_with_fused_bottleneck_blocks_bf16(torch, ee, orc, h, w, ci):
    """Three segments of two bf16 bottleneck blocks served with every block fused, with and without zero-copy compaction (the block that ends a
    segment writes its samples to their slots), on two lanes: what every request gets is that of the separate layers, bit for bit."""
    blob = W.bottleneck_net(h, w, ci, seed=h, blocks=2, stages=3, dtype=W.DT_BF16)
    n, b_max = 96, 8
    pool = W.input_pool(blob, n)
    act = pool[:24]
    for s in range(2):                                                     # thresholds that split the requests at both exits
        act = orc.stage_forward(blob, s, act)
        blob.exits[s]["thr"] = float(np.median(orc.exit_head(blob, s, act, 0.5)[1]))
    say(f"[case] serve bf16 bottleneck net {h}x{w}x{ci}")
    eng = ee.Engine(blob, b_max)
    assert eng.zero_copy_supported() and eng.set_lanes(2) == 2
    lut = synthetic_lut(blob.n_stages, b_max)
    dpool = dev(torch, pool)
    want = None
    for mode, zc in ((0, 0), (2, 1), (0, 1), (2, 0), (2, 1)):
        eng.ir_mode(mode)
        got = eng.serve_stream(np.zeros(n, np.int64), dpool, lut, refill=2, lanes=2, zero_copy=zc)[0]
        want = got if want is None else want
        for f in ("exit_idx", "label", "conf"):
            assert np.array_equal(got[f], want[f]), (f, mode, zc)
    assert np.all(np.bincount(want["exit_idx"], minlength=3) > 0)
    serve_scattered_blocks(torch, eng, pool, b_max, 2, "bneck_block_bf16")
    eng.close()


def test_zero_copy_is_refused_where_it_cannot_run(torch, ee, orc):
    blob = W.load_net("mobilenetv2_small_i8")                               # depthwise / thin layers at the segment boundaries
    eng = ee.Engine(blob, 8)
    n = 16
    dpool = dev(torch, W.input_pool(blob, n))
    lut = synthetic_lut(blob.n_stages, 8)
    if not eng.zero_copy_supported():
        with pytest.raises(ee.EEError):
            eng.serve_stream(np.zeros(n, np.int64), dpool, lut, clock=1, zero_copy=1)
    eng.close()
    blob = W.load_net("tiny_i8")
    eng = ee.Engine(blob, 8)
    eng.set_lanes(3)
    dpool = dev(torch, W.input_pool(blob, n))
    lut = synthetic_lut(blob.n_stages, 8)
    with pytest.raises(ee.EEError):
        eng.serve_stream(np.zeros(n, np.int64), dpool, lut, clock=1, refill=2, lanes=3, zero_copy=1)    # the slots cover two steps in flight
    with pytest.raises(ee.EEError):
        eng.serve_stream(np.zeros(n, np.int64), dpool, lut, clock=1, zero_copy=2)
    eng.close()


def test_serve_stream_lanes_wall_clock(torch, ee, orc):
    """On the wall clock the schedule is a measurement; the per-request results are not (schedule independence)."""
    blob = W.load_net("resnet50_small_i8")
    n, b_max = 400, 16
    pool = W.input_pool(blob, n)
    alone = orc.forward_alone(blob, pool)
    eng = ee.Engine(blob, b_max)
    eng.set_lanes(3)
    lut = eng.measure_lut(reps=2)
    dpool = dev(torch, pool)
    for lanes, arrivals in ((3, np.zeros(n, np.int64)), (2, (np.arange(n) * 3000).astype(np.int64)), (1, np.zeros(n, np.int64))):
        say(f"[case] wall clock, lanes {lanes}")
        got, st, ev = eng.serve_stream(arrivals, dpool, lut, clock=0, refill=2, lanes=lanes, max_events=20000)
        for f in ("exit_idx", "label", "score"):
            assert np.array_equal(got[f], alone[f]), (f, lanes)
        assert np.all(got["latency_ns"] > 0) and st["seg_samples"][0] == n
        assert set(ev["aux"][ev["kind"] == 2].tolist()) <= set(range(lanes))
    eng.close()


# ---- full-size configurations, in the launch configuration the benchmark uses ------------------------------------
def golden(name):
    """tests/golden/full_size_<net>.txt, written by tests/golden/make_full_size_golden.py from the oracle alone"""
    import os
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", f"full_size_{name}.txt")
    rows = [line.split() for line in open(path) if not line.startswith("#")]
    return (np.array([int(r[1]) for r in rows]), np.array([int(r[2]) for r in rows]), np.array([int(r[3]) for r in rows], np.int64),
            np.array([float(r[4]) for r in rows], np.float32))


FULL = [("resnet18_i8", 512, 32, [(0, 1, 0)]),                                      # static batches of 32: the configuration as stated
        ("resnet50_i8", 512, 64, [(2, 2, 0), (2, 1, 0), (1, 1, 32), (0, 1, 0)]),    # what the benchmark times, then the other policies
        ("mobilenetv2_i8", 512, 64, [(2, 2, 0), (1, 1, 1)]),
        ("resnet50_eq_i8", 256, 64, [(2, 2, 0)]),                                   # exits equidistant in work
        ("inception_i8", 256, 64, [(2, 2, 0)])]                                     # rectangular kernels, concatenation, average pooling


@pytest.mark.parametrize("case", FULL)
def test_full_size_every_request_against_the_oracle(torch, ee, orc, case):
    """Every request of a prefix of the benchmark's own pool, under the policies the benchmark runs, against what the oracle
    computed for it alone (stored by tests/golden/make_full_size_golden.py): exit, label and score, bit for bit."""
    name, n, b_max, policies = case
    blob = W.load_net(name)
    g_exit, g_label, g_score, _ = golden(name)
    assert len(g_exit) >= n
    pool = W.input_pool(blob, n)
    eng = ee.Engine(blob, b_max)
    eng.set_lanes(2)
    eng.autotune(reps=2)                                   # the launch configuration the benchmark times
    lut = synthetic_lut(blob.n_stages, b_max)
    dpool = dev(torch, pool)
    for refill, lanes, min_incr in policies:
        say(f"[case] full-size {name} n={n} b_max={b_max} refill={refill} lanes={lanes} min_incr={min_incr}")
        got, st, _ = eng.serve_stream(np.zeros(n, np.int64), dpool, lut, clock=1, refill=refill, lanes=lanes, min_incr=max(1, min_incr))
        assert np.array_equal(got["exit_idx"], g_exit[:n]) and np.array_equal(got["label"], g_label[:n]) and np.array_equal(got["score"], g_score[:n])
        say(f"[info] {name} exit counts {np.bincount(got['exit_idx'], minlength=blob.n_stages).tolist()} "
            f"mean batch {[round(a / max(b, 1), 1) for a, b in zip(st['seg_samples'], st['seg_runs'])]}")
    # on the wall clock, as the benchmark runs it; then with zero-copy compaction where the network allows it
    for zc in ((0, 1) if eng.zero_copy_supported() else (0,)):
        say(f"[case] full-size {name} wall clock zero_copy={zc}")
        got, st, _ = eng.serve_stream(np.zeros(n, np.int64), dpool, eng.measure_lut(reps=1), clock=0, refill=policies[0][0], lanes=policies[0][1], zero_copy=zc)
        assert np.array_equal(got["exit_idx"], g_exit[:n]) and np.array_equal(got["label"], g_label[:n]) and np.array_equal(got["score"], g_score[:n])
    eng.close()


@pytest.mark.parametrize("name,b_max", [("resnet18_i8", 32), ("resnet50_i8", 64), ("mobilenetv2_i8", 64), ("inception_i8", 64)])
def test_full_size_every_segment_element_by_element(torch, ee, orc, name, b_max):
    """All segments at the full benchmark batch with the autotuned table, no exits taken: sampled slots (first, middle,
    last, and the one before a tile boundary) of every segment's output against the oracle's chain for those samples."""
    blob = W.load_net(name)
    pool = W.input_pool(blob, b_max)
    slots = sorted({0, b_max // 2 - 1, b_max // 2, b_max - 1})
    eng = ee.Engine(blob, b_max)
    eng.autotune(reps=2)
    act, ref = dev(torch, pool), pool[slots]
    for s in range(blob.n_stages):
        say(f"[case] full-size {name} segment {s} at b={b_max}")
        if eng.ir_count():                                 # every inverted-residual block fused, whatever the tuned table says
            eng.ir_mode(2)
            forced = eng.stage_forward(s, act, blob.stage_out_shape(s))
            eng.ir_mode(1)
        act = eng.stage_forward(s, act, blob.stage_out_shape(s))
        if eng.ir_count():
            assert torch.equal(forced, act), f"{name} segment {s}: fused blocks differ from the tuned mix"
        ref = orc.stage_forward(blob, s, ref)
        got = act.cpu().numpy()[slots]
        assert np.array_equal(got, ref), f"{name} segment {s}: {np.count_nonzero(got != ref)} of {ref.size} differ"
        thr = float(blob.exits[s]["thr"])
        lab, conf, score, flag = orc.exit_head(blob, s, ref, thr)
        glab, gconf, gscore, gflag = eng.exit_head(s, act, thr)
        assert np.array_equal(glab.cpu().numpy()[slots], lab) and np.array_equal(gscore.cpu().numpy()[slots], score)
        assert np.array_equal(gflag.cpu().numpy()[slots], flag)
    eng.close()


# ---- fused layer pairs (conv2 -> conv3 of a bottleneck block in one launch) ------------------------------
@pytest.mark.parametrize("case", [("resnet50_i8", 5), ("resnet50_i8", 64), ("resnet50_bf16", 3), ("resnet50_bf16", 40)])
def test_fused_pairs_equal_separate_layers_and_oracle(torch, ee, orc, case):
    """Every segment of the ResNet-50-style network with all pairs fused against the same segment with none fused
    (same arithmetic, so equal bit for bit in both dtypes), at a batch with ragged tiles and at a full one; the
    fused first segment also against the oracle on sampled slots."""
    name, b = case
    say(f"[case] fused pairs {name} b={b}")
    blob = W.load_net(name)
    eng = ee.Engine(blob, b)
    # conv2 -> conv3 of the 3 + 4 + 6 blocks with up to 256 mid channels; in bf16 the 256-channel pairs do not fit LDS
    assert eng.pair_count() == (13 if blob.dtype == W.DT_I8 else 7)
    pool = W.input_pool(blob, b)
    act = dev(torch, pool)
    for s in range(blob.n_stages):
        say(f"[case] fused pairs {name} b={b} segment {s}")
        eng.pair_mode(0)
        ref = eng.stage_forward(s, act, blob.stage_out_shape(s))
        eng.pair_mode(2)
        got = eng.stage_forward(s, act, blob.stage_out_shape(s))
        assert torch.equal(got, ref), f"segment {s}"
        if s == 0:
            slots = sorted({0, b // 2, b - 1})
            want = orc.stage_forward(blob, 0, pool[slots])
            if blob.dtype == W.DT_I8:
                assert np.array_equal(host(got, want)[slots], want)
            else:
                r, g = bf16_to_f32(want).astype(np.float64), bf16_to_f32(host(got, want)[slots]).astype(np.float64)
                assert np.abs(g - r).max() <= 2e-2 * np.abs(r).max()
        act = ref
    eng.close()


# ---- bf16 ---------------------------------------------------------------------------------------------
def bf16_to_f32(a):
    return W.bf16_bits_to_f32(a)


def test_full_size_bf16_against_the_oracle(torch, ee, orc):
    """The ResNet-50-style bf16 network at its benchmark configuration (256 slots, autotuned kernel table, stage pools on
    two lanes, then Algorithm 1): the first 64 requests against what the oracle computed for each alone (stored by
    tests/golden/make_full_size_golden.py), under the tolerances for bf16; then every segment at the full batch element
    by element on sampled slots."""
    name, n, b_max = "resnet50_bf16", 320, 256
    say(f"[case] full-size {name} n={n} b_max={b_max}")
    blob = W.load_net(name)
    g_exit, g_label, _, g_conf = golden(name)
    m = len(g_exit)
    assert m >= 32
    pool = W.input_pool(blob, n)
    eng = ee.Engine(blob, b_max)
    eng.set_lanes(2)
    eng.autotune(reps=2)
    lut = synthetic_lut(blob.n_stages, b_max)
    thr = np.array([float(e["thr"]) for e in blob.exits], np.float32)
    for refill, lanes in ((2, 2), (1, 1)):
        got, st, _ = eng.serve_stream(np.zeros(n, np.int64), dev(torch, pool), lut, clock=1, refill=refill, lanes=lanes, min_incr=b_max // 2)
        assert np.bincount(got["exit_idx"], minlength=blob.n_stages).sum() == n and np.all(got["exit_idx"] >= 0)
        same = got["exit_idx"][:m] == g_exit
        # where the exits agree the confidences must: both sides computed the same head on the same path
        assert np.all(np.abs(got["conf"][:m][same] - g_conf[same]) <= 1e-3)
        # where they differ the library's confidence at the earlier of the two exits must sit within the tolerance of that
        # exit's threshold (the decision there was a toss-up); request by request through the oracle
        for sid in np.nonzero(~same)[0]:
            act, cleared = pool[sid:sid + 1], False
            for s_ in range(min(int(got["exit_idx"][sid]), int(g_exit[sid])) + 1):
                act = orc.stage_forward(blob, s_, act)
                _, conf, _, _ = orc.exit_head(blob, s_, act, float(thr[s_]))
                cleared = cleared or abs(float(conf[0]) - float(thr[s_])) < 1e-3
            assert cleared, f"request {sid}: exit {got['exit_idx'][sid]} vs oracle {g_exit[sid]} with no confidence near a threshold"
        say(f"[info] bf16 refill={refill}: {int(np.count_nonzero(~same))} of {m} requests sit within 1e-3 of a threshold")
        assert np.count_nonzero(~same) <= m // 8
    # every segment at the full batch, element by element on sampled slots
    slots = [0, 131, b_max - 1]
    act, ref = dev(torch, pool[:b_max]), pool[:b_max][slots]
    for s_ in range(blob.n_stages):
        say(f"[case] full-size bf16 segment {s_} at b=256")
        act = eng.stage_forward(s_, act, blob.stage_out_shape(s_))
        ref_next = orc.stage_forward(blob, s_, ref)
        r, g = bf16_to_f32(ref_next).astype(np.float64), bf16_to_f32(host(act, ref_next)[slots]).astype(np.float64)
        scale = np.abs(r).reshape(r.shape[0], -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30
        assert np.all(np.abs(g - r) <= 2e-2 * scale), f"segment {s_}: {np.max(np.abs(g - r) / scale)}"
        ref = ref_next
    eng.close()


@pytest.mark.parametrize("name", ["tiny_bf16", "zoo_bf16", "resnet50_small_bf16", "inception_small_bf16", "resnet50_bf16"])
def test_tunings_of_a_bf16_network_agree(torch, ee, name):
    """Contexts tuned apart, one of them for other batches, return the same bits at every batch size: the shapes alone decide in which order a tuned layer adds."""
    blob = W.load_net(name)
    engines = [ee.Engine(blob, b_max) for b_max in (256, 256, 40)]
    for reps, eng in enumerate(engines, 1):
        eng.autotune(reps=reps)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((256,) + tuple(blob.in_shape()), device="cuda", generator=gen).to(torch.bfloat16).view(torch.int16)
    for b in (1, 5, 40, 256):
        say(f"[case] tunings {name} b={b}")
        first = None
        for k, eng in enumerate(engines[:2 if b > 40 else 3]):
            act, out = x[:b], []
            for s in range(blob.n_stages):
                act = eng.stage_forward(s, act, blob.stage_out_shape(s))
                out += [act, *eng.exit_head(s, act, float(blob.exits[s]["thr"]))]
            first = first or out
            assert all(torch.equal(g, w) for g, w in zip(out, first)), f"tuning {k}: outputs {[i for i, (g, w) in enumerate(zip(out, first)) if not torch.equal(g, w)]} differ"
    for eng in engines:
        eng.close()


@pytest.mark.parametrize("name", ["tiny_bf16", "zoo_bf16", "resnet50_small_bf16", "inception_small_bf16"])
def test_bf16_within_tolerance(torch, ee, orc, name):
    blob = W.load_net(name)
    eng = ee.Engine(blob, 16)
    x = W.input_pool(blob, 12)
    for tile in (0, 1, 2, 3, 4, 0x0321, 0x0432, 0x10321, 0x10332, 0x10423, 0x10234):     # tiles, pipelined steps, the slab kernel
        ee.tune_conv_tile(tile)
        act = x
        for s in range(blob.n_stages):
            say(f"[case] {name} tile {tile:#x} segment {s}")
            ref = orc.stage_forward(blob, s, act)
            got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
            r, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(got).astype(np.float64)
            scale = np.abs(r).reshape(r.shape[0], -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30
            assert np.all(np.abs(g - r) <= 2e-2 * scale), f"stage {s}: {np.max(np.abs(g - r) / scale)}"
            thr = float(blob.exits[s]["thr"])
            lab, conf, _, flag, logits = orc.exit_head(blob, s, ref, thr, want_logits=True)
            glab, gconf, _, gflag = eng.exit_head(s, dev(torch, ref), thr)
            glog = eng.last_logits(ref.shape[0], logits.shape[1])
            zmax = np.abs(logits).max(axis=1, keepdims=True)
            assert np.all(np.abs(glog - logits) <= 2e-2 * zmax)
            assert np.all(np.abs(gconf.cpu().numpy() - conf) <= 1e-3)
            clear = np.abs(conf - np.float32(thr)) >= 1e-3
            assert np.array_equal(gflag.cpu().numpy()[clear], flag[clear])
            top2 = np.sort(logits, axis=1)[:, -2:]
            sure = (top2[:, 1] - top2[:, 0]) > 4e-2 * zmax[:, 0]
            assert np.array_equal(glab.cpu().numpy()[sure], lab[sure])
            act = ref
    ee.tune_conv_tile(0)
    eng.close()


# h, w, c_in, kernel, stride, padding, c_out: reductions shorter than the 16 wavefronts and long ones, steps that do not fill the last group of
# loads, channels that fill no block of 32 or 64, taps outside the image, strides
FEW_PIXEL_BF16 = [(7, 7, 512, 3, 1, 1, 72), (5, 6, 24, 1, 1, 0, 40), (9, 9, 8, 5, 2, 2, 16), (14, 14, 64, 1, 2, 0, 136), (6, 4, 40, 3, 1, 0, 8)]


@pytest.mark.parametrize("cfg", SKINNY)
def test_few_pixel_convolution_bf16(torch, ee, orc, cfg):
    """The few-pixel kernel forced on bf16 layers.  One layer against the oracle (double sums, rounded to bf16): the K products of a sum are exact
    in float, every addition of any order errs by at most 2^-23 of the sum of their magnitudes, and the two roundings to bf16 by at
    most 2^-8 of the value each.  Then whole networks (slices, residuals, rectangular kernels) under the tolerance of the tiling tests."""
    old = ee.tune_conv_tile(cfg)
    try:
        for h, w, c, k, stride, pad, co in FEW_PIXEL_BF16:
            blob = W.single_layer_net("conv", h, w, c, k, stride, pad, W.DT_BF16, seed=co, co=co)
            mag = W.Blob(blob.tobytes())
            mag.op_weights(mag.ops[0])[0][:] &= 0x7FFF
            eng = ee.Engine(blob, 3)
            x = W.input_pool(blob, 3)
            for b in (3, 1):
                say(f"[case] cfg {cfg:#x} {h}x{w}x{c} k{k} s{stride} p{pad} -> {co} b={b}")
                ref = orc.stage_forward(blob, 0, x[:b])
                total = bf16_to_f32(orc.stage_forward(mag, 0, x[:b] & 0x7FFF)).astype(np.float64) * (1 + 2.0 ** -8)
                got = bf16_to_f32(host(eng.stage_forward(0, dev(torch, x[:b]), ref.shape[1:]), ref)).astype(np.float64)
                r = bf16_to_f32(ref).astype(np.float64)
                bound = 2 * 2.0 ** -8 * np.maximum(np.abs(r), np.abs(got)) + k * k * c * 2.0 ** -23 * total
                assert np.all(np.abs(got - r) <= bound), f"{np.max(np.abs(got - r) / bound)} of the bound"
            eng.close()
        for name in ("zoo_bf16", "resnet50_small_bf16", "inception_small_bf16"):
            blob = W.load_net(name)
            eng = ee.Engine(blob, 4)
            act = W.input_pool(blob, 3)
            for s in range(blob.n_stages):
                say(f"[case] cfg {cfg:#x} {name} segment {s}")
                ref = orc.stage_forward(blob, s, act)
                got = host(eng.stage_forward(s, dev(torch, act), ref.shape[1:]), ref)
                r, g = bf16_to_f32(ref).astype(np.float64), bf16_to_f32(got).astype(np.float64)
                scale = np.abs(r).reshape(r.shape[0], -1).max(axis=1).reshape(-1, 1, 1, 1) + 1e-30
                assert np.all(np.abs(g - r) <= 2e-2 * scale), f"segment {s}: {np.max(np.abs(g - r) / scale)}"
                act = ref
            eng.close()
    finally:
        ee.tune_conv_tile(old)


def test_bf16_serve_stream_decisions(torch, ee, orc):
    name, n, b_max = "tiny_bf16", 64, 8
    blob = W.load_net(name)
    pool = W.input_pool(blob, n)
    eng = ee.Engine(blob, b_max)
    lut = synthetic_lut(blob.n_stages, b_max)
    got, st, _ = eng.serve_stream(np.zeros(n, np.int64), dev(torch, pool), lut, clock=1)
    # the oracle's view of every sample at every exit it reaches
    act, alive = pool, np.arange(n)
    unclear = np.zeros(n, bool)
    ref_exit = np.full(n, -1)
    for s in range(blob.n_stages):
        act = orc.stage_forward(blob, s, act)
        thr = float(blob.exits[s]["thr"])
        lab, conf, _, flag = orc.exit_head(blob, s, act, thr)
        if s < blob.n_stages - 1:
            unclear[alive[np.abs(conf - np.float32(thr)) < 1e-3]] = True
        ref_exit[alive[flag == 1]] = s
        act, alive = act[flag == 0], alive[flag == 0]
    ok = ~unclear
    assert np.array_equal(got["exit_idx"][ok], ref_exit[ok])
    assert np.bincount(got["exit_idx"], minlength=3).sum() == n
    eng.close()
