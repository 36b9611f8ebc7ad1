"""Kernels at the sizes where a tile, a remainder or a dispatch rule can go wrong, against the oracle (needs an MI355X)."""
import numpy as np
import pytest

import synth
from helpers import check_parity, rel_err, setup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


def forward(torch, net, spec, cfgs, route, x, **kw):
    t = torch.from_numpy(np.ascontiguousarray(x))
    t = (t.to(torch.bfloat16) if spec.dtype == "bf16" else t).to("cuda:0")
    out = net.forward(cfgs, np.asarray(route, np.int32), t, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# fp32 convolutions: reductions of 27 (scalar loads), 72 (one wave per tile), 8..31 and >= 32 steps of 16 (2, 4 and 8
# waves per tile), channel counts around the 16-wide tile, pixel counts around the 16 x waves a block covers.
# Tolerance: a sum of n fp32 terms in another order moves by about sqrt(n) 2^-24 of its size; n <= 1152 and 8 layers
# in a row give 8 * 34 * 6e-8 = 1.6e-5.
@pytest.mark.parametrize("stages,res,batch", [((8, 8, 16), 9, 1), ((16, 24, 40), 17, 3), ((32, 64, 128), 32, 5),
                                              ((56, 72, 120), 11, 2), ((128, 8, 128), 8, 16)])
def test_fp32_conv_tile_edges(torch_mod, stages, res, batch):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.TinySpec(stage_ch=stages, width_choices=(1.0,), res_choices=(res,))
    W, S, C = setup(spec, 2)
    net = sna.Supernet(spec, W, S, 2, 16)
    try:
        for c in (C[0], C[-1]):
            x = synth.make_inputs(spec, batch, res, res, 11)
            print("fp32 conv", stages, res, batch, c.depth, flush=True)
            got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
            check_parity(got, oracle.forward(spec, W, S, c, x), "fp32", f"{stages} {res} x{batch}", tol=1.6e-5)
    finally:
        net.close()


def depthwise_launches(torch, net, spec, cfgs, route, x):
    """-> (problems that ran expand and depthwise as one launch, problems of separate depthwise launches) of a forward."""
    net.profile_enable(True)
    try:
        forward(torch, net, spec, cfgs, route, x)
        lines = [l for l in net.profile_read_launches().split("\n") if " depthwise " in l]
        net.profile_read()                                      # forgets the launches read
    finally:
        net.profile_enable(False)
    fused = sum(l.count("Cin=") for l in lines)
    return fused, sum(l.count("[N=") for l in lines) - fused


# Fused expand + depthwise: images whose stage outputs are 65 x 33, 33 x 17, 17 x 9 .. and 1 x 1 (segments of 16 outputs
# with remainders 1 and 15, several column tiles, several requests per block with a partial last block), every kernel
# size, all of a forward's blocks in one launch each.  Tolerance: the family's 2e-2 (each stored tensor is rounded to bf16
# once); requests are bitwise independent of the batch and of the other subnets of the call they come in.
@pytest.mark.parametrize("h,w,batch", [(130, 66, 2), (36, 140, 3), (260, 30, 1), (8, 9, 17), (57, 57, 5)])
def test_expand_depthwise_tile_edges(torch_mod, h, w, batch):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, res_choices=(260,))
    W, S, C = setup(spec, 4)
    net = sna.Supernet(spec, W, S, 4, 20)
    try:
        x = synth.make_inputs(spec, batch, h, w, 12)
        alone = []
        for c in C:
            c.in_h, c.in_w = h, w
            print("expand + depthwise", h, w, batch, c.block_kernel, flush=True)
            got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
            check_parity(got, oracle.forward(spec, W, S, c, x), "bf16", f"{h} x {w}")
            last = forward(torch_mod, net, spec, [c], np.zeros(1), x[-1:])
            np.testing.assert_array_equal(got[-1:], last)
            assert depthwise_launches(torch_mod, net, spec, [c], np.zeros(batch), x) == (sum(c.depth), 0)
            alone.append(got)
        route = np.arange(batch) * 3 % len(C)
        mixed = forward(torch_mod, net, spec, C, route, x)
        np.testing.assert_array_equal(mixed, np.stack([alone[r][i] for i, r in enumerate(route)]))
    finally:
        net.close()


# Several requests per block of the fused layer, whose squeeze-excite pool sums a request's segments over lanes: outputs of
# 5, 6, 9 and 14 rows, of two and three column segments, and at stride 2, where a request's 3, 5, 6 or 7 segments begin in the
# middle of a lane's four.  One pixel of each request is 2^16 larger, so that the sums round.  Every request has the bits that
# it has alone.
@pytest.mark.parametrize("h,w,k,stride", [(10, 10, 7, 1), (12, 12, 5, 1), (18, 18, 3, 1), (28, 28, 5, 1), (12, 40, 3, 1), (10, 80, 3, 1),
                                          (27, 28, 3, 2), (20, 20, 5, 2)])
def test_pool_sums_at_every_place_of_a_block(torch_mod, h, w, k, stride):
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=200, stage_ch=(160,), stage_stride=(stride,), stage_se=(True,), stage_act=("hswish",),
                          max_depth=(4,), depth_choices=(4,), expand_choices=(6,), kernel_choices=(k,), res_choices=(80,))
    W, S, C = setup(spec, 2)
    c, batch = C[-1], 17
    c.in_h, c.in_w = h, w
    x = synth.make_inputs(spec, batch, h, w, 18)
    for i in range(batch):
        x[i, i % h, (3 * i) % w] *= 2.0 ** 16
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        print("pool sums", h, w, k, stride, flush=True)
        got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
        alone = [forward(torch_mod, net, spec, [c], np.zeros(1), x[i:i + 1])[0] for i in range(batch)]
        assert [i for i in range(batch) if not np.array_equal(got[i], alone[i])] == []
    finally:
        net.close()


# Wide block inputs.  168 and 264 channels: a reduction of more than one pass of five steps, and more weight fragments than
# one per thread.  4800 channels: the expand weights no longer fit in LDS beside the tile, and the block runs as separate
# expand and depthwise launches, with the gate's pool in the depthwise one.  Tolerance: the family's.
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("k", [3, 5, 7])
def test_expand_depthwise_wide_inputs(torch_mod, k, stride):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(168, 264, 4800, 24), stage_stride=(1, 2, 1, stride),
                          stage_se=(False, True, False, True), stage_act=("relu", "hswish", "relu", "hswish"),
                          max_depth=(1, 1, 1, 1), depth_choices=(1,), expand_choices=(0.1,), kernel_choices=(k,),
                          res_choices=(80,), tail_ch=64, fc_ch=64)
    W, S, C = setup(spec, 2)
    c, batch, h, w = C[-1], 3, 70, 62
    c.in_h, c.in_w = h, w
    x = synth.make_inputs(spec, batch, h, w, 16)
    ref = oracle.forward(spec, W, S, c, x)
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        print("wide inputs", k, stride, c.block_mid_ch, flush=True)
        got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
        check_parity(got, ref, "bf16", f"{k} x {k} / {stride}")
        np.testing.assert_array_equal(got[-1:], forward(torch_mod, net, spec, [c], np.zeros(1), x[-1:]))
        assert depthwise_launches(torch_mod, net, spec, [c], np.zeros(batch), x) == (3, 1)
    finally:
        net.close()


# Squeeze-excite gates that no matrix tile can apply, so that a pass of its own scales the tensor: 1632 expanded channels,
# whose project layer sums in two chunks, and 1 x 1 maps of more requests than have room for their gates beside a tile's ring
# (960 channels: 24 have, 40 have not).  The launch list says how many gates were scaled by the pass.  Tolerance: the
# family's; requests are bitwise independent of the batch, which takes them one way or the other, and of their call's subnets.
def scaled_gates(torch, net, spec, cfgs, route, x):
    """-> (gates applied by the project layer, gates applied by a pass of its own) of a forward, by their bytes."""
    net.profile_enable(True)
    try:
        forward(torch, net, spec, cfgs, route, x)
        lines = [l for l in net.profile_read_launches().split("\n") if " squeeze_excite " in l]
        net.profile_read()
    finally:
        net.profile_enable(False)
    n = [0, 0]
    for l in lines:
        gates = [[int(t.split("=")[1]) for t in g.split("]")[0].split()] for g in l.split(" [")[1:]]       # N, HW, C, Q
        left = float(l.split("bytes=")[1].split()[0]) - sum(4.0 * c * q for _, _, c, q in gates)
        # the subnets of a call differ in their channels, so that the bytes tell which of them were scaled
        ways = [m for m in range(1 << len(gates)) if left == sum(4.0 * g[0] * g[1] * g[2] for i, g in enumerate(gates) if m >> i & 1)]
        assert len(ways) == 1, l
        n[1] += bin(ways[0]).count("1")
        n[0] += len(gates) - bin(ways[0]).count("1")
    return tuple(n)


def test_gates_scaled_by_a_pass_of_their_own(torch_mod):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(272,), stage_stride=(2,), stage_se=(True,), stage_act=("hswish",), max_depth=(3,),
                          depth_choices=(3,), expand_choices=(3, 6), kernel_choices=(3,), res_choices=(80,), tail_ch=64, fc_ch=64)
    W, S, C = setup(spec, 2)
    batch, h, w = 5, 28, 36
    x = synth.make_inputs(spec, batch, h, w, 21)
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        alone = []
        for c, mid, want in ((C[0], 816, (3, 0)), (C[-1], 1632, (1, 2))):
            c.in_h, c.in_w = h, w
            assert c.block_mid_ch[0][1] == mid
            print("scaled gates", mid, flush=True)
            got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
            check_parity(got, oracle.forward(spec, W, S, c, x), "bf16", f"mid {mid}")
            assert scaled_gates(torch_mod, net, spec, [c], np.zeros(batch), x) == want
            np.testing.assert_array_equal(got[3:4], forward(torch_mod, net, spec, [c], np.zeros(1), x[3:4]))
            alone.append(got)
        route = np.array([0, 1, 1, 0, 1])
        mixed = forward(torch_mod, net, spec, [C[0], C[-1]], route, x)
        np.testing.assert_array_equal(mixed, np.stack([alone[r][i] for i, r in enumerate(route)]))
        assert scaled_gates(torch_mod, net, spec, [C[0], C[-1]], route, x) == (4, 2)
    finally:
        net.close()


def test_gates_of_many_one_pixel_maps(torch_mod):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(24, 160), stage_stride=(2, 2), stage_se=(False, True), stage_act=("relu", "hswish"),
                          max_depth=(3, 3), depth_choices=(3,), expand_choices=(6,), kernel_choices=(3,), res_choices=(80,), tail_ch=64,
                          fc_ch=64)
    W, S, C = setup(spec, 2)
    c = C[-1]
    c.in_h = c.in_w = 8
    x = synth.make_inputs(spec, 40, 8, 8, 22)
    ref = oracle.forward(spec, W, S, c, x)
    net = sna.Supernet(spec, W, S, 2, 40)
    try:
        alone = [forward(torch_mod, net, spec, [c], np.zeros(1), x[i:i + 1])[0] for i in range(40)]
        check_parity(np.stack(alone), ref, "bf16", "alone")
        for batch, scaled in ((1, 0), (24, 0), (40, 2)):
            print("one-pixel maps", batch, flush=True)
            got = forward(torch_mod, net, spec, [c], np.zeros(batch), x[:batch])
            np.testing.assert_array_equal(got, np.stack(alone[:batch]))
            assert scaled_gates(torch_mod, net, spec, [c], np.zeros(batch), x[:batch])[1] == scaled
    finally:
        net.close()


# A tile that scales its input has waves of its own that fetch (8, 28 and 29): the price of a step that the choice goes by
# holds for scaling only where others compute meanwhile.  Forcing any other variant, or none, leaves one of the three.
@pytest.mark.parametrize("batch,res", [(1, 64), (48, 80)])
def test_gated_layers_run_where_waves_fetch(torch_mod, batch, res):
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(40,), stage_stride=(2,), stage_se=(True,), stage_act=("relu",), max_depth=(3,),
                          depth_choices=(3,), expand_choices=(3,), kernel_choices=(3,), res_choices=(80,), tail_ch=64, fc_ch=64)
    W, S, C = setup(spec, 2)
    c = C[-1]
    c.in_h = c.in_w = res
    x = synth.make_inputs(spec, batch, res, res, 23)
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        ref = None
        for v in [-1] + list(range(sna.lib().sna_tile_variant_count())):
            net.set_tile_variant(v)
            got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
            ref = got if ref is None else ref
            np.testing.assert_array_equal(got, ref)
            net.profile_enable(True)
            try:
                forward(torch_mod, net, spec, [c], np.zeros(batch), x)
                lines = [l for l in net.profile_read_launches().split("\n") if " igemm_conv_linear " in l and " K=40 C=" in l]
                net.profile_read()
            finally:
                net.profile_enable(False)
            lines = [l for l in lines if " M=1 " not in l and f"M={batch} " not in l]             # not the classifier
            assert len(lines) == 3, lines
            ran = {int(l.split("tile=")[1].split(" ")[0]) for l in lines}
            assert ran <= {8, 28, 29}, (v, lines)
            if v == -1 and batch == 48:                            # 1200 blocks of 32x32: beyond two a CU another tile is faster
                assert 28 not in ran, lines
    finally:
        net.close()


# Attention and LayerNorm: token counts around the 16-query waves and the key pairs a lane transposes (odd counts, one
# token, a full block), hidden sizes whose last 64-lane group of octets is partial (9, 65 octets) or full (256).
# Tolerance: the family's.
@pytest.mark.parametrize("tokens,hidden,heads", [(1, 72, 1), (2, 520, 3), (17, 72, 1), (31, 72, 2), (65, 520, 1), (127, 136, 2),
                                                 (128, 2048, 1)])
def test_attention_layernorm_edges(torch_mod, tokens, hidden, heads):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.TransformerSpec(n_classes=40, hidden=hidden, n_heads=heads, ffn=96, max_layers=2, seq_len=tokens,
                                 depth_choices=(1, 2))
    W, S, C = setup(spec, 2)
    net = sna.Supernet(spec, W, S, 2, 5)
    try:
        c = C[-1]
        x = synth.make_inputs(spec, 5, c.in_h, c.in_w, 13)
        print("attention", tokens, hidden, heads, flush=True)
        got = forward(torch_mod, net, spec, [c], np.zeros(5), x)
        check_parity(got, oracle.forward(spec, W, S, c, x), "bf16", f"{tokens} x {hidden}")
    finally:
        net.close()


# MBV3 head: outputs of 14, 15 and 29 rows or columns (14 x 14 tiles), image edges that fall on every window position, and
# a request with a row of one tile only.  Tolerance: the family's.
@pytest.mark.parametrize("h,w", [(27, 29), (28, 30), (29, 57), (58, 26), (31, 15)])
def test_mbv3_head_tile_edges(torch_mod, h, w):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(24,), stage_stride=(1,), stage_se=(False,), stage_act=("relu",),
                          max_depth=(1,), depth_choices=(1,), kernel_choices=(3,), res_choices=(80,), tail_ch=64, fc_ch=64)
    W, S, C = setup(spec, 2)
    net = sna.Supernet(spec, W, S, 2, 3)
    try:
        c = C[-1]
        c.in_h, c.in_w = h, w
        x = synth.make_inputs(spec, 3, h, w, 15)
        print("mbv3 head", h, w, flush=True)
        check_parity(forward(torch_mod, net, spec, [c], np.zeros(3), x), oracle.forward(spec, W, S, c, x), "bf16", f"{h} x {w}")
    finally:
        net.close()


# Non-finite activations of the fused expand + depthwise layer: one pixel of request 0 is so large that the expanded tensor
# overflows to Inf around it.  The depthwise weights are negative, so that every output whose own taps see it is ReLU(-Inf)
# = 0 and the logits stay finite; an output that does not see it keeps its value.  (Inf times the zeros of the band matrix
# would make NaN, and ReLU 0, of all 16 outputs of the row segment.)  The oracle refuses to overflow; a pixel of 2^40 in
# the place of 2^100 drives the same outputs below zero without.  Tolerance: the family's.
@pytest.mark.parametrize("stride,h,w", [(1, 24, 20), (2, 24, 20), (1, 14, 76), (2, 22, 76)])
@pytest.mark.parametrize("k", [3, 5, 7])
def test_overflow_stays_in_its_window(torch_mod, k, stride, h, w):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.MBV3Spec(n_classes=40, stage_ch=(24,), stage_stride=(stride,), stage_se=(False,), stage_act=("relu",),
                          max_depth=(1,), depth_choices=(1,), kernel_choices=(k,), res_choices=(80,), tail_ch=64, fc_ch=64)
    W, S, C = setup(spec, 2)
    W["s0.b0.dw.w"] = -np.abs(W["s0.b0.dw.w"])
    S["s0.b0.sn1"][:, 2] *= 1e10
    S["s0.b0.sn2"][:, 2] *= 1e-10
    S["s0.b0.sn2"][:, 3] += 3.0
    c, batch = C[-1], 3
    c.in_h, c.in_w = h, w
    x = synth.make_inputs(spec, batch, h, w, 14)
    ref_plain = oracle.forward(spec, W, S, c, x)
    x[0, h // 2, w // 2] = 2.0 ** 40
    ref = oracle.forward(spec, W, S, c, x)
    x[0, h // 2, w // 2] = 2.0 ** 100
    assert np.abs(ref[0] - ref_plain[0]).max() > 0.04 * np.abs(ref[0]).max()
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        print("overflow", k, stride, h, w, flush=True)
        got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
        check_parity(got, ref, "bf16", f"{k} x {k} / {stride}, {h} x {w}")
        for i in range(1, batch):
            np.testing.assert_array_equal(got[i:i + 1], forward(torch_mod, net, spec, [c], np.zeros(1), x[i:i + 1]))
    finally:
        net.close()


# A weight of -Inf at the first tap of one fp32 stem channel, over positive pixels: every output whose window holds that tap
# inside the image is ReLU(-Inf) = 0, and the outputs of the first row and column, whose tap lies in the padding, keep their
# value (padding zeros times the weight would make NaN of them, and ReLU 0).  A weight of -2^60 does the same with finite
# numbers.  in_ch 3 takes the scalar loads, 4 the vector ones.  Tolerance: as for the fp32 convolutions above.
@pytest.mark.parametrize("in_ch", [3, 4])
def test_infinite_weight_stays_in_its_tap(torch_mod, in_ch):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.TinySpec(in_ch=in_ch, res_choices=(9,))
    W, S, C = setup(spec, 2)
    c, batch = C[-1], 3
    x = np.abs(synth.make_inputs(spec, batch, 9, 9, 15)) + np.float32(0.1)
    W["stem.w"][1, 0, 0, :] = -2.0 ** 60
    ref = oracle.forward(spec, W, S, c, x)
    all_zero = dict(W)
    all_zero["stem.w"] = W["stem.w"].copy()
    all_zero["stem.w"][1] = -2.0 ** 60
    assert rel_err(oracle.forward(spec, all_zero, S, c, x), ref).min() > 5e-4
    W["stem.w"][1, 0, 0, :] = -np.inf
    net = sna.Supernet(spec, W, S, 2, batch)
    try:
        print("infinite weight", in_ch, flush=True)
        got = forward(torch_mod, net, spec, [c], np.zeros(batch), x)
        check_parity(got, ref, "fp32", f"in_ch {in_ch}", tol=1.6e-5)
    finally:
        net.close()


# Deep-ring tiles of the matrix kernel (the last variants): reductions of 1, 2 and 7..9 steps around the 8 stages of the
# ring, whole and half groups of steps, 25 and 65 steps (two and four chunks, folded or spread over blocks) and 129 steps,
# more than a deep ring walks: unless they are spread, another tile runs them.  Same bits as the 128x64 tile, which walks the same order; the
# oracle's tolerance is the family's.
@pytest.mark.parametrize("hidden,ffn", [(64, 64), (72, 440), (128, 512), (136, 520), (192, 640), (72, 1544), (64, 4160),
                                        (64, 8256)])
def test_deep_ring_step_counts(torch_mod, hidden, ffn):
    import oracle
    import paper_2312_16733_amd as sna
    spec = synth.TransformerSpec(n_classes=40, hidden=hidden, n_heads=1, ffn=ffn, max_layers=1, seq_len=11,
                                 depth_choices=(1,))
    W, S, C = setup(spec, 2)
    net = sna.Supernet(spec, W, S, 2, 7)
    try:
        c = C[-1]
        x = synth.make_inputs(spec, 7, c.in_h, c.in_w, 17)
        net.set_tile_variant(1)
        ref = forward(torch_mod, net, spec, [c], np.zeros(7), x)
        check_parity(ref, oracle.forward(spec, W, S, c, x), "bf16", f"{hidden} x {ffn}")
        nv = sna.lib().sna_tile_variant_count()
        for v in (nv - 3, nv - 2, nv - 1):
            for split in (1, 2):
                net.set_tile_variant(v)
                net.set_k_split(split)
                print("deep ring", hidden, ffn, "variant", v, "split", split, flush=True)
                np.testing.assert_array_equal(forward(torch_mod, net, spec, [c], np.zeros(7), x), ref)
    finally:
        net.close()


# The same tiles with taps: 3x3 layers of 2, 7, 8, 9, 25 and 65 steps, 128 (the longest table, the folding 64x64 kernel's
# whole LDS) and 129, which only fits when it is spread over blocks; odd images whose windows cross every border, two
# requests in a tile.  The launch list says which tile ran.  Same bits as the 128x64 tile.
@pytest.mark.parametrize("mid", [8, 48, 56, 64, 176, 456, 904, 912])
def test_deep_ring_taps(torch_mod, mid):
    import oracle
    import paper_2312_16733_amd as sna
    steps = -(-9 * mid // 64)
    spec = synth.ResNetSpec(n_classes=24, stem_ch=16, stage_ch=(64, 64), stage_stride=(1, 2), max_depth=(2, 1), depth_minus=(0, 1),
                            expand_choices=(mid / 64,), width_choices=(1.0,), res_choices=(40,))
    W, S, C = setup(spec, 2)
    net = sna.Supernet(spec, W, S, 2, 3)
    try:
        c = C[-1]
        c.in_h, c.in_w = 37, 27
        assert c.block_mid_ch[0][0] == mid
        x = synth.make_inputs(spec, 3, c.in_h, c.in_w, 19)
        net.set_tile_variant(1)
        ref = forward(torch_mod, net, spec, [c], np.zeros(3), x)
        check_parity(ref, oracle.forward(spec, W, S, c, x), "bf16", f"mid {mid}")
        nv = sna.lib().sna_tile_variant_count()
        for v in (nv - 3, nv - 2, nv - 1):
            for split in (1, 2, 3):
                net.set_tile_variant(v)
                net.set_k_split(split)
                print("deep ring taps", mid, "variant", v, "split", split, flush=True)
                np.testing.assert_array_equal(forward(torch_mod, net, spec, [c], np.zeros(3), x), ref)
                net.profile_enable(True)
                try:
                    forward(torch_mod, net, spec, [c], np.zeros(3), x)
                    lines = [l for l in net.profile_read_launches().split("\n") if " igemm_conv_linear " in l and " 3x3/" in l]
                    net.profile_read()
                finally:
                    net.profile_enable(False)
                assert len(lines) == sum(c.depth)
                ran = {int(l.split("tile=")[1].split(" ")[0]) for l in lines}
                assert (ran == {v}) == (split > 1 or steps <= 128), (steps, split, lines)
    finally:
        net.close()
