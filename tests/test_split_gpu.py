"""fp32 layers on the f16 matrix instructions (every operand as two f16 values): shapes at the edges of their tiles,
magnitudes far apart, and what lies outside the forms they take."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import paper_1611_07151_amd as sq
    return sq


@pytest.fixture(autouse=True)
def wherever_the_form_fits(sq):
    """Layers too small for it to pay run on split operands too."""
    sq.lib.sq_tune_conv_split(1)
    yield
    sq.lib.sq_tune_conv_split(-1)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def assert_close(got, ref, what):
    err = np.abs(got.astype(np.float64) - ref) / (1 + np.abs(ref.astype(np.float64)))
    assert np.isfinite(got).all() and err.max() <= 1e-4, (what, float(err.max()))


def assert_within_rounding(got, ref, x, w, b, pad, what, stride=1):
    """Every result within the bound of an fp32 sum over the same products: a rounding of 2^-24 per step of 16 terms (two
    accumulators), operands and dropped products 2^-22 of each term, all relative to the sum of the terms' magnitudes."""
    terms = oracle.conv2d(np.abs(x), np.abs(w), np.abs(b), stride, pad, False).astype(np.float64)
    steps = max(w.shape[2] ** 2 * ((w.shape[1] + 15) // 16), 3 * ((w[0].size + 15) // 16))    # (or three roundings per 16 terms)
    bound = (steps + 8) * 2.0 ** -23 * terms
    err = np.abs(got.astype(np.float64) - ref)
    assert np.isfinite(got).all() and (err <= bound).all(), (what, float((err / bound).max()))


# N, Cin, Cout, K, H, W: one pixel, rows shorter and longer than a tile, images that share a tile, input layers that are no
# multiple of 16, output layers that fill no block of 32, contractions dealt out to two and four wavefronts, a map that
# does not fit LDS at once, and batches on both sides of the 32- and 96-pixel tiles
CONVS = [(5, 16, 32, 3, 1, 1), (5, 8, 32, 3, 2, 40), (3, 24, 96, 3, 9, 7), (1, 48, 192, 3, 5, 6), (2, 64, 64, 3, 27, 27), (1, 16, 64, 3, 55, 55),
         (9, 128, 128, 3, 3, 3), (3, 256, 384, 3, 13, 13), (1, 384, 64, 3, 40, 41), (24, 32, 96, 3, 33, 31), (2, 24, 40, 5, 11, 9),
         (1, 3, 8, 5, 4, 70), (11, 48, 256, 5, 21, 20)]


@pytest.mark.parametrize("case", CONVS, ids=lambda c: "x".join(map(str, c)))
def test_conv_on_split_operands(sq, case):
    n, cin, cout, k, h, w_ = case
    rng = np.random.default_rng(n * 100 + cin)
    x = synth.normal01(rng, (n, cin, h, w_))
    w, b = synth.conv_params(rng, cout, cin, k)
    pad = (k - 1) // 2
    ref = oracle.conv2d(x, w, b, 1, pad, True)
    xd, wd, bd = dev(x), dev(w), dev(b)
    sq.sq_profile_begin(8)
    got = sq.sq_conv2d_forward_ws(xd, wd, bd, 1, pad, True)
    names = [r["name"] for r in sq.sq_profile_end()]
    if cout % 32 == 0 and cin % 8 == 0:
        assert any(f"k{k}s1_split" in s for s in names), names
    assert_within_rounding(got.cpu().numpy(), ref, x, w, b, pad, case)
    # into a wider tensor, without bias and ReLU
    out = torch.full((n, cout + 5, h, w_), -7.0, device="cuda")
    sq.sq_conv2d_forward_ws(xd, wd, None, 1, pad, False, out=out, c_offset=3)
    assert_within_rounding(out[:, 3:3 + cout].cpu().numpy(), oracle.conv2d(x, w, None, 1, pad, False), x, w, b, pad, "offset")
    assert bool((out[:, :3] == -7).all()) and bool((out[:, 3 + cout:] == -7).all())


@pytest.mark.parametrize("cin", [16, 64, 384])       # one part, several parts, staged in two goes
@pytest.mark.parametrize("outlier,scale", [(1e30, 1.0), (3e5, 1.0), (1e30, 1e-6), (1.0, 1e-30), (1e38, 1e36)])
def test_magnitudes_far_apart_do_not_disturb_each_other(sq, cin, outlier, scale):
    """A pixel many powers of two above its neighbours: results whose windows do not touch it keep their precision."""
    rng = np.random.default_rng(cin)
    x = (np.maximum(synth.normal01(rng, (2, cin, 11, 13)), 0) * np.float32(scale)).astype(np.float32)
    x[0, 3, 4, 5] = outlier
    x[1, :, 7, :] = 0
    w, b = synth.conv_params(rng, 64, cin, 3)
    w *= np.float32(0.01)
    b *= np.float32(scale)
    got = sq.sq_conv2d_forward_ws(dev(x), dev(w), dev(b), 1, 1, True).cpu().numpy()
    assert_within_rounding(got, oracle.conv2d(x, w, b, 1, 1, True), x, w, b, 1, (cin, outlier, scale))


# the expands of a fire layer: layers that fill no block, blocks shared unevenly, small and large tiles
@pytest.mark.parametrize("n,cin,csq,ce1,ce3,h,w", [(3, 16, 48, 32, 32, 7, 7), (3, 48, 64, 40, 32, 9, 5), (7, 32, 48, 8, 96, 8, 30), (64, 64, 64, 64, 64, 3, 3),
                                                   (3, 128, 48, 160, 160, 27, 13), (24, 32, 64, 100, 64, 33, 34)])
def test_fire_on_split_operands(sq, n, cin, csq, ce1, ce3, h, w):
    rng = np.random.default_rng(n + cin)
    x = synth.uniform01(rng, (n, cin, h, w))
    p = [*synth.conv_params(rng, csq, cin, 1), *synth.conv_params(rng, ce1, csq, 1), *synth.conv_params(rng, ce3, csq, 3)]
    p[1] = (p[1] + 0.5).astype(np.float32)          # relu(b_sq) != 0: the padding must still be zero
    d = [dev(a) for a in [x] + p]
    sq.sq_profile_begin(8)
    got = sq.sq_fire_forward(*d)
    names = [r["name"] for r in sq.sq_profile_end()]
    assert any("split" in s and s.endswith("+k1") for s in names), names
    assert torch.equal(sq.sq_fire_forward_packed(*d, sq.sq_fire_pack_weights(d[5])), got)
    s = sq.sq_conv2d_forward(d[0], d[1], d[2], 1, 0, True).cpu().numpy()
    g = got.cpu().numpy()
    assert_within_rounding(g[:, :ce1], oracle.conv2d(s, p[2], p[3], 1, 0, True), s, p[2], p[3], 0, "expand1x1")
    assert_within_rounding(g[:, ce1:], oracle.conv2d(s, p[4], p[5], 1, 1, True), s, p[4], p[5], 1, "expand3x3")


# N, H, W, pad, Cout: smaller than a tile, one pixel, tiles cut off on either side, even and odd extents, fewer output
# layers than a block and than all three, and more tiles than workgroups
STEMS = [(1, 7, 7, 0, 96), (2, 5, 6, 1, 8), (1, 40, 37, 2, 96), (3, 33, 70, 3, 40), (2, 224, 224, 2, 96), (17, 96, 130, 0, 33)]


@pytest.mark.parametrize("case", STEMS, ids=lambda c: "x".join(map(str, c)))
def test_first_layer_on_split_operands(sq, case):
    n, h, w_, pad, cout = case
    rng = np.random.default_rng(n + h)
    x = synth.uniform01(rng, (n, 3, h, w_))
    w, b = synth.conv_params(rng, cout, 3, 7)
    sq.sq_profile_begin(8)
    got = sq.sq_conv2d_forward(dev(x), dev(w), dev(b), 2, pad, True)
    names = [r["name"] for r in sq.sq_profile_end()]
    assert any("k7s2c3_split" in s for s in names), names
    assert_within_rounding(got.cpu().numpy(), oracle.conv2d(x, w, b, 2, pad, True), x, w, b, pad, case, 2)
    ho, wo = got.shape[2:]
    out = torch.full((n, cout + 5, ho, wo), -7.0, device="cuda")
    sq.sq_conv2d_forward_ex(dev(x), dev(w), None, 2, pad, False, out=out, c_offset=3)
    assert_within_rounding(out[:, 3:3 + cout].cpu().numpy(), oracle.conv2d(x, w, None, 2, pad, False), x, w, b, pad, "offset", 2)
    assert bool((out[:, :3] == -7).all()) and bool((out[:, 3 + cout:] == -7).all())


@pytest.mark.parametrize("outlier,scale", [(1e30, 1.0), (3e5, 1.0), (1.0, 1e-30), (1e38, 1e36)])
def test_first_layer_with_magnitudes_far_apart(sq, outlier, scale):
    rng = np.random.default_rng(3)
    x = (synth.uniform01(rng, (2, 3, 50, 61)) * np.float32(scale)).astype(np.float32)
    x[0, 1, 20, 33] = outlier
    w, b = synth.conv_params(rng, 96, 3, 7)
    w *= np.float32(0.01)
    b *= np.float32(scale)
    got = sq.sq_conv2d_forward(dev(x), dev(w), dev(b), 2, 2, True).cpu().numpy()
    # (a tile with such a pixel is summed one product after another: up to a rounding per product)
    terms = oracle.conv2d(np.abs(x), np.abs(w), np.abs(b), 2, 2, False).astype(np.float64)
    ref = oracle.conv2d(x, w, b, 2, 2, True)
    assert np.isfinite(got).all() and (np.abs(got.astype(np.float64) - ref) <= 160 * 2.0 ** -24 * terms).all()


@pytest.mark.parametrize("k,stride,cin,cout,kg", [(7, 2, 3, 96, 1), (5, 1, 24, 64, 4), (5, 1, 200, 96, 1)])
@pytest.mark.parametrize("where", ["map", "kernels"])
def test_infinities_and_nan_go_where_fp32_sums_take_them(sq, k, stride, cin, cout, kg, where):
    rng = np.random.default_rng(k + cin)
    pad = 2
    x = synth.normal01(rng, (2, cin, 41, 43))
    w, b = synth.conv_params(rng, cout, cin, k)
    if where == "map":
        x[0, 1, 20, 21] = np.inf
        x[1, 2, 30, 7] = np.nan
        x[1, 0, 9, 36] = -np.inf
    else:
        w[5, 1, 2, 2] = np.inf
        w[40, 2, 1, 0] = np.nan
    xi, wi = np.where(np.isfinite(x), x, 0), np.where(np.isfinite(w), w, 0)
    # layers and windows that such a value reaches, summed in fp32 by the kernels that take every shape
    want = sq.sq_conv2d_forward_ex(dev(x), dev(w), dev(b), stride, pad, True, algo=sq.SQ_ALGO_DIRECT).cpu().numpy()
    got = (sq.sq_conv2d_forward_ws if stride == 1 else sq.sq_conv2d_forward)(dev(x), dev(w), dev(b), stride, pad, True).cpu().numpy()
    reached = oracle.conv2d((~np.isfinite(x)).astype(np.float32), np.ones_like(w), None, stride, pad, False) > 0 if where == "map" else \
        np.broadcast_to((~np.isfinite(w)).any(axis=(1, 2, 3))[None, :, None, None], want.shape)
    assert reached.any() and np.isinf(want[reached]).any()
    np.testing.assert_array_equal(got[reached & ~np.isfinite(want)], want[reached & ~np.isfinite(want)])
    np.testing.assert_array_equal(got[reached & (want == 0)], 0)
    ref = oracle.conv2d(xi, wi, b, stride, pad, True)
    got, ref = np.where(reached, 0, got), np.where(reached, 0, ref)
    terms = oracle.conv2d(np.abs(xi), np.abs(wi), np.abs(b), stride, pad, False).astype(np.float64)
    assert (np.abs(got.astype(np.float64) - ref) <= w[0].size * 2.0 ** -24 * terms).all()


@pytest.mark.parametrize("n,split_layers", [(10, 4), (13, 4), (32, 8)])
def test_packed_network_on_split_operands(sq, n, split_layers):
    """From ten images on the packed call computes the first layer, its pooling and the first squeeze in one launch, and
    the expands of the later fire layers, from 32 on of all, on split operands."""
    cfg = synth.config_squeezenet(seed=50 + n, n=n)
    params = [dev(p) for p in cfg["params"]]
    packed = sq.sq_pack_weights(params, sq.SQ_F32)
    x = cfg["x"].copy()
    x[n - 1, :, 100:140, 30:60] *= np.float32(1e7)         # tiles whose magnitudes span more than one scale holds
    sq.sq_profile_begin(64)
    got = sq.sq_squeezenet_forward_packed(dev(x), params, packed)
    names = {r["name"] for r in sq.sq_profile_end()}
    assert any("k7s2c3_split+pool3s2+k1" in s for s in names), names
    assert sum("/e1+e3|k3s1_split" in s for s in names) == split_layers, names
    ref = oracle.squeezenet(np.concatenate([x[:1], x[n - 1:]]), cfg["params"])
    assert_close(got[[0, n - 1]].cpu().numpy(), ref, "one-launch stem vs oracle")
    assert_close(got.cpu().numpy(), sq.sq_squeezenet_forward(dev(x), params).cpu().numpy(), "one-launch stem vs single layers")


# several images per tile and a tile per part of an image, layers staged in parts of 64 and of 128, a last workgroup that is
# not full, and (the fp32 forms then) too little work or too small a workspace for the split kernels
@pytest.mark.parametrize("n,cin,h,w,cout,taken", [(100, 64, 13, 13, 170, True), (9000, 128, 2, 1, 136, True), (170, 192, 9, 12, 130, True), (16, 256, 14, 14, 1000, True),
                                                  (80, 512, 6, 5, 1100, False), (16, 64, 13, 13, 40, False), (10, 2048, 5, 5, 2048, False)])
def test_classifier_on_split_operands(sq, n, cin, h, w, cout, taken):
    rng = np.random.default_rng(n + cin)
    x = synth.uniform01(rng, (n, cin, h, w))
    x[1, cin // 2:] *= np.float32(1e6)                     # scales that change on the way
    x[2] *= np.float32(1e-20)
    wt, b = synth.conv_params(rng, cout, cin, 1)
    sq.sq_profile_begin(16)
    probs, means = sq.sq_classifier_forward(dev(x), dev(wt), dev(b), want_means=True)
    names = [r["name"] for r in sq.sq_profile_end()]
    assert any("k1s1_split_96+planesums" in k for k in names) == taken, names
    ref = oracle.conv2d(x, wt, b, 1, 0, True).astype(np.float64).mean(axis=(2, 3))
    # three roundings per 16 products and one per pixel, relative to the terms
    terms = oracle.conv2d(np.abs(x), np.abs(wt), np.abs(b), 1, 0, False).astype(np.float64).mean(axis=(2, 3))
    err = np.abs(means.cpu().numpy() - ref)
    assert (err <= (3 * cin / 16 + h * w + 16) * 2.0 ** -24 * terms).all(), float((err / terms).max())
    assert_close(probs.cpu().numpy(), oracle.softmax(means.cpu().numpy()), "softmax")
    # an infinity and a NaN: means of the images that hold none stay, the others are those of fp32 sums
    x[3, 1, 0, 0], x[4, 0, h - 1, w - 1] = np.inf, np.nan
    _, odd = sq.sq_classifier_forward(dev(x), dev(wt), dev(b), want_means=True)
    odd = odd.cpu().numpy()
    want = sq.sq_avgpool_global(sq.sq_conv2d_forward_ex(dev(x), dev(wt), dev(b), 1, 0, True, algo=sq.SQ_ALGO_DIRECT)).cpu().numpy()
    assert np.isinf(want[3]).any()
    np.testing.assert_array_equal(np.isinf(odd), np.isinf(want))
    keep = np.isfinite(want) & (np.arange(n) != 4)[:, None]
    assert (np.abs(odd - ref)[keep & (np.arange(n) != 3)[:, None]] <= ((cin + h * w + 16) * 2.0 ** -24 * terms)[keep & (np.arange(n) != 3)[:, None]]).all()


def network_of_single_layers(sq, x, params):
    """The network as single calls of the kernels that take every shape, each a plain fp32 sum per output element."""
    conv = lambda t, i, stride=1, pad=0, **kw: sq.sq_conv2d_forward_ex(t, params[i], params[i + 1], stride, pad, True, algo=sq.SQ_ALGO_DIRECT, **kw)
    t = sq.sq_maxpool(conv(x, 0, 2, 2), 3, 2)
    for f in range(8):
        s = conv(t, 2 + 6 * f)
        ce = params[4 + 6 * f].shape[0]
        t = torch.empty((s.shape[0], 2 * ce, *s.shape[2:]), device="cuda")
        conv(s, 4 + 6 * f, out=t, c_offset=0)
        conv(s, 6 + 6 * f, 1, 1, out=t, c_offset=ce)
        if f in (2, 6):
            t = sq.sq_maxpool(t, 3, 2)
    return sq.sq_softmax(sq.sq_avgpool_global(conv(t, 50)))


@pytest.mark.parametrize("where", ["image", "conv1 kernels", "squeeze kernels"])
def test_one_launch_first_layers_with_infinities_and_nan(sq, where):
    """An infinity or NaN reaches the results that fp32 sums carry it to and no others: maxima and ReLU drop a NaN."""
    n = 10
    cfg = synth.config_squeezenet(seed=77, n=n)
    x, params = cfg["x"].copy(), [p.copy() for p in cfg["params"]]
    if where == "image":
        x[0, 1, 100, 57], x[3, 2, 7, 200], x[3, 0, 150, 3] = np.inf, -np.inf, np.nan
    elif where == "conv1 kernels":
        params[0][17, 1, 3, 4], params[0][90, 0, 2, 5] = np.nan, -np.inf     # (taps that no padding meets)
    else:
        params[2][5, 40], params[2][11, 3] = np.nan, -np.inf
    xd, pd = dev(x), [dev(p) for p in params]
    sq.sq_profile_begin(64)
    got = sq.sq_squeezenet_forward_packed(xd, pd, sq.sq_pack_weights(pd, sq.SQ_F32))
    assert any("k7s2c3_split+pool3s2+k1" in r["name"] for r in sq.sq_profile_end())
    pick = [0, 3, 9]
    want = network_of_single_layers(sq, xd[pick].contiguous(), pd).cpu().numpy()
    assert np.isfinite(want).all()
    assert_close(got[pick].cpu().numpy(), want, where)


# Values far apart that never meet: a sum is as exact as its own terms, whatever lies beside them under zero kernels or meets
# zeros.  2^20, 2^27 and more apart: within a scale's reach, at its end, and far outside it.
APART = [1e6, 2e8, 1e12, 1e30]


@pytest.mark.parametrize("big", APART)
@pytest.mark.parametrize("cin,cout,k,h,w_", [(16, 64, 3, 9, 11), (64, 32, 3, 27, 27), (384, 64, 3, 11, 13), (96, 40, 5, 30, 20), (3, 96, 7, 50, 61)])
@pytest.mark.parametrize("where", ["layer under zero kernels", "kernels over a zero layer", "single kernels over a zero layer", "one kernel"])
def test_sums_are_as_exact_as_their_own_terms(sq, cin, cout, k, h, w_, big, where):
    rng = np.random.default_rng(cin + k)
    stride, pad = (2, 2) if k == 7 else (1, (k - 1) // 2)
    x = np.maximum(synth.normal01(rng, (2, cin, h, w_)), 0)
    w, b = synth.conv_params(rng, cout, cin, k)
    if where == "layer under zero kernels":
        x[:, 1] = big
        w[:, 1] = 0
    elif where == "kernels over a zero layer":
        x[:, 1] = 0
        w[:, 1] *= np.float32(big)
    elif where == "single kernels over a zero layer":
        x[:, 2] = 0
        w[7, 2, 1, 1] = big
    else:                      # a pruned layer: one kernel of ordinary size, over small values beside large ones
        x[:, 0] *= np.float32(1 / big)
        w[3] = 0
        w[3, 0, k // 2, k // 2] = 0.75
        b[3] = 0
    b *= np.float32(1e-3)
    got = (sq.sq_conv2d_forward if k == 7 else sq.sq_conv2d_forward_ws)(dev(x), dev(w), dev(b), stride, pad, True).cpu().numpy()
    assert_within_rounding(got, oracle.conv2d(x, w, b, stride, pad, True), x, w, b, pad, (where, big), stride)


@pytest.mark.parametrize("big", APART)
@pytest.mark.parametrize("n,csq,ce", [(3, 48, 64), (24, 64, 256)])
def test_fire_sums_are_as_exact_as_their_own_terms(sq, n, csq, ce, big):
    rng = np.random.default_rng(csq)
    x = synth.uniform01(rng, (n, 32, 27, 27))
    p = [*synth.conv_params(rng, csq, 32, 1), *synth.conv_params(rng, ce, csq, 1), *synth.conv_params(rng, ce, csq, 3)]
    p[0][5] = np.abs(p[0][5]) * np.float32(big)                            # a squeeze layer that no expand kernel reads
    p[2][:, 5] = p[4][:, 5] = 0
    p[0][6], p[1][6] = -np.abs(p[0][6]), 0                                 # one that is zero after the ReLU, under large kernels
    p[2][3, 6] = p[4][9, 6] = big
    d = [dev(a) for a in [x] + p]
    got = sq.sq_fire_forward(*d)
    assert torch.equal(sq.sq_fire_forward_packed(*d, sq.sq_fire_pack_weights(d[5])), got)
    s = sq.sq_conv2d_forward(d[0], d[1], d[2], 1, 0, True).cpu().numpy()
    assert s[:, 5].min() > 0 and s[:, 6].max() == 0
    g = got.cpu().numpy()
    assert_within_rounding(g[:, :ce], oracle.conv2d(s, p[2], p[3], 1, 0, True), s, p[2], p[3], 0, "expand1x1")
    assert_within_rounding(g[:, ce:], oracle.conv2d(s, p[4], p[5], 1, 1, True), s, p[4], p[5], 1, "expand3x3")


@pytest.mark.parametrize("big", APART)
@pytest.mark.parametrize("first", [True, False])                           # the large layer before and after those that count
def test_classifier_sums_are_as_exact_as_their_own_terms(sq, big, first):
    n, cin, cout, h, w = 40, 256, 500, 13, 13
    rng = np.random.default_rng(9)
    x = synth.uniform01(rng, (n, cin, h, w))
    wt, b = synth.conv_params(rng, cout, cin, 1)
    at, zero = (3, 250) if first else (250, 3)
    x[:20, at], wt[:, at] = big, 0
    x[20:, zero], wt[7, zero] = 0, big
    x[:20, zero] = 0
    x[20:, at] = 0
    sq.sq_profile_begin(16)
    _, means = sq.sq_classifier_forward(dev(x), dev(wt), dev(b), want_means=True)
    assert any("k1s1_split_96+planesums" in r["name"] for r in sq.sq_profile_end())
    ref = oracle.conv2d(x, wt, b, 1, 0, True).astype(np.float64).mean(axis=(2, 3))
    terms = oracle.conv2d(np.abs(x), np.abs(wt), np.abs(b), 1, 0, False).astype(np.float64).mean(axis=(2, 3))
    err = np.abs(means.cpu().numpy() - ref)
    assert (err <= (3 * cin / 16 + h * w + 16) * 2.0 ** -24 * terms).all(), float((err / terms).max())


@pytest.mark.parametrize("big", APART)
@pytest.mark.parametrize("where", ["layer under zero kernels", "kernels over a zero layer", "image layer under zero kernels"])
def test_one_launch_first_layers_are_as_exact_as_their_own_terms(sq, big, where):
    """Layers that count for nothing, large and absent: the same probabilities but for rounding."""
    cfg = synth.config_squeezenet(seed=78, n=10)
    x, params = cfg["x"].copy(), [p.copy() for p in cfg["params"]]
    for c in (2, 40):                                    # the first and the second step that a wavefront adds
        if where == "layer under zero kernels":
            params[0][c], params[2][:, c] = np.abs(params[0][c]) * np.float32(big), 0
        elif where == "kernels over a zero layer":
            params[0][c], params[1][c], params[2][3, c] = -np.abs(params[0][c]), 0, big
        else:
            x[:, 1], params[0][:, 1] = big, 0
    run = lambda x, params: sq.sq_squeezenet_forward_packed(dev(x), params, sq.sq_pack_weights(params, sq.SQ_F32)).cpu().numpy().astype(np.float64)
    got = run(x, [dev(p) for p in params])
    for c in (2, 40):
        if where == "image layer under zero kernels":
            x[:, 1] = 0
        else:
            params[0][c], params[2][:, c] = 0, 0
    want = run(x, [dev(p) for p in params])
    assert np.abs(got / want - 1).max() <= 1e-5, float(np.abs(got / want - 1).max())


def test_first_layer_without_relu_keeps_nan(sq):
    rng = np.random.default_rng(6)
    x = synth.uniform01(rng, (2, 3, 40, 33))
    x[0, 1, 20, 9], x[1, 2, 3, 30] = np.nan, np.inf
    w, b = synth.conv_params(rng, 96, 3, 7)
    want = sq.sq_conv2d_forward_ex(dev(x), dev(w), dev(b), 2, 2, False, algo=sq.SQ_ALGO_DIRECT).cpu().numpy()
    got = sq.sq_conv2d_forward(dev(x), dev(w), dev(b), 2, 2, False).cpu().numpy()
    assert np.isnan(want).any() and np.isinf(want).any()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])


@pytest.mark.parametrize("csq,ce,w_", [(48, 64, 180), (48, 192, 260), (64, 64, 256), (64, 256, 176), (64, 32, 190)])
@pytest.mark.parametrize("n", [1, 3, 6])
def test_packed_fire_runs_the_kernels_of_the_unpacked_call_on_maps_of_any_width(sq, n, csq, ce, w_):
    """Rows too long for the split form's patch in LDS (and around that line): the packed call has the kernels of every form."""
    rng = np.random.default_rng(w_)
    x = synth.uniform01(rng, (n, 16, 5, w_))
    d = [dev(a) for a in [x, *synth.conv_params(rng, csq, 16, 1), *synth.conv_params(rng, ce, csq, 1), *synth.conv_params(rng, ce, csq, 3)]]
    packed = sq.sq_fire_pack_weights(d[5])
    results, names = [], []
    for call, more in ((sq.sq_fire_forward, ()), (sq.sq_fire_forward_packed, (packed,))):
        sq.sq_profile_begin(8)
        results.append(call(*d, *more))
        names.append([r["name"] for r in sq.sq_profile_end() if "transform" not in r["name"] and "split_kernels" not in r["name"]])
    assert names[0] == names[1]
    assert torch.equal(*results)


@pytest.mark.parametrize("n", [2, 3, 10, 33, 64])
def test_packed_network_prepares_no_expand_kernels_inside_the_call(sq, n):
    """Only conv10's kernels are prepared by the call itself, where it runs on split operands."""
    cfg = synth.config_squeezenet(seed=60, n=min(n, 4))
    params = [dev(p) for p in cfg["params"]]
    x = dev(cfg["x"]).repeat((n + 3) // 4, 1, 1, 1)[:n].contiguous()
    packed = sq.sq_pack_weights(params, sq.SQ_F32)
    before = packed.clone()
    sq.sq_profile_begin(128)
    got = sq.sq_squeezenet_forward_packed(x, params, packed)
    names = [r["name"] for r in sq.sq_profile_end()]
    assert not any("transform" in k for k in names), names
    assert [k for k in names if "split_kernels" in k] == (["conv10|split_kernels"] if n >= 16 else []), names
    assert torch.equal(packed, before)
    assert_close(got.cpu().numpy(), sq.sq_squeezenet_forward(x, params).cpu().numpy(), "packed and unpacked")
    # forms that a tuning hook asks for are not among the packed kernels
    for hook, forms in ((sq.lib.sq_tune_expand_pair, (1, 2, 3, 0)), (sq.lib.sq_tune_force_expand, (-3, -1))):
        default = -1 if hook is sq.lib.sq_tune_expand_pair else -2
        for form in forms:
            try:
                hook(form)
                forced, want = sq.sq_squeezenet_forward_packed(x, params, packed), sq.sq_squeezenet_forward(x, params)
            finally:
                hook(default)
            assert_close(forced.cpu().numpy(), want.cpu().numpy(), (hook, form))
    assert torch.equal(packed, before)


@pytest.mark.parametrize("n", [10, 16, 33, 64])
def test_taps_do_not_change_the_packed_network(sq, n):
    cfg = synth.config_squeezenet(seed=61, n=min(n, 4))
    params = [dev(p) for p in cfg["params"]]
    x = dev(cfg["x"]).repeat((n + 3) // 4, 1, 1, 1)[:n].contiguous()
    packed = sq.sq_pack_weights(params, sq.SQ_F32)
    probs, taps = sq.sq_squeezenet_forward_packed(x, params, packed, want_taps=True)
    assert torch.equal(sq.sq_squeezenet_forward_packed(x, params, packed), probs)
    assert torch.equal(taps["probs"], probs)
    want, wtaps = sq.sq_squeezenet_forward(x, params, want_taps=True)
    for k in wtaps:         # (activations of order one: sums of much larger terms that cancel would differ by 2^-24 of those)
        assert_close(taps[k].cpu().numpy(), wtaps[k].cpu().numpy(), k)


# where the split form is the faster one and where it is not: 3x3 layers of one round of short launches, few output layers over
# many input layers, 5x5 layers of any size; fire layers whose blocks of layers leave wavefronts idle
@pytest.mark.parametrize("n,cin,cout,k,h,w_,split", [(1, 16, 64, 3, 7, 7, False), (16, 64, 64, 3, 14, 14, False), (1, 64, 256, 3, 28, 28, False), (16, 64, 64, 3, 56, 56, False),
                                                     (4, 384, 64, 3, 56, 56, False), (4, 8, 384, 3, 56, 56, False), (7, 256, 384, 3, 13, 13, True), (4, 128, 256, 3, 27, 27, True),
                                                     (1, 8, 40, 5, 7, 7, True), (16, 96, 256, 5, 27, 27, True), (2, 384, 16, 5, 40, 41, True)])
def test_layers_run_in_the_faster_form(sq, n, cin, cout, k, h, w_, split):
    rng = np.random.default_rng(n + cin)
    x = synth.normal01(rng, (n, cin, h, w_))
    w, b = synth.conv_params(rng, cout, cin, k)
    pad = k // 2
    names, results = [], []
    for mode in (-1, 0, 1):
        sq.lib.sq_tune_conv_split(mode)
        sq.sq_profile_begin(8)
        results.append(sq.sq_conv2d_forward_ws(dev(x), dev(w), dev(b), 1, pad, True).cpu().numpy())
        names.append([r["name"] for r in sq.sq_profile_end()])
    assert [any("_split_" in s for s in v) for v in names] == [split, False, True], names
    for r in results:
        assert_close(r, results[1], names)


@pytest.mark.parametrize("n,csq,ce,h,w_,split", [(16, 48, 192, 27, 27, True), (64, 64, 256, 27, 27, True), (3, 64, 256, 13, 13, True), (48, 64, 96, 40, 40, False), (20, 64, 96, 56, 56, False)])
def test_fire_layers_run_in_the_faster_form(sq, n, csq, ce, h, w_, split):
    sq.lib.sq_tune_conv_split(-1)
    rng = np.random.default_rng(n)
    x = torch.rand((n, 16, h, w_), device="cuda")
    d = [x] + [dev(a) for a in [*synth.conv_params(rng, csq, 16, 1), *synth.conv_params(rng, ce, csq, 1), *synth.conv_params(rng, ce, csq, 3)]]
    names, results = [], []
    for call, more in ((sq.sq_fire_forward, ()), (sq.sq_fire_forward_packed, (sq.sq_fire_pack_weights(d[5]),))):
        sq.sq_profile_begin(8)
        results.append(call(*d, *more))
        names.append([r["name"] for r in sq.sq_profile_end()])
    assert [any("_split_" in s for s in v) for v in names] == [split, split], names
    assert torch.equal(*results)
    sq.lib.sq_tune_conv_split(0)
    assert_close(results[0].cpu().numpy(), sq.sq_fire_forward(*d).cpu().numpy(), names)


def test_what_first_layer_kernels_lose_does_not_add_up_over_the_image(sq):
    """Two f16 values hold a kernel value up to its last bit, and that error is the same at every pixel: the plane means of the
    layer must be off by clearly less than kernels rounded one by one make them (r0, from the kernels themselves)."""
    rng = np.random.default_rng(21)
    x = synth.uniform01(rng, (4, 3, 112, 112))
    w, _ = synth.conv_params(rng, 96, 3, 7)
    top = 2.0 ** (13 - np.floor(np.log2(np.abs(w).max(axis=(1, 2, 3), keepdims=True))))
    v = w.astype(np.float64) * top
    hi = v.astype(np.float16).astype(np.float64)
    lo = ((v - hi) * 2048).astype(np.float16).astype(np.float64) / 2048
    pd = lambda k: torch.nn.functional.conv2d(dev(x).double(), torch.from_numpy(np.ascontiguousarray(k)).cuda(), None, 2, 2).mean((0, 2, 3))
    r0 = pd((hi + lo - v) / top).pow(2).mean().sqrt().item()
    got = sq.sq_conv2d_forward(dev(x), dev(w), None, 2, 2, False).double().mean((0, 2, 3))
    off = (got - pd(w.astype(np.float64))).pow(2).mean().sqrt().item()
    assert 0 < off < 0.6 * r0, (off, r0)
