"""The kernels of small launches (tiles of 4 or 8 output rows x 16 columns by 64
output channels, the contraction divided over the waves of a block) and of stride-1
and transposed ones (tiles of 8 rows, a wave per 64 channels of a phase): ragged tiles
in both directions, one to five input chunks (all of the window in LDS, two or
three buffers, or one refilled chunk by chunk), kernel sizes up to its spans, the
phases of transposed convolutions (unequal ones without output padding), and the
launches on both sides of the limits of its dispatch.  Sums are whole numbers, so
every path gives the same accumulators, outputs, maxima and codes bit for bit.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host
from paper_2608_01653_amd import hatq, synth
from test_gpu_parity import _layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hatq.load()
    torch.cuda.init()


GEOM = [  # (n, h, w, cin, cout, k, stride, pad, transposed, out_pad, form, hblock)
    (1, 1, 1, 64, 64, 1, 1, 0, False, 0, "DH", 64),        # one point
    (2, 3, 17, 128, 128, 1, 1, 0, False, 0, "WH", 64),
    (1, 9, 33, 320, 64, 3, 1, 1, False, 0, "DH", 16),      # five chunks
    (1, 5, 16, 64, 128, 7, 1, 3, False, 0, "DH", 64),      # span 7
    (1, 11, 20, 64, 64, 8, 1, 2, False, 0, "WH", 16),      # even kernel, span 8
    (1, 8, 15, 64, 192, 2, 1, 0, False, 0, "DH", 64),
    (1, 15, 31, 192, 320, 5, 2, 2, False, 0, "WH", 64),
    (1, 16, 34, 320, 192, 5, 2, 2, False, 0, "DH", 64),    # five chunks in three buffers
    (2, 7, 65, 128, 64, 6, 2, 2, False, 0, "WH", 16),      # the widest stride-2 span
    (1, 18, 33, 64, 192, 4, 2, 1, False, 0, "DH", 64),
    (1, 6, 9, 256, 256, 3, 2, 0, False, 0, "DH", 64),
    (1, 3, 5, 192, 192, 5, 2, 2, True, 1, "DH", 64),
    (1, 4, 17, 128, 64, 3, 2, 1, True, 0, "WH", 64),       # phases of unequal sizes
    (2, 5, 7, 64, 192, 4, 2, 1, True, 0, "DH", 64),
    (1, 9, 16, 320, 64, 6, 2, 2, True, 0, "WH", 16),
]
IDS = [f"{c[1]}x{c[2]}-{c[3]}to{c[4]}-k{c[5]}s{c[6]}{'T' if c[8] else ''}-{c[10]}{c[11]}" for c in GEOM]


@pytest.mark.parametrize("c", GEOM, ids=IDS)
def test_accumulators_exact(orc, c):
    n, h, w, cin, cout, k, s, p, tr, op, form, hb = c
    rng, wt, b, ref, layer = _layer(orc, c, 301)
    xq = synth.int8_codes(rng, (n, h, w, ref.cin_p))
    acc = orc.conv_int8(xq, ref.wq, stride=s, pad=p, transposed=tr, out_pad=op)
    got = hatq.hatq_conv_int8(layer, dev(xq), torch.ones(n, device="cuda"), hatq.HATQ_OUT_I32)
    assert np.array_equal(host(got), acc)


# Batches of small samples: 1, some, and many of them, so that the launches take
# the 4-row tiles, the 8-row tiles and the large-launch kernels of each geometry.
BATCH = [
    (9, 31, 192, 192, 5, 2, 2, False, 0, "DH", 64),
    (9, 31, 192, 320, 5, 2, 2, False, 0, "WH", 64),
    (17, 20, 128, 192, 4, 2, 1, False, 0, "WH", 64),
    (17, 20, 64, 192, 6, 2, 2, False, 0, "DH", 64),
    (9, 17, 64, 128, 5, 2, 2, False, 0, "WH", 64),
    (9, 17, 192, 192, 1, 1, 0, False, 0, "DH", 64),
    (5, 18, 64, 320, 1, 1, 0, False, 0, "WH", 64),
    (9, 17, 128, 64, 3, 1, 1, False, 0, "WH", 64),
    (5, 9, 192, 192, 5, 2, 2, True, 1, "WH", 64),
    (4, 9, 64, 64, 3, 2, 1, True, 0, "DH", 64),
    (3, 5, 320, 192, 5, 2, 2, True, 1, "WH", 64),      # every chunk of five in LDS
    (9, 17, 64, 192, 3, 1, 1, False, 0, "DH", 64),     # three units
    (9, 17, 64, 320, 3, 1, 1, False, 0, "WH", 64),     # five units: some waves take two
    (9, 17, 64, 256, 1, 1, 0, False, 0, "DH", 64),
    (9, 17, 64, 192, 1, 2, 0, False, 0, "WH", 64),     # stride 2, k < 4: back to the large kernels sooner
    (9, 17, 128, 128, 1, 2, 0, False, 0, "DH", 64),
    (9, 17, 64, 320, 2, 2, 0, False, 0, "DH", 64),
    (9, 17, 64, 192, 3, 2, 1, False, 0, "WH", 64),
    (9, 17, 64, 64, 1, 1, 0, False, 0, "WH", 16),
    (4, 9, 64, 192, 3, 2, 1, True, 0, "WH", 64),       # transposed, a first phase of one tap
    (4, 9, 64, 320, 2, 2, 0, True, 0, "DH", 64),
]


@pytest.mark.parametrize("c", BATCH, ids=[f"{c[2]}to{c[3]}-k{c[4]}s{c[5]}{'T' if c[7] else ''}-{c[9]}" for c in BATCH])
@pytest.mark.parametrize("next_b", [1, 64])
def test_launch_sizes_agree(c, next_b):
    h, w, cin, cout, k, s, p, tr, op, form, hb = c
    rng = np.random.default_rng(302)
    wt, b = synth.layer_params(rng, cin, cout, k, tr)
    layer = hatq.hatq_prepare_weights(hatq.desc(cin, cout, k, s, p, hb, tr, op), form, dev(wt), dev(b))
    n = 420
    g = torch.Generator("cuda").manual_seed(5)
    xq = torch.randint(-127, 128, (n, h, w, cin), dtype=torch.int8, device="cuda", generator=g)
    sx = torch.rand(n, device="cuda", generator=g) + 0.5

    def run(q, sc):
        m = torch.full((q.shape[0],), -1.0, device="cuda")
        y = hatq.hatq_conv_int8(layer, q, sc, hatq.HATQ_OUT_F32, next_hblock=next_b, next_absmax=m)
        yq, sq = hatq.hatq_conv_int8_requant(layer, q, sc, next_b, next_absmax=m)
        t, _ = hatq.hatq_int_transition_params(layer, 1.0, 4000.0, next_b)
        return [m, y, yq, sq, hatq.hatq_conv_int8_int_transition(layer, q, next_b, t),
                hatq.hatq_conv_int8(layer, q, sc, hatq.HATQ_OUT_I32)]

    big = run(xq, sx)
    for i, cnt in ((0, 1), (7, 60), (300, 120)):
        part = run(xq[i:i + cnt].contiguous(), sx[i:i + cnt].contiguous())
        for a, e in zip(part, big):
            assert torch.equal(a, e[i:i + cnt])
    # the maxima and codes are those of the output
    q2, s2 = hatq.hatq_fwht_quant_act(big[1], next_b, absmax=big[0])
    q3, s3 = hatq.hatq_fwht_quant_act(big[1], next_b)
    assert torch.equal(s2, s3) and torch.equal(big[3], s2) and torch.equal(big[2], q2)


# Affine activations on the persistent window kernel (several tiles per block, most
# at the image's border: a tap's weight sums staged per tile) and on the kernel of
# small launches: a batch against parts of it, bit for bit, and the 64-bit sums of
# the centered codes on the first sample.
@pytest.mark.parametrize("form", ["DH", "WH"])
def test_affine_launch_sizes_agree(orc, form):
    n, h, w, cin, cout = 150, 18, 21, 64, 192
    rng = np.random.default_rng(303)
    wt, b = synth.layer_params(rng, cin, cout, 5)
    ref = orc.prepare_weights(wt, b, cin=cin, cout=cout, k=5, stride=2, pad=2, form=form, hblock=64)
    layer = hatq.hatq_prepare_weights(hatq.desc(cin, cout, 5, 2, 2, 64), form, dev(wt), dev(b))
    tap = hatq.hatq_weight_tapsums(layer)
    x = torch.randn((n, h, w, cin), device="cuda", generator=torch.Generator("cuda").manual_seed(9)) + 0.7
    q, s, z = hatq.hatq_fwht_quant_act_affine(x, 64 if form == "DH" else 1)
    for mode in (hatq.HATQ_OUT_F32, hatq.HATQ_OUT_I32):
        big = hatq.hatq_conv_int8_affine(layer, q, s, z, tap, out_mode=mode)
        for i, cnt in ((0, 3), (100, 50)):
            part = hatq.hatq_conv_int8_affine(layer, q[i:i + cnt].contiguous(), s[i:i + cnt].contiguous(),
                                              z[i:i + cnt].contiguous(), tap, out_mode=mode)
            assert torch.equal(part, big[i:i + cnt])
    acc = orc.conv_int8(host(q[:1]), ref.wq, stride=2, pad=2, zx=host(z[:1]))
    assert np.array_equal(host(big[:1]), acc)


# The reductions' block sizes: one sample on both sides of the limit, odd counts of
# items per block, and a batch of more samples than blocks; the absmax and minimum
# and maximum against torch's (blocks of 1: exact), the order-64 ones against the
# activation kernel's own codes (no code beyond the scale, and one that reaches it).
@pytest.mark.parametrize("shape", [(1, 16, 16, 4095 * 4), (1, 127, 129, 64), (1, 128, 128, 64), (1, 129, 131, 64),
                                   (3, 61, 67, 192), (700, 5, 3, 64)])
@pytest.mark.parametrize("b", [1, 64])
def test_reduction_block_sizes(shape, b):
    if shape[3] % b:
        shape = shape[:3] + (shape[3] // 64 * 64,)
    n = shape[0]
    x = torch.randn(shape, device="cuda", generator=torch.Generator("cuda").manual_seed(11))
    for i in range(n):   # the largest value at an end of the sample
        x[i].view(-1)[0 if i % 2 else -1] = 9.0 if i % 3 else -9.0
    amax, _ = hatq.hatq_range_expansion(x, b)
    q, s = hatq.hatq_fwht_quant_act(x, b)
    qa, sa, za = hatq.hatq_fwht_quant_act_affine(x, b)
    lim = x.abs().amax(dim=(1, 2, 3))
    assert torch.equal(amax[:n], lim)
    assert torch.equal(s, amax[n:] / torch.full((1,), 127.0, device="cuda"))
    assert torch.equal(q.abs().amax(dim=(1, 2, 3)), torch.full((n,), 127, dtype=torch.int8, device="cuda"))
    if b == 1:
        assert torch.equal(amax[n:], lim)
        hi, lo = x.amax(dim=(1, 2, 3)).clamp_min(0), (-x).amax(dim=(1, 2, 3)).clamp_min(0)
        assert torch.equal(sa, (hi + lo) / torch.full((1,), 255.0, device="cuda"))
    assert bool((qa.amax(dim=(1, 2, 3)) >= 126).all()) and bool((qa.amin(dim=(1, 2, 3)) <= -127).all())


# The transformed maxima of the reductions, exactly: small whole numbers (every
# partial sum of the transform is exact in fp32), the transform a float64 product by the
# order's matrix, samples on both sides of each limit of the launch shapes (threads,
# blocks, own slots, forward order, one item per quad), and the largest positive and
# negative values in the first item, the last and one in between.
@pytest.mark.parametrize("n,b,pixels", [(n, b, p) for n in (1, 3) for b, p in (
    (16, 4133), (64, 16801), (128, 17419), (192, 16567), (320, 16453), (64, 5003), (128, 1201), (192, 2503), (320, 907))]
    + [(1, 64, 67), (2, 128, 6007), (2, 192, 1511), (17, 320, 2203), (131, 64, 2503), (131, 128, 4201)])
def test_reductions_transformed(orc, n, b, pixels):
    c = 64 * 5 if b == 16 else b
    H = torch.from_numpy(orc.activation_transform(np.eye(b, dtype=np.float32).reshape(1, 1, b, b), b)
                         .reshape(b, b).astype(np.float64)).cuda()   # row i: the transform of unit vector i
    g = torch.Generator("cuda").manual_seed(21)
    base = torch.randint(-3, 4, (n, 1, pixels, c), device="cuda", generator=g).float()
    items = pixels * c // b
    for hi, lo in ((0, items - 1), (items - 1, 0), (items // 2 + 1, items // 3), (items - 2, 1)):
        x = base.clone()
        flat = x.view(n, items, b)
        for i in range(n):   # aligned with a row of the transform: b times the entry's size
            col = (5 * i + 3) % b
            flat[i, hi] = 20.0 * torch.sign(H[:, col]).float()
            flat[i, lo] = -17.0 * torch.sign(H[:, col]).float()
        S = (x.view(-1, b).double() @ H).view(n, -1)
        am = S.abs().amax(1).float()
        assert torch.equal(am.double(), S.abs().amax(1)) and int((S.abs() == S.abs().amax(1, True)).sum()) == n
        amax, _ = hatq.hatq_range_expansion(x, b)
        assert torch.equal(amax[n:], am) and torch.equal(amax[:n], x.abs().amax(dim=(1, 2, 3)))
        q, s = hatq.hatq_fwht_quant_act(x, b)
        assert torch.equal(s, am / torch.full((1,), 127.0, device="cuda"))
        qa, sa, za = hatq.hatq_fwht_quant_act_affine(x, b)
        top, bot = S.amax(1).float(), (-S).amax(1).float()
        want = (top + bot) / torch.full((1,), 255.0, device="cuda")
        assert torch.equal(sa, want)
        assert torch.equal(za, (torch.round(bot / want) - 128).clamp(-128, 127).int())


# Orders that span a layer's columns (192, 320): many small samples (the large-launch
# kernels) against few of them (the kernel of small launches on all columns).
@pytest.mark.parametrize("cout,form,hb,nb", [(192, "DH", 64, 192), (192, "WH", 192, 192), (192, "WH", 192, 1),
                                             (320, "WH", 320, 1), (320, "DH", 64, 320)])
def test_wide_order_launch_sizes_agree(cout, form, hb, nb):
    rng = np.random.default_rng(304)
    wt, b = synth.layer_params(rng, 128, cout, 5)
    layer = hatq.hatq_prepare_weights(hatq.desc(128, cout, 5, 2, 2, hb), form, dev(wt), dev(b))
    n = 260
    g = torch.Generator("cuda").manual_seed(6)
    xq = torch.randint(-127, 128, (n, 11, 35, 128), dtype=torch.int8, device="cuda", generator=g)
    sx = torch.rand(n, device="cuda", generator=g) + 0.5

    def run(q, sc):
        m = torch.full((q.shape[0],), -1.0, device="cuda")
        y = hatq.hatq_conv_int8(layer, q, sc, hatq.HATQ_OUT_F32, next_hblock=nb, next_absmax=m)
        m2 = torch.full((q.shape[0],), -1.0, device="cuda")
        hatq.hatq_conv_int8(layer, q, sc, hatq.HATQ_OUT_F32, next_hblock=nb, next_absmax=m2, absmax_only=True)
        yq, sq = hatq.hatq_conv_int8_requant(layer, q, sc, nb, next_absmax=m)
        return [m, y, m2, yq, sq]

    big = run(xq, sx)
    for i, cnt in ((0, 1), (37, 20), (200, 60)):
        for a, e in zip(run(xq[i:i + cnt].contiguous(), sx[i:i + cnt].contiguous()), big):
            assert torch.equal(a, e[i:i + cnt])
