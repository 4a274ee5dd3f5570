"""The next operand's maximum on tiles that reach past the output grid, for every
way an epilogue masks them: orders up to 64 a 64-channel block at a time, the orders
that span several blocks (128, 192, 320), their cancelled and untransformed forms; on
the kernels of small launches, the persistent window kernel and the general one.

Two inputs per launch.  One makes the pixels past the grid dominate: constant codes
without padding and a bias that cancels the sum, so every output is small, while a
pixel past the grid, whose window reaches out of the image, keeps most of the bias.
The other puts one spike per sample, over all samples at every place of the ragged
tile, so a valid pixel that a mask drops is the sample's maximum.  The maximum has to
give the scale and the codes that the two-pass quantizer derives from the stored output
(the same fp32 transform), bit for bit, with the output stored and without it.
"""
import pytest
import torch

from paper_2608_01653_amd import hatq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hatq.load()
    torch.cuda.init()


GEOM = {  # (h, w, k, stride, transposed, samples)
    "s2-small": (21, 41, 5, 2, False, 5),
    "s2-large": (21, 41, 5, 2, False, 300),
    "s2-k4-large": (20, 39, 4, 2, False, 300),
    "s1": (11, 21, 3, 1, False, 5),
    "s1-large": (11, 21, 3, 1, False, 300),
    "1x1": (9, 19, 1, 1, False, 5),
    "1x1-large": (9, 19, 1, 1, False, 300),
    "T": (5, 9, 5, 2, True, 5),
}
ORDERS = [  # (cout, form, hblock, next block, HATQ_PAIRED)
    (192, "DH", 64, 192, False), (192, "WH", 192, 192, False), (192, "WH", 192, 1, False),
    (192, "WH", 64, 192, False), (192, "WH", 192, 64, False),
    (320, "DH", 64, 320, False), (320, "WH", 320, 1, False), (320, "WH", 320, 320, False),
    (128, "DH", 64, 128, False), (128, "WH", 128, 1, False), (128, "WH", 128, 128, False),
    (256, "WH", 64, 128, False), (256, "WH", 128, 64, False),
    (192, "WH", 64, 64, True), (192, "WH", 64, 64, False), (192, "DH", 64, 64, False), (320, "WH", 64, 1, False),
    (128, "WH", 16, 32, False), (64, "DH", 64, 1, False),
]


def _check(layer, q, nb, paired):
    n = q.shape[0]
    sx = torch.ones(n, device="cuda")
    m, mo = torch.full((n,), -1.0, device="cuda"), torch.full((n,), -1.0, device="cuda")
    y = hatq.hatq_conv_int8(layer, q, sx, hatq.HATQ_OUT_F32, next_hblock=nb, next_absmax=m, paired=paired)
    hatq.hatq_conv_int8(layer, q, sx, hatq.HATQ_OUT_F32, next_hblock=nb, next_absmax=mo, absmax_only=True,
                        paired=paired)
    q2, s2 = hatq.hatq_fwht_quant_act(y, nb)
    q1, s1 = hatq.hatq_fwht_quant_act(y, nb, absmax=m)
    assert torch.equal(s1, s2) and torch.equal(q1, q2)
    # (paired, without the output: the maximum of z, which B_next y equals but for
    # the rounding of two six-stage fp32 transforms, 2 * 6 * 2^-24 of sum |z| <= 64 max |z|)
    if paired:
        assert bool(((mo - m).abs() <= 64 * 12 * 2.0 ** -24 * m).all())
    else:
        assert torch.equal(mo, m)
    return y


@pytest.mark.parametrize("geom", list(GEOM))
@pytest.mark.parametrize("c", ORDERS, ids=[f"{c[0]}-{c[1]}{c[2]}to{c[3]}{'p' if c[4] else ''}" for c in ORDERS])
def test_ragged_maxima(c, geom):
    cout, form, hb, nb, paired = c
    h, w, k, s, tr, n = GEOM[geom]
    if tr and paired:
        pytest.skip("the pairing is that of a stack's regular layers")
    cin = 64
    g = torch.Generator("cuda").manual_seed(17)
    wt = torch.randn((cin, cout, k, k) if tr else (cout, cin, k, k), device="cuda", generator=g) * 0.05
    d = hatq.desc(cin, cout, k, s, 0, hb, tr, 0)
    small = 1e-3 * torch.randn(cout, device="cuda", generator=g)
    layer = hatq.hatq_prepare_weights(d, form, wt, small)

    # one spike per sample, at places spread over the image
    q = torch.zeros((n, h * w, cin), dtype=torch.int8, device="cuda")
    at = (torch.arange(n, device="cuda") * (h * w - 1)) // max(n - 1, 1)
    q[torch.arange(n, device="cuda"), at] = torch.randint(-127, 128, (n, cin), dtype=torch.int8, device="cuda",
                                                          generator=g)
    q = q.view(n, h, w, cin)
    _check(layer, q, nb, paired)
    # and at every place of the last rows and columns, where the ragged tiles are
    for pos in ((h - 1, w - 1), (h - 1, 0), (0, w - 1), (h - k, w - k)):
        e = torch.zeros((n, h, w, cin), dtype=torch.int8, device="cuda")
        e[:, pos[0], pos[1]] = q.view(n, h * w, cin)[torch.arange(n, device="cuda"), at]
        _check(layer, e, nb, paired)

    # constant codes, the sum cancelled by the bias
    if not tr:
        q = torch.randint(-127, 128, (1, 1, 1, cin), dtype=torch.int8, device="cuda", generator=g).expand(
            n, h, w, cin).contiguous()
        zero = hatq.hatq_prepare_weights(d, form, wt, torch.zeros(cout, device="cuda"))
        y0 = hatq.hatq_conv_int8(zero, q, torch.ones(n, device="cuda"), hatq.HATQ_OUT_F32)
        b = -y0[0, 0, 0].contiguous()
        y = _check(hatq.hatq_prepare_weights(d, form, wt, b + small), q, nb, paired)
        assert float(y.abs().max()) < 0.05 * float(b.abs().max())
