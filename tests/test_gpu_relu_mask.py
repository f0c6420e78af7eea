"""The GroupNorm backward's recomputed ReLU mask where it is decided by the last
bit: the launchers called directly, every channel's shift chosen so that the
value before the ReLU of one of its pixels is the rounding error of that pixel's
product.  The backward that forms the mask again must then equal the one that
reads the saved output bit for bit, and the other form's mask must not."""
import ctypes as C

import pytest
import torch

from paper_1911_00357_amd import _lib as L
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

V, I, F = C.c_void_p, C.c_int, C.c_float
F2, F4, S_ = "P15HIP_vector_typeIfLj2EE", "PS2_IfLj4EE", "P12ihipStream_t"
NONE, OUT, APPLY, FUSED = range(4)   # GnMask


def _fn(name):
    f = getattr(L.lib(), name)
    f.restype = None
    return f


def gn_forward(form, y, G, gamma, beta, relu, chw):
    """Output and statistics of the three-launch (APPLY) or one-launch (FUSED) form."""
    B, P, Ch = y.shape
    out, stats = torch.full_like(y, float("nan")), torch.empty(B * G, 2, device=DEV)
    s = V(torch.cuda.current_stream().cuda_stream)
    p = lambda t: V(t.data_ptr())
    if form == APPLY:
        S = max(1, min(32, P // 64))
        part = torch.empty(B * S * Ch, 4, device=DEV)
        _fn(f"_Z17launch_gn_forwardPKfiiiifS0_S0_S0_iPfi{F2}{F4}i{S_}")(
            p(y), I(B), I(P), I(Ch), I(G), F(1e-5), p(gamma), p(beta), None, I(relu), p(out), I(chw), p(stats),
            p(part), I(S), s)
    else:
        _fn(f"_Z15launch_gn_fusedPKfimPfiiiifS0_S0_S0_iS1_i{F2}{S_}iS1_iiPK8GnSecond")(
            p(y), I(1), C.c_size_t(0), None, I(B), I(P), I(Ch), I(G), F(1e-5), p(gamma), p(beta), None, I(relu),
            p(out), I(chw), p(stats), s, I(0), None, I(0), I(0), None)
    torch.cuda.synchronize()
    return out, stats


def gn_backward(mask, dout, out, y, G, stats, gamma, beta, chw):
    B, P, Ch = y.shape
    S = max(1, min(32, P // 64))
    dy, dg, db = torch.full_like(y, float("nan")), torch.empty(Ch, device=DEV), torch.empty(Ch, device=DEV)
    bpart, coef = torch.empty(B * S * Ch, 2, device=DEV), torch.empty(B * G, 2, device=DEV)
    p = lambda t: V(t.data_ptr())
    _fn("_Z18launch_gn_backwardPKfS0_6GnMaskiS0_iiiiPK15HIP_vector_typeIfLj2EES0_S0_PfS6_S6_S6_PS3_S7_iP12ihipStream_t")(
        p(dout), p(out), I(mask), I(chw), p(y), I(B), I(P), I(Ch), I(G), p(stats), p(gamma), p(beta), p(dy), None,
        p(dg), p(db), p(bpart), p(coef), I(S), V(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return dy, dg, db


# images, pixels, channels, groups: one pixel (1x1 maps), an odd map, several
# pixel chunks, the 256- and 1024-thread one-launch blocks, 4 to 64 channels a group
SHAPES = [(3, 1, 128, 2), (2, 49, 64, 16), (5, 64, 64, 2), (2, 200, 64, 4), (1, 1024, 128, 8)]


@pytest.mark.parametrize("chw", [0, 1], ids=["nhwc", "chw"])
@pytest.mark.parametrize("form", [APPLY, FUSED], ids=["apply", "fused"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_mask_is_the_saved_outputs_to_the_last_bit(P, shape, form, chw):
    B, Px, Ch, G = shape
    print(f"recomputed mask {shape} form {form} chw {chw}", flush=True)
    gen = torch.Generator().manual_seed(Px + Ch + form)
    y = (torch.randn(B, Px, Ch, generator=gen) * 2 + 0.5).to(DEV)
    dout = torch.randn(B, Px, Ch, generator=gen).to(DEV)     # read as [B][Ch][Px] with chw
    gamma = (torch.rand(Ch, generator=gen) + 0.5).mul(torch.randint(0, 2, (Ch,), generator=gen) * 2 - 1).to(DEV)
    zero = torch.zeros(Ch, device=DEV)
    # the value with no shift is the rounded product; minus that as the shift
    # leaves the product's rounding error, of either sign, at the chosen pixel
    v, _ = gn_forward(form, y, G, gamma, zero, 0, 0)
    b, q = torch.randint(0, B, (Ch,), generator=gen), torch.randint(0, Px, (Ch,), generator=gen)
    c = torch.arange(Ch)
    beta = -v[b.to(DEV), q.to(DEV), c.to(DEV)].contiguous()
    out, stats = gn_forward(form, y, G, gamma, beta, 1, chw)
    at = (b * Ch + c) * Px + q if chw else (b * Px + q) * Ch + c
    border = out.reshape(-1)[at.to(DEV)]
    # |product - its rounding| <= 2^-24 |product|
    assert (border.abs() <= 2.0 ** -24 * beta.abs()).all()
    assert 0 < int((border > 0).sum()) < Ch                  # both sides of the border are there
    ref = gn_backward(OUT, dout, out, y, G, stats, gamma, beta, chw)
    got = gn_backward(form, dout, out, y, G, stats, gamma, beta, chw)
    other = gn_backward(APPLY + FUSED - form, dout, out, y, G, stats, gamma, beta, chw)
    assert all(torch.isfinite(t).all() for t in ref)
    for name, r, g in zip(("dy", "dgamma", "dbeta"), ref, got):
        assert torch.equal(r, g), name
    assert not torch.equal(ref[2], other[2]), "the other form's mask cannot be told apart here"
