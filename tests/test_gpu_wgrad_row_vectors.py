"""The float32 weight gradient by 8-row vectors (at most 32 output channels, 4n but
not 8n input channels) at its edges: tiles of one vector, rows that end half way
through a vector, reductions that end in the middle of a pair, a K tile or a
split."""
import ctypes as C

import pytest
import torch

from paper_1911_00357_amd import _lib as L
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


class Geo(C.Structure):
    _fields_ = [(n, C.c_int) for n in "B H W C Ho Wo Co KH KW stride pad".split()]


class Epi(C.Structure):
    _fields_ = [("C", C.c_void_p), ("ldc", C.c_int), ("bias", C.c_void_p), ("alpha", C.c_float), ("relu", C.c_int),
                ("accumulate", C.c_int), ("partial", C.c_void_p)] + \
               [(n, C.c_int) for n in "rq rwq rs1 rs2 rs3 r0 gm_p gm_cg gm_split_only act".split()]


def wgrad(geo, x, dy):
    out = torch.full((geo.Co, geo.KH, geo.KW, geo.C), float("nan"), device=DEV)
    part = torch.empty(16 << 20, device=DEV)
    f = L.lib()._Z15gemm_conv_wgradiRK7ConvGeoPKfS3_3EpimPfP12ihipStream_t
    f.restype = None
    e = Epi(out.data_ptr(), out[0].numel(), None, 1.0, 0, 0, None, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0)
    f(C.c_int(0), C.byref(geo), C.c_void_p(x.data_ptr()), C.c_void_p(dy.data_ptr()), e, C.c_size_t(64 << 20),
      C.c_void_p(part.data_ptr()), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return out


# frames, input size, input channels, output channels, kernel, stride
@pytest.mark.parametrize("case", [(1, 3, 4, 8, 5, 1), (1, 7, 12, 8, 3, 2), (2, 9, 4, 24, 7, 2), (3, 15, 20, 32, 3, 1),
                                  (5, 32, 4, 32, 7, 2), (7, 16, 28, 16, 3, 1)], ids=lambda c: "x".join(map(str, c)))
def test_weight_gradient(P, case):
    B, hw, ci, co, k, st = case
    print(f"float32 weight gradient {case}", flush=True)
    ho = (hw + 2 * (k // 2) - k) // st + 1
    geo = Geo(B, hw, hw, ci, ho, ho, co, k, k, st, k // 2)
    gen = torch.Generator().manual_seed(hw + ci)
    n = B * hw * hw * ci
    x = torch.randn(B, hw, hw, ci, generator=gen)
    dy = torch.randn(B, ho, ho, co, generator=gen)
    xd = torch.zeros(n + 1, device=DEV)
    got = wgrad(geo, x.to(DEV), dy.to(DEV))
    # the scalar loaders, taken where the input lies between 16-byte addresses: the same sums in the same order
    xd[1:] = x.reshape(-1).to(DEV)
    assert torch.equal(got, wgrad(geo, xd[1:], dy.to(DEV)))

    def ref(x, dy):
        w = torch.nn.grad.conv2d_weight(x.double().permute(0, 3, 1, 2), (co, ci, k, k), dy.double().permute(0, 3, 1, 2),
                                        stride=st, padding=k // 2)
        return w.permute(0, 2, 3, 1)
    # a sum of B ho ho float32 products: at most that many roundings of the sum of magnitudes
    bound = (B * ho * ho + 1) * 2.0 ** -24 * ref(x.abs(), dy.abs())
    assert ((got.cpu().double() - ref(x, dy)).abs() <= bound).all()
