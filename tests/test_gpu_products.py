"""The block's product at the edges of its tile choice: one row, partial row
tiles, each tile size, one k-stage up to more than the ring holds, odd counts,
against fp64 within the rounding of fp32 sums (K ulps of sum |a w|)."""
import numpy as np
import pytest
import torch

from gpu_common import log
from paper_2001_04451_amd import lsh

pytestmark = pytest.mark.gpu


# N = 128: only the smaller tiles; 64 x 64 tiles below 256 tiles of 128, 128 x 128
# from there, 256 x 256 from 192 of them (M = 12033, N = 1024: 48 x 4, the last
# row tile of one row).  K / 64 stages: 1, 2, 3, 5, 7.
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (63, 128, 128), (65, 384, 320), (300, 256, 448), (4097, 1024, 64),
                                   (5000, 896, 192), (12033, 1024, 64), (12033, 1024, 128), (12200, 1024, 448)])
def test_linear_tiles(M, N, K):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g = torch.Generator().manual_seed(M + N + K)
    a = torch.randn(M, K, generator=g).bfloat16().cuda()
    w = torch.randn(N, K, generator=g).bfloat16().cuda()
    bias = torch.randn(N, generator=g).cuda()
    resid = torch.randn(M, N, generator=g).cuda()
    log("linear", M, N, K)
    exact = a.double() @ w.double().t() + bias.double()
    bound = (K + 2) * 2.0 ** -23 * (a.double().abs() @ w.double().abs().t() + bias.double().abs())
    out = lsh.linear_bf16(a, w, bias=bias, resid=resid, sign=-1.0)
    err = (out.double() - (resid.double() - exact)).abs()
    assert (err <= bound + 2.0 ** -23 * (resid.abs() + exact.abs())).all()
    relu = lsh.linear_bf16(a, w, bias=bias, relu_bf16=True)
    assert ((relu.double() - exact.relu()).abs() <= bound + 2.0 ** -8 * exact.abs()).all()
