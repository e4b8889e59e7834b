"""The block's product at the edges of its tile choice: one row, partial row
tiles, each tile size, one k-stage up to more than the ring holds, odd counts,
against fp64 within the rounding of fp32 sums (K ulps of sum |a w|)."""
import numpy as np
import pytest
import torch

from gpu_common import log
from oracle import block as OB
from paper_2001_04451_amd import lsh
from paper_2001_04451_amd import workloads as W

pytestmark = pytest.mark.gpu


# N = 128: only the smaller tiles; 64 x 64 tiles below 256 tiles of 128, 128 x 128 from there (M = 12033, N = 1024:
# 95 x 8, the last row tile of one row).  K / 64 stages: 1, 2, 3, 5, 7.
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


# 256 x 256 tiles on either side of where they begin (218 tiles from K = 576, 256 or 252 at K = 512, 192 from K = 1536;
# the last row tile of one row): K / 64 = 8, 9, 11 and 24 stages.
@pytest.mark.parametrize("M,N,K", [(16129, 1024, 512), (15873, 1024, 512), (15617, 1024, 512), (13825, 1024, 576),
                                   (13569, 1024, 704), (7169, 2048, 704), (12033, 1024, 1536), (11777, 1024, 1536)])
def test_linear_wide_tiles(M, N, K):
    test_linear_tiles(M, N, K)


# The walk over the tiles (bands of an eighth of the row tiles, four columns at a time, an eighth of the tiles to an XCD)
# takes every tile once, whatever their counts: fewer than eight tiles, a short last band, a last group of one to three
# columns.  Row and column counts in tiles of 64 (128 for the last two: 257 and 33 row tiles).
@pytest.mark.parametrize("M,N", [(1, 128), (150, 128), (400, 384), (577, 128), (1100, 640), (1500, 896), (2113, 384),
                                 (32800, 128), (4200, 1152)])
def test_linear_walk(M, N):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g = torch.Generator().manual_seed(M + N)
    a = torch.randint(-4, 5, (M, 64), generator=g).bfloat16().cuda()
    w = torch.randint(-4, 5, (N, 64), generator=g).bfloat16().cuda()
    log("linear-walk", M, N)
    # NaN where a call before this one left its output: a tile that no workgroup takes shows
    torch.full((M, N), float("nan"), device="cuda")
    assert torch.equal(lsh.linear_bf16(a, w), a.float() @ w.float().t())  # whole numbers: exact in any order


# The attention half's products in the [B, H, L, 64] layout, batches ending inside row tiles.  The whole call takes
# 256 x 256 tiles (M = 16362, N = 1024: 256 of them) or 128 x 128 (M = 65000, N = 256: 1016; M = 33330, N = 128: 261),
# a few batches 128 x 128 (M = 4848, N = 1024; M = 26000, N = 256) or 64 x 64 (M = 3333), one batch 64 x 64.  Every
# tile adds a value's products in the same order, so the results are the same bits; one batch is held to the oracle.
@pytest.mark.parametrize("B,H,L,few", [(54, 16, 303, 16), (50, 4, 1300, 20), (30, 2, 1111, 3)])
def test_head_layout_by_tile(B, H, L, few):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    w = W.BLOCKS["revblock_bf16_L65536"].scaled(B=B, H=H, L=L, d_ff=128, n_buckets=8, n_rounds=1, ff_chunk=0, exact=True)
    x = W.make_block_inputs(w)
    host, dev = {}, {}
    for k, a in x.items():
        if k not in ("x1", "x2"):
            bf = a.dtype == np.uint16
            host[k] = W.as_f64(a, "bf16") if bf else a.astype(np.float64)
            t = torch.from_numpy(a.view(np.int16) if bf else a).cuda()
            dev[k] = t.view(torch.bfloat16) if bf else t
    x1, x2 = torch.from_numpy(x["x1"]).cuda(), torch.from_numpy(x["x2"]).cuda()
    wd = lsh.BlockWeights(**dev)

    def call(batches):
        cfg = lsh.BlockConfig.of(w.scaled(B=batches.stop - batches.start))
        log("heads", B, H, L, batches)
        return lsh.rev_attention(cfg, wd, x2[batches].contiguous(), x1[batches].contiguous(), -1.0)

    whole = call(slice(0, B))
    assert torch.equal(call(slice(1, 1 + few)), whole[1:1 + few])
    for b in (0, B // 2, B - 1):
        assert torch.equal(call(slice(b, b + 1)), whole[b:b + 1])
    want = OB.attention_layer(x["x2"][-1:].astype(np.float64), OB.BlockWeights(**host), H, w.chunk, w.causal, w.ln_eps)
    err = np.abs(whole[-1:].cpu().numpy() - (x["x1"][-1:] - want))
    assert err.max() <= 2e-2  # the bf16 attention's bound
