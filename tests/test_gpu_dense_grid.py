"""Dense attention over the kernel's choices: 64 or 256 queries a workgroup
(256 from 512 such workgroups under causal masking, 256 without), one, two, four
or eight slices over the XCDs, whole and partial groups of slices, ragged
lengths, the online maximum; against fp64 torch within the rounding of bf16
weights and outputs (2^-9 each in numerator, denominator and result)."""
import math

import pytest
import torch

from gpu_common import log
from paper_2001_04451_amd import lsh

pytestmark = pytest.mark.gpu


def _reference(q, v, causal):
    """out, lse and sum p |v| of one slice, in fp64."""
    L = q.shape[0]
    i = torch.arange(L, device=q.device)
    s = q @ (q / q.norm(dim=1, keepdim=True)).t().contiguous() / math.sqrt(64)
    s = s - 1e5 * (i[:, None] == i[None, :])
    if causal:
        s = s.masked_fill(i[None, :] > i[:, None], -math.inf)
    lse = torch.logsumexp(s, 1)
    p = torch.exp(s - lse[:, None])
    return p @ v, lse, p @ v.abs()


@pytest.mark.parametrize("B,H,L,causal,big", [
    (3, 19, 2250, True, False),    # one slice at a time, 513 wide workgroups, a partial last group
    (1, 57, 2047, True, False),    # 456: the narrow kernel
    (5, 26, 769, True, True),      # two at a time, 520, the last block of one query, online maximum
    (4, 33, 1000, True, False),    # four at a time, 528
    (8, 9, 2048, True, True),      # eight at a time, 576, groups of eight and one, online maximum
    (1, 37, 1537, False, False),   # no mask, 259 wide workgroups, the last block of one query
    (2, 32, 769, False, True),     # 256: the wide kernel's first
    (1, 51, 1025, False, False),   # 255: the narrow kernel's last
    (1, 1, 65, False, False),      # two narrow workgroups, the second of one query
    (7, 3, 2, True, False),        # two tokens
])
def test_dense_grid(B, H, L, causal, big):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + L)
    q = torch.randn(B, H, L, 64, generator=g, device="cuda")
    if big:
        q[:, :, ::5] *= 64.0  # logit bounds past the range that needs no maximum
    q = q.bfloat16()
    v = torch.randn(B, H, L, 64, generator=g, device="cuda").bfloat16()
    cfg = lsh.Config(B=B, H=H, L=L, n_buckets=2, n_rounds=1, causal=causal)
    log("dense grid", B, H, L, causal, big)
    out, lse = lsh.lsh_dense_attn_fwd(cfg, q, v)
    for b in range(B):
        for h in range(H):
            x = q[b, h].double()
            ref, ref_lse, mass = _reference(x, v[b, h].double(), causal)
            logit = 2.0 ** -20 * x.norm(dim=1)  # fp32 sums of 64 products and the exponential's argument
            assert ((out[b, h].double() - ref).abs()
                    <= 2.0 ** -8 * mass + 2.0 ** -8 * ref.abs() + logit[:, None] * mass + 1e-6).all()
            assert ((lse[b, h].double() - ref_lse).abs() <= 2.0 ** -8 + logit + 2.0 ** -20 * ref_lse.abs()).all()
