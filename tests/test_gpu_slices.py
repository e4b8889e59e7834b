"""The chunk attention's numbering of workgroups over the XCDs (one slice at a time,
four or eight, whole and partial last sets): a call gives each (batch, head)
slice what a call on that slice alone gives, bit for bit, forward and backward."""
import pytest
import torch

from gpu_common import log
from paper_2001_04451_amd import lsh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,L,n_r,causal", [
    (1, 8, 130, 1, True),       # eight slices at a time, one pass
    (2, 12, 1000, 3, False),    # eight, three passes
    (3, 4, 1999, 2, True),      # four, two XCDs each, odd strips
    (1, 4, 64, 1, True),        # four, one strip: half of the workgroups have none
    (1, 6, 700, 2, True),       # neither: one at a time
    (1, 8, 16384, 2, True),     # eight: the last length of at most 4 MB a slice
    (1, 8, 16385, 1, False),    # one at a time
])
def test_slices_stand_alone(B, H, L, n_r, causal):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g = torch.Generator(device="cuda").manual_seed(L)
    q, v, dout = (torch.randn(B, H, L, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    n_b = max(2, L // 64 // 2 * 2)
    R = torch.randn(n_r, 64, n_b // 2, generator=g, device="cuda")

    def call(q, v, dout):
        cfg = lsh.Config(B=q.shape[0], H=q.shape[1], L=L, n_buckets=n_b, n_rounds=n_r, causal=causal)
        f = lsh.lsh_attention_fwd(cfg, q, v, R)
        dq, dv = lsh.lsh_chunk_attn_bwd(cfg, q, v, f.out, dout, f.lse, f.buckets, f.perm, f.undo, f.bstart)
        return f.out, f.lse, dq, dv

    log("slices", B, H, L, n_r, causal)
    whole = call(q, v, dout)
    for b in range(B):
        for h in range(H):
            alone = call(*(x[b:b + 1, h:h + 1].contiguous() for x in (q, v, dout)))
            for w, a in zip(whole, alone):
                assert torch.equal(w[b, h], a[0, 0])
