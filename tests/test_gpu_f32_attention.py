"""The fp32 forward at the edges of its tiles, windows and signature widths,
and with values that are not finite outside a query's keys."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import log, lse_close, small, to_device
from paper_2001_04451_amd import lsh
from paper_2001_04451_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    lsh.lib()


# L: one token, a tile's edge, a partial last chunk of one slot, pieces of the
# window past the sequence; rounds: each signature width.
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("L,chunk,after,n_r,n_b", [(1, 64, 0, 1, 2), (16, 128, 0, 2, 2), (17, 64, 1, 3, 4),
                                                   (129, 64, 0, 6, 2), (193, 128, 1, 16, 6), (321, 64, 1, 8, 2),
                                                   (500, 128, 0, 4, 8)])
def test_f32_forward_edges(gpu, causal, L, chunk, after, n_r, n_b):
    w = small("tiny_f32_L1024", B=1, H=2, L=L, chunk=chunk, n_rounds=n_r, n_buckets=n_b, causal=causal)
    x = W.make_inputs(w)
    ref = oracle.lsh_attention_fwd(W.as_f64(x["q"], "f32"), W.as_f64(x["v"], "f32"), x["R"].astype(np.float64), chunk,
                                   causal, after=after)
    cfg = lsh.Config.of(w, chunks_after=after)
    log("f32-edges", L, chunk, after, n_r, n_b, causal)
    st = lsh.lsh_attention_fwd(cfg, to_device(x["q"], "f32"), to_device(x["v"], "f32"), to_device(x["R"], "f32"))
    assert np.abs(st.out.cpu().numpy() - ref["out"]).max() <= 1e-5
    assert lse_close(st.lse.cpu().numpy(), ref["lse"], "f32").all()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_f32_values_not_finite_stay_with_their_bucket(gpu, bad):
    """A value that is not finite reaches the queries that have its key and no
    others, under a causal mask and across buckets."""
    w = small("tiny_f32_L1024", B=1, H=1, L=256, n_rounds=1, n_buckets=8, causal=True)
    x = W.make_inputs(w)
    q64, v64, R64 = (a.astype(np.float64) for a in (x["q"], x["v"], x["R"]))
    ref = oracle.lsh_attention_fwd(q64, v64, R64, w.chunk, True)
    at = 100
    v = x["v"].copy()
    v[0, 0, at, 3] = bad
    log("f32-not-finite", bad)
    st = lsh.lsh_attention_fwd(lsh.Config.of(w), to_device(x["q"], "f32"), to_device(v, "f32"), to_device(x["R"], "f32"))
    out = st.out.cpu().numpy()[0, 0]
    bucket, perm = ref["buckets"][0, 0, :, 0], ref["perm"][0, 0, 0]
    chunk_of = np.argsort(perm) // w.chunk
    i = np.arange(w.L)
    has = (i > at) & (bucket == bucket[at]) & (chunk_of - chunk_of[at] <= 1) & (chunk_of >= chunk_of[at])
    assert has.any() and not np.isfinite(out[has, 3]).any()
    clean = np.ones_like(out, dtype=bool)
    clean[has, 3] = False
    clean[at, 3] = np.isfinite(out[at, 3])  # its own row: v itself if it has no other key
    assert np.abs(out - ref["out"][0, 0])[clean].max() <= 1e-5
