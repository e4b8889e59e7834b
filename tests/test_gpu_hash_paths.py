"""The hash's last pass (fp64) at the edges of its groups, candidate lists and
fp32 range.  Bucket ids are whole numbers: bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import log, small, to_device
from paper_2001_04451_amd import lsh
from paper_2001_04451_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    lsh.lib()


# copies: columns within an ulp of one another, so that every row has that
# many candidates: two, all of a row's eight candidate lanes, and more (every
# column in fp64).  Lengths: one row, groups of 16 with a remainder, several
# groups.  scale 2^-120 on top of R's 2^-30 leaves fp32's range.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L,n_buckets,copies,k", [(1, 2, 1, 0), (17, 32, 2, 0), (33, 128, 8, 0), (65, 128, 9, 0),
                                                  (300, 1022, 3, 0), (40, 66, 2, -120)])
def test_hash_close_columns(gpu, dtype, L, n_buckets, copies, k):
    w = small("causal_bf16_L16384", B=1, H=2, L=L, n_buckets=n_buckets, n_rounds=2, dtype=dtype)
    x = W.make_inputs(w)
    R = x["R"].copy()
    half = n_buckets // 2
    for c in range(half):  # runs of `copies` columns, each one ulp away in one entry
        base = c - c % copies
        R[:, :, c] = R[:, :, base]
        if c != base:
            R[:, c % 64, c] = np.nextafter(R[:, c % 64, c], np.float32(np.inf))
    q = W.as_f64(x["q"], dtype).astype(np.float32)
    if k:
        q = np.ldexp(q, k).astype(np.float32)
        R = np.ldexp(R, -30).astype(np.float32)
    qin = W.f32_to_bf16_bits(q) if dtype == "bf16" else q
    want, _ = oracle.lsh_hash(W.as_f64(qin, dtype), R.astype(np.float64))
    log("hash-close", dtype, L, n_buckets, copies, k)
    got = lsh.lsh_hash(lsh.Config.of(w), to_device(qin, dtype), to_device(R, "f32")).cpu().numpy()
    assert np.array_equal(got, want)


# Projections outside fp32's range, or of rows or an R near its lower end, where the last pass's fp32 sums say nothing
# (a partial sum may overflow to an infinity, or to NaN, in a column that does not hold the largest): every row has a
# column and its copy one ulp away, so that all rows reach the last pass.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k_q,k_r", [(64, 60), (64, 61), (66, 62), (100, 26), (-75, 40), (-69, 20), (60, -118)])
def test_hash_fp32_range(gpu, dtype, k_q, k_r):
    w = small("causal_bf16_L16384", B=1, H=2, L=300, n_buckets=128, n_rounds=2, dtype=dtype)
    x = W.make_inputs(w)
    R = x["R"].copy()
    R[:, :, 1::2] = R[:, :, ::2]
    R[:, 5, 1::2] = np.nextafter(R[:, 5, 1::2], np.float32(np.inf))
    q = np.ldexp(W.as_f64(x["q"], dtype).astype(np.float32), k_q)
    R = np.ldexp(R, k_r)
    qin = W.f32_to_bf16_bits(q) if dtype == "bf16" else q
    want, _ = oracle.lsh_hash(W.as_f64(qin, dtype), R.astype(np.float64))
    log("hash-range", dtype, k_q, k_r)
    got = lsh.lsh_hash(lsh.Config.of(w), to_device(qin, dtype), to_device(R, "f32")).cpu().numpy()
    assert np.array_equal(got, want), f"{(got != want).sum()} of {got.size}"


# One round (of one head) with columns in equal pairs, so that only its list is long: every block of the last pass
# takes a share of it, past the 64 rounds that a block looks at together (H n_rounds = 1040 in groups of 1024 and 16).
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,H,L,n_r,n_buckets,at", [(1, 2, 9001, 3, 130, (0, 1)), (40, 65, 61, 16, 34, (63, 15)),
                                                    (40, 65, 61, 16, 34, (64, 3)), (60, 70, 61, 1, 66, (2, 0))])
def test_hash_one_long_list(gpu, dtype, B, H, L, n_r, n_buckets, at):
    w = small("causal_bf16_L16384", B=B, H=H, L=L, n_buckets=n_buckets, n_rounds=n_r, dtype=dtype)
    x = W.make_inputs(w)
    per_head = H > 2
    R = np.random.default_rng(9).standard_normal((H if per_head else 1, n_r, 64, n_buckets // 2), dtype=np.float32)
    R[at][:, 1::2] = R[at][:, :-1:2][:, :R[at][:, 1::2].shape[1]]
    R = R if per_head else R[0]
    want, _ = oracle.lsh_hash(W.as_f64(x["q"], dtype), R.astype(np.float64))
    log("hash-long-list", dtype, B, H, L, n_r, n_buckets, at)
    got = lsh.lsh_hash(lsh.Config.of(w, r_per_head=per_head), to_device(x["q"], dtype), to_device(R, "f32")).cpu().numpy()
    assert np.array_equal(got, want)


# One R per head: slices that end inside a workgroup's rows (L = 1, 255, 300),
# one head, and more rounds of R than are hashed together (H n_rounds = 1040).
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,H,L,n_r,n_buckets", [(2, 3, 300, 2, 66), (3, 1, 255, 1, 2), (1, 65, 40, 16, 34),
                                                 (5, 2, 1, 3, 1022), (2, 2, 512, 4, 256)])
def test_hash_per_head_slices(gpu, dtype, B, H, L, n_r, n_buckets):
    w = small("causal_bf16_L16384", B=B, H=H, L=L, n_buckets=n_buckets, n_rounds=n_r, dtype=dtype)
    x = W.make_inputs(w)
    R = np.random.default_rng(7).standard_normal((H, n_r, 64, n_buckets // 2), dtype=np.float32)
    want, _ = oracle.lsh_hash(W.as_f64(x["q"], dtype), R.astype(np.float64))
    log("hash-per-head", dtype, B, H, L, n_r, n_buckets)
    cfg = lsh.Config.of(w, r_per_head=True)
    got = lsh.lsh_hash(cfg, to_device(x["q"], dtype), to_device(R, "f32")).cpu().numpy()
    assert np.array_equal(got, want)


# Above 40 M projections bf16 calls are screened with R's hi plane, then the open rows listed: whole and partial tiles
# and stages of R (1, 2, 3, 10 and 16 tiles), one R or one per head (slices that end inside a workgroup's rows, several
# batches, H n_rounds = 1120: a full and a partial group of heads; 1040: the last head alone, in one pass).  Rows are
# drawn from a pool whose ids come from the oracle: zero rows, bf16 subnormals, a few large values beside small ones,
# scales of 2^-60 .. 2^60, rounds of R at 2^-60 and 2^50.  tied: every column has an equal, a negated or a one-ulp copy,
# so that every row is left open by the screen and by the listed pass (full segments and lists).
@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("B,H,L,n_r,n_buckets,per_head", [
    (1, 2, 41001, 16, 2, False), (1, 2, 20501, 16, 66, False), (2, 1, 13701, 16, 192, False),
    (2, 1, 8201, 8, 640, False), (1, 2, 9001, 5, 1022, False),
    (1, 2, 41001, 16, 2, True), (3, 5, 2801, 16, 66, True), (2, 3, 9001, 4, 1022, True),
    (2, 70, 430, 16, 1022, True), (1, 65, 700, 16, 1022, True)])
def test_hash_screened(gpu, B, H, L, n_r, n_buckets, per_head, tied):
    half = n_buckets // 2
    assert B * H * L * n_r * -(-half // 32) * 32 > 40 << 20
    rng = np.random.default_rng(L + n_buckets)
    pool, sets = 250, H if per_head else 1
    R = rng.standard_normal((sets, n_r, 64, half), dtype=np.float32)
    if tied and half > 1:
        R[..., 1::3] = R[..., :-1:3][..., :R[..., 1::3].shape[-1]]
        R[..., 2::3] = -R[..., 1::3][..., :R[..., 2::3].shape[-1]]
        R[..., 7, 1::6] = np.nextafter(R[..., 7, 1::6], np.float32(np.inf))
    R[:, 0] *= np.float32(2.0 ** -60)
    R[:, -1] *= np.float32(2.0 ** 50)
    q = rng.standard_normal((1, sets, pool, 64)) * np.ldexp(1.0, rng.integers(-60, 61, (1, sets, pool, 1)))
    q[:, :, 1::8] = 0
    q[:, :, 2::8] = rng.standard_normal(q[:, :, 2::8].shape) * 2.0 ** -130
    q[:, :, 3::8, :4] *= 2.0 ** 30
    bits = W.f32_to_bf16_bits(q.astype(np.float32))
    want, _ = oracle.lsh_hash(W.as_f64(bits, "bf16"), (R if per_head else R[0]).astype(np.float64))
    pick = rng.integers(0, pool, (B, H, L))
    head = np.arange(H)[None, :, None] % sets
    w = small("causal_bf16_L16384", B=B, H=H, L=L, n_buckets=n_buckets, n_rounds=n_r)
    log("hash-screened", B, H, L, n_r, n_buckets, per_head, tied)
    got = lsh.lsh_hash(lsh.Config.of(w, r_per_head=per_head), to_device(bits[0][head, pick], "bf16"),
                       to_device(R if per_head else R[0], "f32")).cpu().numpy()
    bad = got != want[0][head, pick]
    assert not bad.any(), f"{bad.sum()} of {got.size}"
