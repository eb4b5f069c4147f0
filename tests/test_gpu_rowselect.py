"""Top-k of full score rows by one workgroup per row: rows that stay in
registers, rows filtered as they stream by a sampled threshold, and rows that
take the radix passes, at the sizes where one form gives way to the next, for
score distributions that crowd or break the histograms (ties, masked rows,
infinities, one cluster, sorted rows), and the fused calls that select from
full scores.  Lists and scores must equal the oracle's selection on the same
float32 scores exactly.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2605_24168_amd import synth
from tests import parity as P
from tests.test_gpu_parity import check_fused

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24168_amd import sparse_decode
    sparse_decode.set_debug(0)
    return sparse_decode


def rows_of_kind(kind, rows, n):
    rng = np.random.default_rng(n * 31 + rows)
    s = rng.standard_normal((rows, n), dtype=np.float32)
    if kind == "ties":
        s = np.round(2 * s)
    elif kind == "masked":
        s[rng.random(s.shape) < 0.99] = -np.inf
    elif kind == "lowest":
        s[rng.random(s.shape) < 0.5] = np.finfo(np.float32).min
    elif kind == "inf":
        s[rng.random(s.shape) < 0.2] = np.inf
    elif kind == "cluster":  # one wave's share holds most of the candidates
        s[:, n // 2:n // 2 + n // 20] += 6
    elif kind == "sorted":
        s.sort(axis=1)
    elif kind == "zeros":
        s = np.where(s < 0, np.float32(-0.0), np.float32(0.0))
    return s


def check(sd, s, L, ratio, n_sink=0, n_local=0):
    rows, n = s.shape
    sp = sd.Sparsity(ratio=ratio, n_sink=n_sink, n_local=n_local)
    idx, vals = sd.sparse_decode_topk(torch.from_numpy(s[None]).cuda(),
                                      torch.tensor([L], dtype=torch.int32, device="cuda"), sp,
                                      with_vals=True)
    torch.cuda.synchronize()
    idx, vals = idx[0].cpu().numpy(), vals[0].cpu().numpy()
    ns = min(n_sink, L)
    nl = min(n_local, L - ns)
    k = min(O.budget(L, ratio, 0), L - ns - nl)
    for r in range(rows):
        # (score descending, position ascending), as a stable sort gives it
        top = np.sort(np.argsort(-s[r, ns:L - nl], kind="stable")[:k]) + ns
        want = np.concatenate([np.arange(ns), top, np.arange(L - nl, L)])
        assert np.array_equal(idx[r, :want.size], want), (r, L, ratio)
        assert (idx[r, want.size:] == -1).all()
        assert np.array_equal(vals[r, :want.size], s[r, want])
        assert (vals[r, want.size:] == -np.inf).all()


@pytest.mark.parametrize("kind", ["normal", "ties", "masked", "lowest", "inf", "cluster", "sorted",
                                  "zeros"])
@pytest.mark.parametrize("rows,n,ratio", [
    (3, 1, 1.0), (3, 65, 4.0), (2, 1025, 10.0),
    (513, 4096, 20.0), (513, 4097, 20.0),        # 256-thread rows, and past them
    (2, 16384, 20.0), (2, 16385, 20.0),          # in registers, and past them
    (2, 50021, 9.0), (2, 50021, 1.5),            # filtered; too many candidates
    (2, 131072, 11.0), (3, 393216, 40.0),        # 8192 samples
    (1, 1048576, 100.0), (1, 1048577, 100.0),    # at 4/5 of the room; 16-bit offsets end
])
def test_topk_rows(sd, kind, rows, n, ratio):
    check(sd, rows_of_kind(kind, rows, n), n, ratio)


@pytest.mark.parametrize("rows,n,nans", [(2, 100, 100), (2, 1040, 64), (3, 1040, 1040), (1, 16384, 200),
                                         (513, 4095, 300)])
def test_topk_rows_of_the_lowest_nans(sd, rows, n, nans):
    # Every position kept, the k-th key being that of the lowest NaN, in the
    # bucket where lanes without a score would be counted too: the lists hold
    # each position once.
    s = np.random.default_rng(n).standard_normal((1, rows, n), dtype=np.float32)
    s.view(np.uint32)[:, :, :nans] = 0xFFFFFFFF
    idx, vals = sd.sparse_decode_topk(torch.from_numpy(s).cuda(),
                                      torch.tensor([n], dtype=torch.int32, device="cuda"),
                                      sd.Sparsity(ratio=1.0), with_vals=True)
    torch.cuda.synchronize()
    assert (idx.cpu().numpy() == np.arange(n)).all()
    np.testing.assert_array_equal(vals.cpu().numpy(), s)


@pytest.mark.parametrize("share", [0.001, 0.03, 0.3])
@pytest.mark.parametrize("n", [4096, 50021, 1048576])
def test_topk_nans_rank_by_their_sign(sd, n, share):
    # Whatever the form that a row takes, NaNs with the sign clear come above
    # every number and the others below (fewer or more of them than k).
    rng = np.random.default_rng(n)
    s = rng.standard_normal((1, 2, n), dtype=np.float32)
    at = rng.random(s.shape) < share
    s.view(np.uint32)[at] = rng.choice(np.array([0x7FC00000, 0x7F800001, 0xFFC00000], np.uint32),
                                       int(at.sum()))
    idx = sd.sparse_decode_topk(torch.from_numpy(s).cuda(),
                                torch.tensor([n], dtype=torch.int32, device="cuda"),
                                sd.Sparsity(ratio=40.0))
    u = s.view(np.uint32).astype(np.int64)
    key = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
    k = O.budget(n, 40.0, 0)
    for r in range(2):
        want = np.sort(np.argsort(-key[0, r], kind="stable")[:k])
        assert np.array_equal(idx[0, r, :k].cpu().numpy(), want)


@pytest.mark.parametrize("L", [0, 1, 63, 16500, 50000])
def test_topk_forced_and_short_sequences(sd, L):
    if L == 0:
        sp = sd.Sparsity(ratio=20.0, n_sink=16, n_local=8)
        idx = sd.sparse_decode_topk(torch.randn((1, 2, 50021), device="cuda"),
                                    torch.zeros(1, dtype=torch.int32, device="cuda"), sp)
        assert (idx == -1).all()
        return
    check(sd, rows_of_kind("normal", 2, 50021), L, 20.0, n_sink=16, n_local=8)


@pytest.mark.parametrize("n,ratio", [
    (4096, 10.0), (16400, 20.0), (50000, 10.0),  # one workgroup per row
    (50000, 2.0),                                # several workgroups per row
])
def test_fused_rows_from_full_scores(sd, n, ratio):
    inp = synth.make_inputs(1, seed=5, B=2, Hq=4, Hkv=2, seq_lens=[n, n // 3 + 7], ncap=n + 5,
                            ratio=ratio)
    q, cache, lens = sd.cache_from_inputs(inp)
    out, idx = sd.sparse_decode_attention(q, cache, lens, sd.sparsity_from_inputs(inp),
                                          k_max=O.k_max_for(inp))
    torch.cuda.synchronize()
    check_fused(inp, P.to_host(out), idx.cpu().numpy(), label=f"{n} at {ratio}x")


@pytest.mark.parametrize("B,Hq,Hkv,n", [
    (1, 3, 3, 262144), (1, 3, 3, 262160),   # one workgroup per row; pieces
    (1, 15, 3, 300000), (1, 16, 2, 300000),  # pieces; one workgroup, enough rows
])
def test_long_rows_by_one_workgroup_or_in_pieces(sd, B, Hq, Hkv, n):
    """Every row from its full scores (debug flag 1): the lists are those of
    the stand-alone selection over the stand-alone scores."""
    g = torch.Generator(device="cuda").manual_seed(n + Hq)
    k = torch.randn((B, Hkv, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn((B, Hq, 128), generator=g, device="cuda").to(torch.bfloat16)
    cache, sp = sd.KVCache(k=k, v=k), sd.Sparsity(ratio=60.0)
    lens = torch.full((B,), n - 3, dtype=torch.int32, device="cuda")
    sd.set_debug(1)
    try:
        idx = sd.sparse_decode_attention(q, cache, lens, sp)[1]
    finally:
        sd.set_debug(0)
    scores = sd.sparse_decode_score(q, cache, lens, sp)
    assert torch.equal(idx, sd.sparse_decode_topk(scores, lens, sp))
