"""Short contexts: calls whose rows the cost rule selects from full scores
(scores, selection, attention) give, bit for bit, the lists and outputs of the
candidate path (debug flag 64 keeps a call on it), for every kind of fused
call, both layouts, ragged batches with empty sequences, capacities beyond
the sequences and budgets set per sequence.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2605_24168_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu

CANDIDATES = 64


@pytest.fixture(scope="module")
def sd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_24168_amd import sparse_decode
    sparse_decode.set_debug(0)
    return sparse_decode


def both(sd, call):
    """(outputs, rows selected from full scores) by the rule and without it."""
    got = []
    for flags in (0, CANDIDATES):
        sd.set_debug(flags)
        sd.set_profiling(True)
        try:
            out = [P.to_host(t) for t in call()]
            torch.cuda.synchronize()
            got.append((out, sd.last_profile()["repaired_rows"]))
        finally:
            sd.set_profiling(False)
            sd.set_debug(0)
    return got


@pytest.mark.parametrize("kind", ["exact", "shared", "forced", "override", "label", "sampled",
                                  "noalloc"])
@pytest.mark.parametrize("layout", ["bhnd", "paged"])
@pytest.mark.parametrize("Hq,Hkv,lens,ncap", [
    (8, 8, [2049, 4096], 4097),            # one row per group
    (32, 8, [8191], 8192),                 # registers hold the rows
    (10, 2, [17003, 0, 1, 9000], 20000),   # 5 heads per group; rows past the registers
    (16, 1, [3000, 64, 65], 30000),        # 16 heads; mostly empty capacity
])
def test_short_context_rule(sd, kind, layout, Hq, Hkv, lens, ncap):
    inp = synth.make_inputs(2, seed=11, seq_lens=lens, ncap=ncap, Hq=Hq, Hkv=Hkv, layout=layout,
                            ratio=20.0, group_shared=kind == "shared",
                            n_sink=70 if kind == "forced" else 0,
                            n_local=33 if kind == "forced" else 0)
    q, cache, sl = sd.cache_from_inputs(inp)
    sp = sd.sparsity_from_inputs(inp)
    kmax = O.k_max_for(inp)
    if kind == "override":
        sp.k_override = torch.tensor([min(kmax, 5 + 97 * b) for b in range(inp.B)],
                                     dtype=torch.int32, device="cuda")
    if kind == "label":
        ch = synth.label_channels(Hkv)
        lab = synth.label_cache_device_layout(inp, synth.label_cache(inp, ch))
        labels = sd.Labels(t=torch.from_numpy(lab).view(torch.bfloat16).cuda(),
                           channels=torch.from_numpy(ch).cuda())
        call = lambda: sd.sparse_decode_label_attention(q, cache, labels, sl, sp, k_max=kmax)
    elif kind == "sampled":
        draws = torch.randint(-2**31, 2**31, (inp.B, Hq, 50), device="cuda").to(torch.int32)
        call = lambda: sd.sparse_decode_sampled_attention(q, cache, sl, sp, draws, k_max=kmax)
    elif kind == "noalloc":
        call = lambda: sd.sparse_decode_attention_noalloc(
            q, cache, sl, sp, torch.empty_like(q),
            torch.empty((inp.B, Hq, kmax), dtype=torch.int32, device="cuda"))
    else:
        call = lambda: sd.sparse_decode_attention(q, cache, sl, sp, k_max=kmax)
    (a, full), (b, cand) = both(sd, call)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)
    if kind != "noalloc":  # (its calls are not profiled)
        assert full > 0 and cand < full, (full, cand)


@pytest.mark.parametrize("layout,lens,Hq,Hkv", [
    ("paged", [32768], 32, 8),          # 32 units of 2048-key waves, halved twice
    ("paged", [65536, 1025], 8, 4),     # 64 units: at 512 keys a whole round
    ("paged", [10000, 8193, 513], 12, 6),  # one head per workgroup: 36 units, four waves a chunk
    ("bhnd", [131071], 8, 2),           # 32 units, the last chunk one key short
])
def test_halved_waves(sd, layout, lens, Hq, Hkv):
    """Calls of few stream units run shorter waves where their workspace has
    room; both give the lists of the stand-alone selection over the
    stand-alone scores, and the same outputs."""
    inp = synth.make_inputs(2, seed=5, seq_lens=lens, ncap=max(lens), Hq=Hq, Hkv=Hkv,
                            layout=layout, ratio=40.0)
    q, cache, sl = sd.cache_from_inputs(inp)
    sp = sd.sparsity_from_inputs(inp)
    kmax = O.k_max_for(inp)
    idx = torch.empty((inp.B, Hq, kmax), dtype=torch.int32, device="cuda")
    buf = torch.empty(sd.workspace_size(q, cache, sp, idx), dtype=torch.uint8, device="cuda")
    sd.set_debug(CANDIDATES)

    def call(room):
        """(out, idx, end of what was written to the workspace)"""
        buf.fill_(0xA5)
        sd.set_workspace(buf[:room])
        try:
            out = [P.to_host(t) for t in sd.sparse_decode_attention(q, cache, sl, sp, k_max=kmax)]
            torch.cuda.synchronize()
            return *out, int((buf != 0xA5).nonzero().max())
        finally:
            sd.set_workspace(None)

    try:
        # The smallest workspace that is taken (too small ones launch
        # nothing): the one of whole-length waves.
        lo, hi = 0, buf.numel() // 256
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                call(256 * mid)
                hi = mid
            except sd.SparseDecodeError:
                lo = mid
        halved, whole = call(buf.numel()), call(256 * hi)
    finally:
        sd.set_debug(0)
    # (two layouts: whole-length waves write less of the workspace)
    assert whole[2] < 256 * hi <= buf.numel() and whole[2] < halved[2], (whole[2], halved[2])
    scores = sd.sparse_decode_score(q, cache, sl, sp)
    want = P.to_host(sd.sparse_decode_topk(scores, sl, sp, k_max=kmax))
    for got in (halved, whole):
        np.testing.assert_array_equal(got[1], want)
    np.testing.assert_array_equal(halved[0], whole[0])


def test_halved_waves_stay_within_the_library_workspace(sd):
    """A call that fits the library's workspace with whole-length waves does
    not have it grown for halved ones: a graph captured over it stays valid,
    and the call itself can be captured.  65 chunks of 131088 keys on 8 KV
    heads keep whole waves, 64 of 131072 would take 1 MB more than them."""
    def make(n):
        q = torch.randn((1, 32, 128), device="cuda").to(torch.bfloat16)
        kv = torch.randn((2, n // 16, 16, 8, 128), device="cuda", dtype=torch.bfloat16)
        table = torch.arange(n // 16, dtype=torch.int32, device="cuda")[None]
        cache = sd.KVCache(k=kv[0], v=kv[1], layout="paged", block_table=table)
        lens = torch.tensor([n], dtype=torch.int32, device="cuda")
        idx = torch.empty((1, 32, sd.k_max_of(cache, sd.Sparsity(ratio=100.0))), dtype=torch.int32,
                          device="cuda")
        return q, cache, lens, torch.empty_like(q), idx

    def call(args):
        q, cache, lens, out, idx = args
        sd.sparse_decode_attention(q, cache, lens, sd.Sparsity(ratio=100.0), out=out, idx=idx)

    longer, shorter = make(131088), make(131072)
    sizes = [sd.workspace_size(q, c, sd.Sparsity(ratio=100.0), idx) for q, c, _, _, idx in (longer, shorter)]
    page = 2 << 20  # (allocations come in pages of 2 MB)
    assert -(-sizes[0] // page) < -(-sizes[1] // page)
    sd.set_workspace(None)
    call(shorter)  # (with room of its own: halved waves)
    torch.cuda.synchronize()
    want = [t.clone() for t in shorter[3:]]
    sd.set_workspace(torch.empty(256, dtype=torch.uint8, device="cuda"))
    sd.set_workspace(None)  # (the library's workspace is given back)
    call(longer)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    call(shorter)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(shorter)
    for _ in range(3):
        for t in shorter[3:]:
            t.zero_()
        call(longer)
        graph.replay()
        torch.cuda.synchronize()
        for t, w in zip(shorter[3:], want):
            assert torch.equal(t, w)


@pytest.mark.parametrize("layout", ["bhnd", "paged"])
@pytest.mark.parametrize("Hq,Hkv,shared", [(4, 4, False), (8, 2, False), (12, 4, True)])
@pytest.mark.parametrize("ncap", [1040, 20000, 400000])
def test_sequences_shorter_than_the_cache(sd, layout, Hq, Hkv, shared, ncap):
    """Calls scored in full (debug flag 1) over ragged sequences in a longer
    cache keep what each sequence keeps in a cache of its own length, and
    stand-alone scores are the same bit for bit, -inf past the sequence."""
    lens = [min(n, ncap) for n in (0, 1, 63, 65, 1039, 4100, 19999)]
    inp = synth.make_inputs(2, seed=6, seq_lens=lens, ncap=max(lens), Hq=Hq, Hkv=Hkv,
                            layout=layout, group_shared=shared)
    q, cache, sl = sd.cache_from_inputs(inp)
    sp = sd.sparsity_from_inputs(inp)
    if layout == "paged":
        wide = torch.full((len(lens), ncap // 16), -1, dtype=torch.int32, device="cuda")
        wide[:, :cache.block_table.shape[1]] = cache.block_table
        big = sd.KVCache(k=cache.k, v=cache.v, layout=layout, block_table=wide)
    else:
        k, v = (torch.zeros((len(lens), Hkv, ncap, 128), dtype=torch.bfloat16, device="cuda")
                for _ in range(2))
        k[:, :, :max(lens)], v[:, :, :max(lens)] = cache.k, cache.v
        big = sd.KVCache(k=k, v=v)
    sd.set_debug(1)
    try:
        out, idx = sd.sparse_decode_attention(q, big, sl, sp)
        scores = sd.sparse_decode_score(q, big, sl, sp)
        for b, L in enumerate(lens):
            k_b = sd.budget(L, sp)
            assert (idx[b, :, k_b:] == -1).all()
            assert torch.isneginf(scores[b, :, L:]).all()
            if L == 0:
                assert (out[b] == 0).all()
                continue
            if layout == "paged":
                own = sd.KVCache(k=cache.k, v=cache.v, layout=layout,
                                 block_table=cache.block_table[b:b + 1, :-(-L // 16)].contiguous())
            else:
                own = sd.KVCache(k=cache.k[b:b + 1, :, :L].contiguous(), v=cache.v[b:b + 1, :, :L].contiguous())
            ref, ridx = sd.sparse_decode_attention(q[b:b + 1].contiguous(), own, sl[b:b + 1], sp)
            assert torch.equal(idx[b, :, :k_b], ridx[0, :, :k_b])
            rscores = sd.sparse_decode_score(q[b:b + 1].contiguous(), own, sl[b:b + 1], sp)
            assert torch.equal(scores[b, :, :L], rscores[0, :, :L])
            ok, worst, _ = P.out_errors(P.to_host(out[b]), P.to_host(ref[0]), "bf16")
            assert ok, worst
    finally:
        sd.set_debug(0)


@pytest.mark.parametrize("n", [16384, 131072])  # full scores; the stream
def test_the_scoring_kernel_that_runs_is_timed(sd, n):
    """Profiling level 2: no scoring kernel reads its keys in less than the
    time that they take at 8 TB/s, whichever one a call takes."""
    kv = torch.randn((2, 2, 8, n, 128), device="cuda", dtype=torch.bfloat16)
    q = torch.randn((2, 32, 128), device="cuda").to(torch.bfloat16)
    cache = sd.KVCache(k=kv[0], v=kv[1])
    lens = torch.full((2,), n, dtype=torch.int32, device="cuda")
    sd.set_profiling(2)
    try:
        for _ in range(3):
            sd.sparse_decode_attention(q, cache, lens, sd.Sparsity(ratio=50.0))
        torch.cuda.synchronize()
        prof = sd.profile_mean()
    finally:
        sd.set_profiling(False)
    assert prof["valid"] == 1 and prof["calls"] == 3
    assert prof["repaired_rows"] == (64 if n == 16384 else 0)
    assert prof["score_ms"] >= kv[0].numel() * 2 / 8e12 * 1e3
