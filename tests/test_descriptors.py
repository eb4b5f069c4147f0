"""The packed descriptors that the binding passes are, byte for byte, the
ctypes structures of the C ABI."""
import ctypes as C

import pytest
import torch

from paper_2605_24168_amd import sparse_decode as sd


@pytest.fixture(autouse=True)
def host_tensors(monkeypatch):
    monkeypatch.setattr(sd, "_need_device", lambda *a, **k: None)


def test_packed_tensors_and_caches():
    for t in (torch.zeros(3), torch.zeros(0, 4), torch.zeros(1, 2, 3, 4, dtype=torch.int32),
              torch.zeros((), dtype=torch.bfloat16)):
        assert sd._desc(t, "t") == bytes(sd._tensor(t, "t"))
    k = torch.zeros(5, 16, 2, 128, dtype=torch.bfloat16)
    table = torch.zeros(3, 7, dtype=torch.int32)
    lab = sd.Labels(torch.zeros(5, 2, 16, 8, dtype=torch.bfloat16), torch.zeros(2, 8, dtype=torch.int32))
    assert sd._labels_desc(lab) == bytes(lab.c())
    for cache in (sd.KVCache(k=k, v=k.clone(), layout="paged", block_table=table),
                  sd.KVCache(k=torch.zeros(1, 2, 30, 128), v=torch.zeros(1, 2, 30, 128))):
        assert sd._kv_desc(cache, "k") == bytes(cache.c("k"))
        assert sd._kv_desc(cache, "k", "v") == (bytes(cache.c("k")), bytes(cache.c("v")))
    with pytest.raises(ValueError):
        sd._kv_desc(sd.KVCache(k=k, v=k, layout="hnd"), "k")
    with pytest.raises(ValueError):
        sd._desc(torch.zeros(1, 1, 1, 1, 1), "t")
    with pytest.raises(ValueError):
        sd._desc(torch.zeros(2, dtype=torch.float64), "t")


@pytest.mark.parametrize("kw", [
    dict(ratio=3.5, rounding=1, group_shared=True, softmax_scale=0.25, n_sink=3, n_local=4),
    dict(ratio=1e-3, rounding=-1, softmax_scale=1e300, n_sink=2**31, n_local=2**32 + 5),
    dict(ratio=float("nan"), softmax_scale=float("-inf"), n_sink=-1),
])
def test_packed_sparsity(kw):
    a, b = bytes(sd.Sparsity(**kw).c()), sd._sparsity_desc(sd.Sparsity(**kw))
    assert a[:20] == b[:20] and a[24:] == b[24:]  # (bytes 20-23: padding)


def test_the_library_takes_its_structures_and_no_others():
    sp = sd.Sparsity(ratio=10.0).c()
    assert sd.lib.sparse_decode_budget(1000, sp) == 100  # (an instance, as its pointer)
    assert sd.lib.sparse_decode_budget(1000, C.byref(sp)) == 100
    assert sd.lib.sparse_decode_budget(1000, C.pointer(sp)) == 100
    assert sd.budget(1000, sd.Sparsity(ratio=10.0)) == 100
    for other in (C.byref(sd.SdTensor()), bytes(sp), 4096):
        with pytest.raises(C.ArgumentError):
            sd.lib.sparse_decode_budget(1000, other)
