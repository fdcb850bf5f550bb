"""The shared merge of many token splits: each split merges a slice of the rows once all have
arrived, and a split that stops waiting leaves its slice to the last one.  With a spin limit of
one poll most splits stop waiting, and the outputs must keep their bits; either way every row
matches the oracle and the workspace's counter region is zero again."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_24957_amd as D
from paper_2606_24957_amd import workloads as W
from tests.gpu_util import bits, check_attention, gpu_rows, scale_of
from tests.test_gpu_attention import _random_selection, _shape

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _counters_clear():
    key = (str(torch.device("cuda", torch.cuda.current_device())), int(torch.cuda.current_stream().cuda_stream), "attn")
    buf = D._WS[key]
    off = (-buf.data_ptr()) % 256
    assert int(buf[off:off + (1 << 18)].count_nonzero()) == 0


# four splits (the fewest that share), an odd number, one slice per row or less, the most; rows of
# one, three, five and eight row tiles; the default rule's own counts (None) at 16 to 63 steps
@pytest.mark.parametrize("splits,B,n,t,Hq,Hkv,k,paged", [
    (4, 1, 1500, 5, 64, 8, 700, False), (5, 2, [1500, 90], [5, 3], 28, 4, 700, True),
    (7, 1, 900, 1, 8, 1, 600, False), (16, 2, [2000, 1111], [9, 4], 64, 8, 900, False),
    (32, 1, 3000, 16, 64, 8, 2000, False), (32, 1, 2500, 2, 8, 1, 1024, True),
    (None, 1, 4000, 5, 64, 8, 512, False), (None, 1, 4000, 5, 8, 1, 480, False),
    (None, 2, [4000, 600], [5, 5], 28, 4, 1024, True), (None, 1, 4000, 7, 64, 8, 2016, False),
])
def test_shared_merge(splits, B, n, t, Hq, Hkv, k, paged, monkeypatch):
    if splits:
        monkeypatch.setenv("DUSTIN_ATTN_SPLITS", str(splits))
    s = _shape(B, n, t, Hq, Hkv, k, paged, seed=31, name=f"merge{splits}")
    L = W.make_layer(s, 0, DEV)
    seq = torch.tensor(s.seq_lens, dtype=torch.int32, device=DEV)
    nq = torch.tensor(s.n_query, dtype=torch.int32, device=DEV)
    idx_np, cnt_np = _random_selection(s, 1, 5, ())
    idx, cnt = torch.from_numpy(idx_np).to(DEV), torch.from_numpy(cnt_np).to(DEV)
    outs = {}
    for spins in (None, 1):
        if spins:
            monkeypatch.setenv("DUSTIN_ATTN_MERGE_SPINS", str(spins))
        for kind in ("sparse", "dense"):
            out = torch.full_like(L.q, float("nan"))
            for _ in range(2):
                if kind == "sparse":
                    D.sparse_verify_attn(L.q, L.k, L.v, idx, cnt, seq, n_query=nq, page_table=L.page_table, out=out)
                else:
                    D.dense_verify_attn(L.q, L.k, L.v, seq, n_query=nq, page_table=L.page_table, out=out)
            torch.cuda.synchronize()
            _counters_clear()
            outs[kind, spins] = out
    kk, vv = L.contiguous_kv(s)
    rows = O.all_rows(s.B, s.n_query, s.num_q_heads)
    for kind in ("sparse", "dense"):
        sel = dict(idx=idx_np, count=cnt_np) if kind == "sparse" else {}
        ref = O.attention(bits(L.q), bits(kk), bits(vv), s.seq_lens, scale_of(s.head_dim), rows, **sel)
        check_attention(gpu_rows(outs[kind, None], rows), ref, f"{s.name} {kind}")
        assert torch.equal(outs[kind, None].view(torch.int16), outs[kind, 1].view(torch.int16))


# one long sequence among short or empty ones: its pairs take more splits than the merge has slices
# (some 60, some 160, and where an empty pair has no step, with four row tiles, all 256)
@pytest.mark.parametrize("Hq,Hkv,n,t", [
    (32, 4, [16000, 90], [5, 3]), (8, 1, [20000] + [40] * 7, [5] * 8), (4, 1, [32752] + [0] * 7, [16] + [0] * 7),
])
@pytest.mark.parametrize("spins", [None, 1])
def test_more_splits_than_slices(Hq, Hkv, n, t, spins, monkeypatch):
    if spins:
        monkeypatch.setenv("DUSTIN_ATTN_MERGE_SPINS", str(spins))
    g = torch.Generator(device=DEV).manual_seed(5)
    B, N, T = len(n), max(n) + max(t), max(t)
    q = torch.randn(B, T, Hq, 128, device=DEV, dtype=torch.bfloat16, generator=g)
    k, v = (torch.randn(B, N, Hkv, 128, device=DEV, dtype=torch.bfloat16, generator=g) for _ in range(2))
    seq, nq = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in (n, t))
    out = torch.full_like(q, float("nan"))
    for _ in range(2):
        D.dense_verify_attn(q, k, v, seq, n_query=nq, out=out)
    torch.cuda.synchronize()
    _counters_clear()
    rows = O.all_rows(B, t, Hq)
    ref = O.attention(bits(q), bits(k), bits(v), n, scale_of(128), rows)
    check_attention(gpu_rows(out, rows), ref, f"{Hq}/{Hkv} {n}")


@pytest.mark.parametrize("B,Hkv,n,units", [(1, 8, 2048, 64), (4, 8, 630, 64), (3, 1, 4000, 45), (2, 4, 512, 16)])
def test_less_scratch_takes_larger_splits(B, Hkv, n, units):
    """A workspace for splits of eight steps, as a program may have sized it for a larger batch of the
    same tokens, still does; a smaller one is refused."""
    Hq, t = Hkv * 8, 5
    g = torch.Generator(device=DEV).manual_seed(n)
    q = torch.randn(B, t, Hq, 128, device=DEV, dtype=torch.bfloat16, generator=g)
    k, v = (torch.randn(B, n + t, Hkv, 128, device=DEV, dtype=torch.bfloat16, generator=g) for _ in range(2))
    seq = torch.tensor([n - 3 * b for b in range(B)], dtype=torch.int32, device=DEV)
    out = torch.full_like(q, float("nan"))
    call = D.plan_dense_verify_attn(q, k, v, seq, max_len=n, out=out)
    rows_pad, full = 48, call._args[-2]
    less = (1 << 18) + sum(-(-units * rows_pad * x * 4 // 256) * 256 for x in (128, 2))
    assert less < full
    with_bytes = lambda x: D.Call(call._fn, call._args[:-2] + (x, call._args[-1]), call._what, call._keep, out)
    with pytest.raises(D.DustinError) as e:
        with_bytes(less - 1)()
    assert e.value.status == D.ERR_WORKSPACE
    for _ in range(2):
        with_bytes(less)()
    torch.cuda.synchronize()
    _counters_clear()
    rows = O.all_rows(B, [t] * B, Hq)
    ref = O.attention(bits(q), bits(k), bits(v), seq.tolist(), scale_of(128), rows)
    check_attention(gpu_rows(out, rows), ref, f"{B} x {Hkv} {n}")
