"""Batches of more than 128 (sequence, KV head) pairs, where pairs of equal length have one split
each: the unit slots that 256 workgroups leave over (past 192 pairs of 8192 tokens and more, as many
again as there are pairs) go to the longest pairs of an uneven batch, and whatever the lengths, every
row matches the oracle and the counters return to zero."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_24957_amd as D
from tests.gpu_util import bits, check_attention, gpu_rows, scale_of
from tests.test_gpu_attention_split_merge import _counters_clear

pytestmark = pytest.mark.gpu
DEV = "cuda"


# 129 pairs (the fewest; 127 slots over), 136 (one very long sequence), 248 (eight slots over, and two
# rounds), 255 (one slot over, and two rounds), 256, 257 (none); 2016 tokens, just below the rule; none at all
@pytest.mark.parametrize("B,Hkv,G,n,t", [
    (43, 3, 2, [6000] + [300 + 7 * b for b in range(42)], 3), (17, 8, 8, [9000] + [500] * 16, 5),
    (31, 8, 8, [3000, 0] + [900 - 20 * b for b in range(29)], 5), (31, 8, 1, [8200, 0] + [90 - b for b in range(29)], 5),
    (85, 3, 4, [2200] * 3 + [64] * 82, 1), (51, 5, 2, [9100] + [33] * 50, 3), (64, 4, 2, [2500] + [200] * 63, 2),
    (257, 1, 4, [2500] + [100] * 256, 2), (17, 8, 1, [300, 1, 0] + [2009] * 14, 2), (20, 8, 8, [2100] * 20, 5),
])
def test_uneven_batches(B, Hkv, G, n, t):
    Hq, N = Hkv * G, max(n)
    g = torch.Generator(device=DEV).manual_seed(B)
    q = torch.randn(B, t, Hq, 128, device=DEV, dtype=torch.bfloat16, generator=g)
    k, v = (torch.randn(B, N + t, Hkv, 128, device=DEV, dtype=torch.bfloat16, generator=g) for _ in range(2))
    nq = [max(1, t - b % 3) for b in range(B)]
    seq, nqt = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in (n, nq))
    rng = np.random.default_rng(B)
    K = min(N, 2048)
    idx_np, cnt_np = np.full((B, 1, K), -1, dtype=np.int32), np.zeros((B, 1), dtype=np.int32)
    for b in range(B):
        c = min(K, n[b])
        idx_np[b, 0, :c], cnt_np[b, 0] = np.sort(rng.choice(n[b], c, replace=False)) if n[b] else [], c
    idx, cnt = torch.from_numpy(idx_np).to(DEV), torch.from_numpy(cnt_np).to(DEV)
    rows = O.all_rows(B, nq, Hq)[::5]
    need = D.lib().dustin_attn_workspace(B, Hq, Hkv, t, N, 0)
    assert (need > 0) == (B * Hkv < 256 and N + t > 63 * 32)
    for sel in (None, dict(idx=idx_np, count=cnt_np)):
        out = torch.full_like(q, float("nan"))
        for _ in range(2):
            if sel is None:
                D.dense_verify_attn(q, k, v, seq, n_query=nqt, out=out)
            else:
                D.sparse_verify_attn(q, k, v, idx, cnt, seq, n_query=nqt, out=out)
        torch.cuda.synchronize()
        if need:
            _counters_clear()
        ref = O.attention(bits(q), bits(k), bits(v), n, scale_of(128), rows, **(sel or {}))
        check_attention(gpu_rows(out, rows), ref, f"{B} x {Hkv}")
