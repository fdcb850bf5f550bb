"""The score's chunk forms against the oracle at the edges of their rules: small calls in one
pass (score_once.hpp) with chunks of 256 and of 512 positions, one layer and a draft's three, one
shared column tile and one per KV head; and K read twice (score_reread.hip) with chunks of 512
and of 1024 positions, summed, per layer and counted by top key digit.  Lengths sit on, before
and after chunk and tile edges, with empty sequences, per-sequence query counts (none among
them), permuted pages, and scales of either sign and zero."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2606_24957_amd as D
from tests.gpu_util import bits, check_score, host, scale_of
from tests.test_gpu_score_single_pass import _paged, _sync_region_clear

pytestmark = pytest.mark.gpu
DEV = "cuda"
TARGET = (64, 8, 128, [0, 17, 34, 51])
DRAFT = (14, 2, 64, [0, 4, 7, 11])
ALL = (14, 2, 64, list(range(14)))


def _inputs(model, lens, nq, n_layers, seed, page_size=0):
    Hq, Hkv, d, _ = model
    B, N = len(lens), max(lens)
    g = torch.Generator(device=DEV).manual_seed(seed)
    qs = [torch.randn((B, max(nq), Hq, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(n_layers)]
    ks = [torch.randn((B, N, Hkv, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(n_layers)]
    kin, pt = ks, None
    if page_size:
        pairs = [_paged(k, page_size, seed + 1) for k in ks]
        kin, pt = [p for p, _ in pairs], pairs[0][1]
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=DEV)
    return qs, ks, kin, pt, i32(lens), i32(nq)


def _reference(model, q, k, lens, nq, scale, check):
    """Per checked sequence the fp64-computed score of one layer."""
    Hq, Hkv, d, heads = model
    return {b: O.score(bits(q[b:b + 1]), bits(k[b:b + 1, :max(lens[b], 1)]), [lens[b]], [nq[b]], heads, scale,
                       num_kv_heads=Hkv)[0, 0, :lens[b]].astype(np.float64) for b in check}


def _check(out, refs, lens, label):
    got = host(out)
    for b, n in enumerate(lens):
        assert np.all(got[b, 0, n:] == -5.0), f"{label}: positions past N_b of sequence {b} written"
        if b in refs:
            check_score(got[b, 0, :n], refs[b], n, f"{label} b={b} N_b={n}")


SMALL = [0, 1, 16, 255, 256, 257, 1023]                  # chunks of 256
LARGE = [11300, 512, 513, 511, 7, 0, 1025, 10000, 4097]  # 9 x 23 chunks of 512


@pytest.mark.parametrize("model,n_layers,nq_max,lens,page_size", [
    (TARGET, 1, 1, SMALL, 0), (TARGET, 1, 1, LARGE, 0), (TARGET, 1, 4, LARGE, 16),
    (DRAFT, 3, 4, SMALL, 0), (DRAFT, 3, 4, LARGE, 0), (DRAFT, 3, 3, SMALL, 4),
    (DRAFT, 3, 5, SMALL, 0), (DRAFT, 3, 6, LARGE, 16), (DRAFT, 3, 8, LARGE, 0),
    (DRAFT, 1, 8, SMALL, 0), (ALL, 1, 4, SMALL, 0), (ALL, 1, 3, SMALL, 64),
    # two and four layers at once, then two after two and one after one
    (DRAFT, 2, 4, SMALL, 0), (DRAFT, 4, 4, LARGE, 16), (DRAFT, 6, 2, SMALL, 0), (DRAFT, 8, 4, LARGE, 0),
    (DRAFT, 5, 4, LARGE, 16), (DRAFT, 7, 3, SMALL, 0),
])
def test_small_calls_in_one_pass(model, n_layers, nq_max, lens, page_size):
    nq = [max(0, nq_max - b % 3) if b else nq_max for b in range(len(lens))]
    qs, ks, kin, pt, seq, nqt = _inputs(model, lens, nq, n_layers, 100 + len(lens) + nq_max, page_size)
    N, d = max(lens), model[2]
    init = torch.rand((len(lens), 1, N), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV) / N
    out = torch.full((len(lens), 1, N), -5.0, device=DEV)
    call = D.plan_score_layers(qs, kin, seq, model[3], n_query=nqt, init=init, out=out, max_len=N, page_table=pt)
    for _ in range(2):  # the counters return to zero
        call()
    torch.cuda.synchronize()
    _sync_region_clear()
    refs = {b: host(init)[b, 0, :n].astype(np.float64) for b, n in enumerate(lens)}
    for q, k in zip(qs, ks):
        for b, r in _reference(model, q, k, lens, nq, scale_of(d), range(len(lens))).items():
            refs[b] = refs[b] + r
    _check(out, refs, lens, "once")


@pytest.mark.parametrize("scale", [-0.11, 0.0])
@pytest.mark.parametrize("model,n_layers,lens", [(DRAFT, 3, [700, 33]), (ALL, 1, [66000, 2100])])
def test_negative_and_zero_scale(scale, model, n_layers, lens):
    nq = [4, 3]
    qs, ks, kin, pt, seq, nqt = _inputs(model, lens, nq, n_layers, 200)
    out = torch.full((2, 1, max(lens)), -5.0, device=DEV)
    D.score_layers(qs, kin, seq, model[3], n_query=nqt, out=out, max_len=max(lens), scale=scale)
    torch.cuda.synchronize()
    _sync_region_clear()
    refs = {b: 0.0 for b in range(2)}
    for q, k in zip(qs, ks):
        for b, r in _reference(model, q, k, lens, nq, scale, range(2)).items():
            refs[b] = refs[b] + r
    _check(out, refs, lens, f"scale {scale}")


# 2 x 129 chunks of 512 positions: chunks of 512; 5 x 137: chunks of 1024
REREAD = [[65700, 1, ], [70000, 1023, 0, 1025, 16]]


@pytest.mark.parametrize("lens", REREAD)
@pytest.mark.parametrize("n_layers,per_layer,page_size", [(1, False, 0), (2, False, 0), (3, False, 16), (3, True, 0)])
def test_k_read_twice(lens, n_layers, per_layer, page_size):
    nq = [4 - b % 4 for b in range(len(lens))]
    qs, ks, kin, pt, seq, nqt = _inputs(ALL, lens, nq, n_layers, 300 + n_layers, page_size)
    N, B = max(lens), len(lens)
    if per_layer:
        out = torch.full((n_layers, B, 1, N), -5.0, device=DEV)
        for _ in range(2):
            D.score_per_layer(qs, kin, seq, ALL[3], n_query=nqt, out=out, max_len=N, page_table=pt)
        torch.cuda.synchronize()
        _sync_region_clear()
        for l in range(n_layers):
            _check(out[l], _reference(ALL, qs[l], ks[l], lens, nq, scale_of(64), range(B) if l == 1 else range(1, B)),
                   lens, f"layer {l}")
            one = torch.full((B, 1, N), -5.0, device=DEV)
            D.score(qs[l], kin[l], seq, ALL[3], n_query=nqt, out=one, max_len=N, page_table=pt)
            assert torch.equal(one, out[l])  # a layer has the same bits in a call of its own
        return
    out = torch.full((B, 1, N), -5.0, device=DEV)
    hist = D.digit_hist(B, DEV)
    plan = D.plan_score_layers(qs, kin, seq, ALL[3], n_query=nqt, out=out, max_len=N, page_table=pt)
    D.plan_score_calls([plan], digit_hists=[hist])()
    torch.cuda.synchronize()
    _sync_region_clear()
    refs = {b: 0.0 for b in range(B)}
    for q, k in zip(qs, ks):
        for b, r in _reference(ALL, q, k, lens, nq, scale_of(64), range(B)).items():
            refs[b] = refs[b] + r
    _check(out, refs, lens, "reread")
    got = host(out)
    for b, n in enumerate(lens):  # positive scores: the key is the bit pattern with the sign set
        keys = (got[b, 0, :n].view(np.uint32) | 0x80000000) >> 20
        assert np.array_equal(np.bincount(keys, minlength=4096), host(hist)[b])


@pytest.mark.parametrize("model,n_layers,nq_max,lens", [
    # small calls in one pass, up to and past their last chunk, in two passes and in 16-wave workgroups
    (TARGET, 3, 1, [9000, 1, 0, 4100]), (TARGET, 3, 1, [32768, 32767, 0, 5]), (TARGET, 3, 1, [32800, 40, 0, 5]),
    (DRAFT, 3, 4, [65536]), (DRAFT, 2, 4, [65537]), (DRAFT, 2, 4, [24700] * 15 + [3]), (DRAFT, 3, 5, [2048] * 4),
    (DRAFT, 3, 5, [2049] * 4), (ALL, 3, 4, [8192]), (ALL, 3, 4, [8193]),
    # K read twice from 512-position chunks on every CU on (fewer than 48 pairs: two), and not before
    (ALL, 3, 4, [32768] * 3 + [32700]), (ALL, 3, 4, [32256] * 4), (ALL, 3, 3, [32768] * 8), (ALL, 3, 3, [32768] * 4),
    # more (layer, sequence) units than there are counters: several launches
    (ALL, 24, 4, [1536] * 85 + [700]), (DRAFT, 32, 4, [257] * 65 + [0]),
])
def test_a_layer_has_the_bits_of_a_call_of_its_own(model, n_layers, nq_max, lens):
    B, N = len(lens), max(lens)
    nq = [max(1, nq_max - b % 3) if b else nq_max for b in range(B)]
    qs, ks, _, _, seq, nqt = _inputs(model, lens, nq, n_layers, 700 + N)
    out = torch.full((n_layers, B, 1, N), -5.0, device=DEV)
    for _ in range(2):
        D.score_per_layer(qs, ks, seq, model[3], n_query=nqt, out=out, max_len=N)
    torch.cuda.synchronize()
    _sync_region_clear()
    for l in range(n_layers):
        one = torch.full((B, 1, N), -5.0, device=DEV)
        D.score(qs[l], ks[l], seq, model[3], n_query=nqt, out=one, max_len=N)
        assert torch.equal(one, out[l]), f"layer {l}"
    sums = (out.double() * (out >= 0)).sum(dim=(2, 3)).cpu()
    want = torch.tensor([len(model[3]) * t if n else 0 for n, t in zip(lens, nq)], dtype=torch.float64)
    assert torch.allclose(sums, want.expand(n_layers, B), rtol=1e-4, atol=0)


@pytest.mark.parametrize("model,n_layers,nq_max,lens", [
    (TARGET, 1, 4, SMALL), (DRAFT, 3, 4, SMALL), (DRAFT, 3, 5, LARGE), (ALL, 1, 3, SMALL),
    (ALL, 1, 4, [65700, 1, 1023]), (ALL, 3, 3, [65700, 300, 1023]),
])
def test_padding_queries_count_for_nothing(model, n_layers, nq_max, lens):
    """Query rows past nq_b and key rows past N_b hold NaN and infinities, with nq_b of 0, 1 and
    some: the outputs are those of the same call with zeros there, to the bit."""
    nq = [(nq_max, 1, 0, nq_max - 1)[b % 4] for b in range(len(lens))]
    qs, ks, _, _, seq, nqt = _inputs(model, lens, nq, n_layers, 500 + nq_max)
    N, outs = max(lens), []
    junk = (0.0, float("nan"), float("inf"))
    for fill in junk:
        for x in qs + ks:
            for b in range(len(lens)):
                x[b, (nq if x.shape[1] == max(nq) else lens)[b]:] = fill
        out = torch.full((len(lens), 1, N), -5.0, device=DEV)
        D.score_layers(qs, ks, seq, model[3], n_query=nqt, out=out, max_len=N)
        outs.append(out)
    torch.cuda.synchronize()
    _sync_region_clear()
    for b, n in enumerate(lens):
        got = outs[0][b, 0, :n]
        if n:  # the softmaxes sum to one
            assert abs(float(got.double().sum()) - n_layers * nq[b] * len(model[3])) <= 1e-4 * max(1, nq[b] * len(model[3]))
    for fill, out in zip(junk[1:], outs[1:]):
        assert torch.equal(out, outs[0]), f"{fill} in the padding shows"


@pytest.mark.parametrize("model,n_layers,lens", [(TARGET, 1, [1000, 40]), (DRAFT, 3, [1000, 40]), (ALL, 1, [65700, 40])])
def test_a_key_that_is_not_finite(model, n_layers, lens):
    """One key of infinities or NaNs: its own position is NaN, and no other (their share of a
    softmax over it is zero)."""
    qs, ks, _, _, seq, nqt = _inputs(model, lens, [3, 3], n_layers, 600)
    N = max(lens)
    for bad in (float("inf"), float("nan")):
        for k in ks:
            k[0, 37, :, 3] = bad
        out = D.score_layers(qs, ks, seq, model[3], n_query=nqt, max_len=N)
        torch.cuda.synchronize()
        _sync_region_clear()
        assert torch.equal(out[0, 0].isnan().nonzero().flatten().cpu(), torch.tensor([37])), bad
        assert not out[1, 0, :lens[1]].isnan().any()


# many chunks of a sequence: merged by all its workgroups together past 64 chunks of 96 columns or
# 128 of 48 while the call fits the chip in one round (the first three), else by each
MANY = [
    (5, [33000, 32768, 40000, 0, 1]), (8, [131072]), (4, [70000, 65536, 513]), (6, [40000] * 6 + [39000]),
]


@pytest.mark.parametrize("nq_max,lens", MANY)
def test_many_chunks_of_a_sequence(nq_max, lens):
    nq = [max(1, nq_max - b) for b in range(len(lens))]
    qs, ks, _, _, seq, nqt = _inputs(DRAFT, lens, nq, 3, 800 + nq_max)
    out = torch.full((len(lens), 1, max(lens)), -5.0, device=DEV)
    for _ in range(2):
        D.score_layers(qs, ks, seq, DRAFT[3], n_query=nqt, out=out, max_len=max(lens))
    torch.cuda.synchronize()
    _sync_region_clear()
    refs = {b: 0.0 for b in range(len(lens))}
    for q, k in zip(qs, ks):
        for b, r in _reference(DRAFT, q, k, lens, nq, scale_of(64), range(len(lens))).items():
            refs[b] = refs[b] + r
    _check(out, refs, lens, f"{lens}")


@pytest.mark.parametrize("model,n_layers,nq_max,lens,per_layer", [
    (TARGET, 1, 4, SMALL, False), (TARGET, 1, 1, LARGE, False), (DRAFT, 3, 4, LARGE, False), (DRAFT, 3, 6, SMALL, False),
    (DRAFT, 3, 8, LARGE, False), (ALL, 1, 4, SMALL, False), (ALL, 3, 4, [700, 2700], True),
    (DRAFT, 2, 4, LARGE, False), (DRAFT, 4, 4, [70000, 65536, 513], False), (DRAFT, 6, 4, SMALL, False),
    (DRAFT, 5, 4, LARGE, False),
    *[(DRAFT, 3, nq, lens, False) for nq, lens in MANY],
    (ALL, 1, 4, REREAD[0], False), (ALL, 3, 4, REREAD[1], False), (ALL, 2, 4, REREAD[1], True),
])
def test_a_wait_that_runs_out_changes_nothing(model, n_layers, nq_max, lens, per_layer, monkeypatch):
    """With one or three more looks at a counter many workgroups stop waiting for the others and form
    their statistics themselves: the outputs and digit counts keep their bits and the counters return to zero."""
    B, N = len(lens), max(lens)
    nq = [max(0, nq_max - b % 3) if b else nq_max for b in range(B)]
    qs, ks, _, _, seq, nqt = _inputs(model, lens, nq, n_layers, 900 + nq_max)
    got = {}
    for polls in (None, "1", "3"):
        if polls:
            monkeypatch.setenv("DUSTIN_SCORE_POLLS", polls)
        hist = D.digit_hist(B, DEV)
        if per_layer:
            out = torch.full((n_layers, B, 1, N), -5.0, device=DEV)
            D.score_per_layer(qs, ks, seq, model[3], n_query=nqt, out=out, max_len=N)
        else:
            out = torch.full((B, 1, N), -5.0, device=DEV)
            plan = D.plan_score_layers(qs, ks, seq, model[3], n_query=nqt, out=out, max_len=N)
            D.plan_score_calls([plan], digit_hists=[hist])()
        torch.cuda.synchronize()
        _sync_region_clear()
        got[polls] = (out, hist)
    for polls in ("1", "3"):
        assert torch.equal(got[polls][0], got[None][0]) and torch.equal(got[polls][1], got[None][1]), polls


@pytest.mark.parametrize("n_layers,gamma", [(1, 4), (2, 4), (3, 3), (3, 6), (4, 4), (5, 2), (6, 4)])
def test_a_pair_of_small_calls_has_the_bits_of_the_separate_calls(n_layers, gamma):
    """A step's target and draft calls in one launch, any count of draft layers, 17 pairs and more (three
    layers), both chunk sizes."""
    for lens in (SMALL, LARGE):
        B, N = len(lens), max(lens)
        qt, _, kt, _, seq, _ = _inputs(TARGET, lens, [1] * B, 1, 400)
        nq = [max(1, gamma - b % 4) for b in range(B)]
        qd, _, kd, _, _, nqt = _inputs(DRAFT, lens, nq, n_layers, 401)
        st, sd = torch.full((B, 1, N), -5.0, device=DEV), torch.full((B, 1, N), -5.0, device=DEV)
        t = D.plan_score(qt[0], kt[0], seq, TARGET[3], out=st, max_len=N)
        d = D.plan_score_layers(qd, kd, seq, DRAFT[3], n_query=nqt, out=sd, max_len=N, ws_tag="score_draft")
        t()
        d()
        ref_t, ref_d = st.clone(), sd.clone()
        st.fill_(-5.0)
        sd.fill_(-5.0)
        D.plan_score_calls([t, d])()
        torch.cuda.synchronize()
        assert torch.equal(st, ref_t) and torch.equal(sd, ref_d)
        for tag in ("score", "score_draft"):
            assert int(D.score_sync_region(tag=tag).count_nonzero()) == 0
