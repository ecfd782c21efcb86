"""Pooling and selection in one launch (csrc/snapkv_topk.hip, pool_select): the first digit has fixed bins of 1/64 octave
around the mean score, so the threshold can fall into either end bin, into a bin that holds more positions than the
candidate list, into one of at most 128 (counted directly) or more (searched by digits), or of more than a workgroup has words
in the exchange; a head may have one
workgroup or many, and rows of votes whose length is no multiple of four are padded.  Whatever the route, the kept
set is exactly the top-k of the call's own pooled scores."""
import numpy as np
import pytest
import torch

from parity import check_against_oracle, check_self_consistency, run_gpu

pytestmark = pytest.mark.gpu

D = 64


def flat(q, k):
    q.zero_()                       # all scores equal: ties down to the first positions


def few_spikes(q, k):               # every other score lies far below the lowest bin
    q[..., 0] += 40.0
    k[:, 100:110, 0] += 12.0


def two_fields(q, k):               # half of the scores equal to the last bit, the others spread
    k[:, ::2] = k[:, :1]


def as_drawn(q, k):
    pass


SHAPES = [  # L, Hq, Hkv, W, C, p, dtype
    (300, 4, 2, 16, 40, 5, torch.float32),         # one workgroup per head
    (515, 4, 4, 32, 33, 7, torch.float32),         # ... and one kept position
    (2081, 2, 2, 32, 1000, 7, torch.bfloat16),
    (6145, 8, 2, 32, 300, 7, torch.bfloat16),      # three workgroups, odd rows, a group of four query heads
    (9003, 2, 1, 16, 8000, 5, torch.float16),      # nearly everything kept
    (20018, 2, 2, 16, 20, 1, torch.bfloat16),      # four kept: with spikes the threshold lies in the top bin
    (131071, 4, 4, 32, 2048, 13, torch.bfloat16),
]


@pytest.mark.parametrize("field", [as_drawn, flat, few_spikes, two_fields], ids=lambda f: f.__name__)
@pytest.mark.parametrize("L,Hq,Hkv,W,C,p,dtype", SHAPES)
def test_kept_set_is_the_exact_top_k(snapkv, field, L, Hq, Hkv, W, C, p, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q = torch.randn((Hq, W, D), generator=gen, device="cuda")
    k = torch.randn((Hkv, L, D), generator=gen, device="cuda")
    field(q, k)
    q, k = q.to(dtype), k.to(dtype)
    v = torch.randn((Hkv, L, D), generator=gen, device="cuda").to(dtype)
    for pool_kind in (0, 1):
        res = run_gpu(snapkv, q, k, v, pool_kind, p, C)
        check_self_consistency(q, k, v, C, *res)


def narrow(q, k):                   # a stretch of scores within one bin, far above the others
    k[:, 1000:1400] = k[:, 1000:1001] + 1e-3 * k[:, 1000:1400]
    k[:, 1000:1400, 0] += 12.0
    q[..., 0] += 8.0


@pytest.mark.parametrize("field", [as_drawn, narrow], ids=lambda f: f.__name__)
@pytest.mark.parametrize("L,groups,heads", [
    (9001, 4, 1), (83983, 40, 1), (83985, 41, 1), (84008, 41, 1), (131072, 63, 1), (165903, 80, 1), (165904, 81, 1), (165921, 81, 1),
    (83983, 40, 3), (83984, 41, 3), (165903, 80, 3), (165904, 81, 3)])
def test_exchange_of_candidates(snapkv, field, L, groups, heads):
    """One head's workgroups exchange 64 words each (up to 40 workgroups), 32 (up to 80) or go the general way; so does a head
    one of whose workgroups has more candidates than words.  40 and 80 workgroups fill a head's words to the last, and
    the next head's bins follow them."""
    assert (L - 16) // 2048 == groups               # a workgroup for every 2048 positions
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q = torch.randn((heads, 16, D), generator=gen, device="cuda")
    k = torch.randn((heads, L, D), generator=gen, device="cuda")
    field(q, k)
    q, k = q.bfloat16(), k.bfloat16()
    for C in (216, 1016):
        res = run_gpu(snapkv, q, k, k, 0, 1, C)
        check_self_consistency(q, k, k, C, *res)


@pytest.mark.parametrize("field", [as_drawn, flat, few_spikes, two_fields], ids=lambda f: f.__name__)
@pytest.mark.parametrize("layers,L,Hq,Hkv,W,C,p,dtype", [
    (40, 9001, 16, 8, 32, 700, 7, torch.bfloat16),   # more heads than the one-launch kernel keeps resident: votes read once
    (66, 4100, 4, 4, 16, 600, 5, torch.float16),     # too short to sample: the separate kernels
    (36, 8209, 8, 8, 32, 8000, 13, torch.bfloat16),  # nearly everything kept: the separate kernels
    (20, 20483, 16, 16, 16, 17, 1, torch.bfloat16),  # one position kept per head
])
def test_many_heads_keep_what_single_calls_keep(snapkv, field, layers, L, Hq, Hkv, W, C, p, dtype):
    """Stacked layers, whose selection samples a lower bound of the threshold and finishes among the positions
    above it (a sample that misleads costs time only): bit for bit the single calls' kept sets."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q = torch.randn((layers * Hq, W, D), generator=gen, device="cuda")
    k = torch.randn((layers * Hkv, L, D), generator=gen, device="cuda")
    field(q, k)
    q, k = q.to(dtype), k.to(dtype)
    ok = torch.empty((layers * Hkv, C, D), dtype=dtype, device="cuda")
    ov = torch.empty_like(ok)
    oi = torch.full((layers * Hkv, C), -1, dtype=torch.int32, device="cuda")
    lists = [list(t.split(t.shape[0] // layers)) for t in (q, k, k, ok, ov, oi)]
    for pool_kind in (0, 1):
        snapkv.snapkv_compress_layers(*lists[:3], pool_kind, p, C, *lists[3:])
        for l in (0, 1, layers - 1):
            res = run_gpu(snapkv, lists[0][l], lists[1][l], lists[2][l], pool_kind, p, C)
            assert (lists[5][l].cpu().numpy() == res[3]).all(), (l, pool_kind)
            assert torch.equal(lists[3][l], res[1]) and torch.equal(lists[4][l], res[2]), (l, pool_kind)


@pytest.mark.parametrize("heads,L,kcount,once", [
    (1024, 616, 100, True),       # too short to sample, but few positions in all
    (512, 1040, 900, True),
    (1024, 617, 100, False),
    (512, 1041, 100, False),
    (1024, 2048, 200, False),
    (1024, 8191, 200, False),
    (1024, 8208, 500, True),
    (1024, 8208, 6000, False),    # the candidates of a head cost more than the scores of all
    (600, 20016, 1000, True),
    (600, 20016, 10000, False),
])
def test_votes_are_read_once_only_where_that_is_faster(snapkv, heads, L, kcount, once):
    """The rule of pool_pick_ok: short prompts and large kept shares go through the kernels that store the scores (the
    stage pool_group), which are twice as fast there.  Either way the kept positions are a single call's."""
    Hkv, W, D = 8, 16, 64
    layers, C = heads // Hkv, kcount + W
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    q = torch.randn((layers * Hkv, W, D), generator=gen, device="cuda").bfloat16()
    k = torch.randn((layers * Hkv, L, D), generator=gen, device="cuda").bfloat16()
    ok = torch.empty((layers * Hkv, C, D), dtype=torch.bfloat16, device="cuda")
    ov = torch.empty_like(ok)
    oi = torch.full((layers * Hkv, C), -1, dtype=torch.int32, device="cuda")
    lists = [list(t.split(Hkv)) for t in (q, k, k, ok, ov, oi)]
    snapkv.snapkv_profile_start(1)
    snapkv.snapkv_compress_layers(*lists[:3], 0, 5, C, *lists[3:])
    stages, calls = snapkv.snapkv_profile_stop()
    assert calls == 1 and (stages["pool_group"] == 0.0) == once, stages
    for l in (0, layers - 1):
        res = run_gpu(snapkv, lists[0][l], lists[1][l], lists[2][l], 0, 5, C)
        assert (lists[5][l].cpu().numpy() == res[3]).all(), l


@pytest.mark.parametrize("pool_kind,p", [(0, 1), (0, 5), (1, 5)])
def test_heads_whose_sample_misleads_are_collected_again(snapkv, pool_kind, p):
    """Only the 2048 sampled positions (runs of four, evenly spread) score high, and more positions than those are kept: the
    sample's lower bound lets too few candidates through and pick_finish has to take all of the head's positions."""
    layers, Hkv, L, W, D, kc = 20, 8, 40032, 16, 64, 3000
    n, C = L - W, kc + W
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    u = torch.zeros(D, device="cuda")
    u[7] = 1.0
    q = torch.randn((layers * Hkv, W, D), generator=gen, device="cuda") * 0.5 + 8 * u
    k = torch.randn((layers * Hkv, L, D), generator=gen, device="cuda")
    sampled = ((n - 4) * torch.arange(512) // 511 & ~3).unsqueeze(1) + torch.arange(4)
    k[:, sampled.flatten().cuda()] += 8 * u
    q, k = q.bfloat16(), k.bfloat16()
    v = torch.randn((layers * Hkv, L, D), generator=gen, device="cuda").bfloat16()
    ok = torch.empty((layers * Hkv, C, D), dtype=torch.bfloat16, device="cuda")
    ov = torch.empty_like(ok)
    oi = torch.full((layers * Hkv, C), -1, dtype=torch.int32, device="cuda")
    lists = [list(t.split(Hkv)) for t in (q, k, v, ok, ov, oi)]
    snapkv.snapkv_profile_start(1)
    snapkv.snapkv_compress_layers(*lists[:3], pool_kind, p, C, *lists[3:])
    stages, calls = snapkv.snapkv_profile_stop()
    assert calls == 1 and stages["pool_group"] == 0.0 and stages["select_topk"] > 0.0, stages
    for l in (0, 7, layers - 1):
        res = run_gpu(snapkv, lists[0][l], lists[1][l], lists[2][l], pool_kind, p, C)
        assert (lists[5][l].cpu().numpy() == res[3]).all(), l
        assert torch.equal(lists[3][l], res[1]) and torch.equal(lists[4][l], res[2]), l
        # the sample's bound as pick_bracket takes it: digits of 2^17 patterns from 1/64 of the mean on
        want = 2048 * kc / n
        rank = int(want + 5 * (4 * want) ** 0.5 + 8)
        lo0 = int(np.float32(np.float32(W / n) * np.float32(1 / 64)).view(np.uint32))
        bits = res[0].view(np.uint32).astype(np.int64)
        digits = np.clip((bits - lo0) >> 17, 0, 2047)
        tlo = lo0 + (np.sort(digits[:, sampled.flatten().numpy()], axis=1)[:, -rank] << 17)
        assert ((bits >= tlo[:, None]).sum(axis=1) < kc).all()


@pytest.mark.parametrize("pool_kind", [0, 1])
@pytest.mark.parametrize("p", [1, 5, 7, 13])
def test_votes_read_once_pool_as_single_calls(snapkv, p, pool_kind):
    """Runs of four positions that share their taps, over two chunks and a ragged end (8210 positions), two query heads a KV
    head; the single call pools the same votes in another kernel."""
    layers, Hq, Hkv, L, W, C = 40, 16, 8, 8226, 16, 120
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p)
    q = torch.randn((layers * Hq, W, D), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((layers * Hkv, L, D), generator=gen, device="cuda").bfloat16() for _ in range(2))
    ok = torch.empty((layers * Hkv, C, D), dtype=torch.bfloat16, device="cuda")
    ov = torch.empty_like(ok)
    oi = torch.full((layers * Hkv, C), -1, dtype=torch.int32, device="cuda")
    lists = [list(t.split(h)) for t, h in ((q, Hq), (k, Hkv), (v, Hkv), (ok, Hkv), (ov, Hkv), (oi, Hkv))]
    snapkv.snapkv_profile_start(1)
    snapkv.snapkv_compress_layers(*lists[:3], pool_kind, p, C, *lists[3:])
    stages, _ = snapkv.snapkv_profile_stop()
    assert stages["pool_group"] == 0.0 and stages["select_topk"] > 0.0, stages
    for l in (0, 21, layers - 1):
        res = run_gpu(snapkv, lists[0][l], lists[1][l], lists[2][l], pool_kind, p, C)
        assert (lists[5][l].cpu().numpy() == res[3]).all(), l
        check_against_oracle(lists[0][l], lists[1][l], lists[2][l], pool_kind, p, C, *res)
