"""Both passes of the two-pass scoring in one launch (wide_once in csrc/snapkv_wide.hip): a single prompt whose slices all find a place at
once.  Its votes are those of the two launches, which layers of a call still take, bit for bit; so are the kept positions."""
import numpy as np
import pytest
import torch

from paper_2404_14469_amd import workloads
from parity import check_against_oracle, run_gpu
from test_gpu_decode import launched
from test_gpu_varlen import compare_with_single_calls, run_batch
from test_gpu_wide import outputs

pytestmark = pytest.mark.gpu


def work(L, g, W, Hkv=2, D=128, dtype="bf16", C=300, p=7, pool_kind=0):
    return workloads.Workload("wide_once", L=L, Hq=g * Hkv, Hkv=Hkv, D=D, W=W, pool_kind=pool_kind, p=p, C=C, dtype=dtype,
                              clusters=(5, 5), radius=6, layers=2, seed=5300)


# Workgroups (units x slices), or None where the two launches run.  Rounds of a slice: 1 (one buffer), 2 (both in LDS when the votes are taken), 3, 4
# (one and two are read again), 5, and last slices of one key.
CASES = {
    "one_round": (dict(L=6000, g=8, W=64), 8 * 47),
    "one_round_last_of_one_key": (dict(L=40 * 128 + 1, g=8, W=64, dtype="f16"), 8 * 41),
    "two_rounds_one_head": (dict(L=18433, g=4, W=32, Hkv=1), 73),
    "three_rounds": (dict(L=18500, g=4, W=32, Hkv=8), 8 * 49),
    "four_rounds": (dict(L=28471, g=4, W=32, Hkv=8, dtype="f16"), 8 * 56),
    "four_rounds_last_of_one_key": (dict(L=50 * 4 * 128 + 1, g=4, W=32, Hkv=8), 8 * 51),
    "five_rounds_last_of_one_key": (dict(L=52 * 5 * 128 + 1, g=4, W=31, Hkv=4, pool_kind=1, p=5), 4 * 53),
    "two_blocks_512_places": (dict(L=63 * 3 * 128 + 1, g=4, W=64, Hkv=4, p=13), 512),     # and a last slice of one key
    "eight_units_512_places": (dict(L=32768, g=4, W=32, Hkv=8), 512),
    # more than eight units: fewer slices, and all of them find a place
    "ten_units_51_slices": (dict(L=12900, g=4, W=64, Hkv=5, p=13), 510),
    "sixteen_units_32_slices": (dict(L=72001, g=4, W=64, Hkv=8, p=13, dtype="f16"), 512),
    "32_units_16_slices": (dict(L=19300, g=1, W=128, Hkv=32, C=300), 512),
    "33_units_64_slices": (dict(L=24400, g=1, W=113, Hkv=33, C=300), None),
    "d64_padded_rows": (dict(L=16500, g=3, W=48, Hkv=3, D=64), 6 * 43),
    "one_row_per_head": (dict(L=150001, g=8, W=1, Hkv=2), 2 * 118),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_one_launch_equals_two(snapkv, tmp_path, name):
    kw, groups = CASES[name]
    w = work(**kw)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)]
    got = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases for _ in range(2)]   # (scratch left by others)
    kernels = launched(lambda: run_gpu(snapkv, *(cases[0][n] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C), tmp_path)
    assert {size for n, size in kernels if "wide_once" in n} == ({groups} if groups else set()), kernels
    assert any("wide_stats" in n for n, _ in kernels) == (groups is None), kernels
    oks, ovs, ois = outputs(w, 2, cases[0]["k"].dtype)
    snapkv.snapkv_compress_layers(*([c[n] for c in cases] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, oks, ovs, ois)
    for l in range(2):
        for r in got[2 * l:2 * l + 2]:
            assert np.array_equal(ois[l].cpu().numpy(), r[3]) and torch.equal(oks[l], r[1]) and torch.equal(ovs[l], r[2]), l
        assert np.array_equal(got[2 * l][0], got[2 * l + 1][0])
    check_against_oracle(*(cases[1][n] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, *got[2], heads=[w.Hkv - 1])
    assert snapkv.snapkv_sync_timeouts() == 0


# From which length on a prompt of so many units comes here: one to three, four to eight, more (min_row_keys); 128, 256 and 512 window rows.
@pytest.mark.parametrize("first,kw,kernel", [(18432, dict(g=4, W=32, Hkv=3), "wide_once"), (16385, dict(g=4, W=32, Hkv=4), "wide_once"),
                                             (16385, dict(g=4, W=32, Hkv=8), "wide_once"), (8193, dict(g=4, W=64, Hkv=4), "wide_once"),
                                             (12288, dict(g=4, W=32, Hkv=9), "wide_once"), (6144, dict(g=4, W=64, Hkv=8), "wide_once"),
                                             (12288, dict(g=4, W=32, Hkv=33), "wide_stats"), (3072, dict(g=8, W=64, Hkv=9), "wide_stats")])
def test_where_the_line_stands(snapkv, tmp_path, first, kw, kernel):
    for L in (first - 1, first):
        w = work(L=L, **kw)
        c = workloads.generate(w, device="cuda")
        got = run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C)
        check_against_oracle(c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C, *got, heads=[0, w.Hkv - 1])
        kernels = {n for n, _ in launched(lambda: run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C), tmp_path)}
        assert any(kernel in n for n in kernels) == (L == first) and any("score_fused" in n for n in kernels) == (L < first), (L, kernels)
    assert snapkv.snapkv_sync_timeouts() == 0


HELPED = {
    "one_block": dict(L=28471, g=4, W=32, Hkv=8),
    "f16": dict(L=18433, g=4, W=32, Hkv=1, dtype="f16"),
    "d64": dict(L=16500, g=3, W=48, Hkv=3, D=64),
    "two_blocks": dict(L=12400, g=4, W=64, Hkv=5, p=13),
    "one_round": dict(L=6000, g=8, W=64),
    "raised": dict(L=18500, g=4, W=32, Hkv=2),               # a stretch of keys 129 nats above the first ones
    "paged": dict(L=18450, g=4, W=32, Hkv=4),
}


@pytest.mark.parametrize("name", sorted(HELPED))
def test_workgroups_that_do_not_wait_help_themselves(snapkv, tmp_path, name):
    """Waits bounded to no polls: a workgroup takes the statistics of every slice that it misses itself.  The same scores, those of
    the oracle, and the same kept positions as layers of a call, which take the two launches; nothing is given up."""
    w = work(**HELPED[name])
    c = workloads.generate(w, device="cuda")
    q, k, v = c["q_win"], c["k"], c["v"]
    if name == "raised":
        q[..., 3] += 12.0
        k[:, 0] = 0
        k[:, 7000:12000, 3] += 122.0
    if name == "paged":
        table, caches = pages_of(w, k, v)
    args = (w.pool_kind, w.p, w.C)
    oks, ovs, ois = outputs(w, 2, k.dtype)
    layers = launched(lambda: snapkv.snapkv_compress_layers([q] * 2, [k] * 2, [v] * 2, *args, oks, ovs, ois), tmp_path)
    assert any("wide_stats" in n for n, _ in layers) and not any("wide_once" in n for n, _ in layers), layers
    scores = [torch.empty((w.Hkv, w.n), dtype=torch.float32, device="cuda") for _ in range(3)]
    try:
        snapkv.snapkv_set_scoring_scheme(2)                  # (a selection without waits)
        for s, polls in zip(scores, (-1, 0, 1)):
            snapkv.snapkv_debug_set_wait_limit(polls)
            (ok,), (ov,), (oi,) = outputs(w, 1, k.dtype)

            def call():
                if name == "paged":
                    snapkv.snapkv_compress_paged(q, *caches, table, w.L, *args, ok, ov, oi)
                else:
                    snapkv.snapkv_compress(q, k, v, *args, ok, ov, oi)
                snapkv.snapkv_pooled_scores(q, k, w.pool_kind, w.p, s)

            kernels = launched(call, tmp_path)
            assert sum("wide_once" in n for n, _ in kernels) == 2 and not any("wide_stats" in n for n, _ in kernels), kernels
            assert torch.equal(oi, ois[1]) and torch.equal(ok, oks[1]) and torch.equal(ov, ovs[1]), polls
        assert snapkv.snapkv_sync_timeouts() == 0
    finally:
        snapkv.snapkv_set_scoring_scheme(0)
        snapkv.snapkv_debug_set_wait_limit(-2)
    assert torch.equal(scores[0], scores[1]) and torch.equal(scores[0], scores[2])
    check_against_oracle(q, k, v, *args, scores[1].cpu().numpy(), ok, ov, oi.cpu().numpy(), w.C, heads=[w.Hkv - 1])


def pages_of(w, k, v, page=16):
    pages = (w.L + page - 1) // page
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(3)).to("cuda", torch.int32)
    caches = []
    for x in (k, v):
        rows = torch.zeros((pages * page, w.Hkv, w.D), dtype=x.dtype, device="cuda")
        rows[:w.L] = x.transpose(0, 1)
        cache = torch.empty((pages, page, w.Hkv, w.D), dtype=x.dtype, device="cuda")
        cache[table.long()] = rows.view(pages, page, w.Hkv, w.D)
        caches.append(cache)
    return table, caches


def test_two_streams_with_workspaces(snapkv, tmp_path):
    """Calls on distinct workspaces may overlap, and none of their launches has the chip to itself then."""
    w = work(L=30011, g=4, W=32, Hkv=8)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)]
    good = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    size = snapkv.snapkv_workspace_bytes(w.L, w.Hq, w.Hkv, w.D, w.W)
    ws = [torch.full((size,), 255, dtype=torch.uint8, device="cuda") for _ in cases]
    outs = [[torch.zeros((w.Hkv, w.C, w.D), dtype=c["k"].dtype, device="cuda") for _ in "kv"]
            + [torch.zeros((w.Hkv, w.C), dtype=torch.int32, device="cuda")] for c in cases]
    status = [torch.zeros(1, dtype=torch.int32, device="cuda") for _ in cases]
    streams = [torch.cuda.Stream() for _ in cases]

    def calls():
        for c, s, space, st, (ok, ov, oi) in zip(cases, streams, ws, status, outs):
            with torch.cuda.stream(s):
                snapkv.snapkv_compress_ws_status(c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C, ok, ov, oi, space, st)

    kernels = launched(calls, tmp_path)
    assert sum("wide_once" in n for n, _ in kernels) == len(cases), kernels
    for _ in range(10):
        calls()
    torch.cuda.synchronize()
    for g, st, (ok, ov, oi) in zip(good, status, outs):
        assert int(st.item()) == w.C and np.array_equal(oi.cpu().numpy(), g[3]) and torch.equal(ok, g[1]) and torch.equal(ov, g[2])


# One prompt of a batch in one launch, more in the two; beside prompts of the joint launches and one that fits the capacity.
@pytest.mark.parametrize("lengths,once,kw", [([8192, 17300, 5000, 290], True, dict(g=4, W=32, Hkv=8)), ([131072, 600], True, dict(g=4, W=64, Hkv=8, p=13, dtype="f16")),
                                             ([16385, 16384], True, dict(g=4, W=31, Hkv=5, pool_kind=1, p=5)), ([17300, 16400, 3000], False, dict(g=4, W=32, Hkv=8)),
                                             ([18561, 2000], False, dict(g=1, W=113, Hkv=33))])
def test_batches(snapkv, tmp_path, lengths, once, kw):
    ws = [work(L=L, **kw).with_(seed=5400 + i) for i, L in enumerate(lengths)]
    for _ in range(2):                   # (the second call's words lie where the first one's were)
        batch = run_batch(snapkv, ws)
        compare_with_single_calls(snapkv, ws, *batch)
    kernels = {n for n, _ in launched(lambda: run_batch(snapkv, ws), tmp_path)}
    assert any("wide_once" in n for n in kernels) == once and any("wide_stats" in n for n in kernels) != once, kernels
    assert snapkv.snapkv_sync_timeouts() == 0
