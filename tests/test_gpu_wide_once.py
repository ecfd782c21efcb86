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


# rounds of a slice: 2 (both in LDS when the votes are taken), 3, 4 (one and two are read again), 5 with a last slice of one key
CASES = {
    "two_rounds_one_head": (dict(L=18433, g=4, W=32, Hkv=1), True),
    "three_rounds": (dict(L=18500, g=4, W=32, Hkv=8), True),
    "four_rounds": (dict(L=28471, g=4, W=32, Hkv=8, dtype="f16"), True),
    "five_rounds_one_key": (dict(L=64 * 4 * 128 + 1, g=4, W=31, Hkv=4, pool_kind=1, p=5), True),
    "two_blocks_512_places": (dict(L=20001, g=4, W=64, Hkv=4, p=13), True),
    # more than eight units: fewer slices, and all of them find a place
    "ten_units_51_slices": (dict(L=9300, g=4, W=64, Hkv=5, p=13), True),
    "sixteen_units_long_slices": (dict(L=70001, g=4, W=64, Hkv=8, p=13, dtype="f16"), True),
    "32_units_16_slices": (dict(L=18561, g=1, W=128, Hkv=32, C=300), True),
    "33_units": (dict(L=18561, g=1, W=113, Hkv=33, C=300), False),                    # 64 slices, the two launches
    "d64_padded_rows": (dict(L=16500, g=3, W=48, Hkv=3, D=64), True),
    "one_row_per_head": (dict(L=150001, g=8, W=1, Hkv=2), True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_one_launch_equals_two(snapkv, tmp_path, name):
    kw, once = CASES[name]
    w = work(**kw)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)]
    got = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases for _ in range(2)]   # (scratch left by others)
    kernels = {n for n, _ in launched(lambda: run_gpu(snapkv, *(cases[0][n] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C), tmp_path)}
    assert any("wide_once" in n for n in kernels) == once and any("wide_stats" in n for n in kernels) != once, kernels
    oks, ovs, ois = outputs(w, 2, cases[0]["k"].dtype)
    snapkv.snapkv_compress_layers(*([c[n] for c in cases] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, oks, ovs, ois)
    for l in range(2):
        for r in got[2 * l:2 * l + 2]:
            assert np.array_equal(ois[l].cpu().numpy(), r[3]) and torch.equal(oks[l], r[1]) and torch.equal(ovs[l], r[2]), l
        assert np.array_equal(got[2 * l][0], got[2 * l + 1][0])
    check_against_oracle(*(cases[1][n] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, *got[2], heads=[w.Hkv - 1])
    assert snapkv.snapkv_sync_timeouts() == 0


# From which length on a prompt of so many units comes here: one to three, four to eight, more (min_row_keys); 128 and 256 window rows.
@pytest.mark.parametrize("first,kw", [(18432, dict(g=4, W=32, Hkv=3)), (16385, dict(g=4, W=32, Hkv=4)), (16385, dict(g=4, W=32, Hkv=8)),
                                      (8193, dict(g=4, W=64, Hkv=4)), (12288, dict(g=4, W=32, Hkv=9)), (6144, dict(g=4, W=64, Hkv=8))])
def test_where_the_line_stands(snapkv, tmp_path, first, kw):
    for L in (first - 1, first):
        w = work(L=L, **kw)
        c = workloads.generate(w, device="cuda")
        got = run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C)
        check_against_oracle(c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C, *got, heads=[0, w.Hkv - 1])
        kernels = {n for n, _ in launched(lambda: run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C), tmp_path)}
        assert any("wide_once" in n for n in kernels) == (L == first) and any("score_fused" in n for n in kernels) == (L < first), (L, kernels)
    assert snapkv.snapkv_sync_timeouts() == 0


@pytest.mark.parametrize("kw", [dict(L=28471, g=4, W=32, Hkv=8), dict(L=18433, g=4, W=32, Hkv=1, dtype="f16"), dict(L=16500, g=3, W=48, Hkv=3, D=64)])
def test_workgroups_that_do_not_wait_help_themselves(snapkv, kw):
    """Waits bounded to no polls: a workgroup takes the statistics of every slice that it misses itself.  Same scores, nothing given up."""
    w = work(**kw)
    c = workloads.generate(w, device="cuda")
    scores = [torch.empty((w.Hkv, w.n), dtype=torch.float32, device="cuda") for _ in range(3)]
    try:
        for s, polls in zip(scores, (-1, 0, 1)):
            snapkv.snapkv_debug_set_wait_limit(polls)
            snapkv.snapkv_pooled_scores(c["q_win"], c["k"], w.pool_kind, w.p, s)
            torch.cuda.synchronize()
        assert snapkv.snapkv_sync_timeouts() == 0
    finally:
        snapkv.snapkv_debug_set_wait_limit(-2)
    assert torch.equal(scores[0], scores[1]) and torch.equal(scores[0], scores[2])


def test_two_streams_with_workspaces(snapkv):
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
    torch.cuda.synchronize()
    for _ in range(10):
        for c, s, space, st, (ok, ov, oi) in zip(cases, streams, ws, status, outs):
            with torch.cuda.stream(s):
                snapkv.snapkv_compress_ws_status(c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C, ok, ov, oi, space, st)
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
