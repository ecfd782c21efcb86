"""Prompts whose KV heads are met by 128 window rows or more, long enough for the two-pass scoring kernels
(csrc/snapkv_wide.hip), or by 64 and longer than 131072 keys (163839 with two query heads of W = 32): edges of rounds (128 keys),
of slices (multiples of 128 keys, at most 64 of them, 256 where a prompt has few units, fewer where it has more than eight) and of the
row blocks (128 rows, whole query heads), every storage type and layout, and rows whose sums leave the fp32 range."""
import re

import numpy as np
import pytest
import torch

from paper_2404_14469_amd import workloads
from paper_2404_14469_amd.workloads import Workload
from parity import check_against_oracle, run_gpu
from test_gpu_decode import launched

pytestmark = pytest.mark.gpu

MIN_ROW_KEYS = 9 << 18   # csrc/snapkv_wide.hip: window rows times keys from which these kernels are used for any number of units (min_row_keys)


def work(L, g, W, Hkv=2, D=128, dtype="bf16", C=300, p=7, pool_kind=0):
    assert g * (-(-W // 16)) >= 8 and g * 16 * (-(-W // 16)) * L >= MIN_ROW_KEYS, "not a shape of the two-pass kernels"
    return Workload("wide", L=L, Hq=g * Hkv, Hkv=Hkv, D=D, W=W, pool_kind=pool_kind, p=p, C=C, dtype=dtype, clusters=(5, 5),
                    radius=6, layers=2, seed=5200)


CASES = {
    "w32_first": work(18432, 4, 32),                       # the shortest of this width; whole rounds
    "w32_one_more": work(18433, 4, 32),                    # one key in the last round
    "w32_round_edge": work(18432 + 127, 4, 32, pool_kind=1, p=5),
    "w64_two_blocks": work(9216 + 31, 4, 64, p=13),        # 256 rows: two blocks per KV head
    "w128_one_head": work(18500, 1, 128, Hkv=3),           # a block is one query head
    "w16_eight_heads": work(18437, 8, 16, p=5),
    "w48_padded": work(16400, 3, 48),                      # nine row units: blocks of six, padded to eight
    "w31_padded_rows": work(18450, 4, 31),
    "g5_uneven_blocks": work(14800, 5, 32),                # five heads of two units: blocks of three and two heads
    "d64_f16": work(18439, 4, 32, D=64, dtype="f16"),
    "f16": work(18441, 4, 32, dtype="f16"),
    "many_slices": work(40001, 4, 32, Hkv=1, C=1024),
    # prompts of few heads are cut into up to 256 slices per head instead of 64, of two rounds at least
    "one_head_256_slices": work(65536, 4, 32, Hkv=1),
    "one_head_171_slices": work(65537, 4, 32, Hkv=1),              # the last one holds one key
    "two_heads_128_slices": work(2 * 16384 - 5, 4, 32),
    "three_heads_85_slices": work(85 * 256, 4, 32, Hkv=3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_against_oracle(snapkv, name):
    w = CASES[name]
    case = workloads.generate(w, device="cuda")
    res = run_gpu(snapkv, case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C)
    check_against_oracle(case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C, *res)


# 64 window rows per KV head: blocks of four row units, prompts longer than 131072 keys
HALF = {
    "w16_first": dict(L=131073, g=4, W=16),                # the shortest; one key in the last round
    "w13_padded_rows": dict(L=131072 + 129, g=4, W=13, pool_kind=1, p=5),
    "w64_one_head": dict(L=131073 + 126, g=1, W=64, Hkv=2, p=13),
    "w50_padded_unit": dict(L=140001, g=1, W=50),          # the fourth row unit holds two rows
    "w32_two_heads": dict(L=163840, g=2, W=32),            # the shortest of this form
    "d64_f16": dict(L=131075, g=4, W=16, D=64, dtype="f16", Hkv=2),
    "five_heads": dict(L=132001, g=4, W=16, Hkv=5, C=5000),   # 64 slices per head
}


def half(L, g, W, Hkv=1, **kw):
    return work(1 << 20, 8, 16, **{"C": 1500, **kw}).with_(L=L, Hq=g * Hkv, Hkv=Hkv, W=W)


@pytest.mark.parametrize("name", sorted(HALF))
def test_64_rows_against_oracle(snapkv, name):
    w = half(**HALF[name])
    case = workloads.generate(w, device="cuda")
    res = run_gpu(snapkv, case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C)
    check_against_oracle(case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C, *res, heads=[w.Hkv - 1])


@pytest.mark.parametrize("L,g,W,two_passes", [(131072, 4, 16, False), (131073, 4, 16, True), (131072, 1, 64, False), (131073, 1, 64, True),
                                              (163839, 2, 32, False), (163840, 2, 32, True)])
def test_which_prompts_with_64_rows_take_the_two_passes(snapkv, tmp_path, L, g, W, two_passes):
    w = half(L, g, W)
    case = workloads.generate(w, device="cuda")
    kernels = launched(lambda: run_gpu(snapkv, case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C), tmp_path)
    for name in ("wide_stats", "wide_votes"):
        assert any(re.search(name + "<.*, 4>", n) for n, _ in kernels) == two_passes, kernels


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("at", [(5,), (60000,), tuple(range(16))])
def test_64_rows_and_keys_that_are_not_finite(snapkv, at, value):
    """Rows with an infinite or undefined logit have no votes to give, and that key's votes are undefined: as the single-read kernel
    (one key less) leaves them, whether the key is among those that the rows' origins come from or not."""
    w = half(131073, 4, 16)
    case = workloads.generate(w, device="cuda")
    q, k = case["q_win"], case["k"].clone()
    k[0, list(at), 3] = value
    votes = []
    for L in (w.L, w.L - 1):
        out = torch.empty((1, L - w.W), device="cuda")
        snapkv.snapkv_pooled_scores(q, k[:, :L].contiguous(), 0, 1, out)
        votes.append(out[0, :w.L - 1 - w.W])
    two, one = votes
    assert torch.equal(two.isnan(), one.isnan()) and torch.equal(two == 0, one == 0)
    real = ~one.isnan()
    # (the longer prompt has one more key in every row's sum: far less than one part in a thousand here)
    assert float(((two - one)[real].abs() - 1e-3 * one[real].abs()).max()) <= 1e-30


@pytest.mark.parametrize("g,W", [(4, 16), (1, 64)])
@pytest.mark.parametrize("nats", [10.0, 40.0, 120.0])
def test_64_rows_whose_reference_is_raised(snapkv, g, W, nats):
    """As test_score_error_does_not_grow_with_the_logits_range, with blocks of four row units and two tiles a wave: a stretch of keys
    lies far above the first sixteen.  The logits and their origins are exact here too, so the bound is the same."""
    L, D = 131099, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(18)
    q = torch.zeros((g, W, D), device="cuda")
    q[..., 3], q[..., 7] = 16.0, 1.0 / 8
    k = torch.zeros((1, L, D), device="cuda")
    k[0, :, 7] = torch.randint(-256, 257, (L,), generator=gen, device="cuda")
    k[0, 70000:75000, 3] = round(nats * D ** 0.5 / 16 * 4) / 4
    q, k = q.bfloat16(), k.bfloat16()
    sc = torch.empty((1, L - W), device="cuda")
    snapkv.snapkv_pooled_scores(q, k, 0, 1, sc)
    logits = (q[0].double() @ k[0].double().t()) / D ** 0.5
    seen = torch.arange(L, device="cuda") <= torch.arange(L - W, L, device="cuda").unsqueeze(1)
    want = g * torch.softmax(logits.masked_fill(~seen, float("-inf")), dim=1)[:, :L - W].sum(0)
    err = float((sc[0].double() - want).norm() / want.norm())
    print(f"score error at {nats} nats: {err:.2e}")
    assert err < 4.5e-7, err


def test_64_rows_one_cache_per_query_head(snapkv):
    """One vote row per query head from blocks of four of them: what every head keeps is what it keeps as a KV head of its own
    (scored by another kernel there: the band decides)."""
    w = half(131100, 4, 16, Hkv=1)
    case = workloads.generate(w, device="cuda")
    q, k, v = case["q_win"], case["k"], case["v"]
    ok = torch.zeros((w.Hq, w.C, w.D), dtype=k.dtype, device="cuda")
    ov = torch.zeros_like(ok)
    oi = torch.full((w.Hq, w.C), -1, dtype=torch.int32, device="cuda")
    kept = snapkv.snapkv_compress_per_query_head(q, k, v, w.pool_kind, w.p, w.C, ok, ov, oi)
    kr, vr = (t.repeat_interleave(w.Hq, dim=0).contiguous() for t in (k, v))
    sc = torch.empty((w.Hq, w.n), device="cuda")
    snapkv.snapkv_pooled_scores(q, kr, w.pool_kind, w.p, sc)
    torch.cuda.synchronize()
    check_against_oracle(q, kr, vr, w.pool_kind, w.p, w.C, sc.cpu().numpy(), ok, ov, oi.cpu().numpy(), kept, heads=[0, 3],
                         own_topk_exact=False)


@pytest.mark.parametrize("g,W", [(4, 16), (1, 64)])
def test_64_rows_on_a_callers_workspace_and_replayed(snapkv, g, W):
    """On a workspace full of ones, and replayed from a graph with other calls' remains in it: bit for bit the own-scratch call."""
    w = half(131101, g, W, Hkv=2)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)]
    want = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    q, k, v = (cases[0][n].clone() for n in ("q_win", "k", "v"))
    ok, ov, oi = (t[0] for t in outputs(w, 1, k.dtype))
    ws = torch.full((snapkv.snapkv_workspace_bytes(w.L, w.Hq, w.Hkv, w.D, w.W),), 255, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), -77, dtype=torch.int32, device="cuda")
    args = (w.pool_kind, w.p, w.C, ok, ov, oi)

    def load(l):
        for t, n in ((q, "q_win"), (k, "k"), (v, "v")):
            t.copy_(cases[l][n])
        ok.zero_(), ov.zero_(), oi.fill_(-1), status.fill_(-77)

    def same(l, what):
        torch.cuda.synchronize()
        assert np.array_equal(oi.cpu().numpy(), want[l][3]), (what, l)
        assert torch.equal(ok, want[l][1]) and torch.equal(ov, want[l][2]), (what, l)

    for l in (0, 1):
        load(l)
        snapkv.snapkv_compress(q, k, v, *args, workspace=ws)
        same(l, "workspace")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        snapkv.snapkv_compress_ws_status(q, k, v, *args, ws, status)
    for rep in range(4):
        load(rep % 2)
        if rep == 2:
            ws.fill_(255)
        graph.replay()
        same(rep % 2, f"replay {rep}")
        assert int(status.item()) == w.C
    assert snapkv.snapkv_sync_timeouts() == 0


@pytest.mark.parametrize("g,W", [(4, 16), (1, 64)])
def test_64_rows_layers_and_batches_equal_single_calls(snapkv, g, W):
    """Stacked and separate layers, paged rows and a batch with prompts on both sides of the rule, bit for bit."""
    w = half(131100, g, W, Hkv=2)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)] + [workloads.generate(w.with_(L=9001), device="cuda")]
    want = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    lists = [[c[n] for c in cases[:2]] for n in ("q_win", "k", "v")]
    for stack in (False, True):
        oks, ovs, ois = outputs(w, 2, cases[0]["k"].dtype)
        if stack:
            lists = [list(torch.stack(x).contiguous()) for x in lists]
            oks, ovs, ois = (list(torch.stack(x).contiguous()) for x in (oks, ovs, ois))
        snapkv.snapkv_compress_layers(*lists, w.pool_kind, w.p, w.C, oks, ovs, ois)
        for l in range(2):
            assert np.array_equal(ois[l].cpu().numpy(), want[l][3]) and torch.equal(oks[l], want[l][1]), (l, stack)
    oks, ovs, ois = outputs(w, 3, cases[0]["k"].dtype)
    snapkv.snapkv_compress_varlen(*([c[n] for c in cases] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, oks, ovs, ois)
    for i in range(3):
        assert np.array_equal(ois[i].cpu().numpy(), want[i][3]) and torch.equal(oks[i], want[i][1]), i
    q, k, v = (cases[0][n] for n in ("q_win", "k", "v"))
    page, pages = 16, -(-w.L // 16)
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(3)).to(torch.int32).cuda()
    pos = torch.arange(w.L, device="cuda")
    paged = []
    for t in (k, v):
        cache = torch.zeros((pages, page, w.Hkv, w.D), dtype=t.dtype, device="cuda")
        cache[table.long()[pos // page], pos % page] = t.permute(1, 0, 2)
        paged.append(cache)
    ok, ov, oi = (t[0] for t in outputs(w, 1, k.dtype))
    snapkv.snapkv_compress_paged(q, *paged, table, w.L, w.pool_kind, w.p, w.C, ok, ov, oi)
    assert np.array_equal(oi.cpu().numpy(), want[0][3])
    assert torch.equal(ok, want[0][1]) and torch.equal(ov, want[0][2])


def relative_error(snapkv, q, k, L):
    """Of the first L keys' votes against float64, over the votes within a factor of two of a head's 1024th (2-norm)."""
    (Hq, W, D), Hkv = q.shape, k.shape[0]
    keys = k[:, :L].contiguous()
    votes = torch.empty((Hkv, L - W), device="cuda")
    snapkv.snapkv_pooled_scores(q, keys, 0, 1, votes)
    seen = torch.arange(L, device="cuda") <= torch.arange(L - W, L, device="cuda").unsqueeze(1)
    errors = []
    for h in range(Hkv):
        want = torch.zeros(L - W, dtype=torch.float64, device="cuda")
        for x in q.view(Hkv, -1, W, D)[h]:
            logits = (x.double() @ keys[h].double().t()) / D ** 0.5
            want += torch.softmax(logits.masked_fill(~seen, float("-inf")), 1)[:, :L - W].sum(0)
        edge = want.topk(1024)[0][-1]
        near = (want > edge / 2) & (want < edge * 2)
        errors.append(((votes[h].double() - want)[near] / want[near]).pow(2).mean())
    return float(torch.stack(errors).mean().sqrt())


@pytest.mark.parametrize("W,spread,sink", [(13, 3.6, 0.0), (16, 3.6, 0.0), (16, 1.8, 8.0), (16, 1.8, 20.0)])
def test_64_rows_are_as_exact_as_the_single_read_kernel(snapkv, W, spread, sink):
    """Logits N(0, spread nats), and a first key `sink` nats above them.  131073 keys take the two passes, 131072 the single-read kernel:
    the error of what the two passes score is no larger than that kernel's."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(29)
    Hkv, g, L, D = 8, 4, 131073, 128
    q = torch.randn((Hkv * g, W, D), generator=gen, device="cuda") + 1.5 * torch.randn((Hkv * g, 1, D), generator=gen, device="cuda")
    k = torch.randn((Hkv, L, D), generator=gen, device="cuda")
    q = q * (spread / q.pow(2).mean().sqrt())
    if sink:
        u = torch.nn.functional.normalize(torch.randn(D, generator=gen, device="cuda"), dim=0)
        q += 8 * u
        k[:, 0] += sink * D ** 0.5 / 8 * u
    q, k = q.bfloat16(), k.bfloat16()
    two, one = relative_error(snapkv, q, k, L), relative_error(snapkv, q, k, L - 1)
    print(f"relative error {two:.3e}, single-read kernel {one:.3e}")
    assert two <= one, (two, one)


def outputs(w, n, dtype):
    return ([torch.zeros((w.Hkv, w.C, w.D), dtype=dtype, device="cuda") for _ in range(n)],
            [torch.zeros((w.Hkv, w.C, w.D), dtype=dtype, device="cuda") for _ in range(n)],
            [torch.full((w.Hkv, w.C), -1, dtype=torch.int32, device="cuda") for _ in range(n)])


def test_layouts_layers_and_batches_equal_single_calls(snapkv):
    """Token-major, paged, separately allocated and stacked layers, a batch with prompts on both sides of the rule:
    every one bit for bit what a single contiguous call gives (a head's result depends on its own prompt only)."""
    w = CASES["w32_one_more"]
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)]
    want = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    q, k, v = (cases[0][n] for n in ("q_win", "k", "v"))

    def same(ok, ov, oi, ref, what):
        assert np.array_equal(oi.cpu().numpy(), ref[3]), what
        assert torch.equal(ok, ref[1]) and torch.equal(ov, ref[2]), what

    ok, ov, oi = (t[0] for t in outputs(w, 1, k.dtype))
    kt, vt = (t.transpose(0, 1).contiguous().transpose(0, 1) for t in (k, v))
    snapkv.snapkv_compress_strided(q, kt, vt, w.pool_kind, w.p, w.C, ok, ov, oi)
    same(ok, ov, oi, want[0], "token-major")

    page, pages = 16, -(-w.L // 16)
    table = torch.randperm(pages, device="cuda").to(torch.int32)
    paged = []
    for t in (k, v):
        pad = torch.zeros((w.Hkv, pages * page, w.D), dtype=t.dtype, device="cuda")
        pad[:, :w.L] = t
        cache = torch.empty((pages, page, w.Hkv, w.D), dtype=t.dtype, device="cuda")
        cache[table.long()] = pad.view(w.Hkv, pages, page, w.D).permute(1, 2, 0, 3)
        paged.append(cache)
    oi.fill_(-1)
    snapkv.snapkv_compress_paged(q, paged[0], paged[1], table, w.L, w.pool_kind, w.p, w.C, ok, ov, oi)
    same(ok, ov, oi, want[0], "paged")

    for stack in (False, True):
        lists = [[c[n] for c in cases] for n in ("q_win", "k", "v")]
        oks, ovs, ois = outputs(w, 2, k.dtype)
        if stack:
            lists = [list(torch.stack(x).contiguous()) for x in lists]
            oks, ovs, ois = (list(torch.stack(x).contiguous()) for x in (oks, ovs, ois))
        snapkv.snapkv_compress_layers(*lists, w.pool_kind, w.p, w.C, oks, ovs, ois)
        for l in range(2):
            same(oks[l], ovs[l], ois[l], want[l], f"layers, stacked={stack}")

    short = workloads.generate(w.with_(L=5000), device="cuda")
    batch = [cases[0], short, cases[1]]
    refs = [want[0], run_gpu(snapkv, short["q_win"], short["k"], short["v"], w.pool_kind, w.p, w.C), want[1]]
    oks, ovs, ois = outputs(w, 3, k.dtype)
    snapkv.snapkv_compress_varlen([c["q_win"] for c in batch], [c["k"] for c in batch], [c["v"] for c in batch],
                                  w.pool_kind, w.p, w.C, oks, ovs, ois)
    for i in range(3):
        same(oks[i], ovs[i], ois[i], refs[i], f"batch, prompt {i}")


@pytest.mark.parametrize("page", [1, 7, 300])
def test_page_sizes_equal_the_contiguous_call(snapkv, page):
    """Pages of one row, of an odd number of rows and longer than a round; an id past the last page is taken for it."""
    w = work(18450, 4, 32)
    case = workloads.generate(w, device="cuda")
    pages = -(-w.L // page)
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(page)).to(torch.int32).cuda()
    pos = torch.arange(w.L, device="cuda")
    paged = []
    for t in (case["k"], case["v"]):
        cache = torch.zeros((pages, page, w.Hkv, w.D), dtype=t.dtype, device="cuda")
        cache[table.long()[pos // page], pos % page] = t.permute(1, 0, 2)
        paged.append(cache)
    ids = table.clone()
    ids[table == pages - 1] = pages + 5                   # clamped to the last page, which is the one it names
    want = run_gpu(snapkv, case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C)
    ok, ov, oi = (t[0] for t in outputs(w, 1, case["k"].dtype))
    snapkv.snapkv_compress_paged(case["q_win"], paged[0], paged[1], ids, w.L, w.pool_kind, w.p, w.C, ok, ov, oi)
    assert np.array_equal(oi.cpu().numpy(), want[3])
    assert torch.equal(ok, want[1]) and torch.equal(ov, want[2])


@pytest.mark.parametrize("Hkv,L", [(1, 18433), (2, 30011)])
def test_few_heads_in_layers_and_batches_equal_single_calls(snapkv, Hkv, L):
    """The cut of a prompt into slices follows its own heads, not those of the call: layers, stacked or separate, and the
    prompts of a batch keep, bit for bit, what single calls keep."""
    w = work(L, 4, 32, Hkv=Hkv)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(2)] + [workloads.generate(w.with_(L=L + 70), device="cuda")]
    want = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    lists = [[c[n] for c in cases[:2]] for n in ("q_win", "k", "v")]
    for stack in (False, True):
        oks, ovs, ois = outputs(w, 2, cases[0]["k"].dtype)
        if stack:
            lists = [list(torch.stack(x).contiguous()) for x in lists]
            oks, ovs, ois = (list(torch.stack(x).contiguous()) for x in (oks, ovs, ois))
        snapkv.snapkv_compress_layers(*lists, w.pool_kind, w.p, w.C, oks, ovs, ois)
        for l in range(2):
            assert np.array_equal(ois[l].cpu().numpy(), want[l][3]) and torch.equal(oks[l], want[l][1]), (l, stack)
    oks, ovs, ois = outputs(w, 3, cases[0]["k"].dtype)
    snapkv.snapkv_compress_varlen(*([c[n] for c in cases] for n in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, oks, ovs, ois)
    for i in range(3):
        assert np.array_equal(ois[i].cpu().numpy(), want[i][3]) and torch.equal(oks[i], want[i][1]), i


def test_logits_far_above_the_first_key(snapkv):
    """The rows' reference is their logit with key 0; here a stretch of keys lies about 130 nats above it (2^187), so
    the sums relative to it overflow and the rows are taken from the keys again."""
    w = work(18461, 4, 32, Hkv=1, C=300)
    case = workloads.generate(w, device="cuda")
    q, k, v = case["q_win"].clone(), case["k"].clone(), case["v"]
    u = torch.zeros(w.D, device="cuda")
    u[3] = 1.0
    q += (12.0 * u).to(q.dtype)
    k[:, 0] = 0
    k[:, 7000:12000] += (122.0 * u).to(k.dtype)          # 12 * 122 / sqrt(128) = 129 nats
    res = run_gpu(snapkv, q, k, v, w.pool_kind, w.p, w.C)
    check_against_oracle(q, k, v, w.pool_kind, w.p, w.C, *res)


@pytest.mark.parametrize("nats", [0.0, 10.0, 40.0, 80.0, 120.0])
def test_score_error_does_not_grow_with_the_logits_range(snapkv, nats):
    """A stretch of keys that the whole window looks for, `nats` above the prompt's first keys.  All rows of the window
    are the same and every logit is exact in fp32 (two non-zero elements of few bits), so what remains is the
    rounding of the exponentials' arguments, which no average over rows hides.  Bound: half an ulp of an argument
    below 16 (2^-21, as a factor 2^-21 ln 2 = 3.3e-7) and one ulp of exp2 (1.2e-7)."""
    Hq, L, W, D = 4, 18461, 32, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    q = torch.zeros((Hq, W, D), device="cuda")
    q[..., 3], q[..., 7] = 16.0, 1.0 / 8
    k = torch.zeros((1, L, D), device="cuda")
    k[0, :, 7] = torch.randint(-256, 257, (L,), generator=gen, device="cuda")              # logits within +-32 / sqrt(128)
    k[0, 7000:12000, 3] = round(nats * D ** 0.5 / 16 * 4) / 4
    q, k = q.bfloat16(), k.bfloat16()
    sc = torch.empty((1, L - W), device="cuda")
    snapkv.snapkv_pooled_scores(q, k, 0, 1, sc)
    logits = (q[0].double() @ k[0].double().t()) / D ** 0.5                                # [W, L]
    seen = torch.arange(L, device="cuda") <= torch.arange(L - W, L, device="cuda").unsqueeze(1)
    p = torch.softmax(logits.masked_fill(~seen, float("-inf")), dim=1)
    want = Hq * p[:, :L - W].sum(0)
    err = float((sc[0].double() - want).norm() / want.norm())
    print(f"score error at {nats} nats: {err:.2e}")
    assert err < 4.5e-7, err


def test_one_cache_per_query_head(snapkv):
    """The per-query-head form takes its votes from the two passes too, one row per query head."""
    w = work(18440, 4, 32, Hkv=2)
    case = workloads.generate(w, device="cuda")
    q, k, v = case["q_win"], case["k"], case["v"]
    ok = torch.zeros((w.Hq, w.C, w.D), dtype=k.dtype, device="cuda")
    ov = torch.zeros_like(ok)
    oi = torch.full((w.Hq, w.C), -1, dtype=torch.int32, device="cuda")
    kept = snapkv.snapkv_compress_per_query_head(q, k, v, w.pool_kind, w.p, w.C, ok, ov, oi)
    kr, vr = (t.repeat_interleave(w.Hq // w.Hkv, dim=0).contiguous() for t in (k, v))
    sc = torch.empty((w.Hq, w.n), device="cuda")
    snapkv.snapkv_pooled_scores(q, kr, w.pool_kind, w.p, sc)          # (scores of another kernel: the band decides)
    torch.cuda.synchronize()
    check_against_oracle(q, kr, vr, w.pool_kind, w.p, w.C, sc.cpu().numpy(), ok, ov, oi.cpu().numpy(), kept,
                         own_topk_exact=False)


def test_callers_scratch_static_scratch_and_replay_equal_own_scratch(snapkv):
    """On a caller's workspace, on the static scratch and replayed from a graph the first pass clears what the selection
    expects to be zero: with scratch full of ones beforehand, and whatever the call before left in it, every call is
    bit for bit the own-scratch call."""
    w = work(18433, 4, 32)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(3)]
    want = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    q, k, v = (cases[0][n].clone() for n in ("q_win", "k", "v"))
    ok, ov, oi = (t[0] for t in outputs(w, 1, k.dtype))
    ws = torch.full((snapkv.snapkv_workspace_bytes(w.L, w.Hq, w.Hkv, w.D, w.W),), 255, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), -77, dtype=torch.int32, device="cuda")
    args = (w.pool_kind, w.p, w.C, ok, ov, oi)

    def load(l):
        for t, n in ((q, "q_win"), (k, "k"), (v, "v")):
            t.copy_(cases[l][n])
        ok.zero_(), ov.zero_(), oi.fill_(-1), status.fill_(-77)

    def same(l, what):
        torch.cuda.synchronize()
        assert np.array_equal(oi.cpu().numpy(), want[l][3]), (what, l)
        assert torch.equal(ok, want[l][1]) and torch.equal(ov, want[l][2]), (what, l)

    for l in (0, 1, 2):
        load(l)
        snapkv.snapkv_compress(q, k, v, *args, workspace=ws)
        same(l, "workspace")
        load(l)
        snapkv.snapkv_compress_ws_status(q, k, v, *args, ws, status)
        same(l, "status")
        assert int(status.item()) == w.C
        load(l)
        snapkv.snapkv_compress_static(q, k, v, *args)
        same(l, "static")
    graphs = {}
    for what, call in (("workspace", lambda: snapkv.snapkv_compress_ws_status(q, k, v, *args, ws, status)),
                       ("static", lambda: snapkv.snapkv_compress_static(q, k, v, *args))):
        graphs[what] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graphs[what]):
            call()
    for rep in range(6):
        for what, graph in graphs.items():
            load(rep % 3)
            if rep == 3:
                ws.fill_(255)
            graph.replay()
            same(rep % 3, f"{what}, replay {rep}")
            assert what == "static" or int(status.item()) == w.C
    assert snapkv.snapkv_sync_timeouts() == 0
