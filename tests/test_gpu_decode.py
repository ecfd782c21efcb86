"""GPU parity of snapkv_decode_attention (through the C ABI) against the fp64 oracle.

Tolerance, from the kernel's arithmetic: logits are exact products accumulated in fp32, the
exponent argument carries one fp32 rounding at magnitude <= ~2^7 (2^-17 relative in the
exponential), the probabilities enter the last product split into two storage-type parts
(<= 2^-16 relative) and everything else is fp32.  The output is a convex combination of value rows, so
|gpu - oracle| <= 1e-4 * max|v| leaves a factor of about three over the sum of those terms; the lse
is compared to 1e-4 absolute.
"""
import json
import time

import numpy as np
import pytest
import torch

from oracle import decode_oracle as dec
from paper_2404_14469_amd import workloads
from paper_2404_14469_amd.workloads import DecodeWorkload

pytestmark = pytest.mark.gpu

TOL = 1e-4


def run(snapkv, w, case, with_lse=True):
    q, k, v, lens = case["q"], case["k_cache"], case["v_cache"], case["lens"]
    out = torch.full((w.B, w.Hq, w.D), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((w.B, w.Hq), float("nan"), dtype=torch.float32, device="cuda") if with_lse else None
    snapkv.snapkv_decode_attention(q, k, v, w.S, out, lse, lens=lens)
    torch.cuda.synchronize()
    return out.cpu().numpy(), lse.cpu().numpy() if with_lse else None


def check(w, case, out, lse, seqs=None):
    seqs = list(range(w.B)) if seqs is None else seqs
    lens = case["lens"].cpu().tolist() if case["lens"] is not None else [w.S] * w.B
    for b in seqs:
        S = lens[b]
        qb = workloads.to_numpy_bits(case["q"][b:b + 1])
        kb = workloads.to_numpy_bits(case["k_cache"][b:b + 1, :, :S])
        vb = workloads.to_numpy_bits(case["v_cache"][b:b + 1, :, :S])
        want, want_lse = dec.decode_attention(qb, kb, vb)
        vmax = float(np.abs(dec.widen(vb)).max())
        err = np.abs(out[b] - want[0]).max()
        assert err <= TOL * vmax, (w.name, b, err, vmax)
        if lse is not None:
            assert np.abs(lse[b] - want_lse[0]).max() <= TOL, (w.name, b)


CASES = [
    DecodeWorkload("one_pair", B=1, Hq=4, Hkv=4, D=128, S=32, cap=32, seed=1),
    DecodeWorkload("one_row", B=2, Hq=2, Hkv=2, D=64, S=1, cap=8, seed=2),
    DecodeWorkload("ragged_tail", B=2, Hq=8, Hkv=8, D=128, S=1000, cap=1100, seed=3),       # S % 32 != 0, S < cap
    DecodeWorkload("gqa4", B=3, Hq=16, Hkv=4, D=128, S=777, cap=800, seed=4),
    DecodeWorkload("gqa8_d64", B=2, Hq=32, Hkv=4, D=64, S=1500, cap=1500, seed=5),
    DecodeWorkload("gqa16", B=1, Hq=32, Hkv=2, D=128, S=300, cap=512, seed=6),             # a full 16-row operand
    DecodeWorkload("split_keys", B=1, Hq=8, Hkv=8, D=128, S=6000, cap=6000, seed=7),        # keys split over workgroups
    DecodeWorkload("split_ragged", B=2, Hq=8, Hkv=2, D=128, S=5000, cap=5003, ragged=True, seed=8),
    DecodeWorkload("many_pairs_no_split", B=40, Hq=32, Hkv=32, D=128, S=200, cap=200, seed=9),
    DecodeWorkload("lens_mixed", B=6, Hq=8, Hkv=4, D=64, S=900, cap=901, ragged=True, seed=10),
    DecodeWorkload("f16", B=2, Hq=8, Hkv=4, D=128, S=1234, cap=1300, dtype="f16", seed=11),
    DecodeWorkload("split_small", B=1, Hq=8, Hkv=2, D=128, S=129, cap=140, seed=13),            # too short to split
    DecodeWorkload("split_first", B=1, Hq=8, Hkv=2, D=128, S=1024, cap=1100, seed=18),          # one step of 32 keys per wave
    DecodeWorkload("split_odd", B=1, Hq=32, Hkv=8, D=128, S=2113, cap=2560, seed=14),           # 17 splits
    DecodeWorkload("split_most", B=1, Hq=2, Hkv=1, D=64, S=16400, cap=16400, seed=15),          # 64 splits
    DecodeWorkload("split_ragged_short", B=3, Hq=16, Hkv=8, D=128, S=3000, cap=3000, ragged=True, seed=16),
    DecodeWorkload("split_rounds", B=3, Hq=32, Hkv=32, D=128, S=2100, cap=2100, seed=17),       # more workgroups than units
    DecodeWorkload("one_step_a_wave", B=1, Hq=32, Hkv=8, D=128, S=4096, cap=4096, seed=31),     # 32 splits of four steps
    DecodeWorkload("a_fifth_step", B=1, Hq=32, Hkv=8, D=128, S=4097, cap=4200, seed=32),
    DecodeWorkload("one_step_unsplit", B=2, Hq=4, Hkv=4, D=64, S=128, cap=200, seed=33),
    DecodeWorkload("one_step_ragged", B=3, Hq=8, Hkv=4, D=128, S=128, cap=128, ragged=True, seed=34),
    DecodeWorkload("one_step_three_to_a_unit", B=1, Hq=32, Hkv=32, D=128, S=2048, cap=2048, dtype="f16", seed=35),
    DecodeWorkload("f16_d64_split", B=1, Hq=4, Hkv=4, D=64, S=4100, cap=4100, dtype="f16", seed=12),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_decode_matches_oracle(snapkv, w):
    case = workloads.generate_decode(w, device="cuda")
    out, lse = run(snapkv, w, case)
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    check(w, case, out, lse)


def test_lse_output_is_optional_and_results_repeat_bitwise(snapkv):
    w = CASES[6]
    case = workloads.generate_decode(w, device="cuda")
    a, _ = run(snapkv, w, case, with_lse=False)
    b, _ = run(snapkv, w, case)
    assert np.array_equal(a, b)


def test_row_order_does_not_matter(snapkv):
    """The property a compacted cache relies on: permuting the cache rows changes nothing beyond
    the rounding order of the sums."""
    w = DecodeWorkload("perm", B=1, Hq=8, Hkv=8, D=128, S=3000, cap=3000, seed=21)
    case = workloads.generate_decode(w, device="cuda")
    a, la = run(snapkv, w, case)
    perm = torch.randperm(w.S, generator=torch.Generator().manual_seed(5)).cuda()
    case2 = dict(case, k_cache=case["k_cache"][:, :, perm].contiguous(), v_cache=case["v_cache"][:, :, perm].contiguous())
    b, lb = run(snapkv, w, case2)
    vmax = float(case["v_cache"].float().abs().max())
    assert np.abs(a - b).max() <= TOL * vmax and np.abs(la - lb).max() <= TOL


def test_lens_beyond_the_step_count_of_S(snapkv):
    """The splits are planned for S rows; lens may ask for more, up to the cache's capacity: several steps a wave then."""
    w = DecodeWorkload("long_lens", B=2, Hq=8, Hkv=4, D=128, S=1100, cap=3000, seed=36)
    case = workloads.generate_decode(w, device="cuda")
    case["k_cache"][:, :, w.S:] = case["k_cache"][:, :, :1].flip(1)     # make the padding rows ordinary
    case["v_cache"][:, :, w.S:] = case["v_cache"][:, :, :1]
    case["lens"] = torch.tensor([3000, 2999], dtype=torch.int32, device="cuda")
    out, lse = run(snapkv, w, case)
    check(w, case, out, lse)


def launched(call, tmp_path):
    """(name, workgroups) of the kernels that a call launches."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        time.sleep(0.02)                 # (the profiler drops kernels near the ends of its window: the clocks differ a little)
        call()
        torch.cuda.synchronize()
        time.sleep(0.02)
    p.export_chrome_trace(str(tmp_path / "trace.json"))
    events = json.loads((tmp_path / "trace.json").read_text())["traceEvents"]
    return [(e["name"], int(np.prod(e["args"]["grid"]))) for e in events if e.get("cat") == "kernel"]


@pytest.mark.parametrize("B,Hkv,S,cap,light", [
    (1, 32, 2048, 2560, False), (3, 8, 2048, 2300, False), (5, 8, 1500, 1900, False), (3, 32, 1024, 1536, False),
    (1, 32, 2048, 2049, False), (1, 32, 2040, 2048, True), (1, 8, 4000, 4096, True)])
def test_splits_are_those_of_the_form_that_runs(snapkv, tmp_path, B, Hkv, S, cap, light):
    """With lens given, sequences may be as long as the cache, and the light form (one step a wave) runs only where even such
    a one has no more.  The other form has one workgroup per compute unit where the pairs leave room; the light form
    takes as many splits as for lens = NULL."""
    w = DecodeWorkload("form", B=B, Hq=32, Hkv=Hkv, D=128, S=S, cap=cap, ragged=True, seed=37)
    case = workloads.generate_decode(w, device="cuda")
    out, lse = run(snapkv, w, case)                              # (allocates the partials' buffer)
    check(w, case, out, lse)
    kernels = launched(lambda: run(snapkv, w, case, with_lse=False), tmp_path)
    (name, groups), = [(n, g) for n, g in kernels if "decode_attn<" in n]
    assert ("true>" in name) == light, name
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if light:
        plain = launched(lambda: run(snapkv, w, dict(case, lens=None), with_lse=False), tmp_path)
        assert (name, groups) in plain
    else:
        assert groups <= cus, (name, groups)


def test_empty_sequence_and_length_clamp(snapkv):
    w = DecodeWorkload("empty", B=3, Hq=4, Hkv=2, D=64, S=50, cap=64, seed=22)
    case = workloads.generate_decode(w, device="cuda")
    case["lens"] = torch.tensor([0, 50, 1000], dtype=torch.int32, device="cuda")   # 1000 is clamped to cap
    case["k_cache"][2, :, 50:] = case["k_cache"][1, :, :14]                        # make the padding rows ordinary
    case["v_cache"][2, :, 50:] = case["v_cache"][1, :, :14]
    out, lse = run(snapkv, w, case)
    assert np.array_equal(out[0], np.zeros_like(out[0])) and np.isneginf(lse[0]).all()
    case_ok = dict(case, lens=torch.tensor([1, 50, 64], dtype=torch.int32, device="cuda"))
    check(w, case_ok, out, lse, seqs=[1, 2])


def test_compressed_cache_feeds_the_decoding_step(snapkv):
    """End to end over the boundary: compress a prompt, decode over the kept rows, and compare with
    the oracle's attention over the rows the oracle's compression keeps."""
    w = workloads.Workload("e2e", Hq=8, Hkv=4, D=128, L=3000, W=32, pool_kind=0, p=7, C=256, dtype="bf16",
                           clusters=(4, 4), radius=6, seed=31)
    case = workloads.generate(w, device="cuda")
    out_k, out_v, out_idx, kept = snapkv.compress(case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C)
    q_new = case["q_win"][:, -1, :].contiguous().unsqueeze(0)                       # stands in for the next token's query
    out = torch.empty((1, w.Hq, w.D), dtype=torch.float32, device="cuda")
    snapkv.snapkv_decode_attention(q_new, out_k.unsqueeze(0), out_v.unsqueeze(0), kept, out)
    torch.cuda.synchronize()
    # the oracle attends to exactly the rows the GPU kept (gathered bit-exactly, checked elsewhere)
    want, _ = dec.decode_attention(workloads.to_numpy_bits(q_new), workloads.to_numpy_bits(out_k.unsqueeze(0)),
                                   workloads.to_numpy_bits(out_v.unsqueeze(0)))
    vmax = float(out_v.float().abs().max())
    assert np.abs(out.cpu().numpy() - want).max() <= TOL * vmax
    # and those rows are the oracle's selection, by the same rule as everywhere: scores within 1e-3, kept
    # positions exact outside the band around the threshold, the exact top-k of the GPU's own scores
    from parity import check_against_oracle
    sc = torch.empty((w.Hkv, w.n), dtype=torch.float32, device="cuda")
    snapkv.snapkv_pooled_scores(case["q_win"], case["k"], w.pool_kind, w.p, sc)
    torch.cuda.synchronize()
    check_against_oracle(case["q_win"], case["k"], case["v"], w.pool_kind, w.p, w.C, sc.cpu().numpy(), out_k, out_v,
                         out_idx.cpu().numpy(), kept)


@pytest.mark.parametrize("B,Hq,Hkv,S", [(9, 32, 32, 2560), (22, 8, 8, 1500), (1, 32, 8, 1023), (3, 8, 8, 900)])
def test_unsplit_steps_on_two_streams_are_independent(snapkv, B, Hq, Hkv, S):
    """Steps of more pairs than two thirds of the compute units, or of fewer than 1024 keys, are not split, so they share
    no buffer: enqueued on two streams without any order between them, both give what they give alone."""
    cases = [workloads.generate_decode(DecodeWorkload("streams", B=B, Hq=Hq, Hkv=Hkv, D=64, S=S, cap=S, seed=s), device="cuda")
             for s in (41, 42)]
    def step(c, o, s):
        snapkv.snapkv_decode_attention(c["q"], c["k_cache"], c["v_cache"], S, o[0], o[1], stream=s)
    new = lambda: (torch.zeros((B, Hq, 64), device="cuda"), torch.zeros((B, Hq), device="cuda"))
    want, got = [new() for _ in cases], [[new() for _ in range(10)] for _ in cases]
    for c, o in zip(cases, want):
        step(c, o, None)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    for i in range(10):
        for c, outs, s in zip(cases, got, streams):
            step(c, outs[i], s)
    torch.cuda.synchronize()
    for w, outs in zip(want, got):
        for o in outs:
            assert torch.equal(o[0], w[0]) and torch.equal(o[1], w[1])


def test_step_captured_before_any_eager_call(snapkv):
    """A capturing stream cannot allocate the partials' buffer: a step captured before the first eager one that is split
    is recorded unsplit, and one captured afterwards as the eager step is; both replay right."""
    w = DecodeWorkload("captured", B=1, Hq=8, Hkv=2, D=128, S=4100, cap=4100, seed=51)
    cases = [workloads.generate_decode(DecodeWorkload(**{**w.__dict__, "seed": 51 + i}), device="cuda") for i in range(2)]
    q, k, v = (torch.empty_like(cases[0][n]) for n in ("q", "k_cache", "v_cache"))
    out, lse = torch.empty((w.B, w.Hq, w.D), device="cuda"), torch.empty((w.B, w.Hq), device="cuda")
    torch.cuda.synchronize()
    snapkv.snapkv_release()                              # as in a process that has not decoded yet
    graphs = []
    for i in range(2):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            snapkv.snapkv_decode_attention(q, k, v, w.S, out, lse)
        if i == 0:
            eager, eager_lse = run(snapkv, w, cases[0])
    for rep in range(4):
        c = cases[rep % 2]
        for t, n in ((q, "q"), (k, "k_cache"), (v, "v_cache")):
            t.copy_(c[n])
        for i, graph in enumerate(graphs):
            out.fill_(float("nan")), lse.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            check(w, c, out.cpu().numpy(), lse.cpu().numpy())
            if i == 1 and rep % 2 == 0:
                assert np.array_equal(out.cpu().numpy(), eager) and np.array_equal(lse.cpu().numpy(), eager_lse)


def test_bad_arguments_are_refused(snapkv):
    w = DecodeWorkload("bad", B=1, Hq=4, Hkv=4, D=64, S=10, cap=16, seed=23)
    case = workloads.generate_decode(w, device="cuda")
    out = torch.empty((1, 4, 64), dtype=torch.float32, device="cuda")
    with pytest.raises(snapkv.SnapKVError):
        snapkv.snapkv_decode_attention(case["q"], case["k_cache"], case["v_cache"], 17, out)      # S > cap
    with pytest.raises(snapkv.SnapKVError):
        snapkv.snapkv_decode_attention(case["q"], case["k_cache"], case["v_cache"], 0, out)
    qf = case["q"].float()
    with pytest.raises(snapkv.SnapKVError):
        snapkv.snapkv_decode_attention(qf, case["k_cache"].float(), case["v_cache"].float(), 10, out)   # fp32 storage
