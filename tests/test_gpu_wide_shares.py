"""Two-pass scoring: the votes' pass is shared out by rounds, so that a workgroup may begin and end in the middle of a slice.  Its results are
those of the oracle, and the same bit for bit in calls whose workgroups begin elsewhere."""
import numpy as np
import pytest
import torch

from paper_2404_14469_amd import workloads
from parity import check_against_oracle, run_gpu
from test_gpu_wide import outputs
from test_gpu_wide_once import work

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(L=9300, g=4, W=64, Hkv=8, p=13),                  # 16 units, slices of 3 rounds
                                dict(L=16513, g=4, W=32, Hkv=4, dtype="f16"),          # 4 units, slices of 3 rounds, the last of one key
                                dict(L=18561, g=1, W=113, Hkv=33),                     # 33 units: also alone more slices than places
                                dict(L=140001, g=4, W=16, Hkv=8)])                     # blocks of 64 rows
def test_layers_whose_shares_end_within_slices(snapkv, kw):
    w = work(**kw)
    cases = [workloads.generate(w, layer=l, device="cuda") for l in range(3)]
    alone = [run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C) for c in cases]
    for n in (2, 3):
        oks, ovs, ois = outputs(w, n, cases[0]["k"].dtype)
        snapkv.snapkv_compress_layers(*([c[x] for c in cases[:n]] for x in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, oks, ovs, ois)
        for l in range(n):
            assert np.array_equal(ois[l].cpu().numpy(), alone[l][3]) and torch.equal(oks[l], alone[l][1]) and torch.equal(ovs[l], alone[l][2]), (n, l)
    check_against_oracle(*(cases[2][x] for x in ("q_win", "k", "v")), w.pool_kind, w.p, w.C, *alone[2], heads=[0, w.Hkv - 1])


def test_paged_prompt_of_more_slices_than_places(snapkv):
    """Paged keys, whose page ids are asked for a round ahead from wherever the workgroup begins."""
    w = work(L=18561, g=1, W=113, Hkv=33)
    c = workloads.generate(w, device="cuda")
    want = run_gpu(snapkv, c["q_win"], c["k"], c["v"], w.pool_kind, w.p, w.C)
    page = 16
    pages = (w.L + page - 1) // page
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(3)).to("cuda", torch.int32)
    caches = []
    for x in (c["k"], c["v"]):
        rows = torch.zeros((pages * page, w.Hkv, w.D), dtype=x.dtype, device="cuda")
        rows[:w.L] = x.transpose(0, 1)
        cache = torch.empty((pages, page, w.Hkv, w.D), dtype=x.dtype, device="cuda")
        cache[table.long()] = rows.view(pages, page, w.Hkv, w.D)
        caches.append(cache)
    (ok,), (ov,), (oi,) = outputs(w, 1, c["k"].dtype)
    snapkv.snapkv_compress_paged(c["q_win"], *caches, table, w.L, w.pool_kind, w.p, w.C, ok, ov, oi)
    assert np.array_equal(oi.cpu().numpy(), want[3]) and torch.equal(ok, want[1]) and torch.equal(ov, want[2])
