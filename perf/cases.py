"""The work that users of this library have it do, as cases that can be timed and compared.

A program that serves or evaluates a model with compressed prompt caches makes four kinds of calls:

  * ``compress``: one prompt, one layer, inside the forward pass (``snapkv_compress`` on the library's scratch or on
    the caller's workspace, ``snapkv_compress_strided`` on token-major caches, ``snapkv_compress_paged`` on paged ones);
  * ``layers``: all layers of one prompt at the end of the prefill (``snapkv_compress_layers``, stacked or one
    allocation per layer);
  * ``varlen``: the prompts of one serving step (``snapkv_compress_varlen``);
  * ``decode``: one decoding step of attention over the compressed caches (``snapkv_decode_attention``).

Sizes, windows, pooling widths and capacities are those of the repository's workloads and of the paper's settings
they stand for; lengths of real prompts are arbitrary, so most lengths here are odd.
"""
import math
import random

import torch

import paper_2404_14469_amd as snapkv

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
POOLS = {"max": snapkv.POOL_MAX, "avg": snapkv.POOL_AVG}
D = 128


def listed():
    mha, gqa = {"Hq": 32, "Hkv": 32, "D": D}, {"Hq": 32, "Hkv": 8, "D": D}
    return [
        # One decoding step of one user: a 2048-row cache and the tokens generated since.  Latency of a step.
        dict(gqa, name="decode_one", kind="decode", dtype="bf16", B=1, S=2113, cap=2560, ragged=False),
        # The decoding step at the batch size and cache cap of Sec. 5.1.2; every sequence is at another token.
        dict(mha, name="decode_batch", kind="decode", dtype="bf16", B=8, S=2560, cap=2560, ragged=True),
        # The smallest prompt worth compressing, fp32 storage, 4 heads of 64: launches and latency.
        dict(name="compress_tiny", kind="compress", layout="plain", dtype="f32", Hq=4, Hkv=4, D=64, L=512, W=32,
             pool="max", p=7, C=128, workspace=False),
        # A 7B multi-head layer at a 16K prompt, the paper's main comparison.
        dict(mha, name="compress_16k", kind="compress", layout="plain", dtype="bf16", L=16384, W=32, pool="max", p=7,
             C=1024, workspace=False),
        # A grouped-query layer in fp16 at a LongBench-like prompt of odd length, on the caller's workspace (what a
        # server with several streams or with graphs uses).
        dict(gqa, name="compress_gqa_odd", kind="compress", layout="plain", dtype="f16", L=28471, W=32, pool="max",
             p=7, C=2048, workspace=True),
        # The same layer of a server that keeps its prompt cache in pages of 16 rows.
        dict(gqa, name="compress_paged", kind="compress", layout="paged", dtype="bf16", L=13339, W=16, pool="max", p=5,
             C=1024, workspace=False),
        # Token-major [L, Hkv, D] caches, as attention libraries write them.
        dict(gqa, name="compress_token_major", kind="compress", layout="token_major", dtype="bf16", L=32749, W=32,
             pool="max", p=7, C=2048, workspace=False),
        # The paper's wide window and pooling (W = 64, p = 13) on a long prompt.
        dict(gqa, name="compress_w64_131k", kind="compress", layout="plain", dtype="bf16", L=131072, W=64, pool="max",
             p=13, C=4096, workspace=False),
        # The longest context the paper reports (Sec. 5.1.1).
        dict(mha, name="compress_380k", kind="compress", layout="plain", dtype="bf16", L=380000, W=16, pool="max", p=5,
             C=1024, workspace=False),
        # The prompts of one serving step, of very different lengths.
        dict(gqa, name="varlen_batch", kind="varlen", dtype="bf16", prompts=8, lo=4096, hi=65536, lengths=1005, W=16,
             pool="avg", p=5, C=1024),
        # A grouped-query model's 32 layers after the prefill, every layer's cache an allocation of its own, odd length.
        dict(gqa, name="layers_gqa_31k", kind="layers", dtype="bf16", layers=32, stacked=False, L=31337, W=32,
             pool="max", p=7, C=2048),
        # The library's headline job: 32 multi-head layers of a 131072-token prompt, 68.7 GB of keys and values.
        dict(mha, name="layers_131k", kind="layers", dtype="bf16", layers=32, stacked=True, L=131072, W=32, pool="max",
             p=7, C=4096),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _selection(rng, L):
    """Window, pooling and capacity as the paper pairs them; the capacity stays below the prompt."""
    W, pool, p = rng.choice([(32, "max", 7), (32, "max", 7), (16, "max", 5), (64, "max", 13), (16, "avg", 5)])
    C = rng.choice([c for c in (256, 1024, 2048, 4096) if c < L // 2] or [128])
    return {"W": W, "pool": pool, "p": p, "C": C}


def draw(rng):
    heads = rng.choice([{"Hq": 32, "Hkv": 32, "D": D}, {"Hq": 32, "Hkv": 8, "D": D}])
    two_byte = rng.choice(["bf16", "bf16", "f16"])
    kind = rng.choice(["decode", "compress", "compress", "compress", "long", "varlen", "layers"])
    if kind == "decode":
        S = _log_uniform(rng, 1024, 16384)
        return dict(heads, kind="decode", dtype=two_byte, B=rng.choice([1, 2, 3, 5, 8, 13]), S=S,
                    cap=S + rng.randrange(0, 512), ragged=rng.random() < 0.5)
    if kind == "compress":
        L = _log_uniform(rng, 512, 131072)
        c = dict(heads, kind="compress", layout=rng.choice(["plain", "plain", "plain", "paged", "token_major"]),
                 dtype=two_byte, L=L, workspace=False, **_selection(rng, L))
        if c["layout"] == "plain":
            c["workspace"] = rng.random() < 0.4
            if rng.random() < 0.15:
                c.update(dtype="f32", D=rng.choice([64, 128]))
        return c
    if kind == "long":
        L = _log_uniform(rng, 131073, 420000)
        return dict(heads, kind="compress", layout="plain", dtype=two_byte, L=L, workspace=False, **_selection(rng, L))
    if kind == "varlen":
        return dict(heads, Hq=32, kind="varlen", dtype=two_byte, prompts=rng.randrange(2, 13),
                    lo=_log_uniform(rng, 1024, 8192), hi=_log_uniform(rng, 8192, 65536), lengths=rng.randrange(1 << 30),
                    W=16, pool=rng.choice(["avg", "max"]), p=5, C=rng.choice([512, 1024]))
    L = _log_uniform(rng, 8192, 131072)
    most = max(2, min(32, (24 << 30) // (heads["Hkv"] * L * D * 4)))
    return dict(heads, kind="layers", dtype=two_byte, layers=rng.randrange(2, most + 1), stacked=rng.random() < 0.5, L=L,
                **_selection(rng, L))


def _lengths(case):
    rng = random.Random(case["lengths"])
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["prompts"])]


def _unit(gen, shape):
    u = torch.randn(shape, generator=gen, device="cuda")
    return u / u.norm(dim=-1, keepdim=True)


def _prompt(gen, heads_q, heads_kv, L, W, d, dtype):
    """q_win [heads_q, W, d] and k, v [heads_kv, L, d] of one or more layers' heads.

    Keys and values are N(0, 1); around 16 places of every KV head the keys of 17 neighbouring tokens lean into a common
    direction that the window's queries look for (the clusters of Sec. 4.3).  The queries at a prompt's end
    look for much the same things, so a head's window rows share a direction beside what each has of its own: the
    votes of a head spread over orders of magnitude, as those of trained models do.
    """
    g, n = heads_q // heads_kv, L - W
    k = torch.empty((heads_kv, L, d), device="cuda", dtype=dtype).normal_(generator=gen)
    v = torch.empty((heads_kv, L, d), device="cuda", dtype=dtype).normal_(generator=gen)
    q = torch.randn((heads_q, W, d), generator=gen, device="cuda")
    q += 1.5 * torch.randn((heads_q, 1, d), generator=gen, device="cuda")
    u = _unit(gen, (heads_kv, 16, d))
    centre = torch.randint(0, n, (heads_kv, 16, 1), generator=gen, device="cuda")
    rows = (centre + torch.arange(-8, 9, device="cuda")).clamp_(0, n - 1)
    head = torch.arange(heads_kv, device="cuda").view(-1, 1, 1).expand_as(rows)
    lean = (3.0 * u).to(dtype).unsqueeze(2).expand(heads_kv, 16, 17, d)
    k.index_put_((head, rows), lean, accumulate=True)
    q += u.sum(1).repeat_interleave(g, dim=0).unsqueeze(1)
    return q.to(dtype), k, v


def _outputs(heads, C, d, dtype):
    k = torch.empty((heads, C, d), device="cuda", dtype=dtype)
    return k, torch.empty_like(k), torch.empty((heads, C), device="cuda", dtype=torch.int32)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype, Hq, Hkv, d = DTYPES[case["dtype"]], case["Hq"], case["Hkv"], case["D"]
    if case["kind"] == "decode":
        return _prepare_decode(case, gen, dtype)
    s = {"case": case, "pool": POOLS[case["pool"]]}
    W, C = case["W"], case["C"]
    if case["kind"] == "varlen":
        made = [_prompt(gen, Hq, Hkv, L, W, d, dtype) for L in _lengths(case)]
        outs = [_outputs(Hkv, C, d, dtype) for _ in made]
    elif case["kind"] == "layers":
        n = case["layers"]
        if case["stacked"]:
            q, k, v = _prompt(gen, n * Hq, n * Hkv, case["L"], W, d, dtype)
            made = list(zip(q.split(Hq), k.split(Hkv), v.split(Hkv)))
        else:
            made = [_prompt(gen, Hq, Hkv, case["L"], W, d, dtype) for _ in range(n)]
        # the compacted caches are small: one tensor for all layers
        s["whole"] = _outputs(n * Hkv, C, d, dtype)
        outs = list(zip(*(t.split(Hkv) for t in s["whole"])))
    else:
        return _prepare_compress(case, gen, dtype, s)
    s["q"], s["k"], s["v"] = ([t[i] for t in made] for i in range(3))
    s["out_k"], s["out_v"], s["out_idx"] = ([t[i] for t in outs] for i in range(3))
    return s


def _prepare_compress(case, gen, dtype, s):
    Hq, Hkv, d, L, W = case["Hq"], case["Hkv"], case["D"], case["L"], case["W"]
    s["q"], k, v = _prompt(gen, Hq, Hkv, L, W, d, dtype)
    s["out_k"], s["out_v"], s["out_idx"] = _outputs(Hkv, case["C"], d, dtype)
    s["workspace"] = None
    if case["layout"] == "token_major":
        # the library is handed [Hkv, L, D] views of tensors stored as [L, Hkv, D]
        k, v = (t.transpose(0, 1).contiguous().transpose(0, 1) for t in (k, v))
    elif case["layout"] == "paged":
        page = 16
        pages = -(-L // page)
        spare = torch.zeros((Hkv, pages * page - L, d), device="cuda", dtype=dtype)
        s["table"] = torch.randperm(pages, generator=gen, device="cuda").to(torch.int32)
        place = s["table"].long()
        paged = []
        for t in (k, v):
            logical = torch.cat([t, spare], dim=1).view(Hkv, pages, page, d).permute(1, 2, 0, 3).contiguous()
            cache = torch.empty_like(logical)
            cache[place] = logical
            paged.append(cache)
        k, v = paged
    elif case["workspace"]:
        need = snapkv.snapkv_workspace_bytes(L, Hq, Hkv, d, W)
        s["workspace"] = torch.empty(need, device="cuda", dtype=torch.uint8)
    s["k"], s["v"] = k, v
    return s


def _prepare_decode(case, gen, dtype):
    """N(0, 1) caches; a few rows of every head are what the head's queries look for, as in a cache that kept them."""
    B, Hq, Hkv, d, S, cap = (case[x] for x in ("B", "Hq", "Hkv", "D", "S", "cap"))
    q = torch.randn((B, Hq, d), generator=gen, device="cuda")
    k = torch.empty((B, Hkv, cap, d), device="cuda", dtype=dtype).normal_(generator=gen)
    v = torch.empty((B, Hkv, cap, d), device="cuda", dtype=dtype).normal_(generator=gen)
    u = _unit(gen, (B, Hkv, d))
    rows = torch.randint(0, S // 2, (4,), generator=gen, device="cuda")
    k[:, :, rows] += (2.0 * u).to(dtype).unsqueeze(2)
    q += 3.0 * u.repeat_interleave(Hq // Hkv, dim=1)
    lens = None
    if case["ragged"]:
        lens = torch.tensor(_decode_lens(case), device="cuda", dtype=torch.int32)
    return {"case": case, "q": q.to(dtype), "k": k, "v": v, "lens": lens, "out": torch.empty((B, Hq, d), device="cuda"),
            "lse": torch.empty((B, Hq), device="cuda")}


def _decode_lens(case):
    """Valid rows per sequence: the kept rows and between none and all of the last fifth, generated since."""
    if not case["ragged"]:
        return [case["S"]] * case["B"]
    rng = random.Random(case["S"])
    return [rng.randint(case["S"] - case["S"] // 5, case["S"]) for _ in range(case["B"])]


def _bits(t):
    """Kept rows are copied, never computed: they are compared as the whole numbers their bits are."""
    return t.view(torch.int32 if t.element_size() == 4 else torch.int16)


def run(s):
    c = s["case"]
    if c["kind"] == "decode":
        snapkv.snapkv_decode_attention(s["q"], s["k"], s["v"], c["S"], s["out"], s["lse"], lens=s["lens"])
        return s["out"], s["lse"]
    args = (s["pool"], c["p"], c["C"], s["out_k"], s["out_v"], s["out_idx"])
    if c["kind"] == "layers":
        snapkv.snapkv_compress_layers(s["q"], s["k"], s["v"], *args)
        k, v, idx = s["whole"]
        return _bits(k), _bits(v), idx
    if c["kind"] == "varlen":
        snapkv.snapkv_compress_varlen(s["q"], s["k"], s["v"], *args)
    elif c["layout"] == "paged":
        snapkv.snapkv_compress_paged(s["q"], s["k"], s["v"], s["table"], c["L"], *args)
    elif c["layout"] == "token_major":
        snapkv.snapkv_compress_strided(s["q"], s["k"], s["v"], *args)
    else:
        snapkv.snapkv_compress(s["q"], s["k"], s["v"], *args, workspace=s["workspace"])
    if c["kind"] == "compress":
        return _bits(s["out_k"]), _bits(s["out_v"]), s["out_idx"]
    return {"k": [_bits(t) for t in s["out_k"]], "v": [_bits(t) for t in s["out_v"]], "idx": s["out_idx"]}


def work(case):
    e, Hq, Hkv, d = DTYPES[case["dtype"]].itemsize, case["Hq"], case["Hkv"], case["D"]
    if case["kind"] == "decode":
        rows = sum(_decode_lens(case))
        return {"bytes": 2 * rows * Hkv * d * e + case["B"] * Hq * (d * (e + 4) + 4), "flops": 4 * rows * Hq * d}
    lengths = _lengths(case) if case["kind"] == "varlen" else [case["L"]] * case.get("layers", 1)
    W, C = case["W"], case["C"]
    total = {"bytes": 0, "flops": 0}
    for L in lengths:
        kept = min(C, L)
        scored = (Hkv * L + Hq * W) * d * e if L > C else 0    # a prompt that fits is copied, not scored
        total["bytes"] += scored + 4 * Hkv * kept * d * e + 4 * Hkv * kept
        total["flops"] += 2 * Hq * W * L * d if L > C else 0
    return total


def tolerance(case):
    if case["kind"] == "decode":
        # probabilities enter the product with V as two 16-bit parts; against float64: rel 8.4e-6, max 3.3e-5
        return {"rel": 3e-5, "max": 1.3e-4}
    # Which rows are kept is decided by comparing fp32 sums.  Where two positions' scores agree to the last bits, another
    # order of summation may keep the other one; in that head every row between the two then moves by one place.  With
    # the sums in the order of the two-pass scoring kernels no position of the listed cases changes (three seeds).
    return {"differ": 0.005}
