"""The workloads whose time and results are watched: what a serving engine has this library do.

One case is one pass of the public entry points of ``paper_2602_10718_amd.snapmla`` at one size:

  step    one decode step of a batch: append + query quantization + decode (one call) and the split-KV
          merge, over the FP8 cache; ``exact_qk`` selects the exact accumulation of the content logits
  bf16    the same step over a BF16 cache (append, decode, merge)
  append  a prefill chunk written into the paged FP8 cache
  fetch   cached prefixes read back as BF16 rows (chunked prefill, prefix reuse)

Inputs are synthetic and made on the GPU from the seed.  The latents are what a normalised compressed
KV looks like: unit-variance channels with a few outlier channels and a mild per-token magnitude
spread; RoPE keys are rotated at their position and have the larger range.  Queries are scaled so
that a row's logits spread over a few units: attention rests on tens to hundreds of tokens.  Pages
are scattered over the pool at random, as a paged allocator leaves them.
"""

import random

import numpy as np
import torch

PAGE, D_C, D_R = 64, 512, 64
TAU = 192.0 ** -0.5
EPS = 2.0 ** -40
FP8_MAX = 448.0


def _step(name, B, H, q_len, lo, hi, lens_seed=1, n_new=None, chunk=0, exact_qk=False, out="bf16", op="step"):
    return {"name": name, "op": op, "B": B, "H": H, "q_len": q_len, "lo": lo, "hi": hi, "lens_seed": lens_seed,
            "n_new": q_len if n_new is None else n_new, "chunk": chunk, "exact_qk": exact_qk, "out": out}


def listed():
    return [
        # one short request on one tensor-parallel rank: launches and latency
        _step("tiny", 1, 16, 1, 256, 256),
        # a few chat requests at a time, all 128 heads on the GPU
        _step("interactive", 4, 128, 1, 1500, 9000),
        # a batch of long documents with few requests: every sequence spread over many workgroups
        _step("few-long", 3, 32, 2, 20000, 60000),
        # 128 heads, short contexts of one length, the batch fits the last-level cache
        _step("heads128", 32, 128, 1, 4096, 4096),
        # the main serving load: 64 heads, ragged 8K-32K contexts
        _step("heads64", 64, 64, 1, 8192, 32768, out="f32"),
        # 128 heads over 8 tensor-parallel ranks: 16 heads against long ragged contexts
        _step("heads16-long", 32, 16, 1, 16384, 131072),
        # 128K contexts cut into fixed 4K chunks
        _step("long-chunks", 8, 64, 1, 131072, 131072, chunk=4096, out="f32"),
        # speculative decoding: two query tokens, causal, 128 heads, ragged 1K-16K
        _step("mtp", 128, 128, 2, 1024, 16384),
        # the main load with exact accumulation of the content logits
        _step("heads64-exact", 48, 64, 1, 4096, 32768, exact_qk=True),
        # the unquantized cache: the same kind of batch over BF16 latents
        _step("bf16-cache", 48, 64, 1, 4096, 24576, op="bf16"),
        # one prefill chunk of 8 requests quantized into their pages
        {"name": "append-prefill", "op": "append", "B": 8, "n_new": 4096, "lo": 4096, "hi": 30000, "lens_seed": 1},
        # cached prefixes of 24 requests fetched for chunked prefill
        {"name": "fetch-prefix", "op": "fetch", "B": 24, "lo": 777, "hi": 40000, "lens_seed": 1},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    seed = rng.randrange(1 << 20)
    kind = rng.choice(["step"] * 8 + ["exact", "bf16", "append", "fetch"])
    if kind == "append":
        B, n = _log(rng, 1, 64), _log(rng, 16, 8192)
        n = max(1, min(n, 32768 // B))
        return {"op": "append", "B": B, "n_new": n, "lo": n, "hi": n + _log(rng, 1, 20000), "lens_seed": seed}
    budget = 400_000 if kind in ("exact", "bf16", "fetch") else 1_000_000      # tokens in the cache
    hi = _log(rng, 200, 131072)
    lo = max(2, int(hi * rng.choice([1.0, 0.7, 0.25, 0.06])))
    B = max(1, min(_log(rng, 1, 128), 2 * budget // (lo + hi)))
    if kind == "fetch":
        return {"op": "fetch", "B": B, "lo": lo, "hi": hi, "lens_seed": seed}
    H = rng.choice([8, 16, 16, 32, 48, 64, 64, 96, 128, 128])
    q_len = rng.choice([1, 1, 1, 2])
    chunk = 64 * _log(rng, 16, 128) if kind == "step" and hi > 16384 and rng.random() < 0.2 else 0
    c = _step("", B, H, q_len, lo, hi, seed, chunk=chunk, exact_qk=kind == "exact", out=rng.choice(["bf16", "f32"]),
              op="bf16" if kind == "bf16" else "step")
    del c["name"]
    return c


def _lens(case):
    r = random.Random("lens %d" % case["lens_seed"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["B"])]


def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, what):
    return torch.Generator(device=_dev()).manual_seed(1_000_003 * seed + what)


def _quantize(x):
    """Per-token E4M3 codes (uint8) and float32 scales of bf16 rows [n, 512]."""
    x = x.float()
    top = x.abs().amax(-1)
    sigma = (top / torch.full_like(top, FP8_MAX)).clamp_min(EPS)     # (a tensor: a number would be multiplied by its reciprocal)
    codes = (x / sigma[:, None]).clamp(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, sigma


def _pages(case, seed, lens):
    """(page table on the host, pages in the pool): scattered pages, -1 past a sequence's end."""
    npg = [(n + PAGE - 1) // PAGE for n in lens]
    perm = np.random.RandomState(seed % (1 << 31)).permutation(sum(npg)).astype(np.int32)
    table = np.full((case["B"], max(npg)), -1, np.int32)
    at = 0
    for b, n in enumerate(npg):
        table[b, :n] = perm[at:at + n]
        at += n
    return table, at


def _tokens(case, seed, lens):
    """Latents and RoPE keys of every token in bf16, the sequences one after another: yields
    (first row, latent [n, 512], rope [n, 64]) in parts of whole pages of a sequence."""
    dev = _dev()
    hot = torch.from_numpy(np.random.RandomState(7).choice(D_C, 4, replace=False)).to(dev)
    theta = 10000.0 ** (-torch.arange(D_R // 2, device=dev, dtype=torch.float32) / (D_R // 2))
    g = _gen(seed, 1)
    row = 0
    for b, N in enumerate(lens):
        for t0 in range(0, N, 32768):
            n = min(32768, N - t0)
            c = torch.randn((n, D_C), device=dev, generator=g)
            c *= torch.exp(0.3 * torch.randn((n, 1), device=dev, generator=g))
            c[:, hot] *= 10.0
            r = 2.0 * torch.randn((n, D_R), device=dev, generator=g)
            ang = torch.arange(t0, t0 + n, device=dev, dtype=torch.float32)[:, None] * theta
            r1, r2 = r[:, :D_R // 2], r[:, D_R // 2:]
            r = torch.cat([r1 * ang.cos() - r2 * ang.sin(), r1 * ang.sin() + r2 * ang.cos()], 1)
            yield b, t0, row, c.bfloat16(), r.bfloat16()
            row += n


def _queries(case, seed):
    g = _gen(seed, 2)
    shape = (case["B"], case["q_len"], case["H"])
    return (torch.randn(shape + (D_C,), device=_dev(), generator=g).bfloat16(),
            torch.randn(shape + (D_R,), device=_dev(), generator=g).bfloat16())


def _slots(table, b, t0, n, dev):
    """Cache slots (page * 64 + place) of tokens t0 .. t0+n-1 of sequence b."""
    t = torch.arange(t0, t0 + n, device=dev)
    return torch.from_numpy(table[b]).to(dev)[t // PAGE].long() * PAGE + t % PAGE


def prepare(case, seed):
    from paper_2602_10718_amd import snapmla as sm
    from paper_2602_10718_amd.runner import prefer_unsplit

    dev, op, B = _dev(), case["op"], case["B"]
    lens = _lens(case)
    table, pages = _pages(case, seed, lens)
    fp8 = op != "bf16"
    latent = torch.zeros((pages, PAGE, D_C), dtype=torch.uint8 if fp8 else torch.bfloat16, device=dev)
    scale = torch.zeros((pages, PAGE), dtype=torch.float32, device=dev) if fp8 else None
    rope = torch.zeros((pages, PAGE, D_R), dtype=torch.bfloat16, device=dev)
    n_new = case.get("n_new", 0)
    new_c = torch.zeros((B, n_new, D_C), dtype=torch.bfloat16, device=dev)
    new_r = torch.zeros((B, n_new, D_R), dtype=torch.bfloat16, device=dev)
    for b, t0, _, c, r in _tokens(case, seed, lens):
        old = max(0, min(len(c), lens[b] - n_new - t0))          # tokens of this part that are in the cache already
        if old < len(c):
            at = t0 + old - (lens[b] - n_new)
            new_c[b, at:at + len(c) - old] = c[old:]
            new_r[b, at:at + len(c) - old] = r[old:]
        if old:
            s = _slots(table, b, t0, old, dev)
            rope.view(-1, D_R)[s] = r[:old]
            if fp8:
                codes, sigma = _quantize(c[:old])
                latent.view(-1, D_C)[s] = codes
                scale.view(-1)[s] = sigma
            else:
                latent.view(-1, D_C)[s] = c[:old]
    st = {"op": op, "sm": sm, "latent": latent, "scale": scale, "rope": rope, "new_c": new_c, "new_r": new_r,
          "table": torch.from_numpy(table).to(dev), "lens": torch.tensor(lens, dtype=torch.int32, device=dev)}
    if op == "append":
        return st
    if op == "fetch":
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        st["cu"] = torch.from_numpy(cu).to(dev)
        st["out"] = torch.empty((int(cu[-1]), D_C + D_R), dtype=torch.bfloat16, device=dev)
        return st
    H, q_len, chunk = case["H"], case["q_len"], case["chunk"]
    st["q_nope"], st["q_rope"] = _queries(case, seed)
    # the split plan, as an engine that knows its batch's lengths picks it
    st["merge"] = True
    if chunk:
        splits = max((n + chunk - 1) // chunk for n in lens)
    elif prefer_unsplit(lens, q_len, H, "e4m3" if fp8 else "bf16"):
        chunk, splits, st["merge"] = table.shape[1] * PAGE, 1, False
    else:
        splits = sm.default_num_splits(q_len, H, total_blocks=sum((n + PAGE - 1) // PAGE for n in lens))
    st.update(B=B, H=H, q_len=q_len, splits=splits, chunk=chunk, causal=q_len > 1, pages=pages,
              flags=sm.DECODE_EXACT_QK if case["exact_qk"] else 0)
    size = sm.snapmla_decode_workspace_size(B, q_len, H, splits, chunk)
    st["workspace"] = torch.empty(size, dtype=torch.uint8, device=dev)
    st["out"] = torch.empty((B, q_len, H, D_C), dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16,
                            device=dev)
    st["lse"] = torch.empty((B, q_len, H), dtype=torch.float32, device=dev)
    return st


def run(st):
    sm, op = st["sm"], st["op"]
    if op == "append":
        sm.snapmla_quantize_append(st["new_c"], st["new_r"], st["table"], st["lens"], st["latent"].shape[0], st["latent"],
                                   st["scale"], st["rope"])
        return {"latent": st["latent"], "scale": st["scale"], "rope": st["rope"]}
    if op == "fetch":
        sm.snapmla_fetch_dequant(st["latent"], st["scale"], st["rope"], st["table"], st["cu"], st["out"])
        return {"out": st["out"]}
    if op == "bf16":
        sm.snapmla_append_bf16(st["new_c"], st["new_r"], st["table"], st["lens"], st["pages"], st["latent"], st["rope"])
        sm.snapmla_decode_bf16(st["q_nope"], st["q_rope"], st["latent"], st["rope"], st["table"], st["lens"], TAU,
                               st["causal"], st["splits"], st["chunk"], st["workspace"], out=st["out"], lse=st["lse"])
    else:
        sm.snapmla_append_decode(st["new_c"], st["new_r"], st["q_nope"], st["q_rope"], st["latent"], st["scale"],
                                 st["rope"], st["table"], st["lens"], TAU, st["causal"], st["splits"], st["chunk"],
                                 st["workspace"], flags=st["flags"], out=st["out"], lse=st["lse"])
    if st["merge"]:
        sm.snapmla_combine(st["workspace"], st["lens"], st["B"], st["q_len"], st["H"], st["splits"], st["chunk"],
                           st["out"], st["lse"])
    got = {"out": st["out"], "lse": st["lse"], "latent": st["latent"], "rope": st["rope"]}
    return got if st["scale"] is None else {**got, "scale": st["scale"]}


def work(case):
    lens, op, B = _lens(case), case["op"], case["B"]
    tokens = sum(lens)
    if op == "append":
        n = B * case["n_new"]
        return {"bytes": n * (2 * (D_C + D_R) + D_C + 4 + 2 * D_R), "flops": 0}
    if op == "fetch":
        return {"bytes": tokens * (D_C + 4 + 2 * D_R + 2 * (D_C + D_R)), "flops": 0}
    per = 2 * (D_C + D_R) if op == "bf16" else D_C + 4 + 2 * D_R
    R, q_len = case["q_len"] * case["H"], case["q_len"]
    seen = sum(n - q_len + 1 + t for n in lens for t in range(q_len))        # (query token, cached token) pairs, causal
    size = 4 if case["out"] == "f32" else 2
    new = B * case["n_new"] * 2 * (D_C + D_R)
    return {"bytes": tokens * per + new + B * R * (2 * (D_C + D_R) + size * D_C + 4),
            "flops": seen * case["H"] * 2 * (D_C + D_R + D_C)}


def tolerance(case):
    # About four times what the outputs were seen to be off exact(): bf16 outputs 1.7e-3, float32 ones up to 1.2e-4
    # over the FP8 cache (the FP8 matrix cores drop low bits beside a larger product, and a probability at the middle
    # of two E4M3 codes goes either way) and somewhat more over the BF16 cache (probabilities rounded to bf16).
    # Single outputs are off by up to 0.045 of the root mean square where a row sees few tokens.
    if case["op"] in ("append", "fetch"):
        return "exact"
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 0.2}
    return {"rel": 4e-3 if case["op"] == "bf16" else 5e-4, "max": 0.2}


def _attend(case, seed, fp8):
    """Outputs and log-sum-exps in 64 bits: softmax attention over the cache as stored, with the
    probabilities times the token scales rounded to E4M3 per 64-token block over the FP8 cache."""
    dev, H, q_len = _dev(), case["H"], case["q_len"]
    lens = _lens(case)
    qn, qr = _queries(case, seed)
    R = q_len * H
    out = torch.zeros((case["B"], q_len, H, D_C), dtype=torch.float64, device=dev)
    lse = torch.zeros((case["B"], q_len, H), dtype=torch.float64, device=dev)
    parts = {}
    for b, t0, _, c, r in _tokens(case, seed, lens):
        parts.setdefault(b, []).append((c, r))
        if t0 + len(c) < lens[b]:
            continue
        c, r = (torch.cat(x) for x in zip(*parts.pop(b)))
        N = lens[b]
        if fp8:
            kc, ks = _quantize(c)
            qc, qs = _quantize(qn[b].reshape(R, D_C))
            q = qc.view(torch.float8_e4m3fn).double() * qs.double()[:, None]
        else:
            q = qn[b].reshape(R, D_C).double()
        qro = qr[b].reshape(R, D_R).double()
        seen = N - q_len + 1 + torch.arange(R, device=dev) // H
        s = torch.empty((R, N), dtype=torch.float64, device=dev)
        for a in range(0, N, 16384):
            e = min(N, a + 16384)
            k = kc[a:e].view(torch.float8_e4m3fn).double() * ks[a:e].double()[:, None] if fp8 else c[a:e].double()
            s[:, a:e] = TAU * (q @ k.t() + qro @ r[a:e].double().t())
            s[:, a:e].masked_fill_(torch.arange(a, e, device=dev)[None, :] >= seen[:, None], -torch.inf)
        top = s.amax(1, keepdim=True)
        total = torch.zeros(R, dtype=torch.float64, device=dev)
        o = torch.zeros((R, D_C), dtype=torch.float64, device=dev)
        for a in range(0, N, 16384):                             # whole 64-token blocks
            e = min(N, a + 16384)
            p = torch.exp(s[:, a:e] - top)
            total += p.sum(1)
            if not fp8:
                o += p @ c[a:e].double()
                continue
            w = torch.nn.functional.pad(p * ks[a:e].double(), (0, -(e - a) % PAGE)).view(R, -1, PAGE)
            sp = (w.amax(2, keepdim=True) / FP8_MAX).clamp_min(EPS)
            w = (w / sp).float().to(torch.float8_e4m3fn).double() * sp
            o += w.view(R, -1)[:, :e - a] @ kc[a:e].view(torch.float8_e4m3fn).double()
        out[b] = (o / total[:, None]).view(q_len, H, D_C)
        lse[b] = (top[:, 0] + torch.log(total)).view(q_len, H)
    return out, lse


def exact(case, seed):
    op, lens, dev = case["op"], _lens(case), _dev()
    if op in ("step", "bf16"):
        out, lse = _attend(case, seed, op == "step")
        got = {"out": out, "lse": lse, "latent": None, "rope": None}
        return got if op == "bf16" else {**got, "scale": None}
    table, pages = _pages(case, seed, lens)
    if op == "append":
        scale = torch.zeros((pages, PAGE), dtype=torch.float64, device=dev)
        for b, t0, _, c, _r in _tokens(case, seed, lens):
            sigma = (c.double().abs().amax(-1) / FP8_MAX).clamp_min(EPS)
            scale.view(-1)[_slots(table, b, t0, len(c), dev)] = sigma
        return {"latent": None, "scale": scale, "rope": None}
    out = torch.empty((sum(lens), D_C + D_R), dtype=torch.float64, device=dev)
    for b, t0, row, c, r in _tokens(case, seed, lens):
        codes, sigma = _quantize(c)
        out[row:row + len(c), :D_C] = codes.view(torch.float8_e4m3fn).double() * sigma.double()[:, None]
        out[row:row + len(c), D_C:] = r.double()
    return {"out": out}
