"""The work this library is used for, as timed cases.

Five kinds of call sequences, each through the public entry points and with the buffers, plans and
workspaces a program keeps between calls:

  prefill        compress() of a prompt's cache, layers folded into the batch dimension
  recluster      compress() of one layer's grown cache at decode time: one round, with its degrees
  decode         one decode step: append() and decode_attn() for every layer
  paged_decode   the same step on block-paged caches
  paged_prefill  a prompt's cache written to pages (paged_scatter) and compressed there (paged_compress)

Keys are first-order autoregressive along the sequence with a few scaled-up channels, values and
queries are normal: the structure the clustering relies on, and what the tests and the benchmark use.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2506_11418_amd as ckv

DEV = "cuda"
_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_MAX_ROWS = 32 * 8 * 131072      # (layer, head) token rows of the largest prefill


# ---- the listed cases -----------------------------------------------------------------------------
def listed():
    return [
        # the smallest cache in use: one head in fp32, half of it kept - nothing but launches and latency
        _prefill("prefill_tiny_f32", layers=1, heads=1, seq=1024, dim=64, dtype="f32", chunk=64, retain=0.5),
        # one layer of a 32k prompt, kept at a quarter: a compression that does not fill the chip for long
        _prefill("prefill_layer_32k", layers=1, heads=8, seq=32768, chunk=1024, retain=0.25),
        # the full-model prompt: 32 layers in one call, the largest job
        _prefill("prefill_model_128k", layers=32, heads=8, seq=131072, chunk=1024, retain=0.25),
        # the method's own defaults on a prompt of no round length: chunk 256, sinks, recents, annealed rounds
        _prefill("prefill_annealed_50k", layers=8, heads=8, seq=50003, chunk=256, retain=0.25, annealed=True,
                 n_sink=16, n_recent=64, assign=False),
        # one layer of an extreme context, the largest chunk
        _prefill("prefill_layer_1m", layers=1, heads=8, seq=1048576, chunk=2048, retain=0.25),
        # decode-time clustering of one layer: a quarter of a 32k prompt plus the tokens decoded since
        dict(name="recluster_8k", kind="recluster", heads=8, seq=8448, dim=128, dtype="bf16", chunk=256, r=0.8,
             n_sink=16, n_recent=64),
        # one layer of a short compressed context: the launch latency of a decode step
        _decode("decode_short", layers=1, batch=1, tokens=515),
        # a full-model decode step over a 128k prompt's compressed cache
        _decode("decode_model_32k", layers=32, batch=1, tokens=32769),
        # serving: 16 sequences of different lengths over compressed caches, four layers of it
        _decode("decode_serving_16x8k", layers=4, batch=16, tokens=8223),
        # the same step over uncompressed caches (no degrees), eight query heads per KV head
        _decode("decode_uncompressed_4x32k", layers=2, batch=4, tokens=32801, group=8, degrees=False),
        # serving on pages of 16 tokens
        _decode("paged_decode_16x8k", kind="paged_decode", layers=4, batch=16, tokens=8223, block=16),
        # prompts arriving in a paged cache and compressed there
        dict(name="paged_prefill_4x16k", kind="paged_prefill", batch=4, heads=8, seq=16384, dim=128, dtype="bf16",
             chunk=1024, retain=0.25, block=16, n_sink=0, n_recent=0),
    ]


def _prefill(name, layers, heads, seq, chunk, retain, dim=128, dtype="bf16", annealed=False, n_sink=0, n_recent=0,
             scope="chunk", assign=True):
    return dict(name=name, kind="prefill", layers=layers, heads=heads, seq=seq, dim=dim, dtype=dtype, chunk=chunk,
                retain=retain, annealed=annealed, n_sink=n_sink, n_recent=n_recent, scope=scope, assign=assign)


def _decode(name, layers, batch, tokens, kind="decode", heads=8, group=4, dim=128, dtype="bf16", degrees=True, block=0):
    return dict(name=name, kind=kind, layers=layers, batch=batch, heads=heads, group=group, tokens=tokens, dim=dim,
                dtype=dtype, degrees=degrees, block=block)


# ---- more cases of the same ranges ----------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "prefill", "recluster", "decode", "decode", "decode", "paged_decode",
                       "paged_prefill"))
    heads = rng.choice((2, 4, 8, 8, 8))
    dim = rng.choice((64, 128, 128, 128))
    if kind == "prefill":
        if rng.random() < 0.15:      # fp32 caches: small ones
            return _unnamed(_prefill("", layers=1, heads=rng.choice((1, 2, 4)), seq=_log(rng, 256, 8192),
                                     dim=rng.choice((64, 128)), dtype="f32", chunk=rng.choice((64, 128, 256)),
                                     retain=rng.choice((0.5, 0.25))))
        layers = rng.choice((1, 1, 2, 4, 8, 16, 32))
        seq = _log(rng, 1024, min(1 << 20, _MAX_ROWS // (layers * heads)))
        if rng.random() < 0.4:       # prompts padded to whole chunks
            seq = max(2048, seq // 2048 * 2048)
        if rng.random() < 0.25 and seq >= 8192:
            return _unnamed(_prefill("", layers, heads, seq, chunk=rng.choice((128, 256, 512)),
                                     retain=rng.choice((0.5, 0.25)), dim=dim, annealed=True, n_sink=16, n_recent=64,
                                     assign=False))
        return _unnamed(_prefill("", layers, heads, seq, chunk=rng.choice((64, 128, 256, 384, 512, 1024, 1024, 2048)),
                                 retain=rng.choice((0.5, 0.3, 0.25, 0.25)), dim=dim,
                                 scope=rng.choice(("chunk", "chunk", "chunk", "head")), assign=rng.random() < 0.5))
    if kind == "recluster":
        return dict(kind=kind, heads=heads, seq=_log(rng, 600, 40000), dim=dim, dtype="bf16",
                    chunk=rng.choice((64, 128, 256, 512, 1024)), r=rng.choice((0.8, 0.5, 1.0)), n_sink=16, n_recent=64)
    if kind == "paged_prefill":
        batch = rng.choice((1, 2, 4, 8))
        sinks = rng.random() < 0.5
        return dict(kind=kind, batch=batch, heads=heads, seq=_log(rng, 1000, 131072 // batch), dim=dim, dtype="bf16",
                    chunk=rng.choice((256, 512, 1024)), retain=rng.choice((0.5, 0.25)), block=rng.choice((16, 32, 64)),
                    n_sink=16 if sinks else 0, n_recent=64 if sinks else 0)
    layers, batch = rng.choice((1, 1, 2, 4)), rng.choice((1, 1, 2, 4, 8, 16, 32))
    tokens = _log(rng, 100, min(1 << 18, (1 << 22) // (layers * batch * heads)))
    dtype = "f32" if rng.random() < 0.1 else "bf16"
    return _unnamed(_decode("", layers, batch, tokens, kind=kind, heads=heads, group=rng.choice((1, 2, 4, 4, 8)), dim=dim,
                            dtype=dtype, degrees=rng.random() < 0.75,
                            block=rng.choice((16, 16, 32, 64)) if kind == "paged_decode" else 0))


def _unnamed(case):
    del case["name"]
    return case


# ---- what a program has in hand before the call ---------------------------------------------------
_ALPHA, _WARM_UP = 0.9, 256      # 0.9**256 < 2e-12: the recursion started at a cold state is stationary by then


def _ar1(gen, out):
    """out [seqs, seq, dim] := per channel k_t = a k_{t-1} + sqrt(1 - a^2) N(0,1), 4 of 128 channels times 10."""
    seqs, seq, dim = out.shape
    at_once = max(1, (1 << 26) // ((_WARM_UP + seq) * dim))
    for i in range(0, seqs, at_once):
        n = min(at_once, seqs - i)
        x = torch.randn((n, _WARM_UP + seq, dim), generator=gen, device=DEV).mul_(math.sqrt(1.0 - _ALPHA * _ALPHA))
        step = 1
        while step < _WARM_UP:       # x_t <- sum over j < 2*step of a^j e_{t-j}
            y = x.clone()
            y[:, step:].add_(x[:, :-step], alpha=_ALPHA ** step)
            x, step = y, 2 * step
        loud = torch.rand((n, dim), generator=gen, device=DEV).topk(dim // 32, dim=1).indices
        x.mul_(torch.ones((n, dim), device=DEV).scatter_(1, loud, 10.0).unsqueeze(1))
        out[i:i + n].copy_(x[:, _WARM_UP:])


def _cache(gen, n_b, heads, seq, dim, dtype, capacity=None):
    """K, V [n_b, heads, capacity, dim] whose first seq rows are filled (the others zero)."""
    shape = (n_b, heads, capacity or seq, dim)
    K, V = torch.zeros(shape, dtype=_DT[dtype], device=DEV), torch.zeros(shape, dtype=_DT[dtype], device=DEV)
    _ar1(gen, K.view(n_b * heads, shape[2], dim)[:, :seq])
    V[:, :, :seq].normal_(generator=gen)
    return K, V


def _degrees(gen, shape):
    """Cluster sizes of a cache compressed to a quarter: 1 and up, four on average."""
    return 1 + torch.empty(shape, device=DEV).exponential_(1.0 / 3.5, generator=gen).to(torch.int32)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    return {"prefill": _prepare_prefill, "recluster": _prepare_recluster, "decode": _prepare_decode,
            "paged_decode": _prepare_paged_decode, "paged_prefill": _prepare_paged_prefill}[case["kind"]](case, gen)


def _schedule(case):
    """(retain_ratio, rounds) as compress() takes them."""
    if not case.get("annealed"):
        return case["retain"], None
    budget = ckv.budget_tokens(case["retain"], case["seq"])
    return 1.0, ckv.schedule_annealed(case["seq"], case["chunk"], budget, r_init=0.8, delta_r=0.2, r_floor=0.2,
                                      n_sink=case["n_sink"], n_recent=case["n_recent"])


def _prepare_prefill(case, gen):
    K, V = _cache(gen, case["layers"], case["heads"], case["seq"], case["dim"], case["dtype"])
    retain, rounds = _schedule(case)
    kw = dict(chunk=case["chunk"], retain_ratio=retain, rounds=rounds, n_sink=case["n_sink"], n_recent=case["n_recent"],
              scope=case["scope"])
    plan = ckv.plan(ckv.layout_of(K), ckv.make_params(**kw))
    shape = (case["layers"], case["heads"], plan.out_seq)
    out = (torch.zeros(shape + (case["dim"],), dtype=K.dtype, device=DEV),
           torch.zeros(shape + (case["dim"],), dtype=K.dtype, device=DEV),
           torch.zeros(shape, dtype=torch.int32, device=DEV),
           torch.zeros(K.shape[:3], dtype=torch.int32, device=DEV) if case["assign"] else None)
    ws = torch.zeros(max(plan.workspace_bytes, 256), dtype=torch.uint8, device=DEV)
    return dict(kind="prefill", K=K, V=V, kw=dict(kw, out=out, workspace=ws, want_assign=case["assign"]))


def _prepare_recluster(case, gen):
    K, V = _cache(gen, 1, case["heads"], case["seq"], case["dim"], case["dtype"])
    deg = _degrees(gen, K.shape[:3])
    kw = dict(chunk=case["chunk"], rounds=[case["r"]], n_sink=case["n_sink"], n_recent=case["n_recent"])
    plan = ckv.plan(ckv.layout_of(K, deg), ckv.make_params(**kw))
    out_K = torch.zeros((1, case["heads"], plan.out_seq, case["dim"]), dtype=K.dtype, device=DEV)
    out = (out_K, torch.zeros_like(out_K), torch.zeros(out_K.shape[:3], dtype=torch.int32, device=DEV), None)
    ws = torch.zeros(max(plan.workspace_bytes, 256), dtype=torch.uint8, device=DEV)
    return dict(kind="recluster", K=K, V=V, kw=dict(kw, deg=deg, out=out, workspace=ws, want_assign=False))


def _lens(case):
    """Tokens per sequence before the step: spread evenly over [half, all], in no particular order."""
    full, n = case["tokens"] - 1, case["batch"]
    return [full - (i * 7 % n) * (full - full // 2) // max(n - 1, 1) for i in range(n)]


def _step_inputs(case, gen):
    L, B, H, D, dt = case["layers"], case["batch"], case["heads"], case["dim"], _DT[case["dtype"]]
    new = [torch.empty((L, B, n, D), dtype=dt, device=DEV).normal_(generator=gen) for n in (H * case["group"], H, H)]
    lens0 = torch.tensor(_lens(case), dtype=torch.int32, device=DEV).expand(L, B).contiguous()
    return dict(kind=case["kind"], layers=L, n=case["tokens"], q=new[0], k_new=new[1], v_new=new[2],
                o=torch.zeros_like(new[0]), lens0=lens0, lens=lens0.clone())


def _prepare_decode(case, gen):
    L, B, H, n = case["layers"], case["batch"], case["heads"], case["tokens"]
    s = _step_inputs(case, gen)
    K, V = _cache(gen, L * B, H, n - 1, case["dim"], case["dtype"], capacity=n + 63)
    K, V = K.view((L, B) + K.shape[1:]), V.view((L, B) + V.shape[1:])
    deg = _degrees(gen, K.shape[:4]) if case["degrees"] else None
    ws = torch.zeros(ckv.decode_attn_workspace(ckv.layout_of(K[0]), H * case["group"]), dtype=torch.uint8, device=DEV)
    return _by_layer(dict(s, batch=B, K=K, V=V, deg=deg, ws=ws))


def _prepare_paged_decode(case, gen):
    L, B, H, D, n, bs = case["layers"], case["batch"], case["heads"], case["dim"], case["tokens"], case["block"]
    s = _step_inputs(case, gen)
    per_seq = -(-n // bs)
    table = torch.randperm(B * per_seq, generator=gen, device=DEV).to(torch.int32).view(B, per_seq)
    K = torch.zeros((L, B * per_seq, H, bs, D), dtype=_DT[case["dtype"]], device=DEV)
    V = torch.empty_like(K).normal_(generator=gen)
    keys = torch.empty((B * H, per_seq * bs, D), dtype=K.dtype, device=DEV)
    for layer in range(L):           # every sequence's keys, block by block, where the table puts them
        _ar1(gen, keys)
        K[layer, table.long()] = keys.view(B, H, per_seq, bs, D).transpose(1, 2)
    deg = _degrees(gen, K.shape[:4]) if case["degrees"] else None
    pl, nbytes = ckv.paged_layout_of(K[0], table), ctypes.c_size_t(0)
    if ckv.lib().ckv_paged_decode_attn_workspace(ctypes.byref(pl), H * case["group"], n, ctypes.byref(nbytes)) != 0:
        raise ValueError("no workspace size for this case")
    ws = torch.zeros(nbytes.value, dtype=torch.uint8, device=DEV)
    return _by_layer(dict(s, K=K, V=V, deg=deg, table=table, ws=ws))


def _by_layer(s):
    """A model keeps one cache per layer: the layers' views beside the tensors they are cut from."""
    views = zip(s["q"], s["k_new"], s["v_new"], s["K"], s["V"], s["deg"] if s["deg"] is not None else [None] * s["layers"],
                s["o"], s["lens"])
    return dict(s, views=list(views))


def _prepare_paged_prefill(case, gen):
    B, H, S, D, bs = case["batch"], case["heads"], case["seq"], case["dim"], case["block"]
    K, V = _cache(gen, B, H, S, D, case["dtype"])
    per_seq = -(-S // bs)
    table = torch.randperm(B * per_seq, generator=gen, device=DEV).to(torch.int32).view(B, per_seq)
    K_pool = torch.zeros((B * per_seq, H, bs, D), dtype=K.dtype, device=DEV)
    V_pool, deg_pool = torch.zeros_like(K_pool), torch.zeros(K_pool.shape[:3], dtype=torch.int32, device=DEV)
    kw = dict(chunk=case["chunk"], retain_ratio=case["retain"], n_sink=case["n_sink"], n_recent=case["n_recent"])
    _, _, nbytes = ckv.paged_compress_plan(ckv.paged_layout_of(K_pool, table), S, ckv.make_params(**kw))
    ws = torch.zeros(max(nbytes, 256), dtype=torch.uint8, device=DEV)
    lens = torch.zeros(B, dtype=torch.int32, device=DEV)
    return dict(kind="paged_prefill", K=K, V=V, pools=(K_pool, V_pool, deg_pool), blocks=table, table=table.clone(),
                lens=lens, seq=S, kw=dict(kw, lens=lens, workspace=ws))


# ---- one pass -------------------------------------------------------------------------------------
def run(s):
    if s["kind"] in ("prefill", "recluster"):
        return ckv.compress(s["K"], s["V"], **s["kw"])
    if s["kind"] == "paged_prefill":
        s["table"].copy_(s["blocks"])              # the block manager hands the blocks out
        ckv.paged_scatter(s["K"], s["V"], None, *s["pools"], s["table"], s["seq"])
        _, freed = ckv.paged_compress(*s["pools"], s["table"], s["seq"], **s["kw"])
        return s["pools"] + (s["table"], s["lens"], freed)
    n, ws = s["n"], s["ws"]
    if s["kind"] == "paged_decode":
        s["lens"].copy_(s["lens0"])                # this step's lengths, before the new token
        table = s["table"]
        for q, k, v, K, V, deg, o, lens in s["views"]:
            ckv.paged_append(k, v, K, V, deg, table, lens)
            ckv.paged_decode_attn(q, K, V, deg, table, lens, n, out=o, workspace=ws)
    elif s["batch"] > 1:
        s["lens"].copy_(s["lens0"])
        for q, k, v, K, V, deg, o, lens in s["views"]:
            ckv.append(k, v, K, V, deg, lens=lens)
            ckv.decode_attn(q, K, V, lens=lens, deg=deg, out=o, workspace=ws)
    else:                                          # one sequence: its length is known to the program
        for q, k, v, K, V, deg, o, lens in s["views"]:
            ckv.append(k, v, K, V, deg, pos=n - 1)
            ckv.decode_attn(q, K[:, :, :n], V[:, :, :n], deg=None if deg is None else deg[:, :, :n], out=o, workspace=ws)
    return s["o"], s["K"], s["V"], s["deg"], s["lens"]


# ---- the same results in 64 bits ------------------------------------------------------------------
def _round64(K, V, deg, chunk, r, n_sink, n_recent, scope):
    """One round on a sequence: K, V [n, dim] in 64 bits, deg [n].  Returns the sums' quotients (64 bits) and the map."""
    n, where = K.shape[0], torch.arange(K.shape[0], device=K.device)
    lo, hi = (0, 0) if n <= n_sink + n_recent else (n_sink, n - n_recent)
    whole = lo + (hi - lo) // chunk * chunk
    src, dst, score, kept = [], [], [], []
    for first, last, size in ((lo, whole, chunk), (whole, hi, hi - whole)):
        if last - first < 2:
            continue
        x = K[first:last].view(-1, size, K.shape[1])
        unit = x / x.norm(dim=2, keepdim=True).clamp_min(1e-300)
        best = torch.bmm(unit[:, 0::2].contiguous(), unit[:, 1::2].transpose(1, 2).contiguous()).max(dim=2)
        t = where[first:last].view(-1, size)
        m = int(r * t[:, 0::2].shape[1] + 1e-9)
        rank = best.values.argsort(dim=1, descending=True, stable=True).argsort(dim=1)
        src.append(t[:, 0::2].reshape(-1))
        dst.append((t[:, :1] + 2 * best.indices + 1).reshape(-1))
        score.append(best.values.reshape(-1))
        kept.append((rank < m).reshape(-1))
    to = where.clone()
    if src:
        src, dst, score, kept = torch.cat(src), torch.cat(dst), torch.cat(score), torch.cat(kept)
        if scope == "head":          # one ranking over the edges of all chunks
            kept = score.argsort(descending=True, stable=True).argsort() < int(r * score.numel() + 1e-9)
        to[src[kept]] = dst[kept]
    left = to == where
    d = torch.zeros_like(deg).index_add_(0, to, deg)[left]
    K, V = (torch.zeros_like(x).index_add_(0, to, x * deg.unsqueeze(1).double())[left] / d.unsqueeze(1).double() for x in (K, V))
    return K, V, d, (left.cumsum(0) - 1)[to]


def _compress64(K, V, deg, dtype, chunk, rounds, n_sink, n_recent, scope):
    """compress() of one sequence.  Between the rounds the cache is held in its own type, as the method has it."""
    assign = torch.arange(K.shape[0], device=K.device)
    for j, r in enumerate(rounds):
        if j:
            K, V = K.to(dtype), V.to(dtype)
        K, V, deg, to = _round64(K.double(), V.double(), deg, chunk, r, n_sink, n_recent, scope)
        assign = to[assign]
    return K.double(), V.double(), deg.to(torch.int32), assign.to(torch.int32)


def _exact_compress(s, rounds):
    kw, K, V = s["kw"], s["K"], s["V"]
    B, H, S = K.shape[:3]
    got = []
    for b in range(B):
        for h in range(H):
            deg = kw["deg"][b, h].long() if kw.get("deg") is not None else torch.ones(S, dtype=torch.long, device=DEV)
            got.append(_compress64(K[b, h], V[b, h], deg, K.dtype, kw["chunk"], rounds, kw["n_sink"], kw["n_recent"],
                                   kw.get("scope", "chunk")))
    outs = []
    for parts in zip(*got):
        x = torch.stack(parts)
        outs.append(x.view((B, H) + x.shape[1:]))
    return outs


def _to_pages(pool, table, rows):
    """pool [n_blocks, heads, block, ...] := the sequences' first rows [batch, heads, n, ...], where the table puts them."""
    n, bs = rows.shape[2], pool.shape[2]
    t = torch.arange(n, device=DEV)
    pool[table[:, t // bs].long(), :, t % bs] = rows.transpose(1, 2)


def _rounds(kw):
    """The merge fractions of the schedule, in 32 bits as the library carries them."""
    rounds = kw.get("rounds")
    if rounds is None:
        retain = float(np.float32(kw["retain_ratio"]))
        n = math.ceil(math.log2(1 / retain) - 1e-6)
        rounds = [1.0] * (n - 1) + [2 * (1 - retain * 2 ** (n - 1))] if n else []
    return [float(np.float32(r)) for r in rounds]


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] in ("prefill", "recluster"):
        K, V, deg, assign = _exact_compress(s, _rounds(s["kw"]))
        return K, V, deg, assign if s["kw"]["want_assign"] else None
    if case["kind"] == "paged_prefill":            # rows behind the new length keep what the prompt wrote there
        outs = _exact_compress(s, _rounds(s["kw"]))
        pools = (s["pools"][0].double(), s["pools"][1].double(), s["pools"][2])
        prompt = (s["K"].double(), s["V"].double(), torch.ones(s["K"].shape[:3], dtype=torch.int32, device=DEV))
        for pool, before, after in zip(pools, prompt, outs):
            _to_pages(pool, s["blocks"], before)
            _to_pages(pool, s["blocks"], after)
        return pools + (None, None, None)
    o = torch.zeros_like(s["o"], dtype=torch.float64)
    G, D, bs = case["group"], case["dim"], case["block"]
    for i, (q, k, v, K, V, deg, _, lens) in enumerate(s["views"]):
        for b, n in enumerate(_lens(case)):
            if bs:                   # this sequence's blocks in order
                blocks = s["table"][b].long()
                Kb, Vb = (x[blocks].transpose(0, 1).reshape(case["heads"], -1, D)[:, :n].double() for x in (K, V))
                db = None if deg is None else deg[blocks].transpose(0, 1).reshape(case["heads"], -1)[:, :n]
            else:
                Kb, Vb, db = K[b, :, :n].double(), V[b, :, :n].double(), None if deg is None else deg[b, :, :n]
            Kb, Vb = torch.cat([Kb, k[b].double().unsqueeze(1)], 1), torch.cat([Vb, v[b].double().unsqueeze(1)], 1)
            z = torch.bmm(q[b].double().view(-1, G, D), Kb.transpose(1, 2).contiguous()) / math.sqrt(D)
            if db is not None:       # the new token's degree is 1: log 1 = 0
                z[:, :, :n] += db.double().log().unsqueeze(1)
            o[i, b] = torch.bmm(z.softmax(dim=2), Vb).view(-1, D)
    return (o, None, None, None, None)               # the caches are copies


# ---- what a pass cannot do without ----------------------------------------------------------------
def _match_flops(tokens, chunk, dim):
    full, tail = divmod(max(tokens, 0), chunk)
    return 2.0 * dim * (full * (chunk // 2) ** 2 + ((tail + 1) // 2) * (tail // 2))


def work(case):
    kind, d, e = case["kind"], case["dim"], 4 if case["dtype"] == "f32" else 2
    row = 2 * d * e                                # a token's key and value
    if kind in ("decode", "paged_decode"):
        tokens = sum(n + 1 for n in _lens(case))
        per_head = tokens * (row + (4 if case["degrees"] else 0)) + case["batch"] * (row + 2 * case["group"] * d * e)
        table = 4 * -(-tokens // case["block"]) if case["block"] else 0
        return {"bytes": case["layers"] * (case["heads"] * per_head + table),
                "flops": 4.0 * d * case["layers"] * case["heads"] * case["group"] * tokens}
    if kind == "recluster":
        n_bh, rounds, retain, deg_in, assign, scope = case["heads"], [case["r"]], 1.0, 4, 0, "chunk"
    else:
        n_bh = case["heads"] * case.get("layers", case.get("batch"))
        retain, rounds = _schedule(case)
        deg_in, assign, scope = 0, 4 if case.get("assign") else 0, case.get("scope", "chunk")
    edge = case["n_sink"] + case["n_recent"]
    lay = ckv.Layout(1, n_bh, case["seq"], d, n_bh * case["seq"] * d, case["seq"] * d, d, int(e == 2), 0)
    plan = ckv.plan(lay, ckv.make_params(case["chunk"], retain, rounds, case["n_sink"], case["n_recent"], scope))
    flops = sum(_match_flops(n - edge, case["chunk"], d) for n in plan.round_len[:-1])
    nbytes = case["seq"] * (row + deg_in + assign) + plan.out_seq * (row + 4)
    if kind == "paged_prefill":                    # and the prompt's own way into its pages
        nbytes += case["seq"] * (row + 4)
    return {"bytes": n_bh * nbytes, "flops": n_bh * flops}


# Measured: every path against itself with the channels of keys and queries in another order (and, for one
# sequence, the cached tokens in reverse), which changes nothing but the order of the fp32 sums.
#   attention   fp32 outputs differed by 9e-7, bf16 outputs (their own rounding flips) by 1.6e-4, single
#               values by 7e-6 and two ulps;
#   clustering  two partners whose similarities agree to the last bits can change places: one match in 1e5 or
#               fewer, each moving a row (rel up to 2.3e-3).  In the annealed schedule a swap at the cut of one
#               round shifts rows of its chunk and so the pairing of the rounds after it: 1.4e-3 of the rows,
#               rel up to 0.055.
# Four times that:
def tolerance(case):
    if case["kind"] in ("decode", "paged_decode"):
        return {"rel": 4e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 7e-4, "max": 0.03}
    if case.get("annealed"):
        return {"rel": 0.22, "differ": 6e-3}
    return {"rel": 1e-2, "differ": 4e-5}
