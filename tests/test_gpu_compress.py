"""GPU parity: ckv_match / ckv_compress (HIP, through the C ABI) vs the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_11418_amd as ckv
from parity_util import DT, TOL, assert_rows_close, check_match, check_round, check_round_head, check_round_with_edges, f64, i64
from synth import kv_host

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _compress(route, *args, **kw):
    """ckv.compress on a named kernel route (the routes give the same bits)."""
    return ckv.compress(*args, route=route, **kw)


def _say(msg):
    print(msg, flush=True)


def _run_rounds_teacher_forced(K, V, chunk, rounds, what, deg=None):
    """Each round: GPU consumes the GPU's previous output; the oracle is fed the same input."""
    dtype = DT[K.dtype]
    curK, curV, curdeg = K, V, deg
    alt = 0
    for j, r in enumerate(rounds):
        gK, gV, gdeg, gas = ckv.compress(curK, curV, chunk, rounds=[r], deg=curdeg)
        torch.cuda.synchronize()
        B, H = curK.shape[:2]
        for b in range(B):
            for h in range(H):
                d_in = np.ones(curK.shape[2], dtype=np.int64) if curdeg is None else i64(curdeg[b, h])
                alt += check_round(f64(curK[b, h]), f64(curV[b, h]), d_in, chunk, r, dtype,
                                   f64(gK[b, h]), f64(gV[b, h]), i64(gdeg[b, h]), i64(gas[b, h]),
                                   what=f"{what} round {j} (b{b},h{h})")
        curK, curV, curdeg = gK, gV, gdeg
    return curK, curV, curdeg, alt


# ---- config 1: 1 x 1 x 1024 x 64 fp32, chunk 64 ---------------------------------------------
def _config1():
    K, V, rng = kv_host(0, 1, 1024, 64, "f32", alpha=0.9, single_stream=True)
    return K.to(DEV), V.to(DEV), rng


def test_match_config1_fp32():
    _say("match config1")
    K, V, _ = _config1()
    dst, score = ckv.match(K, 64)
    torch.cuda.synchronize()
    n = check_match(f64(K[0, 0]), 64, i64(dst[0, 0]), f64(score[0, 0]), "config1")
    assert n == 0


@pytest.mark.parametrize("rho,chunk", [(0.5, 64), (0.75, 64), (0.25, 64), (0.5, 8), (0.375, 16), (1.0, 64)])
def test_compress_config1_fp32(rho, chunk):
    _say(f"compress config1 rho={rho} chunk={chunk}")
    K, V, _ = _config1()
    pl = ckv.plan(ckv.layout_of(K), ckv.make_params(chunk, rho))
    fK, fV, fdeg, alt = _run_rounds_teacher_forced(K, V, chunk, pl.round_r, f"config1 rho={rho}")
    assert alt == 0
    # the one-call multi-round path gives the same bits as the chained single rounds
    gK, gV, gdeg, gas = ckv.compress(K, V, chunk, retain_ratio=rho)
    torch.cuda.synchronize()
    assert gK.shape[2] == pl.out_seq == int(round(rho * 1024))
    if pl.round_r:
        assert torch.equal(gK, fK) and torch.equal(gV, fV) and torch.equal(gdeg, fdeg)
    # and matches the oracle end to end (no near-ties on this input)
    ref = oracle.compress(f64(K[0, 0]), f64(V[0, 0]), chunk, pl.round_r, "f32")
    assert np.array_equal(i64(gas[0, 0]), ref["assign"])
    assert np.array_equal(i64(gdeg[0, 0]), ref["deg"])
    assert np.allclose(f64(gK[0, 0]), ref["K"], rtol=1e-5, atol=1e-6)
    assert np.array_equal(np.bincount(i64(gas[0, 0]), minlength=pl.out_seq), i64(gdeg[0, 0]))


# ---- bf16, several tiles, ragged tails ------------------------------------------------------
@pytest.mark.parametrize("heads,seq,dim,chunk", [
    (2, 4096, 128, 1024),      # two A blocks per chunk
    (2, 3000, 128, 1024),      # tail chunk of 952 tokens
    (1, 2047, 128, 256),       # odd tail
    (1, 5000, 128, 2048),      # largest chunk, ragged
    (2, 1536, 64, 512),        # head_dim 64
    (3, 700, 128, 64),         # small chunks
    (1, 130, 128, 2),          # smallest chunk
    (1, 1, 128, 16),           # single token
])
def test_match_bf16_shapes(heads, seq, dim, chunk):
    _say(f"match bf16 H={heads} S={seq} D={dim} c={chunk}")
    K, _, _ = kv_host(11, heads, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K = K.to(DEV)
    dst, score = ckv.match(K, chunk)
    torch.cuda.synchronize()
    for h in range(heads):
        check_match(f64(K[0, h]), chunk, i64(dst[0, h]), f64(score[0, h]), f"h{h}")


@pytest.mark.parametrize("heads,seq,dim,chunk", [
    (300, 201, 128, 200), (300, 200, 64, 200),      # 4 waves x 32 rows, a block per chunk
    (300, 641, 64, 384), (90, 1153, 128, 384),      # dim 64: 8 x 32 for a few chunks, 4 x 64 for many
    (130, 1537, 128, 1024), (130, 1024, 64, 1024),  # 8 x 32 for a few, 8 x 64 (or the streaming kernel) for many
    (70, 2048 + 515, 128, 2048), (70, 1400, 64, 1400),
])
def test_match_kernels_for_few_and_for_many_rows_agree(heads, seq, dim, chunk):
    """A chunk's matches do not depend on how many others share its launch: same bits, and the oracle's matching."""
    _say(f"match forms H={heads} S={seq} D={dim} c={chunk}")
    K, _, _ = kv_host(61, 2, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K = K.to(DEV)
    few = [x.clone() for x in ckv.match(K, chunk)]
    many = ckv.match(K.repeat(1, heads // 2, 1, 1), chunk)
    torch.cuda.synchronize()
    for a, b in zip(few, many):
        assert torch.equal(a.repeat(1, heads // 2, 1), b)
    for h in range(2):
        check_match(f64(K[0, h]), chunk, i64(few[0][0, h]), f64(few[1][0, h]), f"h{h}")


# ---- chunks of 64, 128 and 256 tokens (the paper's chunk ablation): several chunks per workgroup ----
@pytest.mark.parametrize("batch,heads,seq,dim,chunk,layout", [
    (1, 2, 2048, 128, 64, "bhsd"),       # four full blocks of 512 tokens per sequence
    (2, 3, 1600, 128, 128, "bshd"),      # last block holds one chunk only; token-major storage, two batches
    (1, 2, 3000, 128, 256, "bhsd"),      # 11 whole chunks (the last block holds one) + a tail chunk of 184 tokens
    (1, 3, 1000, 64, 64, "bhsd"),        # head_dim 64; 15 whole chunks + a tail of 40
    (1, 2, 833, 64, 256, "bhsd"),        # head_dim 64; 3 whole chunks + an odd tail of 65
    (1, 1, 64, 128, 64, "bhsd"),         # exactly one chunk
    (1, 2, 191, 128, 128, "bhsd"),       # one whole chunk + a tail of 63
])
def test_match_small_chunk_kernel_bf16(batch, heads, seq, dim, chunk, layout):
    """The kernel that packs 512 tokens (8, 4 or 2 chunks, the last one possibly ragged) into a workgroup."""
    _say(f"match small chunks B={batch} H={heads} S={seq} D={dim} c={chunk} {layout}")
    Ks = [kv_host(41 + b, heads, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)[0] for b in range(batch)]
    K = torch.cat(Ks, dim=0)
    if seq >= 200:
        K[0, 0, 6] = 0                                         # a zero A key and a zero B key
        K[0, 0, 9] = 0
        K[0, -1, chunk:chunk + chunk // 2] = K[0, -1, chunk + 1]   # equal maxima: the lowest index must win
    if layout == "bshd":
        Kd = K.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    else:
        Kd = K.to(DEV)
    dst, score = ckv.match(Kd, chunk)
    torch.cuda.synchronize()
    for b in range(batch):
        for h in range(heads):
            check_match(f64(K[b, h]), chunk, i64(dst[b, h]), f64(score[b, h]), f"b{b} h{h}")
    if seq >= 200:                                             # the tie: every source of that stretch picks its chunk's first B token
        g0 = chunk
        srcs = [t for t in range(g0, g0 + chunk // 2, 2)]
        got = i64(dst[0, heads - 1])[[t // 2 for t in srcs]]
        assert np.all(got == g0 + 1), got


@pytest.mark.parametrize("chunk", [64, 128, 256])
@pytest.mark.parametrize("whole", [512, 768])            # the tail opens a workgroup's block, or follows whole chunks in it
def test_match_small_chunks_ragged_tails_bf16(whole, chunk):
    """Tails of one token (no edge), one pair, around one tile of 32 rows and one short of a chunk."""
    _say(f"match small chunks, tails after {whole}, c={chunk}")
    for tail in sorted({1, 2, 3, 62, 63, min(64, chunk - 2), min(65, chunk - 1), chunk - 1}):
        K, _, _ = kv_host(51 + tail, 2, whole + tail, 128, "bf16", alpha=0.9, n_outlier=4)
        dst, score = ckv.match(K.to(DEV), chunk)
        torch.cuda.synchronize()
        for h in range(2):
            check_match(f64(K[0, h]), chunk, i64(dst[0, h]), f64(score[0, h]), f"tail {tail} h{h}")


# ---- the persistent kernel for whole 1024- or 2048-token chunks of 128-dim bf16 keys --------------
@pytest.mark.parametrize("batch,heads,seq,layout,chunk", [
    (1, 5, 1024, "bhsd", 1024),        # one chunk per sequence: every item starts a new sequence
    (1, 3, 7168, "bhsd", 1024),        # 21 items, one per workgroup
    (2, 3, 5120, "bshd", 1024),        # token-major storage: row stride heads*dim, separate batch stride
    (2, 5, 33792, "bhsd", 1024),       # 330 items on 256 workgroups: ranges of one and of two items
    (1, 3, 2048, "bhsd", 2048),        # two A blocks per chunk, one chunk per sequence
    (2, 2, 10240, "bshd", 2048),       # 40 items; token-major storage
    (1, 7, 40960, "bhsd", 2048),       # 280 items on 256 workgroups: a chunk's two blocks on different workgroups
])
def test_match_streaming_kernel_bf16(batch, heads, seq, layout, chunk):
    _say(f"match streaming B={batch} H={heads} S={seq} {layout} c={chunk}")
    Ks = [kv_host(31 + b, heads, seq, 128, "bf16", alpha=0.9, n_outlier=4)[0] for b in range(batch)]
    K = torch.cat(Ks, dim=0)                                   # [B, H, S, D]
    if seq == 1024:
        K[0, 1, 17] = 0                                        # a zero A key and a zero B key
        K[0, 1, 400:404] = 0
    if layout == "bshd":
        K = K.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
        assert not K.is_contiguous()
    else:
        K = K.to(DEV)
    dst, score = ckv.match(K, chunk)
    torch.cuda.synchronize()
    for b in range(batch):
        for h in range(heads):
            check_match(f64(K[b, h]), chunk, i64(dst[b, h]), f64(score[b, h]), f"b{b}h{h}")


@pytest.mark.parametrize("tail", [1, 2, 511, 513, 1023])
def test_match_streaming_kernel_with_ragged_tails_bf16(tail):
    """From 1024 whole chunks on they take the streaming kernel and the tails a launch of their own: the bits
    of the whole chunks by themselves and of the tails by themselves, on both kernels' own routes."""
    heads, whole, chunk = 64, 16, 1024
    _say(f"match ragged H={heads} S={whole}*{chunk}+{tail}")
    gen = torch.Generator(device=DEV).manual_seed(tail)
    K = torch.randn((1, heads, whole * chunk + tail, 128), generator=gen, device=DEV).to(torch.bfloat16)
    dst, score = ckv.match(K, chunk)
    d0, s0 = ckv.match(K[:, :, :whole * chunk], chunk)
    d1, s1 = ckv.match(K[:, :, whole * chunk:], chunk)
    n = whole * chunk // 2
    assert torch.equal(dst[:, :, :n], d0) and torch.equal(score[:, :, :n], s0)
    assert torch.equal(dst[:, :, n:], torch.where(d1 < 0, d1, d1 + whole * chunk)) and torch.equal(score[:, :, n:], s1)


@pytest.mark.parametrize("chunk", [1024, 2048])
def test_match_streaming_kernel_takes_the_lowest_index_among_equal_maxima(chunk):
    """Exactly equal scores in different tiles, lane halves and accumulators: lowest B index wins."""
    _say(f"match streaming ties c={chunk}")
    rng = np.random.default_rng(77)
    K = torch.from_numpy(rng.standard_normal((1, 2, 4096, 128)).astype(np.float32)).to(torch.bfloat16)
    K[0, 1, 2048:4096] = K[0, 1, 2048]                         # identical keys: every source takes B row 0
    picks = [(0, 10, (37, 411)), (0, 300, (5, 4)), (0, 511, (480, 31)), (2048, 64, (96, 100)), (2048, 7, (3, 259))]
    for g0, a, (j1, j2) in picks:                               # two copies of an A key among the B keys
        K[0, 0, g0 + 2 * j1 + 1] = K[0, 0, g0 + 2 * a]
        K[0, 0, g0 + 2 * j2 + 1] = K[0, 0, g0 + 2 * a]
    K = K.to(DEV)
    dst, score = ckv.match(K, chunk)
    torch.cuda.synchronize()
    d0, d1 = i64(dst[0, 0]), i64(dst[0, 1])
    for g0, a, (j1, j2) in picks:
        assert d0[g0 // 2 + a] == g0 + 2 * min(j1, j2) + 1, (g0, a, j1, j2, d0[g0 // 2 + a])
    for g0 in range(2048, 4096, chunk):
        assert np.all(d1[g0 // 2:(g0 + chunk) // 2] == g0 + 1)
    for h in range(2):
        check_match(f64(K[0, h]), chunk, i64(dst[0, h]), f64(score[0, h]), f"ties h{h}")


@pytest.mark.parametrize("heads,seq,dim,chunk,rounds", [
    (2, 4096, 128, 1024, [1.0, 1.0]),
    (2, 3000, 128, 1024, [1.0, 0.5]),
    (1, 2047, 128, 256, [0.8, 0.6]),
    (1, 5000, 128, 2048, [0.3]),
    (2, 1536, 64, 512, [1.0]),
    (3, 700, 128, 64, [0.75, 0.75, 0.75]),
    (1, 130, 128, 2, [1.0]),
    (1, 1, 128, 16, [1.0]),
    (1, 9, 128, 8, [1.0]),
])
def test_compress_bf16_shapes(heads, seq, dim, chunk, rounds):
    _say(f"compress bf16 H={heads} S={seq} D={dim} c={chunk} rounds={rounds}")
    K, V, _ = kv_host(12, heads, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    fK, fV, fdeg, _ = _run_rounds_teacher_forced(K, V, chunk, rounds, "bf16 shapes")
    gK, gV, gdeg, gas = ckv.compress(K, V, chunk, rounds=rounds)
    torch.cuda.synchronize()
    assert torch.equal(gK, fK) and torch.equal(gV, fV) and torch.equal(gdeg, fdeg)
    for h in range(heads):
        a = i64(gas[0, h])
        assert np.array_equal(np.bincount(a, minlength=gK.shape[2]), i64(gdeg[0, h]))


def test_compress_config2_llama_layer_bf16():
    """8 KV heads x 32768 x 128 bf16, chunk 1024, retain 25% (rounds [1, 1])."""
    _say("compress config2")
    K, V, _ = kv_host(2, 8, 32768, 128, "bf16", alpha=0.9, n_outlier=4)
    K, V = K.to(DEV), V.to(DEV)
    pl = ckv.plan(ckv.layout_of(K), ckv.make_params(1024, 0.25))
    assert pl.round_r == [1.0, 1.0] and pl.out_seq == 8192
    fK, fV, fdeg, alt = _run_rounds_teacher_forced(K, V, 1024, pl.round_r, "config2")
    _say(f"config2: {alt} near-tie rows resolved differently")
    gK, gV, gdeg, gas = ckv.compress(K, V, 1024, retain_ratio=0.25)
    torch.cuda.synchronize()
    assert torch.equal(gK, fK) and torch.equal(gV, fV) and torch.equal(gdeg, fdeg)
    assert int(gdeg.sum()) == 8 * 32768


# ---- rounds of small chunks: one launch of 256 tokens per workgroup -----------------------------
def _timed(call):
    """call(), and the names of the kernels that made it."""
    ckv.timing_reset()
    ckv.timing_enable(True)
    got = call()
    torch.cuda.synchronize()
    ckv.timing_enable(False)
    return got, set(ckv.timing_read())


def _by_separate_kernels(K, V, deg, chunk, r, n_sink=0, n_recent=0):
    """One round with the top-r inside every chunk, by the match kernel and merge_kernel: every chunk as a sequence of its
    own, the only and short chunk of 2048 tokens in it, which no kernel takes for a small one."""
    B, H, S, D = K.shape
    lo, hi = (n_sink, S - n_recent) if S > n_sink + n_recent else (0, 0)
    deg = torch.ones((B, H, S), dtype=torch.int32, device=K.device) if deg is None else deg
    parts = []                                   # K', V', deg', the tokens' places, by part of the sequence

    def copied(a, b):
        if b > a:
            parts.append((K[:, :, a:b], V[:, :, a:b], deg[:, :, a:b],
                          torch.arange(b - a, dtype=torch.int32, device=K.device).expand(B, H, b - a)))

    def clustered(a, b, size):
        n = (b - a) // size
        if n == 0:
            return
        shape = (B, H * n, size)
        k, v, d = (x[:, :, a:b].reshape(shape + x.shape[3:]).contiguous() for x in (K, V, deg))
        (k, v, d, to), names = _timed(lambda: ckv.compress(k, v, 2048, rounds=[r], deg=d))
        assert not any(x.startswith("round") for x in names) and any(x.startswith("merge") for x in names), names
        left = k.shape[2]
        to = to.view(B, H, n, size) + left * torch.arange(n, dtype=torch.int32, device=K.device).view(1, 1, n, 1)
        parts.append((k.reshape(B, H, n * left, D), v.reshape(B, H, n * left, D), d.reshape(B, H, n * left), to.reshape(B, H, n * size)))

    copied(0, lo if hi > lo else S)
    if hi > lo:
        whole = lo + (hi - lo) // chunk * chunk
        clustered(lo, whole, chunk)
        clustered(whole, hi, hi - whole or 1)
        copied(hi, S)
    at, places = 0, []
    for k, _, _, to in parts:
        places.append(to + at)
        at += k.shape[2]
    return [torch.cat([p[i] for p in parts], dim=2) for i in range(3)] + [torch.cat(places, dim=2)]


def _same(got, want, what):
    for n, a, e in zip(["K'", "V'", "deg'", "assign"], got, want):
        assert torch.equal(a, e), f"{n} differs from {what}"


@pytest.mark.parametrize("chunk", [64, 128, 256])
@pytest.mark.parametrize("seq,dim,r,big_degrees,n_sink,n_recent", [
    (256, 128, 0.8, False, 0, 0),
    (257, 128, 1.0, False, 0, 0),            # a one-token chunk in a block of its own
    (512 + 65, 64, 0.5, False, 0, 0),        # chunk 64: a one-token chunk behind a whole one
    (768 + 255, 128, 0.3, True, 0, 0),       # the longest tail; weights beyond the packed route's 256
    (2 * 256 + 130, 64, 1.0, True, 16, 64),
    (80 + 3, 128, 1.0, False, 16, 64),       # three tokens to cluster
    (300, 64, 0.0, False, 0, 9),             # nothing merged
])
def test_rounds_of_small_chunks_in_one_launch(seq, dim, r, big_degrees, n_sink, n_recent, chunk):
    """Against the oracle, and bit for bit against the separate match and merge kernels."""
    _say(f"round in one launch S={seq} D={dim} c={chunk} r={r} n1={n_sink} n2={n_recent}")
    K, V, _ = kv_host(41, 4, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.reshape(2, 2, seq, dim).to(DEV), V.reshape(2, 2, seq, dim).to(DEV)
    deg = np.random.default_rng(seq).integers(1, 9, (2, 2, seq))
    if big_degrees:
        deg[1, 0, seq // 2:] *= 999
    deg = torch.from_numpy(deg.astype(np.int32)).to(DEV)
    got, names = _timed(lambda: ckv.compress(K, V, chunk, rounds=[r], deg=deg, n_sink=n_sink, n_recent=n_recent))
    assert names == {"round_bf16"}
    for b in range(2):
        for h in range(2):
            check_round_with_edges(f64(K[b, h]), f64(V[b, h]), i64(deg[b, h]), chunk, r, "bf16", n_sink, n_recent,
                                   f64(got[0][b, h]), f64(got[1][b, h]), i64(got[2][b, h]), i64(got[3][b, h]),
                                   what=f"b{b} h{h}")
    _same(got, _by_separate_kernels(K, V, deg, chunk, r, n_sink, n_recent), "the separate kernels")


@pytest.mark.parametrize("chunk,dim", [(512, 128), (512, 64), (1024, 64)])
@pytest.mark.parametrize("whole,tail,r,directions", [
    (1, 0, 0.8, 0),
    (2, 1, 1.0, 0),              # a one-token chunk
    (1, 509, 0.3, 0),            # the first rows of the last tile masked
    (0, 33, 1.0, 0),             # a short chunk alone
    (1, 300, 0.6, 5),            # keys of five directions: lists far beyond eight members, scores equal at the cut
    (2, 0, 1.0, 12),
])
def test_rounds_of_one_chunk_per_workgroup(whole, tail, r, directions, chunk, dim):
    """Chunks of 512 and 1024 tokens in one launch, against the oracle, and bit for bit against the separate kernels."""
    from synth.kv import prototype_kv_host
    seq = whole * chunk + tail
    _say(f"round in one launch S={seq} D={dim} c={chunk} r={r} directions={directions}")
    if directions:
        K, V = prototype_kv_host(47, 2, seq, dim, "bf16", directions)
    else:
        K, V, _ = kv_host(47, 2, seq, dim, "bf16", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    deg = torch.from_numpy(np.random.default_rng(seq).integers(1, 9, (1, 2, seq)).astype(np.int32)).to(DEV)
    got, names = _timed(lambda: ckv.compress(K, V, chunk, rounds=[r], deg=deg))
    assert names == {"round_bf16"}
    for h in range(2):
        check_round(f64(K[0, h]), f64(V[0, h]), i64(deg[0, h]), chunk, r, "bf16", f64(got[0][0, h]), f64(got[1][0, h]),
                    i64(got[2][0, h]), i64(got[3][0, h]), what=f"h{h}")
    _same(got, _by_separate_kernels(K, V, deg, chunk, r), "the separate kernels")


@pytest.mark.parametrize("route", [None, "full_rounds", "defer_always"])
@pytest.mark.parametrize("dtype,seq,dim,chunk,rounds", [
    ("bf16", 1, 128, 64, [1.0, 1.0]),                    # a token alone in every round
    ("bf16", 4099, 128, 2, [1.0, 1.0, 0.5]),             # the smallest chunk, a one-token tail
    ("bf16", 3001, 64, 64, [1.0, 1.0, 1.0, 0.6]),        # eight original tokens to an input token of the last round
    ("bf16", 2500, 128, 384, [1.0, 0.7]),
    ("bf16", 2561, 128, 512, [1.0, 1.0]),                # tails of one token and of a half chunk
    ("bf16", 1700, 128, 128, [1.0, 1.0]),
    ("bf16", 3333, 64, 256, [1.0, 1.0, 0.4]),
    ("bf16", 3100, 64, 1024, [1.0, 1.0]),
    ("bf16", 5121, 128, 1024, [1.0, 0.8, 1.0]),          # after a round below 1 the chunks no longer nest
    ("bf16", 9000, 128, 2048, [1.0, 1.0, 0.3]),
    ("f32", 777, 64, 128, [1.0, 1.0, 0.5]),
    ("f32", 1200, 32, 300, [0.9, 1.0]),
])
def test_assignments_of_several_rounds_are_the_rounds_maps_chained(dtype, seq, dim, chunk, rounds, route):
    _say(f"chained maps {dtype} S={seq} D={dim} c={chunk} rounds={rounds} route={route}")
    K, V, _ = kv_host(67, 2, seq, dim, dtype, alpha=0.9)
    K, V = K.to(DEV), V.to(DEV)
    got = _compress(route, K, V, chunk, rounds=rounds)
    k, v, deg, to = K, V, None, None
    for r in rounds:
        k, v, deg, m = ckv.compress(k, v, chunk, rounds=[r], deg=deg)
        to = m if to is None else torch.gather(m, 2, to.long())
    torch.cuda.synchronize()
    for n, a, e in zip(["K'", "V'", "deg'", "assign"], got, (k, v, deg, to)):
        assert torch.equal(a, e), f"{n} differs from the chained rounds"


@pytest.mark.parametrize("dtype,seq,dim,chunk,rounds,n_sink,n_recent", [
    ("bf16", 2049, 128, 256, [1.0, 1.0], 0, 0),
    ("bf16", 5000, 128, 384, [1.0, 1.0], 4, 9),
    ("bf16", 3500, 64, 512, [1.0, 0.7, 1.0], 0, 0),      # the second round ranks the whole sequence
    ("bf16", 70001, 128, 1024, [1.0, 0.4], 0, 0),
    ("f32", 1000, 64, 64, [1.0], 0, 0),
])
def test_ranking_over_the_whole_sequence_where_every_edge_is_merged(dtype, seq, dim, chunk, rounds, n_sink, n_recent):
    """A round at r = 1 gives the bits of every chunk clustered by itself, alone and among others; rounds below 1 are
    ranked over the whole sequence in either chain."""
    _say(f"whole-sequence ranking at r = 1 {dtype} S={seq} D={dim} c={chunk} rounds={rounds}")
    K, V, _ = kv_host(71, 2, seq, dim, dtype, alpha=0.9)
    K, V = K.to(DEV), V.to(DEV)
    got = ckv.compress(K, V, chunk, rounds=rounds, n_sink=n_sink, n_recent=n_recent, scope="head")
    k, v, deg, to = K, V, None, None
    for r in rounds:
        if r == 1.0:
            k, v, deg, m = _by_separate_kernels(k, v, deg, chunk, r, n_sink, n_recent)
        else:
            k, v, deg, m = ckv.compress(k, v, chunk, rounds=[r], deg=deg, n_sink=n_sink, n_recent=n_recent, scope="head")
        to = m if to is None else torch.gather(m, 2, to.long())
    torch.cuda.synchronize()
    for n, a, e in zip(["K'", "V'", "deg'", "assign"], got, (k, v, deg, to)):
        assert torch.equal(a, e), f"{n} differs from the chained rounds"


@pytest.mark.parametrize("dtype,dim,chunk", [("bf16", 128, 384), ("bf16", 128, 1024), ("bf16", 64, 2048), ("f32", 64, 1024),
                                             ("bf16", 128, 2)])
@pytest.mark.parametrize("whole,tail,r,directions", [
    (2, 0, 0.8, 0),
    (1, 333, 0.5, 0),
    (1, 0, 0.999, 0),            # all edges of a long chunk but one
    (2, 5, 0.002, 0),            # one or two, none in the tail
    (1, 77, 0.6, 3),             # keys of three directions: most scores equal, whichever cut is taken
])
def test_the_best_edges_of_a_chunk_are_merged_and_the_earliest_of_equal_ones(whole, tail, r, directions, dtype, dim, chunk):
    """The separate merge kernel's selection against the scores of the match kernel, exactly, and the round against the
    oracle."""
    from synth.kv import prototype_kv_host
    seq = whole * chunk + tail
    _say(f"selection {dtype} S={seq} D={dim} c={chunk} r={r} directions={directions}")
    if directions:
        K, V = prototype_kv_host(53, 2, seq, dim, dtype, directions)
    else:
        K, V, _ = kv_host(53, 2, seq, dim, dtype, alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    deg = torch.from_numpy(np.random.default_rng(seq).integers(1, 9, (1, 2, seq)).astype(np.int32)).to(DEV)
    dst, score = ckv.match(K, chunk)
    got = ckv.compress(K, V, chunk, rounds=[r], deg=deg)
    torch.cuda.synchronize()
    for h in range(2):
        to, first = i64(got[3][0, h]), 0
        for lo in range(0, seq, chunk):
            n = min(chunk, seq - lo)
            n_src, n_edges = (n + 1) // 2, (n + 1) // 2 if n > 1 else 0
            at, sc = i64(dst[0, h])[first:first + n_src], score[0, h][first:first + n_src].cpu().numpy()
            first += n_src
            m = int(np.floor(float(np.float32(r)) * n_edges + 1e-9))
            want = np.zeros(n_src, dtype=bool)
            want[np.argsort(-sc, kind="stable")[:m]] = True
            merged = np.array([j >= 0 and to[lo + 2 * i] == to[j] for i, j in enumerate(at)])
            assert np.array_equal(merged, want), f"h{h} chunk at {lo}: {np.flatnonzero(merged != want)[:8]}"
        check_round(f64(K[0, h]), f64(V[0, h]), i64(deg[0, h]), chunk, r, dtype, f64(got[0][0, h]), f64(got[1][0, h]),
                    i64(got[2][0, h]), i64(got[3][0, h]), what=f"h{h}")


@pytest.mark.parametrize("chunk", [64, 128, 256])
@pytest.mark.parametrize("seq,dim,r,n_sink,n_recent", [
    (256, 64, 0.5, 0, 0),
    (257, 128, 1.0, 0, 0),                   # a one-token chunk
    (3 * 256 + 255, 16, 0.8, 0, 0),          # the longest tail, the narrowest rows
    (512 + 2, 32, 1.0, 16, 64),
    (80 + 1, 128, 1.0, 16, 64),              # one token to cluster
])
def test_fp32_rounds_of_small_chunks_in_one_launch(seq, dim, r, n_sink, n_recent, chunk):
    """As above, for fp32 caches."""
    _say(f"fp32 round in one launch S={seq} D={dim} c={chunk} r={r} n1={n_sink} n2={n_recent}")
    K, V, _ = kv_host(43, 3, seq, dim, "f32", alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    deg = torch.from_numpy(np.random.default_rng(seq).integers(1, 400, (1, 3, seq)).astype(np.int32)).to(DEV)
    got, names = _timed(lambda: ckv.compress(K, V, chunk, rounds=[r], deg=deg, n_sink=n_sink, n_recent=n_recent))
    assert names == {"round_f32"}
    for h in range(3):
        check_round_with_edges(f64(K[0, h]), f64(V[0, h]), i64(deg[0, h]), chunk, r, "f32", n_sink, n_recent, f64(got[0][0, h]),
                               f64(got[1][0, h]), i64(got[2][0, h]), i64(got[3][0, h]), what=f"h{h}")
    _same(got, _by_separate_kernels(K, V, deg, chunk, r, n_sink, n_recent), "the separate kernels")


@pytest.mark.parametrize("dtype,dim,chunk,r", [
    ("bf16", 128, 64, 1.0), ("bf16", 64, 64, 0.5), ("bf16", 128, 128, 0.7), ("bf16", 64, 256, 0.5), ("bf16", 64, 512, 0.6),
    ("bf16", 128, 1024, 0.5), ("f32", 64, 64, 0.5), ("f32", 128, 128, 1.0), ("f32", 32, 256, 0.3), ("f32", 64, 512, 0.5),
])
@pytest.mark.parametrize("rows", ["a source", "a destination", "every source", "every row"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), 3e30])
def test_keys_without_a_cosine_stay_inside_their_chunk(dtype, dim, chunk, r, rows, value):
    """A key that is not finite, or whose norm is not: every other chunk as without it, and in its own chunk as many edges
    merged and every token accounted for."""
    _say(f"keys without a cosine {dtype} D={dim} c={chunk} r={r}: {rows} {value}")
    seq = 3 * chunk + chunk // 2 + 1
    K, V, _ = kv_host(91, 2, seq, dim, dtype, alpha=0.9)
    K, V = K.to(DEV), V.to(DEV)
    bad = {"a source": slice(chunk + 6, chunk + 7), "a destination": slice(chunk + 5, chunk + 6),
           "every source": slice(chunk, 2 * chunk, 2), "every row": slice(chunk, 2 * chunk)}[rows]
    P = K.clone()
    P[0, 0, bad, 3] = value
    want, got = (ckv.compress(k, V, chunk, rounds=[r]) for k in (K, P))
    torch.cuda.synchronize()
    kept = chunk - int(np.floor(float(np.float32(r)) * (chunk // 2) + 1e-9))       # rows a whole chunk leaves
    outside = [slice(0, kept), slice(2 * kept, None)]
    for n, a, e in zip(["K'", "V'", "deg'"], got, want):
        assert torch.equal(a[0, 1], e[0, 1]), n
        for x in outside:
            assert torch.equal(a[0, 0, x], e[0, 0, x]), n
    to = i64(got[3][0, 0])
    assert torch.equal(got[3][0, 1], want[3][0, 1])
    assert np.array_equal(to[:chunk], i64(want[3][0, 0])[:chunk]) and np.array_equal(to[2 * chunk:], i64(want[3][0, 0])[2 * chunk:])
    mine = to[chunk:2 * chunk]
    assert mine.min() >= kept and mine.max() < 2 * kept
    assert np.array_equal(np.bincount(mine - kept, minlength=kept), i64(got[2][0, 0])[kept:2 * kept])
    ref = np.zeros((kept, dim))
    np.add.at(ref, mine - kept, f64(V[0, 0])[chunk:2 * chunk])
    assert_rows_close(f64(got[1][0, 0])[kept:2 * kept], ref / np.bincount(mine - kept)[:, None], TOL[dtype] if dtype == "f32" else 2.0 ** -8,
                      "V' of the chunk")


# ---- attention sinks and recent tokens (Sec. 5.2 / 5.3) ----------------------------------------
@pytest.mark.parametrize("dtype,heads,seq,dim,chunk,rounds,n_sink,n_recent", [
    ("bf16", 2, 4096 + 80, 128, 1024, [1.0, 1.0], 16, 64),
    ("bf16", 2, 3001, 128, 256, [1.0, 0.6], 4, 0),
    ("bf16", 1, 2500, 128, 512, [0.7], 0, 100),
    ("bf16", 2, 700, 64, 64, [1.0, 1.0, 1.0], 3, 33),
    ("f32", 1, 1024, 64, 64, [1.0, 0.5], 4, 32),
    ("bf16", 1, 300, 128, 64, [1.0, 1.0, 1.0, 1.0], 100, 150),   # the middle dries up: 50 -> 25 -> 12 -> 6 -> 3
    ("bf16", 2, 90, 128, 16, [1.0], 40, 50),                      # nothing between sinks and recents
    ("bf16", 1, 50, 128, 16, [1.0], 40, 50),                      # shorter than n1 + n2
])
def test_compress_with_sinks_and_recents(dtype, heads, seq, dim, chunk, rounds, n_sink, n_recent):
    _say(f"sinks/recents {dtype} H={heads} S={seq} D={dim} c={chunk} rounds={rounds} n1={n_sink} n2={n_recent}")
    K, V, _ = kv_host(31, heads, seq, dim, dtype, alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    curK, curV, curdeg, maps = K, V, None, []
    for j, r in enumerate(rounds):
        gK, gV, gdeg, gas = ckv.compress(curK, curV, chunk, rounds=[r], deg=curdeg, n_sink=n_sink, n_recent=n_recent)
        torch.cuda.synchronize()
        for h in range(heads):
            d_in = np.ones(curK.shape[2], dtype=np.int64) if curdeg is None else i64(curdeg[0, h])
            check_round_with_edges(f64(curK[0, h]), f64(curV[0, h]), d_in, chunk, r, dtype, n_sink, n_recent,
                                   f64(gK[0, h]), f64(gV[0, h]), i64(gdeg[0, h]), i64(gas[0, h]),
                                   what=f"sinks/recents round {j} h{h}")
        curK, curV, curdeg = gK, gV, gdeg
        maps.append(gas.to(torch.int64))
    gK, gV, gdeg, gas = ckv.compress(K, V, chunk, rounds=rounds, n_sink=n_sink, n_recent=n_recent)
    torch.cuda.synchronize()
    assert list(gK.shape) == [1, heads, oracle.round_lengths(seq, chunk, rounds, n_sink, n_recent)[-1], dim]
    assert torch.equal(gK, curK) and torch.equal(gV, curV) and torch.equal(gdeg, curdeg)
    comp = maps[0]
    for m in maps[1:]:
        comp = torch.gather(m, 2, comp)
    assert torch.equal(gas.to(torch.int64), comp)
    assert int(gdeg.sum()) == heads * seq


def test_sinks_beside_as_many_chunks_as_one_launch_takes():
    """2^24 - 16 workgroups of 256 threads merge; with those that copy 80 sinks per sequence they would pass the
    2^32 threads of a launch.  Same bits as the two halves of the batch."""
    B, H, n_sink, dim = 4, 4, 80, 16
    seq = n_sink + 2 * ((1 << 20) - 1)
    _say(f"{B * H * ((1 << 20) - 1)} chunks of two tokens, {n_sink} sinks")
    gen = torch.Generator(device=DEV).manual_seed(3)
    K, V = (torch.randn((B, H, seq, dim), generator=gen, device=DEV) for _ in range(2))
    call = lambda k, v: ckv.compress(k, v, 2, rounds=[1.0], n_sink=n_sink, want_assign=False)[:3]
    whole = call(K, V)
    for part in (slice(0, 2), slice(2, 4)):
        for got, want in zip(whole, call(K[part], V[part])):
            assert torch.equal(got[part], want)
    assert torch.equal(whole[0][:, :, :n_sink], K[:, :, :n_sink]) and torch.equal(whole[1][:, :, :n_sink], V[:, :, :n_sink])
    assert bool((whole[2][:, :, :n_sink] == 1).all()) and int(whole[2].sum()) == B * H * seq


def test_sinks_and_recents_with_strided_layout_and_retain_ratio():
    """[B,S,H,D] input, padded output, incoming degrees, retain_ratio schedule with n1=16, n2=64:
    the whole call against the oracle's compress (teacher-forcing is covered above)."""
    _say("sinks/recents bshd")
    B, H, S, D, c, n1, n2 = 2, 2, 2128, 128, 256, 16, 64
    K0, V0, _ = kv_host(32, B * H, S, D, "bf16", alpha=0.9, n_outlier=4)
    rng = np.random.default_rng(5)
    Kb = K0.reshape(B, H, S, D).permute(0, 2, 1, 3).contiguous().to(DEV)      # [B,S,H,D] storage
    Vb = V0.reshape(B, H, S, D).permute(0, 2, 1, 3).contiguous().to(DEV)
    K, V = Kb.permute(0, 2, 1, 3), Vb.permute(0, 2, 1, 3)                     # [B,H,S,D] views
    deg = torch.from_numpy(rng.integers(1, 4, size=(B, H, S)).astype(np.int32)).to(DEV)
    out_len = oracle.round_lengths(S, c, oracle.direct_schedule(0.375), n1, n2)[-1]
    pad = 40
    oK = torch.zeros((B, H, out_len + pad, D), dtype=torch.bfloat16, device=DEV)
    oV = torch.zeros_like(oK)
    odeg = torch.zeros((B, H, out_len + pad), dtype=torch.int32, device=DEV)
    oas = torch.empty((B, H, S), dtype=torch.int32, device=DEV)
    ckv.compress(K, V, c, retain_ratio=0.375, deg=deg, out=(oK, oV, odeg, oas), n_sink=n1, n_recent=n2)
    torch.cuda.synchronize()
    assert not bool(oK[:, :, out_len:].any()) and not bool(odeg[:, :, out_len:].any())
    direct = chained = flagged = 0
    for b in range(B):
        for h in range(H):
            ref = oracle.compress(f64(K[b, h]), f64(V[b, h]), c, oracle.direct_schedule(0.375), "bf16",
                                  deg=i64(deg[b, h]), n_sink=n1, n_recent=n2)
            if np.array_equal(i64(oas[b, h]), ref["assign"]):
                direct += 1
                assert np.array_equal(i64(odeg[b, h, :out_len]), ref["deg"])
                assert_rows_close(f64(oK[b, h, :out_len]), ref["K"], TOL["bf16"], f"b{b}h{h} K'")
                assert_rows_close(f64(oV[b, h, :out_len]), ref["V"], TOL["bf16"], f"b{b}h{h} V'")
                continue
            # a near-tie somewhere sent this sequence down another (valid) path: hold it to the oracle round
            # by round instead (each round on the GPU's own previous output), and the one call to the chained rounds
            curK, curV, curdeg = K[b:b + 1, h:h + 1].contiguous(), V[b:b + 1, h:h + 1].contiguous(), deg[b:b + 1, h:h + 1].contiguous()
            maps = []
            for j, r in enumerate(oracle.direct_schedule(0.375)):
                gK, gV, gdeg, gas = ckv.compress(curK, curV, c, rounds=[r], deg=curdeg, n_sink=n1, n_recent=n2)
                torch.cuda.synchronize()
                n_alt = check_round_with_edges(f64(curK[0, 0]), f64(curV[0, 0]), i64(curdeg[0, 0]), c, r, "bf16", n1, n2,
                                               f64(gK[0, 0]), f64(gV[0, 0]), i64(gdeg[0, 0]), i64(gas[0, 0]),
                                               what=f"b{b}h{h} round {j}")
                flagged += n_alt
                curK, curV, curdeg = gK, gV, gdeg
                maps.append(gas[0, 0].to(torch.int64))
            assert torch.equal(oK[b, h, :out_len], curK[0, 0]) and torch.equal(oV[b, h, :out_len], curV[0, 0])
            assert torch.equal(odeg[b, h, :out_len], curdeg[0, 0])
            comp = maps[0]
            for m in maps[1:]:
                comp = m[comp]
            assert torch.equal(oas[b, h].to(torch.int64), comp)
            chained += 1
    assert direct + chained == B * H and direct >= 1, f"{direct} sequences compared in one piece, {chained} round by round"
    assert chained == 0 or flagged >= 1      # a sequence only leaves the direct path through a flagged near-tie
    assert int(odeg.sum()) == int(deg.sum())


# ---- top-r over all chunks of a sequence (the other reading of Sec. 5.2-5.3) --------------------
@pytest.mark.parametrize("dtype,heads,seq,dim,chunk,rounds,n_sink,n_recent", [
    ("bf16", 2, 8192, 128, 1024, [0.5], 0, 0),
    ("bf16", 2, 4096 + 80, 128, 256, [0.8, 0.6], 16, 64),
    ("bf16", 1, 3001, 128, 512, [0.3, 0.9], 0, 0),                # ragged tail chunk, odd length
    ("bf16", 2, 1000, 64, 16, [0.5, 0.5], 4, 0),                  # many small chunks: a thread per chunk
    ("bf16", 1, 4097, 128, 2, [0.25], 0, 0),                      # chunk 2: one edge per chunk, one-token tail
    ("f32", 1, 1024, 64, 64, [0.7, 0.2], 0, 8),
    ("bf16", 2, 2048, 128, 256, [1.0, 0.0], 0, 0),                # all edges / no edge
    ("bf16", 1, 70000, 128, 2048, [0.45], 0, 0),                  # several scan tiles' worth of edges
])
def test_compress_with_selection_over_the_whole_sequence(dtype, heads, seq, dim, chunk, rounds, n_sink, n_recent):
    _say(f"scope=head {dtype} H={heads} S={seq} D={dim} c={chunk} rounds={rounds} n1={n_sink} n2={n_recent}")
    K, V, _ = kv_host(41, heads, seq, dim, dtype, alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    curK, curV, curdeg, maps, alt = K, V, None, [], 0
    for j, r in enumerate(rounds):
        gK, gV, gdeg, gas = ckv.compress(curK, curV, chunk, rounds=[r], deg=curdeg, n_sink=n_sink, n_recent=n_recent,
                                         scope="head")
        torch.cuda.synchronize()
        for h in range(heads):
            d_in = np.ones(curK.shape[2], dtype=np.int64) if curdeg is None else i64(curdeg[0, h])
            alt += check_round_with_edges(f64(curK[0, h]), f64(curV[0, h]), d_in, chunk, r, dtype, n_sink, n_recent,
                                          f64(gK[0, h]), f64(gV[0, h]), i64(gdeg[0, h]), i64(gas[0, h]),
                                          what=f"scope=head round {j} h{h}", scope="head")
        curK, curV, curdeg = gK, gV, gdeg
        maps.append(gas.to(torch.int64))
    _say(f"  {alt} edges inside the near-tie band resolved differently")
    gK, gV, gdeg, gas = ckv.compress(K, V, chunk, rounds=rounds, n_sink=n_sink, n_recent=n_recent, scope="head")
    torch.cuda.synchronize()
    assert gK.shape[2] == oracle.round_lengths(seq, chunk, rounds, n_sink, n_recent, scope="head")[-1]
    assert torch.equal(gK, curK) and torch.equal(gV, curV) and torch.equal(gdeg, curdeg)
    comp = maps[0]
    for m in maps[1:]:
        comp = torch.gather(m, 2, comp)
    assert torch.equal(gas.to(torch.int64), comp)
    assert int(gdeg.sum()) == heads * seq


def test_whole_sequence_selection_ties_across_identical_chunks():
    """Identical chunks give exactly equal scores in every chunk: the quota of edges ON the cut
    goes to the lowest positions, so the first chunks merge one edge more than the last."""
    _say("scope=head exact ties")
    base, _, _ = kv_host(43, 1, 64, 128, "bf16", alpha=0.9, n_outlier=4)
    K = base.repeat(1, 1, 8, 1).to(DEV)                      # 8 identical chunks of 64
    V = K.clone()
    gK, gV, gdeg, gas = ckv.compress(K, V, 64, rounds=[0.3], scope="head")     # floor(0.3 * 256) = 76 = 9*8 + 4
    torch.cuda.synchronize()
    a = i64(gas[0, 0])
    merged_per_chunk = [64 - len(np.unique(a[g * 64:(g + 1) * 64])) for g in range(8)]
    assert merged_per_chunk == [10, 10, 10, 10, 9, 9, 9, 9]
    check_round_with_edges(f64(K[0, 0]), f64(V[0, 0]), np.ones(512, dtype=np.int64), 64, 0.3, "bf16", 0, 0,
                           f64(gK[0, 0]), f64(gV[0, 0]), i64(gdeg[0, 0]), a, what="ties", scope="head")


# ---- layouts, degrees, degenerate inputs ------------------------------------------------------
@pytest.mark.parametrize("edges,chunk,r,opposed", [
    (8191, 128, 0.3, False),      # one edge less than the scores of a workgroup's step, chunks of 64 sources
    (8192, 128, 0.5, False),
    (8193, 64, 0.9, False),       # one more; chunks of 32 sources, eight at a time
    (16400, 130, 0.01, False),    # chunks of 65 sources: one more than a wave
    (9000, 1026, 0.7, False),     # 513 sources: one more than the scores of a wave's step
    (9000, 256, 0.4, True),       # every similarity below zero
])
def test_whole_sequence_selection_merges_the_best_edges_exactly(edges, chunk, r, opposed):
    """Integer work on the scores ckv_match gives: the number of edges merged in every chunk is exact."""
    _say(f"scope=head counts edges={edges} c={chunk} r={r} opposed={opposed}")
    seq = 2 * edges
    K, V, _ = kv_host(47, 2, seq, 64, "bf16", alpha=0.9, n_outlier=0)
    if opposed:
        K = K.abs()
        K[:, :, 1::2] *= -1
    K, V = K.to(DEV), V.to(DEV)
    _, score = ckv.match(K, chunk)
    _, _, _, gas = ckv.compress(K, V, chunk, rounds=[r], scope="head")
    torch.cuda.synchronize()
    for h in range(2):
        sc = score.view(2, edges)[h].cpu().numpy()
        assert not opposed or (sc < 0).all()
        kept = np.zeros(edges, dtype=np.int64)
        kept[np.argsort(-sc, kind="stable")[:int(float(np.float32(r)) * edges + 1e-9)]] = 1
        want = [kept[i:i + chunk // 2].sum() for i in range(0, edges, chunk // 2)]
        a = i64(gas[0, h])
        assert [len(c) - len(np.unique(c)) for c in (a[i:i + chunk] for i in range(0, seq, chunk))] == want


def test_bshd_layout_and_padded_output():
    _say("compress strided layout")
    K, V, _ = kv_host(13, 2, 1024, 128, "bf16", n_outlier=4)
    # store as [B, S, H, D] and view as [B, H, S, D]
    Kb = K.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    Vb = V.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    ref = ckv.compress(K.to(DEV), V.to(DEV), 256, rounds=[0.5])
    K_out = torch.zeros((1, 800, 2, 128), dtype=torch.bfloat16, device=DEV).permute(0, 2, 1, 3)   # room to spare
    V_out = torch.zeros_like(K_out)
    deg_out = torch.zeros((1, 2, 800), dtype=torch.int32, device=DEV)
    got = ckv.compress(Kb, Vb, 256, rounds=[0.5], out=(K_out, V_out, deg_out, None))
    torch.cuda.synchronize()
    n = ref[0].shape[2]
    assert n == 768
    assert torch.equal(got[0][:, :, :n], ref[0]) and torch.equal(got[1][:, :, :n], ref[1])
    assert torch.equal(deg_out[:, :, :n], ref[2])
    assert float(K_out[:, :, n:].abs().sum()) == 0.0            # rows beyond out_seq untouched


def test_incoming_degrees_weight_the_merge():
    _say("compress with deg_in")
    K, V, _ = kv_host(14, 1, 512, 128, "bf16", n_outlier=4)
    K, V = K.to(DEV), V.to(DEV)
    deg = torch.from_numpy(np.random.default_rng(0).integers(1, 9, (1, 1, 512)).astype(np.int32)).to(DEV)
    _run_rounds_teacher_forced(K, V, 128, [0.75, 0.5], "deg_in", deg=deg)


@pytest.mark.parametrize("rounds", [[1.0, 1.0], [0.7, 0.6, 0.5]])
def test_bf16_centroids_are_bit_identical_to_the_oracle(rounds):
    """Stronger than the tolerance: the single rounding of S/n to bf16 (fp32 accumulation of exact
    products, correctly rounded quotient) lands on the oracle's fp64 -> bf16 value.  Round by round
    (the oracle is fed the GPU's input of that round), wherever the matching agrees, every element
    must match bit for bit, except where the fp32 sum itself lost the last bits of a quotient that
    lies within 1e-6 (relative) of a bf16 rounding boundary: a handful of elements per million,
    each one bf16 step away."""
    _say(f"bit-identity to the oracle, rounds={rounds}")
    K, V, _ = kv_host(71, 3, 8192, 128, "bf16", alpha=0.9, n_outlier=4)
    curK, curV, curdeg = K.to(DEV), V.to(DEV), None
    compared = off = 0
    for j, r in enumerate(rounds):
        gK, gV, gdeg, gas = ckv.compress(curK, curV, 512, rounds=[r], deg=curdeg)
        torch.cuda.synchronize()
        for h in range(3):
            d_in = np.ones(curK.shape[2], dtype=np.int64) if curdeg is None else i64(curdeg[0, h])
            ref = oracle.csm_round(f64(curK[0, h]), f64(curV[0, h]), d_in, 512, r, "bf16")
            if not np.array_equal(ref["assign"], i64(gas[0, h])):
                continue                              # a near-tie resolved differently: covered by the tests above
            assert np.array_equal(i64(gdeg[0, h]), ref["deg"])
            for got, want, exact in ((f64(gK[0, h]), ref["K"], ref["K_exact"]), (f64(gV[0, h]), ref["V"], ref["V_exact"])):
                for idx in np.argwhere(got != want):
                    g, w, x = got[tuple(idx)], want[tuple(idx)], exact[tuple(idx)]
                    boundary = 0.5 * (g + w)          # the two differ by one bf16 step: its midpoint
                    assert abs(g - w) <= 2.0 ** -7 * abs(w) and abs(x - boundary) <= 1e-6 * abs(x), (j, h, idx, g, w, x)
                    off += 1
            compared += 1
        curK, curV, curdeg = gK, gV, gdeg
    assert compared >= 2 * len(rounds) and off <= 6
    _say(f"  {off} elements sit on a rounding boundary to within fp32 accumulation error")


def test_large_incoming_degrees():
    """Degrees far above 256 (the limit of the packed-weight accumulation route) in some chunks and
    small ones in others, through full rounds and through a deferred pair."""
    _say("large degrees")
    heads, seq, chunk = 2, 3000, 256
    K, V, _ = kv_host(61, heads, seq, 128, "bf16", alpha=0.9, n_outlier=4)
    K, V = K.to(DEV), V.to(DEV)
    d = np.random.default_rng(9).integers(1, 4, (1, heads, seq))
    d[0, 0, 700:1400] = np.random.default_rng(10).integers(200, 70000, 700)          # some chunks with wide weights
    d[0, 1, 2990:] = 100000
    deg = torch.from_numpy(d.astype(np.int32)).to(DEV)
    fK, fV, fdeg, _ = _run_rounds_teacher_forced(K, V, chunk, [1.0, 0.7], "large degrees", deg=deg)
    gK, gV, gdeg, _ = _compress("defer_always", K, V, chunk, rounds=[1.0, 0.7], deg=deg)        # deferred pair
    torch.cuda.synchronize()
    assert torch.equal(gK, fK) and torch.equal(gV, fV) and torch.equal(gdeg, fdeg)
    assert int(gdeg.sum()) == int(d.sum())


def test_duplicate_keys_merge_losslessly_on_gpu():
    _say("compress duplicate keys")
    k = torch.randn(128, generator=torch.Generator().manual_seed(3)).to(torch.bfloat16)
    K = k.repeat(1, 1, 512, 1).contiguous().to(DEV)
    V = torch.randn((1, 1, 512, 128), generator=torch.Generator().manual_seed(4)).to(torch.bfloat16).to(DEV)
    gK, gV, gdeg, gas = ckv.compress(K, V, 256, rounds=[1.0])
    torch.cuda.synchronize()
    assert torch.equal(gK, k.to(DEV).expand_as(gK))             # every centroid key == the key
    # exact ties: all 128 sources of a chunk join the chunk's first B token
    assert i64(gdeg[0, 0]).tolist() == ([129] + [1] * 127) * 2
    ref = oracle.csm_round(f64(K[0, 0]), f64(V[0, 0]), np.ones(512, dtype=np.int64), 256, 1.0, "bf16")
    assert np.array_equal(i64(gas[0, 0]), ref["assign"])
    assert np.array_equal(f64(gV[0, 0]), ref["V"])


def test_zero_rounds_and_r_zero_are_identity():
    _say("compress identity")
    K, V, _ = kv_host(15, 2, 300, 64, "bf16")
    K, V = K.to(DEV), V.to(DEV)
    for kw in (dict(retain_ratio=1.0), dict(rounds=[0.0])):
        gK, gV, gdeg, gas = ckv.compress(K, V, 64, **kw)
        torch.cuda.synchronize()
        assert torch.equal(gK, K) and torch.equal(gV, V)
        assert bool((gdeg == 1).all())
        assert torch.equal(gas, torch.arange(300, dtype=torch.int32, device=DEV).expand(1, 2, 300))


def test_zero_keys_and_run_to_run_determinism():
    _say("compress zero keys / determinism")
    K, V, _ = kv_host(16, 2, 2048, 128, "bf16", n_outlier=4)
    K[0, 0, 100:140] = 0                                        # zero-norm keys: similarity 0
    K, V = K.to(DEV), V.to(DEV)
    _run_rounds_teacher_forced(K, V, 512, [0.6], "zero keys")
    a = ckv.compress(K, V, 512, retain_ratio=0.25)
    b = ckv.compress(K, V, 512, retain_ratio=0.25)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_runtime_argument_errors():
    _say("compress argument errors")
    K, V, _ = kv_host(17, 1, 256, 128, "bf16")
    K, V = K.to(DEV), V.to(DEV)
    with pytest.raises(ckv.CkvError) as e:
        ckv.compress(K, V, 64, rounds=[1.0], workspace=torch.empty(256, dtype=torch.uint8, device=DEV))
    assert e.value.status == -4
    with pytest.raises(ckv.CkvError) as e:
        ckv.compress(K, K, 64, rounds=[1.0], out=(K, V, torch.empty((1, 1, 256), dtype=torch.int32, device=DEV), None))
    assert e.value.status == -1                                  # output overlaps input
    K96 = torch.zeros((1, 1, 64, 96), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(ckv.CkvError) as e:
        ckv.compress(K96, K96.clone(), 16, rounds=[1.0])
    assert e.value.status == -5                                  # head_dim without a kernel


# ---- deferred values: rounds after an r = 1 round rebuild their value rows from the original cache ----
@pytest.mark.parametrize("dtype,heads,seq,dim,chunk,rounds,use_deg,n_sink,n_recent", [
    ("bf16", 3, 8192, 128, 1024, [1.0, 1.0], False, 0, 0),
    ("bf16", 2, 8192 + 80, 128, 1024, [1.0, 1.0], False, 16, 64),     # the paper's sinks / recents
    ("bf16", 2, 3000, 128, 256, [1.0, 1.0, 0.5], True, 5, 37),
    ("f32", 1, 700, 64, 64, [1.0, 1.0, 1.0, 1.0], False, 100, 150),    # the middle shrinks to a few tokens
    ("bf16", 1, 260, 128, 16, [1.0, 1.0], False, 100, 159),            # one clustered token: nothing to defer to
    ("bf16", 2, 5000, 128, 1024, [1.0, 0.6], True, 0, 0),          # ragged tail chunk in both rounds
    ("bf16", 2, 4097, 128, 256, [1.0, 1.0, 1.0], False, 0, 0),     # odd length: a one-token tail chunk; pair + one full round
    ("bf16", 1, 6000, 128, 2048, [1.0, 1.0, 1.0, 0.5], True, 0, 0),  # two pairs
    ("bf16", 2, 1026, 64, 2, [1.0, 1.0], False, 0, 0),             # chunk 2
    ("bf16", 1, 3000, 64, 512, [0.5, 1.0, 1.0], True, 0, 0),       # a full round first, then a pair
    ("f32", 2, 1500, 64, 64, [1.0, 0.75], True, 0, 0),
    ("f32", 1, 1024, 128, 128, [1.0, 1.0], False, 0, 0),
    # a pair in the middle of the schedule would write its result over the values it still reads
    # (the staging buffers alternate): such rounds run in full and the pair is taken at the end
    ("bf16", 1, 2566, 64, 1024, [0.5, 1.0, 1.0, 1.0], True, 0, 0),
    ("bf16", 2, 1413, 128, 512, [0.5, 0.8, 1.0, 0.5], False, 0, 7),
    ("bf16", 1, 2395, 128, 1024, [0.8, 1.0, 1.0, 0.5], False, 0, 0),
    ("bf16", 2, 9000, 128, 256, [1.0, 1.0, 1.0, 1.0, 1.0], False, 4, 16),   # pairs (0,1) and (3,4), round 2 in full
    ("f32", 1, 5000, 32, 128, [1.0, 1.0, 1.0, 1.0, 1.0, 0.5], True, 0, 0),
])
def test_deferred_values_are_bit_identical_to_full_rounds(dtype, heads, seq, dim, chunk, rounds, use_deg, n_sink,
                                                          n_recent):
    """By default a round that merges every edge (r = 1) and is followed by another writes keys and
    degrees only, and the next round rebuilds the value rows it needs from the original values.
    On the "full_rounds" route every round runs in full; both must give the same bits (the
    full rounds are checked against the oracle above)."""
    _say(f"deferred values {dtype} H={heads} S={seq} D={dim} c={chunk} rounds={rounds} deg={use_deg} "
         f"n1={n_sink} n2={n_recent}")
    kw = dict(n_sink=n_sink, n_recent=n_recent)
    K, V, _ = kv_host(51, heads, seq, dim, dtype, alpha=0.9, n_outlier=4 if dim == 128 else 0)
    K, V = K.to(DEV), V.to(DEV)
    deg = None
    if use_deg:
        deg = torch.from_numpy(np.random.default_rng(2).integers(1, 7, (1, heads, seq)).astype(np.int32)).to(DEV)
    ckv.timing_reset()
    ckv.timing_enable(True)
    got = _compress("defer_always", K, V, chunk, rounds=rounds, deg=deg, **kw)
    torch.cuda.synchronize()
    ckv.timing_enable(False)
    names = ckv.timing_read()
    suffix = "bf16" if dtype == "bf16" else "f32"
    assert f"merge_keys_{suffix}" in names and f"merge_origin_{suffix}" in names      # the deferred path really ran
    ckv.timing_reset()
    ckv.timing_enable(True)
    ref = _compress("full_rounds", K, V, chunk, rounds=rounds, deg=deg, **kw)
    torch.cuda.synchronize()
    ckv.timing_enable(False)
    assert f"merge_keys_{suffix}" not in ckv.timing_read()
    for n, a, b in zip(["K'", "V'", "deg'", "assign"], got, ref):
        assert a.shape == b.shape, n
        assert torch.equal(a, b), f"{n} differs between deferred and full rounds"


@pytest.mark.parametrize("scope,dim,chunk,seq,rounds,n_sink,n_recent,least", [
    ("chunk", 64, 64, 32768, [1.0, 1.0], 0, 0, "defer_always"),       # faster in one launch a round, smaller with values left
    ("chunk", 128, 256, 131073, [1.0, 1.0, 0.5], 0, 0, "defer_always"),
    ("head", 64, 16, 8192 + 80, [1.0, 1.0], 16, 64, "full_rounds"),   # without the member lists of a pair
])
def test_a_workspace_without_the_value_cache_is_enough(scope, dim, chunk, seq, rounds, n_sink, n_recent, least):
    """Jobs of 1024 chunks and more run in the scratch they take where the size of the job alone decides whether values
    are left to the next round: same bits, and not a byte less."""
    _say(f"least workspace {scope} D={dim} c={chunk} S={seq}")
    gen = torch.Generator(device=DEV).manual_seed(5)
    K, V = (torch.randn((1, 4, seq, dim), generator=gen, device=DEV).to(torch.bfloat16) for _ in range(2))
    kw = dict(rounds=rounds, n_sink=n_sink, n_recent=n_recent, scope=scope)
    need, enough = (ckv.plan(ckv.layout_of(K), ckv.make_params(chunk, route=r, **kw)).workspace_bytes for r in (None, least))
    assert enough < need
    want = ckv.compress(K, V, chunk, **kw)
    ws = torch.empty(enough, dtype=torch.uint8, device=DEV)
    ckv.timing_reset()
    ckv.timing_enable(True)
    got = ckv.compress(K, V, chunk, workspace=ws, **kw)
    torch.cuda.synchronize()
    ckv.timing_enable(False)
    assert ("merge_keys_bf16" in ckv.timing_read()) == (least == "defer_always")
    for n, a, e in zip(["K'", "V'", "deg'", "assign"], got, want):
        assert torch.equal(a, e), n
    with pytest.raises(ckv.CkvError) as e:
        ckv.compress(K, V, chunk, workspace=ws[:enough - 256], **kw)
    assert e.value.status == -4


def test_deferred_values_with_strided_input_and_padded_output():
    _say("deferred values, [B,S,H,D] input")
    B, H, S, D, c = 2, 2, 3072, 128, 512
    K0, V0, _ = kv_host(52, B * H, S, D, "bf16", alpha=0.9, n_outlier=4)
    Kb = K0.reshape(B, H, S, D).permute(0, 2, 1, 3).contiguous().to(DEV)
    Vb = V0.reshape(B, H, S, D).permute(0, 2, 1, 3).contiguous().to(DEV)
    K, V = Kb.permute(0, 2, 1, 3), Vb.permute(0, 2, 1, 3)
    out_len = S // 4
    oK = torch.zeros((B, H, out_len + 24, D), dtype=torch.bfloat16, device=DEV)
    oV = torch.zeros_like(oK)
    odeg = torch.zeros((B, H, out_len + 24), dtype=torch.int32, device=DEV)
    oas = torch.empty((B, H, S), dtype=torch.int32, device=DEV)
    _compress("defer_always", K, V, c, retain_ratio=0.25, out=(oK, oV, odeg, oas))
    ref = ckv.compress(K.contiguous(), V.contiguous(), c, rounds=[1.0])
    ref = ckv.compress(ref[0], ref[1], c, rounds=[1.0], deg=ref[2])         # two full single-round calls
    torch.cuda.synchronize()
    assert torch.equal(oK[:, :, :out_len], ref[0]) and torch.equal(oV[:, :, :out_len], ref[1])
    assert torch.equal(odeg[:, :, :out_len], ref[2]) and not bool(oV[:, :, out_len:].any())


@pytest.mark.parametrize("r", [1.0, 0.7])
@pytest.mark.parametrize("each", [1, 2, 3])
@pytest.mark.parametrize("dim,chunk", [(128, 384), (128, 1024), (128, 2048), (64, 2048)])
def test_rows_of_one_two_and_more_sources_are_emitted_where_they_belong(dim, chunk, each, r):
    """Whole chunks whose destinations have exactly `each` sources or none (one each: as many rows of one source as a
    chunk can have), and a tail in which nobody is alike: bf16, strided, a deferred pair and full rounds (the other forms of
    the merge: the test below)."""
    _say(f"rows by sources D={dim} c={chunk} each={each} r={r}")
    rng = np.random.default_rng(17 * chunk + each)
    seq, half = 4 * chunk + 77, chunk // 2
    K = rng.standard_normal((2, seq, dim))
    for h in range(2):
        for lo in range(0, 4 * chunk, chunk):
            sources = lo + 2 * rng.permutation(half)
            K[h, sources] = K[h, lo + 1 + 2 * (rng.permutation(half)[np.arange(half) // each])]
    K = torch.from_numpy(K).to(torch.bfloat16)[None].to(DEV)
    V = torch.from_numpy(rng.standard_normal((1, 2, seq, dim))).to(torch.bfloat16).to(DEV)
    kw = dict(rounds=[1.0, r])
    got, ref = _compress("defer_always", K, V, chunk, **kw), _compress("full_rounds", K, V, chunk, **kw)
    one = _compress("full_rounds", K, V, chunk, rounds=[r])
    torch.cuda.synchronize()
    for n, a, b in zip(["K'", "V'", "deg'", "assign"], got, ref):
        assert torch.equal(a, b), f"{n} differs between deferred and full rounds"
    ones = np.ones(seq, dtype=np.int64)
    for h in range(2):
        check_round(f64(K[0, h]), f64(V[0, h]), ones, chunk, r, "bf16", f64(one[0][0, h]), f64(one[1][0, h]),
                    i64(one[2][0, h]), i64(one[3][0, h]), what=f"h{h}")
        if r == 1.0:                                 # the chunks really were as described
            sizes = i64(one[2][0, h])[:4 * half]
            assert set(sizes.tolist()) <= {1, 1 + each, 1 + half % each}


@pytest.mark.parametrize("dtype,heads,seq,dim,chunk,r,scope", [
    ("bf16", 2, 2048 + 77, 128, 1024, 1.0, "chunk"),      # 32 workgroups of 16 row groups for 512 rows: output order ...
    ("bf16", 2, 2048 + 77, 128, 1024, 0.998, "chunk"),    # ... for 514: by sources
    ("bf16", 2, 4096 + 5, 64, 2048, 1.0, "chunk"),        # 32 of 32 for 1024
    ("bf16", 28, 4 * 384 + 1, 128, 384, 1.0, "chunk"),    # 9 of 16 for 192: by sources; a tail of one token
    ("bf16", 2, 4000, 128, 1000, 1.0, "chunk"),           # lists of 500, not read in pieces
    ("bf16", 2, 4 * 1024, 128, 1024, 0.5, "head"),        # a number of rows for every chunk
    ("f32", 2, 1024 + 90, 128, 512, 1.0, "chunk"),        # 32 of 8 for 256: output order ...
    ("f32", 2, 1040 + 90, 128, 520, 1.0, "chunk"),        # ... for 260: by sources
    ("f32", 1, 4096 + 3, 32, 2048, 0.7, "head"),
])
def test_rows_in_output_order_and_by_sources_on_strided_caches_and_pages(dtype, heads, seq, dim, chunk, r, scope):
    """Launches on either side of the line up to which every output row has a row group: one round against the oracle, and
    two rounds in full, deferred, and both again over pages, bit for bit."""
    _say(f"rows in output order {dtype} H={heads} S={seq} D={dim} c={chunk} r={r} {scope}")
    K, V, _ = kv_host(61, heads, seq, dim, dtype, alpha=0.9, n_outlier=0)
    K, V = K.to(DEV), V.to(DEV)
    one = _compress("full_rounds", K, V, chunk, rounds=[r], scope=scope)
    kw = dict(rounds=[1.0, r], scope=scope)
    ref = _compress("full_rounds", K, V, chunk, **kw)
    got = _compress("defer_always", K, V, chunk, **kw)
    torch.cuda.synchronize()
    for n, a, b in zip(["K'", "V'", "deg'", "assign"], got, ref):
        assert torch.equal(a, b), f"{n} differs between deferred and full rounds"
    check = check_round if scope == "chunk" else check_round_head
    for h in {0, heads - 1}:
        check(f64(K[0, h]), f64(V[0, h]), np.ones(seq, dtype=np.int64), chunk, r, dtype, f64(one[0][0, h]), f64(one[1][0, h]),
              i64(one[2][0, h]), i64(one[3][0, h]), what=f"h{h}")
    n_blocks = -(-seq // 16)
    for route in ("full_rounds", "defer_always"):
        table = torch.randperm(n_blocks, generator=torch.Generator().manual_seed(3)).to(torch.int32).view(1, -1).to(DEV)
        K_pool = torch.zeros((n_blocks, heads, 16, dim), dtype=K.dtype, device=DEV)
        pools = (K_pool, torch.zeros_like(K_pool), torch.zeros(K_pool.shape[:3], dtype=torch.int32, device=DEV))
        ckv.paged_scatter(K, V, None, *pools, table, seq)
        n, _ = ckv.paged_compress(*pools, table, seq, chunk, route=route, **kw)
        pages = ckv.paged_gather(*pools, table, n)
        torch.cuda.synchronize()
        for name, a, b in zip(["K'", "V'", "deg'"], pages, ref):
            assert torch.equal(a, b), f"{name} differs on pages ({route})"


@pytest.mark.parametrize("dtype,dim", [("bf16", 128), ("f32", 64)])
def test_a_whole_chunk_of_2048_copies(dtype, dim):
    """Chunks in which no edge is merged copy all 2048 tokens: in every chunk (r = 0), in front of a round, and in one
    chunk whose edges are all worse than the next chunk's."""
    _say(f"whole chunks of copies {dtype}")
    seq, chunk = 2 * 2048 + 1, 2048
    K, V, _ = kv_host(62, 1, seq, dim, dtype, alpha=0.9, n_outlier=0)
    K[:, :, 2048:4096:2] = K[:, :, 2049:4096:2]
    K, V = K.to(DEV), V.to(DEV)
    same = ckv.compress(K, V, chunk, rounds=[0.0])
    want, got = ckv.compress(K, V, chunk, rounds=[0.5]), ckv.compress(K, V, chunk, rounds=[0.0, 0.5])
    half = ckv.compress(K, V, chunk, rounds=[0.499], scope="head")      # 1021 of the second chunk's 1024 edges
    torch.cuda.synchronize()
    assert torch.equal(same[0], K) and torch.equal(same[1], V) and bool((same[2] == 1).all())
    assert torch.equal(same[3][0, 0].cpu().long(), torch.arange(seq))
    for n, a, b in zip(["K'", "V'", "deg'", "assign"], got, want):
        assert torch.equal(a, b), n
    assert half[0].shape[2] == seq - 1021
    assert torch.equal(half[0][:, :, :2048], K[:, :, :2048]) and torch.equal(half[1][:, :, :2048], V[:, :, :2048])
    assert torch.equal(half[3][0, 0, :2048].cpu().long(), torch.arange(2048)) and bool((half[2][:, :, :2048] == 1).all())
    check_round_head(f64(K[0, 0]), f64(V[0, 0]), np.ones(seq, dtype=np.int64), chunk, 0.499, dtype, f64(half[0][0, 0]),
                     f64(half[1][0, 0]), i64(half[2][0, 0]), i64(half[3][0, 0]), what="one chunk without an edge")


@pytest.mark.parametrize("dtype,seq,dim,chunk,n_proto,rounds", [
    ("bf16", 4096, 128, 1024, 6, [1.0, 1.0]),
    ("bf16", 4096 + 300, 128, 1024, 40, [1.0, 0.8]),
    ("bf16", 8192, 64, 2048, 12, [1.0, 1.0]),       # chunk 2048: the origin-mode route without resolved lookups
    ("f32", 2048, 64, 256, 5, [1.0, 1.0, 1.0, 1.0]),
])
def test_deferred_values_with_long_clusters(dtype, seq, dim, chunk, n_proto, rounds):
    """Keys from a handful of directions: tens of tokens join one centroid in the first round and
    several such centroids merge in the second, so the origin-mode rebuild walks long member lists
    at both levels.  Same bits as the full rounds, which are also checked against the oracle."""
    from synth.kv import prototype_kv_host
    _say(f"deferred values, long clusters {dtype} S={seq} D={dim} c={chunk} directions={n_proto} rounds={rounds}")
    K, V = prototype_kv_host(61, 2, seq, dim, dtype, n_proto)
    K, V = K.to(DEV), V.to(DEV)
    got = _compress("defer_always", K, V, chunk, rounds=rounds)
    ref = _compress("full_rounds", K, V, chunk, rounds=rounds)
    torch.cuda.synchronize()
    for n, a, b in zip(["K'", "V'", "deg'", "assign"], got, ref):
        assert torch.equal(a, b), f"{n} differs between deferred and full rounds"
    assert int(got[2].max()) >= 24                      # the long lists really occurred
    # the degrees are consistent with the assignment map, and the centroid values are the plain
    # degree-weighted means of the ORIGINAL values (one rounding per round: loose tolerance)
    gas, gdeg = i64(got[3][0, 0]), i64(got[2][0, 0])
    assert np.array_equal(np.bincount(gas, minlength=gdeg.size), gdeg)
    mean = np.zeros((gdeg.size, dim))
    np.add.at(mean, gas, f64(V[0, 0]))
    mean /= gdeg[:, None]
    tol = 2e-2 if dtype == "bf16" else 1e-5
    assert np.allclose(f64(got[1][0, 0]), mean, atol=tol, rtol=tol)


def test_calls_on_separate_streams_do_not_disturb_one_another():
    """Two compressions and an attention issued on three streams at once (own outputs and
    workspaces) give the bits of the same calls issued one after the other."""
    _say("three streams at once")
    jobs = []
    for i, (heads, seq, chunk, rounds) in enumerate([(4, 16384, 1024, [1.0, 1.0]), (3, 9000, 256, [1.0, 0.5, 1.0])]):
        K, V, _ = kv_host(71 + i, heads, seq, 128, "bf16", alpha=0.9, n_outlier=4)
        jobs.append((K.to(DEV), V.to(DEV), chunk, rounds))
    ref = [ckv.compress(K, V, c, rounds=r) for (K, V, c, r) in jobs]
    q = torch.randn((1, 16, 128), generator=torch.Generator().manual_seed(5)).to(torch.bfloat16).to(DEV)
    o_ref = ckv.decode_attn(q, ref[0][0], ref[0][1], deg=ref[0][2], out_dtype=torch.float32)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for _ in range(3):                                  # a few times: the overlap differs from run to run
        got = [None, None]
        for i, (K, V, c, r) in enumerate(jobs):
            with torch.cuda.stream(streams[i]):
                got[i] = ckv.compress(K, V, c, rounds=r)
        with torch.cuda.stream(streams[2]):
            o = ckv.decode_attn(q, ref[0][0], ref[0][1], deg=ref[0][2], out_dtype=torch.float32)
        torch.cuda.synchronize()
        for g, e in zip(got, ref):
            for a, b in zip(g, e):
                assert torch.equal(a, b)
        assert torch.equal(o, o_ref)


def test_compress_can_be_captured_in_a_hip_graph():
    """A whole compression (three rounds, sinks / recents, deferred pair) recorded into a HIP graph:
    every replay, with the outputs cleared and eager work in between, gives the eager bits."""
    _say("compress in a HIP graph")
    heads, seq, chunk, rounds = 4, 8192 + 80, 512, [1.0, 1.0, 0.5]
    K, V, _ = kv_host(81, heads, seq, 128, "bf16", alpha=0.9, n_outlier=4)
    K, V = K.to(DEV), V.to(DEV)
    kw = dict(rounds=rounds, n_sink=16, n_recent=64)
    ref = _compress("defer_always", K, V, chunk, **kw)
    torch.cuda.synchronize()
    out = tuple(torch.zeros_like(t) for t in ref)
    plan = ckv.plan(ckv.layout_of(K), ckv.make_params(chunk, rounds=rounds, n_sink=16, n_recent=64,
                                                      route="defer_always"))      # sized for the route that will run
    ws = torch.empty(max(plan.workspace_bytes, 256), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _compress("defer_always", K, V, chunk, out=out, workspace=ws, **kw)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _compress("defer_always", K, V, chunk, out=out, workspace=ws, **kw)
    for i in range(3):
        for t in out:
            t.zero_()
        ws.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n, a, b in zip(["K'", "V'", "deg'", "assign"], out, ref):
            assert torch.equal(a, b), f"replay {i}: {n}"
        ckv.compress(K, V, chunk, **kw)                  # eager work between replays
        torch.cuda.synchronize()


def test_timing_hooks_can_be_narrowed_to_one_kernel():
    """ckv_timing_select: only launches whose timing name starts with the prefix are bracketed."""
    _say("timing select")
    K, V, _ = kv_host(5, 2, 4096, 128, "bf16", alpha=0.9, n_outlier=4)
    K, V = K.to(DEV), V.to(DEV)
    try:
        ckv.timing_select("merge")
        ckv.timing_reset()
        ckv.timing_enable(True)
        ckv.compress(K, V, 1024, retain_ratio=0.25)
        torch.cuda.synchronize()
        ckv.timing_enable(False)
        names = ckv.timing_read()
        assert names and all(n.startswith("merge") for n in names), names
        ckv.timing_select(None)
        ckv.timing_reset()
        ckv.timing_enable(True)
        ckv.compress(K, V, 1024, retain_ratio=0.25)
        torch.cuda.synchronize()
        ckv.timing_enable(False)
        names = ckv.timing_read()
        assert "match_bf16" in names and any(n.startswith("merge") for n in names), names
    finally:
        ckv.timing_select(None)
        ckv.timing_enable(False)
        ckv.timing_reset()
