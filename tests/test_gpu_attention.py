"""GPU parity: ckv_decode_attn (HIP, through the C ABI) vs the oracle's Eq. 3."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_11418_amd as ckv
from parity_util import ATTN_TOL, assert_rows_close, f64, i64
from synth import kv_host, query_host

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(msg):
    print(msg, flush=True)


def _check(q, K, V, deg, lens, out, tol=ATTN_TOL, what=""):
    B = q.shape[0]
    for b in range(B):
        n = K.shape[2] if lens is None else int(lens[b])
        ref = oracle.app_attn(f64(q[b]), f64(K[b]), f64(V[b]), None if deg is None else i64(deg[b]), n)
        assert_rows_close(f64(out[b]), ref, tol, f"{what} b{b}")


def test_config1_decode_over_compressed_cache_fp32():
    _say("attn config1")
    K, V, rng = kv_host(0, 1, 1024, 64, "f32", alpha=0.9, single_stream=True)
    q = query_host(rng, 1, 1, 64, "f32").to(DEV)
    K, V = K.to(DEV), V.to(DEV)
    cK, cV, cdeg, _ = ckv.compress(K, V, 64, retain_ratio=0.5)
    o = ckv.decode_attn(q, cK, cV, deg=cdeg)
    torch.cuda.synchronize()
    _check(q, cK, cV, cdeg, None, o, tol=1e-4, what="config1")
    # and the approximation is close to attention over the full cache (sanity, loose)
    full = oracle.app_attn(f64(q[0]), f64(K[0]), f64(V[0]))
    assert np.abs(f64(o[0]) - full).max() < 0.5


@pytest.mark.parametrize("B,Hkv,G,L,D,dtype", [
    (1, 8, 4, 8192, 128, "bf16"),      # config 2's compressed cache
    (2, 2, 4, 1000, 128, "bf16"),      # ragged: not a multiple of the slice
    (3, 1, 8, 300, 64, "bf16"),
    (2, 2, 1, 513, 128, "bf16"),
    (1, 2, 2, 77, 32, "f32"),
    (2, 1, 4, 2000, 128, "f32"),
    (1, 1, 1, 1, 64, "f32"),
])
def test_decode_attn_shapes(B, Hkv, G, L, D, dtype):
    _say(f"attn B={B} Hkv={Hkv} G={G} L={L} D={D} {dtype}")
    rng = np.random.default_rng(B * 1000 + L)
    Ks, Vs = [], []
    for b in range(B):
        K, V, _ = kv_host(20 + b, Hkv, L, D, dtype, n_outlier=0)
        Ks.append(K)
        Vs.append(V)
    K, V = torch.cat(Ks).to(DEV), torch.cat(Vs).to(DEV)
    q = query_host(int(rng.integers(1 << 30)), B, Hkv * G, D, dtype).to(DEV)
    deg = torch.from_numpy(rng.integers(1, 6, (B, Hkv, L)).astype(np.int32)).to(DEV)
    lens = torch.from_numpy(rng.integers(1, L + 1, B).astype(np.int32))
    lens[0] = L
    tol = 1e-4 if dtype == "f32" else ATTN_TOL
    o = ckv.decode_attn(q, K, V, lens=lens.to(DEV), deg=deg, out_dtype=torch.float32)
    torch.cuda.synchronize()
    _check(q, K, V, deg, lens, o, tol, "deg+lens")
    o2 = ckv.decode_attn(q, K, V)                                 # vanilla attention, cache dtype out
    torch.cuda.synchronize()
    # a bf16 output carries its own rounding (half an ulp = 2^-9 relative) on top of the bar
    _check(q, K, V, None, None, o2, ATTN_TOL + 2.0 ** -8 if dtype == "bf16" else 1e-4, "vanilla")


@pytest.mark.parametrize("B,Hkv,G,L,D,dtype", [
    (6, 2, 4, 65, 128, "bf16"),        # around one tile (16 tokens) and one tile per wave (64)
    (6, 2, 8, 130, 64, "bf16"),
    (6, 2, 1, 130, 128, "f32"),
    (6, 1, 2, 65, 32, "f32"),
    (1, 2, 4, 8191, 128, "bf16"),      # two pairs: the last length in short slices of four waves ...
    (1, 2, 4, 8192, 128, "bf16"),      # ... and the first in 64 slices of eight
    (2, 1, 8, 24576, 128, "bf16"),     # the last in 64 slices, one sequence far below it
    (1, 1, 2, 32768, 128, "bf16"),     # the last length of one pair with four waves per workgroup ...
    (1, 1, 2, 32769, 128, "bf16"),     # ... and the first with eight
    (3, 2, 8, 8200, 64, "bf16"),       # eight waves, slices that end inside a tile
    (2, 2, 4, 9000, 64, "f32"),
    (17, 1, 4, 2100, 128, "bf16"),     # more pairs than eight waves are taken for
    (520, 1, 1, 300, 64, "bf16"),      # one slice per pair: written without a merge
    (2, 1, 1, 100000, 32, "f32"),      # slices merged in whole blocks and a rest, threads in 16, 8, 4 and 2 groups ...
    (1, 1, 2, 40000, 32, "f32"),
    (2, 1, 4, 2100, 32, "f32"),
    (1, 2, 8, 40000, 32, "f32"),
    (1, 1, 8, 40000, 64, "f32"),       # ... in one, a thread's one pair of channels ...
    (2, 1, 8, 40000, 128, "f32"),      # ... and its two
    (1, 2, 8, 2100, 128, "f32"),
    (1, 1, 8, 8192, 128, "f32"),       # 32 slices by pairs of channels ...
    (1, 1, 8, 8193, 128, "f32"),       # ... and 33 by single ones: a block of 32 and one more ...
    (1, 2, 4, 16384, 128, "f32"),
    (1, 2, 4, 27400, 128, "f32"),      # ... 108: three, one of eight and four
    (2, 1, 8, 18000, 64, "f32"),
    (1, 1, 8, 24000, 64, "bf16"),      # bf16: two blocks of 32 slices and a rest ...
    (1, 1, 8, 32000, 128, "bf16"),     # ... and, with two pairs of channels a thread, seven of 16
])
def test_attn_tile_and_slice_edges(B, Hkv, G, L, D, dtype):
    """Lengths around the tiles and slices of the kernel, most of them far below the cache's capacity, with
    and without degrees.  Logits, weights and sums are fp32: the bar is the file's own."""
    _say(f"attn edges B={B} Hkv={Hkv} G={G} L={L} D={D} {dtype}")
    rng = np.random.default_rng(L + D)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    K, V = (torch.from_numpy(rng.standard_normal((B, Hkv, L, D)).astype(np.float32)).to(td).to(DEV) for _ in range(2))
    q = torch.from_numpy(rng.standard_normal((B, Hkv * G, D)).astype(np.float32)).to(td).to(DEV)
    deg = torch.from_numpy(rng.integers(1, 300, (B, Hkv, L)).astype(np.int32)).to(DEV)
    edges = [L, 1, 15, 16, 17, 63, 64] if B < 17 else [L, 1, L - 1, 16, 129]
    lens = torch.tensor([min(edges[b % len(edges)], L) for b in range(B)], dtype=torch.int32)
    o = ckv.decode_attn(q, K, V, lens=lens.to(DEV), deg=deg, out_dtype=torch.float32)
    plain = ckv.decode_attn(q, K, V, out_dtype=torch.float32)
    torch.cuda.synchronize()
    some = slice(0, min(B, 20))
    tol = 1e-4 if dtype == "f32" else ATTN_TOL
    _check(q[some], K[some], V[some], deg[some], lens[some], o[some], tol, "edges")
    _check(q[some], K[some], V[some], None, None, plain[some], tol, "plain")


@pytest.mark.parametrize("H,cap,lengths", [
    (8, 4352, (4352, 4096, 3742, 4097, 2049, 515, 4352)),        # eight waves above 32768 tokens over all heads, four up to it
    (1, 33000, (32768, 32769, 16384, 33000, 100, 32768)),
])
def test_one_workspace_for_the_capacity_serves_every_length(H, cap, lengths):
    """The bits of calls with a workspace of their own, whatever length came before."""
    _say(f"attn one workspace H={H} capacity={cap}")
    gen = torch.Generator(device=DEV).manual_seed(cap)
    K, V = (torch.randn((1, H, cap, 128), generator=gen, device=DEV).to(torch.bfloat16) for _ in range(2))
    q = torch.randn((1, 4 * H, 128), generator=gen, device=DEV).to(torch.bfloat16)
    deg = torch.randint(1, 9, (1, H, cap), generator=gen, device=DEV, dtype=torch.int32)
    ws = torch.zeros(ckv.decode_attn_workspace(ckv.layout_of(K, deg), 4 * H), dtype=torch.uint8, device=DEV)
    for n in lengths:
        call = lambda w: ckv.decode_attn(q, K[:, :, :n], V[:, :, :n], deg=deg[:, :, :n], out_dtype=torch.float32, workspace=w)
        o, own = call(ws), call(None)
        torch.cuda.synchronize()
        assert torch.equal(o, own), n
        _check(q, K[:, :, :n], V[:, :, :n], deg[:, :, :n], None, o, ATTN_TOL, f"length {n}")


@pytest.mark.parametrize("B,Hkv,G,L,D", [
    (1, 8, 4, 128, 128), (1, 8, 4, 129, 128), (3, 2, 1, 256, 64), (3, 2, 8, 257, 64),     # two steps of four waves, and a row more
    (24, 8, 2, 1536, 128), (24, 8, 1, 1537, 64), (32, 8, 1, 700, 128), (33, 8, 1, 300, 64),   # a workgroup of eight waves per pair
    (24, 8, 1, 128, 128), (24, 8, 4, 129, 128), (32, 8, 8, 128, 64), (32, 8, 1, 129, 64),     # four waves up to 128 tokens of that many
])
def test_caches_of_one_slice(B, Hkv, G, L, D):
    """Sequences of lengths down to zero on both sides of the sizes up to which a cache is not cut."""
    _say(f"one slice B={B} Hkv={Hkv} G={G} L={L} D={D}")
    K, V, _ = kv_host(83, Hkv, L, D, "bf16", n_outlier=0)
    K, V = K.expand(B, Hkv, L, D).contiguous().to(DEV), V.expand(B, Hkv, L, D).contiguous().to(DEV)
    q = query_host(84, B, Hkv * G, D, "bf16").to(DEV)
    deg = torch.from_numpy(np.random.default_rng(L).integers(1, 6, (B, Hkv, L)).astype(np.int32)).to(DEV)
    lens = torch.tensor([L - b * L // max(B - 1, 1) for b in range(B)], dtype=torch.int32, device=DEV)
    o = ckv.decode_attn(q, K, V, lens=lens, deg=deg, out_dtype=torch.float32)
    torch.cuda.synchronize()
    some = [b for b in range(B) if int(lens[b]) > 0 and (B <= 8 or b % 5 == 0)]
    assert B == 1 or not o[B - 1].any()              # an empty cache
    _check(q[some], K[some], V[some], deg[some], lens[some], o[some], what="one slice")


@pytest.mark.parametrize("B,Hkv,G,L,D", [(1, 2, 4, 40, 128), (2, 1, 8, 515, 64), (1, 1, 2, 5000, 128), (1, 4, 1, 9001, 64)])
@pytest.mark.parametrize("scale", [0.0, 1e-6])          # ordinary weights, and all of them within a bit of 1
def test_infinite_values_reach_their_own_channels_only(B, Hkv, G, L, D, scale):
    """A value of infinity under a weight above zero: infinity in that channel, every other channel as the oracle has it."""
    _say(f"attn infinite values B={B} Hkv={Hkv} G={G} L={L} D={D} scale={scale}")
    K, V, _ = kv_host(93, Hkv, L, D, "bf16", n_outlier=0)
    K, V = K.expand(B, Hkv, L, D).contiguous().to(DEV), V.expand(B, Hkv, L, D).contiguous().to(DEV)
    q = query_host(94, B, Hkv * G, D, "bf16").to(DEV)
    deg = torch.from_numpy(np.random.default_rng(L).integers(1, 6, (B, Hkv, L)).astype(np.int32)).to(DEV)
    hit = {0: (0, np.inf), 3: (L // 2, -np.inf), D - 1: (L - 2, np.inf), 5: (17, np.inf)}    # channel: token, value
    P = V.clone()
    for c, (t, x) in hit.items():
        P[:, :, t, c] = x
    o = ckv.decode_attn(q, K, P, deg=deg, scale=scale, out_dtype=torch.float32)
    plain = ckv.decode_attn(q, K, V, deg=deg, scale=scale, out_dtype=torch.float32)
    torch.cuda.synchronize()
    for c, (_, x) in hit.items():
        assert bool((o[:, :, c] == x).all()), (c, o[0, :, c])
    rest = [c for c in range(D) if c not in hit]
    assert torch.equal(o[:, :, rest], plain[:, :, rest])


@pytest.mark.parametrize("dtype,Hkv,G,L,D,low", [
    ("bf16", 2, 4, 64, 128, lambda t, L, D: t % 64 < 16),                        # one wave of four
    ("bf16", 2, 8, 128, 64, lambda t, L, D: t % 128 < 32),
    ("bf16", 1, 1, 40000, 128, lambda t, L, D: t < L // 2),                      # slices, of eight waves each ...
    ("bf16", 2, 2, 4096, 64, lambda t, L, D: t < L // 2),                        # ... and of four
    ("f32", 2, 4, 64, 128, lambda t, L, D: t % (1024 // D) == 0),                # one row group
    ("f32", 2, 2, 64, 32, lambda t, L, D: t % (1024 // D) == 0),
    ("f32", 2, 8, 64, 128, lambda t, L, D: t % (1024 // D) < 256 // D),          # one wave's row groups
    ("f32", 2, 1, 128, 64, lambda t, L, D: t % (1024 // D) < 256 // D),
    ("f32", 1, 8, 3000, 128, lambda t, L, D: t < L // 2),                        # slices
    ("f32", 1, 8, 20000, 128, lambda t, L, D: t < L // 2),                       # ... merged by single channels
])
def test_weights_down_to_the_smallest_denormal_count(dtype, Hkv, G, L, D, low):
    """Parts of a cache whose logits lie 2^-140 below the rest's: their weight is not zero, and an infinite value
    among them gives infinity in its channel, not 0 x infinity.  Every other channel as without it."""
    _say(f"attn small weights {dtype} Hkv={Hkv} G={G} L={L} D={D}")
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    t = torch.arange(L)
    K = torch.zeros((1, Hkv, L, D))
    K[:, :, :, 0] = torch.where(low(t, L, D), 0.0, 97.0)           # 97 log2(e) = 139.9
    V = torch.from_numpy(np.random.default_rng(L).standard_normal((1, Hkv, L, D)).astype(np.float32))
    q = torch.zeros((1, Hkv * G, D))
    q[:, :, 0] = 1.0
    K, V, q = K.to(td).to(DEV), V.to(td).to(DEV), q.to(td).to(DEV)
    P = V.clone()
    P[:, :, 0, 5], P[:, :, 0, D - 1] = np.inf, -np.inf
    o, plain = (ckv.decode_attn(q, K, x, scale=1.0, out_dtype=torch.float32) for x in (P, V))
    torch.cuda.synchronize()
    assert bool((o[:, :, 5] == np.inf).all()) and bool((o[:, :, D - 1] == -np.inf).all())
    rest = [c for c in range(D) if c not in (5, D - 1)]
    assert torch.equal(o[:, :, rest], plain[:, :, rest])
    _check(q * np.sqrt(D), K, V, None, None, plain, 1e-4 if dtype == "f32" else ATTN_TOL, "without it")


@pytest.mark.parametrize("L", [200, 9000, 17000])      # one slice, 36, 67
def test_fp32_caches_with_bf16_outputs(L):
    """The fp32 result, rounded once."""
    _say(f"attn fp32 cache, bf16 output L={L}")
    gen = torch.Generator(device=DEV).manual_seed(L)
    K, V = (torch.randn((1, 2, L, 128), generator=gen, device=DEV) for _ in range(2))
    q = torch.randn((1, 16, 128), generator=gen, device=DEV)
    o, full = (ckv.decode_attn(q, K, V, out_dtype=t) for t in (torch.bfloat16, torch.float32))
    torch.cuda.synchronize()
    assert torch.equal(o, full.to(torch.bfloat16))
    _check(q, K, V, None, None, full, 1e-4, "fp32")


def test_outlier_keys_large_logits_bf16():
    """Keys with x10 outlier channels give logits of several tens: the softmax must stay stable."""
    _say("attn outliers")
    K, V, _ = kv_host(31, 2, 4096, 128, "bf16", n_outlier=4)
    q = query_host(32, 1, 8, 128, "bf16")
    K, V, q = K.to(DEV), V.to(DEV), q.to(DEV)
    cK, cV, cdeg, _ = ckv.compress(K, V, 1024, retain_ratio=0.25)
    o = ckv.decode_attn(q, cK, cV, deg=cdeg, out_dtype=torch.float32)
    torch.cuda.synchronize()
    _check(q, cK, cV, cdeg, None, o, ATTN_TOL, "outliers")


def test_zero_length_and_zero_query():
    _say("attn zero length / zero query")
    K, V, _ = kv_host(33, 1, 256, 128, "bf16")
    K, V = K.to(DEV), V.to(DEV)
    cK, cV, cdeg, _ = ckv.compress(K, V, 64, retain_ratio=0.5)
    q = torch.zeros((1, 4, 128), dtype=torch.bfloat16, device=DEV)
    o = ckv.decode_attn(q, cK, cV, deg=cdeg, out_dtype=torch.float32)
    torch.cuda.synchronize()
    # q = 0: degree-weighted mean of centroids = plain mean of the ORIGINAL values (bf16 storage of V')
    assert np.abs(f64(o[0, 0]) - f64(V[0, 0]).mean(0)).max() < 2e-3
    lens = torch.zeros(1, dtype=torch.int32, device=DEV)
    o0 = ckv.decode_attn(torch.ones_like(q), cK, cV, lens=lens, deg=cdeg)
    torch.cuda.synchronize()
    assert float(o0.float().abs().sum()) == 0.0


def test_strided_cache_layout():
    _say("attn strided layout")
    K, V, _ = kv_host(34, 2, 640, 128, "bf16")
    q = query_host(35, 1, 4, 128, "bf16").to(DEV)
    Kb = K.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)     # [B,S,H,D] storage
    Vb = V.permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    a = ckv.decode_attn(q, Kb, Vb, out_dtype=torch.float32)
    b = ckv.decode_attn(q, K.to(DEV), V.to(DEV), out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_decode_loop_can_be_captured_in_a_hip_graph():
    """The library allocates nothing, synchronises nothing and clears nothing with memset, so the
    per-layer attention calls of a decode step (and an append before them) can be recorded into a
    HIP graph.  Every replay, with eager work and synchronisation between replays, gives the bits of
    the eager calls."""
    _say("attention calls in a HIP graph")
    Ly, Hkv, G, L, D = 6, 4, 4, 3000, 128
    K, V, _ = kv_host(61, Ly * Hkv, L + 1, D, "bf16", n_outlier=0)
    K, V = K.reshape(Ly, Hkv, L + 1, D).to(DEV), V.reshape(Ly, Hkv, L + 1, D).to(DEV)
    rng = np.random.default_rng(3)
    deg = torch.from_numpy(rng.integers(1, 6, (Ly, Hkv, L + 1)).astype(np.int32)).to(DEV)
    q = query_host(9, Ly, Hkv * G, D, "bf16").to(DEV).reshape(Ly, 1, Hkv * G, D)
    k_new, v_new = K[:, :, L].clone(), V[:, :, L].clone()
    ws = torch.zeros(ckv.decode_attn_workspace(ckv.layout_of(K[0:1]), Hkv * G), dtype=torch.uint8, device=DEV)
    o = torch.empty((Ly, 1, Hkv * G, D), dtype=torch.float32, device=DEV)

    def step():
        for l in range(Ly):
            ckv.append(k_new[l:l + 1], v_new[l:l + 1], K[l:l + 1], V[l:l + 1], deg[l:l + 1], pos=L)
            ckv.decode_attn(q[l], K[l:l + 1], V[l:l + 1], deg=deg[l:l + 1], out=o[l], workspace=ws)

    step()
    torch.cuda.synchronize()
    ref = o.clone()
    for l in (0, Ly - 1):
        _check(q[l], K[l:l + 1], V[l:l + 1], deg[l:l + 1], None, ref[l], ATTN_TOL, f"eager layer {l}")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                           # warm-up on the capture stream's side
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for i in range(4):
        o.zero_()
        K[:, :, L].zero_()                               # the captured append has to write the token again
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, ref), f"replay {i}"
        assert torch.equal(K[:, :, L], k_new)
        step()                                           # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(o, ref)


def test_attn_argument_errors():
    _say("attn argument errors")
    K = torch.zeros((1, 2, 64, 128), dtype=torch.bfloat16, device=DEV)
    q = torch.zeros((1, 6, 128), dtype=torch.bfloat16, device=DEV)      # 3 query heads per KV head
    with pytest.raises(ckv.CkvError) as e:
        ckv.decode_attn(q, K, K)
    assert e.value.status == -5
    q = torch.zeros((1, 8, 128), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(ckv.CkvError) as e:
        ckv.decode_attn(q, K, K, workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
    assert e.value.status == -4
