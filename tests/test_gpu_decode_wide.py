"""The eight- and four-wave decode kernel at the edges of its dispatch, against the oracle: one block of
entries, one more than a round of its waves, several slices, more workgroups than compute units, and the
smallest and largest head groups.  Needs an MI355X."""
import ctypes
import math

import numpy as np
import pytest

import oracle
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    (2, 16, 1, 128, 0, 8, 4, 24),     # one block; 16 heads per KV head; fewer table rows than a block has entries
    (2, 8, 4, 64, 4, 100, 60, 256),   # exactly one block per wave
    (2, 8, 8, 64, 4, 100, 60, 257),   # one wave has a second block
    (2, 14, 2, 128, 4, 64, 256, 800), # 7 heads per KV head; several slices
    (1, 8, 2, 128, 4, 200, 100, 530), # several slices with ROPE, one without
    (1, 4, 1, 128, 4, 300, 256, 1100),# several slices with and without ROPE
    (3, 6, 2, 64, 3, 700, 300, 1999), # the same at d = 64
    (33, 16, 8, 128, 2, 20, 10, 75),  # 264 pairs: four waves, two workgroups per compute unit
    (65, 8, 8, 64, 2, 150, 50, 290),  # 520 pairs, several blocks per wave
]


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("S,Hq,Hkv,d,a,s,w,c", CASES)
def test_decode_dispatch_edges(S, Hq, Hkv, d, a, s, w, c, rope):
    import paper_2412_12094_amd as sp

    rng = np.random.default_rng(c + S)
    wcap = c - a - s
    sizes = np.zeros((S, 4), dtype=np.int32)
    for q in range(S):
        tot = int(rng.integers(1, wcap + 1))
        loc = min(w, tot)
        sizes[q] = (int(rng.integers(0, a + 1)), int(rng.integers(0, s + 1)), tot - loc, loc)
    sizes[0] = (a, s, wcap - w, w)  # one full cache
    if S > 1:
        sizes[1] = (0, 0, 0, 1)     # and one with a single entry
    cfg = wl.CacheConfig("wide", S, Hq, Hkv, d, a, s, w, c, 0.1, "bf16", seed=900 + c)
    data = wl.make_cache(cfg, sizes)
    heads = np.stack([rng.integers(0, s, size=S), rng.integers(0, wcap, size=S)], axis=1)
    # slots without a valid entry hold NaN
    Kp, Vp, _, sz6 = wl.cache_to_ring(data["Kc"], data["Vc"], data["win_is_sep"], sizes, heads, a, s, fill=np.nan)
    bf = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda().to(torch.bfloat16)
    q, Kc, Vc, sz = bf(data["q"]), bf(Kp), bf(Vp), torch.from_numpy(sz6).cuda()
    scale = 1.0 / math.sqrt(d)
    if rope:
        table = sp.sepkv_rope_table(c, d, 10000.0, "cuda")
        out, lse = sp.sepattn_decode_rope(q, Kc, Vc, sz, table, a, s, w, scale)
        ref, lref = oracle.decode_rope(data["q"], data["Kc"], data["Vc"], sizes, a, s, scale, 10000.0)
    else:
        out, lse = sp.sepattn_decode(q, Kc, Vc, sz, a, s, w, scale)
        ref, lref = oracle.decode(data["q"], data["Kc"], data["Vc"], sizes, a, s, scale)
    torch.cuda.synchronize()
    assert np.abs(out.float().cpu().numpy() - ref).max() <= 2e-2
    assert np.abs(lse.cpu().numpy() - lref).max() <= (1e-2 if rope else 2e-3)


# slices and waves per workgroup: the edges of decode_wide_shape's rules on a chip of 256 compute units.  `slices`: without and
# with ROPE
SHAPE_CASES = [
    (1, 8, 2, 128, 4, 50, 30, 128, (1, 1)),         # four blocks: four waves
    (1, 8, 2, 128, 4, 50, 30, 129, (1, 1)),         # five: eight waves
    (1, 8, 2, 128, 4, 100, 60, 256, (1, 1)),        # eight blocks: one slice of eight waves
    (1, 8, 2, 128, 4, 100, 60, 385, (1, 4)),        # 13 blocks: one slice of eight waves without ROPE, four of four with
    (4, 32, 8, 128, 4, 64, 256, 800, (7, 7)),       # 25 blocks in seven slices, the last of one block
    (2, 8, 1, 128, 0, 1100, 256, 2600, (16, 16)),   # 82 blocks in sixteen slices
    (9, 56, 8, 128, 4, 500, 100, 1600, (3, 3)),     # 72 pairs of seven heads: three slices
    (16, 128, 8, 128, 4, 200, 100, 800, (1, 1)),    # 128 pairs of sixteen heads, 25 blocks: one slice
    (16, 32, 8, 128, 4, 200, 100, 1100, (1, 2)),    # 128 pairs, 35 blocks: one slice without ROPE, two with
    (16, 32, 8, 128, 4, 800, 100, 1312, (1, 2)),    # 41 blocks: 20 spared, one without
    (16, 32, 8, 128, 4, 800, 100, 1340, (2, 2)),    # 42 blocks: 21 spared, two slices without ROPE too, added in the kernel
    (16, 128, 8, 128, 4, 800, 100, 1400, (2, 2)),   # 128 pairs of sixteen heads, 44 blocks: two slices, merge launch
    (2, 12, 12, 64, 3, 64, 256, 800, (1, 7)),       # d = 64: one slice without ROPE, seven of four waves with
    (4, 8, 8, 64, 4, 900, 256, 2300, (8, 8)),       # nine blocks per slice: eight waves
    (2, 14, 2, 128, 4, 500, 256, 1400, (8, 8)),     # seven heads: eight slices added in the kernel
    (2, 14, 2, 128, 4, 1100, 256, 2600, (16, 16)),  # seven heads: sixteen slices, merge launch
    (1, 4, 2, 64, 4, 2500, 256, 5200, (16, 16)),    # d = 64, 163 blocks: sixteen slices, two fetches of records
    (1, 2, 1, 128, 4, 4000, 256, 6500, (32, 32)),   # 204 blocks, one pair: thirty-two slices, merge launch
    (1, 5, 5, 128, 4, 4000, 256, 6500, (16, 16)),   # 204 blocks, five pairs: sixteen
    (1, 2, 1, 64, 4, 30000, 256, 51300, (64, 64)),  # 1604 blocks: sixty-four
    (33, 8, 8, 64, 4, 500, 100, 1100, (1, 1)),      # 264 pairs at d = 64: one slice of eight waves
]


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("S,Hq,Hkv,d,a,s,w,c,slices", SHAPE_CASES)
def test_decode_slices_and_waves(S, Hq, Hkv, d, a, s, w, c, slices, rope):
    import paper_2412_12094_amd as sp

    # the workspace holds the records of the larger number of slices, and words to count them if there are several
    up = lambda x: -(-x // 256) * 256
    p = sp.binding.SepkvParams(S, Hq, Hkv, d, a, s, w, c, 1.0, 0)
    words = up(S * Hkv * 8) if max(slices) > 1 else 0
    assert sp.load().sepattn_decode_workspace_bytes(ctypes.byref(p)) == words + up(S * Hq * max(slices) * (d + 2) * 4)
    test_decode_dispatch_edges(S, Hq, Hkv, d, a, s, w, c, rope)


def test_decode_workspace_needs_no_clearing():
    """The slices are counted in the workspace, whatever it holds: the same bits from any of it, call after call and
    with calls of other shapes, which lay the workspace out differently, in between."""
    import paper_2412_12094_amd as sp

    def call(S, c, seed, ws):
        g = torch.Generator(device="cuda").manual_seed(seed)
        q = torch.randn((S, 32, 128), device="cuda", generator=g).bfloat16()
        K, V = (torch.randn((S, 8, c, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
        sizes = torch.tensor([[4, 64, c - 4 - 64 - 256, 256, 3, 5]] * S, dtype=torch.int32, device="cuda")
        return [t.clone() for t in sp.sepattn_decode(q, K, V, sizes, 4, 64, 256, 0.09, ws=ws)]

    shapes = [(4, 800, 1), (1, 2600, 2), (9, 700, 3)]
    fresh = [call(*s, torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")) for s in shapes]
    g = torch.Generator(device="cuda").manual_seed(9)
    noise = torch.randint(0, 256, (4 << 20,), dtype=torch.uint8, device="cuda", generator=g)
    for ws in (noise, torch.full_like(noise, 255), torch.full_like(noise, 0x7F)):
        for k in (0, 0, 1, 2, 0, 2, 1):
            for got, ref in zip(call(*shapes[k], ws), fresh[k]):
                assert torch.equal(got, ref)


@pytest.mark.parametrize("left", [1, 3, 6])
def test_decode_heals_from_counts_that_overlapping_calls_left(left):
    """Two calls that overlap on one workspace may leave any count in the words that count the slices.  That spoils
    those calls, and none after them."""
    import paper_2412_12094_amd as sp

    S, Hkv, c, sizes = 4, 8, 800, [[4, 64, 476, 256, 3, 5]]
    ws = torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")
    # a word in front of the records of its (sequence, KV head): four heads, seven slices, 130 floats each
    words = ws.view(torch.int64).as_strided((S * Hkv,), (1 + 4 * 7 * 130 // 2,))
    g = torch.Generator(device="cuda").manual_seed(left)
    sz = torch.tensor(sizes * S, dtype=torch.int32, device="cuda")
    for call in range(4):
        q = torch.randn((S, 32, 128), device="cuda", generator=g).bfloat16()
        K, V = (torch.randn((S, Hkv, c, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
        ref = sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, ws=torch.zeros_like(ws))
        got = sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, ws=ws)
        for x, y in zip(got, ref):
            assert torch.equal(x, y), call
        assert not words.any(), call  # set back, for the next call to find it so
        words += left + (call << 40)  # the lower 8 bits count, the upper ones tell launches apart


def test_decode_alone_after_calls_that_overlapped():
    """The same with an overlap: whatever two streams leave in a workspace that they share, later calls are right."""
    import paper_2412_12094_amd as sp

    g = torch.Generator(device="cuda").manual_seed(21)
    q = torch.randn((4, 32, 128), device="cuda", generator=g).bfloat16()
    K, V = (torch.randn((4, 8, 800, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    sz = torch.tensor([[4, 64, 476, 256, 3, 5]] * 4, dtype=torch.int32, device="cuda")
    ws = torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")
    ref = sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, ws=torch.zeros_like(ws))
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [(torch.empty_like(q), torch.empty((4, 32), device="cuda")) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(16):
        for st, out in zip(streams, outs):
            with torch.cuda.stream(st):
                sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, out=out, ws=ws)
    torch.cuda.synchronize()
    for call in range(3):
        got = sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, ws=ws)
        for x, y in zip(got, ref):
            assert torch.equal(x, y), call


def test_decode_captured_slices_replay():
    """A captured call has several slices too; whatever the workspace holds before a replay, the outputs are those of the
    eager call, bit for bit."""
    import paper_2412_12094_amd as sp

    g = torch.Generator(device="cuda").manual_seed(11)
    q = torch.empty((4, 32, 128), dtype=torch.bfloat16, device="cuda")
    K, V = (torch.randn((4, 8, 800, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    sz = torch.tensor([[4, 64, 476, 256, 3, 5]] * 4, dtype=torch.int32, device="cuda")
    out = (torch.empty_like(q), torch.empty((4, 32), device="cuda"))
    ws, other = (torch.zeros(4 << 20, dtype=torch.uint8, device="cuda") for _ in range(2))
    call = lambda w, o: sp.sepattn_decode(q, K, V, sz, 4, 64, 256, 0.09, out=o, ws=w)
    side = torch.cuda.Stream()
    q.normal_(generator=g)
    with torch.cuda.stream(side):
        call(ws, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(ws, out)
    for k in range(5):
        q.normal_(generator=g)
        ref = [t.clone() for t in call(other, None)]
        ws.random_(0, 256, generator=g) if k % 2 else ws.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, ref):
            assert torch.equal(x, y), k


@pytest.mark.parametrize("S,Hq,Hkv,d,a,s,w,c,blocks", [  # blocks: of the first slice; seven, eight and sixteen slices
    (4, 32, 8, 128, 4, 64, 256, 800, 4), (4, 8, 8, 64, 4, 900, 256, 2300, 9), (1, 4, 2, 64, 4, 2500, 256, 5200, 11)])
def test_decode_slices_far_apart(S, Hq, Hkv, d, a, s, w, c, blocks):
    """Slices whose maxima lie 130 octaves apart: their weights, below the smallest normal number, reach the output where
    the values are as large, and in a captured call as in an eager one, bit for bit.  Scores in octaves: 90 log2(e) at one entry of the
    first slice, 0 at all others, which hold 2^115 (the first slice zeros): each weight of 2^-129.84 keeps 19 bits, so the bf16
    result is within 2^-8 of the exact sum."""
    import paper_2412_12094_amd as sp

    per = 32 * blocks
    sizes = np.array([[a, s, c - a - s - w, w, 0, 0]] * S, dtype=np.int32)
    q, K, V = np.zeros((S, Hq, d), np.float32), np.zeros((S, Hkv, c, d), np.float32), np.full((S, Hkv, c, d), 2.0 ** 115, np.float32)
    q[..., 0], K[:, :, 0, 0], V[:, :, :per] = 1.0, 90.0, 0.0
    bf = lambda x: torch.from_numpy(x).cuda().to(torch.bfloat16)
    args = [bf(q), bf(K), bf(V), torch.from_numpy(sizes).cuda(), a, s, w, 1.0]
    ws = torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")
    eager = [t.clone() for t in sp.sepattn_decode(*args, ws=ws)]
    out = (torch.empty_like(eager[0]), torch.empty_like(eager[1]))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.sepattn_decode(*args, out=out, ws=ws)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, eager):
            assert torch.equal(x, y)
    want = (c - per) * 2.0 ** 115 * math.exp(-90.0)
    assert np.abs(eager[0].float().cpu().numpy() / want - 1).max() <= 2.0 ** -8
