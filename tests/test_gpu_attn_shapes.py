"""Forward and backward at the edges of what the attention kernels' launchers decide (tiles, slices of the
far keys' work, workgroup shapes), against the oracle.  Needs an MI355X."""
import math

import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import assert_close, assert_grads_close, dev, gpu_index, host, make_case, packed_index

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def run(B, Hq, Hkv, L, d, a, n, p, dtype, seed=1):
    """n: a window, or a list with one window per query head."""
    import paper_2412_12094_amd as sp

    tok, Q, K, V, dO = make_case(B, Hq, Hkv, L, d, p, dtype, seed)
    scale = 1.0 / math.sqrt(d)
    flags = oracle.mark_separators(tok, wl.SEPARATOR_IDS)
    q, k, v, do = (dev(x, dtype) for x in (Q, K, V, dO))
    _, idx, cnt, pre = gpu_index(sp, tok)
    heads = isinstance(n, list)
    fwd, bwd = (sp.sepattn_forward_headwise, sp.sepattn_backward_headwise) if heads else (sp.sepattn_forward, sp.sepattn_backward)
    O, LSE = fwd(q, k, v, idx, cnt, pre, a, n, scale)
    grads = bwd(q, k, v, O, LSE, do, idx, cnt, pre, a, n, scale)
    torch.cuda.synchronize()
    n, n_head = (1, n) if heads else (n, None)
    rO, rL = oracle.forward(Q, K, V, flags, a, n, scale, n_head=n_head)
    refs = oracle.backward(Q, K, V, dO, flags, a, n, scale, return_term_rss=True, n_head=n_head)
    assert_close(host(O), rO, dtype, "O")
    assert np.abs(host(LSE) - rL).max() <= (1e-4 if dtype == "fp32" else 2e-3)
    assert_grads_close(grads, refs, dtype)


def run_packed(L, Hq, Hkv, d, a, n, p, cu, seed=1):
    import paper_2412_12094_amd as sp

    tok, Q, K, V, dO = make_case(1, Hq, Hkv, L, d, p, "bf16", seed)
    scale = 1.0 / math.sqrt(d)
    cus = [np.array(cu, dtype=np.int32)]
    flags = oracle.mark_separators(tok, wl.SEPARATOR_IDS)
    _, ds, de, idx, cnt, pre = packed_index(sp, tok, cus, a)
    q, k, v, do = (dev(x, "bf16") for x in (Q, K, V, dO))
    O, LSE = sp.sepattn_forward_packed(q, k, v, ds, de, idx, cnt, pre, n, scale)
    grads = sp.sepattn_backward_packed(q, k, v, O, LSE, do, ds, de, idx, cnt, pre, n, scale)
    torch.cuda.synchronize()
    assert_grads_close(grads, oracle.backward_packed(Q, K, V, dO, flags, cus, a, n, scale, return_term_rss=True), "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p", [
    (1, 1, 1, 1, 64, 0, 1, 0.0),       # one query
    (2, 2, 1, 16, 128, 3, 4, 0.3),     # exactly one tile
    (1, 3, 1, 17, 64, 1, 40, 1.0),     # one row in the second tile; every key on the far list
    (1, 8, 2, 600, 128, 4, 8, 0.15),   # list tiles spread over several slices
    (3, 4, 4, 333, 64, 0, 16, 0.02),   # fewer items than one slice per list tile
])
def test_fp32_tiles_and_slices(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "fp32")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L,a,n,p", [
    (1, 7, 1, 33, 2, 5, 0.1),      # seven heads: one position in the second tile
    (2, 14, 2, 450, 4, 100, 0.1),  # seven heads, several segments and tiles; an odd number of blocks
    (1, 8, 1, 257, 0, 64, 0.2),    # eight heads: two groups of four
    (1, 2, 1, 65, 3, 200, 0.0),    # two heads; the window covers everything
    (1, 3, 3, 129, 1, 1, 0.3),     # one head; one position in the second tile; the smallest window
    (4, 8, 2, 128, 4, 32, 0.1),    # streams that end with a full block
])
def test_bf16_workgroup_shapes(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,a,n,p", [
    (4, 128, 32, 513, 4, 33, 0.1),                   # one position in the last tile, two workgroups per group of heads
    (16, 128, 32, 128, 1, 200, 0.1),                 # the fewest tiles for which eight waves are taken (2048 of four); more groups than compute units
    (16, 128, 32, 96, 1, 20, 0.1),                   # fewer: four waves
    (4, 128, 32, 513, 4, [33, 513, 1, 100] * 32, 0.1),  # a window per head
])
def test_bf16_eight_wave_forward_and_dq(B, Hq, Hkv, L, a, n, p):
    run(B, Hq, Hkv, L, 128, a, n, p, "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,p,nh", [
    (1, 8, 2, 1100, 128, 4, 0.08, [1100] * 4 + [48] * 4),      # a KV head that sees everything next to a short window
    (2, 12, 4, 700, 64, 3, 0.1, [33] * 6 + [700] * 3 + [1] * 3),  # three heads per KV head, two rows of the batch
    (1, 8, 2, 513, 64, 0, 0.0, [513] * 4 + [512] * 4),         # one position from full; no separators
    (2, 14, 2, 400, 128, 2, 0.1, [16] * 7 + [500] * 7),        # seven heads per tile; a window beyond the sequence
    (8, 128, 128, 66, 64, 1, 0.1, [66, 5, 20, 1] * 32),        # more groups than workgroups fit the chip
    (1, 4, 2, 31, 128, 1, 0.3, [31, 31, 2, 2]),                # less than one tile
])
def test_bf16_head_groups_by_work(B, Hq, Hkv, L, d, a, p, nh):
    run(B, Hq, Hkv, L, d, a, nh, p, "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p", [
    (1, 8, 1, 512, 128, 4, 512, 0.1),    # the shortest sequence whose keys are all listed
    (1, 8, 1, 511, 128, 4, 511, 0.1),    # one key fewer: band units
    (2, 8, 2, 1101, 64, 0, 4000, 0.0),   # a last list tile of 13 keys; no separators; a window beyond the sequence
    (1, 4, 1, 8200, 128, 4, 8200, 0.05),  # eight-wave dK/dV workgroups
])
def test_bf16_windows_of_the_whole_sequence(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L,a,n,p", [
    (1, 2, 2, 128, 0, 1, 0.0),     # one head: the waves' streams end with one key each, half a tile apart
    (2, 3, 3, 300, 4, 40, 0.1),    # the last tile's waves 2 and 3 lie past the sequence
    (1, 1, 1, 97, 0, 500, 0.0),    # one position in the last wave; the window covers everything
    (1, 4, 2, 191, 2, 33, 0.2),    # two heads: two position blocks per workgroup
    (1, 2, 1, 224, 100, 8, 0.05),  # more initial tokens than window
])
def test_bf16_waves_whose_streams_end_apart(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p", [
    (1, 8, 2, 600, 128, 4, 96, 0.1),    # a band unit in four parts of one head
    (1, 8, 2, 600, 64, 4, 96, 0.1),
    (1, 7, 1, 130, 64, 2, 100, 0.1),    # seven parts
    (2, 12, 2, 333, 128, 0, 64, 0.0),   # three parts of two heads; nothing on the list
    (4, 32, 8, 256, 128, 4, 128, 0.1),  # two parts of two heads
    (4, 32, 8, 257, 128, 4, 128, 0.1),  # one key more: whole units
    (21, 4, 1, 384, 128, 4, 360, 0.1),  # as many parts as workgroups
    (21, 4, 1, 385, 128, 4, 360, 0.1),  # one key more: two parts
    (1, 8, 1, 8200, 128, 4, 2000, 0.05),  # eight-wave workgroups
    (1, 8, 2, 8201, 128, 4, 256, 0.05),   # whole units: eight waves, the last unit has nine keys
])
def test_bf16_band_units_in_parts(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p", [
    (1, 32, 32, 1970, 128, 4, 189, 0.1),  # 31 units, 16 workgroups: one has a unit less and not all far work
    (1, 32, 32, 1970, 128, 4, 64, 0.9),   # ... enough of it for a slice each
    (1, 32, 32, 1970, 128, 0, 900, 0.01),  # ... so little that one workgroup has it all
    (1, 32, 32, 1090, 128, 4, 60, 0.1),   # 18 units: fourteen share it
    (2, 16, 16, 3000, 64, 4, 100, 0.2),   # 47 units, 24 workgroups
    (2, 16, 16, 3000, 64, 4, [100] * 8 + [300] * 8, 0.2),
    (1, 8, 8, 2646, 64, 4, 22, 0.1),      # 42 units, 43 workgroups: all but one share it, in parts that differ by an item
    (1, 32, 32, 1000, 128, 4, 20, 0.3),   # 16 units, 16 workgroups: none has a unit less
    (1, 16, 16, 2000, 64, 4, [20] * 15 + [30], 0.3),
])
def test_bf16_far_work_beside_uneven_band_units(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


# B, Hq, Hkv, L, d, a, n, p, packed from documents, dQ and dK/dV in one launch (asserted where the rule is tested on the host)
JOINT_CASES = [
    (1, 32, 8, 768, 128, 4, 100, 0.1, False, True),  # four heads, 192 query tiles: the last call with one launch
    (1, 32, 8, 769, 128, 4, 100, 0.1, False, False),  # one position more
    (2, 8, 4, 1536, 64, 0, 33, 0.1, False, True),    # two heads
    (2, 8, 4, 1537, 64, 0, 33, 0.1, False, False),
    (2, 8, 8, 1536, 64, 4, 70, 0.1, False, True),    # one head
    (2, 8, 8, 1537, 128, 4, 70, 0.1, False, False),
    (1, 32, 8, 768, 128, 4, 100, 0.1, True, True),
    (1, 32, 8, 769, 64, 4, 100, 0.1, True, False),
    (1, 8, 8, 3072, 64, 3, 70, 0.1, True, True),
    (1, 8, 8, 3073, 128, 3, 70, 0.1, True, False),
]


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p,docs,one", JOINT_CASES)
def test_bf16_backward_in_one_launch_and_in_two(B, Hq, Hkv, L, d, a, n, p, docs, one):
    if docs:
        run_packed(L, Hq, Hkv, d, a, n, p, [0, L // 3, L // 3 + 5, L // 2, L])
    else:
        run(B, Hq, Hkv, L, d, a, n, p, "bf16")


# one row: dQ and dK/dV in one launch; four: in two (asserted where the rule is tested on the host)
JOINT_ROWS = [(32, 8, 700, 128, 4, 100), (32, 8, 700, 64, 4, 30), (8, 4, 3000, 128, 0, 33), (12, 12, 2011, 64, 4, 64)]


@pytest.mark.parametrize("Hq,Hkv,L,d,a,n", JOINT_ROWS)
def test_bf16_dq_of_one_launch_and_of_two(Hq, Hkv, L, d, a, n):
    """A row's dQ is the same bits in a call that runs dQ beside dK/dV and as part of a batch that does not; dK and dV, whose far work is
    cut for other numbers of workgroups, differ by no more than two roundings to bf16 and the order of fp32 sums."""
    import paper_2412_12094_amd as sp

    B, scale = 4, 1.0 / math.sqrt(d)
    tok, Q, K, V, dO = make_case(B, Hq, Hkv, L, d, 0.1, "bf16", 1)
    q, k, v, do = (dev(x, "bf16") for x in (Q, K, V, dO))
    _, idx, cnt, pre = gpu_index(sp, tok)
    O, LSE = sp.sepattn_forward(q, k, v, idx, cnt, pre, a, n, scale)
    call = lambda b: sp.sepattn_backward(*(x[b].contiguous() for x in (q, k, v, O, LSE, do, idx, cnt, pre)), a, n, scale)
    two = call(slice(0, B))
    for b in range(B):
        one = call(slice(b, b + 1))
        assert torch.equal(one[0][0], two[0][b])
        for x, y in zip(one[1:], two[1:]):
            assert np.abs(host(x[0]) - host(y[b])).max() <= 2.0 ** -7 * np.abs(host(y[b])).max()


def test_bf16_backward_in_one_launch_is_recorded_once():
    """Two handles do not both cover the launch that has dQ and dK/dV side by side: that counts as dK/dV, and the row values in front
    of it, which read and write a fraction of its bytes, as dQ."""
    import paper_2412_12094_amd as sp

    B, H, L, d, a, n = 1, 12, 2011, 128, 4, 64
    tok, Q, K, V, dO = make_case(B, H, H, L, d, 0.1, "bf16", 1)
    q, k, v, do = (dev(x, "bf16") for x in (Q, K, V, dO))
    _, idx, cnt, pre = gpu_index(sp, tok)
    scale = 1.0 / math.sqrt(d)
    O, LSE = sp.sepattn_forward(q, k, v, idx, cnt, pre, a, n, scale)
    us = {}
    for name in ("bwd_dq", "bwd_dkv"):
        prof = sp.sepattn_profile_begin(sp.KERNEL_IDS[name], 40)
        for _ in range(40):
            sp.sepattn_backward(q, k, v, O, LSE, do, idx, cnt, pre, a, n, scale)
        torch.cuda.synchronize()
        ms = sp.sepattn_profile_end(prof)
        assert len(ms) == 40
        us[name] = 1e3 * float(np.median(ms))
    assert us["bwd_dq"] <= 0.6 * us["bwd_dkv"], us


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L,a,n,p", [
    (1, 4, 1, 2560, 4, 2560, 0.1),                         # four heads; the shortest window that may end before the sequence
    (1, 3, 3, 1301, 0, 1301, 0.05),                        # full windows are split from some 1300 positions on
    (1, 4, 2, 1500, 4, 1500, 0.1),                         # two heads
    (1, 4, 2, 1500, 4, 1499, 0.1),                         # a position short of full: whole
    (1, 8, 2, 1430, 4, [1430] * 4 + [30, 7, 1, 64], 0.1),  # one group full and split, the other not
    (1, 2, 1, 2627, 0, 1 << 20, 0.0),                      # two heads, ragged; windows longer than any sequence
    (2, 1, 1, 2689, 4, 2570, 0.1),                         # one head: waves that end before the second half
    (1, 4, 2, 4000, 2, 2600, 0.3),                         # windows that end: many split tiles equally long
    (1, 8, 2, 2600, 4, [2600] * 4 + [40, 7, 1, 64], 0.1),  # one group split, the other not
])
def test_bf16_streams_in_two_parts(B, Hq, Hkv, L, d, a, n, p):
    run(B, Hq, Hkv, L, d, a, n, p, "bf16")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (2, 2), (7, 1)])
@pytest.mark.parametrize("shape", ["grow", "jump"])
def test_bf16_forward_raises_its_maximum(Hq, Hkv, d, shape):
    """Scores that grow along the keys, from -s to s, steadily (every few blocks outgrow the maximum before them) or at
    once (the first exponential after the jump overflows); half the heads see them fall instead.  |V| <= 2: rounding P and O
    to bf16 gives at most 2 * 2^-9 + 2^-8 < 0.008 in O; 2e-3 in LSE is the other tests' bound, |LSE| stays below 110."""
    import paper_2412_12094_amd as sp

    L, a, n, p, top = 700, 4, 300, 0.1, 100.0
    scale = 1.0 / math.sqrt(d)
    tok, Q, K, V, _ = make_case(1, Hq, Hkv, L, d, p, "bf16", 5)
    ramp = np.linspace(-1, 1, L) if shape == "grow" else np.where(np.arange(L) < L // 2, -1.0, 1.0)
    u = np.where(np.arange(d) % 2, 1.0, -1.0)
    sign = np.where(np.arange(Hq) % 2, -1.0, 1.0)
    Q = (0.05 * Q + sign[None, :, None, None] * u).astype(np.float32)
    K = (0.05 * K + (top / math.sqrt(d) * ramp)[None, None, :, None] * u).astype(np.float32)
    q, k, v = (dev(x, "bf16") for x in (Q, K, np.clip(V, -2, 2)))
    _, idx, cnt, pre = gpu_index(sp, tok)
    O, LSE = sp.sepattn_forward(q, k, v, idx, cnt, pre, a, n, scale)
    torch.cuda.synchronize()
    rO, rL = oracle.forward(host(q), host(k), host(v), oracle.mark_separators(tok, wl.SEPARATOR_IDS), a, n, scale)
    assert np.abs(host(O) - rO).max() <= 8e-3
    assert np.abs(host(LSE) - rL).max() <= 2e-3
