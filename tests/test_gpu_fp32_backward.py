"""fp32 backward: dQ and dK/dV in one launch or in two give the same bits, whatever the workspace held.  Needs an MI355X."""
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_12094_amd as sp_

    sp_.load()
    return sp_


# one launch (the last column: yes): a tile, a ragged row, list tiles in many slices, the last size below the line at d = 64 and 128; two:
# the first above
CASES = [
    (1, 1, 1, 1, 64, 0, 1, 0.0, True), (1, 2, 1, 17, 128, 4, 3, 0.5, True), (1, 2, 1, 512, 64, 4, 64, 0.125, True),
    (2, 4, 1, 999, 64, 3, 40, 0.3, True), (1, 4, 4, 300, 128, 0, 100, 0.1, True), (1, 14, 14, 544, 64, 4, 64, 0.1, True),
    (1, 8, 2, 1024, 128, 4, 64, 0.1, True), (1, 8, 8, 1024, 64, 4, 16, 0.1, False), (1, 8, 8, 656, 128, 4, 16, 0.1, False)]


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,p,one", CASES)
def test_one_launch_and_two_give_the_same_bits(sp, B, Hq, Hkv, L, d, a, n, p, one):  # one: asserted where the rule is tested on the host
    g = torch.Generator(device="cuda").manual_seed(L)
    tok = torch.from_numpy(wl.make_token_ids(B, L, p, L).astype("int32")).cuda()
    _, idx, cnt, pre = sp.sepattn_mark_compact(tok, wl.SEPARATOR_IDS.tolist())
    rnd = lambda h: torch.randn((B, h, L, d), device="cuda", generator=g)
    Q, K, V, dO, scale = rnd(Hq), rnd(Hkv), rnd(Hkv), rnd(Hq), d ** -0.5
    O, LSE = sp.sepattn_forward(Q, K, V, idx, cnt, pre, a, n, scale)
    ws = torch.zeros(sp.sepattn_backward_workspace_bytes(Q, K, a, n, scale, L), dtype=torch.uint8, device="cuda")
    out = tuple(torch.empty_like(x) for x in (Q, K, V))
    call = lambda: sp.sepattn_backward(Q, K, V, O, LSE, dO, idx, cnt, pre, a, n, scale, out=out, ws=ws)
    # a captured launch has no number of its own to count slices under: always two launches
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    want = None
    for k in range(3):
        for x in out:
            x.fill_(float("nan"))
        ws.random_(0, 256, generator=g) if k else ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        if want is None:
            want = [x.clone() for x in out]
            assert all(bool(torch.isfinite(x).all()) for x in want)
        assert all(torch.equal(x, y) for x, y in zip(out, want))
    for k in range(6):  # what the workspace holds: noise, one value, what the call before left
        if k < 4:
            ws.random_(0, 256, generator=g) if k % 2 else ws.fill_(k)
        for x in out:
            x.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want)), k
