"""Entry points that write the whole of a fresh buffer (`_filled`, `_zeroed`): what the plain call writes, bit for bit, and the
given value everywhere else, over memory that holds something else.  Needs an MI355X."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 64  # entries behind a buffer that nothing may touch


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_12094_amd as sp_

    sp_.load()
    return sp_


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


# a token, a wave, a chunk of 2048 and its halves, the one-launch limits of 8192 and 32768 tokens, each with its neighbours; a wave with one
# token of its own (1025 and 3073)
@pytest.mark.parametrize("B,L,p", [(1, 1, 0.5), (2, 63, 0.3), (3, 1023, 0.1), (2, 1025, 0.0), (2, 1025, 0.5), (2, 3073, 0.4), (2, 2048, 1.0), (3, 2049, 0.1), (2, 4095, 0.08),
                                   (3, 6145, 0.2), (2, 8192, 0.08), (2, 8193, 0.08), (1, 32768, 0.1), (2, 32769, 0.1)])
def test_list_is_filled_behind_its_last_separator(sp, B, L, p):
    lib = sp.load()
    tok = wl.make_token_ids(B, L, p, 7 + L).astype(np.int32)
    ids = np.concatenate([wl.SEPARATOR_IDS, wl.SEPARATOR_IDS[:1]]).astype(np.int32)  # one id twice
    flags = oracle.mark_separators(tok, wl.SEPARATOR_IDS)
    t = torch.from_numpy(tok).cuda()
    ws = torch.empty(max(256, lib.sepattn_compact_workspace_bytes(B, L)), dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    most = int(flags.sum(1).max())
    for cap in sorted({1, max(1, most // 2), max(1, most), L, L + 1, L + 3000}):
        for fill in (-1, 12345):
            want_idx, want_cnt, want_pre = oracle.compact_indices(flags, cap=cap)
            want_idx = np.where(np.arange(cap)[None, :] < np.minimum(want_cnt, cap)[:, None], want_idx, fill)
            for mark in (True, False):
                sep = torch.full((B * L + GUARD,), 9, dtype=torch.uint8, device="cuda")
                idx = torch.full((B * cap + GUARD,), -77, dtype=torch.int32, device="cuda")
                cnt = torch.full((B,), -77, dtype=torch.int32, device="cuda")
                pre = torch.full((B * (L + 1) + GUARD,), -77, dtype=torch.int32, device="cuda")
                if mark:
                    rc = lib.sepattn_mark_compact_filled(ptr(t), B, L, ids.ctypes.data_as(ctypes.c_void_p), len(ids), ptr(sep), ptr(idx),
                                                         cap, ptr(cnt), ptr(pre), fill, ptr(ws), ws.numel(), st)
                else:
                    sep[:B * L] = torch.from_numpy(flags).cuda().reshape(-1)
                    rc = lib.sepattn_compact_indices_filled(ptr(sep), B, L, ptr(idx), cap, ptr(cnt), ptr(pre), fill, ptr(ws), ws.numel(), st)
                assert rc == 0
                sep, idx, cnt, pre = (x.cpu().numpy() for x in (sep, idx, cnt, pre))
                assert np.array_equal(sep[:B * L].reshape(B, L), flags) and (sep[B * L:] == 9).all()
                assert np.array_equal(idx[:B * cap].reshape(B, cap), want_idx) and (idx[B * cap:] == -77).all()
                assert np.array_equal(cnt, want_cnt)
                assert np.array_equal(pre[:B * (L + 1)].reshape(B, L + 1), want_pre) and (pre[B * (L + 1):] == -77).all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("S,Hkv,L,d,a,s,w,c,nw,p", [
    (2, 2, 300, 128, 4, 40, 16, 4 + 40 + 90, 70, 0.2), (3, 1, 200, 64, 3, 100, 8, 3 + 100 + 40, 40, 0.1),
    (1, 2, 50, 128, 4, 10, 4, 4 + 10 + 30, 0, 0.3), (2, 1, 3, 64, 4, 10, 4, 4 + 10 + 30, 0, 0.5),
    (1, 3, 130, 128, 0, 5, 2, 0 + 5 + 129 + 1, 129, 0.0), (2, 1, 700, 128, 4, 64, 32, 4 + 64 + 301, 300, 1.0)])
def test_caches_are_zero_beyond_their_sizes(sp, dtype, S, Hkv, L, d, a, s, w, c, nw, p):
    lib = sp.load()
    tok = torch.from_numpy(wl.make_token_ids(S, L, p, L).astype(np.int32)).cuda()
    sep, idx, cnt, pre = sp.sepattn_mark_compact(tok, wl.SEPARATOR_IDS.tolist())
    g = torch.Generator(device="cuda").manual_seed(L)
    K, V = (torch.randn((S, Hkv, L, d), device="cuda", generator=g).to(dtype) for _ in range(2))
    n_row, room = S * Hkv * c * d, c - a - s

    def buffers(value, flag, size):
        return [torch.full((n_row + GUARD,), value, dtype=dtype, device="cuda") for _ in range(2)] + \
            [torch.full((S * room + GUARD,), flag, dtype=torch.uint8, device="cuda"), torch.full((S * 6,), size, dtype=torch.int32, device="cuda")]

    params = sp.SepkvParams(S, Hkv, Hkv, d, a, s, w, c, 1.0, sp.SEPATTN_BF16 if dtype == torch.bfloat16 else sp.SEPATTN_FP32)
    want, got = buffers(0, 0, 0), buffers(5, 9, -1)
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for fn, x in ((lib.sepkv_fill_from_prefill, want), (lib.sepkv_fill_from_prefill_zeroed, got)):
        assert fn(ctypes.byref(params), L, nw, ptr(K), ptr(V), ptr(sep), ptr(idx), idx.shape[1], ptr(pre), *[ptr(y) for y in x], st) == 0
    for x, y, n, guard in zip(want, got, (n_row, n_row, S * room, S * 6), (5, 5, 9, -1)):
        assert torch.equal(x[:n], y[:n]) and bool((y[n:] == guard).all())
