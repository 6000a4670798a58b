"""fp32 path: an infinity or a NaN in one position reaches the rows that see that position and no others.
Needs an MI355X."""
import math

import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import dev, gpu_index, host, make_case, packed_index

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B, HQ, HKV, L, A = 1, 4, 2, 150, 0


def visible(flags, cus, heads):
    """[Hq, L, L]: query i of head h sees key j"""
    rows = [oracle.mask(flags[0], A, n) for n in heads]
    M = np.stack(rows).astype(bool)
    if cus is not None:
        doc = np.searchsorted(cus, np.arange(L), side="right")
        M &= doc[:, None] == doc[None, :]
    return M


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("where", ["Q", "K", "V", "dO"])
@pytest.mark.parametrize("t", [0, 37, L - 1])  # the row that padding loads; inside a block; the last row, in a ragged block
@pytest.mark.parametrize("form,d", [("plain", 64), ("plain", 128), ("headwise", 64), ("packed", 64)])
def test_non_finite_values_stay_with_the_rows_that_see_them(form, d, t, where, value):
    import paper_2412_12094_amd as sp

    tok, Q, K, V, dO = make_case(B, HQ, HKV, L, d, 0.1, "fp32", 5)
    x = {"Q": Q, "K": K, "V": V, "dO": dO}[where]
    scale = 1.0 / math.sqrt(d)
    flags = oracle.mark_separators(tok, wl.SEPARATOR_IDS)
    tok[:, t] = tok[flags == 0][0]  # not a separator: the rows beyond its window do not see it
    flags = oracle.mark_separators(tok, wl.SEPARATOR_IDS)
    heads = [9, 20, 33, 5] if form == "headwise" else [20] * HQ
    cus = np.array([[0, 30, 77, L]], dtype=np.int32) if form == "packed" else None
    if form == "packed":
        refs = (*oracle.forward_packed(Q, K, V, flags, cus, A, 20, scale), *oracle.backward_packed(Q, K, V, dO, flags, cus, A, 20, scale))
    else:
        refs = (*oracle.forward(Q, K, V, flags, A, 20, scale, n_head=heads), *oracle.backward(Q, K, V, dO, flags, A, 20, scale, n_head=heads))
    x[:, :, t, 3::5] = value
    q, k, v, do = (dev(y, "fp32") for y in (Q, K, V, dO))
    if form == "packed":
        _, ds, de, *index = packed_index(sp, tok, cus, A)
        O, LSE = sp.sepattn_forward_packed(q, k, v, ds, de, *index, 20, scale)
        grads = sp.sepattn_backward_packed(q, k, v, O, LSE, do, ds, de, *index, 20, scale)
    else:
        _, *index = gpu_index(sp, tok)
        O, LSE = sp.sepattn_forward_headwise(q, k, v, *index, A, heads, scale)
        grads = sp.sepattn_backward_headwise(q, k, v, O, LSE, do, *index, A, heads, scale)
        if form == "plain":
            same = sp.sepattn_forward(q, k, v, *index, A, 20, scale)
            same_grads = sp.sepattn_backward(q, k, v, O, LSE, do, *index, A, 20, scale)
            for a, b in zip((O, LSE, *grads), (*same, *same_grads), strict=True):
                assert torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))
    M = visible(flags, None if cus is None else cus[0], heads)
    if where in ("K", "V"):
        rows = M[:, :, t]  # [Hq, L] the rows whose result may be non-finite
    else:
        rows = np.zeros((HQ, L), dtype=bool)
        rows[:, t] = True
    fwd_rows = rows & (where != "dO")
    keys = np.stack([np.any([(rows[h, :, None] & M[h]).any(axis=0) for h in range(kv * 2, kv * 2 + 2)], axis=0) for kv in range(HKV)])
    assert (~rows).sum() > 0.5 * rows.size and (~keys).sum() > 0.25 * keys.size
    for name, got, ref, hit in zip(("O", "LSE", "dQ", "dK", "dV"), (O, LSE, *grads), refs, (fwd_rows, fwd_rows, rows, keys, keys), strict=True):
        got = host(got)[0]
        assert np.isfinite(got[~hit]).all(), (name, np.argwhere(~np.isfinite(got.reshape(*hit.shape, -1)).all(-1) & ~hit)[:8])
        assert np.abs(got[~hit] - ref[0][~hit]).max() <= 1e-4, name
    first = {"Q": O, "K": O, "V": O, "dO": grads[0]}[where]
    assert not np.isfinite(host(first)[0][rows]).all(axis=-1).any()  # ... and those rows do show it
