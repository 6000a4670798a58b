"""What the binding's extension module refuses before it allocates or launches anything.  Needs no GPU: the
arguments are fake tensors, which have a shape, a type and a device and no memory."""
import pytest

torch = pytest.importorskip("torch")
from torch._subclasses.fake_tensor import FakeTensorMode  # noqa: E402

B, HQ, HKV, L, D = 2, 4, 2, 64, 64
NEW = None  # the call allocates its outputs; without a GPU that fails, with another error than a check


@pytest.fixture(scope="module")
def bd():
    from paper_2412_12094_amd import binding

    binding._native()
    return binding


def fake(*shape, dtype=torch.int32, device="cuda"):
    with FakeTensorMode():
        return torch.empty(*shape, dtype=dtype, device=device)


def attention():
    q, k = fake(B, HQ, L, D, dtype=torch.bfloat16), fake(B, HKV, L, D, dtype=torch.bfloat16)
    return q, k, fake(B, HQ, L, dtype=torch.float32), (fake(B, L), fake(B), fake(B, L + 1))


@pytest.mark.parametrize("start,end", [
    ((L,), (L,)),              # one row's bounds without the batch dimension
    ((1, L), (1, L)),          # one row for a batch of two
    ((B, L - 1), (B, L - 1)),  # a position short
    ((B, L), (L,)),            # only one of the two has the call's shape
    ((B, L), (1, L)),
    ((B, L, 1), (B, L, 1)),
    ((L, B), (L, B)),
])
@pytest.mark.parametrize("call", ["forward", "backward"])
def test_packed_bounds_have_the_shape_of_the_batch(bd, call, start, end):
    q, k, lse, index = attention()
    bounds = fake(*start), fake(*end)
    with pytest.raises(AssertionError, match="doc_start"):
        if call == "forward":
            bd.sepattn_forward_packed(q, k, k, *bounds, *index, 4, 0.1, NEW, NEW)
        else:
            bd.sepattn_backward_packed(q, k, k, q, lse, q, *bounds, *index, 4, 0.1, NEW, NEW)


@pytest.mark.parametrize("call", ["forward", "backward"])
def test_packed_bounds_are_int32(bd, call):
    q, k, lse, index = attention()
    bounds = fake(B, L), fake(B, L, dtype=torch.int64)
    with pytest.raises(AssertionError, match="doc_start"):
        if call == "forward":
            bd.sepattn_forward_packed(q, k, k, *bounds, *index, 4, 0.1, NEW, NEW)
        else:
            bd.sepattn_backward_packed(q, k, k, q, lse, q, *bounds, *index, 4, 0.1, NEW, NEW)


class Watched:
    """Not a tensor; logs when its type is looked at and when it is released."""

    def __init__(self, log):
        self.log = log

    @property
    def __class__(self):
        self.log.append("looked at")
        return object

    def __del__(self):
        self.log.append("released")


def cache_call():
    q, Kc = fake(1, HQ, D, dtype=torch.bfloat16), fake(1, HKV, 32, D, dtype=torch.bfloat16)
    return q, Kc, Kc, fake(1, 6), 4, 8, 8, 0.1


@pytest.mark.parametrize("make", [tuple, list, iter, lambda items: (x for x in items)])
def test_outputs_live_until_the_call_returns(bd, make):
    """`out` may be any iterable, and it may be the only owner of its items."""
    log = []
    with pytest.raises(TypeError, match="tensor") as err:
        bd.sepattn_decode_noalloc(*cache_call(), make(Watched(log) for _ in range(2)))
    assert log[0] == "looked at"
    del err  # (the traceback's frames hold a tuple or a list)
    assert log[-2:] == ["released"] * 2 and log.count("released") == 2


@pytest.mark.parametrize("n", [0, 1, 3])
def test_outputs_are_counted(bd, n):
    q, k, lse, index = attention()
    with pytest.raises(ValueError):
        bd.sepattn_forward(q, k, k, *index, 1, 4, 0.1, (q,) * n)
    with pytest.raises(TypeError):
        bd.sepattn_forward(q, k, k, *index, 1, 4, 0.1, 3)


def test_document_bounds_take_a_sequence(bd):
    cu, row = fake(3), fake(L, dtype=torch.int64)
    with pytest.raises(TypeError):  # an iterator would come back exhausted
        bd.sepattn_doc_bounds(cu, L, 2, None, iter((row, row)))
    with pytest.raises(ValueError, match="number of tensors"):
        bd.sepattn_doc_bounds(cu, L, 2, None, (row,))
    with pytest.raises(ValueError, match="GPU"):  # taken apart; refused for what the second item is
        bd.sepattn_doc_bounds(cu, L, 2, None, [row, fake(L, device="cpu"), row])


def test_decode_with_positions_needs_the_table(bd):
    """Without one it would be the decode without positions."""
    q, Kc, Vc, sizes, *kv = cache_call()
    with pytest.raises(TypeError):
        bd.sepattn_decode_rope(q, Kc, Vc, sizes, None, *kv, (q, fake(1, HQ, dtype=torch.float32)))
    with pytest.raises(AssertionError, match="rope_table"):
        bd.sepattn_decode_rope(q, Kc, Vc, sizes, fake(32, 2, D, dtype=torch.float32), *kv)


def test_flags_and_lists_are_read_as_python_does(bd):
    tokens, flags = fake(B, L), fake(B, L, dtype=torch.uint8)
    with pytest.raises(RuntimeError, match="ambiguous"):  # bool() of this raises
        bd.sepattn_compact_indices(flags, want_prefix=torch.zeros(2))
    with pytest.raises(TypeError):  # no length
        bd.sepattn_mark_separators(tokens, (x for x in [1, 2]))
    ids = [1, 2, 3]

    class Clears:
        def __int__(self):
            ids.clear()
            return 1

    ids[0] = Clears()
    q, k, _, index = attention()
    with pytest.raises(AssertionError, match="n_per_head"):  # the three items that the list had
        bd.sepattn_forward_headwise(q, k, k, *index, 1, ids, 0.1)
    with pytest.raises(ValueError, match="wrong number"):  # float() takes the text, the outputs are looked at next
        bd.sepattn_forward(q, k, k, *index, 1, 4, "0.1", ())


def test_errors_of_torch_keep_their_class(bd):
    q, k, _, (idx, cnt, pre) = attention()
    with pytest.raises(IndexError):  # the list has no second dimension
        bd.sepattn_forward(q, k, k, fake(L), cnt, pre, 1, 4, 0.1)


def test_calls_go_to_the_library_that_was_loaded(bd, monkeypatch, tmp_path):
    import shutil

    from paper_2412_12094_amd import _native

    other = str(tmp_path / "libsepattn.so")
    shutil.copy(bd.LIB_PATH, other)
    bound = []
    monkeypatch.setattr(_native, "bind", lambda path, raise_error: bound.append(path))
    monkeypatch.setattr(bd, "_lib", None)
    monkeypatch.setattr(bd, "_calls", None)
    bd.load(other)  # the first one loaded is the one in use
    bd._native()
    bd.load()
    bd._native()
    assert bound == [other]
    bd.load(bd.LIB_PATH)  # ... until the usual one is asked for
    bd._native()
    assert bound == [other, bd.LIB_PATH]
