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
