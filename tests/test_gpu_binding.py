"""How the binding's extension module calls the library: without the interpreter lock, with the caller's outputs alive.
Needs an MI355X."""
import re
import subprocess

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

S, HQ, HKV, L, D = 2, 4, 2, 32, 64
KV = (4, 8, 8)  # a, s, w


@pytest.fixture(scope="module")
def bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_12094_amd import binding

    binding._native()
    return binding


def z(*shape, dtype=torch.int32):
    return torch.zeros(*shape, dtype=dtype, device="cuda")


def calls(bd):
    bf, f32, u8 = torch.bfloat16, torch.float32, torch.uint8
    q, k, lse = z(S, HQ, L, D, dtype=bf), z(S, HKV, L, D, dtype=bf), z(S, HQ, L, dtype=f32)
    index = z(S, L), z(S), z(S, L + 1)
    bounds = z(S, L), z(S, L)
    q1, flags, sizes, table = z(S, HQ, D, dtype=bf), z(S, L - 12, dtype=u8), z(S, 6), z(L, 2, D // 2, dtype=f32)
    row = z(S, HKV, D, dtype=bf)
    return {
        "sepattn_mark_separators": lambda: bd.sepattn_mark_separators(z(S, L), [1]),
        "sepattn_compact_indices": lambda: bd.sepattn_compact_indices(z(S, L, dtype=u8)),
        "sepattn_mark_compact": lambda: bd.sepattn_mark_compact(z(S, L), [1]),
        "sepattn_doc_bounds": lambda: bd.sepattn_doc_bounds(z(2), L),
        "sepattn_forward": lambda: bd.sepattn_forward(q, k, k, *index, 1, 4, 0.1),
        "sepattn_forward_headwise": lambda: bd.sepattn_forward_headwise(q, k, k, *index, 1, [4] * HQ, 0.1),
        "sepattn_forward_packed": lambda: bd.sepattn_forward_packed(q, k, k, *bounds, *index, 4, 0.1),
        "sepattn_backward": lambda: bd.sepattn_backward(q, k, k, q, lse, q, *index, 1, 4, 0.1),
        "sepattn_backward_headwise": lambda: bd.sepattn_backward_headwise(q, k, k, q, lse, q, *index, 1, [4] * HQ, 0.1),
        "sepattn_backward_packed": lambda: bd.sepattn_backward_packed(q, k, k, q, lse, q, *bounds, *index, 4, 0.1),
        "sepattn_decode": lambda: bd.sepattn_decode(q1, k, k, sizes, *KV, 0.1),
        "sepattn_decode_rope": lambda: bd.sepattn_decode_rope(q1, k, k, sizes, table, *KV, 0.1),
        "sepattn_decode_noalloc": lambda: bd.sepattn_decode_noalloc(q1, k, k, sizes, *KV, 0.1, (q1, None)),
        "sepkv_append": lambda: bd.sepkv_append(row, row, z(S, dtype=u8), k, k, flags, sizes, HQ, *KV),
        "sepkv_evict_window": lambda: bd.sepkv_evict_window(k, k, flags, sizes, HQ, *KV),
        "sepkv_fill_from_prefill": lambda: bd.sepkv_fill_from_prefill(k, k, z(S, L, dtype=u8), *index[::2], HQ, *KV, L, 8),
    }


def test_the_library_is_called_without_the_interpreter_lock(bd, tmp_path):
    """Against a stand-in for the library that launches nothing and answers whether the lock is held."""
    from test_host_abi import declared_functions

    names = declared_functions()
    source = tmp_path / "stand_in.c"
    source.write_text("int PyGILState_Check(void);\n" + "\n".join(
        f"unsigned long {n}(void) {{ return 256; }}" if n.endswith("_bytes") else f"int {n}(void) {{ return PyGILState_Check() ? 98 : 99; }}"
        for n in names))
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(tmp_path / "stand_in.so"), str(source)], check=True)
    table = calls(bd)
    torch.cuda.synchronize()
    bd._native().bind(str(tmp_path / "stand_in.so"), bd._raise_status)
    status = {}
    try:
        for name, call in table.items():
            with pytest.raises(bd.SepattnError, match=name) as err:
                call()
            status[name] = err.value.status
    finally:
        bd._native().bind(bd.LIB_PATH, bd._raise_status)
    assert status == {name: 99 for name in table}
    bound = set(re.findall(r"X\((\w+)\)", open(bd.__file__.replace("binding.py", "csrc/native_binding.cpp")).read()))
    assert set(table) == {n for n in bound if n.startswith("sep") and not n.endswith("_bytes")}


@pytest.mark.parametrize("make", [list, iter, lambda items: map(torch.empty_like, items)])
def test_outputs_of_any_iterable_are_written(bd, make):
    torch.manual_seed(0)
    q, k = (torch.randn(S, h, L, D, device="cuda").to(torch.bfloat16) for h in (HQ, HKV))
    _, *index = bd.sepattn_mark_compact(torch.randint(0, 4, (S, L), dtype=torch.int32, device="cuda"), [1])
    want = bd.sepattn_forward(q, k, k, *index, 1, 4, 0.1)
    got = bd.sepattn_forward(q, k, k, *index, 1, 4, 0.1, make([torch.empty_like(t) for t in want]))
    filler = [torch.full_like(t, 7.0) for t in want for _ in range(2)]  # takes whatever memory has been given back
    want_g = bd.sepattn_backward(q, k, k, *want, q, *index, 1, 4, 0.1)
    got_g = bd.sepattn_backward(q, k, k, *got, q, *index, 1, 4, 0.1, make([torch.empty_like(t) for t in want_g]))
    filler += [torch.full_like(t, 7.0) for t in want_g for _ in range(2)]
    for a, b in zip((*want, *want_g), (*got, *got_g), strict=True):
        assert torch.equal(a, b)


def test_a_failed_allocation_is_an_out_of_memory_error(bd):
    """The class that programs catch to give memory back and try again."""
    q, k = z(1, 64, 4096, 128, dtype=torch.bfloat16), z(1, 8, 4096, 128, dtype=torch.bfloat16)
    index = z(1, 4096), z(1), z(1, 4097)
    torch.cuda.empty_cache()
    allowed = torch.cuda.memory_reserved() + (1 << 20)  # no room for the outputs (64 MiB)
    torch.cuda.set_per_process_memory_fraction(allowed / torch.cuda.get_device_properties(0).total_memory)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            bd.sepattn_forward(q, k, k, *index, 4, 64, 0.1)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert bd.sepattn_forward(q, k, k, *index, 4, 64, 0.1)[0].shape == q.shape
