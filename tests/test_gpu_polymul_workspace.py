"""GPU: a product whose workspace the caller brings."""
import ctypes

import pytest

from paper_2410_05934_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2410_05934_amd as ntt  # noqa: E402


def test_product_workspace_from_the_caller():
    """Too small or missing: the library allocates its own; large enough: used."""
    mods = synth.primes_below(1 << 50, 1 << 17, 2)
    N = 1 << 15
    plan = ntt.Plan(N, mods, 64)
    a = torch.randint(0, mods[-1], (2, 2, N), device="cuda")
    b = torch.randint(0, mods[-1], (2, 2, N), device="cuda")
    want = torch.empty_like(a)
    plan.polymul(want, a, b)
    need = ctypes.c_uint64()
    assert ntt.lib().ntt_polymul_workspace(plan._h, 2, ctypes.byref(need)) == 0
    assert need.value == a.numel() * 8
    ws = torch.full((a.numel() + 16,), -1, dtype=torch.int64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for ptr, size in ((None, 0), (ws.data_ptr(), need.value - 8), (ws.data_ptr(), need.value)):
        out = torch.empty_like(a)
        assert ntt.lib().ntt_polymul_ws(plan._h, out.data_ptr(), a.data_ptr(), b.data_ptr(), 2, ptr,
                                        size, stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert bool((ws[a.numel():] == -1).all())
        assert bool((ws[:a.numel()] == -1).all()) == (size < need.value)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = torch.empty_like(a)
    plan.polymul(out, a, b, stream=side)
    side.synchronize()
    assert torch.equal(out, want)


def test_product_on_any_object_with_a_stream_handle():
    """A two-pass product takes what every other call takes as its stream."""
    mods = synth.primes_below(1 << 50, 1 << 17, 2)
    N = 1 << 15
    plan = ntt.Plan(N, mods, 64)
    a = torch.randint(0, mods[-1], (1, 2, N), device="cuda")
    b = torch.randint(0, mods[-1], (1, 2, N), device="cuda")
    want = plan.polymul(torch.empty_like(a), a, b)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    class Handle:
        cuda_stream = side.cuda_stream

    for stream in (Handle(), torch.cuda.ExternalStream(side.cuda_stream)):
        out = torch.zeros_like(a)
        side.wait_stream(torch.cuda.current_stream())
        plan.polymul(out, a, b, stream=stream)
        side.synchronize()
        assert torch.equal(out, want)


def test_workspace_that_overlaps_or_is_misaligned_is_refused():
    """Before any launch, and only where the call would use it."""
    mods = synth.primes_below(1 << 50, 1 << 17, 1)
    N = 1 << 15
    plan = ntt.Plan(N, mods, 64)
    block = torch.zeros((4, N), dtype=torch.int64, device="cuda")
    a, b, out, ws = (block[i] for i in range(4))
    bad = ntt.lib().ntt_polymul_ws
    stream, size = torch.cuda.current_stream().cuda_stream, N * 8
    for ptr in (a.data_ptr(), b.data_ptr(), out.data_ptr(), out.data_ptr() + 8, ws.data_ptr() - 8,
                ws.data_ptr() + 4):
        assert bad(plan._h, out.data_ptr(), a.data_ptr(), b.data_ptr(), 1, ptr, size, stream) == 1
    assert bad(plan._h, out.data_ptr(), a.data_ptr(), b.data_ptr(), 1, ws.data_ptr(), size, stream) == 0
    # too small: not used, so not looked at
    assert bad(plan._h, out.data_ptr(), a.data_ptr(), b.data_ptr(), 1, ws.data_ptr() + 4, 8, stream) == 0
    torch.cuda.synchronize()
