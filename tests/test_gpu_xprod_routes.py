"""GPU: external products whose workgroup would need more than 64 KiB of LDS run in
one launch only where that is faster than the separate steps; both give the
oracle's words."""
import numpy as np
import pytest

import oracle
from paper_2410_05934_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2410_05934_amd as ntt  # noqa: E402
from paper_2410_05934_amd.tensors import empty_device, to_device, to_host  # noqa: E402


def _one_launch(run):
    """Whether every kernel of run() is the fused one."""
    ntt.stats_reset()
    ntt.stats_enable(True)
    try:
        run()
        torch.cuda.synchronize()
        names = set(ntt.stats_collect())
    finally:
        ntt.stats_enable(False)
        ntt.stats_reset()
    assert names
    return all(n.startswith(("cmux", "xprod")) for n in names)


@pytest.mark.parametrize("bits,wb,logn,rows,groups,fused", [
    (50, 64, 4, 481, 2, True), (50, 64, 4, 482, 2, False), (32, 32, 6, 120, 2, True),
    (32, 32, 6, 121, 2, False), (60, 64, 8, 32, 3, False), (50, 64, 9, 16, 3, False),
    (32, 32, 9, 16, 3, True), (32, 32, 9, 17, 3, False), (32, 32, 9, 16, 512, True),
    (32, 32, 9, 16, 513, False), (60, 64, 10, 8, 3, True), (60, 64, 10, 9, 3, False),
    (50, 64, 10, 16, 3, True), (32, 32, 10, 16, 3, True)])
def test_operands(bits, wb, logn, rows, groups, fused):
    N, cols = 1 << logn, 2
    mods = synth.primes_below(1 << bits, 1 << 17, 1)
    ops = synth.uniform_poly(11 + rows, mods, rows * groups - 1, N)
    key = synth.uniform_poly(12 + rows, mods, rows * cols, N).reshape(rows, cols, 1, N)
    plan = ntt.Plan(N, mods, wb)
    da, dk = to_device(ops, wb), to_device(key, wb)
    out = empty_device((groups, cols, 1, N), wb)
    assert _one_launch(lambda: plan.external_product(out, da, dk, rows, cols)) == fused
    mac = oracle.mac(oracle.forward(ops, mods), key, mods, rows, cols)
    want = oracle.inverse(np.asarray(mac).reshape(-1, 1, N), mods)
    assert np.array_equal(to_host(out, wb).astype(np.uint64).reshape(-1, 1, N), want)


@pytest.mark.parametrize("bits,wb,logn,comps,levels,digits,cmux", [
    (60, 64, 8, 4, 8, False, False), (60, 64, 9, 2, 8, False, False), (50, 64, 9, 2, 8, False, True),
    (32, 32, 9, 2, 8, True, True), (60, 64, 10, 3, 4, True, True), (60, 64, 10, 2, 8, False, True),
    (50, 64, 10, 2, 8, True, True)])
def test_digits_and_cmux(bits, wb, logn, comps, levels, digits, cmux):
    N, num = 1 << logn, 3
    mods = synth.primes_below(1 << bits, 1 << 17, 1)
    rows, beta = comps * levels, -(-(bits + 1) // levels)
    acc = synth.uniform_poly(21 + rows, mods, num * comps, N).reshape(num, comps, 1, N)
    key = synth.uniform_poly(22 + rows, mods, rows * comps, N).reshape(rows, comps, 1, N)
    rot = np.array([1, N, 2 * N - 1], dtype=np.uint32)
    plan = ntt.Plan(N, mods, wb)
    da, dk = to_device(acc, wb), to_device(key, wb)
    dr = torch.from_numpy(rot.view(np.int32)).to("cuda")
    out, ext = empty_device(acc.shape, wb), empty_device(acc.shape, wb)
    assert _one_launch(lambda: plan.external_product_decomposed(ext, da, dk, levels, beta)) == digits
    assert _one_launch(lambda: plan.cmux(out, da, dr, dk, levels, beta)) == cmux
    assert np.array_equal(to_host(ext, wb).astype(np.uint64),
                          oracle.external_product_decomposed(acc, key, mods, levels, beta, comps))
    assert np.array_equal(to_host(out, wb).astype(np.uint64),
                          oracle.cmux(acc, key, mods, rot, levels, beta))


def test_threads_with_workgroups_of_different_sizes():
    """One kernel from two threads, workgroups of 77 and 136 KiB of LDS by turns."""
    import threading
    N, cols, mods = 1 << 10, 1, synth.primes_below(1 << 32, 1 << 17, 1)
    plan = ntt.Plan(N, mods, 32)
    cases = {}
    for rows in (9, 16):
        ops = synth.uniform_poly(31 + rows, mods, rows, N)
        key = synth.uniform_poly(32 + rows, mods, rows, N).reshape(rows, 1, 1, N)
        mac = oracle.mac(oracle.forward(ops, mods), key, mods, rows, cols)
        cases[rows] = (to_device(ops, 32), to_device(key, 32),
                       oracle.inverse(np.asarray(mac).reshape(-1, 1, N), mods), empty_device((1, 1, 1, N), 32))
    torch.cuda.synchronize()
    errors = []

    def work(rows):
        da, dk, _, out = cases[rows]
        try:
            for _ in range(200):
                plan.external_product(out, da, dk, rows, cols)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(r,)) for r in cases]
    [t.start() for t in threads]
    [t.join() for t in threads]
    torch.cuda.synchronize()
    assert not errors
    for _, _, want, out in cases.values():
        assert np.array_equal(to_host(out, 32).astype(np.uint64).reshape(-1, 1, N), want)
