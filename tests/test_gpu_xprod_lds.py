"""GPU parity: external product, its decomposing form and the CMux step in one
launch where a workgroup needs between 64 and 160 KiB of LDS, against the oracle."""
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


@pytest.mark.parametrize("bits,wb", [(32, 32), (50, 64), (60, 64)])
@pytest.mark.parametrize("logn,levels", [(10, 4), (11, 2), (11, 3), (11, 4), (12, 2)])
def test_cmux_and_products_with_large_workgroups(bits, wb, logn, levels):
    N, comps, num = 1 << logn, 2, 5
    mods = synth.primes_below(1 << bits, 1 << 17, 1)
    rows, beta = comps * levels, -(-(bits + 1) // levels)
    acc = synth.uniform_poly(800 + logn, mods, num * comps, N).reshape(num, comps, 1, N)
    key = synth.uniform_poly(900 + levels, mods, rows * comps, N).reshape(rows, comps, 1, N)
    rot = np.array([0, 1, N - 1, N, 2 * N - 1], dtype=np.uint32)
    plan = ntt.Plan(N, mods, wb)
    dk, da = to_device(key, wb), to_device(acc, wb)
    word = lambda t: to_host(t, wb).astype(np.uint64)  # noqa: E731
    out = empty_device(acc.shape, wb)
    ntt.stats_reset()
    ntt.stats_enable(True)
    try:
        plan.cmux(out, da, torch.from_numpy(rot.view(np.int32)).to("cuda"), dk, levels, beta)
        torch.cuda.synchronize()
        assert np.array_equal(word(out), oracle.cmux(acc, key, mods, rot, levels, beta))
        plan.external_product_decomposed(out, da, dk, levels, beta)
        torch.cuda.synchronize()
        want = oracle.external_product_decomposed(acc, key, mods, levels, beta, comps)
        assert np.array_equal(word(out), want)
        ops = synth.uniform_poly(950 + logn, mods, 2 * rows + 1, N)
        prod = empty_device((3, comps, 1, N), wb)
        plan.external_product(prod, to_device(ops, wb), dk, rows, comps)
        torch.cuda.synchronize()
        mac = oracle.mac(oracle.forward(ops, mods), key, mods, rows, comps)
        assert np.array_equal(word(prod).reshape(-1, 1, N),
                              oracle.inverse(np.asarray(mac).reshape(-1, 1, N), mods))
        names = set(ntt.stats_collect())
    finally:
        ntt.stats_enable(False)
        ntt.stats_reset()
    assert names and all(n.startswith(("cmux", "xprod")) for n in names), names
