"""GPU parity: the split and row radix a call takes by default, on both sides of
the rules' lines, against a plan with the split fixed (whose words other tests pin
to the oracle) and, for one row of each, the oracle itself."""
import numpy as np
import pytest

import oracle
from paper_2410_05934_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2410_05934_amd as ntt  # noqa: E402
from paper_2410_05934_amd.tensors import to_host  # noqa: E402

PRIMES = {"u32": (32, 32), "fp64": (50, 64), "i64": (60, 64)}


@pytest.mark.parametrize("cls", list(PRIMES))
@pytest.mark.parametrize("logn,batch", [(13, 1), (13, 21), (13, 22), (13, 70), (14, 1), (14, 31),
                                        (14, 32), (15, 1), (15, 40), (16, 2)])
def test_default_split_gives_the_same_words(cls, logn, batch):
    bits, wb = PRIMES[cls]
    N, L = 1 << logn, 3
    mods = synth.primes_below(1 << bits, 1 << 17, L)
    g = torch.Generator(device="cuda")
    g.manual_seed(logn * 100 + batch)
    dt = torch.int32 if wb == 32 else torch.int64

    def draw():
        return torch.stack([torch.randint(0, q, (batch, N), device="cuda", generator=g).to(dt)
                            for q in mods], dim=1)

    a, b = draw(), draw()
    plan = ntt.Plan(N, mods, wb)
    fixed = ntt.Plan(N, mods, wb, ntt.flag_split(logn - 12))
    got = {}
    for name, p in (("default", plan), ("fixed", fixed)):
        f, i, c, u, v = a.clone(), a.clone(), torch.empty_like(a), a.clone(), b.clone()
        p.forward(f)
        p.inverse(i)
        p.polymul(c, a, b)
        m = torch.empty_like(a)
        p.forward_mul(m, u, v)
        got[name] = (f, i, c, m, u, v)
    torch.cuda.synchronize()
    for x, y in zip(got["default"], got["fixed"]):
        assert torch.equal(x, y)
    word = lambda t: to_host(t, wb).astype(np.uint64)  # noqa: E731
    last = word(a[-1:])
    assert np.array_equal(word(got["default"][0][-1:]), oracle.forward(last, mods))
    assert np.array_equal(word(got["default"][1][-1:]), oracle.inverse(last, mods))


@pytest.mark.parametrize("cls,logn,batch", [("fp64", 14, 48), ("fp64", 13, 40), ("i64", 14, 2),
                                            ("fp64", 15, 2)])
def test_tuner_times_the_product_rows_that_calls_run(cls, logn, batch):
    """The radix the tuner records for products is that of the rows products take with
    the recorded split (N = 2^14 in one pass, which products do not have, included)."""
    bits, wb = PRIMES[cls]
    N, mods = 1 << logn, synth.primes_below(1 << bits, 1 << 17, 3)

    def product_rows(run):
        ntt.stats_reset()
        ntt.stats_enable(True)
        try:
            run()
            torch.cuda.synchronize()
            return {n for n in ntt.stats_collect() if n.startswith("polymul_row")}
        finally:
            ntt.stats_enable(False)
            ntt.stats_reset()

    ntt.tune_clear()
    try:
        timed = product_rows(lambda: ntt.tune_split(N, mods, wb, batch))
        plan = ntt.Plan(N, mods, wb)
        a = torch.randint(0, mods[-1], (batch, 3, N), device="cuda")
        taken = product_rows(lambda: plan.polymul(torch.empty_like(a), a, a))
    finally:
        ntt.tune_clear()
    assert len(timed) == 2 and len(taken) == 1 and taken <= timed


@pytest.mark.parametrize("rows,product,fwdmul", [(31, "polymul_row8", "fwdmul_row8"),
                                                 (32, "polymul_row", "fwdmul_row8")])
def test_wide_product_rows_of_2_12(rows, product, fwdmul):
    """64-bit integers at 2^16: products take radix-16 rows from 32 limb-rows on,
    forward-and-multiply radix-8; the words are those of a radix-8 plan."""
    N, mods = 1 << 16, synth.primes_below(1 << 60, 1 << 17, 1)
    draw = lambda: torch.randint(0, mods[0], (rows, 1, N), device="cuda")  # noqa: E731
    a, b = draw(), draw()
    got = []
    for flags in (0, 1 << 17):
        plan = ntt.Plan(N, mods, 64, flags)
        c, m, u, v = torch.empty_like(a), torch.empty_like(a), a.clone(), b.clone()
        ntt.stats_reset()
        ntt.stats_enable(True)
        try:
            plan.polymul(c, a, b)
            plan.forward_mul(m, u, v)
            torch.cuda.synchronize()
            names = {n.split("_fwd_")[0] for n in ntt.stats_collect()}
        finally:
            ntt.stats_enable(False)
            ntt.stats_reset()
        got.append((c, m))
        if not flags:
            assert product in names and fwdmul in names, names
            assert not names & {"polymul_row", "polymul_row8", "fwdmul_row", "fwdmul_row8"} - {product, fwdmul}
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    one = to_host(a[:1], 64).astype(np.uint64), to_host(b[:1], 64).astype(np.uint64)
    assert np.array_equal(to_host(got[0][0][:1], 64).astype(np.uint64), oracle.polymul(*one, mods))
