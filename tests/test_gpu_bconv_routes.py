"""GPU: which form a basis conversion takes by default, on both sides of each line of
the rule, and that its words are those of both forced forms."""
import pytest

from paper_2410_05934_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2410_05934_amd as ntt  # noqa: E402

N = 1 << 15


def _form(run):
    ntt.stats_reset()
    ntt.stats_enable(True)
    try:
        run()
        torch.cuda.synchronize()
        names = set(ntt.stats_collect())
    finally:
        ntt.stats_enable(False)
        ntt.stats_reset()
    kinds = {"matrix" if "_mfma" in n else "vector" for n in names}
    assert len(kinds) == 1, names
    return kinds.pop()


@pytest.mark.parametrize("mode,L,M,batch,form", [
    ("conv", 8, 4, 1, "vector"), ("conv", 9, 1, 1, "vector"), ("conv", 16, 2, 1, "matrix"),
    ("conv", 16, 2, 2, "vector"), ("conv", 9, 4, 3, "matrix"), ("conv", 9, 4, 4, "vector"),
    ("conv", 9, 5, 5, "matrix"), ("conv", 10, 8, 6, "vector"), ("conv", 10, 9, 6, "matrix"),
    ("conv", 17, 1, 15, "matrix"), ("conv", 17, 2, 16, "vector"), ("conv", 21, 2, 16, "matrix"),
    ("up", 10, 4, 4, "vector"), ("up", 10, 4, 3, "matrix"), ("up", 11, 4, 4, "matrix"),
    ("up", 9, 5, 6, "matrix"), ("down", 16, 8, 1, "matrix"), ("down", 16, 8, 2, "vector"),
    ("down", 12, 9, 7, "matrix"), ("down", 12, 9, 8, "vector"), ("down", 13, 9, 8, "matrix"),
    ("down", 17, 4, 5, "matrix"), ("down", 17, 4, 6, "vector"), ("down", 24, 2, 6, "vector"),
    ("down", 24, 3, 6, "matrix"), ("down", 25, 1, 6, "matrix"), ("down", 37, 4, 6, "vector"),
    ("down", 37, 5, 6, "matrix")])
@pytest.mark.parametrize("wb", [32, 64])
def test_form_and_words(mode, L, M, batch, form, wb):
    """L source and M target moduli."""
    pool = synth.primes_below(1 << (32 if wb == 32 else 50), 1 << 17, L + M)
    src, dst = pool[:L], pool[L:]
    dt = torch.int32 if wb == 32 else torch.int64
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * L + M)
    draw = lambda mods: torch.stack(  # noqa: E731
        [torch.randint(0, q, (batch, N), device="cuda", generator=g).to(dt) for q in mods], dim=1)
    x = draw(src if mode != "down" else dst + src)
    outs = []
    for mfma in (None, False, True):
        if mode == "conv":
            call, rows = ntt.BasisConversion(N, src, dst, wb, mfma=mfma), M
        elif mode == "up":
            call, rows = ntt.BasisExtension(N, src, dst, wb, mfma=mfma).mod_up, L + M
        else:
            call, rows = ntt.BasisExtension(N, dst, src, wb, mfma=mfma).mod_down, M
        out = torch.empty((batch, rows, N), dtype=dt, device="cuda")
        took = _form(lambda: call(out, x))
        assert took == (form if mfma is None else "matrix" if mfma else "vector")
        outs.append(out)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("L,M", [(9, 5), (12, 20), (24, 3), (6, 5)])
@pytest.mark.parametrize("wb", [32, 64])
def test_operands_that_start_at_any_word(L, M, wb):
    """Inputs and outputs one word past an allocation's start: the same words."""
    pool = synth.primes_below(1 << (32 if wb == 32 else 50), 1 << 17, L + M)
    src, dst = pool[:L], pool[L:]
    n, batch = 1 << 12, 2
    dt = torch.int32 if wb == 32 else torch.int64

    def odd(rows):
        return torch.zeros(batch * rows * n + 1, dtype=dt, device="cuda")[1:].view(batch, rows, n)

    x = torch.stack([torch.randint(0, q, (batch, n), device="cuda").to(dt) for q in dst + src], dim=1)
    conv, up = ntt.BasisConversion(n, src, dst, wb), ntt.BasisExtension(n, src, dst, wb)
    down = ntt.BasisExtension(n, dst, src, wb)
    s = x[:, M:].contiguous()
    for call, inp, rows in ((conv, s, M), (up.mod_up, s, L + M), (down.mod_down, x, M)):
        want, got, view = torch.empty((batch, rows, n), dtype=dt, device="cuda"), odd(rows), odd(inp.shape[1])
        view.copy_(inp)
        assert view.is_contiguous() and view.data_ptr() % (2 * wb // 8)
        call(want, inp)
        call(got, view)
        assert torch.equal(got, want)
