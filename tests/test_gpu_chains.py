"""Long reduce chains in the mask and the device advance, against the CPU oracle."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_host_tables import nullable_grammar  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import paper_2607_11951_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.lib()
    return pkg


def _pair(G, oracle_mod, text, tokens):
    """The grammar on the device and its oracle, over all bytes, the tokens and an end-of-sequence token."""
    vocab = [bytes([b]) for b in range(256)] + sorted(tokens) + [b""]
    eos = len(vocab) - 1
    g = G.Grid(text, (), vocab, [eos], eos).to_device("cuda")
    return g, oracle_mod.Oracle(text, (), {}, vocab, [eos], eos), vocab


def _check(g, o, prefixes, status=0):
    cfgs, pool = g.configs(prefixes)
    m, e, s = g.mask(*g.configs_to_device(cfgs, pool), len(prefixes))
    torch.cuda.synchronize()
    assert (s.cpu().numpy() == status).all(), s.cpu().tolist()
    for i, w in enumerate(prefixes):
        want, want_eos = o.mask(w, mode=1)
        assert np.array_equal(m[i].cpu().numpy().view(np.uint32), want), (i, w[-8:])
        assert int(e[i]) == want_eos, (i, w[-8:])


@pytest.mark.parametrize("levels", [1, 4, 7, 9])
def test_long_runs_of_empty_reductions(G, oracle_mod, levels):
    toks = {a + b for a in (b"b", b"c", b"x", b"y", b"bc", b"cb", b"bcbc") for b in (b"x", b"y", b"b", b"c", b"bcx", b"bcy")}
    g, o, _ = _pair(G, oracle_mod, nullable_grammar(levels), toks)
    _check(g, o, [b"", b"b", b"bc", b"x", b"y", b"bcb", b"bcx", b"bcbc"])


# a chain's length is the stack's: reductions that pop two entries each, past any
# fixed number of steps; the end of input at their end, or a terminal
RIGHT = 'start P\ntoken LP "("\ntoken N /[a-z]+/\ntoken E ";"\ntoken WS / +/ ignore\nP : {} ;\nS : LP S | N ;\n'


@pytest.mark.parametrize("depth", [4000, 4094, 4095, 4096, 4097, 4200, 9000])
@pytest.mark.parametrize("form", ["S E", "S", "S E P | S E"])
def test_chains_as_long_as_the_stack(G, oracle_mod, form, depth):
    toks = {b"a;", b"(a;", b"(a ", b"((a;", b"a ;", b"a;a", b"; ", b"a ", b"(( a ;"}
    g, o, vocab = _pair(G, oracle_mod, RIGHT.format(form), toks)
    base = b"(" * depth
    prefixes = [base, base + b" ", base + b"a", base + b"a "] + ([base + b"a ;"] if "E" in form else [])
    _check(g, o, prefixes)
    # the advance by every token the mask allows
    rows = [(w, t) for w in prefixes for t in range(256, len(vocab)) if o.mask(w, tokens=[t])[0][0] and vocab[t]]
    cfgs, pool = g.configs([w for w, _ in rows])
    cap = 10240
    ids = torch.tensor([t for _, t in rows], dtype=torch.int32, device="cuda")
    c2, p2, st = g.accept(*g.configs_to_device(cfgs, pool), ids, len(rows), cap)
    out, area, st = c2.cpu().numpy().view(G.CONFIG_DTYPE), p2.cpu().numpy().view(np.uint16), st.cpu().numpy()
    assert (st == G.ROW_OK).all(), st.tolist()
    for r, (w, t) in enumerate(rows):
        want, stack = g.config(w + vocab[t])
        assert int(out[r]["q"]) == int(want["q"]) and int(out[r]["stk_depth"]) == len(stack), (r, vocab[t])
        assert np.array_equal(area[r * cap:r * cap + len(stack)], stack), (r, vocab[t])
    if depth < 8000:  # in place: within the workgroup's own area
        region = np.zeros(len(rows) * cap, np.uint16)
        c3 = cfgs.copy()
        for r in range(len(rows)):
            off, d = int(cfgs["stk_off"][r]), int(cfgs["stk_depth"][r])
            region[r * cap:r * cap + d] = pool[off:off + d]
            c3["stk_off"][r] = r * cap
        cd, pd = g.configs_to_device(c3, region)
        st = g.accept_inplace(cd, pd, ids, len(rows), cap).cpu().numpy()
        assert (st == G.ROW_OK).all(), st.tolist()
        assert torch.equal(cd.cpu(), c2.cpu())
