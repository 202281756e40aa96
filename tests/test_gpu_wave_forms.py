"""The two forms of the bf16 forward kernel of width 64 (source rows requested a step ahead where
few workgroups run, in the step itself where many do): the hidden rows of a run over one subgraph
against those of the run over all.

Tolerance.  The wavefronts of the two runs are cut at other rows, so the entries of a row fall into
other slots of the 64-entry steps and its fp32 sum of about ten terms is taken in another order:
an error of up to 2^-20 relative, by which an aggregate changes to the neighbouring bf16 number with
a probability of up to 2^-12 (spacing 2^-8).  One such change moves the 64 outputs of its row by up
to 2^-8 of one of their terms: of all outputs up to 64 2^-12 = 1/64 move by about 2^-8, in the
2-norm 2^-8 / 8, doubled for the outputs' own rounding: 2^-10.  The second layer adds as much
again.  One entry left out of the 12 500 rows compared would show as 4 2^-10."""
import numpy as np
import pytest

from paper_2511_09261_amd import inputs
from tests.parity import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,hub", [(2, 0), (3, 200), (3, 700)])   # 700: pre-reduced rows
def test_forms_agree(gco, L, hub):
    n, P = 100_003, 8                      # over 768 workgroups of four 32-row tiles in all
    rs = np.random.RandomState(L + hub)
    u, v = rs.randint(0, n, 250_000), rs.randint(0, n, 250_000)
    if hub:
        u, v = np.append(u, np.full(hub, 17 * P)), np.append(v, P * rs.permutation(n // P)[:hub])
    g = inputs.from_edges(n, u, v)
    part = (np.arange(n) % P).astype(np.int32)
    E, Ws = inputs.init_params(n, part, P, L, 64, 2)
    ctx = gco.Context(num_layers=L, dim=64, storage="bf16")
    ctx.upload_graph(g.n, g.rowptr, g.col, part, P)
    ctx.set_params(E * 20, Ws)
    ctx.forward()
    want = [ctx.get_hidden(l) for l in range(1, L)]
    assert all((H != 0).mean() > 0.1 for H in want)
    for k in (0, 5):
        ctx.set_params(E * 20, Ws)
        ctx.forward()
        ctx.train_subset(1, [k])           # H is that of the parameters before the step
        for l in range(1, L):
            assert rel_l2(ctx.get_hidden(l)[part == k], want[l - 1][part == k]) <= l * 2.0 ** -10
    ctx.destroy()
