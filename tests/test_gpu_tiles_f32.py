"""GPU parity of the fp32 hidden-layer kernels where their 16-row tiles, the shares of a tile's
entries and the classes of row lengths begin and end.  Tolerance as in test_gpu_parity: fp32
sums of at most a few hundred terms against fp64, norm-wise 1e-5."""
import numpy as np
import pytest

from oracle import gcn
from paper_2511_09261_amd import inputs
from tests.parity import rel

pytestmark = pytest.mark.gpu


def ragged_subgraphs(seed):
    """Subgraphs of 1, 15, 16, 17, 32, 33, 64, 65 and 129 rows with random edges, and three with a
    hub of 255, 256 and 257 neighbours (the last class that is summed in place, the first two
    that come pre-reduced), all node ids shuffled."""
    rs = np.random.RandomState(seed)
    us, vs, part, base = [], [], [], 0
    for k, rows in enumerate([1, 15, 16, 17, 32, 33, 64, 65, 129, 256, 300, 700]):
        m = 3 * rows if rows > 1 else 0
        us.append(base + rs.randint(0, rows, m))
        vs.append(base + rs.randint(0, rows, m))
        spokes = {256: 255, 300: 256, 700: 257}.get(rows, 0)
        if spokes:  # the hub is a node the random edges leave alone
            us[-1][us[-1] == base + rows // 2] = base
            vs[-1][vs[-1] == base + rows // 2] = base
            others = np.setdiff1d(np.arange(rows), [rows // 2])[:spokes]
            us.append(np.full(spokes, base + rows // 2))
            vs.append(base + others)
        part.append(np.full(rows, k))
        base += rows
    name = rs.permutation(base)
    ids = np.empty(base, dtype=np.int32)
    ids[name] = np.concatenate(part)
    return inputs.from_edges(base, name[np.concatenate(us)], name[np.concatenate(vs)]), ids, 12


@pytest.mark.parametrize("D", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("L,norm,share", [(2, "sym", False), (3, "mean", False), (3, "sym", True)])
def test_tile_and_row_length_edges(gco, D, L, norm, share):
    g, part, P = ragged_subgraphs(D + L)
    E, Ws = inputs.init_params(g.n, part, 1 if share else P, L, D, 3)
    E, Ws = (E * 5).astype(np.float32), [W * 1.5 for W in Ws]
    ctx = gco.Context(num_layers=L, dim=D, norm=norm, weight_sharing=share)
    ctx.upload_graph(g.n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    spec = gcn.Spec(num_layers=L, norm=norm, weight_sharing=share)
    lg = gcn.local_graph(g.n, g.rowptr, g.col, part, P, norm)
    cache = gcn.forward(lg, E, Ws, spec)
    gE, gWs = gcn.backward(lg, cache, Ws, spec)
    dE, dWs = ctx.get_grads()
    assert rel(ctx.get_probs(), cache["p"]) <= 1e-5
    for l in range(1, L):
        assert rel(ctx.get_hidden(l), cache["H"][l]) <= 1e-5
    assert rel(dE, gE) <= 1e-5
    for l in range(L):
        assert rel(dWs[l], gWs[l]) <= 1e-5, f"layer {l + 1}"
    first = ctx.train(3)
    ctx.set_params(E, Ws)
    assert np.array_equal(first, ctx.train(3))  # one fixed order of additions
    ctx.destroy()


@pytest.mark.parametrize("D,storage", [(8, "fp32"), (16, "fp32"), (32, "fp32"), (64, "fp32"), (128, "fp32"), (64, "bf16"),
                                       (128, "bf16")])
def test_long_rows_reduced_ahead_are_those_of_the_new_embeddings(gco, D, storage):
    """The last launch of a training epoch pre-reduces the long rows for the forward pass after it: bit for bit what that
    pass forms itself from the same parameters, also where a subset trained, first of all or after the others."""
    g, part, P = ragged_subgraphs(D)
    L = 2 + (D >= 32)
    E, Ws = inputs.init_params(g.n, part, P, L, D, 3)
    ctx, fresh = (gco.Context(num_layers=L, dim=D, storage=storage) for _ in range(2))
    for c in (ctx, fresh):
        c.set_scalar_layer_form("streams")
        c.upload_graph(g.n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    subset = lambda *parts: ctx.train_subset(2, np.array(parts, dtype=np.int32))
    for run in (lambda: subset(11), lambda: ctx.train(2), lambda: subset(10)):
        run()
        ctx.forward()
        fresh.set_params(*ctx.get_params())
        fresh.forward()
        assert np.array_equal(ctx.get_probs(), fresh.get_probs())
    ctx.destroy()
    fresh.destroy()


def test_workgroups_grouped_by_xcd(gco):
    """Rows of more than 32 MB in more than eight subgraphs: the launches whose workgroups are
    grouped by XCD, with idle workgroups among them, against the oracle."""
    P, D = 24, 16
    rs = np.random.RandomState(3)
    sizes = (23_000 * (0.7 + 0.6 * rs.random_sample(P))).astype(np.int32)
    n = int(sizes.sum())
    part = np.repeat(np.arange(P), sizes).astype(np.int32)
    u = rs.randint(0, n, 2 * n)
    v = np.clip(u + rs.randint(-30, 31, 2 * n), 0, n - 1)
    name = rs.permutation(n)
    ids = np.empty(n, dtype=np.int32)
    ids[name] = part
    g = inputs.from_edges(n, name[u], name[v])
    row = np.repeat(np.arange(n), np.diff(g.rowptr))
    inside = ids[row] == ids[g.col]
    served = [gco.workgroup_parts("fp32", D, kind, sizes, np.bincount(ids[row[inside]], minlength=P))
              for kind in ("forward", "hidden", "embed")]
    assert all(np.any(np.diff(w) < 0) for w in served)       # out of the subgraphs' order: grouped
    assert any((w < 0).any() for w in served)                # workgroups with nothing to do
    E, Ws = inputs.init_params(n, ids, P, 3, D, 3)
    E, Ws = (E * 5).astype(np.float32), [W * 1.5 for W in Ws]
    ctx = gco.Context(num_layers=3, dim=D)
    ctx.upload_graph(n, g.rowptr, g.col, ids, P)
    ctx.set_params(E, Ws)
    spec = gcn.Spec(num_layers=3)
    lg = gcn.local_graph(n, g.rowptr, g.col, ids, P, "sym")
    cache = gcn.forward(lg, E, Ws, spec)
    gE, gWs = gcn.backward(lg, cache, Ws, spec)
    dE, dWs = ctx.get_grads()
    assert rel(ctx.get_probs(), cache["p"]) <= 1e-5
    assert rel(dE, gE) <= 1e-5
    for l in range(3):
        assert rel(dWs[l], gWs[l]) <= 1e-5, f"layer {l + 1}"
    ctx.destroy()


@pytest.mark.parametrize("storage,D", [("fp32", 32), ("bf16", 64)])
def test_a_listed_subset_has_runs_of_its_own(gco, storage, D):
    """A fine-tune cuts its wavefront runs for the listed subgraphs alone.  Listing all of them
    gives the bits of gco_train; changing lists back and forth, also to longer ones, gives the
    bits of a context that only ever saw that list."""
    g, part, P = ragged_subgraphs(5)
    E, Ws = inputs.init_params(g.n, part, P, 3, D, 3)

    def context():
        ctx = gco.Context(num_layers=3, dim=D, storage=storage, norm="mean")
        ctx.set_scalar_layer_form("streams")
        ctx.upload_graph(g.n, g.rowptr, g.col, part, P)
        ctx.set_params(E, Ws)
        return ctx

    a, b = context(), context()
    assert np.array_equal(a.train(3), b.train_subset(3, np.arange(P)))
    assert np.array_equal(a.get_params()[0], b.get_params()[0])
    for listed in ([11], [0, 4, 9, 10], [3], list(range(P)), [2, 11]):
        c = context()
        b.set_params(E, Ws)
        assert np.array_equal(b.train_subset(4, listed), c.train_subset(4, listed))
        (e1, w1), (e2, w2) = b.get_params(), c.get_params()
        assert np.array_equal(e1, e2) and all(np.array_equal(x, y) for x, y in zip(w1, w2))
        c.destroy()
    a.destroy()
    b.destroy()


@pytest.mark.parametrize("storage,D,sizes", [("fp32", 16, [40] * 300), ("bf16", 64, [33, 400, 0, 2000, 7] * 12),
                                             ("fp32", 32, [30_000] * 9)])
def test_a_longer_list_allocates_nothing(gco, storage, D, sizes):
    """The tables of a subset of the subgraphs lie in one block for every list after the first."""
    rs = np.random.RandomState(1)
    n, P = sum(sizes), len(sizes)
    part = np.repeat(np.arange(P), sizes).astype(np.int32)
    u = rs.randint(0, n, 3 * n)
    g = inputs.from_edges(n, u, np.clip(u + rs.randint(-20, 21, 3 * n), 0, n - 1))
    E, Ws = inputs.init_params(n, part, P, 3, D, 3)
    ctx = gco.Context(num_layers=3, dim=D, storage=storage)
    ctx.set_scalar_layer_form("streams")
    ctx.upload_graph(n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    ctx.train_subset(2, [0])
    asked = []
    empty = ctx._allocator.torch.empty

    class Counting:
        uint8 = ctx._allocator.torch.uint8

        @staticmethod
        def empty(*args, **more):
            asked.append(args)
            return empty(*args, **more)

    ctx._allocator.torch = Counting
    for listed in ([1, 2], [P - 1], list(range(0, P, 2)), list(range(P)), list(range(P - 1)), [3]):
        ctx.train_subset(2, listed)
    assert not asked
    ctx.destroy()


def test_partial_sums_take_the_memory_of_the_workgroups_there_are(gco):
    """Width 128: 512 backward workgroups, 32 MB of partial weight gradients per hidden layer."""
    n, D, L = 140_000, 128, 3
    u = np.arange(n - 1)
    g = inputs.from_edges(n, u, u + 1)
    ctx = gco.Context(num_layers=L, dim=D)
    ctx.upload_graph(n, g.rowptr, g.col)
    total = sum(t.numel() for t in ctx._allocator.live.values())
    rows = (3 + (L - 1) + (L - 2)) * n * D * 4       # E, m, v, the hidden layers, the gradient between two
    assert total <= rows + (L - 1) * 512 * D * D * 4 + 200 * n
    ctx.destroy()


@pytest.mark.parametrize("D,L", [(8, 2), (16, 3), (64, 2), (128, 3)])
def test_hidden_activations_are_those_of_the_last_epoch(gco, D, L):
    """Training keeps the last hidden layer's activations only in its last epoch: they are the ones a forward pass
    at the parameters before that epoch leaves, bit for bit."""
    g, part, P = ragged_subgraphs(7)
    E, Ws = inputs.init_params(g.n, part, P, L, D, 3)
    ctx = gco.Context(num_layers=L, dim=D)
    ctx.set_scalar_layer_form("streams")
    ctx.upload_graph(g.n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    ctx.train(2)
    ctx.forward()
    want = ctx.get_hidden(L - 1)
    assert (want > 0).any()
    ctx.set_params(E, Ws)
    ctx.train(3)
    assert np.array_equal(ctx.get_hidden(L - 1), want)
    ctx.destroy()
