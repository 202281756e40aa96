"""Read-out kernels (cross edges, their ends, conflicts, counts, greedy repair) against the
combinatorial oracle, bit for bit, where the chunks of 2048 entries and the classes of row
lengths begin and end."""
import numpy as np
import pytest

from oracle import combinatorial as cb
from paper_2511_09261_amd import inputs

pytestmark = pytest.mark.gpu


def circulant(n, half):
    """n nodes with 2 half neighbours each."""
    u = np.repeat(np.arange(n), half)
    return inputs.from_edges(n, u, (u + np.tile(np.arange(1, half + 1), n)) % n)


def spokes(n, degrees, rs, core=None):
    """Node 7 (i + 1) has degrees[i] neighbours among the last nodes; the last nodes of all are joined as
    the upper triangle `core` says."""
    us = [np.full(d, 7 * (i + 1)) for i, d in enumerate(degrees)]
    vs = [n - 1 - rs.permutation(n - 7 * (len(degrees) + 2))[:d] for d in degrees]
    if core is not None:
        u, v = np.nonzero(core)
        us.append(n - 1 - u)
        vs.append(n - 1 - v)
    return inputs.from_edges(n, np.concatenate(us), np.concatenate(vs))


def graph(kind):
    rs = np.random.RandomState(5)
    if kind == "whole_chunks":            # 4096 entries, rows begin where chunks do
        return circulant(512, 4)
    if kind == "rows_over_edges":         # rows of 6: a row lies across the end of each chunk
        return circulant(700, 3)
    if kind == "one_entry_more":          # 2050 entries
        u = np.arange(1025)
        return inputs.from_edges(1100, u, u + 1)
    if kind == "row_lengths":             # around 8 lanes, 16 in a pass, 128 in a lane group
        return spokes(900, [1, 7, 8, 9, 15, 16, 17, 127, 128, 129, 255, 256, 257, 600], rs)
    if kind == "hubs":                    # rows longer than a chunk and than two
        return spokes(9000, [2048, 2049, 4500, 7000], rs)
    if kind == "dense":                   # more than 128 neighbours on average: a wavefront per node
        return spokes(1500, [1, 255, 256, 257, 1024, 1025], rs, np.triu(rs.random_sample((700, 700)) < 0.9, 1))
    if kind == "dense_hubs":              # and rows beyond a wavefront's 1024
        return spokes(3000, [1023, 1024, 1025, 2500], rs, np.triu(rs.random_sample((1000, 1000)) < 0.5, 1))
    if kind == "gap":                     # 30 000 rows without entries between two that have some
        u = np.concatenate([rs.randint(0, 400, 1500), 30400 + rs.randint(0, 400, 1500)])
        v = np.concatenate([rs.randint(0, 400, 1500), 30400 + rs.randint(0, 400, 1500)])
        u[0], v[0] = 3, 30500
        return inputs.from_edges(30900, u, v)
    return inputs.from_edges(300, np.array([0]), np.array([299]))  # two entries, at both ends


@pytest.mark.parametrize("kind", ["whole_chunks", "rows_over_edges", "one_entry_more", "row_lengths", "hubs", "dense",
                                  "dense_hubs", "gap", "two_entries"])
def test_read_out_edges(gco, kind):
    g = graph(kind)
    rs = np.random.RandomState(6)
    part = rs.randint(0, 5, g.n).astype(np.int32)
    E, Ws = inputs.init_params(g.n, part, 5, 2, 16, 1)
    ctx = gco.Context(num_layers=2, dim=16)
    ctx.upload_graph(g.n, g.rowptr, g.col, part, 5)
    wu, wv = cb.cut_edges_vectorised(g.n, g.rowptr, g.col, part)
    u, v = ctx.cut_edges()
    np.testing.assert_array_equal(u, wu)
    np.testing.assert_array_equal(v, wv)
    np.testing.assert_array_equal(ctx.cross_mask(), cb.cross_mask(g.n, wu, wv))
    sel = (rs.random_sample(g.n) < 0.6).astype(np.uint8)
    for got, want in zip(ctx.conflict_edges(sel), cb.conflict_edges(wu, wv, sel)):
        np.testing.assert_array_equal(got, want)
    ctx.set_params(E, Ws)
    ctx.forward()
    p = ctx.get_probs()
    for thr in (0.0, float(np.median(p))):       # every node selected, half of them
        x0, obj, before, _ = ctx.round_repair(thr, "none")
        np.testing.assert_array_equal(x0, (p >= np.float32(thr)).astype(np.uint8))
        assert obj == x0.sum() and before == cb.count_conflicts(g.n, g.rowptr, g.col, part, x0, "all")
        for scope in ("local", "all"):
            x, obj, b, after = ctx.round_repair(thr, scope)
            np.testing.assert_array_equal(x, cb.repair(g.n, g.rowptr, g.col, part, p, x0, scope))
            assert b == before and obj == x.sum()
            assert after == cb.count_conflicts(g.n, g.rowptr, g.col, part, x, "all")
    ctx.destroy()
