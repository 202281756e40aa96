"""One Adam step in fp32 is the correctly rounded one, bit for bit, whichever launch takes it.

From the moments the library reports after the first step the step itself follows without a
gradient: x1 = x0 - lr ((m c1) / (sqrt(v) c2 + eps)), every operation rounded once.  The learning
rate is a power of two, so that its product is exact; the sum under the fraction may be one
operation or two (a fused multiply-add), and either is accepted."""
import numpy as np
import pytest

from paper_2511_09261_amd import inputs

pytestmark = pytest.mark.gpu

LR = 2.0 ** -7


def steps(x0, m, v):
    """The two acceptable results of the first step, in float32."""
    f = np.float32
    c1 = f(1.0 / (1.0 - float(f(0.9))))
    c2 = f(1.0 / np.sqrt(1.0 - float(f(0.999))))
    root, top = np.sqrt(v), m * c1
    out = []
    for below in (root * c2 + f(1e-8), (root.astype(np.float64) * float(c2) + float(f(1e-8))).astype(f)):
        out.append(x0 - f(LR) * (top / below))
    return out


@pytest.mark.parametrize("D,L,storage,share,way", [
    (8, 2, "fp32", True, "tiles"), (16, 3, "fp32", True, "tiles"), (32, 2, "fp32", True, "tiles"),
    (64, 3, "fp32", True, "tiles"), (128, 2, "fp32", False, "tiles"), (16, 1, "fp32", False, "tiles"),
    (8, 2, "fp32", False, "small"), (16, 3, "fp32", False, "small"), (32, 2, "fp32", False, "small"),
    (64, 2, "fp32", False, "small"), (64, 2, "bf16", False, "small")])
def test_first_step_is_correctly_rounded(gco, D, L, storage, share, way):
    rs = np.random.RandomState(D + L)
    P, rows, per_node = 250, 60, 1 if D == 64 else 2   # sizes at which one launch is the chosen way for small subgraphs
    n = P * rows
    part = np.repeat(np.arange(P), rows).astype(np.int32)
    m = per_node * n
    base = rs.randint(0, P, m) * rows
    g = inputs.from_edges(n, base + rs.randint(0, rows, m), base + rs.randint(0, rows, m))
    E, Ws = inputs.init_params(n, part, 1 if share else P, L, D, 5)
    ctx = gco.Context(num_layers=L, dim=D, storage=storage, weight_sharing=share, lr=LR)
    ctx.upload_graph(n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    ctx.set_profiling(1)
    ctx.train(1)
    assert (ctx.get_timing()["small_train"]["launches"] > 0) == (way == "small")
    E1, W1 = ctx.get_params()
    mE, vE, mW, vW, _ = ctx.get_opt_state()
    assert (mE != 0).mean() > 0.1
    for x0, x1, m, v in [(E, E1, mE, vE)] + list(zip(Ws, W1, mW, vW)):
        a, b = steps(x0.astype(np.float32), m, v)
        assert not ((x1 != a) & (x1 != b)).any()
    ctx.destroy()
