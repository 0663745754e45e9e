"""GPU: the fused engine's results follow from the graph and the batch alone,
to the last bit, also where sums in 64 bits are rounded."""
import numpy as np
import pytest

from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L

from .gpu_common import say, to_np

pytestmark = pytest.mark.gpu


def _weights(g, rng, spread=30):
    """Symmetric weights over `spread` powers of two: float32 values whose sums
    do not fit 53 bits."""
    row = np.repeat(np.arange(g.n), np.diff(g.off))
    a, b = np.minimum(row, g.idx).astype(np.int64), np.maximum(row, g.idx)
    _, pair = np.unique(a * g.n + b, return_inverse=True)
    return np.exp2(spread * (rng.random(pair.max() + 1) - 0.5)).astype(np.float32)[pair]


def _graphs():
    gs = [gen.planted_partition(2048, 32, 0.12, 0.004, seed=k) for k in range(4)]
    gs += [gen.rmat(12, 16, seed=1), gen.rmat(10, 32, seed=2)]  # vertices of more than 256 edges
    assert max(np.diff(g.off).max() for g in gs) > 600
    rng = np.random.default_rng(3)
    return gs, [(g.off, g.idx, _weights(g, rng)) for g in gs]


@pytest.mark.parametrize("mode", ["df", "ds", "nd"])
def test_fleet_results_do_not_depend_on_timing_or_variant(mode):
    """Six runs without a chosen variant and one of each variant: the same
    bits of memberships, modularity, K, Sigma and 2m after a static run and
    after an update."""
    gs, dev = _graphs()
    rng = np.random.default_rng(4)
    jobs = []
    for k, g in enumerate(gs):
        b = gen.random_batch(g, 300, seed=k)
        w = np.exp2(30 * (rng.random(len(b.ins_u)) - 0.5)).astype(np.float32)
        jobs.append((k, mode, L.make_batch(b.del_u, b.del_v, b.ins_u, b.ins_v, w)))
    first = None
    for v in [None] * 6 + list(range(L.FLEET_VARIANTS)):
        say("fleet order", mode, "variant", v)
        fl = L.Fleet(dev)
        if v is not None:
            fl.set_variant(v)
        out = []
        for run in ([(k, "static", None) for k in range(len(gs))], jobs):
            res, _ = fl.run(run)
            out += [(to_np(r[0]).tobytes(), float(r[1]).hex()) for r in res]
            for k in range(len(gs)):
                C, K, S, m2 = fl.get_state(k)
                out.append((to_np(C).tobytes(), to_np(K).tobytes(), to_np(S).tobytes(), float(m2).hex()))
        fl.close()
        first = first or out
        assert out == first, (v, [k for k, (x, y) in enumerate(zip(out, first)) if x != y])
