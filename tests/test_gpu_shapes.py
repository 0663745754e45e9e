"""GPU: the launch shapes and table sizes of the kernels at the edges of their
ranges, through the C ABI, against the CPU oracle (integer weights, so every
comparison that is not said to be otherwise is exact)."""
import numpy as np
import pytest

import oracle
from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L

from .gpu_common import dev_batch, og, say, to_np
from .test_gpu_async import _check_state, _graph_of

pytestmark = pytest.mark.gpu


def _stars(degrees, seed=1):
    """A hub of each of the given degrees among communities of 64 vertices:
    the hub is joined to the first vertices of a shared pool, every pool
    vertex to 6 others of its community, the first two hubs to each other."""
    rng = np.random.default_rng(seed)
    pool = max(degrees) + 64
    h = len(degrees)
    u, v = [], []
    for k, d in enumerate(degrees):
        mates = rng.permutation(pool)[:d]
        u.append(np.full(d, k))
        v.append(h + mates)
    p = np.arange(pool)
    for _ in range(6):
        u.append(h + p)
        v.append(h + np.minimum(p // 64 * 64 + rng.integers(0, 64, pool), pool - 1))
    g = gen.from_edges(h + pool, np.concatenate(u), np.concatenate(v))
    deg = np.diff(g.off)
    assert [int(x) for x in deg[:h]] == list(degrees)
    return g


@pytest.mark.parametrize("degrees", [
    (256, 257, 2048),            # wavefront and workgroup
    (257, 2048, 2049, 6144),     # and the large workgroup
    (300, 2049, 6144, 6145),     # a chunked hub, alone in its slice or not
    (6145, 6500, 7000, 400, 500, 2500) * 3,
])
@pytest.mark.parametrize("slices", [0, 1])
def test_hub_degree_classes(degrees, slices):
    """Vertices on either side of every degree class of the asynchronous hub
    slices (one slice, and the default 64): modularity, K, Sigma and 2m match
    the oracle's for the returned membership and the communities are connected.
    With the default slices the modularity of the static run is at most 5e-3
    below the oracle's (the single-run bound of the other asynchronous tests;
    hubs that all move at once end where they end)."""
    g = _stars(degrees)
    h = L.leiden_create(g.off, g.idx, g.w, L.leiden_default_params(hub_slices=slices))
    say("hub classes", degrees, "slices", slices)
    C, q, st = L.leiden_static(h)
    qo = _check_state(h, g, C, q)
    if slices == 0:
        ost, _ = oracle.static(og(g))
        assert qo - oracle.modularity(og(g), ost.C) >= -5e-3
    for mode, b in zip(("df", "nd", "ds"), gen.batch_stream(g, 200, 3, seed=3)):
        C, q, st, _ = L.leiden_update(h, dev_batch(b), mode)
        _check_state(h, _graph_of(h), C, q)
