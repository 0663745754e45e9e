"""GPU: refinement joins of vertices that several wavefronts decide at once."""
import numpy as np
import pytest

from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L

from .gpu_common import say, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shifts", [1, 4, 16])
def test_no_vertex_of_a_triangle_stays_alone(shifts):
    """Triangles of two vertices that one wavefront decides together and a
    third one that another wavefront reaches at about the same time (0 to
    shifts - 1 groups earlier; a wavefront takes 256 vertices in order).  Each
    vertex prefers the smallest of the other two, so the first two choose each
    other and the third chooses the first.  Whoever comes first, a vertex
    whose choice was joined by another has that one's community, and nobody
    is left alone: the result of one pass is its refinement."""
    blocks = 64
    base = np.arange(blocks)[:, None] * 512
    p = np.arange(0, 256, 2)[None]
    a = (base + p).ravel()
    b = a + 1
    c = (base + 256 + (p - 2 * (np.arange(blocks) % shifts)[:, None]) % 256).ravel()
    rest = np.setdiff1d(np.arange(512 * blocks), np.concatenate([a, b, c]))
    g = gen.from_edges(512 * blocks, np.concatenate([a, a, b, rest[::2]]), np.concatenate([b, c, c, rest[1::2]]))
    # tau0 = 0: local moving ends when nothing moves, with every triangle whole
    prm = L.leiden_default_params(max_passes=1, tau0=0.0, max_iter=100, verts_per_wave=256)
    for r in range(10):
        say("triangles", shifts, "run", r)
        C = to_np(L.leiden_static(L.leiden_create(g.off, g.idx, g.w, prm))[0])
        assert np.array_equal(C[a], C[b]) and np.array_equal(C[a], C[c])
        assert np.array_equal(C[rest[::2]], C[rest[1::2]])
