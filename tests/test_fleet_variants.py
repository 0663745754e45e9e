"""The fused engine's launch variants: what the library uses by itself is among
those that can be chosen and timed, and the choice can be given back."""
import numpy as np
import pytest

from paper_2405_11658_amd import inputs as gen
from paper_2405_11658_amd import leiden as L


def test_every_launch_can_be_chosen():
    info = [L.fleet_variant_info(v) for v in range(L.FLEET_VARIANTS)]
    assert len(set(info)) == len(info)
    assert (8, 2048) in info and (4, 512) in info  # up to 1024 jobs, and more
    for v in (-1, L.FLEET_VARIANTS):
        with pytest.raises(L.LeidenError):
            L.fleet_variant_info(v)


@pytest.mark.gpu
def test_the_librarys_choice_can_be_set_again():
    g = gen.planted_partition(512, 8, 0.15, 0.01, seed=1)
    fl = L.Fleet([(g.off, g.idx, g.w)] * 3)
    run = lambda: [r[0].cpu().numpy() for r in fl.run([(k, "static", None) for k in range(3)])[0]]
    first = run()
    for v in (0, -1, L.FLEET_VARIANTS - 1, -1):
        fl.set_variant(v)
        assert all(np.array_equal(x, y) for x, y in zip(run(), first))
    for v in (-2, L.FLEET_VARIANTS):
        with pytest.raises(L.LeidenError):
            fl.set_variant(v)
    fl.close()
