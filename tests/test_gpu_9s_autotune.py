"""rd_autotune where every tile is the same kernel: the selected tile stays (a
timing of equals would pick one by noise, and keep it for later problems)."""
import pytest

from gpu_common import make_problem, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision,tiles", [(32, 0, (4, 8, 16)), (64, 0, (4, 8, 16)),
                                               (128, 0, (16, 32)), (32, 1, (4, 16, 8)),
                                               (64, 1, (8, 16)), (128, 1, (32,))])
def test_the_selected_tile_stays(n, precision, tiles):
    need_gpu()
    p, _, _ = make_problem(n, 3, precision=precision)
    for cpt in tiles:  # (the default last: later problems start from it again)
        p.set_tile(0, cpt)
        for _ in range(3):
            assert list(p.autotune()) == [cpt]
    p.close()
