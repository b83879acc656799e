"""The kernels a step takes by the level's size (ppm_get_step_route), on both
sides of each line of the rules, and their results against the staged kernels
bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1008_2801_amd import inputs as I  # noqa: E402
from paper_1008_2801_amd import ppm as P  # noqa: E402

pytestmark = pytest.mark.gpu

# box sizes per axis, precision, (front end, final stage)
CASES = [
    # one launch up to 2048 workgroups: 12 wavefront runs a row of k_front_x of
    # 63 zones, 256 zones a tile of the other axes
    (([32], [69], [70]), 0, (4, 0)), (([29], [69], [77]), 0, (2, 0)),
    (([32], [69], [70]), 1, (4, 0)), (([29], [69], [77]), 1, (2, 0)),
    # y and z in columns from planes of 16 MB and 1024 workgroups on, both
    # reached at 128^3 traced zones in FP64
    (([126], [126], [126]), 0, (3, 1)), (([125], [126], [126]), 0, (2, 1)),
    (([126], [126], [254]), 1, (3, 0)), (([125], [126], [254]), 1, (2, 0)),
    # bricks from 512 of them on
    (([64], [64], [64]), 0, (2, 1)), (([64], [64], [60]), 0, (2, 0)), (([64], [64], [64]), 1, (2, 1)),
    # not where the boxes' extents cut thin ones: rows of 33 (shares of a brick
    # row filled 0.52), 36 (0.56) and 48 zones (0.75), boxes 4, 5, 7 and 8 wide
    (([33] * 4, [33] * 4, [33] * 4), 0, (3, 0)), (([33] * 4, [33] * 4, [33] * 4), 1, (2, 0)),
    (([36] * 4, [36] * 2, [36] * 2), 0, (2, 1)), (([36] * 4, [36] * 2, [36] * 2), 1, (2, 0)),
    (([48] * 3, [48] * 2, [48] * 2), 1, (2, 1)), (([72], [72], [72]), 1, (2, 0)),
    (([4], [256], [256]), 0, (2, 0)), (([4], [256], [256]), 1, (2, 0)),
    (([5] * 8, [5] * 8, [5] * 8), 0, (2, 0)), (([7] * 8, [7] * 8, [7] * 8), 0, (2, 1)),
    (([7] * 8, [7] * 8, [7] * 8), 1, (2, 0)), (([8] * 8, [8] * 8, [8] * 8), 1, (2, 1)),
    # columns from 1536 workgroups on, on boxes of a million zones and more on
    # average: 131 x 12 workgroups here, 49 x 5 a box of the eight
    (([200], [160], [180]), 0, (3, 4)), (([200], [60], [70] * 8), 0, (3, 1)),
    (([200], [160], [180]), 1, (3, 0)),
]


@pytest.mark.parametrize("tiling,precision,route", CASES)
def test_kernels_by_size(tiling, precision, route):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay = I.tensor_tiling(*tiling, bc=(1, 1, 0, 0, 2, 2))
    h = (1.0 / 32, 1.0 / 24, 1.0 / 40)
    p = P.params(gamma=1.4, grav=(0.1, 0.0, -0.4), precision=precision)
    rng = torch.Generator(device="cuda").manual_seed(3)
    outs = []
    for staged in (True, False):
        lev = P.Level(lay)
        if staged:
            lev.set_front_form(0)
            lev.set_step_form(0)
        assert lev.get_step_route(precision) == ((0, 0) if staged else route)
        if staged:
            U = lev.new_state()
            for b in range(lay.nbox):
                o, n = int(lev.offsets[b]), lay.box_size(b)
                v = U[o:o + n].view(5, -1)
                v.copy_(0.2 * torch.rand(v.shape, generator=rng, device="cuda", dtype=torch.float64))
                v[0] += 1.0
                v[4] += 2.5
            lev.fill_boundary(U)
            dt = lev.compute_dt(U, h, p)
        V = torch.zeros_like(U)
        nxt = torch.zeros(2, dtype=torch.float64, device="cuda")
        F = lev.new_fluxes()
        lev.hydro_step(U, V, h, p, dt_dev=dt, dt_next=nxt, fluxes=F)
        assert lev.check_status() == 0
        lev.close()
        outs.append([V, nxt] + list(F))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def test_one_launch_front_end_needs_its_tile_size():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lev = P.Level(I.single_box(16))
    assert lev.get_step_route() == (4, 0)
    lev.set_tiling(128, 8)
    assert lev.get_step_route() == (2, 0)
    with pytest.raises(P.PPMError, match="step_route"):
        lev.get_step_route(2)
    lev.close()


def test_autotuner_leaves_the_front_end_by_size_where_it_takes_columns():
    """Form 3 (columns always) is the same batched step there, but holds for the
    launches of single small boxes as well."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay = I.tensor_tiling([64] * 2, [64] * 2, [64] * 3)
    lev = P.Level(lay)
    p = P.params(gamma=1.4)
    assert lev.get_step_route()[0] == 3
    U = lev.new_state()
    for b in range(lay.nbox):
        o, n = int(lev.offsets[b]), lay.box_size(b)
        v = U[o:o + n].view(5, -1)
        v.fill_(0.1)
        v[0] = 1.0
        v[4] = 2.5
    for _ in range(3):
        lev.autotune(U, (0.1, 0.1, 0.1), p, reps=1)
        assert lev.get_front_form() != 3
    lev.close()
