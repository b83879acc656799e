"""Kernels whose lanes walk columns of a box (a stencil or a carried state in
registers along y or z) against the staged kernels on the same input, bit for
bit, at box sizes around the run lengths and workgroup sizes of the columns:
extents of one and two zones, one run, a run and a remainder, more columns
than one workgroup, several boxes, walls and gravity."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1008_2801_amd import inputs as I  # noqa: E402
from paper_1008_2801_amd import ppm as P  # noqa: E402

pytestmark = pytest.mark.gpu

# per-axis box sizes of a tensor tiling
TILINGS = [([5], [4], [4]), ([1, 7], [3, 1], [2, 5]), ([17], [14], [15]), ([64], [15, 2], [33]),
           ([70, 3], [16, 31], [6, 1, 9]), ([4], [40], [4, 18])]


def _level(tiling, precision, seed=9):
    lay = I.tensor_tiling(*tiling, bc=(0, 0, 0, 0, 2, 2))
    h = (1.0 / 32, 1.0 / 24, 1.0 / 40)
    rng = np.random.default_rng(seed)
    S = [I.ModeSum(rng, 6, 4, (1.0, 1.0, 1.0)) for _ in range(5)]

    def prim(x, y, z):
        left = x < 0.06
        return (np.where(left, 1.0, 0.3) * (1.0 + 0.3 * S[0](x, y, z)), 0.4 * S[1](x, y, z), 0.4 * S[2](x, y, z),
                0.4 * S[3](x, y, z), np.where(left, 1.0, 0.2) * (1.0 + 0.3 * S[4](x, y, z)))
    U = torch.from_numpy(I._fill_state(lay, h, 1.4, prim)).cuda()
    return lay, h, U, P.params(gamma=1.4, grav=(0.1, 0.0, -0.4), precision=precision)


def _step(lay, h, U, p, mode, front, form=0):
    lev = P.Level(lay)
    lev.set_front_form(front)
    lev.set_step_form(form)
    A = U.clone()
    lev.fill_boundary(A)
    B = torch.zeros_like(A)
    F = lev.new_fluxes()
    dt = lev.compute_dt(A, h, p)
    nxt = torch.zeros(2, dtype=torch.float64, device="cuda")
    lev.hydro_step(A, B, h, p, dt_dev=dt, fluxes=F, mode=mode, dt_next=nxt)
    # the intermediates the adjoint reads from the step workspace
    w = torch.ones_like(A)
    G = torch.zeros_like(A)
    lev.hydro_step_adjoint(A, w, G, h, p, dt_dev=dt, saved=True)
    return B, nxt, G, F


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("tiling", TILINGS)
def test_front_columns_agree_bitwise(tiling, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U, p = _level(tiling, precision)
    for mode in (P.BATCHED, P.PER_BOX):
        ref = _step(lay, h, U, p, mode, 0)
        got = _step(lay, h, U, p, mode, 3)
        for a, b in zip(ref[:3], got[:3]):
            assert torch.equal(a, b), (tiling, precision, mode)
        for a, b in zip(ref[3], got[3]):
            assert torch.equal(a, b), (tiling, precision, mode)


@pytest.mark.parametrize("tiling", [([33], [5], [6]), ([4, 1], [9], [5]), ([65, 2], [1, 4], [1, 3])])
def test_bricks_one_zone_thin_agree_bitwise(tiling):
    """Boxes one zone longer than whole bricks (32 x 4 x 4) along x, y or z."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U, p = _level(tiling, 0)
    ref = _step(lay, h, U, p, P.BATCHED, 0)
    got = _step(lay, h, U, p, P.BATCHED, 0, form=1)
    for a, b in zip(list(ref[:3]) + list(ref[3]), list(got[:3]) + list(got[3])):
        assert torch.equal(a, b), tiling


@pytest.mark.parametrize("tiling", [([200], [181], [195]), ([130, 3, 61], [1, 40, 90], [65, 33, 16, 2, 63])])
def test_final_columns_agree_bitwise(tiling):
    """Levels large enough for the final stage in columns (form 0) against the
    brick form: new state, flux outputs, next dt, and the saved adjoint."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # the final stage's rule: planes of 16 MB, 1536 workgroups of 248 columns in runs of 16 planes
    groups = sum(-(-((x + 2) * y) // 248) * -(-z // 16) for x in tiling[0] for y in tiling[1] for z in tiling[2])
    zones = sum((x + 2) * (y + 2) * (z + 2) for x in tiling[0] for y in tiling[1] for z in tiling[2])
    assert zones * 8 >= 16 << 20 and groups >= 1536, (zones, groups)
    lay, h, U, p = _level(tiling, 0)
    ref = _step(lay, h, U, p, P.BATCHED, 0, form=1)
    got = _step(lay, h, U, p, P.BATCHED, 2)
    for a, b in zip(ref[:3], got[:3]):
        assert torch.equal(a, b), tiling
    for a, b in zip(ref[3], got[3]):
        assert torch.equal(a, b), tiling


# one zone; up to, at and beyond the zones of one workgroup; the most
# workgroups the one-launch front end takes (2048) and a few more
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("tiling", [([4], [4], [4]), ([1, 3], [4], [4]), ([14], [14], [15]), ([5, 1], [70, 2], [3, 9]),
                                    ([54], [53], [53]), ([55], [55], [55])])
def test_front_end_in_one_launch_agrees_bitwise(tiling, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U, p = _level(tiling, precision)
    for mode in (P.BATCHED, P.PER_BOX):
        ref = _step(lay, h, U, p, mode, 0)
        got = _step(lay, h, U, p, mode, 2)
        for a, b in zip(ref[:3], got[:3]):
            assert torch.equal(a, b), (tiling, precision, mode)
        for a, b in zip(ref[3], got[3]):
            assert torch.equal(a, b), (tiling, precision, mode)


def test_time_step_of_a_state_without_a_speed():
    """Speeds that are not numbers are left out of the time step; with no other
    the largest speed is 0 and any step is allowed."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U, p = _level(([5, 4], [4], [20]), 0)
    lev = P.Level(lay)
    dt = lev.compute_dt(U, h, p).clone()
    assert dt[0].item() > 0 and dt[0].item() == p.cfl / dt[1].item()
    nan = torch.full_like(U, float("nan"))
    pair = dt.clone()
    for _ in range(2):
        lev.compute_dt(nan, h, p, out=pair)
        assert pair[0] == float("inf") and pair[1] == 0
    lev.compute_dt(U, h, p, out=pair)
    assert torch.equal(pair, dt)


@pytest.mark.parametrize("n,precision", [((52, 52, 100), 0), ((88, 88, 88), 0), ((112, 112, 112), 1)])
def test_plain_and_streaming_stores_agree_bitwise(n, precision):
    """A periodic box whose planes are stored plainly and the same box twice
    along z, whose planes are streamed: 52 x 52 x 100 the fluxes (2.4 and 4.8
    MB a plane, line 3.4), 88^3 FP64 and 112^3 FP32 the primitives (35 and 70
    MB, line 64)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = (1.0 / 32, 1.0 / 24, 1.0 / 40)
    rng = np.random.default_rng(4)
    outs = []
    A = None
    for copies in (1, 2):
        lay = I.tensor_tiling([n[0]], [n[1]], [n[2]] * copies, bc=(0,) * 6)
        lev = P.Level(lay)
        U = lev.new_state()
        if A is None:
            A = 0.2 * torch.from_numpy(rng.normal(size=lay.box_size(0))).cuda()
            v = A.view(lay.stored_shape(0))
            v[0] = 1.0 + 0.4 * v[0].sin()
            v[4] = 3.0 + v[4].sin()
        U.copy_(A.repeat(copies))
        p = P.params(gamma=1.4, precision=precision)
        lev.fill_boundary(U)
        V = torch.zeros_like(U)
        lev.hydro_step(U, V, h, p, dt=2e-3)
        assert lev.check_status() == 0
        outs.append([V[b * lay.box_size(0):(b + 1) * lay.box_size(0)] for b in range(copies)])
    for b in range(2):
        assert torch.equal(outs[0][0], outs[1][b]), (n, precision, b)


# boxes of a million zones in columns with several boxes; 511, 512 and more
# bricks (32 x 4 x 4); FP32 boxes below and above 80^3 zones
@pytest.mark.parametrize("tiling,precision", [(([200, 120], [150], [131, 60]), 0), (([32 * 7], [4 * 73], [4]), 0),
                                              (([64], [64], [64]), 0), (([31, 5], [41, 40], [33, 50]), 0),
                                              (([64], [64], [64]), 1), (([81], [81], [82]), 1)])
def test_final_stage_by_rule_agrees_bitwise(tiling, precision):
    """The form the rule takes (form 0) against the streamed form."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U, p = _level(tiling, precision)
    ref = _step(lay, h, U, p, P.BATCHED, 0, form=2)
    got = _step(lay, h, U, p, P.BATCHED, 2)
    for a, b in zip(ref[:3], got[:3]):
        assert torch.equal(a, b), tiling
    for a, b in zip(ref[3], got[3]):
        assert torch.equal(a, b), tiling
