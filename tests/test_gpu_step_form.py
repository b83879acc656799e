"""The final stage's forms (ppm_set_step_form): each value runs the kernels it
names, and the columns agree with the staged pair bit for bit on boxes of a few
zones (rows shorter than a wavefront's columns, runs of one or two planes) and
around the columns' run and workgroup sizes, with walls and outflow on every
axis and in both launch modes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1008_2801_amd import inputs as I  # noqa: E402
from paper_1008_2801_amd import ppm as P  # noqa: E402

pytestmark = pytest.mark.gpu

STAGED, BRICKS, STREAM, BY_SIZE, COLUMNS = range(5)


def _level(tiling, bc, seed=11):
    lay = I.tensor_tiling(*tiling, bc=bc)
    h = (1.0 / 32, 1.0 / 24, 1.0 / 40)
    rng = np.random.default_rng(seed)
    S = [I.ModeSum(rng, 6, 4, (1.0, 1.0, 1.0)) for _ in range(5)]

    def prim(x, y, z):
        left = x < 0.06
        return (np.where(left, 1.0, 0.3) * (1.0 + 0.3 * S[0](x, y, z)), 0.4 * S[1](x, y, z), 0.4 * S[2](x, y, z),
                0.4 * S[3](x, y, z), np.where(left, 1.0, 0.2) * (1.0 + 0.3 * S[4](x, y, z)))
    return lay, h, torch.from_numpy(I._fill_state(lay, h, 1.4, prim)).cuda()


def _step(lay, h, U, form, precision=0, mode=P.BATCHED):
    lev = P.Level(lay)
    if form is not None:
        lev.set_step_form(form)
        assert lev.get_step_form() == form
    p = P.params(gamma=1.4, grav=(0.1, 0.0, -0.4), precision=precision)
    A = U.clone()
    lev.fill_boundary(A)
    B = torch.zeros_like(A)
    F = lev.new_fluxes()
    dt = lev.compute_dt(A, h, p)
    nxt = torch.zeros(2, dtype=torch.float64, device="cuda")
    lev.hydro_step(A, B, h, p, dt_dev=dt, fluxes=F, mode=mode, dt_next=nxt)
    status = lev.check_status()
    lev.close()
    return [B, nxt] + list(F), status


@pytest.mark.parametrize("precision", [0, 1])
def test_each_form_runs_the_kernels_it_names(precision):
    """Form 0 leaves the final fluxes in the workspace, whose last 15 planes
    they are, on a level whose size picks a fused kernel too; the fused forms
    leave those planes alone.  A level starts by size."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U = _level(([64], [64], [64]), (0,) * 6)
    p = P.params(gamma=1.4, precision=precision)
    real = torch.float32 if precision else torch.float64
    tail = 15 * 66 ** 3
    written = {STAGED: True, BRICKS: False, STREAM: False, BY_SIZE: False, COLUMNS: precision == 1}
    for form, want in list(written.items()) + [(None, False)]:
        lev = P.Level(lay)
        if form is None:
            assert lev.get_step_form() == BY_SIZE
        else:
            lev.set_step_form(form)
        A = U.clone()
        lev.fill_boundary(A)
        B = torch.zeros_like(A)
        lev.ensure_workspace(precision)
        nbytes = lev.workspace_bytes(precision)
        off = (-lev._work.data_ptr()) % 256
        f3 = lev._work[off:off + nbytes].view(real)[-tail:]
        f3.fill_(-7.0)
        lev.hydro_step(A, B, h, p, dt=1e-3)
        torch.cuda.synchronize()
        assert bool((f3 != -7.0).any()) == want, form
        lev.close()
    lev = P.Level(lay)
    for bad in (-1, 5):
        with pytest.raises(P.PPMError, match="step_form"):
            lev.set_step_form(bad)


@pytest.mark.parametrize("bc", [(0, 0, 0, 0, 2, 2), (2, 2, 1, 1, 0, 0), (1, 2, 2, 2, 2, 1)])
@pytest.mark.parametrize("tiling", [([4], [4], [4]), ([1, 7], [3, 1], [2, 5]), ([17], [14], [15]), ([64], [15, 2], [33]),
                                    ([70, 3], [16, 31], [6, 1, 9]), ([61, 1], [2, 40], [3, 16]), ([60], [5], [17])])
def test_columns_agree_with_the_staged_pair_bitwise(tiling, bc):
    """60 to 64 zones along x: rows of about a wavefront's 62 columns."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay, h, U = _level(tiling, bc)
    for mode in (P.BATCHED, P.PER_BOX):
        ref, rs = _step(lay, h, U, STAGED, mode=mode)
        got, gs = _step(lay, h, U, COLUMNS, mode=mode)
        assert rs == gs, (tiling, bc, mode)
        for a, b in zip(ref, got):
            assert torch.equal(a, b), (tiling, bc, mode)
