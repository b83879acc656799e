"""The Riemann solver's arithmetic over strong jumps: one step of a box whose
faces carry shocks, fans and near-vacuum expansions, against the oracle, for
several adiabatic exponents and Newton counts.

Bar: the FP64 parity bar, 1e-12 per field.  A face's flux is 30 to 100
roundings of 2^-53 from the oracle's form, and the update takes differences
of a few such fluxes: some 1e-14 of a field's scale."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1008_2801_amd import inputs as I  # noqa: E402
from paper_1008_2801_amd import ppm as P  # noqa: E402
from tests.helpers import interior, oracle_level  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma,iters,jump", [(1.4, 3, 10.0), (5.0 / 3.0, 3, 1e3), (1.05, 3, 1e2), (1.4, 0, 10.0),
                                              (1.4, 1, 1e3), (1.4, 8, 1e3), (3.0, 16, 1e2)])
def test_step_across_strong_jumps_matches_oracle(gamma, iters, jump):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = (13, 10, 9)
    lay = I.single_box(n)
    h = (1.0 / 16,) * 3
    rng = np.random.default_rng(41)
    k = np.log(jump)
    rho = np.exp(rng.uniform(-0.5 * k, 0.5 * k, n[::-1]))
    p = np.exp(rng.uniform(-0.5 * k, 0.5 * k, n[::-1]))
    c = np.sqrt(gamma * p / rho)
    u = [rng.uniform(-1.0, 1.0, n[::-1]) * c for _ in range(3)]
    wl = I.Workload("jumps", lay, I._fill_state(lay, h, gamma, lambda x, y, z: (rho, u[0], u[1], u[2], p)), h, gamma, 1)
    dt = 0.05 * h[0] / float((np.abs(u).max(axis=0) + c).max())
    ref, _, _, _ = oracle_level(O, wl, 1, dt=dt, riemann_iters=iters)
    lev = P.Level(lay)
    A = torch.from_numpy(wl.arena).cuda()
    B = lev.new_state()
    lev.fill_boundary(A)
    lev.hydro_step(A, B, h, P.params(gamma=gamma, riemann_iters=iters), dt=dt)
    got = interior(lay.view(B.cpu().numpy(), 0))
    want = interior(ref[0])
    for m in range(5):
        scale = np.abs(want[m]).max() if m in (0, 4) else np.sqrt(want[0] * want[4]).max()
        err = np.abs(got[m] - want[m]).max() / scale
        print(f"gamma {gamma:.3f} iters {iters} jump {jump:g} field {m}: {err:.2e}")
        assert err <= 1e-12, (m, err)
