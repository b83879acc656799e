"""Two steps of one context in flight on two streams, each with a workspace of
its own, with the same dt and spacings (the context's step constants): each
leaves the state and the next dt that it leaves alone, whatever the other's
speeds are."""
import pytest

torch = pytest.importorskip("torch")

from paper_1008_2801_amd import inputs as I  # noqa: E402
from paper_1008_2801_amd import ppm as P  # noqa: E402

pytestmark = pytest.mark.gpu


# levels whose final stage is staged (32^3), in bricks (96^3) and in columns
# (200^3 FP64) by size
@pytest.mark.parametrize("n,precision", [(32, 0), (96, 0), (96, 1), (200, 0)])
def test_steps_in_flight_on_two_streams_keep_their_next_dt(n, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lay = I.single_box(n)
    lev = P.Level(lay)
    h = (1.0 / n,) * 3
    p = P.params(gamma=1.4, precision=precision)
    g = torch.Generator(device="cuda").manual_seed(5)
    states = []
    for scale in (9.0, 1.0):  # pressures: speeds about three times apart
        U = lev.new_state()
        v = U.view(5, -1)
        v[0] = 1.0 + 0.1 * torch.rand(v.shape[1], generator=g, device="cuda", dtype=torch.float64)
        v[1:4] = 0.1 * torch.rand(3, v.shape[1], generator=g, device="cuda", dtype=torch.float64)
        v[4] = scale * (2.5 + 0.1 * torch.rand(v.shape[1], generator=g, device="cuda", dtype=torch.float64))
        lev.fill_boundary(U)
        states.append(U)
    out = [torch.zeros_like(U) for U in states]
    nxt = torch.zeros(2, 2, dtype=torch.float64, device="cuda")
    dt = 0.05 / n
    streams = [torch.cuda.Stream() for _ in range(2)]

    def step(k, stream=None):
        lev.select_workspace(k, precision)
        lev.hydro_step(states[k], out[k], h, p, dt=dt, dt_next=nxt[k], stream=stream)
    ref = []
    for k in range(2):
        step(k)
        torch.cuda.synchronize()
        ref.append((out[k].clone(), nxt[k].clone()))
    assert ref[0][1][0] < 0.5 * ref[1][1][0]
    for order in ((0, 1), (1, 0)) * 4:
        nxt.fill_(-1.0)
        torch.cuda.synchronize()
        for k in order:
            step(k, streams[k])
        torch.cuda.synchronize()
        for k in range(2):
            assert torch.equal(nxt[k], ref[k][1]), (order, k, nxt[k].tolist(), ref[k][1].tolist())
            assert torch.equal(out[k], ref[k][0]), (order, k)
    assert lev.check_status() == 0
    lev.release_workspace_slots()
    lev.close()
