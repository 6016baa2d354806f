"""The Gaussian smoothing at the edges of its blocks of 12 outputs: lines of one block,
whole blocks and one sample more or less, tap counts of every remainder of 4 and 16,
radii that reach both ends of a line, last strips of every width and workgroups whose
last lines are missing, out of place and in place, forward and transpose.

Tolerance: positive samples and taps; each of the two passes rounds at most 2 r + 1 <= 143
partial sums by 2^-25 of themselves (rms), so sqrt(2 143) 2^-25 = 5.0e-7 with all of them as
large as the result: 1e-6 in relative L2."""
import numpy as np
import pytest

import synth
from oracle import smooth as OS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# n_theta, n_s, radius, views
CASES = [(12, 24, 1, 1), (13, 23, 2, 2), (24, 25, 11, 3), (11, 40, 10, 9), (36, 37, 35, 2), (90, 91, 7, 5),
         (47, 300, 46, 4), (180, 72, 71, 2), (361, 145, 60, 1), (25, 1381, 24, 2)]


@pytest.mark.parametrize("case", CASES)
def test_smooth_blocks_against_the_oracle(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    K, S, r, V = case
    g = synth.Grid(nu=8, nv=6, du=1.0, dv=1.0, n_theta=K, n_s=S, ds=1.0, nx=4, ny=4, nz=4, vx=1.0, vy=1.0, vz=1.0)
    print("\n[gpu smooth blocks]", case, flush=True)
    plan = P.Plan(g, synth.sinusoid_orbit(V, 750.0, 1200.0))
    x = synth.rand_array((V, K, S), 3, 0.1, 1.0).astype(np.float32)
    sigma = 0.4 * r + 0.3
    for fn, ref in ((P.dc_smooth_weights, OS.smooth_weights), (P.dc_smooth_weights_adjoint, OS.smooth_weights_adjoint)):
        d = torch.as_tensor(x, device="cuda")
        y = torch.full_like(d, float("nan"))
        fn(plan, d, y, sigma, r)
        want = ref(x.astype(np.float64), sigma, r)
        got = y.double().cpu().numpy()
        assert np.linalg.norm(got - want) < 1e-6 * np.linalg.norm(want), np.linalg.norm(got - want) / np.linalg.norm(want)
        fn(plan, d, d, sigma, r)   # in place
        assert torch.equal(d, y)
        part = torch.full_like(d, -3.0)
        fn(plan, torch.as_tensor(x, device="cuda"), part, sigma, r, v0=V // 2, nv=V - V // 2)
        assert torch.equal(part[V // 2:], y[V // 2:]) and bool((part[:V // 2] == -3.0).all())
    plan.close()
