"""The splat's gather form (dc_weight_radon, dc_detector_bp_adjoint where bins are as
wide as pixels and at most twice as wide) at the sizes where its tables change:
angle groups of 4, 2 and 1, a last view group of 1 to 4 views, blocks of rows that
do not divide the image, lines shorter than a wave, anisotropic pixels, the widest
bins it takes, and sinograms shorter than the detector diagonal.

Two forms.  dc_detector_bp_adjoint into float32 rounds each pixel to the view's unit
(largest / qmax) and sums at most 64 rows of one column in float32 (rounding below
sqrt(64) 2^-25 = 2.4e-7 of the sum, rms), the column sums as 32-bit integers (finer).
The others put two integers, each rounded to the unit, on two bins.  qmax is at least
2^31 / (pixels of a bin, below 700 here), and at most 2^21: a unit of 5e-7 of the
largest pixel, rounded twice with an rms of 0.29 units each, against pixels of an rms
of 0.58 of it: 3.5e-7.  So 1e-6 in relative L2 for both.  Into bfloat16 the second form
is compared bit for bit with the same integer sums formed in numpy."""
import math

import numpy as np
import pytest

import synth
from oracle import pipeline as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-6
# nu, nv, dv / du, n_theta, ds / du, n_s (0: the diagonal), views
CASES = {
    "groups-of-4": (128, 96, 1.0, 360, 1.0, 0, 5),
    "groups-of-2": (70, 53, 1.0, 180, 1.0, 0, 3),
    "single-angles": (33, 150, 1.0, 37, 1.0, 0, 4),
    "thin": (5, 67, 1.0, 41, 1.0, 0, 1),
    "anisotropic": (61, 90, 0.8, 200, 1.0, 0, 6),
    "wide-bins": (64, 64, 1.0, 360, 1.4, 0, 2),
    "short-rows": (64, 48, 1.0, 90, 1.0, 40, 7),
}


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.mark.parametrize("name", sorted(CASES))
def test_splat_gather_against_the_oracle(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    nu, nv, av, n_theta, ws, n_s, V = CASES[name]
    du = 1.1
    g = synth.Grid(nu=nu, nv=nv, du=du, dv=av * du, n_theta=n_theta, n_s=n_s or synth.radon_bins(nu, nv), ds=ws * du,
                   nx=6, ny=5, nz=4, vx=1.0, vy=1.0, vz=1.0)
    views = synth.sinusoid_orbit(V, 750.0, 1200.0)
    plan = P.Plan(g, views)
    print("\n[gpu splat gather]", name, g.as_dict(), flush=True)
    pos = synth.rand_array((V, nv, nu), 5, 0.0, 1.0) * np.float32(3.0) ** np.arange(V, dtype=np.float32)[:, None, None]
    sgn = synth.rand_array((V, nv, nu), 6)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    host = lambda t: t.double().cpu().numpy()
    R = torch.full((V, n_theta, g.n_s), float("nan"), device="cuda")
    P.dc_weight_radon(plan, dev(pos), R)
    GH = torch.full_like(R, float("nan"))
    P.dc_detector_bp_adjoint(plan, dev(sgn), GH)
    ref, refh = O.weight_radon(pos.astype(np.float64), g, views), O.detector_bp_adjoint(sgn.astype(np.float64), g)
    for v in range(V):
        assert rel(host(R)[v], ref[v]) < TOL and rel(host(GH)[v], refh[v]) < TOL, (v, rel(host(R)[v], ref[v]))
    # a view's sums do not depend on the views beside it, nor on the run
    part = torch.full_like(R, -7.0)
    v0 = V // 2
    P.dc_weight_radon(plan, dev(pos), part, v0=v0, nv=V - v0)
    assert torch.equal(part[v0:], R[v0:]) and bool((part[:v0] == -7.0).all())
    # storage types: the unrounded result to the nearest bfloat16 (half a unit is at most 2^-8 of a
    # value) or float16 (2^-11, and 2^-25 among the subnormals), which R is within 2^-24 of
    for dt, half, tiny in ((torch.bfloat16, 2.0 ** -8, 0.0), (torch.float16, 2.0 ** -11, 2.0 ** -25)):
        low = torch.empty((V, n_theta, g.n_s), device="cuda", dtype=dt)
        P.dc_weight_radon(plan, dev(pos), low)
        err, r = np.abs(host(low) - host(R)), np.abs(host(R))
        assert np.all(err <= (half + 2.0 ** -23) * r + tiny)
    # a view of zeros, and one far below the others, keep their own scale
    pos[0] = 0.0
    pos[V - 1] *= np.float32(1e-20)
    P.dc_weight_radon(plan, dev(pos), R)
    if V > 1:
        assert not host(R)[0].any() and rel(host(R)[V - 1], 1e-20 * ref[V - 1]) < TOL
    plan.close()


def integer_terms(img, g, kgrid):
    """One view's unit S and its sums of round(x S) - round(x S f) and round(x S f)."""
    A, B, C, qmax = kgrid
    S = np.float32(np.float32(qmax) / np.float32(np.abs(img).max()))
    # round(x S) of the unrounded product (exact in float64), round(xs f) of the float32 one
    qa = np.rint(img.astype(np.float64) * float(S)).astype(np.int64)
    xs2 = (img * S * np.float32(2.0 ** -32)).astype(np.float64)
    out = np.zeros((g.n_theta, g.n_s))
    for k in range(g.n_theta):
        col = abs(B[k]) > abs(A[k])
        line, walk = (np.arange(g.nv), np.arange(g.nu)) if col else (np.arange(g.nu), np.arange(g.nv))
        step = int(np.rint((A[k] if col else B[k]) * 2.0 ** 32))
        # one rounding of line * slope + C, as a fused multiply-add rounds it
        slope = B[k] if col else A[k]
        t0 = np.array([float(np.longdouble(l) * np.longdouble(slope) + np.longdouble(C[k])) for l in line])
        fl = np.floor(t0)
        T = (fl.astype(np.int64) << 32) + ((t0 - fl) * 2.0 ** 32).astype(np.int64)
        T = T[:, None] + walk[None, :].astype(np.int64) * step
        if not col:
            T = T.T
        m, lo = T >> 32, (T & 0xffffffff).astype(np.float32).astype(np.float64)
        qb = np.rint(xs2 * lo).astype(np.int64)   # the product of two float32 is exact
        for bins, q in ((m, qa - qb), (m + 1, qb)):
            ok = (bins >= 0) & (bins < g.n_s)
            out[k] += np.bincount(bins[ok], weights=q[ok], minlength=g.n_s)
    return S, out


@pytest.mark.parametrize("name", sorted(CASES))
def test_splat_gather_integer_terms(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_14900_amd as P
    nu, nv, av, n_theta, ws, n_s, V = CASES[name]
    du = 1.1
    g = synth.Grid(nu=nu, nv=nv, du=du, dv=av * du, n_theta=n_theta, n_s=n_s or synth.radon_bins(nu, nv), ds=ws * du,
                   nx=6, ny=5, nz=4, vx=1.0, vy=1.0, vz=1.0)
    plan = P.Plan(g, synth.sinusoid_orbit(V, 750.0, 1200.0))
    print("\n[gpu splat gather] integer terms", name, g.as_dict(), flush=True)
    sgn = synth.rand_array((V, nv, nu), 6).astype(np.float32)
    out = torch.full((V, n_theta, g.n_s), float("nan"), device="cuda", dtype=torch.bfloat16)
    P.dc_detector_bp_adjoint(plan, torch.as_tensor(sgn, device="cuda"), out)
    mu = [k * math.pi / n_theta for k in range(n_theta)]
    A = [g.du * math.cos(m) / g.ds for m in mu]
    B = [g.dv * math.sin(m) / g.ds for m in mu]
    x0, y0 = -0.5 * (nu - 1) * g.du, -0.5 * (nv - 1) * g.dv
    C = [(x0 * math.cos(m) + y0 * math.sin(m)) / g.ds + 0.5 * (g.n_s - 1) for m in mu]
    terms = 1
    for a, b in zip(A, B):
        a, b = abs(a), abs(b)
        t = min((math.floor(1 / a) + 1 if a > 0 else 1e30) * nv, (math.floor(1 / b) + 1 if b > 0 else 1e30) * nu)
        terms = max(terms, int(min(t, nu * nv)))
    qmax = min(2147483647 // terms - 1, 2 ** 21)
    for v in (0, V - 1):
        S, sums = integer_terms(sgn[v], g, (A, B, C, qmax))
        inv = float(np.float32(math.pi / n_theta)) / float(S)
        want = torch.as_tensor((sums * inv).astype(np.float32)).to(torch.bfloat16)
        assert torch.equal(out[v].cpu(), want), (v, float((out[v].cpu().float() - want.float()).abs().max()))
    plan.close()
