"""b~, D(S) and its factor at the edges of the camera sums' work split: cameras with one
observation more or fewer than a wavefront (64) and a work-group (256) take, both pose
dimensions, at the build, after new values in place and after a new lambda."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ba = pytest.importorskip("paper_2110_04015_amd")


def _h(t):
    return t.detach().cpu().numpy()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype=torch.float64)


def check(g, o, n, tag):
    D, ref = _h(g.precond_blocks()), o.D_blocks()
    assert np.abs(D - ref).max() <= 1e-12 * np.abs(ref).max(), tag
    b, bref = _h(g.rhs()), o.rhs()
    assert np.abs(b - bref).max() <= 1e-12 * np.abs(bref).max(), tag
    r = np.random.default_rng(n).standard_normal(g.n)
    z, zref = _h(g.precond(_dev(r))), o.precond(r)
    assert np.abs(z - zref).max() <= 1e-10 * np.abs(zref).max(), tag   # kappa <= 9 (1 + lambda) / lambda once scaled by diag(U)


@pytest.mark.parametrize("dp", [9, 6])
@pytest.mark.parametrize("n_lms", [30, 63, 64, 65, 255, 256, 257, 513])
def test_camera_sums(n_lms, dp):
    p = synth.tiny(n_cams=4, n_lms=n_lms, seed=n_lms, c_lo=4, c_hi=4, lam=1e-1, shuffle=True)   # every camera sees all
    if dp == 6:
        p = synth.extrinsics_only(p)
    g = ba.System.from_problem(p)
    check(g, oracle.System(p), n_lms, "built")
    q = synth.Problem(**{**p.__dict__, "J_p": 0.75 * p.J_p, "r": p.r[::-1].copy(), "lam": 1e-2})
    g.update(_dev(q.J_p), _dev(q.J_l), _dev(q.r), q.lam)
    check(g, oracle.System(q), n_lms, "updated")
    g.set_lambda(0.5)
    check(g, oracle.System(q, lam=0.5), n_lms, "lambda")
    g.close()
