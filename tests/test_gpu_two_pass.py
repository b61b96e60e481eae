"""The multidirectional product in two passes (landmarks seen from many subsets) against the oracle.

The problems are dense enough for the two-pass form (five subsets or more among a landmark's
observers, on average), at the edges of its work split: one to four tiles of 16 columns and
their remainders, landmarks with more pairs than a row of 16 lanes, cameras with one work-group
and with several, both pose dimensions, new values in place, the skipped problems of a batch, and
systems without room for camera-major records.
"""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ba = pytest.importorskip("paper_2110_04015_amd")

from test_gpu_parity import assert_within_rounding, stored_product  # noqa: E402


def _h(t):
    return t.detach().cpu().numpy()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype=torch.float64)


def problem(name):
    if name == "cap70":       # 5 to 40 observers; cameras from a few to some 900 observations
        return synth.cap_problem(n_cams=70, n_lms=1500, seed=11, name=name)
    if name == "ring64":      # 24 to 40 observers of 64: two and three rounds of pairs
        return synth.ring_problem(n_cams=64, n_lms=257, c_lo=24, c_hi=40, seed=12, name=name, shuffle=True)
    return synth.extrinsics_only(synth.cap_problem(n_cams=65, n_lms=900, seed=13, name=name))


def mean_subsets(p, N):
    grp = oracle.partition(p.n_cams, N)[p.obs_cam]
    pairs = np.unique(p.obs_lm.astype(np.int64) * 64 + grp)
    return float(np.bincount(pairs // 64, minlength=p.n_lms)[p.obs_lm].mean())


def check(p, g, o, N, z, tag, precisions=("fp64", "fp32", "bf16")):
    dp = p.d_p
    grp = np.repeat(oracle.partition(p.n_cams, N), dp)
    for prec in precisions:
        Y = _h(g.matmat_grouped(N, _dev(z), precision=prec))
        assert np.array_equal(Y, _h(g.matmat_grouped(N, _dev(z), precision=prec))), (tag, prec)
        for q in range(N):
            zq = np.where(grp == q, z, 0.0)
            if prec == "fp64":
                ref = o.matvec(zq)
                assert np.abs(Y[q] - ref).max() <= 1e-12 * np.abs(ref).max(), (tag, q)
            else:
                ref, bound = stored_product(p, o, prec, zq)
                assert_within_rounding(Y[q], ref, bound, (tag, prec, q))


@pytest.mark.parametrize("name,N", [("cap70", 9), ("cap70", 16), ("cap70", 17), ("cap70", 33), ("cap70", 64),
                                    ("ring64", 15), ("ring64", 64), ("dp6", 32), ("dp6", 47)])
def test_grouped_product(name, N):
    p = problem(name)
    assert mean_subsets(p, N) >= 5.0
    g = ba.System.from_problem(p)
    z = np.random.default_rng(N).standard_normal(g.n)
    check(p, g, oracle.System(p), N, z, name)
    # new values of the same observations: the camera-major records follow
    q = synth.Problem(**{**p.__dict__, "J_p": 1.25 * p.J_p[::-1].copy(), "J_l": p.J_l[::-1].copy(), "lam": 1e-2})
    g.update(_dev(q.J_p), _dev(q.J_l), _dev(q.r), q.lam)
    check(q, g, oracle.System(q), N, z, name + " updated")
    g.close()


def test_batch_skips_and_layout_change():
    """Problems of a batch on either branch, eager and replayed, and after another partition was asked
    of the batch's system (its layout is made anew, so a captured window must be too)."""
    probs = [synth.cap_problem(n_cams=n, n_lms=40 * n, seed=n, name=f"cap{n}") for n in (24, 40, 33)]
    N, k = 20, 6
    assert min(mean_subsets(p, N) for p in probs) >= 5.0
    b = ba.Batch(probs)
    orc = [oracle.System(p).mcg(N, 3.3, eps=0.0, imax=k) for p in probs]
    z = torch.randn(b.n, dtype=torch.float64, device="cuda")
    for win, other in ((0, 0), (3, 0), (3, 7)):
        if other:
            b.system.matmat_grouped(other, z)
        x, stats, ms, rc = b.mcg(N, 3.3, eps=0.0, max_iter=k, graph_window=win)
        for (xo, so), s, xi in zip(orc, stats, b.split(x)):
            assert s.multi_steps == so.multi_steps
            assert np.linalg.norm(_h(xi) - xo) <= 1e-9 * np.linalg.norm(xo), (win, other)
    b.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_batch_skips_in_reduced_precision(prec):
    """Problems of a batch on either branch of an iteration: each ends with the bits of a batch of its
    own.  (Every chunk is one tile and every sum of a problem runs over that problem alone, in an
    order that does not depend on the others.)"""
    probs = [synth.cap_problem(n_cams=n, n_lms=40 * n, seed=n, name=f"cap{n}") for n in (24, 40, 33)]
    kw = dict(eps=1e-13, max_iter=8, precision=prec, max_outer=1, max_inner=8, inner_eps=1e-13)
    b = ba.Batch(probs)
    x, stats, _, _ = b.mcg(20, 10.0, **kw)
    assert all(0 < s.multi_steps < s.iterations for s in stats)
    for p, xi, s in zip(probs, b.split(x), stats):
        alone = ba.Batch([p])
        y, so, _, _ = alone.mcg(20, 10.0, **kw)
        assert so[0].multi_steps == s.multi_steps and torch.equal(xi, y), p.name
        alone.close()
    b.close()


@pytest.mark.parametrize("name,N", [("cap70", 17), ("ring64", 64), ("dp6", 47)])
def test_without_room_for_records(name, N):
    """The product reads the tile stream then, to the same bits: after a solve whose history fits no
    device, and for a copy that is made in a workspace with room for the copy alone."""
    p = problem(name)
    g = ba.System.from_problem(p)
    z = _dev(np.random.default_rng(N).standard_normal(g.n))
    ref = {}
    for prec in ("fp64", "fp32", "bf16"):
        ref[prec] = g.matmat_grouped(N, z, precision=prec)
    with pytest.raises(ba.BAError) as e:
        g.mcg(N, 3.3, max_history_cols=2 ** 31 - 1)
    assert e.value.status == ba.BA_ERR_NOMEM
    for prec, y in ref.items():
        assert torch.equal(g.matmat_grouped(N, z, precision=prec), y), prec
    tiles = g.info()["n_tiles"]
    g.close()
    kw = dict(ws_groups=N, ws_max_iter=2)
    nbytes = ba.System.from_problem(p, size_only=True, **kw).ws_bytes
    for prec, words in (("fp32", 24), ("bf16", 12)):
        copy = tiles * 64 * words * 4
        ws = torch.empty(nbytes + copy, dtype=torch.uint8, device="cuda")
        g = ba.System.from_problem(p, workspace=ws, **kw)
        assert torch.equal(g.matmat_grouped(N, z, precision=prec), ref[prec]), prec
        assert torch.equal(g.matmat_grouped(N, z), ref["fp64"]), prec
        g.close()


def test_first_use_in_a_workspace():
    """Subsets that no layout was reserved for take no records from the caller's workspace."""
    p = synth.cap_problem(n_cams=24, n_lms=60000, seed=14, name="cap24")
    N = 12
    assert mean_subsets(p, N) >= 5.0
    nbytes = ba.System.from_problem(p, size_only=True).ws_bytes
    ws = torch.empty(nbytes + 24 * 8 * p.n_obs, dtype=torch.uint8, device="cuda")
    g = ba.System.from_problem(p, workspace=ws)
    check(p, g, oracle.System(p), N, np.random.default_rng(N).standard_normal(g.n), "cap24", ("fp64",))
    g.close()
