"""The chunks of the one-column product: their number follows from the problem's size and the
device, FP32 and BF16 copies have chunks of their own, and back-substitution shares a chunk
between wavefronts.  Against the FP64 oracle (products 1e-12 of the largest entry in FP64; the
FP32 and BF16 terms of the S product within 64 roundings of the sum of their sizes)."""
import numpy as np
import pytest

import oracle
import synth
from oracle import reduced as R

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ba = pytest.importorskip("paper_2110_04015_amd")

from test_gpu_parity import assert_within_rounding, stored_product  # noqa: E402


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype=torch.float64)


# one tile; fewer tiles than chunks would be made; one more than that; several per chunk; a
# dense problem whose chunks see more than 128 cameras
@pytest.mark.parametrize("make", [
    lambda: synth.ring_problem(n_cams=5, n_lms=9, c_lo=2, c_hi=4, seed=1, name="ring5"),
    lambda: synth.ring_problem(n_cams=40, n_lms=5000, c_lo=2, c_hi=8, seed=2, name="ring40"),
    lambda: synth.ring_problem(n_cams=60, n_lms=9700, c_lo=2, c_hi=8, seed=3, name="ring60"),
    lambda: synth.walk_problem(n_cams=150, n_lms=26000, seed=4, name="walk150"),
    lambda: synth.cap_problem(n_cams=300, n_lms=24000, seed=5, name="cap300"),
], ids=["ring5", "ring40", "ring60", "walk150", "cap300"])
def test_products_and_back_substitution(make):
    p = make()
    o = oracle.System(p)
    v = np.random.default_rng(6).standard_normal(9 * p.n_cams)
    ref = o.matvec(v)
    plain = ba.System.from_problem(p)
    g = ba.System.from_problem(p, store_fp32=True, store_bf16=True)
    try:
        y = plain.matvec(_dev(v))
        assert np.abs(y.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
        assert torch.equal(g.matvec(_dev(v)), y)   # whatever copies are kept
        lamd = R.lambda_diag(o.U_blocks(), p.lam)
        for prec in ("fp32", "bf16"):
            yr, ya = R.schur_matvec_stored(p.obs_cam, p.obs_lm, p.n_cams, p.n_lms, R.stored(p.J_p, prec),
                                           R.stored(p.J_l, prec), o.Vinv_blocks(), lamd, v)
            y16 = g.matvec(_dev(v), precision=prec)
            assert np.all(np.abs(y16.cpu().numpy() - yr) <= 64 * 2.0 ** -24 * ya), prec
            assert torch.equal(g.matvec_noalloc(_dev(v), torch.empty_like(y), precision=prec), y16)
            assert torch.equal(plain.matvec(_dev(v), precision=prec), y16)   # a copy made when asked for
        assert torch.equal(plain.matvec(_dev(v)), y)
        step = 1e-3 * v
        dl = g.back_substitute(_dev(step)).cpu().numpy().reshape(-1)
        rl = np.asarray(o.back_substitute(step)).reshape(-1)
        assert np.abs(dl - rl).max() <= 1e-11 * np.abs(rl).max()
    finally:
        plain.close()
        g.close()


@pytest.mark.parametrize("make", [
    lambda: synth.walk_problem(n_cams=150, n_lms=26000, seed=4, name="walk150"),   # few camera rows a tile
    lambda: synth.cap_problem(n_cams=300, n_lms=24000, seed=5, name="cap300"),     # many
    lambda: synth.ring_problem(n_cams=60, n_lms=9700, c_lo=2, c_hi=18, seed=6, name="ring60"),   # a tile a chunk
], ids=["walk150", "cap300", "ring60"])
def test_copies_of_poses_without_intrinsics(make):
    p = synth.extrinsics_only(make())
    o = oracle.System(p)
    v = np.random.default_rng(8).standard_normal(6 * p.n_cams)
    g = ba.System.from_problem(p, store_fp32=True, store_bf16=True)
    try:
        for prec in ("fp32", "bf16"):
            ref, bound = stored_product(p, o, prec, v)
            assert_within_rounding(g.matvec(_dev(v), precision=prec).cpu().numpy(), ref, bound, prec)
    finally:
        g.close()


@pytest.mark.parametrize("prec,words", [("fp32", 24), ("bf16", 12)])
def test_workspace_without_room_for_the_copys_chunks(prec, words):
    """A copy made when asked for, in a workspace that has no room for its chunk arrays: the
    product takes the FP64 product's chunks and nothing but the copy is taken."""
    p = synth.walk_problem(n_cams=150, n_lms=26000, seed=4, name="walk150")
    v = _dev(np.random.default_rng(7).standard_normal(9 * p.n_cams))
    nbytes = ba.System.from_problem(p, size_only=True).ws_bytes
    plain = ba.System.from_problem(p)
    copy = plain.info()["n_tiles"] * 64 * words * 4
    ws = torch.empty(nbytes + copy + 40_000, dtype=torch.uint8, device="cuda")
    g = ba.System.from_problem(p, workspace=ws)
    try:
        used = g.workspace_used()
        y = g.matvec(v, precision=prec)
        assert used + copy <= g.workspace_used() < used + copy + 256
        # the same partial products, added up over other chunks in FP64
        yp = plain.matvec(v, precision=prec)
        assert (y - yp).abs().max() <= 1e-12 * yp.abs().max()
    finally:
        plain.close()
        g.close()


@pytest.mark.parametrize("prec,words", [("fp32", 24), ("bf16", 12)])
def test_copy_takes_nothing_else_from_a_workspaces_spare_room(prec, words):
    """A copy made when asked for, in a workspace with room for its chunk arrays as well: they were
    not counted, so what is left is for what the caller has in mind (a solve of its own, here)."""
    p = synth.walk_problem(n_cams=150, n_lms=26000, seed=4, name="walk150")
    v = _dev(np.random.default_rng(7).standard_normal(9 * p.n_cams))
    nbytes = ba.System.from_problem(p, size_only=True, ws_groups=1, ws_max_iter=300).ws_bytes
    plain = ba.System.from_problem(p)
    copy = plain.info()["n_tiles"] * 64 * words * 4
    # (vectors that the solve needs longer are taken anew: some kilobytes, a tenth of the chunk arrays at most)
    ws = torch.empty(nbytes + copy + 65536, dtype=torch.uint8, device="cuda")
    g = ba.System.from_problem(p, workspace=ws)
    try:
        used = g.workspace_used()
        g.matvec(v, precision=prec)
        assert used + copy <= g.workspace_used() < used + copy + 256
        x, st = g.mcg(1, 3.3, max_iter=300)
        y, su = plain.mcg(1, 3.3, max_iter=300)
        assert torch.equal(x, y) and st.iterations == su.iterations
    finally:
        plain.close()
        g.close()
