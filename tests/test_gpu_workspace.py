"""Systems built into a caller-owned workspace (ba_build_workspace_bytes,
ba_build_system_ws) against systems whose memory the library allocates.

  - The sizing pass's byte count is exact: a build into exactly that many bytes succeeds
    and uses them all (after the reserved solves have run too), and one 256 bytes short
    fails with BA_ERR_WORKSPACE.
  - Same layout, same kernels: S v (FP64 and a stored FP32 copy), b~, D(S), the
    multidirectional product, and PCG / MCG / mixed-precision solves equal the ordinary
    build's bit for bit, for an implicit and an explicit S.
  - Solves outside the reservation (another N) fail with BA_ERR_WORKSPACE and leave the
    system usable; ba_set_lambda and ba_update_system work in place.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ba = pytest.importorskip("paper_2110_04015_amd")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype=torch.float64)


def _same(a, b):
    torch.cuda.synchronize()
    return torch.equal(a, b)


@pytest.mark.parametrize("name,explicit", [("walk200", False), ("ring50", True), ("cap120", False)])
def test_workspace_build_equals_library_build(name, explicit):
    print(f"\n[case] workspace build {name} explicit={explicit}", flush=True)
    p = {"walk200": lambda: synth.walk_problem(n_cams=200, n_lms=20_000, seed=3),
         "ring50": lambda: synth.config0(seed=1),
         "cap120": lambda: synth.cap_problem(n_cams=120, n_lms=5000, seed=4)}[name]()
    N, its = 8, 300
    kw = dict(store_fp32=True, explicit_schur=explicit, ws_groups=N, ws_max_iter=its)
    nbytes = ba.System.from_problem(p, size_only=True, **kw).ws_bytes
    assert nbytes > 0 and nbytes % 256 == 0
    short = torch.empty(nbytes - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(ba.BAError) as e:
        ba.System.from_problem(p, workspace=short, **kw)
    assert e.value.status == ba.BA_ERR_WORKSPACE
    del short
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    g = ba.System.from_problem(p, workspace=ws, **kw)
    ref = ba.System.from_problem(p, **kw)
    v = _dev(np.random.default_rng(1).standard_normal(g.n))
    assert _same(g.matvec(v), ref.matvec(v))
    assert _same(g.matvec(v, precision="fp32"), ref.matvec(v, precision="fp32"))
    assert _same(g.rhs(), ref.rhs()) and _same(g.precond_blocks(), ref.precond_blocks())
    assert _same(g.matmat_grouped(N, v), ref.matmat_grouped(N, v))
    for f in (lambda s: s.pcg(max_iter=its, trace=True), lambda s: s.mcg(N, 3.3, max_iter=its),
              lambda s: s.mcg(N, 3.3, max_iter=its, precision="fp32"), lambda s: s.mcg(1, 3.3, max_iter=its)):
        xa, sa = f(g)
        xb, sb = f(ref)
        assert _same(xa, xb) and sa.iterations == sb.iterations and sa.status == sb.status
    assert g.workspace_used() <= nbytes
    assert g.workspace_used() > nbytes - 256     # the reservation covered every solve: nothing more was taken
    # outside the reservation: another N
    with pytest.raises(ba.BAError) as e:
        g.mcg(N + 1, 3.3, max_iter=its)
    assert e.value.status == ba.BA_ERR_WORKSPACE
    xa, sa = g.mcg(N, 3.3, max_iter=its)       # still usable
    assert sa.status == ba.BA_OK
    # a new lambda in place
    g.set_lambda(1e-2)
    ref.set_lambda(1e-2)
    assert _same(g.matvec(v), ref.matvec(v))
    g.close()
    ref.close()
    del ws


def test_memory_per_observation():
    """What a system keeps is what its kernels read: per tile slot the FP64 record, the observation
    and the slot word; per observation its places in the camera order; and the sums and tables of
    landmarks, cameras and chunks.  A map of eight bytes per observation would be 4.8 MB more."""
    p = synth.ring_problem(n_cams=64, n_lms=10_000, c_lo=60, c_hi=60, seed=5)
    g = ba.System.from_problem(p)
    info = g.info()
    g.close()
    slots, m = 64 * info["n_tiles"], p.n_obs
    blocks = m // 256 + p.n_cams
    kept = (slots * (24 * 8 + 8 + 4) + m * (8 + 4 + 4 + 4) + p.n_lms * (18 * 8 + 4 + 4 + 8 + 4) +
            info["n_chunks"] * p.n_cams * (9 * 8 + 4 + 4) + blocks * (108 * 8 + 12))
    nbytes = ba.System.from_problem(p, size_only=True).ws_bytes
    assert nbytes <= kept + 1_000_000   # cameras' blocks, a PCG solve's vectors, alignment
