"""Batches (ba_batch_*) whose problems stop at different iterations: an iteration's state in
two buffers, the history written by the S product, restarts of some of the problems."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ba = pytest.importorskip("paper_2110_04015_amd")


# FP32 with subsets of one or two cameras (17 to 32 cameras, N = 16) stops short of 1e-10:
# the inner solves break down on the rounding of their products
@pytest.mark.parametrize("count,N,precision,window",
                         [(c, n, "fp64", w) for c, n in [(2, 4), (7, 16), (27, 3), (27, 16), (3, 1)] for w in (0, 8)] +
                         [(c, n, "fp32", 8) for c, n in [(2, 4), (27, 3), (3, 1)]])
def test_uneven_problems(count, N, precision, window):
    probs = [synth.ring_problem(n_cams=17 + 5 * (k % 4), n_lms=900 + 130 * (k % 7), c_lo=2, c_hi=6, seed=10 + k, name=f"p{k}")
             for k in range(count)]
    b = ba.Batch(probs, store_fp32=precision == "fp32")
    try:
        x, stats, ms, rc = b.mcg(N, 3.3, eps=1e-10, precision=precision, graph_window=window)
        assert rc == 0
        xs = x.detach().cpu().numpy()
        for p, a, c, st in zip(probs, b.row0, b.cams, stats):
            o = oracle.System(p)
            seg = slice(int(a), int(a) + 9 * int(c))
            bt = o.rhs()
            # the stop test bounds the recursive residual (refined solves: the FP64 one) by
            # 1e-10; the recursion drifts from b~ + S x by rounding, far below as much again
            assert np.linalg.norm(o.matvec(xs[seg]) + bt) <= 2e-10 * np.linalg.norm(bt)
            if precision == "fp64":
                # one block per iteration, N columns wide after a failed tau-test
                assert st.history_cols == st.iterations + (N - 1) * st.multi_steps
        # a second solve, and each problem's work, do not depend on what ran before
        x2, stats2, _, _ = b.mcg(N, 3.3, eps=1e-10, precision=precision, graph_window=window)
        assert torch.equal(x, x2)
        assert [s.iterations for s in stats] == [s.iterations for s in stats2]
    finally:
        b.close()
