"""Orthogonalisation kernels of the one-vector GMRES where their launch shape or
their chunking changes: vectors of one block, of a partial last block and on
both sides of the length (2^18) from which a finishing kernel sums the
partials, odd lengths, and cycles of more than 32 basis vectors, with one and
two Gram-Schmidt passes.

The oracle's GMRES (modified Gram-Schmidt) is the reference: iteration counts
within 2 per step with two passes (at tol 1e-8: at 1e-12 the oracle's update
x += P^{-1}(V y) can leave its true residual just above the tolerance and take a
further cycle, 64 iterations against the flexible form's 61 at 71^2, restart
64), the solution against the dense LU to 1e-10 relative (tol 1e-12) on small
grids, and on the large ones the true residual recomputed by the oracle, at most
(tol + 1e-12) ||b||.
"""

import numpy as np
import pytest
import torch

import oracle as O
from workloads.configs import domain_mask, make_config, SHAPES

pytestmark = pytest.mark.gpu

rsfde = pytest.importorskip("paper_2102_11576_amd")
from paper_2102_11576_amd import RsfdePlan, make_opts  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV).reshape(-1)


@pytest.mark.parametrize("name,n,restart,reorth,side", [
    ("c1", 3, 20, 0, "right"),      # N = 9: one block, most lanes idle
    ("c1", 15, 20, 0, "right"),     # N = 225: one block
    ("c1", 16, 20, 0, "left"),      # N = 256: one full block
    ("c1", 17, 20, -1, "right"),    # N = 289: a second, partial block; one pass
    ("c3", 71, 32, 0, "right"),     # cycles of exactly 32 vectors
    ("c3", 71, 33, 0, "right"),     # one vector more: two chunks
    ("c3", 71, 64, 0, "right"),     # two full chunks
    ("c3", 71, 64, 0, "left"),
    ("c3", 71, 64, -1, "right"),
])
def test_one_vector_solve_matches_lu(name, n, restart, reorth, side):
    w = make_config(name, n=n, m=2)
    p = O.problem_from_workload(w)
    ref = O.march_lu(p, w.u0, w.m, w.f_kind)
    with RsfdePlan.from_workload(w, max_restart=restart) as pl:
        u, _, _ = pl.march(_t(w.u0), w.m, w.f_kind,
                           make_opts(restart, 100000, 1e-12, sstep=0, reorth=reorth, side=side))
        _, its, _ = pl.march(_t(w.u0), w.m, w.f_kind,
                             make_opts(restart, 100000, 1e-8, sstep=0, reorth=reorth, side=side))
        u = u.cpu().numpy().reshape(w.n2, w.n1)
    assert np.abs(u - ref).max() / np.abs(ref).max() <= (1e-10 if side == "right" else 1e-9)
    if reorth == 0:  # one classical pass may lose orthogonality and take more
        _, it_ref = O.march_gmres(p, w.u0, w.m, w.f_kind, restart, 1e-8, side=side)
        assert all(abs(a - b) <= 2 for a, b in zip(its, it_ref)), (its, it_ref)


# N = 262143 and 262144: the consumers sum the partials; 262656 (even) and 264195
# (odd): a finishing kernel does
@pytest.mark.parametrize("n1,n2", [(511, 513), (512, 512), (513, 512), (513, 515)])
def test_one_vector_step_around_the_length_limit(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["disk"](0.5, 0.5, 0.4))
    p = O.Problem(n1, n2, box, 1.3, 1.6, 1.0, 1.0, 1e-6, 1.0 / 32, mask)
    x, y = np.arange(1, n1 + 1) / (n1 + 1), np.arange(1, n2 + 1) / (n2 + 1)
    u = np.exp(-40.0 * ((x[None, :] - 0.45) ** 2 + (y[:, None] - 0.55) ** 2)) * mask
    tol = 1e-8
    b = O.rhs(p, u, O.F_LOGISTIC)
    lam = O.tau_eigs_xy(p)
    _, it_ref, ok = O.gmres(lambda V: O.matvec_fast(p, V), b, u, 30, tol,
                            Pinv=lambda V: O.precond_apply_fft(p, V, lam))
    assert ok
    with RsfdePlan(n1, n2, box, 1.3, 1.6, 1.0, 1.0, torch.as_tensor(mask), 1e-6, 1.0 / 32) as pl:
        out, st = pl.step(_t(u), None, O.F_LOGISTIC, make_opts(30, 10000, tol, sstep=0))
        out = out.cpu().numpy().reshape(n2, n1)
    r = np.linalg.norm(b - O.matvec_fast(p, out)) / np.linalg.norm(b)
    assert r <= tol + 1e-12, r
    assert abs(st.iters - it_ref) <= 2, (st.iters, it_ref)


# N = 1046529 (odd): 256 blocks, chunks of 32 and 16 vectors, and the one-pass form
@pytest.mark.parametrize("reorth", [0, -1])
def test_long_vectors_in_two_chunks(reorth):
    w = make_config("c2", n=1023)
    p = O.problem_from_workload(w)
    tol = 1e-8
    with RsfdePlan.from_workload(w, max_restart=48) as pl:
        out, st = pl.step(_t(w.u0), None, w.f_kind, make_opts(48, 1000, tol, sstep=0, reorth=reorth))
        out = out.cpu().numpy().reshape(w.n2, w.n1)
    b = O.rhs(p, w.u0, w.f_kind)
    assert np.linalg.norm(b - O.matvec_fast(p, out)) <= (tol + 1e-12) * np.linalg.norm(b)
    assert st.iters > 32 and st.status == 0
