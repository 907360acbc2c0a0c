"""The smallest lattice, 2^4, where the forward and backward neighbour along
every axis is the same site and every Dirichlet block is a single tile: the
GPU operators against the oracle, and GPU solves against an LU solve of the
full dense matrix built from the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import TOL, ctx, np_of, on_parity, rel  # noqa: F401
from util_fields import dense_matrix

pytestmark = pytest.mark.gpu

L = pytest.importorskip("paper_1109_2935_amd.lqcd")
from paper_1109_2935_amd import ops  # noqa: E402

DIMS = (2, 2, 2, 2)


@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (1, 12), (2, 12), (3, 18)])
def test_wilson_dslash_2x2x2x2(ctx, prec, recon):
    U = synth.gauge_field(DIMS, 0.25, 121)
    psi = synth.gaussian_spinor(DIMS, 122)
    o = ops.wilson_clover(ctx, U, DIMS, 0.124, 1.0, prec, recon)
    for p in (0, 1):
        for dagger in (0, 1):
            src = on_parity(psi, oracle.parity_mask(DIMS, 1 - p))
            out = o.spinor()
            L.lqcd_dslash(ctx, o.op, out, o.import_spinor(src, 1 - p), p, dagger)
            ref = oracle.wilson_dslash(DIMS, U, src, out_parity=p, dagger=bool(dagger))
            assert rel(np_of(o.export_spinor(out, p)), ref) < TOL[prec]


@pytest.mark.parametrize("precond", [0, 1])
def test_gcr_2x2x2x2_against_dense_lu(ctx, precond):
    U = synth.gauge_field(DIMS, 0.25, 123)
    b = synth.gaussian_spinor(DIMS, 124)
    op = oracle.WilsonClover(DIMS, U, 0.124, 1.0, bc_t=-1)
    M, _ = dense_matrix(op.M, oracle.shape4(DIMS) + (4, 3))
    ref = np.linalg.solve(M, b.reshape(-1)).reshape(b.shape)
    Ud = torch.from_numpy(U).cuda()
    o64 = ops.wilson_clover(ctx, U, DIMS, 0.124, 1.0, 0, 18, U_device=Ud)
    o32 = ops.wilson_clover(ctx, U, DIMS, 0.124, 1.0, 1, 18, U_device=Ud)
    x = o64.spinor(full=True)
    prm = ops.gcr_params(1e-10, 8, 1e-3, precond=precond, block=DIMS, mr_steps=4)
    st, info = L.lqcd_gcr_solve(ctx, o64.op, o32.op, o32.op if precond else None, prm, x, o64.import_spinor(b, -1))
    assert st == L.LQCD_OK, L.lqcd_last_error(ctx)
    xs = np_of(o64.export_spinor(x, -1))
    assert np.linalg.norm(b - op.M(xs)) / np.linalg.norm(b) <= 1.05e-10
    assert rel(xs, ref) < 1e-8


def test_staggered_cg_2x2x2x2_against_dense_lu(ctx):
    U = synth.gauge_field(DIMS, 0.2, 125)
    fat = synth.fat_links(DIMS, U, seed=126)
    chi = synth.gaussian_spinor(DIMS, 127, inner=(3,))
    even = oracle.parity_mask(DIMS, 0)
    b = np.where(even[..., None], chi, 0)
    stag = oracle.Staggered(DIMS, fat, oracle.long_links(DIMS, U), 0.01)
    N, idx = dense_matrix(stag.normal_even, oracle.shape4(DIMS) + (3,), mask=even)
    ref = np.linalg.solve(N, b.reshape(-1)[idx])
    o = ops.staggered(ctx, fat, U, DIMS, 0.01, 0, 18)
    x = o.spinor()
    st, info = L.lqcd_cg_solve(ctx, o.op, None, ops.cg_params(1e-10, 1000, 0.1, L.LQCD_CG_STAG_NORMAL), x,
                               o.import_spinor(b, 0))
    assert st == L.LQCD_OK, L.lqcd_last_error(ctx)
    xs = np_of(o.export_spinor(x, 0)).reshape(-1)[idx]
    assert rel(xs, ref) < 1e-8


# CGNE in one precision on at most 16384 even sites iterates without a host round
# trip; a solve that records its iterates takes the host's loop. Both run the
# same recurrences (sums in another order): less than one workgroup, a workgroup
# that is not full, several, the largest size, and the first beyond it.
@pytest.mark.parametrize("dims,recon", [((2, 2, 2, 2), 18), ((6, 2, 6, 2), 12), ((8, 4, 6, 8), 8), ((16, 16, 8, 16), 18),
                                        ((16, 16, 8, 18), 18)])
@pytest.mark.parametrize("max_iter", [1, 3, 1000])
def test_cgne_device_iterations_equal_host_loop(ctx, dims, recon, max_iter):
    import ctypes
    U = synth.gauge_field(dims, 0.25, 131)
    o = ops.wilson_clover(ctx, U, dims, 0.12, 1.0, 0, recon)
    b = o.import_spinor(synth.gaussian_spinor(dims, 132), -1)
    runs = []
    for record in (False, True):
        prm = ops.cg_params(1e-10, max_iter, history=1000)
        if record:
            rec, err, zero = o.spinor(nrhs=1), o.spinor(nrhs=1), o.spinor()
            count = ctypes.c_int32(0)
            prm.record_r, prm.record_e, prm.record_xstar = rec.data_ptr(), err.data_ptr(), zero.data_ptr()
            prm.record_every, prm.record_max, prm.record_count = 1000, 1, ctypes.pointer(count)
        x = o.spinor(full=True)
        st, info = L.lqcd_cg_solve(ctx, o.op, None, prm, x, b)
        runs.append((st, info.iters, info.restarts, info.matvecs, ops.residual_history(prm, info),
                     np_of(o.export_spinor(x, -1))))
    dev, host = runs
    assert dev[:4] == host[:4]
    assert dev[0] == (L.LQCD_OK if max_iter == 1000 else L.LQCD_ERR_NOT_CONVERGED)
    assert len(dev[4]) == dev[1] == len(host[4])
    # FP64 sums in another order: the recurrences amplify 1e-16 by the steps taken
    assert np.allclose(dev[4], host[4], rtol=1e-9)
    assert rel(dev[5], host[5]) < 1e-11


def cgne_both_ways(ctx, o, prm_of, x0, b):
    """The device-driven solve, then the host's loop (which a solve that records its iterates takes)."""
    import ctypes
    runs = []
    for record in (False, True):
        prm = prm_of()
        if record:
            rec, err, zero = o.spinor(nrhs=1), o.spinor(nrhs=1), o.spinor()
            count = ctypes.c_int32(0)
            prm.record_r, prm.record_e, prm.record_xstar = rec.data_ptr(), err.data_ptr(), zero.data_ptr()
            prm.record_every, prm.record_max, prm.record_count = 100000, 1, ctypes.pointer(count)
        x = x0.clone()
        try:
            st, info = L.lqcd_cg_solve(ctx, o.op, None, prm, x, b)
        except L.LqcdError as e:
            st, info = e.status, None
        runs.append((st, info, np_of(o.export_spinor(x, -1))))
    return runs


# A residual that overflows to NaN in an iteration is a breakdown only if another
# iteration would follow; at max_iter the solve has not converged. Clover entries of
# 1e198 and a source of 1e-50 keep |p|^2 finite (1e300) and overflow the operator's
# second application.
@pytest.mark.parametrize("max_iter", [1, 2])
def test_cgne_residual_not_a_number(ctx, max_iter):
    dims = (4, 4, 4, 4)
    o = ops.wilson_clover(ctx, synth.gauge_field(dims, 0.25, 171), dims, 0.12, 1.0, 0, 18)
    o._keep["clover"].view(torch.float64).mul_(1e198)
    b = o.import_spinor(1e-50 * synth.gaussian_spinor(dims, 172), -1)
    dev, host = cgne_both_ways(ctx, o, lambda: ops.cg_params(1e-10, max_iter), o.spinor(full=True).zero_(), b)
    assert host[0] == (L.LQCD_ERR_NOT_CONVERGED if max_iter == 1 else L.LQCD_ERR_BREAKDOWN)
    assert dev[0] == host[0]
    if max_iter == 1:
        assert (dev[1].iters, dev[1].matvecs) == (host[1].iters, host[1].matvecs)


# From a first guess 1e6 times the solution, adding the correction leaves an error of
# a few 1e-16 * 1e6 in x, so the true residual fails the stop of 1e-10 that the
# iterated one has passed, and the device's iterations are entered again from it. The
# solution then meets the stop; two such solutions differ by at most the condition of
# the operator (below 1e3 here) times twice the stop.
@pytest.mark.parametrize("dims,recon", [((4, 4, 4, 4), 18), ((8, 4, 6, 8), 12)])
def test_cgne_device_iterations_after_a_failed_true_residual(ctx, dims, recon):
    o = ops.wilson_clover(ctx, synth.gauge_field(dims, 0.25, 173), dims, 0.12, 1.0, 0, recon)
    b = o.import_spinor(synth.gaussian_spinor(dims, 174), -1)
    x0 = o.import_spinor(1e6 * synth.gaussian_spinor(dims, 175), -1)
    dev, host = cgne_both_ways(ctx, o, lambda: ops.cg_params(1e-10, 1000), x0, b)
    for st, info, _ in (dev, host):
        assert st == L.LQCD_OK, L.lqcd_last_error(ctx)
        assert info.restarts >= 2
        assert info.true_residual <= 1e-10 * (1 + 1e-6)
    assert rel(dev[2], host[2]) < 1e3 * 2e-10
