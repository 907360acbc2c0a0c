"""GPU parity of the Wilson-clover kernels against the FP64 CPU oracle."""
import functools

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import TOL, check, ctx, np_of, on_parity, rel  # noqa: F401

pytestmark = pytest.mark.gpu

L = pytest.importorskip("paper_1109_2935_amd.lqcd")
from paper_1109_2935_amd import ops  # noqa: E402

# (dims, tile): plain lexicographic layouts (tile = dims) with a non-power-of-two
# extent, and tiled layouts that span several tiles with a ragged tile count.
LAYOUTS = [((4, 4, 6, 8), None), ((8, 8, 8, 8), (4, 4, 4, 4)), ((4, 8, 4, 12), (2, 4, 2, 4))]
PREC_RECON = [(0, 18), (0, 12), (0, 8), (1, 18), (1, 12), (1, 8), (2, 18), (2, 12), (3, 18), (3, 12)]


# Schwarz K with 8 MR steps, by storage precision. Each MR step stores r, the
# intermediate odd spinor, q and x in the storage format: independent
# round-to-nearest errors of relative RMS u / sqrt(3), u the unit roundoff
# (2^-11 for FP16, 2^-8 for BF16). An error in r_k reaches x through the
# remaining steps, which approximate Mhat_B^-1; Mhat_B = A - kappa^2 (...) with
# kappa^2 = 0.015 is close to the identity, so that factor is taken as 1. The
# 32 roundings added in quadrature give sqrt(32 / 3) u = 3.3 u; a factor 3 for
# the spread of a statistical bound gives 10 u: 5e-3 for FP16 and 4e-2 for
# BF16.
SCHWARZ_TOL = {0: 1e-12, 1: 1e-5, 2: 5e-3, 3: 4e-2}


class Fields:
    cache = {}

    @classmethod
    def get(cls, dims, seed=11):
        key = (dims, seed)
        if key not in cls.cache:
            U = synth.gauge_field(dims, 0.25, seed)
            psi = synth.gaussian_spinor(dims, seed + 1)
            cls.cache[key] = (U, psi, torch.from_numpy(U).cuda())
        return cls.cache[key]


def make_op(ctx, dims, prec, recon, tile=None, kappa=0.124, csw=1.0, bc_t=-1):
    U, psi, Ud = Fields.get(dims)
    return ops.wilson_clover(ctx, U, dims, kappa, csw, prec, recon, tile=tile, bc_t=bc_t, U_device=Ud)


@pytest.mark.parametrize("layout", LAYOUTS, ids=lambda l: "x".join(map(str, l[0])))
@pytest.mark.parametrize("prec,recon", PREC_RECON, ids=lambda v: str(v))
@pytest.mark.parametrize("dagger", [0, 1])
def test_dslash_parity(ctx, layout, prec, recon, dagger):
    dims, tile = layout
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon, tile)
    for p in (0, 1):
        mask_in = oracle.parity_mask(dims, 1 - p)
        src = on_parity(psi, mask_in)
        inp = o.import_spinor(src, 1 - p)
        out = o.spinor()
        L.lqcd_dslash(ctx, o.op, out, inp, p, dagger)
        got = np_of(o.export_spinor(out, p))
        ref = oracle.wilson_dslash(dims, U, src, bc_t=-1, out_parity=p, dagger=bool(dagger))
        check(got, ref, TOL[prec], "parity %d" % p)


# grids of every remainder over the 8 XCDs (544 .. 1056 sites of a parity in workgroups
# of 64 to 256): every site is computed once, by whichever XCD owns it
@pytest.mark.parametrize("lt", [34, 38, 42, 46, 50, 54, 58, 62, 66])
def test_dslash_any_number_of_workgroups(ctx, lt):
    dims = (4, 4, 2, lt)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, 2, 12)
    src = on_parity(psi, oracle.parity_mask(dims, 1))
    out = o.spinor()
    L.lqcd_dslash(ctx, o.op, out, o.import_spinor(src, 1), 0, 0)
    ref = oracle.wilson_dslash(dims, U, src, bc_t=-1, out_parity=0)
    check(np_of(o.export_spinor(out, 0)), ref, TOL[2], "dslash")


@pytest.mark.parametrize("prec,recon", [(0, 18), (1, 12), (2, 12)])
@pytest.mark.parametrize("block", [(4, 4, 4, 4), (2, 4, 4, 2), (8, 8, 2, 8)])
def test_dslash_dirichlet_cut(ctx, prec, recon, block):
    dims = (8, 8, 8, 8)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon, tile=(4, 4, 4, 4))
    for dagger in (0, 1):
        for p in (0, 1):
            src = on_parity(psi, oracle.parity_mask(dims, 1 - p))
            inp = o.import_spinor(src, 1 - p)
            out = o.spinor()
            L.lqcd_dslash(ctx, o.op, out, inp, p, dagger, block=block)
            got = np_of(o.export_spinor(out, p))
            ref = oracle.wilson_dslash(dims, U, src, out_parity=p, dagger=bool(dagger), block=block)
            check(got, ref, TOL[prec], "dagger %d parity %d" % (dagger, p))


@pytest.mark.parametrize("prec,recon", [(0, 18), (1, 12), (2, 12), (3, 12), (4, 12)])
def test_dslash_cut_never_reads_other_blocks(ctx, prec, recon):
    """With a cut at the tile faces, values in another block must not reach an
    output, not even as 0 * NaN: one block's input is NaN, and every output
    outside that block is finite and equals the oracle's cut operator applied
    to the input with that block zeroed."""
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon, tile=block)
    lab = oracle.block_labels(dims, block)
    for p in (0, 1):
        src = on_parity(psi, oracle.parity_mask(dims, 1 - p))
        bad = np.where((lab == 5)[..., None, None], np.nan + 0j, src)
        out = o.spinor()
        L.lqcd_dslash(ctx, o.op, out, o.import_spinor(bad, 1 - p), p, 0, block=block)
        got = np_of(o.export_spinor(out, p))
        ref = oracle.wilson_dslash(dims, U, np.where((lab == 5)[..., None, None], 0, src), out_parity=p, block=block)
        keep = (lab != 5)[..., None, None] & np.ones(got.shape, bool)
        assert np.isfinite(got[keep]).all()
        check(np.where(keep, got, 0), np.where(keep, ref, 0), TOL[prec] if prec < 4 else 6e-4, "parity %d" % p)


@pytest.mark.parametrize("bc_t", [1, -1])
def test_dslash_periodic_and_antiperiodic(ctx, bc_t):
    dims = (4, 4, 6, 8)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, 0, 18, bc_t=bc_t)
    src = on_parity(psi, oracle.parity_mask(dims, 1))
    out = o.spinor()
    L.lqcd_dslash(ctx, o.op, out, o.import_spinor(src, 1), 0, 0)
    ref = oracle.wilson_dslash(dims, U, src, bc_t=bc_t, out_parity=0)
    assert rel(np_of(o.export_spinor(out, 0)), ref) < 1e-12


@pytest.mark.parametrize("layout", LAYOUTS[:2], ids=lambda l: "x".join(map(str, l[0])))
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_clover_build_and_apply(ctx, layout, prec):
    dims, tile = layout
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, 18, tile)
    A = oracle.clover_build(dims, U, 0.124, 1.0)
    Ainv = oracle.clover_invert(dims, A)
    for p in (0, 1):
        src = on_parity(psi, oracle.parity_mask(dims, p))
        inp = o.import_spinor(src, p)
        for inverse, M in ((0, A), (1, Ainv)):
            out = o.spinor()
            L.lqcd_clover_apply(ctx, o.op, out, inp, p, inverse)
            ref = oracle.clover_apply(dims, M, src, parity=p)
            check(np_of(o.export_spinor(out, p)), ref, TOL[prec], "parity %d inverse %d" % (p, inverse))


@pytest.mark.parametrize("layout", LAYOUTS, ids=lambda l: "x".join(map(str, l[0])))
@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (1, 12), (1, 8), (2, 12), (3, 12)])
def test_schur_parity(ctx, layout, prec, recon):
    dims, tile = layout
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon, tile)
    ref_op = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    src = on_parity(psi, ref_op.even)
    inp = o.import_spinor(src, 0)
    for dagger in (0, 1):
        out = o.spinor()
        L.lqcd_schur_apply(ctx, o.op, out, inp, dagger)
        ref = ref_op.schur(src, dagger=bool(dagger))
        check(np_of(o.export_spinor(out, 0)), ref, TOL[prec], "dagger %d" % dagger)


@pytest.mark.parametrize("block", [(4, 4, 4, 4), (2, 2, 2, 2)])
def test_schur_cut_parity(ctx, block):
    dims = (8, 8, 8, 8)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, 0, 18, tile=(4, 4, 4, 4))
    ref_op = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    src = on_parity(psi, ref_op.even)
    out = o.spinor()
    L.lqcd_schur_apply(ctx, o.op, out, o.import_spinor(src, 0), 0, block=block)
    assert rel(np_of(o.export_spinor(out, 0)), ref_op.schur(src, block=block)) < 1e-12


@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), (4, 4, 4, 4)), ((4, 4, 8, 8), (2, 2, 2, 2)),
                                        ((16, 8, 8, 8), (8, 8, 8, 8))])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_schwarz_parity(ctx, dims, block, prec):
    """K r = block-Jacobi of 8 MR steps on each Dirichlet block (FP64: 1e-12)."""
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, 18 if prec in (0, 1) else 12, tile=block)
    ref_op = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    from oracle import solvers
    src = on_parity(psi, ref_op.even)
    ref = solvers.schwarz(ref_op, src, block, 8)
    inp = o.import_spinor(src, 0)
    out = o.spinor()
    L.lqcd_schwarz_precond(ctx, o.op, ops.schwarz_params(block, 8), out, inp)
    check(np_of(o.export_spinor(out, 0)), ref, SCHWARZ_TOL[prec])


@pytest.mark.parametrize("omega,cycles", [(1.3, 0), (0.8, 1)])
def test_schwarz_over_relaxed(ctx, omega, cycles):
    """MR with over-relaxation omega in the additive (8 steps) and the
    multiplicative (4 steps per visit) K, FP64, against the oracle (1e-12); it
    differs from plain MR; omega outside (0, 2) is refused."""
    from oracle import solvers
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, 0, 18, tile=block)
    ref_op = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    src = on_parity(psi, ref_op.even)
    steps = 8 if cycles == 0 else 4
    if cycles == 0:
        ref = solvers.schwarz(ref_op, src, block, steps, omega=omega)
        plain = solvers.schwarz(ref_op, src, block, steps)
    else:
        ref = solvers.sap(ref_op, src, block, steps, cycles, omega=omega)
        plain = solvers.sap(ref_op, src, block, steps, cycles)
    assert rel(ref, plain) > 1e-5
    out = o.spinor()
    L.lqcd_schwarz_precond(ctx, o.op, ops.schwarz_params(block, steps, cycles, omega=omega), out,
                           o.import_spinor(src, 0))
    check(np_of(o.export_spinor(out, 0)), ref, 1e-12)
    with pytest.raises(L.LqcdError) as ei:
        L.lqcd_schwarz_precond(ctx, o.op, ops.schwarz_params(block, steps, cycles, omega=2.5), out,
                               o.import_spinor(src, 0))
    assert ei.value.status == L.LQCD_ERR_INVALID_ARG


def test_dslash_deterministic(ctx):
    dims = (8, 8, 8, 8)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, 1, 12, tile=(4, 4, 4, 4))
    inp = o.import_spinor(on_parity(psi, oracle.parity_mask(dims, 1)), 1)
    a, b = o.spinor(), o.spinor()
    L.lqcd_dslash(ctx, o.op, a, inp, 0)
    L.lqcd_dslash(ctx, o.op, b, inp, 0)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (1, 12), (2, 12)])
def test_multi_rhs_equals_single(ctx, prec, recon):
    """nrhs right-hand sides interleaved per site: each equals its single-field
    result bit for bit (same arithmetic per site), for dslash, clover and Schur."""
    dims = (4, 4, 6, 8)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon)
    nr = 3
    srcs = np.stack([on_parity(synth.gaussian_spinor(dims, 100 + r), oracle.parity_mask(dims, 1)) for r in range(nr)])
    inp = o.import_spinor(srcs, 1, nrhs=nr)
    out = o.spinor(nrhs=nr)
    L.lqcd_dslash(ctx, o.op, out, inp, 0, nrhs=nr)
    multi = np_of(o.export_spinor(out, 0, nrhs=nr))
    esrc = np.stack([on_parity(synth.gaussian_spinor(dims, 200 + r), oracle.parity_mask(dims, 0)) for r in range(nr)])
    ein = o.import_spinor(esrc, 0, nrhs=nr)
    eout, cout = o.spinor(nrhs=nr), o.spinor(nrhs=nr)
    L.lqcd_schur_apply(ctx, o.op, eout, ein, nrhs=nr)
    L.lqcd_clover_apply(ctx, o.op, cout, ein, 0, 1, nrhs=nr)
    emulti = np_of(o.export_spinor(eout, 0, nrhs=nr))
    cmulti = np_of(o.export_spinor(cout, 0, nrhs=nr))
    for r in range(nr):
        single = o.spinor()
        L.lqcd_dslash(ctx, o.op, single, o.import_spinor(srcs[r], 1), 0)
        assert np.array_equal(np_of(o.export_spinor(single, 0)), multi[r])
        ref = oracle.wilson_dslash(dims, U, srcs[r], out_parity=0)
        check(multi[r], ref, TOL[prec], "rhs %d" % r)
        es = o.spinor()
        e1 = o.import_spinor(esrc[r], 0)
        L.lqcd_schur_apply(ctx, o.op, es, e1)
        assert np.array_equal(np_of(o.export_spinor(es, 0)), emulti[r])
        L.lqcd_clover_apply(ctx, o.op, es, e1, 0, 1)
        assert np.array_equal(np_of(o.export_spinor(es, 0)), cmulti[r])


@pytest.fixture
def matrix_cores(monkeypatch):
    """Link products of 16-bit multi-source hops on the matrix cores."""
    monkeypatch.setenv("LQCD_MRHS_MFMA", "1")


@pytest.mark.parametrize("prec,recon", [(2, 18), (2, 12), (3, 18), (3, 12)])
@pytest.mark.parametrize("dims,nr", [((6, 6, 2, 2), 4), ((4, 4, 6, 8), 8), ((4, 4, 4, 4), 12)])
def test_multi_rhs_matrix_cores(ctx, matrix_cores, prec, recon, dims, nr):
    """16-bit operators with a multiple of 4 sources take the link products on
    the matrix cores: every source of dslash (both parities, dagger) and of the
    Schur operator against the oracle, and against its single-source result,
    within the storage-precision bound. (6,6,2,2) with 4 sources leaves half a
    wave of idle lanes at the end."""
    U = synth.gauge_field(dims, 0.25, 31)
    o = ops.wilson_clover(ctx, U, dims, 0.124, 1.0, prec, recon)
    ref_op = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    for p in (0, 1):
        srcs = np.stack([on_parity(synth.gaussian_spinor(dims, 300 + r), oracle.parity_mask(dims, 1 - p))
                         for r in range(nr)])
        inp = o.import_spinor(srcs, 1 - p, nrhs=nr)
        for dagger in (0, 1):
            out = o.spinor(nrhs=nr)
            L.lqcd_dslash(ctx, o.op, out, inp, p, dagger, nrhs=nr)
            multi = np_of(o.export_spinor(out, p, nrhs=nr))
            for r in (0, nr // 2, nr - 1):
                ref = oracle.wilson_dslash(dims, U, srcs[r], out_parity=p, dagger=bool(dagger))
                check(multi[r], ref, TOL[prec], "parity %d dagger %d rhs %d" % (p, dagger, r))
                single = o.spinor()
                L.lqcd_dslash(ctx, o.op, single, o.import_spinor(srcs[r], 1 - p), p, dagger)
                check(multi[r], np_of(o.export_spinor(single, p)), TOL[prec], "vs single rhs %d" % r)
    esrc = np.stack([on_parity(synth.gaussian_spinor(dims, 400 + r), ref_op.even) for r in range(nr)])
    eout = o.spinor(nrhs=nr)
    L.lqcd_schur_apply(ctx, o.op, eout, o.import_spinor(esrc, 0, nrhs=nr), nrhs=nr)
    emulti = np_of(o.export_spinor(eout, 0, nrhs=nr))
    for r in (0, nr - 1):
        check(emulti[r], ref_op.schur(esrc[r]), TOL[prec], "schur rhs %d" % r)


@pytest.mark.parametrize("prec", [2, 3])
def test_multi_rhs_matrix_cores_dirichlet_cut(ctx, matrix_cores, prec):
    dims, block, nr = (8, 8, 8, 8), (4, 4, 4, 4), 4
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, 12, tile=(4, 4, 4, 4))
    srcs = np.stack([on_parity(synth.gaussian_spinor(dims, 500 + r), oracle.parity_mask(dims, 1)) for r in range(nr)])
    out = o.spinor(nrhs=nr)
    L.lqcd_dslash(ctx, o.op, out, o.import_spinor(srcs, 1, nrhs=nr), 0, 1, block=block, nrhs=nr)
    multi = np_of(o.export_spinor(out, 0, nrhs=nr))
    for r in range(nr):
        ref = oracle.wilson_dslash(dims, U, srcs[r], out_parity=0, dagger=True, block=block)
        check(multi[r], ref, TOL[prec], "rhs %d" % r)


@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (1, 12), (2, 12), (3, 12)])
def test_batched_persistent_uneven_lattices(ctx, prec, recon):
    """One persistent launch over lattices of different size and rhs count
    equals the per-operator dslash (bitwise) and the oracle (per-precision bound)."""
    run_batch(ctx, prec, recon)


@pytest.mark.parametrize("prec", [2, 3])
def test_batched_persistent_matrix_cores(ctx, matrix_cores, prec):
    """The persistent launch takes the same matrix-core path per job as the
    per-operator dslash (4- and 12-source jobs), the vector path for 1 source."""
    run_batch(ctx, prec, 12)


def run_batch(ctx, prec, recon):
    shapes = [((4, 4, 4, 8), 4), ((6, 6, 6, 12), 4), ((8, 8, 8, 8), 12), ((4, 6, 4, 6), 1)]
    jobs, ref_single, refs = [], [], []
    keep = []
    for k, (dims, nr) in enumerate(shapes):
        U = synth.gauge_field(dims, 0.25, 4001 + 10 * k)
        o = ops.wilson_clover(ctx, U, dims, 0.122, 1.0, prec, recon)
        srcs = np.stack([on_parity(synth.gaussian_spinor(dims, 4002 + 10 * k + r), oracle.parity_mask(dims, 1))
                         for r in range(nr)])
        inp = o.import_spinor(srcs, 1, nrhs=nr)
        out = o.spinor(nrhs=nr)
        single = o.spinor(nrhs=nr)
        L.lqcd_dslash(ctx, o.op, single, inp, 0, nrhs=nr)
        jobs.append((o.op, out, inp, 0, nr))
        keep.append((o, out, inp, single, srcs, U, dims, nr))
    L.lqcd_dslash_batch(ctx, jobs)
    L.lqcd_dslash_batch(ctx, jobs)  # second call: tuned parameters
    torch.cuda.synchronize()
    check_batch(keep, prec)


def check_batch(keep, prec):
    for o, out, inp, single, srcs, U, dims, nr in keep:
        assert torch.equal(out, single)
        got = np_of(o.export_spinor(out, 0, nrhs=nr))
        if nr == 1:
            got = got[None]
        for r in range(nr):
            ref = oracle.wilson_dslash(dims, U, srcs[r], out_parity=0)
            check(got[r], ref, TOL[prec], "rhs %d" % r)


def test_invalid_arguments_write_nothing(ctx):
    dims = (4, 4, 6, 8)
    o = make_op(ctx, dims, 1, 12)
    out = o.spinor()
    out.fill_(7)
    inp = o.spinor()
    for kwargs, code in [(dict(out_parity=2), L.LQCD_ERR_INVALID_ARG),
                         (dict(out_parity=0, nrhs=0), L.LQCD_ERR_INVALID_ARG),
                         (dict(out_parity=0, block=(3, 4, 6, 8)), L.LQCD_ERR_INVALID_ARG)]:
        with pytest.raises(L.LqcdError) as ei:
            L.lqcd_dslash(ctx, o.op, out, inp, **kwargs)
        assert ei.value.status == code
    with pytest.raises(L.LqcdError) as ei:
        L.lqcd_dslash(ctx, o.op, int(out.data_ptr()) + 4, inp, 0)
    assert ei.value.status == L.LQCD_ERR_INVALID_ARG
    torch.cuda.synchronize()
    assert bool((out == 7).all())


# the clover build takes 64 sites per workgroup, in columns along t of the
# largest even extents up to 8 that divide Ly and Lz: lattices that end inside a
# workgroup, columns of 2, 6 and 8, extents of 2 (both neighbours are one site)
@pytest.mark.parametrize("dims,tile", [((2, 2, 2, 2), None), ((6, 2, 10, 2), (2, 2, 10, 2)), ((2, 14, 6, 4), None),
                                       ((4, 8, 16, 2), (4, 4, 8, 2))])
@pytest.mark.parametrize("prec,recon", [(0, 18), (2, 12), (3, 18)])
def test_clover_build_edges(ctx, dims, tile, prec, recon):
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon, tile)
    A = oracle.clover_build(dims, U, 0.124, 1.0)
    for inverse, M in ((0, A), (1, oracle.clover_invert(dims, A))):
        for p in (0, 1):
            src = on_parity(psi, oracle.parity_mask(dims, p))
            out = o.spinor()
            L.lqcd_clover_apply(ctx, o.op, out, o.import_spinor(src, p), p, inverse)
            check(np_of(o.export_spinor(out, p)), oracle.clover_apply(dims, M, src, parity=p), TOL[prec])


def test_clover_build_refuses_indefinite_blocks(ctx):
    """A clover term with an eigenvalue below zero has no inverse here."""
    dims = (4, 4, 2, 2)
    U = synth.gauge_field(dims, 1.0, 17)
    with pytest.raises(L.LqcdError) as ei:
        ops.wilson_clover(ctx, U, dims, 0.5, 8.0, 0, 18)
    assert ei.value.status == L.LQCD_ERR_BREAKDOWN


# launches of at most 16384 points (site, source) run a site's hops in eight
# waves, larger ones one site per thread: 6 sources of 2560 sites are the first,
# 8 the second, and both equal the single-source launches bit for bit
@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (0, 8), (1, 18), (1, 12), (1, 8)])
@pytest.mark.parametrize("block", [None, (4, 4, 4, 10)])
@pytest.mark.parametrize("dagger", [0, 1])
def test_split_launch_equals_plain(ctx, prec, recon, block, dagger):
    dims = (8, 8, 8, 10)
    o = make_op(ctx, dims, prec, recon, (4, 4, 2, 10))
    fields = np.stack([synth.gaussian_spinor(dims, 400 + j) for j in range(8)])
    for n in (6, 8):
        for p in (0, 1):
            src = np.stack([on_parity(f, oracle.parity_mask(dims, p)) for f in fields[:n]])
            inp, hop, schur = o.import_spinor(src, p, nrhs=n), o.spinor(nrhs=n), o.spinor(nrhs=n)
            L.lqcd_dslash(ctx, o.op, hop, inp, 1 - p, dagger, block=block, nrhs=n)
            got = [np_of(o.export_spinor(hop, 1 - p, nrhs=n))]
            if p == 0:
                L.lqcd_schur_apply(ctx, o.op, schur, inp, dagger, block=block, nrhs=n)
                got.append(np_of(o.export_spinor(schur, 0, nrhs=n)))
            for j in range(n):
                one, out = o.import_spinor(src[j], p), o.spinor()
                L.lqcd_dslash(ctx, o.op, out, one, 1 - p, dagger, block=block)
                assert np.array_equal(got[0][j], np_of(o.export_spinor(out, 1 - p)))
                if p == 0:
                    L.lqcd_schur_apply(ctx, o.op, out, one, dagger, block=block)
                    assert np.array_equal(got[1][j], np_of(o.export_spinor(out, 0)))


# The kernels of one thread per site, which take the launches above 16384 points: one
# source on 18360 sites of a parity, which leaves the last workgroup of 64, 128 or 256
# threads partly empty, daggered or not, cut or not
@pytest.mark.parametrize("prec,recon", [(0, 18), (0, 12), (0, 8), (1, 18), (1, 12), (1, 8)])
@pytest.mark.parametrize("block", [None, (6, 6, 2, 34)])
@pytest.mark.parametrize("dagger", [0, 1])
def test_one_thread_kernels_with_a_partial_workgroup(ctx, prec, recon, block, dagger):
    dims = (18, 6, 10, 34)
    U, psi, _ = Fields.get(dims)
    o = make_op(ctx, dims, prec, recon)
    ref = one_thread_oracle(dims, block, dagger)
    for p in (0, 1):
        src = on_parity(psi, oracle.parity_mask(dims, p))
        inp, out = o.import_spinor(src, p), o.spinor()
        L.lqcd_dslash(ctx, o.op, out, inp, 1 - p, dagger, block=block)
        check(np_of(o.export_spinor(out, 1 - p)), ref[p], TOL[prec], "dslash from parity %d" % p)
        if p == 0:
            L.lqcd_schur_apply(ctx, o.op, out, inp, dagger, block=block)
            check(np_of(o.export_spinor(out, 0)), ref[2], TOL[prec], "schur")


@functools.lru_cache(maxsize=None)
def one_thread_oracle(dims, block, dagger):
    U, psi, _ = Fields.get(dims)
    ref = oracle.WilsonClover(dims, U, 0.124, 1.0, bc_t=-1)
    src = [on_parity(psi, oracle.parity_mask(dims, p)) for p in (0, 1)]
    return [ref.D(src[p], out_parity=1 - p, dagger=bool(dagger), block=block) for p in (0, 1)] + [
        ref.schur(src[0], dagger=bool(dagger), block=block)]
