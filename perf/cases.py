"""The work that programs have this library do, as cases to be timed and compared.

A case is a dict of plain values. `prepare` makes what a program holds before
the call (operators with packed links, source fields, output buffers), `run`
is one pass through the public entry points, `work` the bytes and operations
that the pass cannot do without, and `exact` the same result from plain torch
in 64-bit arithmetic. Lattices are written "LxxLyxLzxLt".
"""
import math

import numpy as np
import torch

from paper_1109_2935_amd import lqcd as L
from paper_1109_2935_amd import ops, ptc

DEVICE = "cuda"
BC_T = -1
EPS = 0.25       # spread of the synthetic links about the identity
CSW = 1.0
MASS = 0.01      # staggered
PRECISION = {"f64": L.LQCD_F64, "f32": L.LQCD_F32, "f16": L.LQCD_F16, "bf16": L.LQCD_BF16}
STORED = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
LINK_SEED = 7919  # the links' random stream is kept apart from the sources'

_context = []


def context():
    """One library context for the whole program."""
    if not _context:
        _context.append(L.lqcd_context_create())
    return _context[0]


def listed():
    return [
        # one application of the FP64 hopping term on the smallest lattice: the call's own cost
        {"name": "dslash_f64_8x8x8x8", "kind": "wilson", "op": "dslash", "dims": "8x8x8x8", "prec": "f64", "recon": 18},
        # the smallest whole solve: even-odd CGNE in FP64, as the training data and reference solutions are made
        {"name": "cgne_f64_8x8x8x8", "kind": "cgne", "dims": "8x8x8x8", "kappa": 0.12},
        # the hopping term of the large lattice in the Krylov precision
        {"name": "dslash_f32_32x32x32x64", "kind": "wilson", "op": "dslash", "dims": "32x32x32x64", "prec": "f32",
         "recon": 12, "tile": "32x32x4x4"},
        # the sloppy operator of mixed-precision BiCGstab and CGNE, two applications a step
        {"name": "schur_f16_32x32x32x64", "kind": "wilson", "op": "schur", "dims": "32x32x32x64", "prec": "f16",
         "recon": 12, "tile": "32x32x4x4"},
        # a lattice with no power of two in it, default site order, adjoint operator in FP64 (reliable updates)
        {"name": "schur_f64_20x12x28x36", "kind": "wilson", "op": "schur", "dims": "20x12x28x36", "prec": "f64",
         "recon": 18, "dagger": 1},
        # the Schwarz preconditioner of GCR-DD, one application a step
        {"name": "schwarz_f16_32x32x32x64", "kind": "schwarz", "dims": "32x32x32x64", "prec": "f16", "recon": 18,
         "block": "8x8x8x8", "steps": 8},
        # a propagator's 12 sources in one launch
        {"name": "dslash_f32_12src_24x24x24x48", "kind": "wilson", "op": "dslash", "dims": "24x24x24x48",
         "prec": "f32", "recon": 12, "nrhs": 12, "kappa": 0.122, "tile": "24x8x8x8"},
        # the staggered normal operator of the sloppy CG, one application a step
        {"name": "stag_f32_48x48x48x96", "kind": "staggered", "dims": "48x48x48x96", "prec": "f32", "recon": 12},
        # the learned preconditioner, one application a step of flexible GCR
        {"name": "ptc_apply_32x32x32x64", "kind": "ptc_apply", "dims": "32x32x32x64", "channels": "1-16-16-16-1",
         "recon": 12, "tile": "8x8x8x8"},
        # one step of its training on a pair (gradient of the residual loss, Adam update)
        {"name": "ptc_train_16x16x16x16", "kind": "ptc_train", "dims": "16x16x16x16", "channels": "1-16-16-16-1",
         "recon": 12, "loss": "residual"},
        # a new gauge configuration: packed links, clover term and its inverse
        {"name": "setup_f32_32x32x32x64", "kind": "setup", "dims": "32x32x32x64", "prec": "f32", "recon": 12,
         "tile": "32x32x4x4"},
        # a whole solve of the large lattice: mixed-precision GCR with the Schwarz preconditioner
        {"name": "gcr_dd_32x32x32x64", "kind": "gcr", "dims": "32x32x32x64", "block": "8x8x8x8", "steps": 8,
         "recon": 18},
    ]


def _pick_dims(rng, least, most, unit=(2, 2, 2, 2), longest=(32, 32, 32, 64)):
    """Extents that are multiples of `unit`, of a volume spread over the logarithm of [least, most]."""
    want = math.exp(rng.uniform(math.log(least), math.log(most)))
    while True:
        d = [u * rng.randint(max(1, -(-4 // u)), m // u) for u, m in zip(unit, longest)]
        if 0.6 * want <= math.prod(d) <= min(1.5 * want, most):
            return "x".join(map(str, d))


def draw(rng):
    big, mid = 32 ** 3 * 64, 24 ** 3 * 48
    kind = rng.choice(["wilson", "wilson", "wilson", "sources", "sources", "schwarz", "staggered", "ptc_apply",
                       "ptc_train", "setup", "cgne", "gcr"])
    prec = rng.choice(["f64", "f32", "f16", "bf16"])
    recon = rng.choice({"f64": [18, 12], "f32": [18, 12, 8]}.get(prec, [18, 12]))
    if kind in ("wilson", "sources"):
        c = {"kind": "wilson", "op": rng.choice(["dslash", "schur"]), "prec": prec, "recon": recon,
             "dagger": rng.randint(0, 1)}
        if kind == "sources":
            c["nrhs"] = rng.choice([2, 3, 4, 6, 8, 12])
            c["dims"] = _pick_dims(rng, 4096, mid)
        else:
            c["dims"] = _pick_dims(rng, 4096, big)
            d = _ints(c["dims"])
            if d[2] % 4 == 0 and d[3] % 4 == 0 and rng.random() < 0.5:
                c["tile"] = "%dx%dx4x4" % (d[0], d[1])
        return c
    if kind == "schwarz":
        block = rng.choice(["4x4x4x4", "8x4x4x4", "8x8x4x4", "8x8x8x8"])
        return {"kind": kind, "dims": _pick_dims(rng, 16384, big, _ints(block)), "block": block,
                "prec": rng.choice(["f16", "bf16"]), "recon": rng.choice([18, 12]), "steps": rng.randint(4, 10)}
    if kind == "staggered":
        prec = rng.choice(["f64", "f32", "f16"])
        return {"kind": kind, "dims": _pick_dims(rng, 4096, 48 ** 3 * 96, longest=(48, 48, 48, 96)), "prec": prec,
                "recon": rng.choice([18, 12])}
    if kind.startswith("ptc"):
        c = {"kind": kind, "channels": rng.choice(["1-16-16-16-1", "1-16-16-1", "1-8-8-1", "1-16-8-1"]),
             "recon": rng.choice([18, 12])}
        if kind == "ptc_train":
            return dict(c, dims=_pick_dims(rng, 4096, 16 ** 4), loss=rng.choice(["residual", "error"]))
        return dict(c, dims=_pick_dims(rng, 4096, big))
    if kind == "setup":
        return {"kind": kind, "dims": _pick_dims(rng, 4096, big), "prec": prec, "recon": 18 if recon == 8 else recon}
    if kind == "cgne":
        return {"kind": kind, "dims": _pick_dims(rng, 4096, 16 ** 4), "kappa": 0.12}
    block = rng.choice(["4x4x4x4", "8x8x8x8"])
    return {"kind": kind, "dims": _pick_dims(rng, 65536, mid, _ints(block)), "block": block, "steps": rng.randint(4, 8),
            "recon": rng.choice([18, 12])}


def _ints(text, by="x"):
    return tuple(int(v) for v in text.split(by))


def _dims(case):
    return _ints(case["dims"])


def _tile(case):
    return _ints(case.get("tile") or case.get("block") or case["dims"])


def _kappa(case):
    return case.get("kappa", 0.124)


# ---------------------------------------------------------------------------
# inputs

def _random(seed, *shape):
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))
    return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float64)


def _gaussian(seed, *shape):
    """Complex Gaussian field, real and imaginary parts N(0, 1)."""
    return torch.view_as_complex(_random(seed, *shape, 2))


def _cross_conj(a, b):
    return torch.cross(a, b, dim=-1).conj()


def _links(dims, seed, eps=EPS):
    """SU(3) links [t,z,y,x,mu,3,3] about the identity: the unitary part of 1 + i eps H - (eps H)^2 / 2, H a
    Gaussian traceless Hermitian matrix."""
    lx, ly, lz, lt = dims
    h = _random(LINK_SEED * (seed + 1), lt, lz, ly, lx, 4, 8) / 2
    H = torch.empty((lt, lz, ly, lx, 4, 3, 3), dtype=torch.complex128, device=DEVICE)
    s = h[..., 7] / math.sqrt(3)
    H[..., 0, 0], H[..., 1, 1], H[..., 2, 2] = h[..., 2] + s, s - h[..., 2], -2 * s
    for (i, j), (a, b) in {(0, 1): (0, 1), (0, 2): (3, 4), (1, 2): (5, 6)}.items():
        H[..., i, j] = torch.complex(h[..., a], -h[..., b])
        H[..., j, i] = torch.complex(h[..., a], h[..., b])
    del h
    rows = []
    for i in range(2):  # two rows of the series
        m = 1j * eps * H[..., i, :]
        for k in range(3):
            m -= (eps * eps / 2) * H[..., i, k, None] * H[..., k, :]
        m[..., i] += 1
        rows.append(m)
    u, v = rows
    u = u / torch.linalg.vector_norm(u, dim=-1, keepdim=True)
    v = v - (u.conj() * v).sum(-1, keepdim=True) * u
    v = v / torch.linalg.vector_norm(v, dim=-1, keepdim=True)
    return torch.stack([u, v, _cross_conj(u, v)], dim=-2, out=H)


def _fat_links(U, seed):
    """General complex links near the thin ones."""
    return U + 0.05 * _gaussian(LINK_SEED * (seed + 1) + 1, *U.shape)


def _sources(case, seed):
    lx, ly, lz, lt = _dims(case)
    inner = (3,) if case["kind"] == "staggered" else (4, 3)
    n = case.get("nrhs", 1)
    return _gaussian(seed, *((n,) if n > 1 else ()), lt, lz, ly, lx, *inner)


def _weights(channels, seed):
    """Network weights: the identity through channel 0 and complex noise on every entry."""
    out = []
    for l, (ci, co) in enumerate(zip(channels[:-1], channels[1:])):
        W = 0.3 / math.sqrt(36 * ci) * _gaussian(31 * (seed + 1) + l, co, ci, 9, 4, 4)
        W[0, 0, 0] += torch.eye(4, device=DEVICE)
        out.append(W)
    return out


# ---------------------------------------------------------------------------
# what a program holds, and one pass

def prepare(case, seed):
    kind, dims, ctx = case["kind"], _dims(case), context()
    U = _links(dims, seed, 0.2 if kind == "staggered" else EPS)
    s = {"case": case, "ctx": ctx}
    if kind == "setup":
        s["links"] = U
        return s
    if kind in ("cgne", "gcr"):
        def make(prec, recon, tile):
            return ops.wilson_clover(ctx, None, dims, _kappa(case), CSW, prec, recon, tile=tile, U_device=U)
        if kind == "cgne":
            s["hi"] = make(L.LQCD_F64, 18, None)
            s["params"] = ops.cg_params(1e-12, max_iter=20000)
        else:
            block = _ints(case["block"])
            tile = (dims[0], dims[1], 4, 4)
            s["hi"], s["krylov"] = make(L.LQCD_F64, 18, tile), make(L.LQCD_F32, 12, tile)
            s["precond"] = make(L.LQCD_F16, case["recon"], block)
            s["params"] = ops.gcr_params(1e-12, 16, 1e-3, max_iter=4000, precond=L.LQCD_PRECOND_SCHWARZ, block=block,
                                         mr_steps=case["steps"])
        s["b"] = s["hi"].import_spinor(_sources(case, seed), -1)
        s["x"] = s["hi"].spinor(full=True)
        return s
    if kind.startswith("ptc"):
        op = ops.wilson_clover(ctx, None, dims, _kappa(case), CSW, L.LQCD_F32, case["recon"], tile=_tile(case),
                               U_device=U)
        channels = _ints(case["channels"], "-")
        net = ptc.Network(ctx, channels)
        net.set_weights([W.cpu().numpy() for W in _weights(channels, seed)])
        s.update(op=op, net=net, r=op.import_spinor(_sources(case, seed), 0), y=op.spinor())
        if kind == "ptc_train":
            s["e"] = op.import_spinor(_sources(case, seed + (1 << 40)), 0)
            # the optimiser's state in the middle of a training
            net.step = 1000
            net.m.copy_(1e-3 * _random(seed + (1 << 41), net.m.numel()))
            net.v.fill_(1e-5)
        return s
    prec = PRECISION[case["prec"]]
    if kind == "staggered":
        op = ops.staggered(ctx, None, None, dims, MASS, prec, case["recon"], fat_device=_fat_links(U, seed),
                           U_device=U)
    else:
        op = ops.wilson_clover(ctx, None, dims, _kappa(case), CSW, prec, case["recon"], tile=_tile(case), U_device=U)
    n = case.get("nrhs", 1)
    parity = 1 if case.get("op") == "dslash" else 0
    s.update(op=op, inp=op.import_spinor(_sources(case, seed), parity, nrhs=n), out=op.spinor(nrhs=n))
    if kind == "schwarz":
        s["params"] = ops.schwarz_params(_ints(case["block"]), case["steps"])
    return s


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "setup":
        op = ops.wilson_clover(ctx, None, _dims(case), _kappa(case), CSW, PRECISION[case["prec"]], case["recon"],
                               tile=_tile(case), U_device=state["links"])
        return [op._keep[k].view(STORED[case["prec"]]) for k in ("gauge", "clover", "clover_inv")]
    if kind in ("cgne", "gcr"):
        x = state["x"].zero_()
        if kind == "cgne":
            status, info = L.lqcd_cg_solve(ctx, state["hi"].op, None, state["params"], x, state["b"])
        else:
            status, info = L.lqcd_gcr_solve(ctx, state["hi"].op, state["krylov"].op, state["precond"].op,
                                            state["params"], x, state["b"])
        if status != L.LQCD_OK:
            raise RuntimeError("not converged: %s" % info.as_dict())
        return state["hi"].export_spinor(x, -1)
    if kind == "ptc_apply":
        state["net"].apply(state["op"], state["y"], state["r"])
        return state["y"].view(torch.float32)
    if kind == "ptc_train":
        net = state["net"]
        if case["loss"] == "residual":
            loss = net.residual_gradient(state["op"], state["r"])
        else:
            loss = net.gradient(state["op"], state["r"], state["e"])
        net.adam(2e-4)
        return [loss, net.grad, net.weights]
    op, out, inp, n = state["op"], state["out"], state["inp"], case.get("nrhs", 1)
    if kind == "schwarz":
        L.lqcd_schwarz_precond(ctx, op.op, state["params"], out, inp)
    elif kind == "staggered":
        L.lqcd_schur_apply(ctx, op.op, out, inp)
    elif case["op"] == "dslash":
        L.lqcd_dslash(ctx, op.op, out, inp, 0, dagger=case.get("dagger", 0), nrhs=n)
    else:
        L.lqcd_schur_apply(ctx, op.op, out, inp, dagger=case.get("dagger", 0), nrhs=n)
    return out.view(STORED[case["prec"]])


def work(case):
    """Inputs read once, outputs written once. Flops of a hop: 1320 a site (Wilson), 1146 (staggered), clover 504."""
    kind, vh = case["kind"], math.prod(_dims(case)) // 2
    n, size, recon = case.get("nrhs", 1), SIZE.get(case.get("prec"), 4), case.get("recon", 18)
    schur = 2 * 1320 + 2 * 504 + 48
    if kind == "wilson":
        both = case["op"] == "schur"
        return {"bytes": vh * size * (48 * n + 8 * recon + (144 if both else 0)), "flops": vh * n * (schur if both else 1320)}
    if kind == "schwarz":
        return {"bytes": vh * size * (48 + 8 * recon + 144), "flops": vh * case["steps"] * (schur + 24 * 12)}
    if kind == "staggered":
        return {"bytes": vh * size * (12 + 8 * (18 + recon)), "flops": vh * 2 * 1146}
    if kind == "setup":
        return {"bytes": 2 * vh * (4 * 144 + size * (4 * recon + 144)), "flops": 2 * vh * 17000}
    if kind.startswith("ptc"):
        ch = _ints(case["channels"], "-")
        flops = 0
        for l, (ci, co) in enumerate(zip(ch[:-1], ch[1:])):
            # the input vanishes on odd sites and the output is read on even ones
            parities = 1 if l == 0 or l == len(ch) - 2 else 2
            flops += parities * vh * ci * (3456 * co + 8 * 4 * 66)
        step = 3 if kind == "ptc_train" else 1  # data and weight gradients beside the forward pass
        return {"bytes": vh * 4 * (48 + 8 * recon + (144 if step > 1 else 0)), "flops": step * flops}
    # solves: an application of the operator a step, for about the steps that these fields take
    if kind == "cgne":
        return {"bytes": 60 * vh * 8 * (2 * (48 + 144 + 144) + 8 * 24), "flops": 60 * vh * 2 * schur}
    per = 4 * (48 + 96 + 144 + 10 * 24) + 2 * (48 + 8 * recon + 144)
    return {"bytes": 57 * vh * per, "flops": 57 * vh * (schur + case["steps"] * (schur + 288) + 20 * 96)}


# ---------------------------------------------------------------------------
# the same results in 64-bit arithmetic

GAMMA_COLUMN = ((3, 2, 1, 0), (3, 2, 1, 0), (2, 3, 0, 1), (2, 3, 0, 1))
GAMMA_ENTRY = ((-1j, -1j, 1j, 1j), (-1, 1, 1, -1), (-1j, 1j, 1j, -1j), (1, 1, 1, 1))


def _gamma(mu, psi):
    """gamma_mu psi, psi [..., spin, colour]."""
    f = torch.tensor(GAMMA_ENTRY[mu], dtype=torch.complex128, device=psi.device)
    return psi[..., GAMMA_COLUMN[mu], :] * f[:, None]


def _mv(U, v):
    """U v for U [..., 3, 3] and v [..., n, 3]."""
    return (U[..., None, :, :] * v[..., None, :]).sum(-1)


def _mm(A, B):
    return (A[..., :, :, None] * B[..., None, :, :]).sum(-2)


def _dag(U):
    return U.transpose(-1, -2).conj()


def _phase(f, axis, step, keep=None):
    """f[x] shifted to f[x + step] along mu, with the boundary sign in t."""
    n = f.shape[3 - axis]
    g = torch.roll(f, -step, dims=3 - axis)
    if axis == 3 and BC_T < 0:
        k = abs(step)
        for j in range(k):
            at = (n - 1 - j) % n if step > 0 else j % n
            g = torch.cat([g[:at], -g[at:at + 1], g[at + 1:]])
    return g


def _cut(f, axis, step, block):
    """Drop the hops that leave a block."""
    if block is None or block[axis] == f.shape[3 - axis]:
        return f
    c = torch.arange(f.shape[3 - axis], device=f.device) % block[axis]
    keep = (c != (block[axis] - 1 if step > 0 else 0)).to(torch.float64)
    shape = [1] * f.dim()
    shape[3 - axis] = -1
    return f * keep.view(shape)


def _hopping(U, psi, dagger=0, block=None):
    out = 0
    for mu in range(4):
        sign = -1 if dagger else 1
        Um = U[..., mu, :, :]
        f = _cut(_phase(psi, mu, +1), mu, +1, block)
        f = _mv(Um, f - sign * _gamma(mu, f))
        g = _mv(_dag(Um), psi + sign * _gamma(mu, psi))
        out = out + f + _cut(_phase(g, mu, -1), mu, -1, block)
    return out


def _clover(U, kappa):
    """The clover term as two Hermitian 6x6 blocks a site: [t,z,y,x,2,6,6]."""
    g = [torch.zeros(4, 4, dtype=torch.complex128, device=U.device) for _ in range(4)]
    for mu in range(4):
        for s in range(4):
            g[mu][s, GAMMA_COLUMN[mu][s]] = GAMMA_ENTRY[mu][s]
    A = torch.zeros(U.shape[:4] + (2, 6, 6), dtype=torch.complex128, device=U.device)
    A += torch.eye(6, dtype=torch.complex128, device=U.device)

    def at(f, mu, step):
        return torch.roll(f, -step, dims=3 - mu)

    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            am, bn, bm, an = at(a, mu, -1), at(b, nu, -1), at(b, mu, -1), at(a, nu, -1)
            Q = _mm(_mm(a, at(b, mu, 1)), _mm(_dag(at(a, nu, 1)), _dag(b)))
            Q += _mm(_mm(b, _dag(at(am, nu, 1))), _mm(_dag(bm), am))
            Q += _mm(_mm(_dag(am), _dag(at(bm, nu, -1))), _mm(at(am, nu, -1), bn))
            Q += _mm(_mm(_dag(bn), an), _mm(at(bn, mu, 1), _dag(a)))
            F = (Q - _dag(Q)) / 8
            del Q, am, bn, bm, an
            S = -kappa * CSW * (g[mu] @ g[nu])  # i sigma = -gamma_mu gamma_nu
            for c in range(2):
                s = S[2 * c:2 * c + 2, 2 * c:2 * c + 2]
                for i in range(2):
                    for j in range(2):
                        if s[i, j] != 0:
                            A[..., c, 3 * i:3 * i + 3, 3 * j:3 * j + 3] += s[i, j] * F
    return A


def _inverse(A):
    """Inverses of positive definite 6x6 blocks (Gauss-Jordan)."""
    A = A.clone()
    for k in range(6):
        p = 1 / A[..., k, k]
        row = A[..., k, :] * p[..., None]
        col = A[..., :, k].clone()
        A -= col[..., :, None] * row[..., None, :]
        A[..., k, :] = row
        A[..., :, k] = -col * p[..., None]
        A[..., k, k] = p
    return A


def _clover_mul(A, psi):
    return (A * psi.reshape(psi.shape[:4] + (2, 1, 6))).sum(-1).reshape(psi.shape)


def _grid_parity(dims):
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device=DEVICE) for n in reversed(dims)), indexing="ij")
    return (x + y + z + t) % 2


def _on(f, dims, parity):
    return f * (_grid_parity(dims) == parity).view(f.shape[:4] + (1,) * (f.dim() - 4))


class _Schur:
    """The even-odd operator on natural fields that vanish on odd sites."""

    def __init__(self, dims, U, kappa):
        self.dims, self.U, self.kappa = dims, U, kappa
        self.A = _clover(U, kappa)
        self.Ainv = _inverse(self.A)

    def __call__(self, x, dagger=0, block=None):
        t = _clover_mul(self.Ainv, _hopping(self.U, x, dagger, block))
        return _clover_mul(self.A, x) - self.kappa ** 2 * _hopping(self.U, t, dagger, block)

    def solve(self, b, tol=1e-14, most=400):
        """M x = b: BiCGstab on the even sites, then the odd ones."""
        be, bo = _on(b, self.dims, 0), _on(b, self.dims, 1)
        rhs = be + self.kappa * _hopping(self.U, _clover_mul(self.Ainv, bo))

        def dot(u, v):
            return torch.view_as_real(u.conj() * v).sum(dim=tuple(range(u.dim())))

        def cdot(u, v):
            return complex(*dot(u, v).tolist())

        x, r = torch.zeros_like(rhs), rhs.clone()
        shadow, p, rho, goal = r.clone(), r.clone(), cdot(r, r), tol ** 2 * cdot(rhs, rhs).real
        for _ in range(most):
            v = self(p)
            alpha = rho / cdot(shadow, v)
            r -= alpha * v
            t = self(r)
            omega = cdot(t, r) / cdot(t, t).real
            x += alpha * p + omega * r
            r -= omega * t
            if cdot(r, r).real <= goal:
                break
            new = cdot(shadow, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
        return x + _clover_mul(self.Ainv, bo + self.kappa * _on(_hopping(self.U, x), self.dims, 1))


def _schwarz(op, r, block, steps):
    """MR on every block at once, from zero."""
    lt, lz, ly, lx = r.shape[:4]

    def sums(u, v):
        d = (u.conj() * v).sum((-1, -2))
        d = d.reshape(lt // block[3], block[3], lz // block[2], block[2], ly // block[1], block[1], lx // block[0],
                      block[0]).sum((1, 3, 5, 7))
        for axis, n in ((0, block[3]), (1, block[2]), (2, block[1]), (3, block[0])):
            d = d.repeat_interleave(n, dim=axis)
        return d[..., None, None]

    x = torch.zeros_like(r)
    for _ in range(steps):
        q = op(r, block=block)
        a = sums(q, r) / sums(q, q).real
        x += a * r
        r = r - a * q
    return x


def _staggered_hopping(fat, lng, chi):
    lt, lz, ly, lx = chi.shape[:4]
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device=chi.device) for n in (lt, lz, ly, lx)), indexing="ij")
    out = 0
    for mu, e in enumerate((0 * x, x, x + y, x + y + z)):
        eta = (1 - 2 * (e % 2)).to(torch.float64)[..., None]
        for U, step in ((fat[..., mu, :, :], 1), (lng[mu], 3)):
            f = _mv(U, _phase(chi, mu, step)[..., None, :])[..., 0, :]
            g = _phase(_mv(_dag(U), chi[..., None, :])[..., 0, :], mu, -step)
            out = out + eta * (f - g)
    return out


def _network(channels, weights, U, psi):
    """Parallel-transport convolution network; psi [t,z,y,x,4,3] -> the same."""
    act = psi[..., None, :, :]
    for W in weights:
        co, ci = W.shape[:2]
        out = 0
        for p in range(9):
            y = act
            if p:
                mu, fwd = (p - 1) // 2, p % 2 == 1
                flat = act.reshape(act.shape[:4] + (ci * 4, 3))
                if fwd:
                    y = _mv(U[..., mu, :, :], _phase(flat, mu, 1))
                else:
                    y = _phase(_mv(_dag(U[..., mu, :, :]), flat), mu, -1)
            # [site, colour, (channel, spin)] times W_p^T
            y = y.reshape(act.shape[:4] + (ci * 4, 3)).transpose(-1, -2)
            out = out + y @ W[:, :, p].permute(0, 2, 1, 3).reshape(co * 4, ci * 4).transpose(0, 1)
        act = out.transpose(-1, -2).reshape(act.shape[:4] + (co, 4, 3))
    return act[..., 0, :, :]


def _site_order(dims, tile, parity):
    """Flat natural index of every site of one parity, in packed order."""
    lx, ly, lz, lt = dims
    i = torch.arange(lx * ly * lz * lt, device=DEVICE).view(lt, lz, ly, lx)
    i = i.masked_fill(_grid_parity(dims) != parity, -1)
    i = i.view(lt // tile[3], tile[3], lz // tile[2], tile[2], ly // tile[1], tile[1], lx // tile[0], tile[0])
    i = i.permute(0, 2, 4, 6, 1, 3, 5, 7).reshape(-1)
    return i[i >= 0]


def _chunks(rows, width):
    """[n, reals] -> chunk-major packed order."""
    return rows.view(rows.shape[0], -1, width).transpose(0, 1).reshape(-1)


def _packed(f, dims, tile, parity, n=1):
    """Natural spinors (n fields) as the library stores one parity of them."""
    V, reals = math.prod(dims), 6 if f.shape[-2:] != (4, 3) else 24
    f = torch.view_as_real(f.contiguous()).reshape(n, V, reals)[:, _site_order(dims, tile, parity)]
    R = 4 if n % 4 == 0 else 2 if n % 2 == 0 else 1
    f = f.view(n // R, R, -1, reals).transpose(1, 2).reshape(-1, reals)
    return _chunks(f, 4 if reals == 24 else 2)


def _packed_sites(rows, dims, tile, size):
    """A per-site field of both parities ([V, reals]) as the library stores it."""
    width = 16 // size
    while rows.shape[1] % width:
        width //= 2
    return [_chunks(rows[_site_order(dims, tile, p)], width) for p in (0, 1)]


def exact(case, seed):
    kind, dims, tile = case["kind"], _dims(case), _tile(case)
    U = _links(dims, seed, 0.2 if kind == "staggered" else EPS)
    if kind == "staggered":
        fat, chi = _fat_links(U, seed), _on(_sources(case, seed), dims, 0)
        lng = []
        for mu in range(4):
            a = U[..., mu, :, :]
            lng.append(_mm(a, _mm(torch.roll(a, -1, dims=3 - mu), torch.roll(a, -2, dims=3 - mu))))
        out = _staggered_hopping(fat, lng, _staggered_hopping(fat, lng, chi))
        return _packed(MASS ** 2 * chi - out / 4, dims, tile, 0)
    if kind == "setup":
        size, recon = SIZE[case["prec"]], case["recon"]
        rows = torch.view_as_real(U).reshape(-1, 4, 18)[:, :, :recon]
        gauge = torch.cat([t for mu in range(4) for t in _packed_sites(rows[:, mu], dims, tile, size)])
        out, A = [gauge], _clover(U, _kappa(case))
        low = [(i, j) for i in range(6) for j in range(i)]
        for B in (A, _inverse(A)):
            B = B.reshape(-1, 2, 6, 6)
            diag = torch.diagonal(B, dim1=-2, dim2=-1).real
            tri = torch.view_as_real(torch.stack([B[..., i, j] for i, j in low], -1)).flatten(-2)
            out.append(torch.cat(_packed_sites(torch.cat([diag, tri], -1).reshape(-1, 72), dims, tile, size)))
        return out
    b = _sources(case, seed)
    if kind.startswith("ptc"):
        channels = _ints(case["channels"], "-")
        weights, r = _weights(channels, seed), _on(b, dims, 0)
        if kind == "ptc_apply":
            with torch.no_grad():
                return _packed(_network(channels, weights, U, r), dims, tile, 0)
        for W in weights:
            W.requires_grad_(True)
        y = _on(_network(channels, weights, U, r), dims, 0)
        if case["loss"] == "residual":
            with torch.no_grad():
                op = _Schur(dims, U, _kappa(case))
            d, norm = op(y) - r, r
        else:
            norm = _on(_sources(case, seed + (1 << 40)), dims, 0)
            d = y - norm
        loss = torch.view_as_real(d).square().sum() / torch.view_as_real(norm).square().sum()
        loss.backward()
        grad = torch.cat([torch.view_as_real(W.grad).reshape(-1) for W in weights]) / 2
        w = torch.cat([torch.view_as_real(W.detach()).reshape(-1) for W in weights])
        m = 0.9 * 1e-3 * _random(seed + (1 << 41), grad.numel()) + 0.1 * grad
        v = 0.999 * 1e-5 + 0.001 * grad * grad
        w = w - 2e-4 * (m / (1 - 0.9 ** 1001)) / ((v / (1 - 0.999 ** 1001)).sqrt() + 1e-8)
        return [loss.detach(), grad, w]
    if kind == "wilson" and case["op"] == "dslash":
        fields = [b] if case.get("nrhs", 1) == 1 else list(b)
        out = torch.stack([_hopping(U, _on(f, dims, 1), case.get("dagger", 0)) for f in fields])
        return _packed(out, dims, tile, 0, len(fields))
    op = _Schur(dims, U, _kappa(case))
    if kind == "wilson":
        fields = [b] if case.get("nrhs", 1) == 1 else list(b)
        out = torch.stack([op(_on(f, dims, 0), case.get("dagger", 0)) for f in fields])
        return _packed(out, dims, tile, 0, len(fields))
    if kind == "schwarz":
        return _packed(_schwarz(op, _on(b, dims, 0), _ints(case["block"]), case["steps"]), dims, tile, 0)
    return op.solve(b)
