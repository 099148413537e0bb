"""Workloads of the library as its users' programs call it, for timing.

Each case is one call or one short chain of calls through the public entry
points (``paper_1701_07559_amd.mdwf``) on device-resident data: operator
applications (one right-hand side, or a batch that shares its launches), whole
solves, the gradient flow of the links, and the source and sink steps around a
propagator solve.  Lattices, fifth dimensions, masses and action parameters
are those of the benchmark and of the tests, or lie between them.

    listed()            the cases that are always timed
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call
    run(state)          one pass; returns its outputs
    work(case)          bytes and flops that a pass cannot do without
    exact(case, seed)   the outputs of run in 64 bits from plain torch
"""
import math

import numpy as np
import torch

from paper_1701_07559_amd import mdwf as M

M5, B5, C5 = 1.3, 1.5, 0.5            # the action of every configuration here
PREC = {"f64": M.MDWF_F64, "f32": M.MDWF_F32, "f16": M.MDWF_F16}
# bytes of one 5D site and of one real of a link in the native layouts
SITE_BYTES = {"f64": 192, "f32": 96, "f16": 52}
REAL_BYTES = {"f64": 8, "f32": 4, "f16": 2}
OPS = {
    "d5": M.MDWF_OP_D5, "d5_dag": M.MDWF_OP_D5_DAG, "schur": M.MDWF_OP_SCHUR, "schur_dag": M.MDWF_OP_SCHUR_DAG,
    "hop_eo": M.MDWF_OP_HOP_EO, "hop_oe": M.MDWF_OP_HOP_OE, "schur_rp": M.MDWF_OP_SCHUR_RP,
    "schur_rp_dag": M.MDWF_OP_SCHUR_RP_DAG, "k5inv": M.MDWF_OP_K5INV,
}
FULL_OPS = ("d5", "d5_dag", "k5inv")
# operator forms of a batched application: (operator, adjoint)
FORMS = {"schur": ("schur", "schur_dag"), "schur_rp": ("schur_rp", "schur_rp_dag")}


# ------------------------------------------------------------------ cases
def listed():
    return [
        # the smallest lattice of the tests: launch latency of one operator call
        dict(name="apply_small", kind="apply", op="schur", prec="f64", X=4, Y=4, Z=4, T=8, L5=8, mq=0.05),
        # the bare Wilson hop in single precision at the benchmark's lattice
        dict(name="hop_f32", kind="apply", op="hop_eo", prec="f32", X=24, Y=24, Z=24, T=64, L5=8, mq=0.0102),
        # the double precision even-odd operator (plain CG, reliable updates), 16^3 x 48
        dict(name="schur_f64", kind="apply", op="schur", prec="f64", X=16, Y=16, Z=16, T=48, L5=12, mq=0.0158),
        # a program that keeps canonical fields: pack, adjoint D5, unpack, on a ragged lattice
        dict(name="canon_d5_ragged", kind="canon", op="d5_dag", prec="f32", X=6, Y=10, Z=14, T=18, L5=5, mq=0.02),
        # the operator and its adjoint as the benchmark's solve launches them: 12 columns, 16-bit storage
        dict(name="batch_rp_12", kind="batch", form="schur_rp", prec="f16", X=24, Y=24, Z=24, T=64, L5=8, nrhs=12,
             masses=1, mq=0.0102),
        # three masses on the largest benchmark volume, the reference even-odd form
        dict(name="batch_s_3mass", kind="batch", form="schur", prec="f16", X=32, Y=32, Z=32, T=64, L5=10, nrhs=3,
             masses=3, mq=0.0074),
        # a small solve: one column, double precision, latency of the CG loop
        dict(name="solve_small", kind="solve", inner="f64", form=0, X=8, Y=8, Z=8, T=16, L5=8, nrhs=1, source="gauss",
             mq=0.05),
        # plain double precision CG at 16^3 x 48
        dict(name="solve_f64", kind="solve", inner="f64", form=0, X=16, Y=16, Z=16, T=48, L5=12, nrhs=1,
             source="gauss", mq=0.0158),
        # the twelve columns of a propagator, 16-bit inner solve
        dict(name="solve_f16_12", kind="solve", inner="f16", form=2, X=16, Y=16, Z=16, T=48, L5=12, nrhs=12,
             source="point", mq=0.0158),
        # gradient flow of the benchmark's links (ten steps of 0.01)
        dict(name="flow", kind="flow", X=24, Y=24, Z=24, T=64, steps=10),
        # twelve smeared sources and their 5D right-hand sides
        dict(name="source_12", kind="source", X=24, Y=24, Z=24, T=64, L5=8, nvec=12, niter=30),
        # wall and midpoint fields and the correlators of twelve solutions
        dict(name="sink_12", kind="sink", X=24, Y=24, Z=24, T=64, L5=8, nvec=12),
    ]


def _extent(rng, lo, hi):
    """An even extent, spread over the logarithm of its range."""
    return 2 * int(round(math.exp(rng.uniform(math.log(lo / 2), math.log(hi / 2)))))


def draw(rng):
    kind = rng.choice(["apply", "apply", "canon", "batch", "batch", "solve", "solve", "flow", "source", "sink"])
    big = kind in ("apply", "batch", "flow", "source", "sink")
    while True:
        d = dict(X=_extent(rng, 4, 32 if big else 16), Y=_extent(rng, 4, 32 if big else 16),
                 Z=_extent(rng, 4, 32 if big else 16), T=_extent(rng, 4, 64 if big else 48))
        L5 = rng.choice([4, 5, 6, 7, 8, 8, 10, 12, 16])
        n = rng.choice([1, 2, 3, 4, 6, 8, 11, 12])
        V = d["X"] * d["Y"] * d["Z"] * d["T"]
        sites = V * L5 * (n if kind in ("batch", "solve", "source", "sink") else 1)
        if sites <= (28_000_000 if kind == "solve" else 84_000_000) and V <= 900_000:
            break
    mq = round(math.exp(rng.uniform(math.log(0.01), math.log(0.05))), 4)
    if kind == "apply" or kind == "canon":
        op = rng.choice(["schur", "schur_dag", "hop_oe", "d5", "d5_dag", "schur_rp", "schur_rp_dag"] +
                        (["k5inv"] if kind == "canon" else []))
        return dict(kind=kind, op=op, prec=rng.choice(["f64", "f32", "f16"] if kind == "apply" else ["f64", "f32"]),
                    L5=L5, mq=mq, **d)
    if kind == "batch":
        return dict(kind=kind, form=rng.choice(["schur", "schur_rp", "schur_rp"]),
                    prec=rng.choice(["f16", "f16", "f32", "f64"]), L5=L5, nrhs=n, masses=rng.choice([1, 1, 2, 3]),
                    mq=mq, **d)
    if kind == "solve":
        inner = rng.choice(["f16", "f16", "f32", "f64"])
        return dict(kind=kind, inner=inner, form=rng.choice([0, 1, 2, 2]) if inner != "f64" else rng.choice([0, 0, 2]),
                    L5=L5, nrhs=n, source=rng.choice(["gauss", "point"]), mq=mq, **d)
    if kind == "flow":
        return dict(kind=kind, steps=rng.choice([1, 3, 5, 10]), **d)
    if kind == "source":
        return dict(kind=kind, L5=L5, nvec=n, niter=rng.choice([1, 5, 12, 30]), **d)
    return dict(kind=kind, L5=L5 + L5 % 2, nvec=n, **d)   # the midpoint needs an even L5


def _dims(case):
    return case["X"], case["Y"], case["Z"], case["T"]


def _masses(case):
    """Per-column quark masses: `masses` of them, in turn."""
    k = case.get("masses", 1)
    return [case["mq"] * (1.0 + 1.7 * (r % k)) for r in range(case["nrhs"])]


# ----------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 7919 + salt) & 0x7FFFFFFF)
    return g


def _mm(a, b):
    """Product of stacks of 3x3 matrices, element by element."""
    return (a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :]) + a[..., :, 2:3] * b[..., 2:3, :]


def _dag(a):
    return a.transpose(-1, -2).conj()


def _expm(A):
    """exp of stacks of small matrices: Taylor polynomial of A / 16, squared back."""
    A = A / 16.0
    one = torch.eye(3, dtype=A.dtype, device=A.device)
    R = one + A / 12.0
    for d in range(11, 0, -1):
        R = one + _mm(A, R) / d
    for _ in range(4):
        R = _mm(R, R)
    return R


def _links(dims, seed, eps=0.25):
    """Smooth random SU(3) links U[t][z][y][x][mu][a][b] = exp(i eps H) with E tr H^2 = 10."""
    X, Y, Z, T = dims
    g = _gen(seed, 11)
    U = torch.empty((T, Z, Y, X, 4, 3, 3), dtype=torch.complex128, device="cuda")
    r3 = 1.0 / math.sqrt(3.0)
    for t in range(T):
        h = torch.randn((8, Z, Y, X, 4), dtype=torch.float64, device="cuda", generator=g) * math.sqrt(0.625)
        H = torch.empty((Z, Y, X, 4, 3, 3), dtype=torch.complex128, device="cuda")
        H[..., 0, 0] = h[2] + r3 * h[7]
        H[..., 1, 1] = r3 * h[7] - h[2]
        H[..., 2, 2] = -2.0 * r3 * h[7]
        H[..., 0, 1] = torch.complex(h[0], -h[1])
        H[..., 0, 2] = torch.complex(h[3], -h[4])
        H[..., 1, 2] = torch.complex(h[5], -h[6])
        H[..., 1, 0] = H[..., 0, 1].conj()
        H[..., 2, 0] = H[..., 0, 2].conj()
        H[..., 2, 1] = H[..., 1, 2].conj()
        U[t] = _expm(1j * eps * H)
    return U


def _randc(shape, g):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), dtype=torch.float64, device="cuda", generator=g))


def _half_input(case, seed, k):
    """Canonical parity-compressed field of right-hand side k: [s][t][z][y][x/2][spin][col]."""
    X, Y, Z, T = _dims(case)
    return _randc((case["L5"], T, Z, Y, X // 2, 4, 3), _gen(seed, 101 + k))


def _full_input(case, seed, k):
    X, Y, Z, T = _dims(case)
    return _randc((case["L5"], T, Z, Y, X, 4, 3), _gen(seed, 101 + k))


def _source(case, seed, k):
    """Right-hand side k of a solve: a Gaussian 5D field or a spin-colour column of a point source."""
    if case["source"] == "gauss":
        return _full_input(case, seed, k)
    X, Y, Z, T = _dims(case)
    r = np.random.default_rng(int(seed))
    x, y, z, t = (int(r.integers(0, e)) for e in (X, Y, Z, T))
    b = torch.zeros((case["L5"], T, Z, Y, X, 4, 3), dtype=torch.complex128, device="cuda")
    b[case["L5"] - 1 if k % 12 < 6 else 0, t, z, y, x, (k % 12) // 3, k % 3] = 1.0
    return b


class _Context:
    """A library context on a stream of its own, released with the state."""

    def __init__(self, dims, L5, mq, U):
        self.stream = torch.cuda.Stream()
        self.h = M.mdwf_create(dims, hip_stream=self.stream.cuda_stream)
        M.mdwf_set_action(self.h, M5, B5, C5, mq, L5)
        torch.cuda.synchronize()
        M.mdwf_load_gauge_dev(self.h, U.data_ptr())

    def __del__(self):
        if getattr(self, "h", None):
            torch.cuda.synchronize()
            M.mdwf_destroy(self.h)
            self.h = None


def _view(buf, prec, vh):
    """A native half field's values, without the layout's padding."""
    if prec == "f64":
        return buf[: 192 * vh].view(torch.float64).view(12, vh, 2)
    if prec == "f32":
        return buf[: 96 * vh].view(torch.float32).view(6, vh, 4)
    off = (48 * vh + 255) // 256 * 256
    return buf[: 48 * vh].view(torch.float16).view(3, vh, 8), buf[off: off + 4 * vh].view(torch.float32)


def _views(buf, prec, vh):
    """Batched _view of the fields [nrhs][stride]: all values as one or two tensors."""
    n = buf.shape[0]
    if prec == "f64":
        return buf[:, : 192 * vh].view(torch.float64).view(n, 12, vh, 2)
    if prec == "f32":
        return buf[:, : 96 * vh].view(torch.float32).view(n, 6, vh, 4)
    off = (48 * vh + 255) // 256 * 256
    return [buf[:, : 48 * vh].view(torch.float16).view(n, 3, vh, 8), buf[:, off: off + 4 * vh].view(torch.float32)]


def prepare(case, seed):
    dims, kind = _dims(case), case["kind"]
    st = {"case": case}
    if kind == "flow":
        st["links"] = _links(dims, seed)
        st["U"] = st["links"].clone()
        return st
    if kind == "source":
        st["U"] = _links(dims, seed)
        X, Y, Z, T = dims
        n = case["nvec"]
        g = _gen(seed, 101)
        st["eta"] = torch.stack([_randc((T, Z, Y, X, 4, 3), g) for _ in range(n)])
        st["smeared"] = torch.empty_like(st["eta"])
        st["b"] = torch.empty((n, case["L5"], T, Z, Y, X, 4, 3), dtype=torch.complex128, device="cuda")
        return st
    if kind == "sink":
        st["x"] = torch.stack([_full_input(case, seed, k) for k in range(case["nvec"])])
        X, Y, Z, T = dims
        st["q"] = torch.empty((case["nvec"], T, Z, Y, X, 4, 3), dtype=torch.complex128, device="cuda")
        st["mid"] = torch.empty_like(st["q"])
        return st
    L5 = case["L5"]
    st["ctx"] = ctx = _Context(dims, L5, case["mq"], _links(dims, seed))
    vh = L5 * dims[0] * dims[1] * dims[2] * dims[3] // 2
    if kind == "solve":
        st["b"] = [_source(case, seed, k) for k in range(case["nrhs"])]
        st["x"] = [torch.empty_like(b) for b in st["b"]]
        st["opts"] = dict(tol=1e-11, inner=PREC[case["inner"]], schur_form=case["form"])
        torch.cuda.synchronize()
        return st
    prec = PREC[case["prec"]]
    full = kind == "canon" or case.get("op") in FULL_OPS
    st["vh"] = vh
    hb = M.mdwf_field_bytes(ctx.h, prec, M.MDWF_HALF_EVEN)
    if kind == "canon":
        st["in"] = (_full_input if case["op"] in FULL_OPS else _half_input)(case, seed, 0)
        st["out"] = torch.empty_like(st["in"])
        fb = M.mdwf_field_bytes(ctx.h, prec, M.MDWF_FULL)
        st["nin"] = torch.empty(fb, dtype=torch.uint8, device="cuda")
        st["nout"] = torch.empty(fb, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        return st
    n = case.get("nrhs", 1)
    fb = 2 * hb if full else hb
    st["in"] = torch.zeros((n, fb), dtype=torch.uint8, device="cuda")
    kin = M.OP_KINDS[OPS[case["op"]]][0] if kind == "apply" else M.MDWF_HALF_EVEN
    for k in range(n):
        c = (_full_input if full else _half_input)(case, seed, k)
        torch.cuda.synchronize()
        M.mdwf_pack_dev(ctx.h, prec, kin, c.data_ptr(), st["in"][k].data_ptr())
        torch.cuda.synchronize()
    st["out"] = torch.zeros_like(st["in"])
    if kind == "batch":
        st["out2"] = torch.zeros_like(st["in"])
        st["masses"] = _masses(case)
    torch.cuda.synchronize()
    return st


def run(st):
    case = st["case"]
    kind, dims = case["kind"], _dims(case)
    if kind == "flow":
        st["U"].copy_(st["links"])   # the flow works in place
        p0, p1 = M.mdwf_wilson_flow_dev(dims, st["U"].data_ptr(), 0.01, case["steps"])
        return [st["U"], p0, p1]
    if kind == "source":
        M.mdwf_gauss_smear_dev(dims, st["U"].data_ptr(), case["nvec"], st["eta"].data_ptr(), st["smeared"].data_ptr(),
                               4.0, case["niter"])
        M.mdwf_wall_source_dev(dims, (M5, B5, C5, 0.01, case["L5"]), st["U"].data_ptr(), case["nvec"],
                               st["smeared"].data_ptr(), st["b"].data_ptr())
        return [st["smeared"], st["b"]]
    if kind == "sink":
        M.mdwf_project_4d_dev(dims, case["L5"], case["nvec"], st["x"].data_ptr(), st["q"].data_ptr(),
                              st["mid"].data_ptr())
        cpp, cmp_, mres = M.mdwf_mres_correlators_dev(dims, case["L5"], case["nvec"], st["x"].data_ptr())
        pion = M.mdwf_pion_correlator_dev(dims, case["nvec"], st["q"].data_ptr())
        return [st["q"], st["mid"], cpp, cmp_, mres, pion]
    h = st["ctx"].h
    if kind == "solve":
        status, _ = M.mdwf_solve_dev(h, [b.data_ptr() for b in st["b"]], [x.data_ptr() for x in st["x"]],
                                     opts=st["opts"])
        if status != M.MDWF_OK:
            raise RuntimeError("the solve did not converge")
        return st["x"]
    prec = PREC[case["prec"]]
    if kind == "canon":
        kin, kout = M.OP_KINDS[OPS[case["op"]]]
        M.mdwf_pack_dev(h, prec, kin, st["in"].data_ptr(), st["nin"].data_ptr())
        M.mdwf_apply_dev(h, OPS[case["op"]], prec, st["nin"].data_ptr(), st["nout"].data_ptr())
        M.mdwf_unpack_dev(h, prec, kout, st["nout"].data_ptr(), st["out"].data_ptr())
        return st["out"]
    if kind == "apply":
        M.mdwf_apply_dev(h, OPS[case["op"]], prec, st["in"].data_ptr(), st["out"].data_ptr())
        if case["op"] in FULL_OPS:
            hb = st["out"].shape[1] // 2
            return [_view(st["out"][0, k * hb: (k + 1) * hb], case["prec"], st["vh"]) for k in range(2)]
        return _view(st["out"][0], case["prec"], st["vh"])
    fwd, adj = FORMS[case["form"]]
    n, stride = st["in"].shape
    for op, out in ((fwd, st["out"]), (adj, st["out2"])):
        M.mdwf_apply_batch_dev(h, OPS[op], prec, n, st["in"].data_ptr(), out.data_ptr(), stride, st["masses"])
    # the first columns apart: those are the ones `exact` computes
    k = min(n, 2)
    return [_views(o[a:b], case["prec"], st["vh"]) for o in (st["out"], st["out2"]) for a, b in ((0, k), (k, n))
            if b > a]


# ------------------------------------------------------------ needed work
def _op_work(op, prec, V, L5):
    """Bytes and flops of one application: every spinor field read once and
    written once per hop kernel (the odd intermediate of the Schur operators
    included, the links beside it), flops as in the library's own model."""
    vh, s = V * L5 // 2, SITE_BYTES[prec]
    links, hop = V * 72 * REAL_BYTES[prec], 1320 * vh
    if op in ("hop_eo", "hop_oe"):
        return 2 * s * vh, links, hop
    if op in ("d5", "d5_dag"):
        return 4 * s * vh, links, 2 * hop + 2 * 192 * vh
    if op == "k5inv":
        return 4 * s * vh, 0, 2 * 48 * L5 * vh
    dense = 48 * L5 * vh
    return 4 * s * vh, links, 2 * hop + (dense if op.startswith("schur_rp") else 0) + dense + 192 * vh


def work(case):
    X, Y, Z, T = _dims(case)
    V, kind = X * Y * Z * T, case["kind"]
    if kind == "flow":
        # three stages a step: links and the accumulator read and written once each
        return dict(bytes=3 * case["steps"] * 4 * V * 395.0 + 2 * 4 * V * 144.0,
                    flops=3 * case["steps"] * 4 * V * 5616.0)
    if kind == "source":
        n = case["nvec"]
        step = V * n * 384.0 + V * 3 * 144.0
        return dict(bytes=case["niter"] * step + V * n * 192.0 * (1 + case["L5"]) + V * 576.0,
                    flops=case["niter"] * V * n * 1632.0 + V * n * 2640.0)
    if kind == "sink":
        # the four slices of x that enter, the two fields written, q read again for its correlator
        return dict(bytes=V * case["nvec"] * (2 * 192.0 + 2 * 192.0), flops=V * case["nvec"] * 3 * 48.0)
    L5 = case["L5"]
    if kind == "canon":
        b, l, f = _op_work(case["op"], case["prec"], V, L5)
        half = 1 if case["op"] in FULL_OPS else 2
        return dict(bytes=float(b + l + 2 * V * L5 * 192 // half + 2 * V * L5 * SITE_BYTES[case["prec"]] // half),
                    flops=float(f))
    if kind == "apply":
        b, l, f = _op_work(case["op"], case["prec"], V, L5)
        return dict(bytes=float(b + l), flops=float(f))
    if kind == "batch":
        b, l, f = _op_work(FORMS[case["form"]][0], case["prec"], V, L5)
        return dict(bytes=2.0 * (case["nrhs"] * b + l), flops=2.0 * case["nrhs"] * f)
    # a solve: CG iterations to 1e-11 as the library's runs at these masses take them
    iters = 150 * (0.05 / case["mq"]) ** 0.5
    b, l, f = _op_work("schur_rp" if case["form"] == 2 else "schur", case["inner"], V, L5)
    vec = 6.5 * SITE_BYTES[case["inner"]] * V * L5 // 2
    return dict(bytes=iters * (case["nrhs"] * (2.0 * b + vec) + 2.0 * l), flops=2.0 * iters * case["nrhs"] * f)


# ------------------------------------------------- plain torch in 64 bits
# Full-lattice fields psi[s][t][z][y][x][spin][col], complex128, chiral basis
# g5 = diag(1, 1, -1, -1), g_mu = [[0, G], [G^+, 0]], G = (-i s1, -i s2, -i s3, 1).
_AXIS = {0: 4, 1: 3, 2: 2, 3: 1}


def _link_mul(U, h):
    """U[t][z][y][x][a][b] times the colour index of h[...][spin][col]."""
    return (U[..., None, :, 0] * h[..., 0:1] + U[..., None, :, 1] * h[..., 1:2]) + U[..., None, :, 2] * h[..., 2:3]


def _G(mu, d, dag):
    """G_mu (or its adjoint) on a spin pair d[..., 2, 3]."""
    d0, d1 = d[..., 0, :], d[..., 1, :]
    if mu == 0:
        o = (-1j * d1, -1j * d0) if not dag else (1j * d1, 1j * d0)
    elif mu == 1:
        o = (-d1, d0) if not dag else (d1, -d0)
    elif mu == 2:
        o = (-1j * d0, 1j * d1) if not dag else (1j * d0, -1j * d1)
    else:
        return d
    return torch.stack(o, dim=-2)


def _hop(U, psi, anti=True, dag=False):
    """Dslash on every slice: sum_mu (1 - g_mu) U psi(x+mu) + (1 + g_mu) U^+ psi(x-mu); dag: g5 Dslash g5."""
    out = torch.zeros_like(psi)
    T = psi.shape[1]
    for mu in range(4):
        Um = U[..., mu, :, :]
        if mu == 3 and anti:
            Um = Um.clone()
            Um[T - 1] = -Um[T - 1]
        for d in (1, -1):
            sg = float(d) * (-1.0 if dag else 1.0)
            nb = torch.roll(psi, -d, dims=_AXIS[mu])
            L = Um if d > 0 else _dag(torch.roll(Um, 1, dims=_AXIS[mu] - 1))
            w = _link_mul(L, nb[..., :2, :] - sg * _G(mu, nb[..., 2:, :], False))
            out[..., :2, :] += w
            out[..., 2:, :] -= sg * _G(mu, w, True)
    return out


def _mats(L5, mq):
    """The fifth-dimension operators as L5 x L5 matrices on (P+ spins, P- spins)."""
    up = torch.zeros((L5, L5), dtype=torch.float64, device="cuda")
    for s in range(L5):
        up[s, (s - 1) % L5] += -mq if s == 0 else 1.0
    dn = torch.zeros_like(up)
    for s in range(L5):
        dn[s, (s + 1) % L5] += -mq if s == L5 - 1 else 1.0
    one = torch.eye(L5, dtype=torch.float64, device="cuda")
    r = {}
    for name, C in (("p", up), ("m", dn)):
        B = B5 * one + C5 * C
        K = (4.0 - M5) * B + one - C
        r[name] = dict(C=C, B=B, K=K, Ki=torch.linalg.inv(K), Bi=torch.linalg.inv(B))
    return r


def _five(m, names, psi, dag=False):
    """Product of fifth-dimension matrices (left to right) on psi, or its adjoint."""
    out = torch.empty_like(psi)
    for h, sl in (("p", slice(0, 2)), ("m", slice(2, 4))):
        A = m[h][names[0]]
        for n in names[1:]:
            A = A @ m[h][n]
        if dag:
            A = A.t()
        v = torch.view_as_real(psi[..., sl, :].contiguous())
        out[..., sl, :] = torch.view_as_complex((A @ v.reshape(A.shape[0], -1)).view(v.shape))
    return out


def _apply_ref(op, U, psi, m):
    if op in ("hop_eo", "hop_oe"):
        return _hop(U, psi)
    if op == "k5inv":
        return _five(m, ["Ki"], psi)
    if op == "d5":
        w = _five(m, ["B"], psi)
        return _five(m, ["K"], psi) - 0.5 * _hop(U, w)
    if op == "d5_dag":
        return _five(m, ["K"], psi, True) - 0.5 * _five(m, ["B"], _hop(U, psi, dag=True), True)
    if op == "schur":
        return _five(m, ["K"], psi) - 0.25 * _hop(U, _five(m, ["B", "Ki"], _hop(U, _five(m, ["B"], psi))))
    if op == "schur_rp":
        return _five(m, ["K", "Bi"], psi) - 0.25 * _hop(U, _five(m, ["B", "Ki"], _hop(U, psi)))
    q = _hop(U, _five(m, ["B", "Ki"], _hop(U, psi, dag=True), True), dag=True)
    if op == "schur_dag":
        return _five(m, ["K"], psi, True) - 0.25 * _five(m, ["B"], q, True)
    return _five(m, ["K", "Bi"], psi, True) - 0.25 * q


def _mask_index(dims, parity):
    """x of the parity-compressed sites, [t][z][y][x/2]."""
    X, Y, Z, T = dims
    t, z, y, h = torch.meshgrid(*[torch.arange(n, device="cuda") for n in (T, Z, Y, X // 2)], indexing="ij")
    return 2 * h + ((y + z + t + parity) & 1)


def _expand(h, dims, parity):
    X, Y, Z, T = dims
    idx = _mask_index(dims, parity)[None, ..., None, None].expand(h.shape)
    out = torch.zeros((h.shape[0], T, Z, Y, X, 4, 3), dtype=h.dtype, device=h.device)
    return out.scatter_(4, idx, h)


def _compress(f, dims, parity):
    X, Y, Z, T = dims
    idx = _mask_index(dims, parity)[None, ..., None, None].expand((f.shape[0], T, Z, Y, X // 2, 4, 3))
    return torch.gather(f, 4, idx)


def _native(h, prec):
    """The native layout of a parity-compressed canonical field, in 64 bits."""
    v = torch.view_as_real(h.permute(1, 2, 3, 4, 0, 5, 6).contiguous()).reshape(-1, 24)
    if prec == "f64":
        return v.view(-1, 12, 2).transpose(0, 1).contiguous()
    if prec == "f32":
        return v.view(-1, 6, 4).transpose(0, 1).contiguous()
    n = v.abs().amax(1)
    s = v / torch.where(n > 0, n, torch.ones_like(n))[:, None]
    return [s.view(-1, 3, 8).transpose(0, 1).contiguous(), n]


def _true_solution(case, U, b):
    """D5 x = b by CG on the normal equations of D5 in 64 bits, to a residual of 2e-14."""
    m = _mats(case["L5"], case["mq"])
    x, r = torch.zeros_like(b), b.clone()
    s = _apply_ref("d5_dag", U, r, m)
    p = s.clone()
    gamma, nb = float(torch.linalg.vector_norm(s)) ** 2, float(torch.linalg.vector_norm(b))
    for k in range(3000):
        q = _apply_ref("d5", U, p, m)
        a = gamma / float(torch.linalg.vector_norm(q)) ** 2
        x += a * p
        r -= a * q
        if k % 50 == 49:
            r = b - _apply_ref("d5", U, x, m)
        if float(torch.linalg.vector_norm(r)) < 2e-14 * nb:
            break
        s = _apply_ref("d5_dag", U, r, m)
        g2 = float(torch.linalg.vector_norm(s)) ** 2
        p = s + (g2 / gamma) * p
        gamma = g2
    return x


def _force(U):
    out = torch.empty_like(U)
    one = torch.eye(3, dtype=U.dtype, device=U.device)
    ax = {0: 3, 1: 2, 2: 1, 3: 0}
    for mu in range(4):
        A, S = U[..., mu, :, :], 0.0
        for nu in range(4):
            if nu == mu:
                continue
            N = U[..., nu, :, :]
            S = S + _mm(torch.roll(N, -1, ax[mu]), _dag(_mm(N, torch.roll(A, -1, ax[nu]))))
            Nm = torch.roll(N, 1, ax[nu])
            S = S + _mm(_dag(_mm(torch.roll(A, 1, ax[nu]), torch.roll(Nm, -1, ax[mu]))), Nm)
        O = _mm(A, S)
        O = O - _dag(O)
        tr = O[..., 0, 0] + O[..., 1, 1] + O[..., 2, 2]
        out[..., mu, :, :] = -0.5 * O + (tr / 6.0)[..., None, None] * one
    return out


def _plaquette(U):
    ax, tot = {0: 3, 1: 2, 2: 1, 3: 0}, 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            A, N = U[..., mu, :, :], U[..., nu, :, :]
            P = _mm(_mm(A, torch.roll(N, -1, ax[mu])), _dag(_mm(N, torch.roll(A, -1, ax[nu]))))
            tot += float((P[..., 0, 0] + P[..., 1, 1] + P[..., 2, 2]).real.mean()) / 18.0
    return tot


def exact(case, seed):
    dims, kind = _dims(case), case["kind"]
    if kind == "flow":
        U = _links(dims, seed)
        p0 = _plaquette(U)
        for _ in range(case["steps"]):
            E = 0.25 * 0.01 * _force(U)
            U = _mm(_expm(E), U)
            E = (8.0 / 9.0) * 0.01 * _force(U) - (17.0 / 9.0) * E
            U = _mm(_expm(E), U)
            E = 0.75 * 0.01 * _force(U) - E
            U = _mm(_expm(E), U)
        return [U, p0, _plaquette(U)]
    if kind == "source":
        U = _links(dims, seed)
        X, Y, Z, T = dims
        g = _gen(seed, 101)
        kap = 16.0 / (4.0 * case["niter"])
        sm, bs = [], []
        for _ in range(case["nvec"]):
            e = _randc((T, Z, Y, X, 4, 3), g)
            for _ in range(case["niter"]):
                lap = -6.0 * e
                for mu in range(3):
                    Um, ax = U[..., mu, :, :], _AXIS[mu] - 1
                    lap += _link_mul(Um, torch.roll(e, -1, ax))
                    lap += torch.roll(_link_mul(_dag(Um), e), 1, ax)
                e = e + kap * lap
            b = torch.zeros((case["L5"],) + tuple(e.shape), dtype=e.dtype, device=e.device)
            for s, lo, hi in ((case["L5"] - 1, 2, 4), (0, 0, 2)):
                p = torch.zeros_like(e)
                p[..., lo:hi, :] = e[..., lo:hi, :]
                b[s] += (1.0 - C5 * (4.0 - M5)) * p + 0.5 * C5 * _hop(U, p[None])[0]
            sm.append(e)
            bs.append(b)
        return [torch.stack(sm), torch.stack(bs)]
    if kind == "sink":
        L = case["L5"]
        q, mid = [], []
        for k in range(case["nvec"]):
            x = _full_input(case, seed, k)
            q.append(torch.cat([x[L - 1][..., :2, :], x[0][..., 2:, :]], dim=-2))
            mid.append(torch.cat([x[L // 2 - 1][..., :2, :], x[L // 2][..., 2:, :]], dim=-2))
        q, mid = torch.stack(q), torch.stack(mid)
        cpp, cmp_ = ((f.real.square() + f.imag.square()).sum(dim=(0, 2, 3, 4, 5, 6)) for f in (q, mid))
        return [q, mid, cpp, cmp_, cmp_ / cpp, cpp]
    sites = case["L5"] * dims[0] * dims[1] * dims[2] * dims[3]
    U = _links(dims, seed)
    if kind == "solve":
        if sites * case["nrhs"] > 600_000:
            return None
        return [_true_solution(case, U, _source(case, seed, k)) for k in range(case["nrhs"])]
    if kind == "batch":
        n, k, first, res = case["nrhs"], min(case["nrhs"], 2), _masses(case), []
        for op in FORMS[case["form"]]:
            outs = []
            for r in range(k):
                m = _mats(case["L5"], first[r])
                full = _apply_ref(op, U, _expand(_half_input(case, seed, r), dims, 0), m)
                outs.append(_native(_compress(full, dims, 0), case["prec"]))
                del full
            if case["prec"] == "f16":
                res.append([torch.stack([o[0] for o in outs]), torch.stack([o[1] for o in outs])])
                rest = [None, None]
            else:
                res.append(torch.stack(outs))
                rest = None
            if n > k:
                res.append(rest)
        return res
    op, m = case["op"], _mats(case["L5"], case["mq"])
    if op in FULL_OPS:
        full = _apply_ref(op, U, _full_input(case, seed, 0), m)
        if kind == "canon":
            return full
        return [_native(_compress(full, dims, p), case["prec"]) for p in (0, 1)]
    pin = 1 if op == "hop_eo" else 0
    pout = 1 - pin if op in ("hop_eo", "hop_oe") else 0
    full = _compress(_apply_ref(op, U, _expand(_half_input(case, seed, 0), dims, pin), m), dims, pout)
    return full if kind == "canon" else _native(full, case["prec"])
