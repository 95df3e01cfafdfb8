"""Performance cases of the MRHS setup library: what a program that uses it calls, over its
range of lattices, right-hand sides, precisions and block solvers.

Kinds:
  setup    the initial setup phase: SAP on random test vectors, FP64 residual norms, block
           Gram-Schmidt, coarse operator
  sap      the smoother alone (plain MR or even-odd block solver, any precision)
  batch    the smoother on several lattices of uneven size in one call
  dirac    the stencil on all right-hand sides
  rebuild  Gram-Schmidt and coarse operator alone, with Q and D_c stored in binary16: the last
           line of the refinement loop with a half-precision coarse grid
  transfer restriction and prolongation
  solve    the low-accuracy coarse solve (FP32 or half-precision coarse grid)
  refine   one pass of the refinement phase over all test vectors

The lattices, mass, sweeps and test-vector counts are those of the benchmark and the tests
(4^4, 16^4, 24^3x48, 32^3x64, the uneven batch); drawn cases take others from the same ranges,
ragged vector counts and blocks of other shapes among them.
"""
import numpy as np
import torch

from paper_1601_03184_amd import mrhs

CSW = 1.0
PRECS = {"f64": mrhs.PREC_F64, "f32": mrhs.PREC_F32, "f16": mrhs.PREC_F32_F16STORE}
DTYPES = {"f64": mrhs.DTYPE_F64, "f32": mrhs.DTYPE_F32, "f16": mrhs.DTYPE_F16}
REAL_BYTES = {"f64": 8, "f32": 4, "f16": 2}
S = 4                     # short-vector length of the multiple-right-hand-side layout
M_COARSE, TOL_COARSE = 8, 0.05   # the refinement phase's coarse solve
BATCH = (("8x8x8x8", 8), ("12x12x12x12", 16), ("16x16x16x32", 24))
LARGEST = 32 ** 3 * 64 * 32      # site x right-hand side of the largest listed case
EXACT_MOST = 20_000_000          # site x right-hand side up to which exact() is quick enough


def listed():
    c = []

    def add(name, kind, L, n, prec="f32", block="4x4x4x4", **opt):
        c.append(dict(dict(name=name, kind=kind, L=L, n=n, prec=prec, block=block, n_sap=3, n_mr=4, tile=0, solver="mr",
                           coarse="f32", sigma=0.3, m0=-0.3), **opt))

    # the smallest call a user makes: the whole phase on the smoke lattice, FP64; launches count
    add("setup_4x4x4x4_f64_n8", "setup", "4x4x4x4", 8, "f64", "2x2x2x2", n_sap=2, n_mr=3, m0=-0.1)
    # an ordinary lattice of the tests and the earlier benchmark, with the operator as created
    add("setup_16x16x16x16_f32_n20", "setup", "16x16x16x16", 20)
    # the benchmark's step on the largest lattice whose state fits the card several times, with
    # the benchmark's vector count and the tile that the autotuner picks on large lattices
    add("setup_32x32x32x64_f32_n32", "setup", "32x32x32x64", 32, tile=4, sigma=0.25, m0=-0.33)
    # several small lattices at once (an odd number of blocks per direction among them)
    add("batch_3_lattices_f32", "batch", "16x16x16x32", 24, tile=4)
    # FP16 storage of the vectors
    add("sap_24x24x24x48_f16_n24", "sap", "24x24x24x48", 24, "f16", tile=4, sigma=0.25, m0=-0.33)
    # the even-odd block solver with the operator as created
    add("sap_eo_16x16x16x32_f32_n24", "sap", "16x16x16x32", 24, solver="eo", n_mr=3)
    # full precision, odd block counts and a ragged last group
    add("sap_12x12x12x24_f64_n10", "sap", "12x12x12x24", 10, "f64")
    # the operator itself, as an outer solver calls it
    add("dirac_32x32x32x64_f32_n24", "dirac", "32x32x32x64", 24, sigma=0.25, m0=-0.33)
    # the rebuild that closes a refinement pass, half-precision coarse grid
    add("rebuild_24x24x24x48_q16_n24", "rebuild", "24x24x24x48", 24, sigma=0.25, m0=-0.33)
    # the two grid transfers of a cycle
    add("transfer_24x24x24x48_f32_n32", "transfer", "24x24x24x48", 32)
    # the coarse solve of a large lattice
    add("solve_32x32x32x64_f32_n32", "solve", "32x32x32x64", 32)
    # a whole refinement pass on an ordinary lattice: a small coarse grid, many launches
    add("refine_16x16x16x16_f32_n20", "refine", "16x16x16x16", 20)
    return c


def draw(rng):
    kind = rng.choice(["setup", "sap", "sap", "sap", "batch", "dirac", "rebuild", "transfer", "solve", "refine"])
    prec = rng.choice(["f32", "f32", "f32", "f16", "f64"]) if kind in ("sap", "dirac", "setup") else "f32"
    block = rng.choice([(4, 4, 4, 4), (4, 4, 4, 4), (4, 4, 4, 4), (2, 4, 4, 4), (4, 4, 4, 2), (2, 2, 2, 2), (3, 3, 3, 3),
                        (4, 2, 4, 6)])
    if kind in ("solve", "refine", "transfer", "rebuild", "batch"):
        block = (4, 4, 4, 4)
    if kind == "setup" and block == (4, 2, 4, 6):
        block = (4, 4, 4, 4)   # the coarse operator takes aggregates with faces up to 64 sites
    eo = kind == "sap" and all(b % 2 == 0 for b in block) and rng.random() < 0.35
    n = rng.choice([1, 3, 5, 7, 8, 12, 13, 16, 20, 24, 25, 29, 31, 32])
    if kind in ("setup", "rebuild", "refine", "solve", "transfer"):
        n = max(n, 3)
    most = LARGEST // {"f64": 8, "f32": 2, "f16": 2}[prec]
    target = 2.0 ** rng.uniform(8, 21)
    while True:
        L = [max(1, int(round(target ** 0.25 * rng.uniform(0.6, 1.6) / b))) * b for b in block]
        if np.prod(L) <= 32 ** 3 * 64 and np.prod(L) * n <= most and max(l // b for l, b in zip(L, block)) <= 64 and \
                np.prod(L) // np.prod(block) * n * n <= 8192 * 32 * 32:
            break
        target *= 0.7
    return dict(kind=kind, L="x".join(map(str, L)), n=n, prec=prec, block="x".join(map(str, block)),
                n_sap=rng.choice([1, 2, 3, 4]), n_mr=rng.choice([2, 3, 4, 5]),
                tile=rng.choice([0, 4]) if prec != "f64" else 0,
                solver="eo" if eo else "mr", coarse=rng.choice(["f32", "f16"]) if kind == "solve" else "f32",
                sigma=rng.choice([0.2, 0.25, 0.3]), m0=rng.choice([-0.1, -0.3, -0.33]))


# ---- inputs -----------------------------------------------------------------------------------

def ints(text):
    return [int(v) for v in text.split("x")]


def device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def normals(seed, shape, dtype=torch.float32):
    gen = torch.Generator(device=device())
    gen.manual_seed(int(seed))
    return torch.randn(shape, generator=gen, dtype=dtype, device=device())


def mul3(a, b):
    """Products of 3x3 matrices over the leading indices, by columns of a and rows of b."""
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def links(L, sigma, seed):
    """SU(3) links near unity, complex128 [4][V][3][3]: 1 + i sigma H - sigma^2 H^2 / 2 with H
    Hermitian, traceless and Gaussian, made unitary by Gram-Schmidt on the rows."""
    V = int(np.prod(L))
    out = torch.empty((4, V, 3, 3), dtype=torch.complex128, device=device())
    eye = torch.eye(3, dtype=torch.complex128, device=device())
    for mu in range(4):
        A = torch.view_as_complex(normals(seed * 1009 + mu, (V, 3, 3, 2)).double())
        H = 0.5 * (A + A.conj().transpose(-1, -2))
        H = H - (torch.diagonal(H, dim1=-2, dim2=-1).sum(-1).real / 3.0)[:, None, None] * eye
        X = 1j * sigma * H
        U = eye + X + 0.5 * mul3(X, X)
        r0 = U[:, 0]
        r0 = r0 / (r0.abs() ** 2).sum(-1, keepdim=True).sqrt()
        r1 = U[:, 1] - (r0.conj() * U[:, 1]).sum(-1, keepdim=True) * r0
        r1 = r1 / (r1.abs() ** 2).sum(-1, keepdim=True).sqrt()
        r2 = torch.stack([r0[:, (k + 1) % 3] * r1[:, (k + 2) % 3] - r0[:, (k + 2) % 3] * r1[:, (k + 1) % 3]
                          for k in range(3)], -1).conj()
        out[mu] = torch.stack([r0, r1, r2], 1)
    return out


def vectors(L, n, seed, first=0):
    """Vectors first .. first + n - 1 of a set of complex Gaussian test vectors, complex128 [n][V][4][3]."""
    V = int(np.prod(L))
    return torch.stack([torch.view_as_complex(normals(seed * 100003 + 17 + first + k, (V, 4, 3, 2)).double())
                        for k in range(n)])


def smoothed(L, n, seed, first=0):
    """Vectors with the overlaps that smoothing leaves: each shares a part with its successor."""
    v = vectors(L, n + 1, seed, first)
    return v[:-1] + 0.6 * v[1:]


def packed(op, make, n, dtype):
    """n native vectors from make(count, first), one group of the layout at a time."""
    out = op.empty(n, dtype)
    per = mrhs.mrhs_vector_bytes(op.handle, op.S, dtype) // out.element_size()
    for g in range((n + op.S - 1) // op.S):
        m = min(op.S, n - g * op.S)
        mrhs.mrhs_pack(op.handle, torch.view_as_real(make(m, g * op.S)), out[g * per:(g + 1) * per], dtype, m)
    return out


def coarse_blocks(Vc, n_tv, seed):
    """D_c of a coarse lattice, float32 [Vc][9][2N][2N][2]: Gaussian blocks with the self blocks
    dominating, which the coarse solve reduces to 0.05 in a few iterations."""
    N2 = 2 * n_tv
    D = normals(seed * 7919 + 3, (Vc, 9, N2, N2, 2))
    D *= 0.5 / N2 ** 0.5
    D[:, 0, range(N2), range(N2), 0] += 4.0
    return D


def coarse_vectors(Vc, n_tv, n, seed):
    """Coarse vectors, float32 [Vc][2N][2][ldc] with zero padding."""
    v = normals(seed * 6007 + 5, (Vc, 2 * n_tv, 2, (n + 3) // 4 * 4))
    v[..., n:] = 0.0
    return v


def operator(case, L, seed):
    op = mrhs.Operator(L, ints(case["block"]), ints(case["block"]), links(L, case["sigma"], seed), case["m0"], CSW,
                       prec=PRECS[case["prec"]], short_len=S)
    if case["tile"]:
        if case["kind"] == "dirac":
            mrhs.mrhs_set_tiles(op.handle, 0, case["tile"])
        else:
            mrhs.mrhs_set_tiles(op.handle, case["tile"], 0)
    if case["solver"] == "eo":
        mrhs.mrhs_set_block_solver(op.handle, mrhs.BLOCK_EO_MR)
    return op


def batch_of(case):
    """The lattices of a batch: the two small ones of every batch and the case's own."""
    return [(ints(l), n) for l, n in BATCH[:2]] + [(ints(case["L"]), case["n"])]


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    st = dict(case=case, n=n)
    if kind == "batch":
        st["ops"], st["b"], st["x"], st["ns"] = [], [], [], []
        for k, (L, m) in enumerate(batch_of(case)):
            op = operator(case, L, seed + 50 * k)
            st["ops"].append(op)
            st["ns"].append(m)
            st["b"].append(packed(op, lambda c, f, L=L, k=k: vectors(L, c, seed + 50 * k, f), m, op.dtype))
            st["x"].append(op.empty(m))
        st["handles"] = [o.handle for o in st["ops"]]
        st["ws"] = torch.empty(mrhs.mrhs_batched_workspace_bytes(st["handles"], st["ns"]), dtype=torch.uint8, device="cuda")
        return st
    L = ints(case["L"])
    op = st["op"] = operator(case, L, seed)
    make = vectors if kind in ("setup", "sap", "dirac") else smoothed
    if kind != "solve":
        st["b"] = packed(op, lambda c, f: make(L, c, seed, f), n, op.dtype)
    if kind in ("setup", "sap", "dirac"):
        st["x"] = op.empty(n)
    if kind in ("setup", "sap", "rebuild"):
        st["ws"] = op.workspace(n)
    if kind == "setup":
        st["res"] = torch.empty(n, dtype=torch.float64, device="cuda")
        st["qdt"] = DTYPES[case["prec"] if case["prec"] != "f16" else "f32"]
    if kind == "rebuild":
        st["qdt"] = mrhs.DTYPE_F16
    if kind in ("setup", "rebuild"):
        st["Q"] = op.empty(n, st["qdt"])
        st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        st["Dc"] = torch.empty(op.n_agg * 9 * (2 * n) ** 2 * 2, dtype=torch.float16 if kind == "rebuild" else torch.float32,
                               device="cuda")
    if kind in ("transfer", "refine"):
        # Q with the magnitudes of orthonormal columns, given to the calls as data
        scale = (6.0 * np.prod(ints(case["block"]))) ** -0.5
        st["Q"] = packed(op, lambda c, f: scale * 0.5 ** 0.5 * vectors(L, c, seed + 1, f), n, mrhs.DTYPE_F32)
    if kind == "transfer":
        st["yc"], st["y"] = op.coarse_empty(n, n), op.empty(n)
    if kind in ("solve", "refine"):
        D = coarse_blocks(op.n_agg, n, seed)
        st["Dc"] = D.half() if case["coarse"] == "f16" else D
    if kind == "solve":
        st["bc"] = coarse_vectors(op.n_agg, n, n, seed)
        st["uc"] = torch.empty_like(st["bc"])
        st["res"] = torch.empty(n, dtype=torch.float64, device="cuda")
        size = mrhs.mrhs_coarse_solve_f16_workspace_bytes if st["Dc"].dtype == torch.float16 else \
            mrhs.mrhs_coarse_solve_workspace_bytes
        st["ws"] = torch.empty(size(op.handle, n, n, M_COARSE), dtype=torch.uint8, device="cuda")
    if kind == "refine":
        st["V"] = torch.empty_like(st["b"])
        st["ws"] = torch.empty(mrhs.mrhs_refine_workspace_bytes(op.handle, n, M_COARSE), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    case, n = st["case"], st["n"]
    kind, n_sap, n_mr = case["kind"], case["n_sap"], case["n_mr"]
    if kind == "batch":
        mrhs.sap_smooth_mrhs_batched(st["handles"], st["b"], st["x"], st["ns"], n_sap, n_mr, st["ws"])
        return {"x": st["x"]}
    h = st["op"].handle
    if kind == "sap":
        mrhs.sap_smooth_mrhs(h, st["b"], st["x"], n, n_sap, n_mr, st["ws"])
        return {"x": st["x"]}
    if kind == "dirac":
        mrhs.dirac_apply_mrhs(h, st["b"], st["x"], n)
        return {"x": st["x"]}
    if kind == "setup":
        mrhs.sap_smooth_mrhs(h, st["b"], st["x"], n, n_sap, n_mr, st["ws"])
        mrhs.mrhs_residual_norms(h, st["b"], st["x"], n, st["res"], st["ws"])
        mrhs.block_orthonormalize(h, st["x"], st["op"].dtype, st["Q"], st["qdt"], n, st["status"], st["ws"])
        mrhs.coarse_op_build(h, st["Q"], st["qdt"], n, st["Dc"], st["ws"])
        return {"x": st["x"], "res": st["res"], "Q": st["Q"], "Dc": st["Dc"], "status": st["status"]}
    if kind == "rebuild":
        mrhs.block_orthonormalize(h, st["b"], st["op"].dtype, st["Q"], st["qdt"], n, st["status"], st["ws"])
        mrhs.coarse_op_build_f16(h, st["Q"], st["qdt"], n, st["Dc"])
        return {"Q": st["Q"], "Dc": st["Dc"], "status": st["status"]}
    if kind == "transfer":
        mrhs.restrict_mrhs(h, st["Q"], mrhs.DTYPE_F32, n, st["b"], st["op"].dtype, st["yc"], n)
        mrhs.prolong_mrhs(h, st["Q"], mrhs.DTYPE_F32, n, st["yc"], st["y"], st["op"].dtype, n)
        return {"yc": st["yc"], "y": st["y"]}
    if kind == "solve":
        call = mrhs.coarse_solve_f16_mrhs if st["Dc"].dtype == torch.float16 else mrhs.coarse_solve_mrhs
        call(h, st["Dc"], n, st["bc"], st["uc"], n, M_COARSE, TOL_COARSE, st["ws"], res_out=st["res"])
        return {"u": st["uc"], "res": st["res"]}
    # a refinement pass replaces its vectors: it starts from the same ones every time
    st["V"].copy_(st["b"])
    mrhs.setup_refine_mrhs(h, st["V"], n, st["Q"], mrhs.DTYPE_F32, st["Dc"], n_sap, n_mr, M_COARSE, TOL_COARSE, st["ws"])
    return {"x": st["V"]}


# ---- what a pass cannot do without --------------------------------------------------------------

def sap_flops(case, V, n):
    """Residuals and block solves; hops inside a block only, and of a residual after a block's
    first visit only those across its faces."""
    inside = float(np.mean([(b - 1) / b for b in ints(case["block"])]))
    extra = 504 if case["solver"] == "eo" else 0
    return V * n * case["n_sap"] * (case["n_mr"] * (528 + extra + 1320 * inside + 336) + 1320 * (1 - inside) + 24)


def work(case):
    kind, n = case["kind"], case["n"]
    e = REAL_BYTES[case["prec"]]
    f = 8 if case["prec"] == "f64" else 4
    if kind == "batch":
        parts = [(int(np.prod(L)), m) for L, m in batch_of(case)]
        return {"bytes": sum(V * (144 * f + 48 * e * m) for V, m in parts),
                "flops": sum(sap_flops(case, V, m) for V, m in parts)}
    V = int(np.prod(ints(case["L"])))
    a = ints(case["block"])
    Vc = V // int(np.prod(a))
    vec, fields, dc = 24 * V * n, 144 * V, Vc * 9 * (2 * n) ** 2 * 2
    gs = 96.0 * V * n * n                                    # V^dag V and V R^-1, half of each
    build = 96.0 * V * 2 * n * n * (1 + sum(1.0 / b for b in a)) + V * 2 * n * (252 + 660 + 330 * sum(1.0 / b for b in a))
    apply_f = Vc * 9 * 8.0 * (2 * n) ** 2 * n
    if kind == "sap":
        return {"bytes": fields * f + 2 * vec * e, "flops": sap_flops(case, V, n)}
    if kind == "dirac":
        return {"bytes": fields * f + 2 * vec * e, "flops": 1848.0 * V * n}
    if kind == "setup":
        q = max(e, 4)
        return {"bytes": fields * (f + (8 if f == 4 else 0)) + vec * (2 * e + q) + dc * 4,
                "flops": sap_flops(case, V, n) + 1896.0 * V * n + gs + build}
    if kind == "rebuild":
        return {"bytes": fields * f + vec * (e + 2) + dc * 2, "flops": gs + build}
    if kind == "transfer":
        return {"bytes": vec * 4 * 3 + Vc * 4 * n * n * 4, "flops": 2 * 96.0 * V * n * n}
    cv = Vc * 2 * n * 2 * n * 4
    solve_f = 4 * (apply_f + 4 * 8.0 * Vc * 2 * n * n)      # a few iterations
    if kind == "solve":
        return {"bytes": dc * (2 if case["coarse"] == "f16" else 4) + 2 * cv, "flops": solve_f}
    return {"bytes": fields * f + vec * 4 * 3 + dc * 4, "flops": 2 * 96.0 * V * n * n + solve_f + sap_flops(case, V, n)}


# ---- the same results in 64 bits, in plain torch --------------------------------------------------

PERM = [[3, 2, 1, 0], [3, 2, 1, 0], [2, 3, 0, 1], [2, 3, 0, 1]]
PHASE = [[1j, 1j, -1j, -1j], [-1, 1, 1, -1], [1j, -1j, -1j, 1j], [1, 1, 1, 1]]


def gamma(mu, v):
    """gamma_mu on the spin index of [..., 4, 3]."""
    ph = torch.tensor(PHASE[mu], dtype=torch.complex128, device=v.device)
    return v[..., PERM[mu], :] * ph[:, None]


class Lattice:
    """Sites in native (block-major) order, the operator's fields, and the hops, in 64 bits."""

    def __init__(self, L, block, sigma, m0, seed):
        dev = device()
        self.L, self.b = L, block
        self.nb = [l // b for l, b in zip(L, block)]
        self.V, self.Vb, self.nblk = int(np.prod(L)), int(np.prod(block)), int(np.prod(self.nb))
        lex = lambda ext: np.stack(np.unravel_index(np.arange(int(np.prod(ext))), ext[::-1])[::-1])  # noqa: E731
        bc, lc = lex(self.nb), lex(block)
        x = bc[:, :, None] * np.array(block)[:, None, None] + lc[:, None, :]
        self.x = x.reshape(4, -1)                                   # coordinates of native sites
        stride = np.cumprod([1] + L[:-1])
        self.canon = (self.x * stride[:, None]).sum(0)
        native_of = np.empty(self.V, np.int64)
        native_of[self.canon] = np.arange(self.V)
        t = lambda a: torch.as_tensor(a, device=dev)  # noqa: E731
        self.nbr, self.same = {}, {}
        for mu in range(4):
            for s in (1, -1):
                y = self.x.copy()
                y[mu] = (y[mu] + s) % L[mu]
                self.nbr[mu, s] = t(native_of[(y * stride[:, None]).sum(0)])
                l = self.x[mu] % block[mu] + s
                # hops that cross no block face; a block spanning the direction has none
                self.same[mu, s] = t(((l >= 0) & (l < block[mu])))
        self.colour = t(bc.sum(0) % 2)
        self.odd = t((lc.sum(0) % 2).astype(bool)).repeat(self.nblk)
        self.U = links(L, sigma, seed)[:, t(self.canon)]
        self.A = self.clover(m0)

    def clover(self, m0):
        dev, U = device(), self.U
        dag = lambda m: m.conj().transpose(-1, -2)  # noqa: E731
        at = lambda idx, mu, s: idx[self.nbr[mu, s]]  # noqa: E731
        here = torch.arange(self.V, device=dev)

        def path(steps):
            # product of the links along steps (mu, +-1) from every site
            site, P = here, None
            for mu, s in steps:
                if s > 0:
                    m = U[mu][site]
                    site = self.nbr[mu, 1][site]
                else:
                    site = self.nbr[mu, -1][site]
                    m = dag(U[mu][site])
                P = m if P is None else mul3(P, m)
            return P

        g = torch.zeros((4, 4, 4), dtype=torch.complex128)
        for mu in range(4):
            g[mu, range(4), PERM[mu]] = torch.tensor(PHASE[mu], dtype=torch.complex128)
        A = torch.zeros((self.V, 4, 3, 4, 3), dtype=torch.complex128, device=dev)
        for mu in range(4):
            for nu in range(mu + 1, 4):
                Q = sum(path(p) for p in ([(mu, 1), (nu, 1), (mu, -1), (nu, -1)], [(nu, 1), (mu, -1), (nu, -1), (mu, 1)],
                                          [(mu, -1), (nu, -1), (mu, 1), (nu, 1)], [(nu, -1), (mu, 1), (nu, 1), (mu, -1)]))
                F = (-CSW / 16.0) * (Q - dag(Q))
                sig = g[mu] @ g[nu]
                for r in range(4):
                    for c in range(4):
                        if abs(complex(sig[r, c])) > 0:
                            A[:, r, :, c, :] += complex(sig[r, c]) * F
        A = A.reshape(self.V, 12, 12)
        A += (4.0 + m0) * torch.eye(12, dtype=torch.complex128, device=dev)
        return A

    def hop(self, v, mu, s, mask=None):
        """-1/2 (1 - s gamma_mu) U v of the neighbour in direction s mu, v [n][V][4][3]."""
        idx = self.nbr[mu, s]
        chi = v[:, idx]
        W = self.U[mu] if s > 0 else self.U[mu][idx].conj().transpose(-1, -2)
        if mask is not None:
            W = W * mask[:, None, None]
        w = sum(W[None, :, None, :, c] * chi[:, :, :, c, None] for c in range(3))
        return -0.5 * (w - s * gamma(mu, w))

    def hops(self, v, mask=None):
        return sum(self.hop(v, mu, s, None if mask is None else mask[mu, s]) for mu in range(4) for s in (1, -1))

    def site(self, M, v):
        n = v.shape[0]
        w = v.reshape(n, self.V, 12)
        return sum(M[None, :, :, c] * w[:, :, c, None] for c in range(12)).reshape(v.shape)

    def dirac(self, v):
        return self.site(self.A, v) + self.hops(v)

    def block_sum(self, v):
        """Sums over a block's sites and components, spread back to the sites, [n][V][1][1]."""
        n = v.shape[0]
        s = v.reshape(n, self.nblk, -1).sum(-1)
        return s[:, :, None].expand(n, self.nblk, self.Vb).reshape(n, self.V, 1, 1)

    def sap(self, b, n_sap, n_mr, eo, x=None):
        # a block that spans a direction keeps its wrap-around hop
        mask = {k: self.same[k] | (self.nb[k[0]] == 1) for k in self.same}
        x = torch.zeros_like(b) if x is None else x
        of = [(self.colour == c)[:, None].expand(self.nblk, self.Vb).reshape(1, self.V, 1, 1) for c in (0, 1)]
        odd = self.odd[None, :, None, None]
        Ainv = torch.linalg.inv(self.A) if eo else None

        def step(apply, r, e):
            q = apply(r)
            qq, qr = self.block_sum(q.abs() ** 2), self.block_sum(q.conj() * r)
            al = torch.where(qq > 0, qr / torch.where(qq > 0, qq, 1.0), 0.0)
            return r - al * q, e + al * r

        for _ in range(n_sap):
            for c in (0, 1):
                r = (b - self.dirac(x)) * of[c]
                e = torch.zeros_like(r)
                if eo:
                    S = lambda v: (self.site(self.A, v) - self.hops(  # noqa: E731
                        self.site(Ainv, self.hops(v, mask) * odd), mask)) * ~odd
                    ro = r * odd
                    re = r * ~odd - self.hops(self.site(Ainv, ro), mask) * ~odd
                    for _ in range(n_mr):
                        re, e = step(S, re, e)
                    e = e + self.site(Ainv, ro - self.hops(e, mask) * odd) * odd
                else:
                    for _ in range(n_mr):
                        r, e = step(lambda v: self.site(self.A, v) + self.hops(v, mask), r, e)
                x = x + e
        return x

    # vectors: canonical -> [n][V][4][3] in native order -> native layout
    def native(self, v, dtype):
        n = v.shape[0]
        v = v[:, torch.as_tensor(self.canon, device=v.device)]
        return torch.complex(stored(v.real, dtype), stored(v.imag, dtype)) if dtype else v.reshape(n, self.V, 4, 3)

    def layout(self, v):
        n = v.shape[0]
        r = torch.view_as_real(v.reshape(n, self.nblk, self.Vb, 12).contiguous()).reshape(n, self.nblk, self.Vb, 24)
        pad = -n % S
        r = torch.cat([r, torch.zeros((pad,) + r.shape[1:], dtype=r.dtype, device=r.device)]) if pad else r
        return r.reshape(-1, S, self.nblk, self.Vb, 24).permute(0, 2, 4, 3, 1).reshape(-1)

    # aggregates are the blocks: [n][V][4][3] -> [Vc][2][6 Va][n]
    def halves(self, v):
        n = v.shape[0]
        return v.reshape(n, self.nblk, self.Vb, 2, 6).permute(1, 3, 2, 4, 0).reshape(self.nblk, 2, 6 * self.Vb, n)

    def whole(self, h):
        n = h.shape[-1]
        return h.reshape(self.nblk, 2, self.Vb, 6, n).permute(4, 0, 2, 1, 3).reshape(n, self.V, 4, 3)

    def orthonormal(self, v):
        """Gram-Schmidt per aggregate half, every column orthogonalised twice."""
        X = self.halves(v).clone()
        for k in range(X.shape[-1]):
            c = X[..., k:k + 1].contiguous()
            for _ in range(2 if k else 0):
                P = X[..., :k].contiguous()
                c = c - P @ (P.conj().transpose(-1, -2).contiguous() @ c)
            X[..., k:k + 1] = c / (c.abs() ** 2).sum(-2, keepdim=True).sqrt()
        return self.whole(X)

    def coarse(self, Q):
        """The 9 blocks of D_c, [Vc][9][2N][2N]: row and column dof h N + k."""
        n = Q.shape[0]
        Qd = self.halves(Q).conj().transpose(-1, -2).contiguous()    # [Vc][2][n][6Va]
        out = torch.empty((self.nblk, 9, 2 * n, 2 * n), dtype=torch.complex128, device=Q.device)
        order = [(mu, 1) for mu in range(4)] + [(mu, -1) for mu in range(4)]
        for hp in range(2):
            P = Q.clone()
            P[:, :, 2 * (1 - hp):2 * (1 - hp) + 2] = 0
            for d in range(9):
                w = self.site(self.A, P) + self.hops(P, self.same) if d == 0 else \
                    self.hop(P, *order[d - 1], ~self.same[order[d - 1]])
                out[:, d, :, hp * n:(hp + 1) * n] = (Qd @ self.halves(w)).reshape(self.nblk, 2 * n, n)
        return out


def stored(v, dtype):
    """Values as a storage type holds them, in 64 bits."""
    return v.to({"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[dtype]).double()


def coarse_layout(yc):
    """[Vc][2N][n] complex -> [Vc][2N][2][ldc]."""
    n = yc.shape[-1]
    r = torch.stack([yc.real, yc.imag], 2)
    return torch.nn.functional.pad(r, (0, -n % 4))


def coarse_apply(na, D, y):
    """D [Vc][9][2N][2N], y [Vc][2N][n] (complex128)."""
    idx = np.arange(len(y)).reshape(na[::-1])
    out = D[:, 0].contiguous() @ y
    for d in range(1, 9):
        mu, s = (d - 1) % 4, 1 if d <= 4 else -1
        j = torch.as_tensor(np.roll(idx, -s, axis=3 - mu).reshape(-1).copy(), device=y.device)
        out = out + D[:, d].contiguous() @ y[j]
    return out


def gmres(na, D, b):
    """GMRES from zero per right-hand side to TOL_COARSE or M_COARSE iterations: u and the relative residuals."""
    Vc, N2, n = b.shape
    dot = lambda x, y: (x.conj() * y).sum((0, 1))  # noqa: E731
    beta = dot(b, b).real.sqrt()
    basis, H = [b / beta], torch.zeros((n, M_COARSE + 1, M_COARSE), dtype=torch.complex128, device=b.device)
    u, res, done = torch.zeros_like(b), torch.ones_like(beta), torch.zeros(n, dtype=torch.bool, device=b.device)
    for j in range(M_COARSE):
        w = coarse_apply(na, D, basis[j])
        for _ in range(2):
            hs = [dot(v, w) for v in basis]
            for i, (h, v) in enumerate(zip(hs, basis)):
                H[:, i, j] += h
                w = w - h * v
        H[:, j + 1, j] = dot(w, w).real.sqrt()
        basis.append(w / H[:, j + 1, j])
        rhs = torch.zeros((n, j + 2, 1), dtype=torch.complex128, device=b.device)
        rhs[:, 0, 0] = beta
        Hj = H[:, :j + 2, :j + 1]
        Hd = Hj.conj().transpose(-1, -2).contiguous()
        y = torch.linalg.solve(Hd @ Hj.contiguous(), Hd @ rhs)
        r = (rhs - Hj.contiguous() @ y).abs().square().sum((1, 2)).sqrt() / beta
        uj = sum(y[:, i, 0] * basis[i] for i in range(j + 1))
        u, res = torch.where(done, u, uj), torch.where(done, res, r)
        done = done | (r <= TOL_COARSE)
    return u, res


def exact(case, seed):
    kind, n, prec = case["kind"], case["n"], case["prec"]
    L, block = ints(case["L"]), ints(case["block"])
    if kind == "batch":
        if sum(int(np.prod(l)) * m for l, m in batch_of(case)) > EXACT_MOST:
            return None
        xs = []
        for k, (l, m) in enumerate(batch_of(case)):
            lat = Lattice(l, block, case["sigma"], case["m0"], seed + 50 * k)
            b = lat.native(vectors(l, m, seed + 50 * k), prec)
            xs.append(lat.layout(lat.sap(b, case["n_sap"], case["n_mr"], False)))
        return {"x": xs}
    V = int(np.prod(L))
    Vc, na = V // int(np.prod(block)), [l // b for l, b in zip(L, block)]
    comp = lambda r: torch.complex(r[..., 0, :n].double(), r[..., 1, :n].double()).contiguous()  # noqa: E731
    blocks = lambda D: torch.complex(D[..., 0].double(), D[..., 1].double())  # noqa: E731
    if kind == "solve":
        D = coarse_blocks(Vc, n, seed)
        u, res = gmres(na, blocks(D.half() if case["coarse"] == "f16" else D), comp(coarse_vectors(Vc, n, n, seed)))
        return {"u": coarse_layout(u), "res": res}
    if V * n > EXACT_MOST * (2 if kind in ("transfer", "dirac") else 1):
        return None
    make = vectors if kind in ("setup", "sap", "dirac") else smoothed
    lat = Lattice(L, block, case["sigma"], case["m0"], seed)
    b = lat.native(make(L, n, seed), prec)
    if kind == "dirac":
        return {"x": lat.layout(lat.dirac(b))}
    if kind == "sap":
        return {"x": lat.layout(lat.sap(b, case["n_sap"], case["n_mr"], case["solver"] == "eo"))}
    real = lambda D: torch.view_as_real(D).reshape(-1)  # noqa: E731
    if kind == "rebuild":
        Q = lat.orthonormal(b)
        return {"Q": lat.layout(Q), "Dc": real(lat.coarse(Q)), "status": None}
    if kind == "setup":
        x = lat.sap(b, case["n_sap"], case["n_mr"], False)
        r = b - lat.dirac(x)
        norm = lambda v: (v.abs() ** 2).reshape(n, -1).sum(-1).sqrt()  # noqa: E731
        Q = lat.orthonormal(x)
        return {"x": lat.layout(x), "res": norm(r) / norm(b), "Q": lat.layout(Q), "Dc": real(lat.coarse(Q)), "status": None}
    scale = (6.0 * np.prod(block)) ** -0.5
    Q = lat.halves(lat.native(scale * 0.5 ** 0.5 * vectors(L, n, seed + 1), "f32")).contiguous()
    yc = (Q.conj().transpose(-1, -2).contiguous() @ lat.halves(b).contiguous()).reshape(Vc, 2 * n, n)
    up = lambda c: lat.whole(Q @ c.reshape(Vc, 2, n, n))  # noqa: E731
    if kind == "transfer":
        return {"yc": coarse_layout(yc).reshape(-1), "y": lat.layout(up(yc))}
    u, _ = gmres(na, blocks(coarse_blocks(Vc, n, seed)), yc)
    return {"x": lat.layout(lat.sap(b, case["n_sap"], case["n_mr"], False, up(u)))}
