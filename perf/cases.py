"""The performance cases of the framework: what its users have it do, over the
range of sizes they have it done at.

A case names a kind of work and its sizes; prepare() makes the inputs on the
GPU from the seed alone (finite element matrices of jittered meshes, element
data, right-hand sides) and builds the handles a program keeps; run() is one
pass through the public entry points.

The matrices are those of the benchmark workloads: P1 triangles and Kuhn
tetrahedra and Q1 hexahedra, Laplacian (one unknown per node) or linear
elasticity (three), in the mesh generator's numbering or with the nodes in
random order, with the Dirichlet nodes of the whole boundary or of the face
x = 0 removed, or none.  A solve with `mass` > 0 is one implicit time step:
the stiffness matrix plus mass times its diagonal.
"""
import itertools
import math

import numpy as np
import torch

import paper_1501_00324_amd as fe

DEV = "cuda"


# ------------------------------------------------------------------- meshes
def _element(name):
    """Sub-elements of a grid cell (local node offsets), shape gradients at
    the quadrature points and their weights."""
    if name == "tri":
        subs = [[(0, 0), (1, 0), (1, 1)], [(0, 0), (1, 1), (0, 1)]]
    elif name == "tet":
        subs = []
        for s in itertools.permutations(range(3)):
            t = [np.zeros(3, int)]
            for ax in s:
                t.append(t[-1] + np.eye(3, dtype=int)[ax])
            if np.linalg.det(np.array(t[1:]) - t[0]) < 0:
                t[1], t[2] = t[2], t[1]
            subs.append([tuple(int(v) for v in p) for p in t])
    else:
        nodes = list(itertools.product((0, 1), repeat=3))
        g = 0.5 / math.sqrt(3.0)
        grads = []
        for q in itertools.product((0.5 - g, 0.5 + g), repeat=3):
            row = []
            for nd in nodes:
                f = [q[k] if nd[k] else 1 - q[k] for k in range(3)]
                s = [1.0 if nd[k] else -1.0 for k in range(3)]
                row.append([s[0] * f[1] * f[2], f[0] * s[1] * f[2], f[0] * f[1] * s[2]])
            grads.append(row)
        return [nodes], np.array(grads), np.full(8, 0.125)
    d = len(subs[0][0])
    grads = np.concatenate([-np.ones((1, d)), np.eye(d)])[None]
    return subs, grads, np.array([1.0 / math.factorial(d)])


def _shape(case):
    """Nodes per direction, and the first and end kept index per direction."""
    d = 2 if case["element"] == "tri" else 3
    n = [case["n"] + (case.get("odd", 0) if k == 0 else 0) for k in range(d)]
    bc = case["bc"]
    lo = [1 if bc == "all" or (bc == "x0" and k == 0) else 0 for k in range(d)]
    hi = [v - 1 if bc == "all" else v for v in n]
    return n, lo, hi


def _offsets(case):
    """Neighbour offsets of the mesh graph, in the order of node numbers."""
    subs = _element(case["element"])[0]
    return sorted({tuple(b[k] - a[k] for k in range(len(a))) for t in subs for a in t for b in t})


def _dof(case):
    return 3 if case["physics"] == "elastic" else 1


def _counts(case):
    """Rows and non-zeros of the case's matrix."""
    _, lo, hi = _shape(case)
    m = [h - l for l, h in zip(lo, hi)]
    pairs = sum(math.prod(max(0, m[k] - abs(o[k])) for k in range(len(m))) for o in _offsets(case))
    return math.prod(m) * _dof(case), pairs * _dof(case) ** 2


class Mesh:
    """Geometry and element matrices of a case, on the GPU."""

    def __init__(self, case, gen):
        self.case = case
        self.n, self.lo, self.hi = _shape(case)
        self.d, self.dof = len(self.n), _dof(case)
        axes = [torch.arange(v, dtype=torch.float64, device=DEV) / (v - 1) for v in self.n]
        X = torch.stack(torch.meshgrid(*axes, indexing="ij"), -1)
        move = torch.rand(X.shape, generator=gen, dtype=torch.float64, device=DEV) * 0.4 - 0.2
        inner = (slice(1, -1),) * self.d
        X[inner] += move[inner] / (torch.tensor(self.n, device=DEV) - 1)
        self.subs, grads, self.w = _element(case["element"])
        self.grads = torch.tensor(grads, device=DEV)
        self.X = X
        # number of every node among the kept ones, -1 where it is removed
        kept = [h - l for l, h in zip(self.lo, self.hi)]
        count = math.prod(kept)
        num = torch.full(self.n, -1, dtype=torch.int64, device=DEV)
        order = torch.randperm(count, generator=gen, device=DEV) if case["numbering"] == "random" else torch.arange(count, device=DEV)
        num[tuple(slice(l, h) for l, h in zip(self.lo, self.hi))] = order.reshape(kept)
        self.num, self.count = num, count

    def at(self, field, o):
        """The node field at local node o of every cell."""
        return field[tuple(slice(o[k], self.n[k] - 1 + o[k]) for k in range(self.d))]

    def gradients(self, t):
        """Physical shape gradients (quadrature, cells, node, d) and weights of sub-element t."""
        x = torch.stack([self.at(self.X, o).reshape(-1, self.d) for o in t], 1)
        J = torch.einsum("qai,caj->qcij", self.grads, x)
        if self.d == 2:
            det = J[..., 0, 0] * J[..., 1, 1] - J[..., 0, 1] * J[..., 1, 0]
            adj = torch.stack([torch.stack([J[..., 1, 1], -J[..., 0, 1]], -1), torch.stack([-J[..., 1, 0], J[..., 0, 0]], -1)], -2)
        else:
            r = [J[..., k, :] for k in range(3)]
            adj = torch.stack([torch.linalg.cross(r[(k + 1) % 3], r[(k + 2) % 3]) for k in range(3)], -1)
            det = (r[0] * adj[..., 0]).sum(-1)
        G = torch.einsum("qcji,qai->qcaj", adj / det[..., None, None], self.grads)
        return G, det * torch.tensor(self.w, device=DEV)[:, None]

    def block(self, G, w, a, b):
        """Element stiffness between local nodes a and b: (cells, dof, dof)."""
        ga, gb = G[:, :, a], G[:, :, b]
        gg = ((ga * gb).sum(-1) * w).sum(0)
        if self.dof == 1:
            return gg[:, None, None]
        lam, mu = 0.3 / (1.3 * 0.4), 1.0 / 2.6          # E = 1, nu = 0.3
        ab = (ga[..., :, None] * gb[..., None, :] * w[..., None, None]).sum(0)
        return lam * ab + mu * ab.transpose(1, 2) + mu * gg[:, None, None] * torch.eye(3, dtype=torch.float64, device=DEV)

    def csr(self):
        """rowptr, col, val of the assembled matrix (columns ascending)."""
        offs = _offsets(self.case)
        S = torch.zeros([len(offs)] + self.n + [self.dof, self.dof], dtype=torch.float64, device=DEV)
        for t in self.subs:
            G, w = self.gradients(t)
            for a, b in itertools.product(range(len(t)), repeat=2):
                o = offs.index(tuple(t[b][k] - t[a][k] for k in range(self.d)))
                part = self.at(S[o], t[a])
                part += self.block(G, w, a, b).reshape(part.shape)
        nbr = torch.full([len(offs)] + self.n, -1, dtype=torch.int64, device=DEV)
        for k, o in enumerate(offs):
            here = tuple(slice(max(0, -v), n - max(0, v)) for v, n in zip(o, self.n))
            there = tuple(slice(max(0, v), n - max(0, -v)) for v, n in zip(o, self.n))
            nbr[k][here] = self.num[there]
        keep = self.num.reshape(-1) >= 0
        row = torch.empty(self.count, dtype=torch.int64, device=DEV)
        row[self.num.reshape(-1)[keep]] = keep.nonzero()[:, 0]
        nbr = nbr.reshape(len(offs), -1)[:, row].T.contiguous()           # (node, offset)
        S = S.reshape(len(offs), -1, self.dof, self.dof)[:, row].permute(1, 0, 2, 3)
        if self.case["numbering"] == "random":
            nbr, by = torch.sort(nbr, 1)
            S = torch.gather(S, 1, by[:, :, None, None].expand(-1, -1, self.dof, self.dof))
        S = S.permute(0, 2, 1, 3)                                         # (node, c, offset, c2)
        there = (nbr >= 0)[:, None, :, None].expand(S.shape)
        comp = torch.arange(self.dof, device=DEV)
        col = (nbr[:, None, :, None] * self.dof + comp).expand(S.shape)[there].to(torch.int32)
        val = S[there]
        rowptr = torch.zeros(self.count * self.dof + 1, dtype=torch.int32, device=DEV)
        rowptr[1:] = (nbr >= 0).sum(1).mul(self.dof).repeat_interleave(self.dof).cumsum(0)
        mass = self.case.get("mass", 0.0)
        if mass:
            r = torch.repeat_interleave(torch.arange(len(rowptr) - 1, device=DEV), rowptr.diff())
            val = torch.where(col == r, val * (1.0 + mass), val)
        return rowptr, col, val

    def elements(self, gen):
        """Element map, matrices and load vectors, cell by cell."""
        edof, ke, re = [], [], []
        comp = torch.arange(self.dof, device=DEV)
        for t in self.subs:
            nodes = torch.stack([self.at(self.num, o).reshape(-1) for o in t], 1)
            e = nodes[:, :, None] * self.dof + comp
            edof.append(torch.where(nodes[:, :, None] >= 0, e, -1).reshape(len(nodes), -1))
            G, w = self.gradients(t)
            k = torch.empty(len(nodes), len(t), self.dof, len(t), self.dof, dtype=torch.float64, device=DEV)
            for a, b in itertools.product(range(len(t)), repeat=2):
                k[:, a, :, b, :] = self.block(G, w, a, b)
            ke.append(k.reshape(len(nodes), len(t) * self.dof, -1))
            load = torch.rand(len(nodes), 1, generator=gen, dtype=torch.float64, device=DEV) * w.sum(0)[:, None] / len(t)
            re.append(load.expand(-1, len(t) * self.dof))
        nde = edof[0].shape[1]
        return (torch.stack(edof, 1).reshape(-1, nde).to(torch.int32).contiguous(),
                torch.stack(ke, 1).reshape(-1, nde, nde).contiguous(), torch.stack(re, 1).reshape(-1, nde).contiguous())


# -------------------------------------------------------------------- cases
def listed():
    return [
        # the product inside a solver on a mesh of ten thousand nodes: latency
        dict(name="product small", kind="product", element="tet", n=22, physics="laplace", numbering="natural", bc="none"),
        # the product on the largest matrix of the sweep, the headline
        dict(name="product large", kind="product", element="hex", n=87, physics="elastic", numbering="natural", bc="none"),
        # a single product in the caller's numbering, one unknown per node, a
        # mesh generator's arbitrary node order, odd sizes
        dict(name="product caller", kind="caller", element="tet", n=101, odd=2, physics="laplace", numbering="random", bc="none"),
        # sixteen right-hand sides at once on the elasticity system
        dict(name="product 16 columns", kind="columns", k=16, element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # the low-precision product inside mixed-precision refinement
        dict(name="product bf16", kind="lowp", dtype="bf16", element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # a Newton step that has new values in CSR order: value refresh (FP64
        # and the FP32 copy), then the residual's product
        dict(name="newton refresh", kind="refresh", dtype="f32", element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # a Newton step from element data: assembly of matrix and load, then
        # the residual's product
        dict(name="newton assembly", kind="assembly", element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # one solve on a small plane mesh: latency of the iteration
        dict(name="solve small", kind="solve", precision="f64", k=1, mass=0.2, element="tri", n=64, physics="laplace", numbering="natural", bc="all"),
        # one implicit step of the large elasticity system
        dict(name="solve large", kind="solve", precision="f64", k=1, mass=0.2, element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # the same in mixed precision
        dict(name="solve refined", kind="solve", precision="f32", k=1, mass=0.2, element="tet", n=64, physics="elastic", numbering="random", bc="x0"),
        # eight load cases of one system at once (a served request)
        dict(name="solve 8 columns", kind="solve", precision="f64", k=8, mass=0.2, element="tet", n=41, physics="elastic", numbering="random", bc="x0"),
        # many small systems, one per patient or material point
        dict(name="solve 64 systems", kind="systems", m=64, mass=0.2, element="tri", n=48, physics="laplace", numbering="natural", bc="all"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product", "product", "caller", "columns", "lowp", "refresh", "assembly", "solve", "solve", "systems"])
    c = dict(kind=kind, physics=rng.choice(["laplace", "elastic"]), element=rng.choice(["tet", "tet", "hex"]),
             numbering=rng.choice(["natural", "random"]), bc=rng.choice(["none", "x0"]), odd=rng.randrange(4))
    most = 60 if c["physics"] == "elastic" else 110
    if kind == "columns":
        c["k"], most = rng.randrange(2, 17), most * 3 // 4
    elif kind in ("lowp", "refresh"):
        c["dtype"] = rng.choice(["f32", "bf16"])
    elif kind == "assembly":
        most = 40 if c["physics"] == "elastic" else 70
    elif kind == "solve":
        k = rng.choice([1, 1, 1, rng.randrange(2, 17)])
        c.update(precision=rng.choice(["f64", "f64", "f32"]) if k == 1 else "f64", k=k, mass=0.2, bc="x0")
        most = 50 if c["physics"] == "elastic" else 70
        if k > 1:
            most = most * 3 // 4
    elif kind == "systems":
        return dict(kind=kind, physics="laplace", element="tri", numbering=c["numbering"], bc="all", odd=c["odd"],
                    m=_log(rng, 8, 128), mass=0.2, n=_log(rng, 16, 56))
    c["n"] = _log(rng, 10, most)
    return c


# ---------------------------------------------------------------- the passes
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, dtype=torch.float64, device=DEV) * 2 - 1


def _lowp(case):
    return fe.DT_BF16 if case["dtype"] == "bf16" else fe.DT_F32


def _inputs(case, seed):
    """What both the framework's pass and the plain one start from."""
    gen = _gen(seed)
    if case["kind"] == "systems":
        mats = [Mesh(case, gen).csr() for _ in range(case["m"])]
        return mats, [_uniform(gen, len(m[0]) - 1) for m in mats]
    mesh = Mesh(case, gen)
    csr = mesh.csr()
    n = len(csr[0]) - 1
    if case["kind"] == "assembly":
        return csr, _uniform(gen, n), mesh.elements(gen)
    if case["kind"] in ("columns", "solve"):
        return csr, _uniform(gen, n, case["k"]) if case["k"] > 1 else _uniform(gen, n)
    if case["kind"] == "refresh":
        return csr, _uniform(gen, n), csr[2] * (1.0 + 0.1 * _uniform(gen, len(csr[2])))
    return csr, _uniform(gen, n)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "systems":
        mats, b = _inputs(case, seed)
        return dict(case=case, A=[fe.csr_create(*m) for m in mats], b=b, x=[torch.empty_like(v) for v in b])
    csr, x, *more = _inputs(case, seed)
    A = fe.csr_create(*csr)
    s = dict(case=case, A=A, x=x)
    if kind in ("lowp", "refresh"):
        fe.csr_add_dtype(A, _lowp(case))
    if kind in ("product", "lowp", "refresh", "assembly"):
        s["x"] = fe.csr_permute(A, fe.TO_LAYOUT, x)
    if kind == "lowp":
        s["x"] = s["x"].float()
    if kind == "refresh":
        s["val"] = more[0]
    if kind == "assembly":
        edof, s["ke"], s["re"] = more[0]
        s["plan"] = fe.asm_create(A, edof)
        s["r"] = torch.empty_like(x)
    if kind == "solve" and case["precision"] == "f32":
        fe.csr_add_dtype(A, fe.DT_F32)
    s["y"] = torch.empty_like(s["x"])
    return s


def run(s):
    case, A = s["case"], s["A"]
    kind = case["kind"]
    if kind == "product":
        return fe.spmv_perm(A, s["x"], s["y"])
    if kind == "caller":
        return fe.spmv(A, s["x"], s["y"])
    if kind == "columns":
        return fe.spmm(A, s["x"], s["y"])
    if kind == "lowp":
        return fe.spmv_lowp(A, _lowp(case), s["x"], s["y"])
    if kind == "refresh":
        fe.csr_update_values(A, s["val"])
        return fe.spmv_perm(A, s["x"], s["y"])
    if kind == "assembly":
        fe.asm_system(s["plan"], s["ke"], s["re"], s["r"])
        return fe.spmv_perm(A, s["x"], s["y"]), s["r"]
    if kind == "systems":
        return torch.cat(fe.cg_solve_batch_wg(A, s["b"], s["x"], x0_zero=1)[0])
    if case["k"] > 1:
        return fe.cg_solve_multi(A, s["x"], s["y"], x0_zero=1)[0]
    precision = fe.PREC_IR_F32 if case["precision"] == "f32" else fe.PREC_F64
    return fe.cg_solve(A, s["x"], s["y"], x0_zero=1, precision=precision)[0]


# ------------------------------------------------------------- what it needs
#: Iterations a solve with mass = 0.2 takes to 1e-8, to within a few.
ITERATIONS = 35


def work(case):
    """Each matrix value once per product with the column of each pair of
    nodes, each vector once; a solve its iterations' products and vectors."""
    n, nnz = _counts(case)
    kind, index = case["kind"], 4 * nnz // _dof(case) ** 2
    if kind == "columns":
        return dict(bytes=8 * nnz + index + 16 * n * case["k"], flops=2 * nnz * case["k"])
    if kind == "lowp":
        return dict(bytes=(2 if case["dtype"] == "bf16" else 4) * nnz + index + 8 * n, flops=2 * nnz)
    product = 8 * nnz + index + 16 * n
    if kind == "refresh":
        return dict(bytes=(16 + (2 if case["dtype"] == "bf16" else 4)) * nnz + product, flops=2 * nnz)
    if kind == "assembly":
        cells = math.prod(v - 1 for v in _shape(case)[0])
        subs = _element(case["element"])[0]
        nde = len(subs[0]) * _dof(case)
        entries = cells * len(subs) * nde * nde
        return dict(bytes=8 * entries + 8 * nnz + cells * len(subs) * nde * 12 + 8 * n + product, flops=entries + 2 * nnz)
    if kind in ("solve", "systems"):
        k, m = case.get("k", 1), case.get("m", 1)
        v = 4 if case.get("precision") == "f32" else 8
        step = v * nnz + index + 11 * v * n * k
        return dict(bytes=ITERATIONS * m * step, flops=ITERATIONS * m * k * (2 * nnz + 13 * n))
    return dict(bytes=product, flops=2 * nnz)


# -------------------------------------------------------- the same in 64 bits
def _product(csr, x):
    rowptr, col, val = csr
    r = torch.repeat_interleave(torch.arange(len(rowptr) - 1, device=DEV), rowptr.diff())
    terms = val * x[col.long()] if x.dim() == 1 else val[:, None] * x[col.long()]
    return torch.zeros(len(rowptr) - 1, *x.shape[1:], dtype=torch.float64, device=DEV).index_add_(0, r, terms)


def _pcg(csr, b):
    """Textbook conjugate gradients with Jacobi scaling to |r| <= 1e-8 |b|, columns apart."""
    rowptr, col, val = csr
    A = torch.sparse_csr_tensor(rowptr.long(), col.long(), val, size=(len(b), len(b)))
    r = torch.repeat_interleave(torch.arange(len(b), device=DEV), rowptr.diff())
    D = torch.zeros_like(b).index_add_(0, r, torch.where(col == r, val, 0.0))
    x, res = torch.zeros_like(b), b.clone()
    z = res / D
    p, rho, stop = z.clone(), torch.dot(res, z), 1e-16 * float(torch.dot(b, b))
    for _ in range(2000):
        q = A @ p
        alpha = rho / torch.dot(p, q)
        x += alpha * p
        res -= alpha * q
        if float(torch.dot(res, res)) <= stop:
            break
        z = res / D
        rho, old = torch.dot(res, z), rho
        p = z + (rho / old) * p
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "systems":
        mats, b = _inputs(case, seed)
        return torch.cat([_pcg(m, v) for m, v in zip(mats, b)])
    csr, x, *more = _inputs(case, seed)
    if kind == "solve":
        if case["precision"] == "f32":
            return None     # refinement steps end where their own rounding puts them
        return torch.stack([_pcg(csr, x[:, c].contiguous()) for c in range(case["k"])], 1) if case["k"] > 1 else _pcg(csr, x)
    if kind in ("caller", "columns"):
        if kind == "columns":
            return torch.stack([_product(csr, x[:, c].contiguous()) for c in range(case["k"])], 1)
        return _product(csr, x)
    # layout numbering: rows in the order of the handle's permutation
    A = fe.csr_create(*csr)
    perm = torch.tensor(fe.csr_get_perm(A), device=DEV).long()
    A.close()
    if kind == "product":
        return _product(csr, x)[perm]
    if kind == "lowp":
        # the stored values and vector are rounded; the sum is not
        v = csr[2].float().bfloat16().double() if case["dtype"] == "bf16" else csr[2].float().double()
        return _product((csr[0], csr[1], v), x.float().double())[perm]
    if kind == "refresh":
        return _product((csr[0], csr[1], more[0]), x)[perm]
    edof, ke, re = more[0]
    # K x element by element
    d = edof.long()
    xe = torch.where(d >= 0, x[d.clamp(min=0)], 0.0)
    kept = d.reshape(-1) >= 0
    out = []
    for v in ((ke * xe[:, None, :]).sum(-1), re):
        out.append(torch.zeros_like(x).index_add_(0, d.reshape(-1)[kept], v.reshape(-1)[kept]))
    return out[0][perm], out[1]
