"""Workloads of symmetric CTM on one GPU, each through the package's public calls.

The sizes are those of the paper's square-lattice runs as this repository
configures them: bond dimension D = 4..8 on the charges {-2, 0, 2} (U(1)), on
parities (Z2) or on multiplets (SU(2)), chi = 16..200 over binomially weighted
charge sectors, a spin-1/2 physical leg.  Values are standard normals, the site
tensor `a` the double layer of a normal site tensor.

  contract   one contraction step of a corner (C T, or X a over two legs)
  corner     one enlarged corner C T T a
  batch      many independent corners of mixed sizes in grouped launches
  move       one CTM move toward a side (corners, halves, FP64 projectors with
             truncation, renormalisation) and the column it leaves
  step       one CTM step: a move toward each side, then the partition
             function per site, as an iteration does it
  su2        one move of an SU(2) environment
  double     the double layer of a site tensor

A moved environment is fixed up to a rotation of its new bonds, which rounding
turns where singular values are close; so a move returns the column
C1' T4' C4' (over both new bonds), the cut's spectrum and, in FP64, the updated
tensors themselves.  Which sectors the truncation keeps depends on the values,
and with them the sizes of these buffers: each comes at the front of an array
of the size that it could at most have.
"""
import itertools
import math

import numpy as np
import torch

import paper_1808_10804_amd as st

IN, OUT = 1, -1
VIRT_U1 = {4: (1, 2, 1), 5: (1, 3, 1), 6: (1, 4, 1), 7: (2, 3, 2), 8: (2, 4, 2)}
# doubled spin: multiplets (virtual leg of total dimension 10, chi = 100)
VIRT_SU2 = {0: 1, 1: 3, 2: 1}
CHI_SU2 = {0: 11, 1: 13, 2: 13, 3: 6}
DOUBLE_SU2 = {0: 11, 1: 12, 2: 12, 3: 6, 4: 1}      # the double layer's legs


# ------------------------------------------------------------------- sizes --
def _virt(group, D):
    if group == "z2":
        return {0: D - D // 2, 1: D // 2}
    return dict(zip((-2, 0, 2), VIRT_U1[D]))


def _chi(group, chi):
    """chi states over the charge sectors: binomial weights, largest remainder."""
    if group == "z2":
        return {0: chi - chi // 2, 1: chi // 2}
    n = 2 if chi < 32 else 4 if chi < 100 else 6
    raw = [chi * math.comb(n, k) / 2 ** n for k in range(n + 1)]
    base = [int(x) for x in raw]
    order = sorted(range(n + 1), key=lambda k: (base[k] - raw[k], abs(k - n // 2), k))
    for k in order[:chi - sum(base)]:
        base[k] += 1
    return {2 * (k - n // 2): d for k, d in enumerate(base) if d > 0}


def _batch_sizes(count, layout):
    """(D, chi) of the corners of a batch: D of 4..8, chi of 32..160."""
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([layout, 999])))
    return [(int(rng.choice((4, 5, 6, 7, 8))), int(rng.integers(32, 161))) for _ in range(count)]


def _fused(sectors, mod):
    """Double-layer leg of `sectors`: its sectors, and per fused state the ket
    and bra states (ordered by q_ket - q_bra, q_ket, i_ket, i_bra)."""
    qs = [q for q in sorted(sectors) for _ in range(sectors[q])]
    norm = (lambda q: q % mod) if mod else (lambda q: q)
    es = sorted((norm(qk - qb), qk, i, j) for i, qk in enumerate(qs) for j, qb in enumerate(qs))
    dims = {}
    for e in es:
        dims[e[0]] = dims.get(e[0], 0) + 1
    return dims, [e[2] for e in es], [e[3] for e in es]


# --------------------------------- dense arrays with sectors, in 64 bits -----
class Sym:
    """Legs, the labels of the blocks that are there and, for values, a dense
    FP64 array (None: sizes only)."""

    def __init__(self, legs, flux, mod, blocks=None, t=None):
        self.legs, self.flux, self.mod, self.t = legs, flux, mod, t
        self.blocks = blocks
        if blocks is None:
            self.blocks = [b for b in itertools.product(*[sorted(s) for s, _ in legs])
                           if self._norm(sum(d * q for (_, d), q in zip(legs, b)) - flux) == 0]

    def _norm(self, q):
        return q % self.mod if self.mod else q

    def size(self, b):
        return math.prod(s[q] for (s, _), q in zip(self.legs, b))

    @property
    def nnz(self):
        return sum(self.size(b) for b in self.blocks)

    def _offsets(self, leg):
        out, o = {}, 0
        for q in sorted(self.legs[leg][0]):
            out[q] = o
            o += self.legs[leg][0][q]
        return out

    def slices(self, b):
        return tuple(slice(self._offsets(i)[q], self._offsets(i)[q] + self.legs[i][0][q]) for i, q in enumerate(b))

    def embed(self, values):
        """Dense array from the blocks' values in canonical order."""
        self.t = torch.zeros([sum(s.values()) for s, _ in self.legs], dtype=torch.float64, device=values.device)
        pos = 0
        for b in self.blocks:
            n = self.size(b)
            sl = self.slices(b)
            self.t[sl] = values[pos:pos + n].double().view(self.t[sl].shape)
            pos += n
        return self

    def canonical(self):
        return torch.cat([self.t[self.slices(b)].reshape(-1) for b in self.blocks])

    def flip(self, legs):
        """The listed legs reversed: direction and charges negated."""
        new, t = list(self.legs), self.t
        for i in legs:
            s, d = self.legs[i]
            off = self._offsets(i)
            new[i] = ({self._norm(-q): n for q, n in s.items()}, -d)
            idx = [off[q] + k for q in sorted(s, key=lambda q: self._norm(-q)) for k in range(s[q])]
            if t is not None:
                t = t.index_select(i, torch.tensor(idx, device=t.device))
        blocks = sorted(tuple(self._norm(-q) if i in legs else q for i, q in enumerate(b)) for b in self.blocks)
        return Sym(new, self.flux, self.mod, blocks, t)

    def permute(self, perm):
        return Sym([self.legs[p] for p in perm], self.flux, self.mod, sorted(tuple(b[p] for p in perm) for b in self.blocks),
                   None if self.t is None else self.t.permute(perm))


class Product:
    """X Y over the legs lx, ly: the result, its useful flops (over matched
    block pairs) and its buffer: one row-major matrix per contracted charge,
    ascending, rows X's open labels, columns Y's."""

    def __init__(self, X, Y, lx, ly, perm=None):
        fx = [i for i in range(len(X.legs)) if i not in lx]
        fy = [i for i in range(len(Y.legs)) if i not in ly]
        self.rows, self.cols, self.groups, self.flops = [X.legs[i] for i in fx], [Y.legs[i] for i in fy], [], 0
        tab = {}
        for side, (T, free, con) in enumerate(((X, fx, lx), (Y, fy, ly))):
            for b in T.blocks:
                key = T._norm((1, -1)[side] * sum(T.legs[i][1] * b[i] for i in con))
                tab.setdefault(key, ({}, {}))[side].setdefault(tuple(b[i] for i in free), set()).add(tuple(b[i] for i in con))
        blocks = []
        for key in sorted(tab):
            al, be = tab[key]
            kap = set().union(*al.values(), set()) & set().union(*be.values(), set())
            rows, cols = sorted(a for a in al if al[a] & kap), sorted(b for b in be if be[b] & kap)
            if not rows or not cols:
                continue
            self.groups.append((rows, cols))
            kd = {k: math.prod(X.legs[i][0][q] for i, q in zip(lx, k)) for k in kap}
            for a in rows:
                for b in cols:
                    common = al[a] & be[b]
                    if common:
                        blocks.append(a + b)
                        self.flops += 2 * self._dim(self.rows, a) * self._dim(self.cols, b) * sum(kd[k] for k in common)
        perm = list(range(len(fx) + len(fy))) if perm is None else perm
        legs = self.rows + self.cols
        self.t = None if X.t is None else torch.tensordot(X.t, Y.t, dims=(list(lx), list(ly)))
        self.out = Sym([legs[p] for p in perm], X._norm(X.flux + Y.flux), X.mod, sorted(tuple(b[p] for p in perm) for b in blocks),
                       None if self.t is None else self.t.permute(perm))

    @staticmethod
    def _dim(legs, labels):
        return math.prod(s[q] for (s, _), q in zip(legs, labels))

    @property
    def elems(self):
        return sum(sum(self._dim(self.rows, a) for a in r) * sum(self._dim(self.cols, b) for b in c) for r, c in self.groups)

    def _states(self, legs, labels):
        """Flat states of label tuples over `legs`, in order."""
        helper = Sym(legs, 0, 0, [], None)
        strides = [math.prod(sum(s.values()) for s, _ in legs[i + 1:]) for i in range(len(legs))]
        out = []
        for b in labels:
            idx = np.zeros(1, dtype=np.int64)
            for i, q in enumerate(b):
                o = helper._offsets(i)[q]
                idx = (idx[:, None] + strides[i] * np.arange(o, o + legs[i][0][q])[None]).reshape(-1)
            out.append(idx)
        return torch.from_numpy(np.concatenate(out)).to(self.t.device)

    def buffer(self):
        m = self.t.reshape(math.prod(sum(s.values()) for s, _ in self.rows), -1)
        return torch.cat([m[self._states(self.rows, r)][:, self._states(self.cols, c)].reshape(-1) for r, c in self.groups])


# legs of the three steps of each enlarged corner: (C Ta), (. Tb), (. a)
CORNER = {1: (([1], [0]), ([0], [2]), ([3, 0], [0, 1])), 2: (([0], [2]), ([0], [0]), ([1, 2], [1, 2])),
          3: (([1], [0]), ([0], [2]), ([3, 0], [2, 3])), 4: (([0], [2]), ([0], [0]), ([2, 1], [0, 3]))}


def _corner(which, C, Ta, Tb, a):
    steps = []
    X = C
    for (lx, ly), Y in zip(CORNER[which], (Ta, Tb, a)):
        steps.append(Product(X, Y, lx, ly))
        X = steps[-1].out
    return steps


def _projectors(Hu, Hd, chi):
    """Spectrum per sector of the cut (key ascending) and the kept P, P~."""
    (sx, dx), (sd, dd) = Hu.legs[:2]
    charge = lambda legs: np.array([Hu._norm(d0 * a + d1 * b) for (s0, d0), (s1, d1) in [legs]
                                    for a in sorted(s0) for _ in range(s0[a]) for b in sorted(s1) for _ in range(s1[b])])
    ru, cu, cd = charge(Hu.legs[:2]), charge(Hu.legs[2:]), charge(Hd.legs[2:])
    nr = len(ru)
    MU, MD = Hu.t.reshape(nr, -1), Hd.t.reshape(nr, -1)
    secs = []
    for v in set(ru.tolist()):
        pick = lambda c, q: torch.from_numpy(np.flatnonzero(c == q)).to(MU.device)
        r, u, d = pick(ru, v), pick(cu, Hu._norm(-v)), pick(cd, v)   # H_d's rows carry -v
        if not len(u) or not len(d):
            continue
        hu, hd = MU[r][:, u], MD[r][:, d]
        Y = hu.T @ hd
        J = torch.zeros((len(u) + len(d),) * 2, dtype=Y.dtype, device=Y.device)
        J[:len(u), len(u):] = Y
        J[len(u):, :len(u)] = Y.T
        w, z = torch.linalg.eigh(J)
        n = min(len(r), len(u), len(d))
        s, z = w.flip(0)[:n], z.flip(1)[:, :min(n, chi)] * math.sqrt(2.0)
        secs.append((Hu._norm(v * dx), r, s, z[:len(u)], z[len(u):], hu, hd))
    secs.sort(key=lambda x: x[0])
    cut = sorted((x for q in secs for x in q[2].tolist()), reverse=True)
    floor = cut[chi] if chi < len(cut) else -1.0
    P, Pt, kept, lab = [], [], {}, []
    for q, r, s, u, v, hu, hd in secs:
        k = int((s > max(floor, 1e-14 * cut[0])).sum())
        if not k:
            continue
        kept[q] = k
        full = torch.zeros((2, nr, k), dtype=s.dtype, device=s.device)
        full[0, r] = hd @ v[:, :k] / s[:k].sqrt()
        full[1, r] = hu @ u[:, :k] / s[:k].sqrt()
        P.append(full[0])
        Pt.append(full[1])
        lab += [(a, b, q) for a in sorted(sx) for b in sorted(sd) if Hu._norm(dx * a + dd * b - dx * q) == 0]
    n0, n1 = sum(sx.values()), sum(sd.values())
    P, Pt = torch.cat(P, 1).reshape(n0, n1, -1), torch.cat(Pt, 1).T.reshape(-1, n0, n1)
    return (torch.cat([q[2] for q in secs]),
            Sym([(sx, OUT), (sd, IN), (kept, IN)], 0, Hu.mod, sorted(lab), P),
            Sym([(kept, OUT), (sx, IN), (sd, OUT)], 0, Hu.mod, sorted((q, a, b) for a, b, q in lab), Pt))


def _move_parts(C, T, a, chi):
    """Left move: (products, C1', T4', C4', spectrum); sizes only (kept as
    chi's sectors) where the tensors hold no values."""
    ks = [_corner(w, C[w - 1], x, y, a) for w, x, y in ((1, T[0], T[3]), (2, T[0], T[1]), (3, T[2], T[1]), (4, T[2], T[3]))]
    k = [x[2].out for x in ks]
    hu, hd = Product(k[0], k[1], [0, 2], [0, 2]), Product(k[3], k[2], [0, 3], [0, 2])
    if a.t is None:
        (sx, _), (sd, _) = T[3].legs[0], a.legs[3]
        s, P = None, Sym([(sx, OUT), (sd, IN), (sx, IN)], 0, a.mod)
        Pt = Sym([(sx, OUT), (sx, IN), (sd, OUT)], 0, a.mod)
    else:
        s, P, Pt = _projectors(hu.out, hd.out, chi)
    c1 = Product(ks[0][0].out, P, [0, 1], [0, 1], [1, 0])
    c4 = Product(ks[3][0].out, Pt, [0, 2], [1, 2])
    x = Product(Pt, T[3], [1], [2])
    xx = Product(x.out, a, [1, 3], [1, 0])
    t4 = Product(xx.out, P, [1, 3], [0, 1], [2, 1, 0])
    for p in (c1, t4, c4):
        if p.t is not None:
            p.out.t = p.out.t / p.out.t.norm()
    return [p for q in ks for p in q] + [hu, hd, c1, c4, x, xx, t4], c1.out, t4.out, c4.out, s


def _turn(C, T, a):
    """The network a quarter turn counterclockwise."""
    return (C[1:] + C[:1], [T[1].flip([1]), T[2], T[3].flip([1]), T[0]], a.permute([1, 2, 3, 0]).flip([1, 3]))


def _moved(C, T, a, chi, direction):
    for _ in range(direction):
        C, T, a = _turn(C, T, a)
    C, T = list(C), list(T)
    _, C[0], T[3], C[3], s = _move_parts(C, T, a, chi)
    for _ in range(direction, 4):
        C, T, a = _turn(C, T, a)
    return C, T, s


def _column(Ca, Te, Cb):
    """C1' T4' C4' -> [x3, r, x1]."""
    return Product(Cb, Product(Te, Ca, [2], [0]).out, [1], [0])


def _kappa(C, T, a):
    e = lambda spec, x, y: torch.einsum(spec, x, y)
    C, T, a = [c.t for c in C], [x.t for x in T], a.t
    top = e("auc,cd->aud", e("ab,buc->auc", C[0], T[0]), C[1])
    bot = e("duf,fg->dug", e("de,euf->duf", C[2], T[2]), C[3])
    z00 = e("ac,ca->", C[0] @ C[1], C[2] @ C[3])
    z10 = e("aud,dua->", top, bot)
    z01 = e("frc,crf->", e("frb,bc->frc", T[3], C[0] @ C[1]), e("crd,df->crf", T[1], C[2] @ C[3]))
    x = e("aure,lurq->aelq", e("aud,dre->aure", top, T[1]), a)
    x = e("aelq,eqg->alg", x, bot)                    # bot[e, q, g]: C3 T3 C4
    z11 = e("alg,gla->", x, T[3])
    return z11 * z00 / (z10 * z01), [z00, z10, z01, z11]


# ------------------------------------------------------------------ inputs --
def _mod(case):
    return 2 if case.get("group") == "z2" else 0


def _dtype(case):
    return "f64" if case["prec"] == "f64" else "f32"


def _site(group, D, mod):
    v = _virt(group, D)
    phys = {0: 1, 1: 1} if group == "z2" else {-1: 1, 1: 1}
    return Sym([(phys, IN), (v, IN), (v, IN), (v, OUT), (v, OUT)], 0 if mod else 1, mod)


def _shapes(group, D, chi, mod):
    """Empty C1..C4, T1..T4, a (clockwise bonds)."""
    x, (dd, _, _) = _chi(group, chi), _fused(_virt(group, D), mod)
    C = [Sym([(x, IN), (x, OUT)], 0, mod) for _ in range(4)]
    T = [Sym([(x, IN), (dd, d), (x, OUT)], 0, mod) for d in (OUT, IN, IN, OUT)]
    return C, T, Sym([(dd, IN), (dd, IN), (dd, OUT), (dd, OUT)], 0, mod)


def _rand(gen, n, f64):
    return torch.randn(n, generator=gen, device="cuda", dtype=torch.float64 if f64 else torch.float32)


def _double(A, D, mod):
    """Dense double layer of the dense site tensor A."""
    _, ket, bra = _fused(D, mod)
    n = sum(D.values())
    m = A.reshape(A.shape[0], -1)
    g = (m.T @ m).reshape((n,) * 8).permute(0, 4, 1, 5, 2, 6, 3, 7).reshape((n * n,) * 4)
    idx = torch.tensor([k * n + b for k, b in zip(ket, bra)], device=A.device)
    for ax in range(4):
        g = g.index_select(ax, idx)
    return g


def _network(case, gen):
    """Values (canonical order, storage type) of one site's C1..C4, T1..T4, a."""
    group, mod, f64 = case.get("group", "u1"), _mod(case), _dtype(case) == "f64"
    C, T, a = _shapes(group, case["D"], case["chi"], mod)
    A = _site(group, case["D"], mod)
    A.embed(_rand(gen, A.nnz, True))
    vals = [_rand(gen, x.nnz, f64) for x in C + T]
    a.t = _double(A.t, _virt(group, case["D"]), mod)
    vals.append(a.canonical().to(torch.float64 if f64 else torch.float32))
    a.t = None
    return C + T + [a], vals


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


class _Shared:
    """A library tensor's device buffer for torch (which keeps it alive)."""

    def __init__(self, t, f64, first=0):
        ptr, n = t.device_ptr()
        es = 8 if f64 else 4
        self.owner = t
        self.__cuda_array_interface__ = {"shape": (n - first,), "typestr": "<f%d" % es, "data": (ptr + first * es, False),
                                         "version": 2}


def _view(t, f64, first=0):
    return torch.as_tensor(_Shared(t, f64, first), device="cuda")


def _front(values, size):
    out = values.new_zeros(size)
    out[:values.numel()] = values
    return out


def _most(case):
    """Largest sizes of the column, a corner and an edge after a move."""
    if case["kind"] == "su2":
        x, d, k = sum(_chi_su2(case).values()), sum(DOUBLE_SU2.values()), case["chi"]
    else:
        x, d, k = case["chi"], case["D"] ** 2, case["chi"]
    return x * d * x, max(k, x) ** 2, max(k, x) ** 2 * d


def _chi_su2(case):
    return {j: max(1, round(n * case["scale"])) for j, n in CHI_SU2.items()}


def _upload(shape, values, group):
    f64 = values.dtype == torch.float64
    t = st.Tensor.create(shape.legs, shape.flux, "f64" if f64 else "f32", group=group)
    _view(t, f64).copy_(values)
    return t


def _operands(case):
    """Shapes and legs of a single contraction: C T1, or X a with X the
    corner's [u, x1, x4, l] before the site tensor."""
    C, T, a = _shapes(case.get("group", "u1"), case["D"], case["chi"], _mod(case))
    if case["step"] == 1:
        return C[0], T[0], [1], [0]
    X = Product(Product(C[0], T[0], [1], [0]).out, T[3], [0], [2]).out
    return Sym(X.legs, 0, X.mod), a, [3, 0], [0, 1]


def _corner_inputs(which):
    return [(0, 4, 7), (1, 4, 5), (2, 6, 5), (3, 6, 7)][which - 1]


def prepare(case, seed):
    gen, group, kind = _generator(seed), case.get("group", "u1"), case["kind"]
    if kind == "contract":
        X, Y, lx, ly = _operands(case)
        f64 = _dtype(case) == "f64"
        return {"case": case, "X": _upload(X, _rand(gen, X.nnz, f64), group), "Y": _upload(Y, _rand(gen, Y.nnz, f64), group),
                "lx": lx, "ly": ly, "f64": f64}
    if kind == "double":
        A = _site(group, case["D"], _mod(case))
        f64 = _dtype(case) == "f64"
        return {"case": case, "A": _upload(A, _rand(gen, A.nnz, f64), group), "f64": f64}
    if kind == "batch":
        ins, first, pos = [], [], 0
        for D, chi in _batch_sizes(case["count"], case["layout"]):
            c = dict(case, D=D, chi=chi)
            shapes, vals = _network(c, gen)
            ins.append([_upload(shapes[i], vals[i], group) for i in (0, 4, 7, 8)])
            first.append(pos)      # the corners follow one another, each on a multiple of 32 values
            pos += -(-_corner(1, *[shapes[i] for i in (0, 4, 7, 8)])[2].elems // 32) * 32
        return {"case": case, "ins": list(zip(*ins)), "first": first, "f64": _dtype(case) == "f64"}
    if kind == "su2":
        A = st.Tensor.create([({1: 1}, IN), (VIRT_SU2, IN), (VIRT_SU2, IN), (VIRT_SU2, OUT), (VIRT_SU2, OUT)], 0, "f32", group="su2")
        _view(A, False).copy_(_rand(gen, A.nnz, False))
        a = st.double_layer(A)
        dd, x = DOUBLE_SU2, _chi_su2(case)
        t = [st.Tensor.create([(x, IN), (x, OUT)], 0, "f32", group="su2") for _ in range(4)]
        t += [st.Tensor.create([(x, IN), (dd, d), (x, OUT)], 0, "f32", group="su2") for d in (OUT, IN, IN, OUT)]
        for q in t:
            _view(q, False).copy_(_rand(gen, q.nnz, False))
        chi = sum((j + 1) * n for j, n in x.items())
        return {"case": dict(case, chi=chi, prec="f32", direction=0), "t": t, "a": a, "env": st.CtmEnv(t[:4], t[4:]), "f64": False}
    shapes, vals = _network(case, gen)
    t = [_upload(s, v, group) for s, v in zip(shapes, vals)]
    s = {"case": case, "t": t[:8], "a": t[8], "f64": _dtype(case) == "f64"}
    if kind != "corner":
        s["env"] = st.CtmEnv(t[:4], t[4:8])
    return s


# --------------------------------------------------------------- one pass ---
def _spectrum(env, f64):
    s = env.singular_values()
    return s if f64 else s.astype(np.float32)   # an FP32 move's spectrum is good to FP32


def run(state):
    case, f64 = state["case"], state["f64"]
    kind = case["kind"]
    if kind == "contract":
        return _view(st.contract(state["X"], state["Y"], state["lx"], state["ly"], prec=case["prec"]), f64)
    if kind == "double":
        return _view(st.double_layer(state["A"]), f64)
    if kind == "corner":
        i, j, k = _corner_inputs(case["which"])
        t = state["t"]
        return _view(st.enlarged_corner(case["which"], t[i], t[j], t[k], state["a"], prec=case["prec"])[0], f64)
    if kind == "batch":
        outs, _ = st.enlarged_corners_batched(*state["ins"], prec=case["prec"], use_graph=case["graph"])
        return [_view(t, f64, first) for t, first in zip(outs, state["first"])]
    env = state["env"]
    for k, t in enumerate(state["t"]):    # every pass from the same environment
        env.set(k, t)
    if kind == "step":
        for d in range(4):
            env.move(state["a"], case["chi"], prec="f64", direction=d, stats=False)
        kappa, z = env.site_partition(state["a"])
        _, corner, edge = _most(case)
        spectrum = torch.from_numpy(env.singular_values())
        return {"kappa": kappa, "z": np.array(z), "spectrum": _front(spectrum, case["chi"] * case["D"] ** 2),
                "env": [_front(_view(env.get(k), True), corner if k < 4 else edge) for k in range(8)]}
    env.move(state["a"], case["chi"], prec=case["prec"], direction=case["direction"], stats=False)
    d, e = case["direction"], (case["direction"] + 3) % 4
    Ca, Te, Cb = env.get(d), env.get(4 + e), env.get(e)
    column = st.contract(Cb, st.contract(Te, Ca, [2], [0], prec=case["prec"]), [1], [0], prec=case["prec"])
    most, corner, edge = _most(case)
    out = {"column": _front(_view(column, f64), most), "spectrum": _spectrum(env, f64)}
    if f64:
        out["env"] = [_front(_view(t, True), n) for t, n in ((Ca, corner), (Te, edge), (Cb, corner))]
    return out


# ------------------------------------------------- what a pass cannot avoid --
def work(case):
    kind, es = case["kind"], 8 if case.get("prec") == "f64" else 4
    mod = _mod(case)
    if kind == "contract":
        X, Y, lx, ly = _operands(case)
        p = Product(X, Y, lx, ly)
        return {"bytes": es * (X.nnz + Y.nnz + p.elems), "flops": p.flops}
    if kind == "double":
        A, (_, _, a) = _site(case.get("group", "u1"), case["D"], mod), _shapes(case.get("group", "u1"), case["D"], 16, mod)
        return {"bytes": es * (A.nnz + a.nnz), "flops": 4 * a.nnz}
    if kind == "su2":
        x, dd = _chi_su2(case), DOUBLE_SU2
        nnz = lambda *legs: st.Tensor.meta(list(legs), 0, "f32", group="su2").nnz
        moved = 2 * nnz((x, IN), (x, OUT)) + nnz((x, IN), (dd, OUT), (x, OUT))
        read = 4 * nnz((x, IN), (x, OUT)) + 4 * nnz((x, IN), (dd, OUT), (x, OUT)) + nnz((dd, IN), (dd, IN), (dd, OUT), (dd, OUT))
        # reduced block pairs at scale 1; the cut grows with chi
        return {"bytes": 4 * (read + moved), "flops": 2.6e10 * case["scale"] ** 3}
    sizes = _batch_sizes(case["count"], case["layout"]) if kind == "batch" else [(case["D"], case["chi"])]
    total = {"bytes": 0, "flops": 0}
    for D, chi in sizes:
        C, T, a = _shapes(case.get("group", "u1"), D, chi, mod)
        if kind in ("batch", "corner"):
            i, j, k = _corner_inputs(case.get("which", 1))
            t = C + T
            steps = _corner(case.get("which", 1), t[i], t[j], t[k], a)
            total["bytes"] += es * (t[i].nnz + t[j].nnz + t[k].nnz + a.nnz + steps[2].elems)
            total["flops"] += sum(p.flops for p in steps)
            continue
        prods, c1, t4, c4, _ = _move_parts(C, T, a, chi)
        cut = {}
        for (q, n), (p, m) in itertools.product(T[3].legs[0][0].items(), a.legs[3][0].items()):
            key = (q - p) % mod if mod else q - p
            cut[key] = cut.get(key, 0) + n * m
        # Y = H_u^T H_d per sector, then the spectrum of every sector's Y
        flops = sum(p.flops for p in prods) + sum(2 * n ** 3 + 8 * n ** 3 // 3 for n in cut.values())
        times = 4 if kind == "step" else 1
        total["flops"] += times * flops
        total["bytes"] += times * es * (sum(x.nnz for x in C + T) + a.nnz + c1.nnz + t4.nnz + c4.nnz)
    return total


# -------------------------------------------------------- 64-bit references --
def exact(case, seed):
    gen, kind, mod = _generator(seed), case["kind"], _mod(case)
    if kind == "su2":
        return None      # reduced tensors: no plain array of their own
    if kind == "contract":
        X, Y, lx, ly = _operands(case)
        f64 = _dtype(case) == "f64"
        X.embed(_rand(gen, X.nnz, f64))
        Y.embed(_rand(gen, Y.nnz, f64))
        return Product(X, Y, lx, ly).buffer()
    if kind == "double":
        A = _site(case.get("group", "u1"), case["D"], mod)
        A.embed(_rand(gen, A.nnz, _dtype(case) == "f64"))
        a = _shapes(case.get("group", "u1"), case["D"], 16, mod)[2]
        a.t = _double(A.t, _virt(case.get("group", "u1"), case["D"]), mod)
        return a.canonical()
    if kind == "batch":
        out = []
        for D, chi in _batch_sizes(case["count"], case["layout"]):
            shapes, vals = _network(dict(case, D=D, chi=chi), gen)
            out.append(_corner(1, *[shapes[i].embed(vals[i]) for i in (0, 4, 7, 8)])[2].buffer())
        return out
    shapes, vals = _network(case, gen)
    t = [s.embed(v) for s, v in zip(shapes, vals)]
    if kind == "corner":
        return _corner(case["which"], *[t[i] for i in _corner_inputs(case["which"])], t[8])[2].buffer()
    C, T, a = t[:4], t[4:8], t[8]
    if kind == "step":
        for d in range(4):
            C, T, s = _moved(C, T, a, case["chi"], d)
        kappa, z = _kappa(C, T, a)
        return {"kappa": float(kappa), "z": torch.stack(z), "spectrum": _front(s, case["chi"] * case["D"] ** 2), "env": None}
    d, e = case["direction"], (case["direction"] + 3) % 4
    C, T, s = _moved(C, T, a, case["chi"], d)
    out = {"column": _front(_column(C[d], T[e], C[e]).buffer(), _most(case)[0]), "spectrum": s}
    if _dtype(case) == "f64":
        out["env"] = None
    return out


# ------------------------------------------------------------------- cases --
def listed():
    return [
        # the smallest call: two small operands, where launches and the host's
        # work on the call count
        {"name": "contract_ct_D4_chi16_f64", "kind": "contract", "step": 1, "D": 4, "chi": 16, "prec": "f64"},
        # the absorption of a site tensor on its own, with odd leg sizes
        {"name": "contract_xa_D5_chi53_f32", "kind": "contract", "step": 3, "D": 5, "chi": 53, "prec": "f32"},
        # the same in FP64, as convergence checks and energies run it
        {"name": "contract_xa_D7_chi90_f64", "kind": "contract", "step": 3, "D": 7, "chi": 90, "prec": "f64"},
        # an ordinary enlarged corner, one call
        {"name": "corner_D6_chi64_f32", "kind": "corner", "which": 1, "D": 6, "chi": 64, "prec": "f32"},
        # the largest corner, in the split precision that holds FP32's accuracy
        {"name": "corner_D8_chi200_bf16x6", "kind": "corner", "which": 3, "D": 8, "chi": 200, "prec": "bf16x6"},
        # throughput: 64 corners of mixed sizes per call, replayed from a graph
        {"name": "batch64_bf16x3", "kind": "batch", "count": 64, "layout": 1813, "prec": "bf16x3", "graph": True},
        # one step of a small FP64 iteration, all four sides and kappa
        {"name": "step_D4_chi16_f64", "kind": "step", "D": 4, "chi": 16, "prec": "f64"},
        # the ordinary move of an optimisation, in FP32 and in FP64
        {"name": "move_D6_chi64_f32", "kind": "move", "D": 6, "chi": 64, "prec": "f32", "direction": 0},
        {"name": "move_D6_chi64_f64", "kind": "move", "D": 6, "chi": 64, "prec": "f64", "direction": 0},
        # the largest move: cut sectors of up to 3144 states
        {"name": "move_D8_chi200_f32", "kind": "move", "D": 8, "chi": 200, "prec": "f32", "direction": 0},
        # the move of a non-abelian environment, D = 10 and chi = 100 in all
        {"name": "su2_move_f32", "kind": "su2", "scale": 1.0},
        # the double layer, formed once per update of the site tensor
        {"name": "double_D8_f32", "kind": "double", "D": 8, "prec": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["contract", "contract", "corner", "batch", "step", "move", "move", "move", "su2", "double"])
    group = rng.choice(["u1", "u1", "z2"])
    D = rng.randint(4, 8)
    if kind == "contract":
        return {"kind": kind, "group": group, "step": rng.choice([1, 3]), "D": D, "chi": _log(rng, 16, 160 if D > 6 else 200),
                "prec": rng.choice(["f64", "f32", "bf16", "bf16x3", "bf16x6"])}
    if kind == "corner":
        return {"kind": kind, "group": group, "which": rng.randint(1, 4), "D": D, "chi": _log(rng, 16, 120 if group == "z2" else 200),
                "prec": rng.choice(["f64", "f32", "bf16", "bf16x3", "bf16x6"])}
    if kind == "batch":
        return {"kind": kind, "count": _log(rng, 2, 60), "layout": rng.randint(1, 9999),
                "prec": rng.choice(["f32", "bf16", "bf16x3", "bf16x6"]), "graph": rng.random() < 0.7}
    if kind == "step":
        return {"kind": kind, "D": rng.randint(4, 5), "chi": rng.randint(16, 40), "prec": "f64"}
    if kind == "move":
        prec = rng.choice(["f32", "f32", "f64", "bf16x6"])
        D = rng.randint(4, 6 if prec == "f64" or group == "z2" else 8)
        return {"kind": kind, "group": group, "D": D, "chi": _log(rng, 20, 64 if prec == "f64" else 100 if group == "z2" else 180),
                "prec": prec, "direction": rng.randint(0, 3)}
    if kind == "su2":
        return {"kind": kind, "scale": round(rng.uniform(0.3, 1.0), 2)}
    return {"kind": kind, "group": group, "D": D, "prec": rng.choice(["f64", "f32"])}
