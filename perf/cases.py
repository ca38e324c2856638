"""What a user of the layout transform has it do, as measurable cases.

Each case is a dict of plain values: an entry point, an element type, an op
with its scalars, the shape of A, and the two layouts.  A layout is block
cyclic (block sizes, process grid, rank and storage order; for the ScaLAPACK
routines also the first process, a padded leading dimension and a window) or
a general grid of random cuts with random owners, drawn from a seed that is
part of the case.

`prepare` makes what a program holds before the call: layout handles, the
relabeling where it uses one, and one device buffer per rank.  `run` is the
call.  Outputs are the local buffers of A, whole, in the order of the labels
(the relabeling moves a label to another rank; its contents stay the same), laid
out in one arena a matrix.
`exact` forms the same buffers with plain torch from global matrices.
"""
import math
import random

import numpy as np
import torch

import paper_2106_06601_amd as costa

ELEM = {"f64": 8, "c128": 16, "f32": 4, "c64": 8}
TORCH = {"f64": torch.float64, "c128": torch.complex128, "f32": torch.float32, "c64": torch.complex64}
DEVICE = "cuda"
WIDE = {"f64": torch.float64, "c128": torch.complex128, "f32": torch.float64, "c64": torch.complex128}


# ---------------------------------------------------------------------------
# layouts
# ---------------------------------------------------------------------------
def _numroc(n, b, iproc, src, nprocs):
    """Rows (or columns) of an n-long dimension in blocks of b that process
    `iproc` holds when the first block sits on process `src`."""
    nblocks = n // b
    d = (iproc - src) % nprocs
    size = nblocks // nprocs * b
    extra = nblocks % nprocs
    return size + (b if d < extra else n % b if d == extra else 0)


class Grid:
    """A layout of a case: side "s" (source B) or "t" (target A) of rows x
    cols elements; for the ScaLAPACK routines the full matrix and the window
    in it."""

    def __init__(self, case, side, rows, cols, seed=0):
        g = lambda k, d=None: case.get(f"{side}_{k}", d)  # noqa: E731
        self.rows, self.cols = rows, cols
        self.col_major = g("store", "col") == "col"
        self.cuts = g("cuts", 0)
        if self.cuts:
            self.nranks = case["ranks"]
            rng = random.Random(g("seed") + (seed << 32 if case["entry"] == "volume" else 0))
            cut = lambda n: [0] + sorted(rng.sample(range(1, n), min(self.cuts, n - 1))) + [n]  # noqa: E731
            if g("even", False):  # contiguous near-equal blocks, one a rank
                k = self.cuts + 1
                self.rs, self.cs = [i * rows // k for i in range(k + 1)], [i * cols // k for i in range(k + 1)]
                self.owners = [i % self.nranks for i in range(k * k)]
            else:
                self.rs, self.cs = cut(rows), cut(cols)
                self.owners = [rng.randrange(self.nranks) for _ in range((len(self.rs) - 1) * (len(self.cs) - 1))]
            return
        self.mb, self.nb = g("mb"), g("nb")
        self.prow, self.pcol = g("prow"), g("pcol")
        self.rank_order = g("rank", "row")
        self.nranks = self.prow * self.pcol
        self.rsrc, self.csrc, self.pad = g("rsrc", 0), g("csrc", 0), g("pad", -1)
        # 1-based window of a larger matrix (ScaLAPACK routines only)
        self.i, self.j, self.tail = g("i", 1), g("j", 1), g("tail", 0)
        if case["entry"] == "volume" and side == "s":  # the inputs are the layouts: the seed picks the window
            rng = random.Random(seed)
            self.i, self.j = 1 + rng.randrange(2 * self.mb), 1 + rng.randrange(2 * self.nb)
            self.rsrc, self.csrc, self.pad = rng.randrange(self.prow), rng.randrange(self.pcol), 0
        self.m, self.n = rows + self.i - 1 + self.tail, cols + self.j - 1 + self.tail
        self.lld = max(_numroc(self.m, self.mb, p, self.rsrc, self.prow) for p in range(self.prow)) + self.pad \
            if self.pad >= 0 else 0
        self.lld = max(self.lld, 1) if self.pad >= 0 else 0

    def place(self, r):
        """(process row, process column) of rank r."""
        return (r // self.pcol, r % self.pcol) if self.rank_order == "row" else (r % self.prow, r // self.prow)

    def local(self, r):
        """Local matrix of rank r: (rows, columns, leading dimension)."""
        pr, pc = self.place(r)
        lr = _numroc(self.m, self.mb, pr, self.rsrc, self.prow)
        lc = _numroc(self.n, self.nb, pc, self.csrc, self.pcol)
        return lr, lc, self.lld or max(1, lr if self.col_major else lc)

    def size(self, r):
        """Elements of rank r's buffer."""
        if self.cuts:
            nbc = len(self.cs) - 1
            return sum((self.rs[k // nbc + 1] - self.rs[k // nbc]) * (self.cs[k % nbc + 1] - self.cs[k % nbc])
                       for k, o in enumerate(self.owners) if o == r)
        lr, lc, ld = self.local(r)
        return 0 if lr == 0 or lc == 0 else (ld * (lc - 1) + lr if self.col_major else ld * (lr - 1) + lc)

    def handle(self):
        if self.cuts:
            return costa.Layout.general(self.rows, self.cols, self.rs, self.cs, self.owners, self.nranks,
                                        "col" if self.col_major else "row")
        if self.pad >= 0:
            d, grid = self.desc()
            return costa.Layout.scalapack(d, *grid).submatrix(self.i - 1, self.j - 1, self.rows, self.cols)
        return costa.Layout.block_cyclic(self.m, self.n, self.mb, self.nb, self.prow, self.pcol, self.rank_order,
                                         "col" if self.col_major else "row")

    def desc(self):
        """ScaLAPACK array descriptor and grid."""
        return ([1, 0, self.m, self.n, self.mb, self.nb, self.rsrc, self.csrc, self.lld],
                (self.prow, self.pcol, self.rank_order))

    def tiles(self, bufs):
        """(row indices, column indices, strided view of the buffer) of every
        rectangular part of the matrix, for the plain-torch reference."""
        if self.cuts:
            at = [0] * self.nranks
            nbc = len(self.cs) - 1
            for k, o in enumerate(self.owners):
                bi, bj = k // nbc, k % nbc
                h, w = self.rs[bi + 1] - self.rs[bi], self.cs[bj + 1] - self.cs[bj]
                st = (1, h) if self.col_major else (w, 1)
                yield (torch.arange(self.rs[bi], self.rs[bi + 1]), torch.arange(self.cs[bj], self.cs[bj + 1]),
                       torch.as_strided(bufs[o], (h, w), st, bufs[o].storage_offset() + at[o]))
                at[o] += h * w
            return
        for r in range(self.nranks):
            lr, lc, ld = self.local(r)
            if lr == 0 or lc == 0:
                continue
            pr, pc = self.place(r)
            own = lambda n, b, p, src, np_: torch.arange(n)[(torch.arange(n) // b + src) % np_ == p]  # noqa: E731
            yield (own(self.m, self.mb, pr, self.rsrc, self.prow), own(self.n, self.nb, pc, self.csrc, self.pcol),
                   torch.as_strided(bufs[r], (lr, lc), (1, ld) if self.col_major else (ld, 1),
                                    bufs[r].storage_offset()))


def _pairs(case, seed=0):
    """Per pair of the case: (op, A's grid, B's grid)."""
    out = []
    for k in range(case.get("pairs", 1)):
        op = case["op"]
        if k < case.get("n_pairs", 0):
            op = "N"
        m, n = case["m"], case["n"]
        rows, cols = (m, n) if op == "N" else (n, m)
        out.append((op, Grid(case, "t", m, n, seed), Grid(case, "s", rows, cols, seed)))
    return out


def _scalars(case):
    a = complex(case.get("alpha", 1.0), case.get("alpha_im", 0.0))
    b = complex(case.get("beta", 0.0), case.get("beta_im", 0.0))
    return (a, b) if case["dtype"] in ("c128", "c64") else (a.real, b.real)


def _split(flat, grid):
    """The ranks' buffers in an arena: one after another, each on a 256-byte
    line."""
    step = 256 // flat.element_size()
    out, at = [], 0
    for r in range(grid.nranks):
        n = grid.size(r)
        out.append(flat[at:at + n])
        at += -(-n // step) * step
    return out


def _inputs(case, seed):
    """Seeded arenas, uniform on [-1, 1): per pair, A's (its buffers by label)
    and B's."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    step = 256 // ELEM[case["dtype"]]

    def arena(grid):
        n = sum(-(-grid.size(r) // step) * step for r in range(grid.nranks))
        t = torch.empty(n, dtype=TORCH[case["dtype"]], device=DEVICE)
        (torch.view_as_real(t) if t.is_complex() else t).uniform_(-1.0, 1.0, generator=gen)
        return t

    return [(arena(ga), arena(gb)) for _, ga, gb in _pairs(case)]


# ---------------------------------------------------------------------------
# what is measured
# ---------------------------------------------------------------------------
def prepare(case, seed):
    pairs = _pairs(case, seed)
    if case["entry"] == "volume":
        op, ga, gb = pairs[0]
        return {"case": case, "A": ga.handle(), "B": gb.handle(), "op": op}
    data = _inputs(case, seed)
    alpha, beta = _scalars(case)
    st = {"case": case, "alpha": alpha, "beta": beta}
    if case["entry"] in ("gemr2d", "tran"):
        op, ga, gb = pairs[0]
        st.update(op=op, a=_split(data[0][1], gb), c=_split(data[0][0], ga), out=data[0][0], da=gb.desc(), dc=ga.desc(), sa=(gb.i, gb.j), sc=(ga.i, ga.j))
        return st
    hs = [(ga.handle(), gb.handle()) for _, ga, gb in pairs]
    P = pairs[0][1].nranks
    sigma = None
    if case.get("relabel", False):
        V = sum(costa.costa_volume_matrix(h[0], h[1], p[0]) for h, p in zip(hs, pairs))
        sigma = costa.costa_relabel(V)[0]
    sg = list(range(P)) if sigma is None else sigma
    descs = []
    for (op, ga, gb), (ha, hb), (a, b) in zip(pairs, hs, data):
        a, b = _split(a, ga), _split(b, gb)
        phys = [None] * P
        for t in range(P):
            phys[sg[t]] = a[t]
        descs.append(dict(op=op, alpha=alpha, beta=beta, A=ha, A_local=phys, B=hb, B_local=b))
    st.update(descs=descs, sigma=sigma, out=[d[0] for d in data])
    return st


def run(st):
    c = st["case"]
    if c["entry"] == "volume":
        return costa.costa_volume_matrix(st["A"], st["B"], st["op"])
    if c["entry"] == "gemr2d":
        costa.costa_pxgemr2d(c["dtype"], c["m"], c["n"], st["a"], *st["sa"], *st["da"], st["c"], *st["sc"],
                             *st["dc"])
        return st["out"]
    if c["entry"] == "tran":
        costa.costa_pxtran(c["dtype"], st["op"], c["m"], c["n"], st["alpha"], st["a"], *st["sa"], *st["da"],
                           st["beta"], st["c"], *st["sc"], *st["dc"])
        return st["out"]
    if c["entry"] == "transform":
        d = st["descs"][0]
        costa.costa_transform(c["dtype"], d["op"], d["alpha"], d["beta"], d["A"], d["A_local"], d["B"], d["B_local"],
                              st["sigma"])
    elif c["entry"] == "batched":
        costa.costa_transform_batched(c["dtype"], st["descs"], st["sigma"])
    else:
        costa.costa_transform_batched_noalloc(c["dtype"], st["descs"], st["sigma"])
    return st["out"]


def work(case):
    if case["entry"] == "volume":
        # the two grids' cut points in, the P x P matrix out; one addition an
        # interval of each dimension's overlay
        op, ga, gb = _pairs(case)[0]
        cuts = 0
        for g in (ga, gb):
            cuts += len(g.rs) + len(g.cs) if g.cuts else math.ceil(g.m / g.mb) + math.ceil(g.n / g.nb)
        return {"bytes": 8 * cuts + 8 * ga.nranks ** 2, "flops": cuts}
    elems = case["m"] * case["n"] * case.get("pairs", 1)
    alpha, beta = _scalars(case)
    cplx = case["dtype"] in ("c128", "c64")
    per = 0 if alpha == 1 and beta == 0 else (6 if cplx else 1) if beta == 0 else (14 if cplx else 3)
    return {"bytes": elems * ELEM[case["dtype"]] * (3 if beta != 0 else 2), "flops": elems * per}


def tolerance(case):
    alpha, beta = _scalars(case)
    if case["entry"] == "volume" or (alpha == 1 and beta == 0):
        return "exact"  # counts, and permutations of the input's values
    # two products and a sum (four and three for complex numbers) of the
    # type's own precision; an implementation that fuses a product into the
    # sum differs by about a third of this
    return {"rel": 2e-7 if case["dtype"] in ("f32", "c64") else 4e-16}


def exact(case, seed):
    if case["entry"] == "volume":
        return _exact_volume(case, seed)
    alpha, beta = _scalars(case)
    wide = WIDE[case["dtype"]]
    out = []
    for (op, ga, gb), (a, b) in zip(_pairs(case), _inputs(case, seed)):
        G = torch.zeros(gb.rows if gb.cuts else gb.m, gb.cols if gb.cuts else gb.n, dtype=wide, device=DEVICE)
        for r, c, v in gb.tiles(_split(b, gb)):
            G[r.to(DEVICE)[:, None], c.to(DEVICE)[None, :]] = v.to(wide)
        if not gb.cuts:
            G = G[gb.i - 1:gb.i - 1 + gb.rows, gb.j - 1:gb.j - 1 + gb.cols]
        if op != "N":
            G = G.t()
        if op == "C" and G.is_complex():
            G = G.conj().resolve_conj()
        res = a.to(wide)
        views = [res[v.storage_offset():v.storage_offset() + v.numel()] for v in _split(a, ga)]
        r0, c0 = (0, 0) if ga.cuts else (ga.i - 1, ga.j - 1)
        for r, c, v in ga.tiles(views):
            kr, kc = (r >= r0) & (r < r0 + ga.rows), (c >= c0) & (c < c0 + ga.cols)
            if not kr.any() or not kc.any():
                continue
            # the kept rows and columns of a local matrix are contiguous runs
            kr, kc = kr.nonzero()[:, 0], kc.nonzero()[:, 0]
            w = v[int(kr[0]):int(kr[-1]) + 1, int(kc[0]):int(kc[-1]) + 1]
            x = G[(r[kr] - r0).to(DEVICE)[:, None], (c[kc] - c0).to(DEVICE)[None, :]]
            w.copy_(x if alpha == 1 and beta == 0 else alpha * x if beta == 0 else alpha * x + beta * w)
        out.append(res)
    return out if case["entry"] in ("transform", "batched", "noalloc") else out[0]


def _exact_volume(case, seed):
    op, ga, gb = _pairs(case, seed)[0]
    V = np.zeros((gb.nranks, ga.nranks), dtype=np.int64)
    if gb.cuts:
        # every pair of overlay intervals, by the owners of the blocks over it
        def overlay(a, b):
            pts = np.union1d(a, b)
            mid = pts[:-1]
            return np.searchsorted(a, mid, "right") - 1, np.searchsorted(b, mid, "right") - 1, np.diff(pts)

        ra, rb, rl = overlay(ga.rs, gb.rs if op == "N" else gb.cs)
        ca, cb, cl = overlay(ga.cs, gb.cs if op == "N" else gb.rs)
        oa = np.array(ga.owners).reshape(len(ga.rs) - 1, -1)[ra][:, ca]
        ob = np.array(gb.owners).reshape(len(gb.rs) - 1, -1)
        ob = ob[rb][:, cb] if op == "N" else ob[cb][:, rb].T
        np.add.at(V, (ob.ravel(), oa.ravel()), np.outer(rl, cl).ravel())
        return V

    def owners(g, transposed):
        """Per process: its rows and its columns of op(window), as 0/1 rows."""
        i, j = np.arange(g.rows) + g.i - 1, np.arange(g.cols) + g.j - 1
        rows = np.array([(i // g.mb + g.rsrc) % g.prow == p for p in range(g.prow)], dtype=np.float64)
        cols = np.array([(j // g.nb + g.csrc) % g.pcol == p for p in range(g.pcol)], dtype=np.float64)
        return (cols, rows) if transposed else (rows, cols)

    ar, ac = owners(ga, False)
    br, bc = owners(gb, op != "N")
    hr, hc = br @ ar.T, bc @ ac.T  # counts below 2^53: exact in float64
    for s in range(gb.nranks):
        i, j = gb.place(s)
        i, j = (j, i) if op != "N" else (i, j)
        for t in range(ga.nranks):
            k, l = ga.place(t)
            V[s, t] = int(hr[i, k]) * int(hc[j, l])
    return V


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _bc(side, mb, nb, prow, pcol, rank="row", store="col", **kw):
    d = {"mb": mb, "nb": nb, "prow": prow, "pcol": pcol, "rank": rank, "store": store, **kw}
    return {f"{side}_{k}": v for k, v in d.items()}


def listed():
    f64 = {"dtype": "f64", "alpha": 1.0, "beta": 0.0}
    return [
        # the smallest call: a subspace matrix of a few hundred rows moved
        # between two solvers' grids inside an iteration; launches and host
        # time are all of it
        {"name": "small_subspace_c64", "entry": "transform", "dtype": "c64", "op": "C", "m": 320, "n": 200,
         "alpha": 1.0, "beta": 0.0, **_bc("s", 32, 32, 2, 2), **_bc("t", 48, 40, 2, 2, "col")},
        # a 1024^2 reshuffle with transpose and relabeling
        {"name": "reshuffle_transpose_1k", "entry": "transform", "op": "T", "m": 1024, "n": 1024, "relabel": True,
         **f64, **_bc("s", 32, 32, 2, 2), **_bc("t", 64, 64, 2, 2, "col")},
        # a serving loop that must not allocate: a small batch through the
        # static scratch array
        {"name": "noalloc_batch_2k", "entry": "noalloc", "dtype": "f32", "op": "T", "m": 2048, "n": 1536,
         "alpha": 2.0, "beta": 0.0, "pairs": 4, "n_pairs": 2, **_bc("s", 64, 64, 2, 4), **_bc("t", 128, 96, 4, 2)},
        # odd sizes and odd blocks in single precision, row-major blocks into
        # column-major ones, accumulated
        {"name": "ragged_f32_7001x4999", "entry": "transform", "dtype": "f32", "op": "N", "m": 7001, "n": 4999,
         "alpha": -1.5, "beta": 0.25, **_bc("s", 37, 53, 3, 2, "row", "row"), **_bc("t", 64, 41, 2, 3, "row", "col")},
        # a ScaLAPACK block-size change of a large matrix, relabeled
        {"name": "blocksize_change_16k", "entry": "transform", "op": "N", "m": 16384, "n": 16384, "relabel": True,
         **f64, **_bc("s", 128, 128, 4, 4), **_bc("t", 256, 256, 4, 4)},
        # scaled, accumulated transpose whose blocks do not fit one another
        {"name": "scaled_transpose_20k", "entry": "transform", "dtype": "f64", "op": "T", "m": 20000, "n": 20000,
         "alpha": 2.0, "beta": 0.5, **_bc("s", 64, 64, 8, 4, "row", "col"), **_bc("t", 100, 100, 4, 8, "row", "row")},
        # random grid to contiguous blocks (a matrix-multiply library's
        # layout), conjugate-transposed complex numbers
        {"name": "cosma_complex_16k", "entry": "transform", "dtype": "c128", "op": "C", "m": 16384, "n": 16384,
         "alpha": 1.0, "beta": 0.0, "ranks": 64, "s_cuts": 40, "s_seed": 5, "t_cuts": 7, "t_even": True, "t_seed": 0},
        # tall-and-skinny operands of a batch of products, accumulated; half
        # of them transposed on the way
        {"name": "tall_skinny_batch", "entry": "batched", "dtype": "f64", "op": "T", "m": 4096, "n": 16384,
         "alpha": 1.0, "beta": 1.0, "pairs": 8, "n_pairs": 4, **_bc("s", 64, 64, 1, 64),
         **_bc("t", 512, 512, 8, 8)},
        # pdgemr2d of a submatrix that starts inside a block, padded local
        # matrices, 256 ranks, small blocks into large ones
        {"name": "pdgemr2d_window_16k", "entry": "gemr2d", "op": "N", "m": 16384, "n": 16384, **f64,
         **_bc("s", 32, 32, 16, 16, i=17, j=273, tail=223, pad=8), **_bc("t", 128, 128, 16, 16, rsrc=3, csrc=5, pad=8)},
        # pdtran of the same shape
        {"name": "pdtran_window_16k", "entry": "tran", "op": "T", "m": 16384, "n": 16384, **f64,
         **_bc("s", 32, 32, 16, 16, i=17, j=273, tail=223, pad=8), **_bc("t", 128, 128, 16, 16, rsrc=3, csrc=5, pad=8)},
        # pztranc of a submatrix, complex scalars, accumulated
        {"name": "pztranc_window_8k", "entry": "tran", "dtype": "c128", "op": "C", "m": 8192, "n": 8192,
         "alpha": 1.0, "alpha_im": -1.0, "beta": 0.5,
         **_bc("s", 64, 64, 8, 8, "col", i=50, j=51, tail=49, rsrc=1, csrc=2, pad=4), **_bc("t", 96, 96, 8, 8, pad=0)},
        # the communication volumes of a large redistribution, which a
        # program asks for before it relabels
        {"name": "volume_100k_blocks_30", "entry": "volume", "dtype": "f64", "op": "N", "m": 100000, "n": 100000,
         **_bc("s", 30, 30, 10, 10), **_bc("t", 10000, 10000, 10, 10, "col")},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    dtype = rng.choice(["f64", "f64", "c128", "f32", "c64"])
    entry = rng.choice(["transform", "transform", "transform", "batched", "noalloc", "gemr2d", "tran", "tran",
                        "volume"])
    op = "N" if entry == "gemr2d" else rng.choice("TC") if entry == "tran" else rng.choice("NTC")
    case = {"entry": entry, "dtype": dtype, "op": op}
    cplx = dtype in ("c128", "c64")
    mode = "copy" if entry in ("gemr2d", "volume") else rng.choice(["copy", "copy", "scale", "axpby", "axpby"])
    case["alpha"] = 1.0 if mode == "copy" else rng.choice([2.0, -1.5, 0.3])
    case["beta"] = rng.choice([0.5, 1.0]) if mode == "axpby" else 0.0
    if cplx and mode != "copy":
        case["alpha_im"] = rng.choice([0.0, -1.0])
    if entry == "volume":
        case["m"], case["n"] = _log(rng, 1000, 100000), _log(rng, 1000, 100000)
        if rng.random() < 0.3:  # two general grids, random owners
            case.update({"ranks": rng.choice([4, 16, 64]), "s_cuts": _log(rng, 20, 400),
                         "s_seed": rng.randrange(1 << 30), "t_cuts": _log(rng, 4, 100),
                         "t_seed": rng.randrange(1 << 30)})
            return case
        p = rng.choice([2, 4, 10])
        case.update(_bc("s", _log(rng, 16, 1000), _log(rng, 16, 1000), p, p, "row"))
        case.update(_bc("t", _log(rng, 100, 10000), _log(rng, 100, 10000), p, p, "col"))
        return case
    # elements of all pairs together: from a few ten thousand to 1.2e8 (5.8 GB
    # moved by an accumulated complex128 transform, below the largest case)
    pairs = rng.choice([2, 4]) if entry in ("batched", "noalloc") else 1
    elems = _log(rng, 2 ** 15, 2 ** 24 if entry == "noalloc" else 1.2e8) // pairs
    aspect = math.exp(rng.uniform(math.log(1 / 8), math.log(8)))
    m = max(33, int(math.sqrt(elems * aspect)))
    n = max(33, elems // m)
    case["m"], case["n"] = m, n
    if pairs > 1:
        case["pairs"], case["n_pairs"] = pairs, rng.choice([0, pairs // 2])
    # process grids of the same number of ranks; blocks of at least a 300th of
    # a dimension (at most a few hundred thousand overlay blocks; a 48th for
    # the entry point whose plan tables must fit its scratch array)
    pr, pc = rng.choice([(1, 1), (1, 4), (2, 2), (2, 3), (4, 4), (4, 8), (8, 8)])

    def side(s, rows, cols):
        a, b = (pr, pc) if rng.random() < 0.5 else (pc, pr)

        def block(d):
            lo = max(32, d // 48) if entry == "noalloc" else max(8, d // 300)
            b_ = _log(rng, lo, max(lo, min(512, d)))
            return max(lo, b_ // 16 * 16) if rng.random() < 0.5 else b_

        extra = {}
        if entry in ("gemr2d", "tran"):
            extra = {"i": rng.randrange(1, 100), "j": rng.randrange(1, 100), "tail": rng.randrange(0, 64),
                     "rsrc": rng.randrange(a), "csrc": rng.randrange(b), "pad": rng.choice([0, 1, 4, 8])}
        mb, nb = block(rows), block(cols)
        if entry in ("batched", "noalloc"):  # one layout rule for both orientations
            mb = nb = max(mb, nb)
        case.update(_bc(s, mb, nb, a, b, rng.choice(["row", "col"]),
                        "col" if entry in ("gemr2d", "tran") else rng.choice(["col", "col", "row"]), **extra))

    general = entry == "transform" and rng.random() < 0.3
    if general:
        case["ranks"] = pr * pc
        case.update({"s_cuts": rng.randrange(1, 40), "s_seed": rng.randrange(1 << 30),
                     "s_store": rng.choice(["col", "col", "row"])})
    else:
        side("s", *((m, n) if op == "N" else (n, m)))
    side("t", m, n)
    if entry == "transform":
        case["relabel"] = rng.random() < 0.3
    return case
