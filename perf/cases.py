"""The measured work: builds, solves and products of close-coupling Hamiltonians.

Each case is one call (or the two calls of a step) that a user of this
framework makes: `build` (the contracted matrix), `solve` (its lowest
eigenpairs), `step` (both, the benchmark's unit), `batch` (many instances in
one replay), `eig` (every eigenpair of a dense matrix) and `apply` (H V). The
sizes are the repository's own workloads, with ragged ones between them.
Inputs follow the laws of the repository's generator (decaying random
integrals, CISD-like determinant spaces, random orthonormal CI vectors), drawn
here on the GPU from the seed alone.
"""
import itertools
import math
import random

import numpy as np
import torch

import paper_1709_03005_amd as cc

SD2 = 0.1   # standard deviation of the two-electron integrals before their decay


def listed():
    return [
        # the smallest whole build (D = 110): launches and latency
        dict(name="build_tiny", kind="build", n_o=10, n_elec=6, n_irrep=1, n_c=20, n_sym=1, dets=40, states=3, l2=50),
        # odd sizes, two irreps, two-word determinants (D = 4815)
        dict(name="build_ragged", kind="build", n_o=36, n_elec=8, n_irrep=2, n_c=101, n_sym=2, dets=611, states=9,
             l2=2997),
        # the usual size of the repository's tests and benchmark: four symmetries (D = 8000)
        dict(name="build_medium", kind="build", n_o=30, n_elec=10, n_irrep=4, n_c=150, n_sym=4, dets=500, states=5,
             l2=5000),
        # a large contracted part: 8000 target determinants, 40 states (D = 40000)
        dict(name="build_precision", kind="build", n_o=40, n_elec=12, n_irrep=1, n_c=300, n_sym=1, dets=8000,
             states=40, l2=28000),
        # the reduced-precision option of the expansion, three slices (D = 20000)
        dict(name="build_bf16x3", kind="build", n_o=40, n_elec=12, n_irrep=1, n_c=300, n_sym=1, dets=4000, states=20,
             l2=14000, slices=3),
        # many uneven instances built together (symmetry-packed integrals, D from 500 to 6000)
        dict(name="batch_16", kind="batch", count=16, shapes=400),
        # the lowest ten pairs of a built matrix of ordinary size, vectors to the host (D = 8000)
        dict(name="solve_medium", kind="solve", n_o=30, n_elec=10, n_irrep=2, n_c=150, n_sym=2, dets=500, states=10,
             l2=5000, k=10, rounds=20),
        # the benchmark's step: build and lowest ten eigenvalues (D = 60000)
        dict(name="step_large", kind="step", n_o=40, n_elec=12, n_irrep=1, n_c=400, n_sym=1, dets=8000, states=50,
             l2=40000, k=10, rounds=58),
        # an L2-heavy matrix with classes 2 and 8 as CSR, build and solve (D = 50712)
        dict(name="step_sparse", kind="step", n_o=40, n_elec=12, n_irrep=1, n_c=178, n_sym=1, dets=2000, states=4,
             l2=50000, k=10, rounds=50, sparse=True),
        # a whole spectrum where launches count
        dict(name="eig_small", kind="eig", n=301),
        # a whole spectrum of the usual built size
        dict(name="eig_large", kind="eig", n=8000),
        # the product that an iterative solver of the user's own makes (device vectors, D = 24011)
        dict(name="apply_block", kind="apply", n_o=36, n_elec=10, n_irrep=1, n_c=201, n_sym=1, dets=300, states=11,
             l2=21800, b=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _space(n_o, na, nb):
    """Determinants within a double substitution of the aufbau reference."""
    va, vb = n_o - na, n_o - nb
    return (1 + na * va + nb * vb + math.comb(na, 2) * math.comb(va, 2) + math.comb(nb, 2) * math.comb(vb, 2)
            + na * va * nb * vb)


def _shape(rng, d_lo, d_hi, ni=(1, 2, 4), states=(2, 40), cc_bytes=2 << 30, most_dets=4000):
    while True:
        n_o, n_elec, n_irrep = rng.randint(10, 40), rng.choice([4, 6, 8, 10, 12]), rng.choice(ni)
        if n_elec // 2 + 1 > n_o - 2:
            continue
        n_c, s, d = _log(rng, 12, 300), _log(rng, *states), _log(rng, d_lo, d_hi)
        l2 = d - n_irrep * s * n_c
        na = n_elec // 2
        m = min(int(0.6 * _space(n_o, na, na) / n_irrep), _log(rng, 2 * s, 40 * s), most_dets)
        if l2 < 20 or l2 > 0.6 * _space(n_o, na + 1, na) / n_irrep or m < s:
            continue
        if 8 * (n_o * n_irrep * n_c) ** 2 > cc_bytes:
            continue
        return dict(n_o=n_o, n_elec=n_elec, n_irrep=n_irrep, n_c=n_c, n_sym=n_irrep, dets=m, states=s, l2=l2)


def draw(rng):
    kind = rng.choice(["build", "build", "build", "split", "batch", "solve", "solve", "step", "sparse", "eig", "eig",
                       "apply"])
    if kind == "build":
        return dict(kind="build", **_shape(rng, 110, 40000))
    if kind == "split":
        return dict(kind="build", slices=rng.randint(2, 4), **_shape(rng, 500, 12000, ni=(1, 2)))
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(3, 16), shapes=rng.randint(0, 1 << 20))
    if kind == "solve":
        d = _shape(rng, 600, 20000, cc_bytes=1 << 29, most_dets=1000)
        return dict(kind="solve", k=rng.randint(3, 10), rounds=20, **d)
    if kind == "step":
        return dict(kind="step", k=rng.randint(5, 10), rounds=25, **_shape(rng, 2000, 40000, cc_bytes=1 << 30))
    if kind == "sparse":
        d = _shape(rng, 4000, 40000, ni=(1, 2), states=(2, 6), cc_bytes=1 << 29, most_dets=1500)
        return dict(kind="step", k=rng.randint(5, 10), rounds=30, sparse=True, **d)
    if kind == "eig":
        return dict(kind="eig", n=_log(rng, 100, 6000))
    d = _shape(rng, 1000, 30000, cc_bytes=1 << 29, most_dets=400)
    return dict(kind="apply", b=rng.randint(1, 16), **d)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Input:
    """What a user's program holds before the call (the fields that
    paper_1709_03005_amd.from_instance reads)."""
    total_irrep, e_core, packed, l2_csf_start = 0, 0.25, False, None


class _Sym:
    def __init__(self, irrep, dets, ci):
        self.irrep, self.dets, self.ci = irrep, dets, ci


def _substituted(n_o, n_e, level):
    """Orbital masks of `level`-fold substitutions of the aufbau string, and the orbitals' parity by irrep bit."""
    ref = (1 << n_e) - 1
    holes = [sum(1 << o for o in c) for c in itertools.combinations(range(n_e), level)]
    parts = [sum(1 << o for o in c) for c in itertools.combinations(range(n_e, n_o), level)]
    h, p = np.array(holes, dtype=np.uint64), np.array(parts, dtype=np.uint64)
    return (np.uint64(ref) ^ h[:, None] ^ p[None, :]).ravel()


def _det_space(rng, n_o, na, nb, tgt_irrep, n_irrep, irrep, count):
    """`count` determinants of one irrep by substitution level from the aufbau reference, in seeded order within a
    level, as 64-bit words over the spin-orbitals 2 * orbital + spin."""
    def irreps(masks):
        r = np.zeros(masks.size, np.int64)
        for o in range(n_o):
            r ^= ((masks >> np.uint64(o)) & np.uint64(1)).astype(np.int64) * int(tgt_irrep[o])
        return r
    got_a, got_b, have, level = [], [], 0, 0
    while have < count:
        if level > na + nb:
            raise ValueError("determinant space too small")
        la, lb = [], []
        for x in range(level + 1):
            if x > min(na, n_o - na) or level - x > min(nb, n_o - nb):
                continue
            sa, sb = _substituted(n_o, na, x), _substituted(n_o, nb, level - x)
            i, j = np.nonzero((irreps(sa)[:, None] ^ irreps(sb)[None, :]) == irrep)
            la.append(sa[i])
            lb.append(sb[j])
        a, b = np.concatenate(la), np.concatenate(lb)
        order = rng.permutation(a.size)[:count - have]
        got_a.append(a[order])
        got_b.append(b[order])
        have += order.size
        level += 1
    a, b = np.concatenate(got_a), np.concatenate(got_b)
    dets = np.zeros((count, (2 * n_o + 63) // 64), np.uint64)
    one = np.uint64(1)
    for o in range(n_o):
        dets[:, (2 * o) // 64] |= ((a >> np.uint64(o)) & one) << np.uint64((2 * o) % 64)
        dets[:, (2 * o) // 64] |= ((b >> np.uint64(o)) & one) << np.uint64((2 * o + 1) % 64)
    return dets


def _integrals(inp, gen, dev):
    """Real integrals with their permutational symmetries, decay and symmetry zeros, on `dev`."""
    n_o, nc = inp.n_o, int(inp.n_c.sum())
    n = n_o + nc
    f = dict(dtype=torch.float64, device=dev)
    irr = torch.from_numpy(np.concatenate([inp.tgt_irrep, np.repeat(np.arange(inp.n_irrep), inp.n_c)])).to(dev).long()
    g = torch.arange(n, **f)

    def randn(*shape):
        return torch.randn(*shape, generator=gen, **f)
    dec = torch.exp(-(g[:, None] - g[None, :]).abs() / 4)
    x = randn(n, n)
    inp.h = (x + x.T) / math.sqrt(2) * dec * (irr[:, None] == irr[None, :])
    t, c = slice(0, n_o), slice(n_o, n)
    pair = irr[:, None] ^ irr[None, :]
    x = randn(n_o, n_o, n_o, n_o)
    x = (x + x.transpose(0, 1)) / math.sqrt(2)
    x = (x + x.transpose(2, 3)) / math.sqrt(2)
    x = (x + x.permute(2, 3, 0, 1)) / math.sqrt(2)
    inp.tttt = SD2 * x * dec[t, t][:, :, None, None] * dec[t, t] * (pair[t, t][:, :, None, None] == pair[t, t])
    x = randn(n_o, n_o, n_o, nc)
    x = (x + x.transpose(0, 1)) / math.sqrt(2)
    inp.tttc = SD2 * x * dec[t, t][:, :, None, None] * dec[t, c] * (pair[t, t][:, :, None, None] == pair[t, c])
    # in place from here on: these two are the large ones
    x = randn(n_o, n_o, nc, nc)
    w = dec[c, c] * SD2
    for p in range(n_o):
        for q in range(p + 1):
            y = x[p, q]
            y = (y + y.T).mul_(w * (math.exp(-(p - q) / 4) / math.sqrt(2)))
            x[p, q] = y
            if p != q:
                x[q, p] = y
    x *= (pair[t, t][:, :, None, None] == pair[c, c])
    inp.ttcc = x
    x = randn(n_o, nc, n_o, nc)
    for p in range(n_o):
        x[p, :, p, :] = (x[p, :, p, :] + x[p, :, p, :].T) / math.sqrt(2)
        for q in range(p):
            x[q, :, p, :] = x[p, :, q, :].T
    x *= (SD2 * dec[t, c])[:, :, None, None]
    x *= dec[t, c]
    x *= (pair[t, c][:, :, None, None] == pair[t, c])
    inp.tctc = x


def _pack(inp):
    """(tt|cc) and (tc|tc) in the symmetry-packed layout that cch_set_integrals_packed documents."""
    n_o, nc, ni = inp.n_o, inp.n_c.astype(np.int64), inp.n_irrep
    n = int(nc.sum())
    cs = np.concatenate([[0], np.cumsum(nc)])
    pair_x = (inp.tgt_irrep[:, None] ^ inp.tgt_irrep[None, :]).ravel()
    at = []
    for x in range(ni):
        at.append(np.concatenate([(np.arange(cs[a], cs[a + 1])[:, None] * n + np.arange(cs[a ^ x], cs[(a ^ x) + 1])
                                   [None, :]).ravel() for a in range(ni)]))
    rec = np.concatenate([[0], np.cumsum([at[x].size for x in pair_x])])
    out = []
    for v in (inp.ttcc, inp.tctc.permute(0, 2, 1, 3)):
        v = v.reshape(n_o * n_o, n * n)
        o = torch.empty(int(rec[-1]), dtype=torch.float64, device=v.device)
        for x in range(ni):
            pairs = np.nonzero(pair_x == x)[0]
            if pairs.size and at[x].size:
                idx = torch.from_numpy(at[x]).to(v.device)
                to = torch.from_numpy(rec[pairs]).to(v.device)[:, None] + torch.arange(at[x].size, device=v.device)
                o[to] = v[torch.from_numpy(pairs).to(v.device)][:, idx]
        out.append(o)
    inp.ttcc, inp.tctc = out
    inp.packed = True


def make_input(case, seed, device="cuda", packed=False):
    dev = torch.device(device)
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * seed + 17)
    rng = np.random.default_rng(seed)
    inp = _Input()
    inp.n_o, inp.n_elec, inp.n_irrep = case["n_o"], case["n_elec"], case["n_irrep"]
    inp.tgt_irrep = (np.arange(inp.n_o) % inp.n_irrep).astype(np.uint8)
    # irreps beyond the first hold a few continuum orbitals fewer when the size is odd
    inp.n_c = np.array([case["n_c"] - (a if case["n_c"] % 2 else 0) for a in range(inp.n_irrep)], np.int32)
    _integrals(inp, gen, dev)
    if packed:
        _pack(inp)
    na = inp.n_elec // 2
    inp.syms = []
    for a in range(case["n_sym"]):
        dets = _det_space(rng, inp.n_o, na, na, inp.tgt_irrep, inp.n_irrep, a, case["dets"])
        q, _ = np.linalg.qr(rng.standard_normal((case["dets"], case["states"])))
        inp.syms.append(_Sym(a, dets, np.ascontiguousarray(q)))
    inp.l2_dets = _det_space(rng, inp.n_o, na + 1, na, inp.tgt_irrep, inp.n_irrep, 0, case["l2"])
    return inp


def _dim(case):
    return case["l2"] + case["states"] * sum(case["n_c"] - (a if case["n_c"] % 2 else 0) for a in range(case["n_sym"]))


def _batch_shapes(case):
    """The instances of one batch: the repository's batching ranges (D from 500 to 6000, 12 to 40 orbitals, one, two
    or four symmetries, 5 to 30 states, 50 to 200 continuum orbitals)."""
    rng, got = random.Random(case["shapes"]), []
    while len(got) < case["count"]:
        d, n_o, ni, s = rng.randint(500, 6000), rng.randint(12, 40), rng.choice([1, 2, 4]), rng.randint(5, 30)
        n_c, n_elec = rng.randint(50, 200), rng.choice([4, 6, 8, 10, 12])
        l2, na = d - ni * s * n_c, n_elec // 2
        m = rng.randint(2 * s, 8 * s)
        if l2 < 1 or na + 1 > n_o - 2 or 8 * (n_o * ni * n_c) ** 2 > (1 << 30):
            continue
        if l2 > 0.6 * _space(n_o, na + 1, na) / ni or m > 0.6 * _space(n_o, na, na) / ni:
            continue
        got.append(dict(n_o=n_o, n_elec=n_elec, n_irrep=ni, n_c=n_c, n_sym=ni, dets=m, states=s, l2=l2))
    return got


# ---------------------------------------------------------------------------
# the measured calls
# ---------------------------------------------------------------------------

class _Matrix:
    """The resident matrix of a context, shared with torch; it keeps the context alive."""

    def __init__(self, ctx):
        self.ctx = ctx
        ptr, ld = ctx.matrix_device()
        d, _ = ctx.dim()
        self.__cuda_array_interface__ = dict(shape=(d, d), strides=(8 * ld, 8), typestr="<f8", data=(ptr, False),
                                             version=2)


def _matrix(ctx):
    return torch.as_tensor(_Matrix(ctx), device="cuda")


def _context(case, seed, packed=False):
    plan = {}
    if case.get("slices"):
        plan = dict(precision=cc.CCH_PREC_SPLIT_BF16, split_slices=case["slices"])
    if case.get("sparse"):
        plan = dict(sparse_l2=True)
    return cc.from_instance(make_input(case, seed, packed=packed), device=0,
                            stream=torch.cuda.current_stream().cuda_stream, **plan)


def _spectrum_input(case, seed, device="cuda"):
    gen = torch.Generator(device=device)
    gen.manual_seed(7919 * seed + 5)
    n = case["n"]
    x = torch.randn(n, n, generator=gen, dtype=torch.float64, device=device)
    a = (x + x.T) / math.sqrt(2 * n)
    a.diagonal().add_(torch.linspace(-1, 1, n, dtype=torch.float64, device=device))
    return a, torch.randn(n, generator=gen, dtype=torch.float64, device=device)


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "eig":
        s["A"], s["ref"] = _spectrum_input(case, seed)
        s["ctx"] = cc.Context(0, torch.cuda.current_stream().cuda_stream)
        return s
    if case["kind"] == "batch":
        s["ctxs"] = [_context(c, 1000 * seed + i, packed=True) for i, c in enumerate(_batch_shapes(case))]
        s["batch"] = cc.Batch(s["ctxs"], autotune=True)
        return s
    s["ctx"] = _context(case, seed)
    d = _dim(case)
    s["ref"] = np.random.default_rng(seed + 1).standard_normal(d)
    if case["kind"] in ("solve", "apply"):
        s["ctx"].build()
    if case["kind"] == "apply":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        s["V"] = torch.randn(case["b"], d, generator=gen, dtype=torch.float64, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "build":
        s["ctx"].build()
        if "H" not in s:
            s["H"] = _matrix(s["ctx"])
        return s["H"]
    if kind == "batch":
        s["batch"].build()
        if "H" not in s:
            s["H"] = [_matrix(c) for c in s["ctxs"]]
        return s["H"]
    if kind == "eig":
        w, v, _ = s["ctx"].eig_all(s["A"], device=True)
        # an eigenvector's sign is free: the program's own convention
        v *= torch.sign(v @ s["ref"])[:, None]
        return dict(w=w, v=v)
    if kind == "apply":
        v = s["V"]
        w = torch.empty_like(v)
        s["ctx"]._ck(cc.lib.cch_apply(s["ctx"].h, v.data_ptr(), v.shape[1], v.shape[0], w.data_ptr(), w.shape[1],
                                      cc.CCH_MEM_DEVICE))
        return w
    ctx, k = s["ctx"], case["k"]
    if kind == "solve":
        ev, vec, _, _ = ctx.davidson(k, tol=1e-8)
        vec *= np.sign(vec @ s["ref"])[:, None]
        return dict(ev=ev, vec=vec)
    ctx.build()
    ev, _, _, _ = ctx.davidson(k, tol=1e-8, want_vectors=False)
    if case.get("sparse"):
        return dict(ev=ev, diagonal=ctx.get_diagonal())
    if "H" not in s:
        s["H"] = _matrix(ctx)
    return dict(ev=ev, H=s["H"])


# ---------------------------------------------------------------------------
# the work of one pass
# ---------------------------------------------------------------------------

def _build_work(case):
    d = _dim(case)
    nc = [case["n_c"] - (a if case["n_c"] % 2 else 0) for a in range(case["n_irrep"])]
    n_o, ni, s = case["n_o"], case["n_irrep"], case["states"]
    slots = n_o * n_o / ni
    # one multiply-add of each distinct two-continuum integral with its density
    flops = 0.0
    for a in range(case["n_sym"]):
        for b in range(a + 1):
            rows = s * (s + 1) / 2 if a == b else s * s
            distinct = nc[a] * nc[b] * slots * (0.25 + 0.5 if a == b else 0.5 + 1.0)
            flops += 2 * rows * distinct
    ints = 8.0 * (n_o ** 4 / ni + n_o ** 3 * sum(nc) / ni + 2 * n_o * n_o * sum(x * x for x in nc))
    dense = 8.0 * (d * d if not case.get("sparse") else 2 * d * (d - case["l2"]))
    return dict(bytes=ints + dense, flops=flops)


def work(case):
    if case["kind"] == "eig":
        n = float(case["n"])
        return dict(bytes=16 * n * n + 8 * n, flops=4 / 3 * n ** 3 + 2 * n ** 3)
    if case["kind"] == "batch":
        w = [_build_work(c) for c in _batch_shapes(case)]
        return dict(bytes=sum(x["bytes"] for x in w), flops=sum(x["flops"] for x in w))
    d = _dim(case)
    if case["kind"] == "apply":
        return dict(bytes=4.0 * d * (d + 1) + 16.0 * case["b"] * d, flops=2.0 * case["b"] * d * d)
    w = dict(bytes=0.0, flops=0.0) if case["kind"] == "solve" else _build_work(case)
    if "rounds" in case:   # each round of the solver multiplies k vectors by the matrix
        c = d - case["l2"]
        size = d * d / 2 if not case.get("sparse") else 2 * d * c
        w["bytes"] += case["rounds"] * 8.0 * size
        w["flops"] += case["rounds"] * 4.0 * case["k"] * size
    return w


# ---------------------------------------------------------------------------
# the same results in 64 bits from the definitions
# ---------------------------------------------------------------------------

def _occ(dets, n_o, dev):
    bits = np.stack([(dets[:, k // 64] >> np.uint64(k % 64)) & np.uint64(1) for k in range(2 * n_o)], 1)
    return torch.from_numpy(bits.astype(np.int64)).to(dev)


def _between(cum, lo, hi):
    """Occupied spin-orbitals strictly between lo and hi (cum: occupied up to and including each)."""
    a, b = torch.minimum(lo, hi), torch.maximum(lo, hi)
    c = torch.gather(cum, 1, (b - 1).clamp(min=0)[:, None]) - torch.gather(cum, 1, a[:, None])
    return torch.where(b - a > 1, c[:, 0], torch.zeros_like(a))


def _first_two(x):
    i = x.argmax(1)
    y = x.clone()
    y[torch.arange(len(y), device=y.device), i] = 0
    return i, y.argmax(1)


def _excitations(A, B, x, y):
    """Holes, particles and sign of the pairs (x of A as bra, y of B as ket)."""
    a, b = A[x], B[y]
    h1, h2 = _first_two(b * (1 - a))
    p1, p2 = _first_two(a * (1 - b))
    cum = torch.cumsum(b, 1)
    c1 = _between(cum, h1, p1)
    c2 = _between(cum, h2, p2)
    lo, hi = torch.minimum(h2, p2), torch.maximum(h2, p2)
    c2 = c2 - ((h1 > lo) & (h1 < hi)).long() + ((p1 > lo) & (p1 < hi)).long()
    return h1, h2, p1, p2, c1, c2


def _slater(inp, A, B):
    """<A|H|B> over target orbitals, dense, and the list of single substitutions (x, y, P, Q, spin, sign)."""
    n_o, dev = inp.n_o, A.device
    h, g = inp.h[:n_o, :n_o].to(dev), inp.tttt.to(dev)
    out = torch.zeros(len(A), len(B), dtype=torch.float64, device=dev)
    ne = int(A[0].sum())
    jj = torch.einsum("ppqq->pq", g).contiguous()
    kk = torch.einsum("pqqp->pq", g).contiguous()
    g1 = torch.einsum("phkk->phk", g).contiguous()
    g2 = torch.einsum("pkkh->phk", g).contiguous()
    singles = []
    Bf = B.to(torch.float32)
    for r in range(0, len(A), 512):
        deg = ne - torch.round(A[r:r + 512].to(torch.float32) @ Bf.T).long()
        x, y = torch.nonzero(deg <= 2, as_tuple=True)
        d = deg[x, y]
        x = x + r
        i = d == 0
        if i.any():
            na, nb = A[x[i]][:, 0::2].double(), A[x[i]][:, 1::2].double()
            n = na + nb
            e = inp.e_core + n @ torch.diagonal(h) + 0.5 * ((n @ jj) * n).sum(1)
            e -= 0.5 * (((na @ kk) * na).sum(1) + ((nb @ kk) * nb).sum(1))
            out[x[i], y[i]] = e
        i = d == 1
        if i.any():
            h1, _, p1, _, c1, _ = _excitations(A, B, x[i], y[i])
            P, H, sp = p1 // 2, h1 // 2, p1 % 2
            ok = sp == h1 % 2
            na, nb = B[y[i]][:, 0::2].double(), B[y[i]][:, 1::2].double()
            same = torch.where(sp[:, None] == 0, na, nb)
            v = h[P, H] + (g1[P, H] * (na + nb)).sum(1) - (g2[P, H] * same).sum(1)
            sign = 1.0 - 2.0 * (c1 % 2)
            out[x[i], y[i]] = torch.where(ok, sign * v, torch.zeros_like(v))
            singles.append([t[ok] for t in (x[i], y[i], P, H, sp, sign)])
        i = d == 2
        if i.any():
            h1, h2, p1, p2, c1, c2 = _excitations(A, B, x[i], y[i])
            s = [t % 2 for t in (h1, h2, p1, p2)]
            H1, H2, P1, P2 = h1 // 2, h2 // 2, p1 // 2, p2 // 2
            v = g[P1, H1, P2, H2] * ((s[2] == s[0]) & (s[3] == s[1]))
            v = v - g[P1, H2, P2, H1] * ((s[2] == s[1]) & (s[3] == s[0]))
            out[x[i], y[i]] = (1.0 - 2.0 * ((c1 + c2) % 2)) * v
    if not singles:
        return out, None
    return out, [torch.cat(t) for t in zip(*singles)]


def exact_matrix(inp, device="cuda"):
    """The contracted matrix from its definition (Slater's rules, one dense sum per pair of symmetries)."""
    dev = torch.device(device)
    n_o = inp.n_o
    cs = np.concatenate([[0], np.cumsum(inp.n_c)])
    occ = [_occ(s.dets, n_o, dev) for s in inp.syms]
    ci = [torch.from_numpy(s.ci).to(dev) for s in inp.syms]
    hc = inp.h.to(dev)
    row, at = 0, []
    for s in inp.syms:
        at.append(row)
        row += s.ci.shape[1] * int(inp.n_c[s.irrep])
    D = row + len(inp.l2_dets)
    M = torch.zeros(D, D, dtype=torch.float64, device=dev)
    for a, sa in enumerate(inp.syms):
        for b in range(a + 1):
            sb = inp.syms[b]
            ja, jb = slice(cs[sa.irrep], cs[sa.irrep + 1]), slice(cs[sb.irrep], cs[sb.irrep + 1])
            Sa, Sb, nca, ncb = ci[a].shape[1], ci[b].shape[1], ja.stop - ja.start, jb.stop - jb.start
            ht, one = _slater(inp, occ[a], occ[b])
            dens = torch.zeros(2, n_o * n_o, Sa * Sb, dtype=torch.float64, device=dev)   # all spins, alpha
            for i in range(0, len(one[0]) if one else 0, 4096):
                x, y, P, Q, sp, sg = (t[i:i + 4096] for t in one)
                v = (sg[:, None, None] * ci[a][x][:, :, None] * ci[b][y][:, None, :]).reshape(len(x), -1)
                dens[0].index_add_(0, P * n_o + Q, v)
                dens[1].index_add_(0, (P * n_o + Q)[sp == 0], v[sp == 0])
            over = None
            if a == b:
                both = (ci[a][:, :, None] * ci[a][:, None, :]).reshape(len(ci[a]), -1)
                o = occ[a].double()
                diag = torch.arange(n_o, device=dev) * (n_o + 1)
                dens[0][diag] += (o[:, 0::2] + o[:, 1::2]).T @ both
                dens[1][diag] += o[:, 0::2].T @ both
                over = ci[a].T @ ci[a]
            J = inp.ttcc.to(dev)[:, :, ja, jb].reshape(n_o * n_o, nca * ncb)
            K = inp.tctc.to(dev)[:, jb, :, ja].permute(0, 2, 3, 1).reshape(n_o * n_o, nca * ncb)
            blk = (dens[0].T @ J - dens[1].T @ K).reshape(Sa, Sb, nca, ncb)
            if ja == jb:
                blk += (ci[a].T @ ht @ ci[b])[:, :, None, None] * torch.eye(nca, dtype=torch.float64, device=dev)
            if over is not None:
                blk += over[:, :, None, None] * hc[n_o:, n_o:][ja, jb]
            blk = blk.permute(0, 2, 1, 3).reshape(Sa * nca, Sb * ncb)
            M[at[a]:at[a] + Sa * nca, at[b]:at[b] + Sb * ncb] = blk
            M[at[b]:at[b] + Sb * ncb, at[a]:at[a] + Sa * nca] = blk.T
    L = _occ(inp.l2_dets, n_o, dev)
    M[row:, row:] = _slater(inp, L, L)[0]
    t3 = inp.tttc.to(dev)
    kkh = torch.einsum("kkhj->khj", t3).contiguous()   # (KK|H j)
    khk = torch.einsum("khkj->khj", t3).contiguous()   # (KH|K j)
    top = 2 * n_o
    for a, sa in enumerate(inp.syms):
        j = slice(cs[sa.irrep], cs[sa.irrep + 1])
        nc, S = j.stop - j.start, ci[a].shape[1]
        out = torch.zeros(len(L), S * nc, dtype=torch.float64, device=dev)
        T = occ[a]
        N = int(T[0].sum())
        for r in range(0, len(L), 256):
            deg = N + 1 - torch.round(L[r:r + 256].to(torch.float32) @ T.to(torch.float32).T).long()
            lx, ty = torch.nonzero(deg <= 2, as_tuple=True)
            d = deg[lx, ty]
            step = max(1, (1 << 27) // max(1, S * nc))
            for i0 in range(0, len(lx), step):
                x, y, dd = lx[i0:i0 + step] + r, ty[i0:i0 + step], d[i0:i0 + step]
                l, t = L[x], T[y]
                h1, h2 = _first_two(l * (1 - t))
                pt = (t * (1 - l)).argmax(1)
                cum = torch.cumsum(l, 1)
                v = torch.zeros(len(x), nc, dtype=torch.float64, device=dev)
                i = torch.nonzero(dd == 1)[:, 0]
                if len(i):
                    H = h1[i] // 2
                    na, nb = t[i][:, 0::2].double(), t[i][:, 1::2].double()
                    w = hc[n_o:, :n_o][j].T[H].clone()
                    for k in range(n_o):
                        w += (na + nb)[:, k:k + 1] * kkh[k][:, j][H] - na[:, k:k + 1] * khk[k][:, j][H]
                    above = N + 1 - torch.gather(cum[i], 1, h1[i][:, None])[:, 0]
                    v[i] = (1.0 - 2.0 * (above % 2))[:, None] * w * (h1[i] % 2 == 0)[:, None]
                i = torch.nonzero(dd == 2)[:, 0]
                if len(i):
                    a1, a2, p = h1[i], h2[i], pt[i]
                    c = _between(cum[i], a1, p)
                    # above a2 after a1 has left and p has come in
                    c = c + N + 1 - torch.gather(cum[i], 1, a2[:, None])[:, 0] + (p > a2).long()
                    w = t3[p // 2, a1 // 2, a2 // 2][:, j] * ((p % 2 == a1 % 2) & (a2 % 2 == 0))[:, None]
                    w = w - t3[p // 2, a2 // 2, a1 // 2][:, j] * ((p % 2 == a2 % 2) & (a1 % 2 == 0))[:, None]
                    v[i] = (1.0 - 2.0 * (c % 2))[:, None] * w
                out.index_add_(0, x, (ci[a][y][:, :, None] * v[:, None, :]).reshape(len(x), -1))
        M[row:, at[a]:at[a] + S * nc] = out
        M[at[a]:at[a] + S * nc, row:] = out.T
    assert top == L.shape[1]
    return M


def _small(case):
    return (case["l2"] <= 6000 and case["dets"] <= 1000 and _dim(case) <= 9000
            and 8 * (case["n_o"] * case["n_irrep"] * case["n_c"]) ** 2 <= 3 << 30)


def exact(case, seed):
    kind = case["kind"]
    if kind == "eig":
        if case["n"] > 2500:
            return None
        a, ref = _spectrum_input(case, seed)
        w, v = np.linalg.eigh(a.cpu().numpy())
        v = np.ascontiguousarray(v.T)
        return dict(w=w, v=v * np.sign(v @ ref.cpu().numpy())[:, None])
    if kind == "batch" or not _small(case):
        return None
    m = exact_matrix(make_input(case, seed))
    if kind == "build":
        return m
    if kind == "apply":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        return torch.randn(case["b"], len(m), generator=gen, dtype=torch.float64, device="cuda") @ m
    if len(m) > 2500:
        return dict(ev=None, H=m) if kind == "step" and not case.get("sparse") else None
    w, v = np.linalg.eigh(m.cpu().numpy())
    if kind == "solve":
        v = np.ascontiguousarray(v.T[:case["k"]])
        ref = np.random.default_rng(seed + 1).standard_normal(len(m))
        return dict(ev=w[:case["k"]], vec=v * np.sign(v @ ref)[:, None])
    if case.get("sparse"):
        return dict(ev=w[:case["k"]], diagonal=torch.diagonal(m).clone())
    return dict(ev=w[:case["k"]], H=m)
