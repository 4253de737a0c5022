"""The work that programs have this library do, as cases that can be timed.

Every case runs on a level-structured symmetric matrix of the benchmark's recipe (levels coupled to
themselves and to their neighbours, diagonal 10 level + U(-1, 1), floor(d/2) draws N(0, 0.5^2) per
row, values rounded to float32), drawn on the GPU from the seed.  Kinds:

  spmm    Y = H X through a context (sppc_spmm): the cost unit of the method
  basis   E = (I - Q Q^T) Psi (sppc_mpnn_target): the passes over a tall-skinny basis
  train   the learned preconditioner's forward, loss and gradient (sppc_mpnn_eval with targets)
  solve   context, whole solve and release, from the matrix to eigenpairs (sppc_setup, sppc_solve)
"""
import json
import math
import os

import torch

import paper_2407_08901_amd as P

_DEV = "cuda"
_PKG = os.path.dirname(os.path.abspath(P.__file__))


def listed():
    l3 = "100/800/4000"                      # the three-level shape of the tests, smoke run and training set
    l4_tenth = "200/2000/15000/100000"       # the four-level training shape
    l4 = "2000/20000/150000/1000000"         # the four-level benchmark shape
    l5_20th = "100/1000/10000/75000/300000"             # the five-level training shape
    l5 = "2000/20000/200000/1500000/6000000"            # the five-level benchmark shape (bench.py's default)
    return [
        # one product on the smallest matrix anybody solves here: launch and latency
        dict(name="spmm-4900-b4", kind="spmm", levels=l3, d=60, small=1, k=4, b=4, x="f64", val="f32"),
        # a medium matrix whose values do not fit float32 (the float64 store)
        dict(name="spmm-117k-b8-val64", kind="spmm", levels=l4_tenth, d=200, small=2, k=8, b=8, x="f64", val="f64"),
        # the product of every step of the plain float64 solve, k = 8
        dict(name="spmm-1.17M-b8", kind="spmm", levels=l4, d=200, small=2, k=8, b=8, x="f64", val="f32"),
        # the product of the mixed form's early steps, k = 16
        dict(name="spmm-1.17M-b16-x32", kind="spmm", levels=l4, d=200, small=2, k=16, b=16, x="f32", val="f32"),
        # one vector: a single pair (Algorithm 1), or the last unconverged pair of a continuation
        dict(name="spmv-1.17M", kind="spmm", levels=l4, d=200, small=2, k=1, b=1, x="f64", val="f32"),
        # a wide block of odd width on ragged levels (up to 32 columns a call: samples of the network,
        # blocks of other solvers)
        dict(name="spmm-772k-b27", kind="spmm", levels="211/2003/20011/150007/600011", d=300, small=2, k=16,
             b=27, x="f64", val="f32"),
        # the benchmark's own matrix at full size, float64 X (half of its products; all of plain float64's)
        dict(name="spmm-7.72M-b16", kind="spmm", levels=l5, d=300, small=2, k=16, b=16, x="f64", val="f32"),
        # the projection out of a basis of 16 steps of k = 8
        dict(name="basis-1.17M-m128", kind="basis", levels=l4, d=200, small=2, k=8, m=128, S=8),
        # a training step's gradient on the three-level training set (basis target, as the trainer calls it)
        dict(name="train-4900", kind="train", levels=l3, d=60, small=1, k=4, m=48, S=4),
        # the same on the five-level training set (pair target: no basis), all 16 pairs
        dict(name="train-386k", kind="train", levels=l5_20th, d=300, small=2, k=16, m=0, S=16),
        # a whole solve with the defaults on the smallest matrix: latency, host path
        dict(name="solve-4900", kind="solve", levels=l3, d=60, small=1, k=4, mode="plain"),
        # a whole solve of the four-level benchmark in the mixed SPPC + RMM-DIIS form
        dict(name="solve-1.17M", kind="solve", levels=l4, d=200, small=2, k=8, mode="mixed+rmmdiis"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of the ranges above: 3 to 5 levels of any sizes, every width, type and storage."""
    kind = rng.choice(["spmm", "spmm", "spmm", "spmm", "basis", "train", "solve"])
    top = {"spmm": 7.0e6, "basis": 1.4e6, "train": 4.5e5, "solve": 1.2e6}[kind]
    n = _log(rng, 4500, top)
    L = 3 if n < 2e4 else 4 if n < 2.5e5 else rng.choice([4, 5])
    ratio = _log(rng, 5.0, 8.0)              # size of a level against the one before
    levels = [max(60, int(n * (ratio - 1) / (ratio ** L - 1) * ratio ** i * rng.uniform(0.9, 1.1))) for i in range(L)]
    small = 1 if L == 3 else 2
    d = rng.randint(48, 90) if L == 3 else rng.randint(150, 300)
    k = rng.choice([1, 2, 3, 4, 5, 8, 11, 16]) if kind == "spmm" else rng.randint(4, 8) if L == 3 else rng.randint(4, 16)
    c = dict(kind=kind, levels="/".join(map(str, levels)), d=d, small=small, k=k)
    if kind == "spmm":
        big = n > 2.5e6
        c["b"] = rng.choice([1, 2, 3, 4, 5, 7, 8, 11, 13, 16] if big else
                            [1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 20, 24, 27, 31, 32])
        c["x"] = rng.choice(["f64", "f64", "f32"])
        c["val"] = "f32" if c["x"] == "f32" or big else rng.choice(["f32", "f32", "f64"])
    elif kind == "basis":
        c["S"] = rng.randint(1, 32)
        c["m"] = rng.randint(3, 256 if n < 4e5 else 160)
    elif kind == "train":
        c["S"] = rng.randint(1, k)
        c["m"] = rng.choice([0, rng.randint(max(4, c["S"]), 128)])
    else:
        c["mode"] = rng.choice(["plain", "mixed+rmmdiis"])
    return c


# ------------------------------------------------------------------------------------------ inputs


def _gen(seed, salt):
    g = torch.Generator(device=_DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _levels(case):
    return [int(x) for x in case["levels"].split("/")]


def _offsets(levels):
    off = [0]
    for s in levels:
        off.append(off[-1] + int(s))
    return off


def _matrix(levels, d, seed, wide):
    """Upper CSR (row_ptr int64, col int32, val) on the GPU; wide: values that need float64."""
    g = _gen(seed, 1)
    off = _offsets(levels)
    n, h, L = off[-1], d // 2, len(levels)
    keys = torch.empty(n * (h + 1), dtype=torch.int64, device=_DEV)
    at = 0
    for l in range(L):
        lo, hi = off[max(0, l - 1)], off[min(L, l + 2)]
        step = max(1, (1 << 26) // h)  # rows at a time
        for r0 in range(off[l], off[l + 1], step):
            r = torch.arange(r0, min(r0 + step, off[l + 1]), device=_DEV).repeat_interleave(h)
            c = torch.randint(lo, hi, (r.numel(),), device=_DEV, generator=g)  # c == r: the diagonal's key
            keys[at:at + r.numel()] = torch.minimum(r, c) * n + torch.maximum(r, c)
            at += r.numel()
    i = torch.arange(n, device=_DEV)
    keys[at:] = i * n + i
    keys = torch.unique(keys)
    rp = torch.searchsorted(keys, torch.arange(n + 1, device=_DEV) * n)
    val = torch.empty(keys.numel(), dtype=torch.float64 if wide else torch.float32, device=_DEV)
    col = torch.empty(keys.numel(), dtype=torch.int32, device=_DEV)
    for e in range(0, keys.numel(), 1 << 26):
        part = keys[e:e + (1 << 26)]
        col[e:e + part.numel()] = part % n
        v = 0.5 * torch.randn(part.numel(), device=_DEV, generator=g)
        if wide:
            v = v.double() * (1.0 + 1e-7 * torch.randn(part.numel(), device=_DEV, generator=g, dtype=torch.float64))
        val[e:e + part.numel()] = v
    del keys
    lev = torch.repeat_interleave(torch.arange(L, device=_DEV), torch.tensor(levels, device=_DEV))
    dg = 10.0 * lev + 2.0 * torch.rand(n, device=_DEV, generator=g, dtype=torch.float64) - 1.0
    val[rp[:-1]] = dg.float().to(val.dtype)
    return rp, col, val


def _localised(levels, b, g):
    """Columns as the method's vectors are: weight falling by a factor of 10 from level to level."""
    off = _offsets(levels)
    X = torch.randn(off[-1], b, device=_DEV, generator=g, dtype=torch.float64)
    for l in range(len(levels)):
        X[off[l]:off[l + 1]] *= 0.1 ** l / math.sqrt(levels[l])
    return X / X.norm(dim=0)


def _basis(n, m, g):
    """m orthonormal columns: random ones of the n cosines, with random signs of the rows."""
    j = torch.randperm(n, device=_DEV, generator=g)[:m]
    angle = (2 * torch.arange(n, device=_DEV)[:, None] + 1) * j % (4 * n)
    scale = torch.full((m,), math.sqrt(2.0 / n), dtype=torch.float64, device=_DEV)
    scale[j == 0] = math.sqrt(1.0 / n)
    sign = 2.0 * torch.randint(0, 2, (n, 1), device=_DEV, generator=g) - 1.0
    return torch.cos(angle.double() * (math.pi / (2 * n))) * sign * scale


def _outside(Y, Q):
    """Y - Q (Q^T Y), on the host."""
    q, y = Q.cpu(), Y.cpu()
    return (y - q @ (q.T @ y)).to(Y.device)


def _weights(levels, m):
    """The trained weights of the target (a basis or one pair) and shape."""
    name = "mpnn_weights.json" if m else "mpnn_weights_rmm_L5.json" if len(levels) >= 5 else "mpnn_weights_rmm.json"
    with open(os.path.join(_PKG, name)) as f:
        return json.load(f)["weights"]


def _vectors(case, seed):
    """The dense inputs of a case."""
    g = _gen(seed, 2)
    levels = _levels(case)
    if case["kind"] == "spmm":
        X = _localised(levels, case["b"], g)
        return dict(X=X.float() if case["x"] == "f32" else X)
    S, m = case["S"], case["m"]
    Q = _basis(sum(levels), m, g) if m else None
    Psi = _localised(levels, S, g)
    if case["kind"] == "basis":
        return dict(Q=Q, Psi=Psi)
    X = Q[:, :S].contiguous() if m else Psi
    R = 1e-3 / math.sqrt(X.shape[0]) * torch.randn(X.shape[0], S, device=_DEV, generator=g, dtype=torch.float64)
    E = _localised(levels, S, g)
    E = _outside(E, Q) if m else E - X * (X * E).sum(dim=0)
    theta = [-8.0 + 0.35 * s for s in range(S)]
    return dict(R=R, X=X, Q=Q, E=E.contiguous(), theta=theta)


def _opts(case):
    """Options of the context: the solve's own; a program that only multiplies keeps no basis."""
    if case["kind"] == "solve":
        mixed = case["mode"].startswith("mixed")
        return P.sppc_default_opts(precision=P.SPPC_PREC_MIXED if mixed else P.SPPC_PREC_FP64,
                                   precond=P.SPPC_CORR_RMMDIIS if "rmmdiis" in case["mode"] else P.SPPC_CORR_JACOBI)
    if case["kind"] == "spmm":
        return P.sppc_default_opts(maxiter=0, p_switch=0, m_max=2 * case["k"], precision=P.SPPC_PREC_MIXED)
    return P.sppc_default_opts(maxiter=0, p_switch=0, m_max=2 * case["k"])


def prepare(case, seed):
    rp, col, val = _matrix(_levels(case), case["d"], seed, case.get("val") == "f64")
    torch.cuda.empty_cache()
    off = _offsets(_levels(case))
    st = dict(case=case, H=(rp, col, val), off=off, opts=_opts(case))
    if case["kind"] == "solve":
        st["ws"] = P.workspace_tensor(P.sppc_workspace_size(rp, col, val, off, case["small"], case["k"], st["opts"]))
        return st
    st["ctx"] = P.sppc_setup(rp, col, val, off, case["small"], case["k"], st["opts"])
    st.update(_vectors(case, seed))
    if case["kind"] == "spmm":
        st["Y"] = torch.empty(off[-1], case["b"], dtype=torch.float64, device=_DEV)
    elif case["kind"] == "train":
        st["w"] = _weights(_levels(case), case["m"])
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "spmm":
        P.sppc_spmm(state["ctx"], state["X"], state["Y"])
        return state["Y"]
    if case["kind"] == "basis":
        return P.sppc_mpnn_target(state["ctx"], state["Q"], state["Psi"])
    if case["kind"] == "train":
        T, loss, grad = P.sppc_mpnn_eval(state["ctx"], state["w"], state["R"], state["X"], state["theta"],
                                         E=state["E"], Q=state["Q"])
        return T, torch.tensor(loss, dtype=torch.float64), torch.tensor(grad, dtype=torch.float64)
    rp, col, val = state["H"]
    ctx = P.sppc_setup(rp, col, val, state["off"], case["small"], case["k"], state["opts"], workspace=state["ws"])
    ev, Z, _, _, status = P.sppc_solve(ctx)
    P.sppc_destroy(ctx)
    return torch.tensor(ev, dtype=torch.float64), Z, status


# ------------------------------------------------------------------------------------------- floors


def work(case):
    """Bytes and operations of one pass: the stored triangle (float32 values where they are exact, int32
    columns, row pointers), inputs and outputs once; 2 operations per entry of the whole matrix and column."""
    n = sum(_levels(case))
    nnz_up = n * (case["d"] // 2 + 1)
    nnz = 2 * nnz_up - n
    H = nnz_up * (4 + (8 if case.get("val") == "f64" else 4)) + 8 * (n + 1)
    if case["kind"] == "spmm":
        xb = 4 if case["x"] == "f32" else 8
        return dict(bytes=H + n * case["b"] * (xb + 8), flops=2.0 * nnz * case["b"])
    if case["kind"] == "basis":
        return dict(bytes=8 * n * (case["m"] + 2 * case["S"]), flops=4.0 * n * case["m"] * case["S"])
    if case["kind"] == "train":
        S, m = case["S"], case["m"]
        # forward and backward of the two layers: 3 products with H, 2 x 2 x 289 operations a row and
        # sample, the projections of the output and of its gradient
        return dict(bytes=H + 8 * n * (4 * S + m), flops=S * (6.0 * nnz + 1156.0 * n + 8.0 * n * m))
    k = case["k"]
    return dict(bytes=H + 8 * n * k, flops=2.0 * nnz * k * 16)  # the products of 15 orders and the check


# ------------------------------------------------------------------------------------- exact values


def _product(H, X, skip_diag=False):
    """H X in float64 from the upper triangle."""
    rp, col, val = H
    n, b = X.shape
    Y = torch.zeros(n, b, dtype=torch.float64, device=_DEV)
    X = X.double()
    step = max(1, (1 << 28) // (b * max(1, int(col.numel() // n))))
    cuts = rp[::step].tolist() + [int(rp[-1])]
    for q in range(len(cuts) - 1):
        r0, r1 = q * step, min(n, (q + 1) * step)
        if r0 >= n:
            break
        e0, e1 = cuts[q], int(rp[r1])
        row = torch.repeat_interleave(torch.arange(r0, r1, device=_DEV), rp[r0 + 1:r1 + 1] - rp[r0:r1])
        c = col[e0:e1].long()
        v = val[e0:e1].double()
        off = (c != row).double()
        Y.index_add_(0, row, (v * off if skip_diag else v)[:, None] * X[c])
        Y.index_add_(0, c, (v * off)[:, None] * X[row])
    return Y


def _csr(H, n0):
    """Both triangles of the leading n0 x n0 block as a torch CSR matrix in float64, on the host."""
    rp, col, val = (t.cpu() for t in H)
    row = torch.repeat_interleave(torch.arange(rp.numel() - 1), rp[1:] - rp[:-1])
    keep = (row < n0) & (col < n0)
    r, c, v = row[keep], col[keep].long(), val[keep].double()
    o = r != c
    key = torch.cat([r * n0 + c, c[o] * n0 + r[o]])
    v = torch.cat([v, v[o]])
    key, p = torch.sort(key)
    ptr = torch.searchsorted(key, torch.arange(n0 + 1) * n0)
    return torch.sparse_csr_tensor(ptr, key % n0, v[p], size=(n0, n0))


def _lowest(A, k, seed):
    """The k lowest eigenpairs of A by a Chebyshev-filtered block to the rounding of float64."""
    n = A.shape[0]
    nb = min(n, k + 16)
    cum = torch.cat([torch.zeros(1, dtype=torch.float64), torch.cumsum(A.values().abs(), 0)])
    bound = float((cum[A.crow_indices()[1:]] - cum[A.crow_indices()[:-1]]).max())
    X = torch.linalg.qr(torch.randn(n, nb, generator=torch.Generator().manual_seed(int(seed) & 0x7FFFFFFF),
                                    dtype=torch.float64))[0]
    for _ in range(60):
        AX = A @ X
        w, V = torch.linalg.eigh(X.T @ AX)
        X, AX = X @ V, AX @ V
        res = (AX[:, :k] - X[:, :k] * w[:k]).norm(dim=0) / w[:k].abs().clamp(min=1.0)
        if float(res.max()) < 2e-13 or nb == n:
            break
        e, c = 0.5 * (bound - float(w[-1])), 0.5 * (bound + float(w[-1]))
        sig = e / (float(w[0]) - c)
        tau = 2.0 / sig
        Y0, Y1 = X, (AX - c * X) * (sig / e)
        deg = max(12, min(80, int(25.0 / math.acosh(max(1.0 + 1e-9, (c - float(w[0])) / e)))))
        for _ in range(deg - 1):
            sn = 1.0 / (tau - sig)
            Y0, Y1 = Y1, (A @ Y1 - c * Y1) * (2.0 * sn / e) - Y0 * (sig * sn)
            sig = sn
        X = torch.linalg.qr(Y1)[0]
    return w[:k], X[:, :k]


def exact(case, seed):
    n = sum(_levels(case))
    if case["kind"] == "basis":
        v = _vectors(case, seed)
        return _outside(v["Psi"], v["Q"])
    if case["kind"] == "solve":
        if n * case["d"] > 3e6:  # a minute and more on the host
            return None
        H = _matrix(_levels(case), case["d"], seed, False)
        n0 = sum(_levels(case)[:case["small"]])
        w, Z = _lowest(_csr(H, n), case["k"], seed)
        # signs: the largest coefficient on the small space's eigenvectors is positive, and their largest entry
        _, P0 = _lowest(_csr(H, n0), case["k"], seed)
        P0 = P0 * torch.sign(P0.gather(0, P0.abs().argmax(dim=0)[None]))
        c = P0.T @ Z[:n0]
        return w, Z * torch.sign(c.gather(0, c.abs().argmax(dim=0)[None])), None
    H = _matrix(_levels(case), case["d"], seed, case.get("val") == "f64")
    v = _vectors(case, seed)
    if case["kind"] == "spmm":
        return _product(H, v["X"])
    return _network(case, H, v)


def _network(case, H, v):
    """The network's projected output, loss and mean gradient in float64 with bfloat16-rounded weights."""
    levels, S = _levels(case), case["S"]
    n, off = sum(levels), _offsets(levels)
    rp, _, val = H
    d = val[rp[:-1]].double()[:, None]
    ones = torch.ones(n, 1, dtype=torch.float64, device=_DEV)
    lev = torch.zeros(n, 1, dtype=torch.float64, device=_DEV)
    for l in range(len(levels)):
        lev[off[l]:off[l + 1]] = 0.5 * min(2, max(0, l - case["small"] + 1))
    stat = _product(H, torch.cat([d, ones, lev], dim=1), skip_diag=True)
    th = torch.tensor(v["theta"], dtype=torch.float64, device=_DEV)
    w = torch.tensor(_weights(levels, case["m"]), device=_DEV).bfloat16().double().requires_grad_(True)
    R, X, Q, E = v["R"], v["X"], v["Q"], v["E"]
    fr = R / (R.pow(2).mean(dim=0)).sqrt()
    sc = 1.0 + th.abs()
    feats = [fr, (d - th) / sc, lev.expand(n, S)]
    msgs = [_product(H, fr, skip_diag=True), (stat[:, :1] - th * stat[:, 1:2]) / sc, stat[:, 2:].expand(n, S)]

    class Agg(torch.autograd.Function):  # A u with the symmetric A = H - diag(d)
        @staticmethod
        def forward(ctx, u):
            return _product(H, u, skip_diag=True)

        @staticmethod
        def backward(ctx, g):
            return _product(H, g.contiguous(), skip_diag=True)

    hs = u = 0.0
    for j in range(32):
        pre = w[192 + j]
        for q in range(3):
            pre = pre + w[3 * j + q] * feats[q] + w[96 + 3 * j + q] * msgs[q]
        hj = torch.tanh(pre)
        hs, u = hs + w[224 + j] * hj, u + w[256 + j] * hj
    o = hs + Agg.apply(u) + w[288]
    den = d - th
    fl = 1e-2 * th.abs().clamp(min=1.0)
    den = torch.where(den.abs() < fl, torch.where(den >= 0, fl.expand_as(den), -fl.expand_as(den)), den)
    t = R / den * (1.0 + o)
    t = _outside(t, Q) if Q is not None else t - X * (X * t).sum(dim=0)
    loss = 1.0 - (t * E).sum(dim=0).pow(2) / (t.pow(2).sum(dim=0) * E.pow(2).sum(dim=0))
    loss.mean().backward()
    return t.detach(), loss.detach(), w.grad
