"""The measured cases: what a user of this package has it do, through its public calls.

Real Schur forms of Hessenberg matrices (one matrix, and batches of uneven
order), the Hessenberg reduction before them, the two together on a dense
matrix, the reordering after them, and a training step of the proposal network.
Sizes run from the smallest calls, where launches and round trips count, to the
orders of the benchmark; odd orders and padded leading dimensions are among them.

A Schur form is not unique: the order of its diagonal blocks and the signs of
its vectors depend on rounding.  So a Schur case returns what its factors are
used for and what the input alone determines: up to order 1100 the whole matrix
put together again, Z S Z^T; above, its product with a block of vectors,
Z (S (Z^T B)); and, where the eigenvalues are well conditioned, all of them
sorted.  The Hessenberg form is unique and comes back as it is.
"""
import math

import numpy as np
import torch

from paper_2002_05024_amd import autotune, autotune_single
from paper_2002_05024_amd import binding as neig

WHOLE = 1100  # orders up to which a factorisation is multiplied out whole
BLOCK = 320   # vectors it is applied to above


def listed():
    return [
        # the smallest call: one matrix that fits in LDS, all launch and round-trip time
        dict(name="schur_40", kind="schur", family="random", n=40, pad=0, tuned=False),
        # the benchmark's small workload
        dict(name="schur_256", kind="schur", family="random", n=256, pad=0, tuned=False),
        # Hessenberg form of a dense matrix, odd order, a view into a wider array, library defaults
        dict(name="schur_dense_1003", kind="schur", family="dense", n=1003, pad=9, tuned=False),
        # the same kind of input at the order of the mid-size benchmark, with the saved tuning
        dict(name="schur_dense_4000", kind="schur", family="dense", n=4000, pad=0, tuned=True),
        # the headline benchmark: random Hessenberg, order 20000, with the saved tuning
        dict(name="schur_random_20000", kind="schur", family="random", n=20000, pad=0, tuned=True),
        # many tiny problems in one launch (a serving loop)
        dict(name="batched_small", kind="batched", count=256, lo=32, hi=96),
        # the batched benchmark: 512 problems of order 32 to 1024
        dict(name="batched_512", kind="batched", count=512, lo=32, hi=1024),
        # Hessenberg reduction with its factor: ordinary, and large
        dict(name="hessenberg_1000", kind="hessenberg", n=1000, pad=0),
        dict(name="hessenberg_8000", kind="hessenberg", n=8000, pad=0),
        # dense matrix to Schur form, both steps: the whole eigenvalue computation
        dict(name="eig_2000", kind="eig", n=2000, tuned=True),
        # half of the eigenvalues of a Schur form moved to its leading block
        dict(name="reorder_4000", kind="reorder", n=4000, pad=0),
        # one step of the proposal network's training, at its default batch
        dict(name="train_4096", kind="train", batch=4096),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["schur", "schur", "schur", "batched", "hessenberg", "eig", "reorder", "train"])
    if kind == "schur":
        family = rng.choice(["random", "dense", "graded"])
        n = _between(rng, 24, {"random": 20000, "dense": 4000, "graded": 4000}[family])
        return dict(kind=kind, family=family, n=n, pad=rng.choice([0, 0, 1, 7]), tuned=rng.random() < 0.5)
    if kind == "batched":
        hi = _between(rng, 48, 1024)
        return dict(kind=kind, count=_between(rng, 32, 512), lo=rng.randint(24, 40), hi=hi)
    if kind == "hessenberg":
        return dict(kind=kind, n=_between(rng, 100, 8000), pad=rng.choice([0, 0, 1, 7]))
    if kind == "eig":
        return dict(kind=kind, n=_between(rng, 64, 3000), tuned=rng.random() < 0.5)
    if kind == "reorder":
        return dict(kind=kind, n=_between(rng, 100, 4000), pad=rng.choice([0, 0, 1, 7]))
    return dict(kind=kind, batch=_between(rng, 64, 32768))


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _host(seed):
    return np.random.Generator(np.random.PCG64(int(seed)))


def _empty(n, pad=0):
    """A column-major n x n matrix with leading dimension n + pad."""
    return torch.empty(n, n + pad, dtype=torch.float64, device="cuda")[:, :n].t()


def _randn(n, g, pad=0):
    A = _empty(n, pad)
    A.copy_(torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g).t())
    return A


def _identity(Z):
    Z.zero_()
    Z.diagonal().fill_(1.0)


def _chi(n, h):
    """Subdiagonal of the Hessenberg form of an n x n N(0,1) matrix: independent
    chi variables of n-1, ..., 1 degrees of freedom (Householder reduction leaves
    the rest N(0,1))."""
    return torch.from_numpy(np.sqrt(h.chisquare(np.arange(n - 1, 0, -1)))).cuda()


def _hessenberg_input(family, n, pad, seed):
    g, h = _generator(seed), _host(seed)
    H = _randn(n, g, pad)
    H.triu_(-1)
    if family == "dense":
        H.diagonal(-1).copy_(_chi(n, h))
    elif family == "graded":
        H.mul_(10.0 ** (-8.0 * torch.arange(n, dtype=torch.float64, device="cuda") / n)[:, None])
    return H


def _vectors(n, seed):
    g = _generator(seed + 7919)
    return torch.randn(n, BLOCK, dtype=torch.float64, device="cuda", generator=g)


def _schur_form(n, seed, pad):
    """A standardised real Schur form: half of the eigenvalues real in [-1, 1], half
    conjugate pairs in the unit disk, in random order; N(0, 1/(100 n)) above."""
    g, h = _generator(seed), _host(seed)
    S = _randn(n, g, pad)
    S.triu_(1).mul_(0.1 / math.sqrt(n))
    npair = n // 4
    size = np.array([1] * (n - 2 * npair) + [2] * npair)
    h.shuffle(size)
    at = np.concatenate([[0], np.cumsum(size)[:-1]])
    one, two = at[size == 1], at[size == 2]
    re, im = np.empty(n), np.zeros(n)
    re[one] = h.uniform(-1.0, 1.0, len(one))
    z = np.sqrt(h.uniform(0.0, 1.0, npair)) * np.exp(1j * h.uniform(0.05, np.pi - 0.05, npair))
    re[two] = re[two + 1] = z.real
    im[two], im[two + 1] = z.imag, -z.imag
    S.diagonal().copy_(torch.from_numpy(re))
    t = torch.from_numpy(two).cuda()
    zi = torch.from_numpy(z.imag).cuda()
    S[t, t + 1] = zi
    S[t + 1, t] = -zi
    return S, re, im


def _orthogonal(n, g, pad):
    """A dense orthogonal matrix: two random reflections."""
    Z = _empty(n, pad)
    _identity(Z)
    for _ in range(2):
        u = torch.randn(n, 1, dtype=torch.float64, device="cuda", generator=g)
        u /= torch.linalg.norm(u)
        Z -= 2.0 * (Z @ u) @ u.t()
    return Z


def _theta(seed):
    h = _host(seed)
    parts = [h.standard_normal(24), np.full(24, 1.0) + h.uniform(0.0, 1.0, 24),
             h.standard_normal((64, 24)) * math.sqrt(2.0 / 24), np.zeros(64),
             h.standard_normal((64, 64)) * math.sqrt(2.0 / 64), np.zeros(64),
             h.standard_normal((16, 64)) * math.sqrt(2.0 / 64), np.zeros(16)]
    return np.concatenate([p.ravel() for p in parts]).astype(np.float32)


def _parameters(n, tuned):
    neig.set_params(ns=0, nw=0, chain=0, chase_w=0, nibble=0)
    if tuned:
        autotune_single.apply(n)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case)
    if kind in ("schur", "eig", "reorder", "hessenberg"):
        n, pad = case["n"], case.get("pad", 0)
        s["Z"] = _empty(n, pad)
        s["H"] = _empty(n, pad)
        if n > WHOLE and kind != "hessenberg":
            s["B"] = _vectors(n, seed)
    if kind == "schur":
        s["H0"] = _hessenberg_input(case["family"], n, pad, seed)
        _parameters(n, case["tuned"])
    elif kind == "eig":
        s["H0"] = _empty(n)
        s["H0"].copy_(torch.rand(n, n, dtype=torch.float64, device="cuda", generator=_generator(seed)) * 2.0 - 1.0)
        _parameters(n, case["tuned"])
    elif kind == "hessenberg":
        s["H0"] = _randn(n, _generator(seed), pad)
    elif kind == "reorder":
        s["H0"], re, _ = _schur_form(n, seed, pad)
        s["Z0"] = _orthogonal(n, _generator(seed + 1), pad)
        s["select"] = (re < 0.0).astype(np.int32)
    elif kind == "batched":
        g, h = _generator(seed), _host(seed)
        count = case["count"]
        sizes = h.integers(case["lo"], case["hi"] + 1, size=count)
        big = max(case["lo"], case["hi"]) | 1
        # problem b in the leading corner of plane b; column-major, so plane[j, i] is entry (i, j)
        H0 = torch.randn(count, big, big, dtype=torch.float64, device="cuda", generator=g)
        i = torch.arange(big, device="cuda")
        H0.mul_(i[None, :] <= i[:, None] + 1)
        nb = torch.from_numpy(sizes).cuda()
        H0.mul_((i[None, :] < nb[:, None])[:, :, None]).mul_((i[None, :] < nb[:, None])[:, None, :])
        # even problems random Hessenberg, odd ones the Hessenberg form of a dense matrix
        for b in range(1, count, 2):
            k = int(sizes[b])
            H0[b, :k, :k].diagonal(1).copy_(_chi(k, h))
        s["ones"] = (i[None, :] < nb[:, None]).double()
        s["H0"], s["H"], s["Z"] = H0, torch.empty_like(H0), torch.zeros_like(H0)
        s["B"] = torch.randn(count, big, 16, dtype=torch.float64, device="cuda", generator=g)
        s["call"] = neig.batched_tables([s["H"][b, :k, :k].t() for b, k in enumerate(sizes)],
                                        [s["Z"][b, :k, :k].t() for b, k in enumerate(sizes)])
        neig.set_params(ns=0, nw=0, chain=0, chase_w=0, nibble=0)
        autotune.apply_saved()
    else:
        g, h = _generator(seed), _host(seed)
        b = case["batch"]
        th = _theta(seed)
        mu, sd = torch.from_numpy(th[:24]).cuda(), torch.from_numpy(th[24:48]).cuda()
        s["X"] = torch.randn(b, 24, device="cuda", generator=g) * sd + mu
        s["a"] = torch.from_numpy(h.integers(0, 8, b).astype(np.int32)).cuda()
        s["c"] = torch.from_numpy(h.integers(0, 8, b).astype(np.int32)).cuda()
        s["w"] = torch.from_numpy(h.exponential(1.0, b).astype(np.float32)).cuda()
        s["theta"] = torch.from_numpy(th).cuda()
        s["m"], s["v"] = torch.zeros_like(s["theta"]), torch.zeros_like(s["theta"])
        s["step"] = 0
    return s


def _together(s, S, Z):
    """The factorisation put to use: Z S Z^T, or its product with the block B."""
    if "B" in s:
        return Z @ (S @ (Z.t() @ s["B"]))
    return (Z @ S) @ Z.t()


def _sorted(wr, wi):
    """Eigenvalues by real part (the two of a pair share it and keep their order, + then -)."""
    wr, at = torch.sort(wr, stable=True)
    return wr, wi[at]


def run(s):
    kind = s["kind"]
    if kind == "train":
        s["step"] += 1
        loss, grad = neig.mlp_grad(s["X"], s["a"], s["c"], s["w"], s["theta"])
        neig.mlp_adam(s["theta"], grad, s["m"], s["v"], s["step"], 2e-3)
        return dict(loss=loss, grad=grad, theta=s["theta"], m=s["m"], v=s["v"])
    H, Z = s["H"], s["Z"]
    H.copy_(s["H0"])
    if kind == "batched":
        Z.zero_()
        Z.diagonal(dim1=1, dim2=2).copy_(s["ones"])
        neig.launch_batched(s["call"])
        out = torch.bmm(Z.transpose(1, 2), torch.bmm(H.transpose(1, 2), torch.bmm(Z, s["B"])))
        return dict(together=out, info=s["call"].info)
    if kind == "reorder":
        Z.copy_(s["Z0"])
        wr, wi, m, info = neig.reorder(H, Z, s["select"])
        return dict(together=_together(s, H, Z), wr=wr, wi=wi, m=m, info=info)
    _identity(Z)
    if kind == "hessenberg":
        neig.hessenberg(H, Z)
        return dict(H=H, Q=Z)
    if kind == "eig":
        neig.hessenberg(H, Z)
    r = neig.schur(H, Z)
    out = dict(together=_together(s, H, Z), info=r.info)
    if kind == "eig" or s["family"] == "dense":
        out["wr"], out["wi"] = _sorted(r.wr, r.wi)
    return out


def work(case):
    kind = case["kind"]
    if kind == "train":
        b, p = case["batch"], 24 * 64 + 64 * 64 + 64 * 16
        return dict(bytes=4.0 * (27 * b + 7 * 6848), flops=6.0 * b * p)
    if kind == "batched":
        lo, hi = case["lo"], max(case["lo"], case["hi"])
        sizes = np.arange(lo, hi + 1, dtype=np.float64)
        return dict(bytes=32.0 * case["count"] * np.mean(sizes ** 2), flops=8.0 * case["count"] * np.mean(sizes ** 3))
    n = float(case["n"])
    if kind == "hessenberg":
        # 10/3 n^3 for H, 4/3 n^3 for Q; the trailing block is read once per column
        return dict(bytes=8.0 * n ** 3 / 3 + 32 * n * n, flops=14.0 / 3 * n ** 3)
    if kind == "reorder":
        # every selected row passes the unselected ones: 6 flops on each of the 2 n entries of S and Z
        return dict(bytes=32.0 * n * n, flops=6.0 * (n / 2) ** 2 / 2 * 2 * n)
    if kind == "eig":
        return dict(bytes=8.0 * n ** 3 / 3 + 64 * n * n, flops=(14.0 / 3 + 10) * n ** 3)
    # Schur: a dense matrix's form takes sweeps (order 10 n^3 flops); a random
    # Hessenberg matrix deflates window by window (about 600 n^2)
    return dict(bytes=32.0 * n * n, flops=10.0 * n ** 3 if case["family"] == "dense" else min(10.0 * n ** 3, 600.0 * n * n))


def _exact_hessenberg(A):
    """Householder reduction column by column, in place; returns (H, Q)."""
    n = A.shape[0]
    Q = torch.eye(n, dtype=torch.float64, device=A.device)
    for j in range(n - 2):
        x = A[j + 1:, j].clone()
        nrm = torch.linalg.norm(x)
        beta = torch.where(x[0] >= 0, -nrm, nrm)
        v = x / (x[0] - beta)
        v[0] = 1.0
        tau = (beta - x[0]) / beta
        A[:, j + 1:].addr_(A[:, j + 1:] @ v, v * tau, alpha=-1.0)
        A[j + 1:, j:].addr_(v * tau, v @ A[j + 1:, j:], alpha=-1.0)
        Q[:, j + 1:].addr_(Q[:, j + 1:] @ v, v * tau, alpha=-1.0)
        A[j + 2:, j] = 0.0
    return A, Q


def _exact_train(s):
    th = s["theta"].double()
    cut = np.cumsum([24, 24, 64 * 24, 64, 64 * 64, 64, 16 * 64, 16])
    p = [t.clone().requires_grad_(True) for t in torch.tensor_split(th, list(cut[:-1]))]
    x = (s["X"].double() - p[0].detach()) / p[1].detach()
    h = torch.relu(x @ p[2].view(64, 24).t() + p[3])
    h = torch.relu(h @ p[4].view(64, 64).t() + p[5])
    z = h @ p[6].view(16, 64).t() + p[7]
    w = s["w"].double()
    at = torch.arange(len(w), device="cuda")
    loss = -(w * (torch.log_softmax(z[:, :8], 1)[at, s["a"].long()] +
                  torch.log_softmax(z[:, 8:], 1)[at, s["c"].long()])).mean()
    grad = torch.cat([torch.zeros(48, dtype=torch.float64, device="cuda")] + list(torch.autograd.grad(loss, p[2:])))
    m, v = 0.1 * grad, 0.001 * grad * grad
    theta = th - 2e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    theta[:48] = th[:48]
    return dict(loss=loss.detach().reshape(1), grad=grad, theta=theta, m=m, v=v)


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "train":
        return _exact_train(s)
    H0 = s["H0"]
    if kind == "batched":
        return dict(together=torch.bmm(H0.transpose(1, 2), s["B"]), info=None)
    if kind == "hessenberg":
        H, Q = _exact_hessenberg(H0.clone(memory_format=torch.contiguous_format))
        return dict(H=H, Q=Q)
    if kind == "reorder":
        _, re, im = _schur_form(case["n"], seed, 0)
        order = np.concatenate([np.flatnonzero(s["select"]), np.flatnonzero(s["select"] == 0)])
        return dict(together=_together(s, H0, s["Z0"]), wr=torch.from_numpy(re[order]),
                    wi=torch.from_numpy(im[order]), m=None, info=None)
    out = dict(together=H0 @ s["B"] if "B" in s else H0, info=None)
    if kind == "eig" or case["family"] == "dense":
        out["wr"] = out["wi"] = None
        if case["n"] <= WHOLE:
            lam = np.linalg.eigvals(H0.cpu().numpy())
            # by real part, the two of a pair next to each other, + then -
            lam = lam[np.lexsort((-lam.imag, lam.real))]
            out["wr"], out["wi"] = torch.from_numpy(lam.real.copy()), torch.from_numpy(lam.imag.copy())
    return out
