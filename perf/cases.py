"""Cases of use of this library, for timing and comparing versions of it.

Each case is one pass of a user's program through the public Python entry
points: the full CGTP (forward, real basis, channels with path weights,
gradients) and the signal products (Gaunt, vector and rank-2; forward,
gradients, real basis).  Sizes are those of the library's own workloads where
it has one, else generic.  Features are iid N(0, 1), as in its workloads.

    listed()            the cases, dicts of plain values
    draw(rng)           one more case of the same ranges
    prepare(case, s)    plan and inputs on the GPU, from the seed alone
    run(state)          one pass; returns its outputs
    work(case)          bytes and flops a pass cannot do without
    tolerance(case)     how far another correct implementation may be off
    exact(case, s)      what run() returns, in 64 bits from the definitions
"""
import math

import numpy as np
import torch

import paper_2602_21466_amd as lib

# op: "cgtp"            Plan.forward
#     "cgtp_real"       Plan.forward_real
#     "cgtp_channels"   Plan.forward_weighted, x2 shared by the C channels, weights per channel or per pair
#     "cgtp_backward"   Plan.backward
#     "cgtp_step"       Plan.forward and Plan.backward, a layer's share of a training step
#     "istp"            IstpPlan.forward (spin 0, 1, 2)
#     "istp_backward"   IstpPlan.backward
#     "istp_real_step"  IstpPlan.forward_real and backward_real (spin 0)
#     "istp_channels"   IstpPlan.forward_weighted, x2 shared, per-channel weights


def listed():
    return [
        # the smallest call: a few molecules' worth of low-degree features in double precision; launch and latency
        {"name": "cgtp_L2_N64_fp64", "op": "cgtp", "L": 2, "N": 64, "dtype": "fp64"},
        # the common low degree over many pairs (edges of a large graph batch)
        {"name": "cgtp_L4_N100000", "op": "cgtp", "L": 4, "N": 100_000, "dtype": "fp32"},
        # the two headline degrees
        {"name": "cgtp_L16_N8192", "op": "cgtp", "L": 16, "N": 8192, "dtype": "fp32"},
        {"name": "cgtp_L32_N1024", "op": "cgtp", "L": 32, "N": 1024, "dtype": "fp32"},
        # real-basis features of a ragged batch at an odd middle degree
        {"name": "cgtp_real_L11_N4001", "op": "cgtp_real", "L": 11, "N": 4001, "dtype": "fp32"},
        # a message-passing layer: 16 channels per edge, the edge's harmonics shared, one weight per path
        {"name": "cgtp_channels_L16_N512_C16", "op": "cgtp_channels", "L": 16, "N": 512, "C": 16, "dtype": "fp32",
         "per_pair": False},
        # gradients at a headline degree
        {"name": "cgtp_backward_L16_N8192", "op": "cgtp_backward", "L": 16, "N": 8192, "dtype": "fp32"},
        # forward and gradients of a layer at a usual training degree, ragged batch
        {"name": "cgtp_step_L7_N4099", "op": "cgtp_step", "L": 7, "N": 4099, "dtype": "fp32"},
        # the multiple-input, multiple-output products: vector and Gaunt
        {"name": "vector_L16_N65536", "op": "istp", "spin": 1, "L": 16, "N": 65_536, "dtype": "fp32"},
        {"name": "gaunt_L32_N65536", "op": "istp", "spin": 0, "L": 32, "N": 65_536, "dtype": "fp32"},
        {"name": "vector_backward_L16_N16384", "op": "istp_backward", "spin": 1, "L": 16, "N": 16_384,
         "dtype": "fp32"},
        # a training step of a real-basis Gaunt layer, the form equivariant networks use most
        {"name": "gaunt_real_step_L10_N20011", "op": "istp_real_step", "spin": 0, "L": 10, "N": 20_011,
         "dtype": "fp32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["cgtp", "cgtp", "cgtp_real", "cgtp_channels", "cgtp_backward", "cgtp_step", "istp",
                     "istp_backward", "istp_real_step", "istp_channels"])
    dtype = "fp64" if rng.random() < 0.12 else "fp32"
    if op.startswith("cgtp"):
        L = rng.randint(1, 32 if dtype == "fp32" else 8)
        # total outputs: from one small batch to a fraction of the headline batches
        most = {"cgtp_backward": 2.0e8, "cgtp_step": 1.5e8}.get(op, 4.0e8) / (4 if dtype == "fp64" else 1)
        N = max(1, min(100_000, int(_log_int(rng, 2.0e4, most) / (L + 1) ** 4)))
        case = {"op": op, "L": L, "N": N, "dtype": dtype}
        if op == "cgtp_channels":
            case["C"] = rng.choice([1, 3, 8, 16, 17])
            case["N"] = max(1, N // case["C"])
            case["per_pair"] = rng.random() < 0.5
        return case
    if op == "istp_real_step":
        spin, L = 0, rng.randint(1, 12 if dtype == "fp64" else 20)
    elif op == "istp_backward":
        spin = rng.choice([0, 1, 1, 2])
        L = rng.randint(1, {0: 30, 1: 18, 2: 11}[spin] if dtype == "fp32" else 8)
    else:
        spin = rng.choice([0, 1, 1, 2])
        L = rng.randint(1, {0: 32, 1: 32, 2: 16}[spin] if dtype == "fp32" else 10)
    most = {"istp_backward": 4.0e7, "istp_real_step": 4.0e7}.get(op, 1.2e8) / (8 if dtype == "fp64" else 1)
    N = max(1, min(100_000, int(_log_int(rng, 2.0e4, most) / ((2 * spin + 1) * (2 * L + 1) ** 2))))
    case = {"op": op, "spin": spin, "L": L, "N": N, "dtype": dtype}
    if op == "istp_channels":
        case["C"] = rng.choice([1, 4, 16])
        case["N"] = max(1, N // case["C"])
    return case


# ---------------------------------------------------------------- inputs and the pass

_DT = {"fp32": torch.float32, "fp64": torch.float64}


def _inputs(case, seed):
    """The pass's input tensors by name, on the GPU, from the seed alone."""
    g = torch.Generator("cuda").manual_seed(int(seed))
    dt, op, L, N = _DT[case["dtype"]], case["op"], case["L"], case["N"]

    def randn(*shape):
        return torch.randn(*shape, dtype=dt, device="cuda", generator=g)

    if op.startswith("cgtp"):
        nin, nout = (L + 1) ** 2, (L + 1) ** 4
        if op == "cgtp_channels":
            C, P = case["C"], (L + 1) * (2 * L * L + 4 * L + 3) // 3
            return {"x1": randn(N, C, nin), "x2": randn(N, nin),
                    "w": randn(N, C, P) if case["per_pair"] else randn(C, P)}
        d = {"x1": randn(N, nin), "x2": randn(N, nin)}
        if op in ("cgtp_backward", "cgtp_step"):
            d["g"] = randn(N, nout)
        return d
    s = case["spin"]
    nin, nout = (2 * s + 1) * (L + 1) ** 2, (2 * s + 1) * (2 * L + 1) ** 2
    if op == "istp_channels":
        C, nl, nlo = case["C"], len(_labels(s, L)), len(_labels(s, 2 * L))
        return {"x1": randn(N, C, nin), "x2": randn(N, nin), "w1": randn(C, nl), "w2": randn(C, nl),
                "wo": randn(C, nlo)}
    d = {"x1": randn(N, nin), "x2": randn(N, nin)}
    if op in ("istp_backward", "istp_real_step"):
        d["g"] = randn(N, nout)
    return d


def prepare(case, seed):
    state = _inputs(case, seed)
    state["op"] = case["op"]
    if case["op"].startswith("cgtp"):
        state["plan"] = lib.Plan(case["L"], dtype=case["dtype"])
    else:
        state["plan"] = lib.IstpPlan(case["L"], case["spin"], case["dtype"])
    return state


def run(state):
    op, plan, x1, x2 = state["op"], state["plan"], state["x1"], state["x2"]
    if op in ("cgtp", "istp"):
        return plan.forward(x1, x2)
    if op == "cgtp_real":
        return plan.forward_real(x1, x2)
    if op == "cgtp_channels":
        return plan.forward_weighted(x1, x2, state["w"])
    if op == "istp_channels":
        return plan.forward_weighted(x1, x2, state["w1"], state["w2"], state["wo"])
    if op in ("cgtp_backward", "istp_backward"):
        return plan.backward(x1, x2, state["g"])
    if op == "cgtp_step":
        z = plan.forward(x1, x2)
        return (z,) + tuple(plan.backward(x1, x2, state["g"]))
    z = plan.forward_real(x1, x2)   # istp_real_step
    return (z,) + tuple(plan.backward_real(x1, x2, state["g"]))


# ---------------------------------------------------------------- the work a pass cannot do without

def _cg_terms(L):
    """Nonzero terms C^{l3 m3}_{l1 m1 l2 m2} of all paths: per (l1, l2) and m3 a square matrix over (l3, m1)."""
    total = 0
    for l1 in range(L + 1):
        for l2 in range(L + 1):
            for M in range(l1 + l2 + 1):
                n = min(2 * min(l1, l2) + 1, l1 + l2 - M + 1)
                total += n * n * (1 if M == 0 else 2)
    return total


def work(case):
    op, L, N = case["op"], case["L"], case["N"]
    esz = 4 if case["dtype"] == "fp32" else 8
    rows = N * case.get("C", 1)
    if op.startswith("cgtp"):
        nin, nout, t = (L + 1) ** 2, (L + 1) ** 4, _cg_terms(L)
        fwd_b, fwd_f = 2 * nin + nout, 2.0 * t + nout        # each term once, each product x1 x2 once
        bwd_b, bwd_f = 4 * nin + nout, 2.0 * t + 4.0 * nout  # the transposed sum, then both factors
        if op == "cgtp_channels":
            P = (L + 1) * (2 * L * L + 4 * L + 3) // 3
            b = rows * (nin + nout) + N * nin + (rows if case["per_pair"] else case["C"]) * P
            return {"bytes": float(esz * b), "flops": rows * (fwd_f + nout)}
        if op == "cgtp_real":   # complex products, both parts of each order
            return {"bytes": float(esz * N * fwd_b), "flops": N * (2.0 * t + 3.0 * nout)}
        if op == "cgtp_backward":
            return {"bytes": float(esz * N * bwd_b), "flops": N * bwd_f}
        if op == "cgtp_step":
            return {"bytes": float(esz * N * (fwd_b + bwd_b)), "flops": N * (fwd_f + bwd_f)}
        return {"bytes": float(esz * N * fwd_b), "flops": N * fwd_f}
    # signal products on the smallest exact grid: Legendre sums (parity-folded),
    # longitude transforms of Hermitian series at 2.5 n log2 n, pointwise products
    s = case["spin"]
    C = 2 * s + 1
    nin, nout = C * (L + 1) ** 2, C * (2 * L + 1) ** 2

    def product(la, lb, lo):
        R, Phi = (la + lb + lo + 2) // 2, la + lb + lo + 1
        fft = 2.5 * Phi * math.log2(Phi)
        mults = {0: 1, 1: 6, 2: 19}[s]
        return C * R * (2.0 * (la + 1) ** 2 + 2.0 * (lb + 1) ** 2 + 2.0 * (lo + 1) ** 2 + 3 * fft) + 6.0 * mults * R * Phi / 2

    fwd_f, bwd_f = product(L, L, 2 * L), 2 * product(2 * L, L, L)
    if op == "istp_channels":
        return {"bytes": float(esz * (rows * (nin + nout) + N * nin)), "flops": rows * fwd_f}
    if op == "istp_backward":
        return {"bytes": float(esz * N * (4 * nin + nout)), "flops": N * bwd_f}
    if op == "istp_real_step":
        return {"bytes": float(esz * N * (6 * nin + 2 * nout)), "flops": N * (fwd_f + bwd_f)}
    return {"bytes": float(esz * N * (2 * nin + nout)), "flops": N * fwd_f}


def tolerance(case):
    """About four times the error against exact() that was measured: at most 2.2e-7 (largest value 9.4e-6, over the
    1.2e9 outputs of L = 32) with 32-bit tables and sums, 5.3e-16 (1.5e-15) in 64 bits at small degrees."""
    if case["dtype"] == "fp64":
        return {"rel": 4e-15, "max": 1e-13}
    return {"rel": 1e-6, "max": 4e-5}


# ---------------------------------------------------------------- the definitions, in 64 bits

_CG = {}


def _cg(l1, l2):
    """Per M = 0..l1+l2: the coefficients C^{l3 M}_{l1 m1 l2 M-m1}, an orthogonal matrix [l3][m1] (both ascending).

    Its rows are the eigenvectors of J^2 = (J1 + J2)^2 in the basis |m1, M - m1> (a tridiagonal matrix with
    eigenvalues l3 (l3 + 1)); signs follow the Condon-Shortley convention, carried down from M = l3, where
    component m1 has the sign (-1)^(l1 - m1), by the lowering operator."""
    if (l1, l2) in _CG:
        return _CG[l1, l2]
    mats = [None] * (l1 + l2 + 1)
    above = None   # (rows by l3, first m1) of M + 1
    for M in range(l1 + l2, -1, -1):
        lo, hi = max(-l1, M - l2), min(l1, M + l2)
        m1 = np.arange(lo, hi + 1)
        m2 = M - m1
        a = np.diag((l1 * (l1 + 1) + l2 * (l2 + 1) + 2 * m1 * m2).astype(np.float64))
        k = np.arange(len(m1) - 1)
        off = np.sqrt((l1 - m1[:-1]) * (l1 + m1[:-1] + 1.0) * (l2 + m2[:-1]) * (l2 - m2[:-1] + 1.0))
        a[k, k + 1] = off
        a[k + 1, k] = off
        v = np.linalg.eigh(a)[1].T   # row i: l3 = lmin + i
        lmin = max(abs(l1 - l2), M)
        if above is not None:   # <l3 M | J- | l3 M+1> > 0
            up, ulo, ulmin = above
            p1 = ulo + np.arange(up.shape[1])
            p2 = M + 1 - p1
            low = np.zeros((up.shape[0], len(m1) + 2))   # column m1 - lo + 1
            low[:, p1 - lo] += np.sqrt((l1 + p1) * (l1 - p1 + 1.0)) * up
            low[:, p1 - lo + 1] += np.sqrt((l2 + p2) * (l2 - p2 + 1.0)) * up
            flip = np.sum(low[:, 1:-1] * v[ulmin - lmin:], axis=1) < 0
            v[ulmin - lmin:][flip] *= -1.0
        if lmin == M:
            b = int(np.argmax(np.abs(v[0])))
            if v[0, b] * (1.0 if (l1 - m1[b]) % 2 == 0 else -1.0) < 0:
                v[0] = -v[0]
        mats[M] = v
        above = (v, lo, lmin)
    _CG[l1, l2] = mats
    return mats


def _orders(L):
    """Per block (l1, l2) and M >= 0: index lists of the term's factors and outputs, and the coefficients."""
    off = 0
    for l1 in range(L + 1):
        for l2 in range(L + 1):
            d = abs(l1 - l2)
            mats = _cg(min(l1, l2), max(l1, l2))
            for M in range(l1 + l2 + 1):
                if l1 <= l2:
                    A = mats[M]
                    lo = max(-l1, M - l2)
                    m1 = torch.arange(lo, lo + A.shape[1])
                    m2 = M - m1
                else:   # C_{l1 l2} = (-1)^(l1 + l2 - l3) C_{l2 l1}
                    lo = max(-l2, M - l1)
                    l3 = max(d, M) + np.arange(mats[M].shape[0])
                    A = mats[M] * np.where((l1 + l2 - l3) % 2 == 0, 1.0, -1.0)[:, None]
                    m2 = torch.arange(lo, lo + A.shape[1])
                    m1 = M - m2
                l3 = torch.arange(max(d, M), l1 + l2 + 1)
                par = 1.0 - 2.0 * ((l1 + l2 - l3) % 2).double()
                yield {"i1": l1 * l1 + l1 + m1, "j1": l1 * l1 + l1 - m1, "i2": l2 * l2 + l2 + m2,
                       "j2": l2 * l2 + l2 - m2, "o": off + l3 * l3 - d * d + l3 + M,
                       "p": off + l3 * l3 - d * d + l3 - M, "par": par, "M": M, "A": torch.from_numpy(np.ascontiguousarray(A))}
            off += (2 * l1 + 1) * (2 * l2 + 1)


def _cgtp(L, x1, x2):
    z = torch.zeros(x1.shape[0], (L + 1) ** 4, dtype=torch.float64, device=x1.device)
    t1, t2 = x1.double().t().contiguous(), x2.double().t().contiguous()
    for b in _orders(L):
        A = b["A"].to(z.device)
        z[:, b["o"]] = (A @ (t1[b["i1"]] * t2[b["i2"]])).t()
        if b["M"]:
            z[:, b["p"]] = ((b["par"][:, None].to(z.device) * A) @ (t1[b["j1"]] * t2[b["j2"]])).t()
    return z


def _cgtp_vjp(L, x1, x2, g):
    t1, t2, tg = x1.double().t().contiguous(), x2.double().t().contiguous(), g.t()
    g1, g2 = torch.zeros_like(t1), torch.zeros_like(t2)
    for b in _orders(L):
        A = b["A"].to(t1.device)
        signs = [("o", "i1", "i2", A)]
        if b["M"]:
            signs.append(("p", "j1", "j2", b["par"][:, None].to(t1.device) * A))
        for o, i, j, a in signs:
            T = a.t() @ tg[b[o]].double()
            g1[b[i]] += T * t2[b[j]]
            g2[b[j]] += T * t1[b[i]]
    return g1.t().contiguous(), g2.t().contiguous()


def _to_complex(L, r):
    """Complex coefficients of real-basis rows, [(L+1)^2, N]: c_0 = r_0, c_m = (-1)^m (r_m - i r_-m) / sqrt 2, c_-m = (r_m + i r_-m) / sqrt 2."""
    t = r.double().t().contiguous()
    c = t.to(torch.complex128)
    for l in range(L + 1):
        for m in range(1, l + 1):
            rp, rm = t[l * l + l + m] / math.sqrt(2), t[l * l + l - m] / math.sqrt(2)
            c[l * l + l + m] = (-1) ** m * torch.complex(rp, -rm)
            c[l * l + l - m] = torch.complex(rp, rm)
    return c


def _cgtp_real(L, x1, x2):
    z = torch.zeros(x1.shape[0], (L + 1) ** 4, dtype=torch.float64, device=x1.device)
    c1, c2 = _to_complex(L, x1), _to_complex(L, x2)
    for b in _orders(L):
        # the path at order -M; odd l1 + l2 + l3 after a factor i
        w = (b["par"][:, None].to(z.device) * b["A"].to(z.device)).to(torch.complex128) @ (c1[b["j1"]] * c2[b["j2"]])
        w = torch.where(b["par"][:, None].to(z.device) < 0, 1j * w, w)
        if b["M"] == 0:
            z[:, b["o"]] = w.real.t()
        else:
            z[:, b["o"]] = math.sqrt(2) * w.real.t()
            z[:, b["p"]] = math.sqrt(2) * w.imag.t()
    return z


def _labels(s, L):
    return [(j, l) for l in range(L + 1) for j in range(abs(l - s), l + s + 1)]


_GRID = {}


def _grid(L, device):
    """An exact grid for products of degree 4 L: harmonics [(l, m) up to 2 L][point], real and imaginary parts, and weights."""
    if L in _GRID:
        return _GRID[L]
    _GRID.clear()
    x, w = np.polynomial.legendre.leggauss(2 * L + 1)
    Phi, lm = 4 * L + 1, 2 * L
    p = np.zeros((lm + 1, lm + 1, len(x)))   # normalised P_l^m, Condon-Shortley phase
    p[0, 0] = math.sqrt(1 / (4 * math.pi))
    sx = np.sqrt(1 - x * x)
    for m in range(1, lm + 1):
        p[m, m] = -math.sqrt((2 * m + 1) / (2 * m)) * sx * p[m - 1, m - 1]
    for m in range(lm):
        p[m + 1, m] = math.sqrt(2 * m + 3) * x * p[m, m]
        for l in range(m + 2, lm + 1):
            a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
            b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1))
            p[l, m] = a * (x * p[l - 1, m] - b * p[l - 2, m])
    phi = 2 * math.pi * np.arange(Phi) / Phi
    yr, yi = np.zeros(((lm + 1) ** 2, len(x), Phi)), np.zeros(((lm + 1) ** 2, len(x), Phi))
    for l in range(lm + 1):
        for m in range(l + 1):
            re, im = p[l, m][:, None] * np.cos(m * phi), p[l, m][:, None] * np.sin(m * phi)
            yr[l * l + l + m], yi[l * l + l + m] = re, im
            yr[l * l + l - m], yi[l * l + l - m] = (-1) ** m * re, -(-1) ** m * im
    wt = np.repeat(w * 2 * math.pi / Phi, Phi)
    n = (lm + 1) ** 2
    _GRID[L] = tuple(torch.from_numpy(t).to(device) for t in (yr.reshape(n, -1), yi.reshape(n, -1), wt))
    return _GRID[L]


def _lift(s, L, device):
    """Per component q = -s..s: the matrix from label coefficients to scalar-harmonic ones, C^{j, m+q}_{l, m, s, q}."""
    nin = (2 * s + 1) * (L + 1) ** 2
    mats = np.zeros((2 * s + 1, nin, (L + 1) ** 2))
    off = 0
    for j, l in _labels(s, L):
        tab = _cg(l, s)
        for m3 in range(-j, j + 1):
            M = abs(m3)
            lo, lmin = max(-l, M - s), max(abs(l - s), M)
            row = tab[M][j - lmin]
            for t, c in enumerate(row):
                m, sg = lo + t, 1.0
                if m3 < 0:   # C at reversed orders: (-1)^(l + s - j)
                    m, sg = -m, (-1.0) ** (l + s - j)
                q = m3 - m
                mats[q + s, off + j + m3, l * l + l + m] = sg * c
        off += 2 * j + 1
    return [torch.from_numpy(mats[i]).to(device) for i in range(2 * s + 1)]


def _spin_product(s, L, x1, x2):
    """The (s, s, s) signal product of rows x1, x2 (64 bits), differentiable."""
    yr, yi, w = _grid(L, x1.device)
    n = (L + 1) ** 2
    lift, proj = _lift(s, L, x1.device), _lift(s, 2 * L, x1.device)
    f = []
    for x in (x1, x2):
        a = [x @ m for m in lift]
        f.append([(t @ yr[:n], t @ yi[:n]) for t in a])
    out = 0
    tab = _cg(s, s)
    for q in range(-s, s + 1):
        gr = gi = 0
        M = abs(q)
        row = tab[M][s - M]   # j = s; rows start at l3 = max(0, M)
        lo = max(-s, M - s)
        for t, c in enumerate(row):
            q1, sg = lo + t, float(c)
            if q < 0:
                q1, sg = -q1, sg * (-1.0) ** s
            q2 = q - q1
            (ar, ai), (br, bi) = f[0][q1 + s], f[1][q2 + s]
            gr = gr + sg * (ar * br - ai * bi)
            gi = gi + sg * (ar * bi + ai * br)
        b = (gr * w) @ yr.t() + (gi * w) @ yi.t()   # real: the coefficients are
        out = out + b @ proj[q + s].t()
    return out


def _gaunt_real(L, x1, x2):
    yr, yi, w = _grid(L, x1.device)
    lm = 2 * L
    rows = []
    for l in range(lm + 1):
        for m in range(-l, l + 1):
            k = l * l + l + abs(m)
            sg = math.sqrt(2) * (-1) ** m
            rows.append(yr[k] if m == 0 else sg * (yr[k] if m > 0 else yi[k]))
    y = torch.stack(rows)
    n = (L + 1) ** 2
    return ((x1 @ y[:n]) * (x2 @ y[:n]) * w) @ y.t()


def _in_chunks(fn, size, *rows):
    parts = [fn(*(r[k:k + size] for r in rows)) for k in range(0, rows[0].shape[0], size)]
    if isinstance(parts[0], tuple):
        return tuple(torch.cat(p) for p in zip(*parts))
    return torch.cat(parts)


def _with_grads(fn):
    def both(x1, x2, g):
        a, b = x1.double().requires_grad_(True), x2.double().requires_grad_(True)
        z = fn(a, b)
        g1, g2 = torch.autograd.grad(z, (a, b), g.double())
        return z.detach(), g1, g2
    return both


def exact(case, seed):
    d = _inputs(case, seed)
    op, L = case["op"], case["L"]
    if op == "cgtp":
        return _cgtp(L, d["x1"], d["x2"])
    if op == "cgtp_real":
        return _cgtp_real(L, d["x1"], d["x2"])
    if op == "cgtp_channels":
        N, C = case["N"], case["C"]
        z = _cgtp(L, d["x1"].reshape(N * C, -1), d["x2"].repeat_interleave(C, 0))
        sizes = [2 * l3 + 1 for l1 in range(L + 1) for l2 in range(L + 1) for l3 in range(abs(l1 - l2), l1 + l2 + 1)]
        path = torch.repeat_interleave(torch.arange(len(sizes)), torch.tensor(sizes)).to(z.device)
        z = z.reshape(N, C, -1)
        z *= d["w"].double()[..., path]
        return z
    if op == "cgtp_backward":
        return _cgtp_vjp(L, d["x1"], d["x2"], d["g"])
    if op == "cgtp_step":
        return (_cgtp(L, d["x1"], d["x2"]),) + _cgtp_vjp(L, d["x1"], d["x2"], d["g"])
    s = case["spin"]
    size = max(64, int(1.5e8 / ((2 * s + 1) * (2 * L + 1) * (4 * L + 1))) // (6 if "backward" in op or "step" in op else 2))
    if op == "istp":
        return _in_chunks(lambda a, b: _spin_product(s, L, a.double(), b.double()), size, d["x1"], d["x2"])
    if op == "istp_backward":
        return _in_chunks(lambda a, b, g: _with_grads(lambda u, v: _spin_product(s, L, u, v))(a, b, g)[1:], size,
                          d["x1"], d["x2"], d["g"])
    if op == "istp_real_step":
        return _in_chunks(_with_grads(lambda u, v: _gaunt_real(L, u, v)), size, d["x1"], d["x2"], d["g"])
    N, C = case["N"], case["C"]   # istp_channels
    li = [torch.repeat_interleave(torch.arange(len(lab)), torch.tensor([2 * j + 1 for j, _ in lab])).to(d["x1"].device)
          for lab in (_labels(s, L), _labels(s, 2 * L))]
    x1 = (d["x1"].double() * d["w1"].double()[:, li[0]]).reshape(N * C, -1)
    x2 = (d["x2"].double()[:, None, :] * d["w2"].double()[:, li[0]]).reshape(N * C, -1)
    z = _in_chunks(lambda a, b: _spin_product(s, L, a, b), size, x1, x2).reshape(N, C, -1)
    return z * d["wo"].double()[:, li[1]]
