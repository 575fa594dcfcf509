"""The workloads whose time is watched: tensor products as an equivariant network calls them.

A case names one entry point of ``Plan`` (``op``), the degrees, the largest spin, the real basis,
the element type and the sizes.  ``exact`` is the same product in float64, written here from its
definition (fields on an exact quadrature grid) with plain torch.
"""

import functools
import math

import numpy as np
import torch

from paper_2607_01408_amd import BASIS_M0_PAIRED, BASIS_PAPER, BASIS_PARITY, Plan, paths_host

_BASES = {"paper": BASIS_PAPER, "paired": BASIS_M0_PAIRED, "parity": BASIS_PARITY}
_DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}

# op: the entry points of one pass.
#   forward   forward: x1, x2 per (edge, channel)
#   backward  backward: both gradients of forward
#   edge      forward_v1 and backward_v1: x2 one row per edge, shared by its channels
#   unit      forward_weighted and backward_weighted: a weight per channel and path, x2 per channel
#   channel   forward_v1_weighted and backward_v1_weighted: the same with x2 one row per edge
#   depthwise forward_depthwise and backward_depthwise: the same with V rows of x2 per edge
#   full      forward_fully_connected and backward_fully_connected: all channel pairs mixed


def _case(name, op, L, N, C, dtype="fp32", basis="paper", smax=1, V=1, W=0):
    L1, L2, Lout = L
    case = {"op": op, "L1": L1, "L2": L2, "Lout": Lout, "smax": smax, "basis": basis, "dtype": dtype, "N": N, "C": C,
            "V": V, "W": W}
    return dict({"name": name}, **case) if name else case


def listed():
    return [
        # one small molecule through one layer: a handful of edges, so the launch is what counts
        _case("small_forward", "forward", (2, 2, 2), 64, 8),
        # message passing on a batch of small molecules (20,000 edges, 64 channels)
        _case("molecule_forward", "forward", (4, 4, 4), 20_000, 64),
        # the headline workload: a large batch of organic molecules at degree 6 in fp32
        _case("organic_forward", "forward", (6, 6, 6), 100_000, 128),
        # its training step's gradients, bf16 coefficients in the parity-labelled basis, a quarter of the batch
        _case("organic_backward", "backward", (6, 6, 6), 25_000, 128, dtype="bf16", basis="parity"),
        # inference on catalyst slabs: degree 8, bf16 coefficients
        _case("catalyst_forward", "forward", (8, 8, 8), 100_000, 128, dtype="bf16"),
        # high angular resolution: degree 12
        _case("sweep_forward", "forward", (12, 12, 12), 8_192, 32),
        # gradients at the largest degree, over a batch that fills no whole number of tiles
        _case("sweep_backward", "backward", (16, 16, 16), 1_999, 33),
        # chirality: spins -2..2 at degree 2, many small molecules
        _case("chiral_forward", "forward", (2, 2, 2), 200_000, 64, smax=2),
        # a training step with an edge feature shared by the channels (no weights), uneven channel count
        _case("edge_train", "edge", (3, 3, 3), 8_192, 100),
        # the depthwise layer of the published runtime table: 1,024 edges, 64 channels, a weight per channel and path
        _case("channel_train", "channel", (2, 2, 2), 1_024, 64),
        # the same layer with several edge features, first input capped at degree 1
        _case("depthwise_train", "depthwise", (1, 3, 3), 1_024, 128, basis="parity", V=4),
        # the fully connected layer: every input channel to every output channel
        _case("full_train", "full", (2, 2, 2), 1_024, 64, W=64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("forward", "forward", "forward", "backward", "backward", "edge", "unit", "channel", "depthwise", "full"))
    basis = rng.choice(("paper", "paper", "paired", "parity"))
    dtype = rng.choice(("fp32", "fp32", "bf16"))
    if op in ("forward", "backward"):
        kind = rng.choice(("square", "square", "square", "square", "chiral", "mixed"))
        if kind == "chiral":
            L, smax, units = (rng.choice((2, 2, 3)),) * 3, 2, 4_000_000
        elif kind == "mixed":
            L, smax, units = rng.choice(((1, 3, 3), (2, 1, 3), (3, 2, 4), (4, 2, 4))), 1, 2_000_000
        else:
            l = rng.randint(1, 16)
            L, smax = (l, l, l), 1
            units = int(min(12_000_000, 2.0e9 / (l + 1) ** 3 if l <= 8 else 4.0e8 / (l + 1) ** 3))
        C = rng.choice((8, 16, 32, 64, 128, _log(rng, 1, 200)))
        N = _log(rng, 8, max(8, units // (2 if op == "backward" else 1) // C))
        return _case("", op, L, N, C, dtype=dtype, basis=basis, smax=smax)
    if op == "edge":
        L = rng.randint(1, 6)
        C = rng.choice((16, 32, 64, 128, _log(rng, 1, 200)))
        return _case("", op, (L, L, L), _log(rng, 16, 1_500_000 // C // L), C, dtype=dtype, basis=basis)
    L = rng.choice(((1, 1, 1), (2, 2, 2), (1, 3, 3)))
    C = rng.choice((16, 64, 128, _log(rng, 4, 160)))
    N = _log(rng, 16, 2_048)
    if op == "full":
        return _case("", op, L, N, C, basis=basis, W=rng.choice((C, _log(rng, 4, 160))))
    V = rng.randint(2, 6) if op == "depthwise" else 1
    return _case("", op, L, N, C, dtype=dtype, basis=basis, V=V)


def _spins(case):
    return tuple(range(-case["smax"], case["smax"] + 1))


def _inputs(case, seed, n_paths):
    """The coefficients and weights of one pass, drawn on the GPU from the seed alone."""
    dev, spins = torch.device("cuda"), _spins(case)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))

    def coefficients(rows, channels, L):
        # normal coefficients of about the same power in every degree; there is no basis function at l < |s|
        live = torch.tensor([[l >= abs(s) for l in range(L + 1) for _ in range(2 * l + 1)] for s in spins],
                            device=dev)
        out = torch.empty((rows, channels) + tuple(live.shape), dtype=_DTYPES[case["dtype"]], device=dev)
        step = max(1, (1 << 28) // max(1, channels * live.numel()))
        for i in range(0, rows, step):
            part = out[i:i + step]
            part.copy_(torch.randn(part.shape, generator=gen, device=dev) * live)
        return out

    N, C, op = case["N"], case["C"], case["op"]
    x2_channels = {"forward": C, "backward": C, "unit": C}.get(op, case["V"])
    x1, x2 = coefficients(N, C, case["L1"]), coefficients(N, x2_channels, case["L2"])
    g = coefficients(N, case["W"] if op == "full" else C, case["Lout"]) if op != "forward" else None
    w = None
    shape = {"unit": (C, n_paths), "channel": (C, n_paths), "depthwise": (case["V"], C, n_paths),
             "full": (n_paths, C, case["V"], case["W"])}.get(op)
    if shape is not None:
        w = torch.randn(shape, generator=gen, device=dev)
        if op == "full":
            w = w / math.sqrt(C * case["V"])
    return x1, x2, g, w


def prepare(case, seed):
    weighted = case["op"] in ("unit", "channel", "depthwise")
    plan = Plan(case["L1"], case["L2"], case["Lout"], _spins(case), case["dtype"], basis=_BASES[case["basis"]],
                channel_weights=weighted, fully_connected=case["op"] == "full")
    x1, x2, g, w = _inputs(case, seed, plan.n_paths)
    return {"op": case["op"], "plan": plan, "x1": x1, "x2": x2, "g": g, "w": w}


def run(state):
    plan, x1, x2, g, w = (state[k] for k in ("plan", "x1", "x2", "g", "w"))
    op = state["op"]
    if op == "forward":
        return [plan.forward(x1, x2)]
    if op == "backward":
        return list(plan.backward(x1, x2, g))
    if op == "edge":
        return [plan.forward_v1(x1, x2), *plan.backward_v1(x1, x2, g)]
    if op == "unit":
        return [plan.forward_weighted(x1, x2, w), *plan.backward_weighted(x1, x2, w, g)]
    if op == "channel":
        return [plan.forward_v1_weighted(x1, x2, w), *plan.backward_v1_weighted(x1, x2, w, g)]
    if op == "depthwise":
        return [plan.forward_depthwise(x1, x2, w), *plan.backward_depthwise(x1, x2, w, g)]
    return [plan.forward_fully_connected(x1, x2, w), *plan.backward_fully_connected(x1, x2, w, g)]


# ---------------------------------------------------------------------------
# float64 reference


@functools.lru_cache(maxsize=8)
def _functions(L, Lmax_sum, smax, basis):
    """The real basis functions on an exact grid: complex [n_spins, n_coef, points] (sector s of each), and the
    points' weights.  Goldberg's explicit sum for the spin-weighted harmonics; real combinations of (s, m) and
    (-s, -m); the parity basis combines the sectors -|s| and +|s|."""
    spins = list(range(-smax, smax + 1))
    n_theta, n_phi = Lmax_sum // 2 + 1, Lmax_sum + 1
    z, w = np.polynomial.legendre.leggauss(n_theta)
    half, phi = np.arccos(z) / 2, 2 * math.pi * np.arange(n_phi) / n_phi
    n = (L + 1) ** 2

    def harmonic(s, l, m):
        norm = math.sqrt((2 * l + 1) / (4 * math.pi) * (math.factorial(l + m) * math.factorial(l - m))
                         / (math.factorial(l + s) * math.factorial(l - s)))
        total = np.zeros(n_theta)
        for r in range(l - s + 1):
            if 0 <= r + s - m <= l + s:
                k = 2 * r + s - m
                total += (-1) ** r * math.comb(l - s, r) * math.comb(l + s, r + s - m) * np.sin(half) ** (2 * l - k) * np.cos(half) ** k
        return np.outer((-1) ** (m + l - s) * norm * total, np.exp(1j * m * phi)).ravel()

    E = np.zeros((len(spins), len(spins) * n, n_theta * n_phi), dtype=np.complex128)
    r2 = 1 / math.sqrt(2)

    def add(col, s, l, m, c):
        E[s + smax, col] += c * harmonic(s, l, m)

    for i, s in enumerate(spins):
        for l in range(abs(s), L + 1):
            for k in range(-l, l + 1):
                col, a = i * n + l * l + l + k, abs(k)
                sign = (-1) ** (a + s)
                if k > 0:
                    add(col, s, l, k, r2)
                    add(col, -s, l, -k, sign * r2)
                elif k < 0:
                    add(col, s, l, a, 1j * r2)
                    add(col, -s, l, -a, -1j * sign * r2)
                elif s == 0 or basis != "paired":
                    add(col, s, l, 0, 1)
                else:
                    c = r2 if s > 0 else 1j * r2
                    add(col, abs(s), l, 0, c)
                    add(col, -abs(s), l, 0, (1 if s > 0 else -1) * (-1) ** s * c)
    if basis == "parity":
        for s in range(1, smax + 1):
            for l in range(s, L + 1):
                lo, hi = (smax - s) * n + l * l, (smax + s) * n + l * l
                a, b = E[:, lo:lo + 2 * l + 1].copy(), (-1) ** l * E[:, hi:hi + 2 * l + 1]
                E[:, lo:lo + 2 * l + 1], E[:, hi:hi + 2 * l + 1] = r2 * (a + b), r2 * (a - b)
    return E, np.repeat(w, n_phi) * (2 * math.pi / n_phi)


@functools.lru_cache(maxsize=4)
def _maps(L1, L2, Lout, smax, basis):
    dev, total = "cuda", L1 + L2 + Lout
    fields = []
    for L in (L1, L2, Lout):
        E, weight = _functions(L, total, smax, basis)
        if len(fields) == 2:
            E = E * weight
        # [n_coef, n_spins * 2 * points]: real and imaginary parts of each sector
        flat = np.stack([E.real, E.imag], axis=1).transpose(2, 0, 1, 3).reshape(E.shape[1], -1)
        fields.append(torch.from_numpy(np.ascontiguousarray(flat)).to(dev))
    return fields


def _product(x1, x2, maps, smax):
    """The product of rows x1 [units, n1] and x2 [units, n2] (or [1, n2]) in float64."""
    m1, m2, m3 = maps
    ns = 2 * smax + 1
    a = (x1 @ m1).reshape(x1.shape[0], ns, 2, -1)
    b = (x2 @ m2).reshape(x2.shape[0], ns, 2, -1)
    sectors = []
    for s3 in range(-smax, smax + 1):
        re = im = 0
        for s1 in range(-smax, smax + 1):
            s2 = s3 - s1
            if abs(s2) <= smax:
                p, q = a[:, s1 + smax], b[:, s2 + smax]
                re = re + p[:, 0] * q[:, 0] - p[:, 1] * q[:, 1]
                im = im + p[:, 0] * q[:, 1] + p[:, 1] * q[:, 0]
        sectors += [re, im]
    return torch.cat(sectors, dim=1) @ m3.T


def _tensor(case):
    """T [n1, n2, n3] of the product, and its paths: the block triples (slots) with a nonzero entry, in order."""
    maps = _maps(case["L1"], case["L2"], case["Lout"], case["smax"], case["basis"])
    n1, n2 = maps[0].shape[0], maps[1].shape[0]
    e1 = torch.eye(n1, dtype=torch.float64, device="cuda").repeat_interleave(n2, 0)
    e2 = torch.eye(n2, dtype=torch.float64, device="cuda").repeat(n1, 1)
    T = _product(e1, e2, maps, case["smax"]).reshape(n1, n2, -1)
    T = torch.where(T.abs() > 1e-12, T, torch.zeros_like(T))

    def blocks(L):
        n = (L + 1) ** 2
        return [slice(i * n + l * l, i * n + (l + 1) ** 2) for i in range(2 * case["smax"] + 1) for l in range(L + 1)]

    live = (T != 0).cpu().numpy()
    paths = [(a, b, c) for a in blocks(case["L1"]) for b in blocks(case["L2"]) for c in blocks(case["Lout"])
             if live[a, b, c].any()]
    return T, paths


def _flat64(t):
    return None if t is None else t.reshape(t.shape[0], t.shape[1], -1).double()


def _gradients(y, leaves, g):
    return [y.detach(), *torch.autograd.grad(y, leaves, g)]


def _shaped(rows, like, case):
    return rows.reshape(like, -1, 2 * case["smax"] + 1, rows.shape[-1] // (2 * case["smax"] + 1))


def exact(case, seed):
    op = case["op"]
    if op in ("forward", "backward", "edge"):
        x1, x2, g, _ = _inputs(case, seed, 0)
        maps = _maps(case["L1"], case["L2"], case["Lout"], case["smax"], case["basis"])
        N, C = case["N"], case["C"]
        step = max(1, int(3e8 / (C * maps[0].shape[1])))  # edges at a time
        parts = []
        for i in range(0, N, step):
            a, b = _flat64(x1[i:i + step]), _flat64(x2[i:i + step])
            n = a.shape[0]
            if op == "forward":
                y = _product(a.reshape(n * C, -1), b.reshape(n * C, -1), maps, case["smax"])
                parts.append([y.reshape(n, C, -1)])
                continue
            a.requires_grad_()
            b.requires_grad_()
            y = _product(a.reshape(n * C, -1), b.expand(n, C, b.shape[2]).reshape(n * C, -1), maps, case["smax"])
            got = _gradients(y.reshape(n, C, -1), (a, b), _flat64(g[i:i + step]))
            parts.append(got if op == "edge" else got[1:])
        whole = [torch.cat(p) for p in zip(*parts)]
        return [_shaped(t, N, case) for t in whole]
    T, paths = _tensor(case)
    x1, x2, g, w = _inputs(case, seed, len(paths))
    a, b, g = _flat64(x1).requires_grad_(), _flat64(x2).requires_grad_(), _flat64(g)
    w = w.double().requires_grad_()
    y = torch.zeros(g.shape, dtype=torch.float64, device=g.device)
    for p, (i, j, k) in enumerate(paths):
        t = T[i, j, k]
        n1, n2, n3 = t.shape
        left = (a[:, :, i].reshape(-1, n1) @ t.reshape(n1, -1)).reshape(a.shape[0], a.shape[1], n2, n3)
        if op in ("unit", "channel"):
            part = (left * b[:, :, j, None]).sum(2) * w[:, p, None]
        elif op == "depthwise":
            mixed = (w[:, :, p].T.unsqueeze(0).unsqueeze(-1) * b[:, None, :, j]).sum(2)  # [N, C, n2]
            part = (left * mixed.unsqueeze(-1)).sum(2)
        else:  # V = 1: the pairs are the channels of x1
            r = (left * b[:, :, j, None]).sum(2)
            part = (r.transpose(1, 2).reshape(-1, r.shape[1]) @ w[p, :, 0]).reshape(r.shape[0], n3, -1).transpose(1, 2)
        y = y + torch.nn.functional.pad(part, (k.start, g.shape[2] - k.stop))
    out = _gradients(y, (a, b, w), g)
    N = case["N"]
    return [_shaped(out[0], N, case), _shaped(out[1], N, case), _shaped(out[2], N, case), out[3]]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far two right answers can be apart


@functools.lru_cache(maxsize=64)
def _nonzeros(L1, L2, Lout, smax):
    """A bound on the nonzero entries of the real tensor: one per pair of orders and allowed degree triple."""
    total = 0
    for s1 in range(-smax, smax + 1):
        for s2 in range(-smax, smax + 1):
            s3 = s1 + s2
            if abs(s3) > smax:
                continue
            for l1 in range(abs(s1), L1 + 1):
                for l2 in range(abs(s2), L2 + 1):
                    for l3 in range(max(abs(s3), abs(l1 - l2)), min(Lout, l1 + l2) + 1):
                        total += min((2 * l1 + 1) * (2 * l2 + 1), (2 * l1 + 1) * (2 * l3 + 1), (2 * l2 + 1) * (2 * l3 + 1))
    return total


def _product_flops(case):
    """One product: the sparse tensor's entries, or the separable transforms where those are fewer."""
    L1, L2, Lout, smax = case["L1"], case["L2"], case["Lout"], case["smax"]
    direct = 3 * _nonzeros(L1, L2, Lout, smax)
    ns, n_theta, n_phi = 2 * smax + 1, (L1 + L2 + Lout) // 2 + 1, L1 + L2 + Lout + 1
    theta = sum(2 * ns * (L + 1) ** 2 for L in (L1, L2, Lout))
    phi = sum(ns * n_phi * (2 * L + 1) for L in (L1, L2, Lout))  # even and odd parts apart: half the products
    return min(direct, n_theta * (theta + phi + 2 * ns * ns * n_phi))


def work(case):
    ns = 2 * case["smax"] + 1
    n1, n2, n3 = (ns * (case[k] + 1) ** 2 for k in ("L1", "L2", "Lout"))
    size = 2 if case["dtype"] == "bf16" else 4
    N, C, V, op = case["N"], case["C"], case["V"], case["op"]
    product = _product_flops(case)
    if op == "forward":
        return {"bytes": N * C * size * (n1 + n2 + n3), "flops": N * C * product}
    if op == "backward":
        return {"bytes": N * C * size * (2 * n1 + 2 * n2 + n3), "flops": 2 * N * C * product}
    if op == "edge":
        return {"bytes": N * size * (C * (2 * n1 + 2 * n3) + 2 * n2), "flops": 3 * N * C * product}
    # forward and gradients of a weighted product: weights read, their gradient written
    widths = _path_outputs(case["L1"], case["L2"], case["Lout"], case["smax"], case["basis"])
    n_paths, direct = len(widths), 3 * _nonzeros(case["L1"], case["L2"], case["Lout"], case["smax"])
    if op == "full":
        W = case["W"]
        return {"bytes": 4 * (N * (2 * C * n1 + 2 * V * n2 + 2 * W * n3) + 2 * n_paths * C * V * W),
                "flops": 3 * N * C * V * (direct + 2 * sum(widths) * W)}
    x2_rows = C if op == "unit" else V
    return {"bytes": size * N * (2 * C * n1 + 2 * x2_rows * n2 + 2 * C * n3) + 8 * V * C * n_paths,
            "flops": 3 * N * C * V * (direct + 2 * sum(widths))}


@functools.lru_cache(maxsize=64)
def _path_outputs(L1, L2, Lout, smax, basis):
    """The widths of the output blocks of the weighted paths."""
    triples = paths_host(L1, L2, Lout, tuple(range(-smax, smax + 1)), _BASES[basis])
    return [2 * (int(b3) % (Lout + 1)) + 1 for _, _, b3 in triples]


def tolerance(case):
    # four times the measured error against exact(): bf16 results are 1.7e-3 off (their rounding), fp32 ones
    # up to 3e-7 (1.1e-6 where a gradient sums over all channel pairs or edges in the fully connected product)
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 0.05}
    rel = 4.5e-6 if case["op"] == "full" else 1.2e-6
    return {"rel": rel, "max": 40 * rel}
