"""The calls that a program using this package makes, over the sizes it makes them at.

Each case is one call (or, for the MASTER pipeline, the three calls that go together) through the
public entry points of ``paper_2602_15605_amd.couple``.  ``listed`` gives the standard ones,
``draw`` others of the same ranges; ``prepare`` holds what a program has in hand before the call
(context, windows, bin edges, measured spectra), ``run`` is one pass, ``work`` the bytes and
operations that the pass cannot do without, and ``exact`` the same outputs from float64 matrix
products in plain torch, without this package.
"""
import math

import numpy as np
import torch

from paper_2602_15605_amd import couple

F_SKY = 0.4
POL4 = "TT,TE,EE,BB"


def listed():
    return [
        # the smallest standard workload: one temperature window, where launches and latency count
        {"name": "tt_lmax256_fp64", "kind": "matrix", "lmax": 256, "spectra": "TT", "precision": "fp64", "lc": 100.0},
        # an ordinary survey at HEALPix-like resolution, all four spectra in the default precision
        {"name": "pol4_lmax2000_fp64", "kind": "matrix", "lmax": 2000, "spectra": POL4, "precision": "fp64",
         "lc": 250.0},
        # the headline workload in both precisions that it is quoted in
        {"name": "pol4_lmax6000_fp32c", "kind": "matrix", "lmax": 6000, "spectra": POL4, "precision": "fp32c",
         "lc": 1500.0},
        {"name": "pol4_lmax6000_fp64", "kind": "matrix", "lmax": 6000, "spectra": POL4, "precision": "fp64",
         "lc": 1500.0},
        # the two single-spectrum kernels that the paper times at lmax = 10^4
        {"name": "tt_lmax10000_fp64", "kind": "matrix", "lmax": 10000, "spectra": "TT", "precision": "fp64",
         "lc": 1500.0},
        {"name": "ee_lmax10000_fp64", "kind": "matrix", "lmax": 10000, "spectra": "EE", "precision": "fp64",
         "lc": 1500.0},
        # many masks of uneven lmax in one call, in its default precision
        {"name": "batched32_lmax500to4000_mfma_fp32", "kind": "batched", "n_masks": 32, "lmax_lo": 500,
         "lmax_hi": 4000, "sizes_seed": 3000, "spectra": POL4, "precision": "mfma_fp32"},
        # band-limited windows of eight masks, binned: few multipoles of the window, many of the map
        {"name": "band8_lmax10000_cut1000_fp32c", "kind": "band", "n_masks": 8, "lmax": 10000, "l3_hi": 1000,
         "bin_width": 50, "spectra": "TT,EE,BB", "precision": "fp32c", "lc": 250.0},
        # a power-spectrum estimate end to end: binned E/B coupling (odd L too), binned spectra, solve;
        # an odd lmax whose last bin is short
        {"name": "master_lmax1499_bins25_fp64", "kind": "master", "lmax": 1499, "bin_width": 25, "lc": 300.0,
         "precision": "fp64"},
        # the E/B system of narrow bins (three multipoles at lmax = 6000): 4000 unknowns
        {"name": "solve_eb_4000", "kind": "solve", "n": 2000, "pol": True, "n_rhs": 1},
        # rows of 3j symbols: the lensing weights (-1 1 0) and the largest family, (2 2 -4)
        {"name": "rows_m1_2000pairs_lmax6000", "kind": "rows", "n_pairs": 2000, "lmax": 6000, "m1": -1, "m2": 1},
        {"name": "rows_224_2000pairs_lmax6000", "kind": "rows", "n_pairs": 2000, "lmax": 6000, "m1": 2, "m2": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["matrix", "matrix", "matrix", "batched", "band", "master", "solve", "rows"])
    if kind == "matrix":
        # lmax up to 6000 (four spectra, with or without odd L) or 10000 (one spectrum)
        spectra = rng.choice(["TT", "EE", "TE", "TT,EE", "EE,BB", POL4, POL4, POL4 + ",EB", "EB", "EE,BB,EB"])
        hi = 10000 if spectra in ("TT", "EE") else 4500 if "EB" in spectra else 6000
        lmax = _log_int(rng, 48, hi)
        return {"kind": kind, "lmax": lmax, "spectra": spectra, "precision": rng.choice(["fp64", "fp64", "fp32c"]),
                "lc": max(10.0, lmax * rng.uniform(0.1, 0.4)), "xi": rng.random() < 0.2}
    if kind == "batched":
        lo = _log_int(rng, 100, 1000)
        return {"kind": kind, "n_masks": rng.randint(2, 32), "lmax_lo": lo, "lmax_hi": min(4000, int(lo * rng.uniform(1.2, 8.0))),
                "sizes_seed": rng.randrange(1 << 20), "spectra": rng.choice([POL4, POL4, "TT", "TT,EE,BB"]),
                "precision": rng.choice(["mfma_fp32", "mfma_bf16x3", "fp32c", "fp64"])}
    if kind == "band":
        lmax = _log_int(rng, 500, 10000)
        return {"kind": kind, "n_masks": rng.randint(1, 8), "lmax": lmax, "l3_hi": _log_int(rng, 50, min(lmax, 1200)),
                "bin_width": rng.randint(5, 60), "spectra": rng.choice(["TT,EE,BB", "TT", "EE,BB,EB", POL4]),
                "precision": rng.choice(["fp32c", "fp64"]), "lc": rng.uniform(50.0, 300.0)}
    if kind == "master":
        lmax = _log_int(rng, 200, 3000)
        return {"kind": kind, "lmax": lmax, "bin_width": rng.randint(max(5, lmax // 120), max(6, lmax // 20)),
                "lc": lmax * rng.uniform(0.1, 0.3), "precision": rng.choice(["fp64", "fp32c"])}
    if kind == "solve":
        pol = rng.random() < 0.6
        m = _log_int(rng, 40, 4000)
        return {"kind": kind, "n": max(2, m // 2 if pol else m), "pol": pol, "n_rhs": rng.choice([1, 1, 1, 2, 5])}
    m1, m2 = rng.choice([(0, 0), (-1, 1), (-2, 2), (1, 1), (2, 2), (2, -1), (-1, -1), (2, 1)])
    return {"kind": kind, "n_pairs": _log_int(rng, 50, 2000), "lmax": _log_int(rng, 100, 6000), "m1": m1, "m2": m2}


# ---------------------------------------------------------------------------------------------
# inputs


def _window(lmax, lc, seed, cut=None):
    """A survey window's spectrum: steeply falling, positive, with a log-normal scatter of a tenth."""
    ell = np.arange(2 * lmax + 1, dtype=np.float64)
    z = np.random.default_rng(seed).standard_normal(2 * lmax + 1)
    w = 4.0 * math.pi * F_SKY * (ell + 1.0) ** -2 * np.exp(-(ell / lc) ** 2 + 0.1 * z)
    w[0] = 4.0 * math.pi * F_SKY
    if cut is not None:
        w[cut + 1:] = 0.0
    return w


def _masks(case, seed):
    """Per mask (lmax, [W_TT, W_TP, W_PP]) as numpy arrays, None for a window that no spectrum uses."""
    sp = _spectra(case)
    need = ("TT" in sp, "TE" in sp, bool({"EE", "BB", "EB"} & set(sp)))
    if case["kind"] == "batched":
        lm = np.random.default_rng(case["sizes_seed"]).integers(case["lmax_lo"], case["lmax_hi"] + 1, case["n_masks"])
        sizes = [(int(x), int(x) / 4.0) for x in lm]
    else:
        sizes = [(case["lmax"], case["lc"])] * case.get("n_masks", 1)
    return [(L, [_window(L, lc, [seed, m, x], case.get("l3_hi")) if need[x] else None for x in range(3)])
            for m, (L, lc) in enumerate(sizes)]


def _spectra(case):
    return ("EE", "BB", "EB") if case["kind"] == "master" else tuple(case["spectra"].split(","))


def _edges(case):
    first = 2 if case["kind"] == "master" else 0
    e = list(range(first, case["lmax"] + 1, case["bin_width"]))
    return e + [case["lmax"] + 1]


def _measured(case, seed):
    """Pseudo-spectra [2, lmax+1] (EE, BB) of a falling signal with scatter."""
    ell = np.arange(case["lmax"] + 1, dtype=np.float64)
    z = np.random.default_rng([seed, 77]).standard_normal((2, case["lmax"] + 1))
    return np.stack([(ell + 10.0) ** -2, 0.1 * (ell + 10.0) ** -2]) * np.exp(0.05 * z)


def _system(case, seed):
    """A binned coupling matrix ([n, n], or [3, n, n] for EE, BB, EB) and its right-hand sides, on the GPU."""
    n, pol, r = case["n"], case["pol"], case["n_rhs"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    i = torch.arange(n, dtype=torch.float64, device="cuda")
    fall = (1.0 + (i[:, None] - i[None, :]).abs()) ** -2
    scatter = 1.0 + 0.1 * torch.randn((3 if pol else 1, n, n), dtype=torch.float64, device="cuda", generator=gen)
    K = F_SKY * 0.1 * fall * scatter
    K[: 2 if pol else 1] += F_SKY * 0.9 * torch.eye(n, dtype=torch.float64, device="cuda")
    if pol:
        K[2] *= 0.2
    m = 2 * n if pol else n
    rhs = torch.rand((r, m), dtype=torch.float64, device="cuda", generator=gen) + 0.5
    return K if pol else K[0], rhs


def _pairs(case, seed):
    l12 = np.random.default_rng([seed, 5]).integers(2, case["lmax"] + 1, (2, case["n_pairs"]))
    return l12[0].astype(np.int32), l12[1].astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        K, rhs = _system(case, seed)
        m = rhs.shape[1]
        work = torch.empty(m * (m + rhs.shape[0]), dtype=torch.float64, device="cuda")
        return {"case": case, "ctx": couple.couple_init(64), "K": K, "rhs": rhs, "work": work}
    if kind == "rows":
        l1, l2 = (torch.as_tensor(x).cuda() for x in _pairs(case, seed))
        return {"case": case, "ctx": couple.couple_init(case["lmax"]), "l1": l1, "l2": l2}
    masks = _masks(case, seed)
    w = [[None if x is None else torch.as_tensor(x).cuda() for x in ws] for _, ws in masks]
    state = {"case": case, "ctx": couple.couple_init(max(L for L, _ in masks)), "lmax": [L for L, _ in masks],
             "spectra": _spectra(case), "w": w,
             "lists": [[ws[x] for ws in w] if w[0][x] is not None else None for x in range(3)]}
    if kind == "batched":
        couple.couple_reserve_batched(state["ctx"], state["lmax"])
    if kind in ("band", "master"):
        state["edges"] = _edges(case)
    if kind == "master":
        state["measured"] = torch.as_tensor(_measured(case, seed)).cuda()
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "matrix":
        return couple.couple_matrix(ctx, *state["w"][0], case["lmax"], spectra=state["spectra"],
                                    precision=case["precision"], xi=case.get("xi", False))
    if kind == "batched":
        return couple.couple_matrix_batched(ctx, state["lmax"], *state["lists"], spectra=state["spectra"],
                                            precision=case["precision"])
    if kind == "band":
        return couple.couple_band_batched(ctx, 0, case["l3_hi"], *state["lists"], case["lmax"],
                                          spectra=state["spectra"], precision=case["precision"],
                                          bin_edges=state["edges"])
    if kind == "master":
        K = couple.couple_band(ctx, 0, 2 * case["lmax"], None, None, state["w"][0][2], case["lmax"],
                               spectra=state["spectra"], precision=case["precision"], bin_edges=state["edges"])
        cb = couple.couple_bin_spectra(ctx, state["measured"], state["edges"])
        return {"K": K, "C": couple.couple_master_solve(ctx, K, cb.reshape(-1), pol=True)}
    if kind == "solve":
        return couple.couple_master_solve(ctx, state["K"], state["rhs"], pol=case["pol"], work=state["work"])
    if case["m1"] == -case["m2"] and case["m2"] >= 0:
        return couple.couple_threej_rows(ctx, state["l1"], state["l2"], case["m2"], stride=2 * case["lmax"] + 1)
    return couple.couple_threej_rows_m(ctx, state["l1"], state["l2"], case["m1"], case["m2"],
                                       stride=2 * case["lmax"] + 1)


# ---------------------------------------------------------------------------------------------
# bytes and operations


def _triples(lmax, l3_hi):
    """(l1, l2, l3) of one parity of L with l1 <= l2 <= lmax and l3 <= l3_hi, and their pairs."""
    d = np.arange(min(lmax, l3_hi) + 1, dtype=np.float64)
    most = np.floor((l3_hi - d) / 2.0)            # the largest k (l3 = d + 2k) inside the band
    rows = lmax - d                               # l1 = 0 .. lmax - d, k = 0 .. min(l1, most)
    full = np.minimum(rows, most)
    terms = (full + 1.0) * (full + 2.0) / 2.0 + (rows - full) * (most + 1.0) * (rows > most)
    return float(terms.sum()), float((rows + 1.0).sum())


def _per_triple(spectra):
    """Operations per triple once every factor of two of the three multipoles is a table: one product and
    sum per spectrum, the polynomial N' (2) and its products with the symbol."""
    sp, n = set(spectra), 0
    n += 2 if "TT" in sp else 0
    if sp & {"TE", "EE", "BB"}:
        n += 3 + (2 if "TE" in sp else 0) + (3 if sp & {"EE", "BB"} else 0)
    return n + (5 if "EB" in sp else 0)


def work(case):
    kind = case["kind"]
    if kind == "solve":
        m = case["n"] * (2 if case["pol"] else 1)
        return {"bytes": 8.0 * ((3 if case["pol"] else 1) * case["n"] ** 2 + 2 * m * case["n_rhs"]),
                "flops": 2.0 / 3.0 * m ** 3 + 2.0 * m ** 2 * case["n_rhs"]}
    if kind == "rows":
        return {"bytes": 8.0 * case["n_pairs"] * (2 * case["lmax"] + 1),
                "flops": 10.0 * case["n_pairs"] * (2.0 / 3.0) * case["lmax"]}
    sp = _spectra(case)
    windows = len({{"TT": 0, "TE": 1}.get(s, 2) for s in sp})
    nbytes = flops = 0.0
    if kind == "batched":
        sizes = [int(x) for x in np.random.default_rng(case["sizes_seed"]).integers(
            case["lmax_lo"], case["lmax_hi"] + 1, case["n_masks"])]
    else:
        sizes = [case["lmax"]] * case.get("n_masks", 1)
    for L in sizes:
        hi = min(case.get("l3_hi", 2 * L), 2 * L)
        n = len(_edges(case)) - 1 if kind in ("band", "master") else L + 1
        flops += _triples(L, hi)[0] * _per_triple(sp)
        nbytes += 8.0 * (windows * (hi + 1) + len(sp) * n * n)
    if kind == "master":
        m = 2 * (len(_edges(case)) - 1)
        flops += 2.0 / 3.0 * m ** 3
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------------------------
# the same outputs in float64, in plain torch


def _tables(n):
    """g(p) and 1 / ((2p + 1) g(p)), p = 0 .. n, from the running product in extended precision."""
    p = np.arange(n + 1, dtype=np.longdouble)
    r = np.ones(n + 1, dtype=np.longdouble)
    r[1:] = (2 * p[1:] - 1) / (2 * p[1:])
    g = np.cumprod(r)
    return (torch.as_tensor(x.astype(np.float64)).cuda() for x in (g, 1 / ((2 * p + 1) * g)))


def _product(g, h, par, lmax, l3_hi):
    """For l3 = 2i + par, s = l1 + l2 = 2j + par, d = l2 - l1 = 2k + par: the squared (0 0 0) symbol as
    B[j, i] A[i, k], and the three index vectors."""
    ni = (min(l3_hi, 2 * lmax) - par) // 2 + 1
    nj = lmax + 1 - par
    nk = (min(lmax, l3_hi) - par) // 2 + 1
    i, j, k = (torch.arange(max(0, n), device="cuda") for n in (ni, nj, nk))
    A = torch.where(i[:, None] >= k[None, :], g[(i[:, None] - k[None, :]).clamp(min=0)] * g[i[:, None] + k[None, :] + par], 0.0)
    B = torch.where(j[:, None] >= i[None, :], g[(j[:, None] - i[None, :]).clamp(min=0)] * h[j[:, None] + i[None, :] + par], 0.0)
    return B, A, i, j, k


def _couplings(lmax, windows, spectra, l3_hi, xi):
    """K^X (or Xi_X) [lmax+1, lmax+1] of each spectrum for one mask."""
    g, h = _tables(2 * lmax + 2)
    l3_hi = min(l3_hi, 2 * lmax)
    ell = torch.arange(lmax + 1, dtype=torch.float64, device="cuda")
    cl = torch.where(ell >= 2, 1.0 / torch.sqrt(((ell - 1) * ell * (ell + 1) * (ell + 2)).clamp(min=1.0)), 0.0)
    out = {s: torch.zeros((lmax + 1, lmax + 1), dtype=torch.float64, device="cuda") for s in spectra if s != "BB"}
    if "BB" in spectra:
        out.setdefault("EE", torch.zeros((lmax + 1, lmax + 1), dtype=torch.float64, device="cuda"))
    wp = [None if w is None else torch.as_tensor(w * (2.0 * np.arange(len(w)) + 1.0) / (4.0 * math.pi)).cuda() for w in windows]

    def put(name, X, l1, l2):
        ok = (l1 >= 0) & (l2 >= l1) & (l2 <= lmax)
        a, b, v = l1[ok], l2[ok], X[ok]
        out[name][a, b] = v if xi else v * (2.0 * b + 1.0)
        out[name][b, a] = v if xi else v * (2.0 * a + 1.0)

    for par in (0, 1):
        if set(spectra) - {"EB"}:
            B, A, i, j, k = _product(g, h, par, lmax, l3_hi)
            if not len(k):
                continue
            l3, s, d = 2 * i + par, 2 * j + par, 2 * k + par
            l1, l2 = j[:, None] - k[None, :], j[:, None] + k[None, :] + par
            if "TT" in out:
                put("TT", B @ (wp[0][l3][:, None] * A), l1, l2)
            if "TE" in out or "EE" in out:
                # N' = f e + G with f = c - (s+1)^2 + 1, e = c - d^2 + 2 and G of s and d alone
                c = (l3 * (l3 + 1)).double()
                S, D = ((s + 1) ** 2).double(), (d ** 2).double()
                Bf = B * (c[None, :] - S[:, None] + 1.0)
                e = c[:, None] - D[None, :] + 2.0
                G = ((S[:, None] - D[None, :]) ** 2 + 6.0 * S[:, None] - 2.0 * D[None, :] - 7.0) / 8.0
                sf = 0.5 * cl[l1.clamp(0, lmax)] * cl[l2.clamp(0, lmax)]
                if "TE" in out:
                    U = wp[1][l3][:, None] * A
                    put("TE", sf * (Bf @ (U * e) + G * (B @ U)), l1, l2)
                if "EE" in out:
                    U = wp[2][l3][:, None] * A
                    t0, t1 = B @ U, Bf @ (U * e)
                    Bf *= c[None, :] - S[:, None] + 1.0
                    put("EE", sf * sf * (Bf @ (U * e * e) + 2.0 * G * t1 + G * G * t0), l1, l2)
        if "EB" in out:
            # odd L: the (0 0 0) symbol of (l1, l2 + 1, l3), s = l1 + l2 + 1 and d = l2 + 1 - l1
            B, A, i, j, k = _product(g, h, par, lmax + 1, l3_hi)
            l3, s, d = 2 * i + par, 2 * j + par, 2 * k + par
            l1, l2 = j[:, None] - k[None, :], j[:, None] + k[None, :] + par - 1
            c = (l3 * (l3 + 1)).double()
            B = B * ((s * (s + 1)).double()[:, None] - c[None, :])
            U = wp[2][l3][:, None] * A * (c[:, None] - (d * (d - 1)).double()[None, :])
            mu = (2 * (l1 + 2) * (l2 + 2) - (s[:, None] + 1) * (s[:, None] + 2)).double()
            sf = 0.5 * cl[l1.clamp(0, lmax)] * cl[l2.clamp(0, lmax)]
            X = B @ (U * c[:, None] ** 2) + 2.0 * mu * (B @ (U * c[:, None])) + mu * mu * (B @ U)
            put("EB", sf * sf * X, l1, l2)
    return [out["EE" if s == "BB" else s] for s in spectra]


def _bin_matrix(edges, lmax):
    """[n_bins, lmax + 1]: 1 where a multipole is in the bin."""
    lo, hi = (torch.as_tensor(edges[q:len(edges) - 1 + q], device="cuda") for q in (0, 1))
    ell = torch.arange(lmax + 1, device="cuda")
    return ((ell >= lo[:, None]) & (ell < hi[:, None])).double()


def _rows_exact(case, seed):
    l1, l2 = (torch.as_tensor(x).cuda().long()[:, None] for x in _pairs(case, seed))
    g, h = _tables(2 * case["lmax"] + 2)
    i = torch.arange(2 * case["lmax"] + 1, device="cuda")[None, :]
    l3 = (l1 - l2).abs() + i
    inside = l3 <= l1 + l2
    l3 = torch.where(inside, l3, (l1 - l2).abs())
    m = (case["m1"], case["m2"], -case["m1"] - case["m2"])
    ls = (l1, l2, l3)
    # columns rotated so that the first two magnetic numbers share a sign, then flipped to >= 0
    for rot in range(3):
        a, b = m[rot], m[(rot + 1) % 3]
        if 0 <= a <= 2 and 0 <= b <= 2 or -2 <= a <= 0 and -2 <= b <= 0:
            break
    flip = a < 0 or b < 0
    a, b = abs(a), abs(b)
    x, y, z = ls[rot], ls[(rot + 1) % 3], ls[(rot + 2) % 3]
    L = l1 + l2 + l3
    odd = (L & 1).bool()
    P = (L + 1) // 2
    base = g[P - l1] * g[P - l2] * g[P - l3] * h[P]
    base = torch.where(odd, base * (8.0 * (P - l1).double() * (P - l2) * (P - l3)) * (L + 2), base)
    A, B, C = (v.double() * (v + 1) for v in (x, y, z))
    s, t = A - B, A + B
    even_n, odd_n = {
        (0, 0): (2.0 + 0 * C, 0 * C),
        (0, 1): (s - C, 1.0 + 0 * C),
        (0, 2): (C * C - C * (t + s + 2) + s * s + 2 * s, s - C + 2),
        (1, 0): (-(s + C), -1.0 + 0 * C),
        (1, 1): (C * t - s * s, -s + 0 * C),
        (1, 2): (-C * C * A + C * ((s * s + 3 * s * t) / 2 + s + 3 * t) - s ** 3 - 3 * s * s - s * t, C * A - s * s - 3 * s - t),
        (2, 0): (C * C - C * (t - s + 2) + s * s - 2 * s, s + C - 2),
        (2, 1): (-C * C * B + C * ((s * s - 3 * s * t) / 2 - s + 3 * t) + s ** 3 - 3 * s * s + s * t, -C * B + s * s - 3 * s + t),
        (2, 2): (C * C * ((s * s + t * t) / 2 - 2 * t) + C * (-2 * s * s * t + s * s - 3 * t * t + 12 * t) + s * s * (s * s + 4 * t - 12),
                 s * (C * (2 - t) + s * s + 4 * t - 12)),
    }[(a, b)]
    d2 = torch.ones_like(C)
    for v, q in ((A, a), (B, b), (C, a + b)):
        for r in range(q):
            d2 = d2 * (v - r * (r + 1))
    v = torch.sqrt(base) * torch.where(odd, odd_n, even_n) / (2.0 * torch.sqrt(d2))
    v = torch.where((P & 1).bool() ^ (odd & flip), -v, v)
    return torch.where(inside & (x >= a) & (y >= b) & (z >= a + b), v, 0.0)


def exact(case, seed):
    kind = case["kind"]
    if kind == "rows":
        return _rows_exact(case, seed)
    if kind == "solve":
        K, rhs = (t.cpu().numpy() for t in _system(case, seed))
        M = np.block([[K[0], K[2]], [K[2], K[1]]]) if case["pol"] else K
        return torch.as_tensor(np.ascontiguousarray(np.linalg.solve(M, rhs.T).T))
    sp, masks = _spectra(case), _masks(case, seed)
    if kind == "matrix":
        return torch.stack(_couplings(case["lmax"], masks[0][1], sp, 2 * case["lmax"], case.get("xi", False)))
    if kind == "batched":
        return [torch.stack(_couplings(L, ws, sp, 2 * L, False)) for L, ws in masks]
    R = _bin_matrix(_edges(case), case["lmax"])
    binned = [torch.stack([(R @ K @ R.T.contiguous()) / R.sum(1)[:, None] for K in
                           _couplings(L, ws, sp, case.get("l3_hi", 2 * L), False)]) for L, ws in masks]
    if kind == "band":
        return torch.stack(binned)
    EE, BB, EB = (k.cpu().numpy() for k in binned[0])
    cb = R.cpu().numpy() @ _measured(case, seed).T / R.sum(1).cpu().numpy()[:, None]
    C = np.linalg.solve(np.block([[EE, EB], [EB, BB]]), cb.T.reshape(-1))
    return {"K": binned[0], "C": torch.as_tensor(C)}
