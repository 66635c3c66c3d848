"""Cases that time the public entry points of the MBE(3)-OSV-MP2 library.

A case is one pass of what a user's program has the library do: the energy of
a molecule call by call, energy and gradient, a recorded step replayed, the
integral stage alone at the sizes of a large system, the split-precision
form, integrals over sparse fitting domains, pair screening and weak pairs,
randomized OSVs, and the localization that comes before all of them.

Molecules are stood in for by chains (short oligomers), jittered lattices of
four-orbital units (water clusters) and helices (peptides) with the sizes per
unit, the cutoff and the value distributions of the repository's workloads.
The geometry (and with it the pair and trimer lists and the OSV counts)
belongs to the case; every value (Fock matrix, virtual energies, OSVs, slabs)
is drawn from the seed.
"""
import math

import numpy as np
import torch

import paper_2603_16575_amd as m

DEV = "cuda:0"
AO_PER_ATOM = (14, 5, 5)  # AOs of the three atoms of a lattice unit


def listed():
    return [
        # a short oligomer, everything kept: the smallest call, latency and
        # launches count
        dict(name="chain8_energy", kind="energy", shape="chain", n=8, n_vir=64, n_aux=192,
             r_lo=12, r_hi=12, cutoff=99.0, tol=1e-8, precision="fp64", warm=True),
        # an oligomer in a differentiable program: caller's own integrals,
        # ragged sizes, energy_fn forward and backward
        dict(name="chain13_autograd", kind="autograd", shape="chain", n=13, n_vir=75, n_aux=205,
             r_lo=5, r_hi=19, cutoff=9.5, tol=1e-8, precision="fp64", warm=True),
        # one step of a geometry-scan or dynamics loop on a small cluster:
        # energy and gradient recorded once, replayed per step
        dict(name="lattice8_replay", kind="replay", shape="lattice", n=8, n_vir=160, n_aux=480,
             r_lo=12, r_hi=28, cutoff=6.0, tol=1e-7, precision="fp64", warm=True),
        # an energy in a basis with many OSVs per orbital (pair domains to 128)
        dict(name="lattice24_wide_energy", kind="energy", shape="lattice", n=24, n_vir=456,
             n_aux=1320, r_lo=24, r_hi=64, cutoff=6.0, tol=1e-7, precision="fp64", warm=True),
        # the 160-orbital water lattice: energy, and energy with gradient
        dict(name="lattice40_energy", kind="energy", shape="lattice", n=40, n_vir=800,
             n_aux=2400, r_lo=20, r_hi=40, cutoff=6.0, tol=1e-7, precision="fp64", warm=True),
        dict(name="lattice40_gradient", kind="gradient", shape="lattice", n=40, n_vir=800,
             n_aux=2400, r_lo=20, r_hi=40, cutoff=6.0, tol=1e-7, precision="fp64", warm=True),
        # the split-precision projection, odd dimensions
        dict(name="lattice18_split_energy", kind="energy", shape="lattice", n=18, n_vir=513,
             n_aux=1485, r_lo=20, r_hi=47, cutoff=6.0, tol=1e-7, precision="proj", warm=True),
        # integrals of a 48-orbital part of the 512-orbital lattice: its slab
        # dimensions, where the projection is the largest product there is
        dict(name="integrals_n2432", kind="integrals", shape="lattice", n=12, n_vir=2432,
             n_aux=7040, r_lo=24, r_hi=64, cutoff=6.0, tol=1e-7, precision="fp64", warm=True),
        # a peptide-like chain with sparse fitting domains at the paper's
        # threshold: metric, restricted slabs, restricted exchange integrals
        dict(name="helix128_fit", kind="fit", shape="helix", n=128, n_vir=512, n_aux=1536,
             r_lo=24, r_hi=80, cutoff=6.0, l_fit=1e-6),
        # all candidate pairs of the 160-orbital lattice screened and classed,
        # the energies of those beyond the fragment cutoff
        dict(name="lattice40_weak", kind="weak", shape="lattice", n=40, n_vir=800, n_aux=2400,
             r_lo=20, r_hi=40, cutoff=6.0),
        # OSVs of a peptide-like chain generated before anything else
        dict(name="helix96_rosv", kind="rosv", shape="helix", n=96, n_vir=384, n_aux=1152,
             l_fit=1e-6, n_max=96),
        # occupied orbitals of a 24-unit cluster localized
        dict(name="localize24", kind="localize", shape="lattice", n=24),
    ]


def draw(rng):
    """One more case of the listed ranges."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["energy", "energy", "gradient", "autograd", "replay", "wide", "split",
                       "integrals", "fit", "weak", "rosv", "localize"])
    if kind == "localize":
        return dict(kind=kind, shape="lattice", n=rng.randint(3, 24))
    if kind == "rosv":
        n = log_int(16, 96)
        return dict(kind=kind, shape="helix", n=n, n_vir=log_int(130, 420),
                    n_aux=log_int(300, 1300), l_fit=rng.choice([1e-6, 1e-7]),
                    n_max=rng.randint(40, 110))
    if kind == "fit":
        n = log_int(24, 140)
        return dict(kind=kind, shape="helix", n=n, n_vir=4 * n + rng.randint(0, 33),
                    n_aux=12 * n + rng.randint(0, 65), r_lo=rng.randint(8, 24),
                    r_hi=rng.randint(32, 80), cutoff=6.0, l_fit=rng.choice([1e-6, 1e-5, 1e-7]))
    if kind == "weak":
        n = log_int(8, 40)
        return dict(kind=kind, shape="lattice", n=n, n_vir=20 * n + rng.randint(0, 17),
                    n_aux=60 * n + rng.randint(0, 65), r_lo=rng.randint(10, 20),
                    r_hi=rng.randint(24, 40), cutoff=6.0)
    rest = dict(tol=1e-7, precision="fp64", warm=rng.random() < 0.75)
    if kind == "integrals":
        return dict(kind=kind, shape="lattice", n=rng.randint(2, 12), n_vir=log_int(300, 2432),
                    n_aux=log_int(900, 7040), r_lo=rng.randint(12, 24),
                    r_hi=rng.randint(32, 64), cutoff=6.0, **rest)
    if kind == "autograd" or (kind == "energy" and rng.random() < 0.5):
        rest["tol"] = 1e-8
        n, r_lo = rng.randint(3, 13), rng.randint(4, 12)
        return dict(kind=kind, shape="chain", n=n, n_vir=rng.randint(48, 140),
                    n_aux=rng.randint(150, 430), r_lo=r_lo, r_hi=r_lo + rng.randint(0, 10),
                    cutoff=rng.choice([6.5, 9.5, 99.0]), **rest)
    if kind == "wide":  # to the widest domains of the 1024-orbital helix's OSV counts
        n, r_lo = log_int(4, 18), rng.randint(16, 32)
        return dict(kind="energy", shape="lattice", n=n, n_vir=19 * n + rng.randint(120, 200),
                    n_aux=55 * n + rng.randint(0, 65), r_lo=r_lo, r_hi=rng.randint(48, 72),
                    cutoff=6.0, **rest)
    if kind == "split":
        rest["precision"] = rng.choice(["proj", "both"])
    n = log_int(4, 27) if kind != "replay" else log_int(2, 12)
    r_lo = rng.randint(8, 20)
    return dict(kind="energy" if kind == "split" else kind, shape="lattice", n=n,
                n_vir=20 * n + rng.randint(40, 90), n_aux=60 * n + rng.randint(0, 90),
                r_lo=r_lo, r_hi=r_lo + rng.randint(4, 20), cutoff=6.0, **rest)


# ---- geometry and lists (the case's own) -----------------------------------

def _lattice(n_units, spacing=2.8):
    """Orbital centres (four per unit) and atom centres (three per unit)."""
    g = np.random.default_rng([28, n_units])
    side = int(math.ceil(n_units ** (1.0 / 3.0) - 1e-9))
    tet = np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]]) / math.sqrt(3.0)
    orb, atom = [], []
    for u in range(n_units):
        c = spacing * np.array([u % side, (u // side) % side, u // side ** 2], dtype=float)
        c = c + g.uniform(-0.35, 0.35, 3)
        q, rr = np.linalg.qr(g.standard_normal((3, 3)))
        d = tet @ (q * np.sign(np.diag(rr))).T
        orb.append(c + 0.7 * d)
        atom += [c, c + 0.96 * d[0], c + 0.96 * d[1]]
    return np.concatenate(orb), np.array(atom)


def _centres(case):
    n = case["n"]
    k = np.arange(n, dtype=float)
    if case["shape"] == "chain":
        return np.stack([1.5 * k, 0 * k, 0 * k], 1)
    if case["shape"] == "helix":
        th = 2.0 * math.pi * k / 3.6
        return np.stack([2.3 * np.cos(th), 2.3 * np.sin(th), 1.5 * k], 1)
    return _lattice(n)[0]


def _dist(a, b):
    return np.sqrt(((a[:, None, :] - b[None, :, :]) ** 2).sum(-1))


def _lists(case):
    """Centres, OSV counts, kept pairs and fragments (rows padded with -1)."""
    x = _centres(case)
    n = len(x)
    r = np.random.default_rng([29, n]).integers(case.get("r_lo", 4), case.get("r_hi", 4) + 1, n)
    if case["kind"] == "rosv":  # no pairs yet at that stage
        adj = np.zeros((n, n), dtype=bool)
    else:
        adj = _dist(x, x) <= case["cutoff"]
    pairs = np.argwhere(np.triu(adj, 1)).astype(np.int32)
    frags = [np.stack([np.arange(n), np.full(n, -1), np.full(n, -1)], 1)]
    if len(pairs):
        frags.append(np.concatenate([pairs, np.full((len(pairs), 1), -1)], 1))
    if case["kind"] in ("energy", "gradient", "autograd", "replay"):
        for i, j in pairs:
            k = np.nonzero(adj[i] & adj[j])[0]
            k = k[k > j]
            if len(k):
                frags.append(np.stack([np.full(len(k), i), np.full(len(k), j), k], 1))
    return x, r.astype(np.int32), pairs, np.concatenate(frags).astype(np.int32)


def _values(case, seed):
    """Every input value, on the host; the slab seed among them."""
    x, r, pairs, frags = _lists(case)
    n, nv, na = len(x), case["n_vir"], case["n_aux"]
    g = np.random.default_rng([31, seed])
    lo, hi = x.min(0), x.max(0)
    x_vir = lo + (hi - lo) * g.uniform(size=(nv, 3))
    x_aux = lo + (hi - lo) * g.uniform(size=(na, 3))
    f = 0.05 * g.standard_normal((n, n)) * np.exp(-_dist(x, x) / 2.0)
    f = np.triu(f, 1)
    f = f + f.T + np.diag(g.uniform(-1.2, -0.4, n))
    eps = np.sort(g.uniform(0.2, 4.0, nv))
    d_ov = _dist(x, x_vir)
    Q = [np.linalg.qr(g.standard_normal((nv, int(ri))) * np.exp(-d_ov[i] / 2.0)[:, None])[0].T
         for i, ri in enumerate(r)]
    return dict(x=x, r=r, pairs=pairs, frags=frags, f=f, eps=eps, Q=Q, seed=int(seed) + 17,
                w_ia=0.1 * np.exp(-d_ov / 3.0), w_iP=np.exp(-_dist(x, x_aux) / 3.0))


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


def _explicit(case):
    return case["kind"] in ("autograd", "weak")


def _given_slab(v, case):
    """The caller's own (ia|P), [n_occ, n_vir, n_aux]."""
    g = torch.Generator(device=DEV)
    g.manual_seed(v["seed"])
    z = torch.randn((len(v["r"]), case["n_vir"], case["n_aux"]), generator=g,
                    dtype=torch.float64, device=DEV)
    z *= _dev(v["w_ia"])[:, :, None]
    z *= _dev(v["w_iP"])[:, None, :]
    return z


def _charges_input(case, seed):
    """Delocalized orthonormal MO coefficients and the AO offsets of the atoms."""
    x, atoms = _lattice(case["n"])
    n_ao = np.tile(AO_PER_ATOM, case["n"])
    off = np.concatenate([[0], np.cumsum(n_ao)]).astype(np.int32)
    g = np.random.default_rng([37, seed])
    d = _dist(np.repeat(atoms, n_ao, axis=0), x)
    c, _ = np.linalg.qr(g.standard_normal(d.shape) * np.exp(-2.0 * d))
    mix, _ = np.linalg.qr(g.standard_normal((len(x), len(x))))
    return c @ mix, off


def _weak_inputs(case, v):
    """Candidate pairs, those beyond the cutoff (the weak ones, left out of the
    fragment list), and diagonal-pair amplitudes."""
    n = len(v["r"])
    cand = np.argwhere(np.triu(np.ones((n, n), dtype=bool), 1)).astype(np.int32)
    far = cand[_dist(v["x"], v["x"])[cand[:, 0], cand[:, 1]] > case["cutoff"]]
    g = np.random.default_rng([41, v["seed"]])
    T = []
    for ri in v["r"]:
        a = 1e-2 * g.standard_normal((int(ri), int(ri)))
        T.append(a + a.T)
    return cand, far, T


# ---- what a user's program has in hand, and one pass ------------------------

PRECISION = dict(fp64=m.MBE3_FP64, proj=m.MBE3_MIXED_BF16_PROJ, both=m.MBE3_MIXED_BF16)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "localize":
        C, off = _charges_input(case, seed)
        return dict(kind=kind, C=_dev(C), off=off)
    v = _values(case, seed)
    slab = _given_slab(v, case) if _explicit(case) else None
    f = _dev(v["f"])
    if kind == "autograd":
        slab.requires_grad_(True)
        f.requires_grad_(True)
    src = dict(slab=slab) if slab is not None else dict(w_ia=_dev(v["w_ia"]),
                                                        w_iP=_dev(v["w_iP"]))
    h = m.Mbe3(r=v["r"], Q=_dev(np.concatenate(v["Q"])), eps_vir=_dev(v["eps"]), f_occ=f,
               pairs=v["pairs"], frags=v["frags"], seed=v["seed"], tol=case.get("tol", 1e-7),
               precision=PRECISION[case.get("precision", "fp64")],
               warm_start=case.get("warm", True), **src)
    st = dict(kind=kind, h=h, case=case, f=f, slab=slab)
    if kind == "replay":
        st["buffers"] = h.capture_step(grad=True)
    if kind == "weak":
        st["cand"], st["far"], T = _weak_inputs(case, v)
        st["gamma"] = h.osv_project(h.empty_gamma())
        W = np.zeros(int(h.layout.k_elems))
        for i, t in enumerate(T):
            W[h.k_off[i]:h.k_off[i + 1]] = t.reshape(-1)
        st["W"] = _dev(W)
    return st


def run(st):
    kind = st["kind"]
    if kind == "localize":
        return m.pm_localize(st["C"], st["off"])
    h = st["h"]
    if kind == "energy":
        out = h.forward()
        out["E"] = np.float64(out["E"])
        return {k: out[k] for k in ("E", "e_frag", "iters", "gamma", "K")}
    if kind == "gradient":
        out = h.forward(grad=True)
        dF = torch.empty_like(st["f"])
        dB, _ = h.mbe3_backward(out["gamma"], out["W"], dEdF=dF)
        out["E"] = np.float64(out["E"])
        out = {k: out[k] for k in ("E", "e_frag", "iters", "gamma", "K", "W")}
        return dict(out, dB=dB, dF=dF)
    if kind == "autograd":
        st["slab"].grad = st["f"].grad = None
        E = m.energy_fn(h, st["slab"], st["f"])
        E.backward()
        return dict(E=E, dB=st["slab"].grad, dF=st["f"].grad)
    if kind == "replay":
        E = h.graph_launch()
        b = st["buffers"]
        out = {k: b[k] for k in ("e_frag", "iters", "gamma", "K", "W", "dB")}
        return dict(out, E=np.float64(E), dF=b["dEdF"])
    if kind == "integrals":
        gamma = h.osv_project(h.empty_gamma())
        return dict(gamma=gamma, K=h.pair_K(gamma, h.empty_K()))
    if kind == "fit":
        s = h.fit_metric()
        gamma = h.project_fit(s, st["case"]["l_fit"], h.empty_gamma())
        K = h.pair_K_fit(s, st["case"]["l_fit"], h.empty_K())
        return dict(s_fit=s, gamma=gamma, K=K)
    if kind == "weak":
        s2b = h.screen(st["cand"])
        lists = m.screen_lists(h.n_occ, st["cand"], s2b.cpu().numpy())
        e = h.weak_pairs(st["far"], st["gamma"], st["W"])
        return dict(s2b=s2b, classes=lists["classes"], e=e)
    s = h.fit_metric()  # rosv
    out = h.rosv(n_max=st["case"]["n_max"], s_fit=s, l_fit=st["case"]["l_fit"])
    return dict(out, s_fit=s)


# ---- what a pass cannot do without ------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "localize":  # charges, then at least two sweeps over all pairs
        n, na = 4 * case["n"], 3 * case["n"]
        n_ao = sum(AO_PER_ATOM) * case["n"]
        return dict(bytes=8.0 * (n_ao * n + n * n * (na + 1)),
                    flops=2.0 * n * n * n_ao + 2 * (n * (n - 1) / 2) * 6.0 * n * na)
    x, r, pairs, frags = _lists(case)
    n, nv, na = len(x), case["n_vir"], case["n_aux"]
    r = r.astype(float)
    rows = r.copy()  # gamma rows per LMO
    np.add.at(rows, pairs[:, 0], r[pairs[:, 1]])
    np.add.at(rows, pairs[:, 1], r[pairs[:, 0]])
    d2 = np.concatenate([r, r[pairs[:, 0]] + r[pairs[:, 1]]]) ** 2
    read = 8.0 * (r.sum() * nv + n * (nv + na) + n * n + nv)
    if _explicit(case):
        read += 8.0 * n * nv * na
    project, pair_K = 2.0 * rows.sum() * nv * na, 2.0 * d2.sum() * na
    gamma_K = 8.0 * (rows.sum() * na + d2.sum())
    if kind == "integrals":
        return dict(bytes=read + gamma_K, flops=project + pair_K)
    if kind == "fit":  # a few percent of the columns are kept at these thresholds
        return dict(bytes=read + gamma_K + 8.0 * n * na, flops=2.0 * n * nv * na)
    if kind == "weak":
        c = r.sum() ** 2 / 2.0  # sum of r_i r_j over all pairs
        far = 1.0 - 2.0 * len(pairs) / (n * (n - 1.0))
        return dict(bytes=8.0 * (r.sum() * (nv + na) + n * n),
                    flops=c * (2.0 * nv + far * (2.0 * na + 8.0 * r.mean())))
    if kind == "rosv":
        return dict(bytes=read + 8.0 * n * (case["n_max"] * nv + na),
                    flops=2.0 * n * nv * na + 4.0 * n * 30 * nv * nv)
    # residual products of two evaluations per fragment, 2 d_t d_s (d_t + d_s)
    # per coupling term
    def term(dt, ds):
        return 2.0 * dt * ds * (dt + ds)

    solve = 0.0
    p, q = r[pairs[:, 0]], r[pairs[:, 1]]
    solve += 2 * (2 * term(p, p + q) + 2 * term(q, p + q)).sum()
    t = frags[frags[:, 2] >= 0]
    if len(t):
        a, b, c = r[t[:, 0]], r[t[:, 1]], r[t[:, 2]]
        s = 0.0
        for u, w, z in ((a, b, c), (b, c, a), (c, a, b)):
            s = s + 2 * term(u, u + w) + 2 * term(w, u + w) + 2 * term(u + w, u + z)
        solve += 2 * s.sum()
    flops, nbytes = project + pair_K + solve, read + gamma_K + 12.0 * len(frags)
    if kind != "energy":  # the products' adjoints, each as large as the product
        flops += project + 2 * pair_K + 0.5 * solve
        nbytes += 8.0 * (d2.sum() + n * nv * na + n * n)
    return dict(bytes=nbytes, flops=flops)


# ---- the same results in plain 64-bit arithmetic ------------------------------

def _mulhi(a, b):
    """High words of the unsigned 64 x 64 bit products (int64 tensors, int b)."""
    lo32 = 0xFFFFFFFF
    a0, a1, b0, b1 = a & lo32, (a >> 32) & lo32, b & lo32, b >> 32
    p = (a0 * b0 >> 32) & lo32
    m1, m2 = a1 * b0, a0 * b1
    mid = p + (m1 & lo32) + (m2 & lo32)
    return a1 * b1 + ((m1 >> 32) & lo32) + ((m2 >> 32) & lo32) + ((mid >> 32) & lo32)


def _signed(x):
    x &= 0xFFFFFFFFFFFFFFFF
    return x - (1 << 64) if x >> 63 else x


def _normals(seed, stream, lmo, rows, cols):
    """Box-Muller normals of words 0, 1 of the Philox4x64-10 blocks at counters
    (col, row, lmo, 0) under key (seed, stream), [rows, cols]."""
    i64 = dict(dtype=torch.int64, device=DEV)
    c = [torch.arange(cols, **i64).expand(rows, cols), torch.arange(rows, **i64)[:, None].expand(rows, cols),
         torch.full((rows, cols), lmo, **i64), torch.zeros((rows, cols), **i64)]
    M0, M1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    k0, k1 = seed, stream
    for _ in range(10):
        hi0, lo0 = _mulhi(c[0], M0), c[0] * _signed(M0)
        hi1, lo1 = _mulhi(c[2], M1), c[2] * _signed(M1)
        c = [hi1 ^ c[1] ^ _signed(k0), lo1, hi0 ^ c[3] ^ _signed(k1), lo0]
        k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    w0, w1 = (c[0] >> 11) & ((1 << 53) - 1), (c[1] >> 11) & ((1 << 53) - 1)
    u1, u2 = (w0.double() + 0.5) * 2.0 ** -53, w1.double() * 2.0 ** -53
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)


def _slab(v, case, i, given=None):
    if given is not None:
        return given[i]
    z = _normals(v["seed"], 0, i, case["n_vir"], case["n_aux"])
    return z * _dev(v["w_ia"][i])[:, None] * _dev(v["w_iP"][i])[None, :]


def _neighbours(v):
    n = len(v["r"])
    adj = np.eye(n, dtype=bool)
    adj[v["pairs"][:, 0], v["pairs"][:, 1]] = adj[v["pairs"][:, 1], v["pairs"][:, 0]] = True
    return [np.nonzero(a)[0] for a in adj]


def _gamma_blocks(v, case, given=None):
    """G[i][x] = Q_x^T B_i over x in N+(i)."""
    Q = [_dev(q) for q in v["Q"]]
    out = []
    for i, nb in enumerate(_neighbours(v)):
        B = _slab(v, case, i, given)
        g = torch.cat([Q[x] for x in nb]) @ B
        out.append(dict(zip(nb.tolist(), g.split([int(v["r"][x]) for x in nb]))))
    return out


def _pair_list(v):
    n = len(v["r"])
    return [(i, i) for i in range(n)] + [tuple(int(k) for k in p) for p in v["pairs"]]


def _orbs(p, q):
    return (p,) if p == q else (p, q)


def _K_blocks(v, G, keep=None):
    """K_pq by pair; keep(p, q): the auxiliary columns summed over."""
    K = {}
    for p, q in _pair_list(v):
        L = torch.cat([G[p][x] for x in _orbs(p, q)])
        R = torch.cat([G[q][x] for x in _orbs(p, q)])
        if keep is not None:
            c = keep(p, q)
            L, R = L[:, c], R[:, c]
        K[p, q] = L @ R.T
    return K


def _flat(blocks):
    return torch.cat([b.reshape(-1) for b in blocks])


class _Host:
    """The residual equations of every fragment, block by block on the host."""

    def __init__(self, v, K):
        self.v, self.r, self.f = v, v["r"], v["f"]
        self.K = {t: b.cpu().numpy() for t, b in K.items()}
        self.S0, self.basis_ = {}, {}

    def blocks(self, A, B, weight=None):
        Q = self.v["Q"]
        V, U = np.concatenate([Q[a] for a in A]), np.concatenate([Q[b] for b in B])
        return (V if weight is None else V * weight) @ U.T

    def S(self, A, B):
        if (A, B) not in self.S0:
            self.S0[A, B] = self.blocks(A, B)
        return self.S0[A, B]

    def basis(self, t):
        if t not in self.basis_:
            o = _orbs(*t)
            S, F = self.blocks(o, o), self.blocks(o, o, self.v["eps"])
            s, U = np.linalg.eigh(S)
            X0 = U[:, s > 1e-8] / np.sqrt(s[s > 1e-8])
            e, Z = np.linalg.eigh(X0.T @ F @ X0)
            self.basis_[t] = X0 @ Z, e, F
        return self.basis_[t]

    def T(self, T, p, q):
        """Amplitudes of the ordered pair, rows in the order of (p, q)'s domain."""
        if p <= q:
            return T[p, q]
        a = int(self.r[q])
        t = T[q, p].T
        return np.block([[t[a:, a:], t[a:, :a]], [t[:a, a:], t[:a, :a]]])

    def residual(self, t, frag, T):
        p, q = t
        o = _orbs(p, q)
        S, F = self.S(o, o), self.basis(t)[2]
        R = self.K[t] + F @ T[t] @ S + S @ T[t] @ F
        for k in frag:
            A = self.S(o, _orbs(k, q))
            R = R - self.f[p, k] * (A @ self.T(T, k, q) @ A.T)
            A = self.S(o, _orbs(p, k))
            R = R - self.f[k, q] * (A @ self.T(T, p, k) @ A.T)
        return R

    def solve(self, frag, tol, start):
        slots = [(p, q) for a, p in enumerate(frag) for q in frag[a:]]
        T = {t: np.zeros_like(self.K[t]) if start is None else start[t] for t in slots}
        for _ in range(101):
            R = {t: self.residual(t, frag, T) for t in slots}
            X = {t: self.basis(t)[0] for t in slots}
            Rt = {t: X[t].T @ R[t] @ X[t] for t in slots}
            if max(np.abs(Rt[t]).max() for t in slots) < tol:
                break
            new = {}
            for t in slots:
                e = self.basis(t)[1]
                den = self.f[t[0], t[0]] + self.f[t[1], t[1]] - e[:, None] - e[None, :]
                new[t] = T[t] + X[t] @ (Rt[t] / den) @ X[t].T
            T = new
        E = sum((1 if p == q else 2) * np.sum((2 * T[p, q] - T[p, q].T)
                                              * (self.K[p, q] + R[p, q])) for p, q in slots)
        return E, T

    def all(self, case):
        """Fragment energies, amplitudes and MBE(3) coefficients."""
        e, Ts, own = [], [], {}
        frags = [tuple(int(k) for k in f if k >= 0) for f in self.v["frags"]]
        c = {f: 1.0 for f in frags}
        for f in frags:
            if len(f) == 3:
                for g in ((f[0], f[1]), (f[0], f[2]), (f[1], f[2])):
                    c[g] -= 1.0
        for f in frags:  # a monomer's coefficient: 1 - those of what contains it
            if len(f) == 1:
                c[f] = 1.0 - sum(c[g] for g in frags if len(g) > 1 and f[0] in g)
        for f in frags:  # monomers, dimers, trimers
            E, T = self.solve(f, case["tol"], own if len(f) == 3 and case["warm"] else None)
            if len(f) < 3:
                own[f[0], f[-1]] = T[f[0], f[-1]]
            e.append(E)
            Ts.append(T)
        return frags, np.array(e), Ts, np.array([c[f] for f in frags])




def _exact_localize(case, seed):
    C, off = _charges_input(case, seed)
    n, na = C.shape[1], len(off) - 1
    P = np.zeros((n, n, na))
    for a in range(na):
        c = C[off[a]:off[a + 1]]
        P[:, :, a] = c.T @ c
    U, dL, rot = np.eye(n), [], []
    while not dL or (dL[-1] > m.L_LOC and len(dL) < 100):
        gain, count = 0.0, 0
        for i in range(n):
            for j in range(i + 1, n):
                d = P[i, i] - P[j, j]
                a = P[i, j] @ P[i, j] - 0.25 * (d @ d)
                b = P[i, j] @ d
                th = 0.25 * math.atan2(b, -a)
                if abs(math.sin(th)) < 1e-10:
                    continue
                co, si = math.cos(th), math.sin(th)
                gain += math.hypot(a, b) * (1.0 - math.cos(4.0 * th))
                count += 1
                G = np.array([[co, -si], [si, co]])
                U[:, [i, j]] = U[:, [i, j]] @ G
                rows = P[[i, j]].reshape(2, -1)
                P[[i, j]] = (G.T @ rows).reshape(2, n, na)
                ci, cj = P[:, i].copy(), P[:, j].copy()
                P[:, i], P[:, j] = co * ci + si * cj, co * cj - si * ci
        dL.append(gain)
        rot.append(count)
    return dict(U=U, P=P, dL=np.array(dL), rotations=None, sweeps=None, status=None)


def _exact_rosv(case, v):
    """Kept singular values of the adaptive range finder, per LMO."""
    n, nv, nm = len(v["r"]), case["n_vir"], case["n_max"]
    s_fit = torch.zeros((n, case["n_aux"]), dtype=torch.float64)
    w = np.zeros((n, nm))
    for i in range(n):
        B = _slab(v, case, i)
        s_fit[i] = (B * B).sum(0).cpu()
        B = B[:, (s_fit[i] > case["l_fit"]).to(B.device)]
        den = _dev(v["eps"])[:, None] + _dev(v["eps"])[None, :] - 2.0 * v["f"][i, i]
        T = ((B @ B.T) / den).cpu().numpy()
        G = _normals(v["seed"], 11, i, 10 + nm, nv).cpu().numpy()
        Y = G @ T
        pending, Z, nxt = list(Y[:10]), np.zeros((0, nv)), 10
        thr = 1e-4 / (10.0 * math.sqrt(2.0 / math.pi))
        while len(Z) < nm and max(np.linalg.norm(y) for y in pending) > thr:
            y = pending.pop(0)
            y = y - Z.T @ (Z @ y)
            z = y / np.linalg.norm(y)
            new = Y[nxt] - Z.T @ (Z @ Y[nxt])
            nxt += 1
            pending.append(new)
            Z = np.concatenate([Z, z[None]])
            pending = [y - z * (z @ y) for y in pending]
        s = np.linalg.svd(Z @ T, compute_uv=False) if len(Z) else np.zeros(0)
        s = s[s >= 1e-4]
        w[i, :len(s)] = s
    return dict(Q=None, w=w, n_osv=None, rows=None, s_fit=s_fit)


def _exact_weak(case, v):
    given = _given_slab(v, case)
    cand, far, T = _weak_inputs(case, v)
    n = len(v["r"])
    s2b = np.array([np.sum((v["Q"][i] @ v["Q"][j].T) ** 2) / math.sqrt(len(v["Q"][i]) * len(v["Q"][j]))
                    for i, j in cand])
    G = [(_dev(v["Q"][i]) @ given[i]).cpu().numpy() for i in range(n)]
    base = []
    for i in range(n):
        q = v["Q"][i]
        s, U = np.linalg.eigh(q @ q.T)
        X0 = U / np.sqrt(s)
        e, Z = np.linalg.eigh(X0.T @ ((q * v["eps"]) @ q.T) @ X0)
        base.append((X0 @ Z, e))
    e = []
    for i, j in far:
        K = G[i] @ G[j].T
        S = v["Q"][i] @ v["Q"][j].T
        f = v["f"]
        Xi, Xj = base[i][0], base[j][0]
        Kt = Xi.T @ K @ Xj
        D = Xi.T @ (T[i] @ S + S @ T[j]) @ Xj
        den = f[i, i] + f[j, j] - base[i][1][:, None] - base[j][1][None, :]
        e.append(4.0 * np.sum(Kt * (Kt - f[i, j] * D) / den))
    return dict(s2b=s2b, classes=None, e=np.array(e))


def exact(case, seed):
    kind = case["kind"]
    if kind == "localize":
        return _exact_localize(case, seed)
    v = _values(case, seed)
    if kind == "rosv":
        return _exact_rosv(case, v)
    if kind == "weak":
        return _exact_weak(case, v)
    given = _given_slab(v, case) if _explicit(case) else None
    nbr = _neighbours(v)
    if kind == "fit":
        return _exact_fit(case, v, nbr)
    if kind == "autograd":
        return _exact_autograd(case, v, given)
    G = _gamma_blocks(v, case, given)
    K = _K_blocks(v, G)
    out = dict(gamma=_flat([g for Gi in G for g in Gi.values()]), K=_flat(K.values()))
    if kind == "integrals":
        return out
    none = dict(E=None, e_frag=None, iters=None)
    if kind != "energy":
        none.update(W=None, dB=None, dF=None)
    if len(v["frags"]) <= 600 and kind == "energy":
        _, e, _, c = _Host(v, K).all(case)
        none.update(E=np.float64(math.fsum(e * c)), e_frag=e)
    return dict(none, **out)


def _exact_fit(case, v, nbr):
    n = len(v["r"])
    s = torch.stack([(_slab(v, case, i) ** 2).sum(0) for i in range(n)])
    D = s > case["l_fit"]
    G = _gamma_blocks(v, case)
    K = _K_blocks(v, G, keep=lambda p, q: D[p] | D[q])
    rows = []
    for i, Gi in enumerate(G):
        C = D[torch.as_tensor(nbr[i], device=D.device)].any(0)
        for x, g in Gi.items():
            rows.append(g * (C if x == i else D[i] | D[x]))
    return dict(s_fit=s, gamma=_flat(rows), K=_flat(K.values()))


def _exact_autograd(case, v, given):
    """The functional's explicit derivatives at the converged amplitudes."""
    n = len(v["r"])
    with torch.no_grad():
        K = _K_blocks(v, _gamma_blocks(v, case, given))
    host = _Host(v, K)
    frags, e, Ts, c = host.all(case)
    W, dF = {}, np.zeros((n, n))
    for frag, T, cF in zip(frags, Ts, c):
        for t, x in T.items():
            W[t] = W.get(t, 0.0) + cF * (2.0 * x - x.T)
        for x in frag:
            for y in frag:
                acc = 0.0
                for q in frag:
                    A = host.S(_orbs(x, q), _orbs(y, q))
                    t = host.T(T, x, q)
                    acc += np.sum((2.0 * t - t.T) * (A @ host.T(T, y, q) @ A.T))
                    A = host.S(_orbs(q, y), _orbs(q, x))
                    t = host.T(T, q, y)
                    acc += np.sum((2.0 * t - t.T) * (A @ host.T(T, q, x) @ A.T))
                dF[x, y] -= cF * acc
    dB = torch.zeros_like(given)
    Q = [_dev(q) for q in v["Q"]]
    for p, q in _pair_list(v):
        V = torch.cat([Q[x] for x in _orbs(p, q)])
        w = _dev(W[p, q])
        if p == q:
            dB[p] += 2.0 * V.T @ ((w + w.T) @ (V @ given[p]))
        else:
            dB[p] += 4.0 * V.T @ (w @ (V @ given[q]))
            dB[q] += 4.0 * V.T @ (w.T @ (V @ given[p]))
    return dict(E=np.float64(math.fsum(e * c)), dB=dB, dF=0.5 * (dF + dF.T))
