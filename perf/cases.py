"""Cases that stand for the work of a program using this library.

The usual program is a self-consistency loop: the geometry (block pattern,
groups, plan) stays, every pass brings new values of K in device memory and
takes D, N = Tr D and E = Tr(D K) back.  A case therefore fixes the geometry,
``prepare`` loads it into a context and draws new values from the seed, and
``run`` is one pass of the loop through the public entry points.

Kinds of cases:
  density  K -> D, N, E by the sign iteration (every precision mode)
  grad     the same and the gradient of a loss through the torch function
  fermi    K -> D, N, E at an electronic temperature (diagonalisation)
  mu       Algorithm 1: the chemical potential of a given electron count
  split    the density path on element-level sub-submatrices, D back in K's layout
"""

from __future__ import annotations

import functools
import math
import types

import numpy as np
import torch

import paper_2004_10811_amd as smx
from waterbox import WATER_CONFIGS, random_block_system, water_system

# block sizes of the ragged systems (single functions to large blocks)
RAGGED = (13, 5, 5, 17, 9, 31, 22, 13, 27, 11, 5, 25, 1, 7, 3)
SPREAD = 0.1        # relative change of K's elements from pass to pass
STEPS = 15          # Newton-Schulz steps of a typical group, for work()


def _water(name, kind="density", precision="fp64", config=None, **more):
    c = dict(WATER_CONFIGS[config or name.split("_")[0]])
    return dict(dict(name=name, kind=kind, system="water", precision=precision, elem=c.get("elem_decay", False),
                     n_mol=c["n_mol"], box=c["box"], r_cut=c["r_cut"], geometry=c["seed"], groups="molecule"), **more)


def listed():
    return [
        # the smallest call: a fragment of twelve blocks, one submatrix per block column
        dict(name="ragged12_fp64", kind="density", system="ragged", precision="fp64", nblk=12, density=0.45,
             geometry=101, groups="column"),
        # one molecular cell inside a self-consistency loop, in full and in reduced precision
        _water("water16_fp64"),
        _water("water16_fp16x2", precision="fp16x2"),
        # a medium cell whose molecule count fits nothing, shorter cutoff
        dict(name="water100_fp64", kind="density", system="water", precision="fp64", elem=False, n_mol=100, box=14.4,
             r_cut=5.0, geometry=11, groups="molecule"),
        # the ordinary production cell in the production precision
        _water("water256_fp16x2", precision="fp16x2"),
        # the same cell grouped by k-means (uneven groups), bulk in single precision
        _water("water256_kmeans_fp32", precision="fp32", groups="kmeans", clusters=384),
        # element-sparse cell, one sub-submatrix per column: thousands of small groups
        _water("water256e_split_fp16x2", kind="split", precision="fp16x2", eps=1e-5),
        # forces: D and the gradient of a loss of D, N and E in K (mu is held fixed: with a gap
        # at mu the derivative in mu is zero but for rounding)
        _water("water256_grad_fp64", kind="grad"),
        # metallic smearing: Fermi occupation at kT = 0.01 Ha
        _water("water256_fermi", kind="fermi", kT=0.01),
        # chemical potential for a fixed electron count, small cell
        dict(name="water32_mu", kind="mu", system="water", precision="fp64", elem=False, n_mol=32, box=9.85, r_cut=4.5,
             geometry=21, groups="molecule", kT=0.01),
        # the large cell in the production precision, and its full-precision reference run
        _water("water1024_fp16x2", precision="fp16x2"),
        _water("water1024_fp64"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["density"] * 6 + ["grad", "fermi", "mu", "split"])
    precision = "fp64"
    if kind == "density":
        precision = rng.choice(["fp64", "fp64", "fp16x2", "fp16x2", "fp32", "bf16x3"])
    elif kind == "grad":
        precision = rng.choice(["fp64", "fp16x2"])
    elif kind == "split":
        precision = rng.choice(["fp64", "fp16x2"])
    if kind in ("density", "grad") and rng.random() < 0.25:
        return dict(kind=kind, system="ragged", precision=precision, nblk=rng.randint(6, 60),
                    density=round(rng.uniform(0.2, 0.6), 2), geometry=rng.randrange(1000),
                    groups=rng.choice(["column", "pairs"]))
    hi = {"density": 500, "grad": 150, "fermi": 200, "mu": 64, "split": 200}[kind]
    n_mol = log_int(8, hi)
    case = dict(kind=kind, system="water", precision=precision, elem=kind == "split", n_mol=n_mol,
                box=round(3.1 * n_mol ** (1 / 3), 2), r_cut=round(rng.uniform(4.0, 6.0), 2),
                geometry=rng.randrange(1000), groups="molecule")
    if kind == "split":
        case["eps"] = 1e-5
    if kind in ("fermi", "mu"):
        case["kT"] = rng.choice([0.005, 0.01, 0.05])
    if kind == "density" and rng.random() < 0.25:
        case["groups"] = "kmeans"
        case["clusters"] = max(2, int(n_mol * rng.uniform(0.7, 1.5)))
    return case


# ---- geometry and values ----------------------------------------------------

@functools.lru_cache(maxsize=2)
def _geometry(key):
    case = dict(key)
    if case["system"] == "ragged":
        sizes = [RAGGED[i % len(RAGGED)] for i in range(case["nblk"])]
        return random_block_system(case["geometry"], sizes, density=case["density"], coupling=0.04,
                                   groups=case["groups"], mu=0.01)
    s = water_system(case["n_mol"], case["box"], case["r_cut"], case["geometry"], elem_decay=case["elem"],
                     eps_filter=1e-5 if case["elem"] else 0.0)
    if case["groups"] == "kmeans":
        s.grp_ptr, s.grp_blocks = smx.group_kmeans(s.coords, case["clusters"], box=case["box"], seed=3)
    return s


def _system(case):
    return _geometry(tuple(sorted((k, v) for k, v in case.items()
                                  if k not in ("name", "kind", "precision", "kT", "eps"))))


def _positions(s, device):
    """Row, column and mirrored position (the transposed element's) of every stored value."""
    bs = torch.as_tensor(s.blk_size.astype(np.int64), device=device)
    boff = torch.cumsum(bs, 0) - bs
    cols = torch.repeat_interleave(torch.arange(s.nblk, device=device),
                                   torch.as_tensor(np.diff(s.col_ptr), device=device))
    rows = torch.as_tensor(s.row_idx.astype(np.int64), device=device)
    voff = torch.as_tensor(s.val_off(), device=device)
    key = cols * s.nblk + rows                       # ascending: storage order
    mirror = torch.searchsorted(key, rows * s.nblk + cols)
    blk = torch.repeat_interleave(torch.arange(len(rows), device=device), voff[1:] - voff[:-1])
    at = torch.arange(len(blk), device=device) - voff[blk]
    bi, bj = bs[rows[blk]], bs[cols[blk]]
    r, c = at % bi, at // bi
    return boff[rows[blk]] + r, boff[cols[blk]] + c, voff[mirror[blk]] + c + r * bj


def _values(s, seed, device="cuda"):
    """K of one pass: the geometry's elements changed by about ten per cent, symmetric."""
    g = torch.Generator(device=device).manual_seed(int(seed))
    base = torch.as_tensor(s.values, device=device)
    f = torch.randn(len(base), generator=g, device=device, dtype=torch.float64)
    _, _, mirror = _positions(s, device)
    return base * (1.0 + SPREAD * math.sqrt(0.5) * (f + f[mirror]))


def _weights(s, seed, device="cuda"):
    """dL/dD of the grad cases' loss L = E + 0.1 N + <G, D>."""
    g = torch.Generator(device=device).manual_seed(int(seed) + 1_000_003)
    return 0.1 * torch.randn(len(s.values), generator=g, device=device, dtype=torch.float64)


# ---- one pass ----------------------------------------------------------------

def prepare(case, seed):
    s = _system(case)
    st = types.SimpleNamespace(kind=case["kind"], mu=s.mu)
    st.ctx = smx.Context(0, stream=torch.cuda.current_stream().cuda_stream)
    st.k = _values(s, seed)
    if case["kind"] == "split":
        part = smx.split_columns(s, case["eps"])
        st.ctx.load(part)
        st.src = part.src
        st.k_split = st.k[torch.as_tensor(part.src, device="cuda")]
        st.d = torch.empty_like(st.k)
    else:
        st.ctx.load(s)
        st.d = torch.empty_like(st.k)
    st.ctx.configure(precision=case["precision"], kT=case.get("kT"))
    if case["kind"] == "grad":
        st.gd = _weights(s, seed)
        st.sign = smx.SubmatrixSign(st.ctx)
    if case["kind"] == "mu":
        st.n_target = 0.5 * s.n
    return st


def run(st):
    h = st.ctx.handle
    if st.kind == "grad":
        k = st.k.detach().requires_grad_()
        d, n, e = st.sign(k, st.mu)
        (e + 0.1 * n + (st.gd * d).sum()).backward()
        return dict(d=d.detach(), n=n.detach(), e=e.detach(), dk=k.grad)
    if st.kind == "mu":
        smx.smx_update_values(h, st.k)
        smx.smx_set_mu(h, st.mu)
        mu, steps, _ = smx.smx_find_mu_eig(h, st.n_target)
        smx.smx_get_d(h, st.d)
        return dict(d=st.d, n=smx.smx_trace(h), e=smx.smx_energy(h), mu=mu, steps=steps)
    if st.kind == "split":
        smx.smx_update_values(h, st.k_split)
        smx.smx_evaluate(h)
        smx.smx_wait(h)
        smx.smx_get_d_expanded(h, st.src, len(st.k), st.d)
        return dict(d=st.d, n=smx.smx_trace(h), e=smx.smx_energy(h))
    smx.smx_update_values(h, st.k)
    r = st.ctx.evaluate(out=st.d)
    return dict(d=r.d_values, n=r.n_elec, e=r.energy)


# ---- work a pass cannot do without --------------------------------------------

def _group_rows(s):
    """Block rows of every group's submatrix (the union of its columns' stored rows)."""
    out = []
    for g in range(s.ngroups):
        cols = s.grp_blocks[s.grp_ptr[g]:s.grp_ptr[g + 1]]
        out.append(np.unique(np.concatenate([s.row_idx[s.col_ptr[j]:s.col_ptr[j + 1]] for j in cols])))
    return out


def work(case):
    s = _system(case)
    if case["kind"] == "split":
        part = smx.split_columns(s, case["eps"])
        first = part.grp_blocks[part.grp_ptr[:-1]]
        n = np.diff(part.col_ptr)[first].astype(np.float64)
    else:
        n = np.array([s.blk_size[r].sum() for r in _group_rows(s)], dtype=np.float64)
    n3 = float((n ** 3).sum())
    bytes_ = 16.0 * len(s.values)                    # K in, D out
    if case["kind"] == "grad":
        # symmetric products of n^3 flops: two a step forwards; backwards a square and the
        # combine, and two general products of 2 n^3
        return dict(bytes=bytes_ + 16.0 * len(s.values), flops=(2 + 6) * STEPS * n3)
    if case["kind"] in ("fermi", "mu"):
        return dict(bytes=bytes_, flops=4.0 / 3.0 * n3)       # the reduction to tridiagonal form
    return dict(bytes=bytes_, flops=2 * STEPS * n3)           # two symmetric products a step


# ---- the same in plain 64-bit torch ---------------------------------------------

def _sign(a, da=None):
    """sign(A) by Newton-Schulz in float64, and its Frechet derivative in direction da."""
    s = a.abs().sum(1).max()
    x, dx = a / s, None if da is None else da / s
    eye = torch.eye(len(a), dtype=a.dtype, device=a.device)
    more = 2
    for _ in range(200):
        x2 = x @ x
        if float((x2 - eye).abs().max()) < 1e-11:
            more -= 1
        if dx is not None:
            dx = 1.5 * dx - 0.5 * (dx @ x2 + x @ (dx @ x) + x2 @ dx)
        x = 1.5 * x - 0.5 * (x @ x2)
        x = 0.5 * (x + x.T)
        if more == 0:
            break
    return x, dx


def exact(case, seed):
    s = _system(case)
    eig = case["kind"] in ("fermi", "mu")
    blocks = _group_rows(s)
    if eig and sum(float(s.blk_size[r].sum()) ** 3 for r in blocks) > 1e10:
        return None                                  # minutes of plain eigendecompositions
    k = _values(s, seed)
    row, col, mirror = _positions(s, "cuda")
    kd = torch.zeros(s.n, s.n, dtype=torch.float64, device="cuda")
    kd[row, col] = k
    stored = torch.zeros(s.n, s.n, dtype=torch.bool, device="cuda")
    stored[row, col] = True
    boff = np.concatenate([[0], np.cumsum(s.blk_size)])

    def functions(b):
        return torch.as_tensor(np.concatenate([np.arange(boff[i], boff[i + 1]) for i in b]), device="cuda")

    if case["kind"] == "split":
        # one submatrix per column: its rows are the elements kept by the cutoff
        part = smx.split_columns(s, case["eps"])
        jobs = []
        for g in range(len(part.grp_ptr) - 1):
            own = part.grp_blocks[part.grp_ptr[g]:part.grp_ptr[g + 1]]
            rows = part.row_idx[part.col_ptr[own[0]]:part.col_ptr[own[0] + 1]]
            jobs.append((torch.as_tensor(rows.astype(np.int64), device="cuda"),
                         torch.as_tensor(own.astype(np.int64), device="cuda")))
        kept = torch.zeros_like(stored)
        at = torch.as_tensor(part.src, device="cuda")
        kept[row[at], col[at]] = True
        stored = kept
        kd = torch.where(kept, kd, torch.zeros_like(kd))
    else:
        jobs = [(functions(blocks[g]), functions(s.grp_blocks[s.grp_ptr[g]:s.grp_ptr[g + 1]]))
                for g in range(s.ngroups)]

    dd = torch.zeros_like(kd)
    grad = torch.zeros_like(kd) if case["kind"] == "grad" else None
    if grad is not None:
        gd = torch.zeros_like(kd)
        gd[row, col] = _weights(s, seed)
        seed_d = torch.where(stored, kd + gd + 0.1 * torch.eye(s.n, dtype=kd.dtype, device="cuda"),
                             torch.zeros_like(kd))  # dL/dD of L = E + 0.1 N + <G, D>
    if eig:
        pairs = []
        for r, own in jobs:
            lam, q = torch.linalg.eigh(kd[r][:, r].cpu())
            pairs.append((lam, q, q[torch.searchsorted(r, own).cpu()]))

        def fermi(lam, mu):
            return 0.5 * (1.0 - torch.tanh((lam - mu) / (2.0 * case["kT"])))

        mu = s.mu
        if case["kind"] == "mu":
            lo, hi = -50.0, 50.0
            for _ in range(100):
                mu = 0.5 * (lo + hi)
                n = sum(float((qo.square().sum(0) * fermi(lam, mu)).sum()) for lam, _, qo in pairs)
                lo, hi = (mu, hi) if n < 0.5 * s.n else (lo, mu)
        for (r, own), (lam, q, qo) in zip(jobs, pairs):
            dd[r[:, None], own[None, :]] = ((q * fermi(lam, mu)) @ qo.T).cuda()
    else:
        for r, own in jobs:
            a = kd[r][:, r]
            a.diagonal().sub_(s.mu)
            at = torch.searchsorted(r, own)
            ds = None
            if grad is not None:
                ds = torch.zeros_like(a)
                ds[:, at] = -0.5 * seed_d[r][:, own]
                ds = 0.5 * (ds + ds.T)
            sgn, da = _sign(a, ds)
            d = -0.5 * sgn[:, at]
            d[at, torch.arange(len(at), device="cuda")] += 0.5
            dd[r[:, None], own[None, :]] = d
            if da is not None:
                grad[r[:, None], r[None, :]] += da
    dd = torch.where(stored, dd, torch.zeros_like(dd))
    out = dict(d=dd[row, col], n=float(dd.diagonal().sum()), e=float((dd * kd).sum()))
    if case["kind"] == "mu":
        out.update(mu=None, steps=None)
    if grad is not None:
        out["dk"] = (grad + dd)[row, col]
        out["n"], out["e"] = (torch.tensor(out[q], dtype=torch.float64) for q in ("n", "e"))
    return out
