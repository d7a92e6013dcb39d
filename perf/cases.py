"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values.  ``listed()`` gives the standing ones,
``draw(rng)`` one more of the same ranges; ``prepare(case, seed)`` makes what a
user's program has in hand before the call, ``run(state)`` is one pass through
the public entry points, ``work(case)`` the bytes and operations the pass cannot
do without, and ``exact(case, seed)`` the outputs in plain FP64 tensor algebra.

Kinds of case (``kind``):

* ``product``: y = H_eff x, ny = N_eff x at one site (``SPMPS.heff_apply``), the
  call a Davidson (or any other) local solver makes over and over.
* ``step``: what surrounds the products of a site step, in both directions:
  the left environment of a bond, diagonals and product at the site right of
  it, then the right environment of the same bond, diagonals and product at
  the site left of it.
* ``sweep``: a new guess into an existing handle (site tensors, right
  environments) and one sweep with few Davidson iterations per site, as the
  first sweeps of a run are done; ``batch``: the same for several guesses
  together.  Broken-symmetry (Neel) guesses, as such runs start from.
* ``expect``: <O P>/<P> of a spin-free operator in the current state, the call
  that density matrices, correlations and energy components consist of.
* ``mlp``: one training step of the learned preconditioner and the corrections
  of the updated model.

The block tables, integrals and guesses are the seeded recipes of the
workloads; MPOs are inputs of the calls and come from the MPO builders.
"""
import math

import numpy as np
import torch

import paper_1703_04789_amd as sp
import workloads as W

SIGMA = ((0, 0), (1, -1), (1, 1), (2, 0))  # (N, 2M) of a site's four states


def _hubbard(kind, L, D, G, U, N=None, twoS=0, twoM=0, **more):
    return dict(kind=kind, model="hubbard", L=L, N=L if N is None else N, twoM=twoM, twoS=twoS, D=D, G=G, U=U, **more)


def _abinitio(kind, K, D, G, N=None, twoS=0, twoM=0, **more):
    return dict(kind=kind, model="abinitio", L=K, N=K if N is None else N, twoM=twoM, twoS=twoS, D=D, G=G, **more)


def listed():
    return [
        # the smallest call: the 8-site chain whose sweeps are compared with
        # the oracle; launches and latency are all there is
        dict(_hubbard("product", 8, 16, 5, 4.0, site=4, precision="fp64"), name="product_hubbard_L8_D16"),
        # the ordinary one: the centre site of the benchmark's chain
        dict(_hubbard("product", 32, 256, 9, 8.0, site=16, precision="fp64"), name="product_hubbard_L32_D256"),
        # the longest Hubbard chain in use, high spin
        dict(_hubbard("product", 48, 512, 9, 6.0, twoS=4, site=24, precision="fp64"), name="product_hubbard_L48_D512"),
        # the FP32 mode at the widest batch guess
        dict(_hubbard("product", 32, 512, 9, 8.0, site=16, precision="fp32"), name="product_fp32_L32_D512"),
        # a wide MPO (dense two-electron integrals), the benchmark's 12 orbitals
        dict(_abinitio("product", 12, 128, 11, site=6, precision="fp64"), name="product_abinitio_K12_D128"),
        # the split-BF16 mode on wider particle-number blocks, off the centre,
        # an odd bond dimension
        dict(_abinitio("product", 14, 181, 11, site=6, precision="bf16x3"), name="product_bf16x3_K14_D181"),
        # what surrounds the products of a site step
        dict(_hubbard("step", 32, 256, 9, 8.0, site=16, precision="fp64"), name="step_hubbard_L32_D256"),
        dict(_abinitio("step", 12, 128, 11, site=6, precision="fp64"), name="step_abinitio_K12_D128"),
        # whole calls: first sweeps of the benchmark's chain, and of several
        # guesses together (the batch recipe's sizes)
        dict(_hubbard("sweep", 32, 256, 9, 8.0, iters=8, sub=6), name="sweep_hubbard_L32_D256"),
        dict(_hubbard("batch", 16, 96, 9, 4.0, iters=8, sub=6, states=6), name="batch_hubbard_6_states"),
        # one entry of a one-body density matrix
        dict(_hubbard("expect", 32, 128, 9, 8.0, op="epq"), name="expect_epq_L32_D128"),
        # one optimiser step of the learned preconditioner and its corrections
        dict(kind="mlp", hidden=256, rows=60001, name="mlp_step_60001_rows"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product"] * 5 + ["step"] * 3 + ["sweep", "batch", "expect", "mlp"])
    if kind == "mlp":
        return dict(kind="mlp", hidden=rng.choice([16, 64, 200, 256]), rows=_log(rng, 100, 60000))
    if kind in ("sweep", "batch"):
        L = 2 * rng.randint(4, 16 if kind == "sweep" else 8)
        c = _hubbard(kind, L, _log(rng, 16, 250 if kind == "sweep" else 96), rng.randint(5, 9), rng.choice([4.0, 8.0]),
                     iters=rng.randint(3, 8), sub=rng.choice([5, 6, 32]))
        if kind == "batch":
            c["states"] = rng.randint(2, 6)
        return c
    spin = lambda N: (N % 2, N % 2 + 2 * rng.randint(0, 2))  # noqa: E731
    if kind == "expect":
        L = rng.randint(6, 32)
        N = L + rng.randint(-2, 2)
        m, s = spin(N)
        return _hubbard(kind, L, _log(rng, 8, 128), rng.randint(3, 9), 4.0, N=N, twoM=m, twoS=s,
                        op=rng.choice(["epq", "spin", "hubbard"]))
    wide = rng.random() < 0.4
    prec = rng.choice(["fp64", "fp64", "fp32", "bf16x3"]) if kind == "product" else "fp64"
    if wide:
        K = rng.randint(6, 12)
        N = K + rng.randint(-1, 1)
        m, s = spin(N)
        c = _abinitio(kind, K, _log(rng, 12, 128), rng.randint(3, 11), N=N, twoM=m, twoS=s, precision=prec)
    else:
        L = rng.randint(6, 40)
        N = L + rng.randint(-2, 2)
        m, s = spin(N)
        c = _hubbard(kind, L, _log(rng, 8, 480 if kind == "product" else 256), rng.randint(3, 9), rng.choice([4.0, 6.0, 8.0]),
                     N=N, twoM=m, twoS=s, precision=prec)
    c["site"] = rng.randint(1, c["L"] - 1) if rng.random() < 0.4 else max(1, c["L"] // 2 + rng.randint(-2, 1))
    return c


# ---- inputs ----------------------------------------------------------------

_INTEGRALS = {}


def _mpo(case):
    if case["model"] == "hubbard":
        return sp.mpo_hubbard(case["L"], 1.0, case["U"])
    K = case["L"]
    if K not in _INTEGRALS:  # one molecule: the states of all seeds share its MPO
        _INTEGRALS[K] = sp.mpo_abinitio(*W.abinitio_integrals(K, 4))
    return _INTEGRALS[K]


def _operator(case):
    L = case["L"]
    if case["op"] == "epq":
        return sp.mpo_epq(L, 2, L // 2)
    if case["op"] == "spin":
        return sp.mpo_spin_corr(L, 2, L // 2)
    return sp.mpo_hubbard(L, 1.0, case["U"])


def _table(case):
    return W.make_block_table(case["L"], case["N"], case["twoM"], case["D"])


def _blocks(case, table, seed):
    return W.neel_blocks(table, seed) if case["kind"] in ("sweep", "batch") else W.random_blocks(table, seed)


def _left_sites(case, table, seed):
    """Left-orthonormal tensors (per right sector) of the sites left of the
    centre, as a sweep leaves them; a step case moves the centre past its site."""
    flat, off, out = _blocks(case, table, seed + 1), 0, []
    for k in range(1, case["site"] + (case["kind"] == "step")):
        A = flat[off:off + table.site_size(k)].copy()
        off += A.size
        of, at = {}, 0
        for _, _, ib, r, c in table.site_blocks(k):
            of.setdefault(ib, []).append((at, r, c))
            at += r * c
        for parts in of.values():
            Q, R = np.linalg.qr(np.concatenate([A[o:o + r * c].reshape(r, c) for o, r, c in parts]))
            Q, row = Q * np.where(np.diag(R) < 0, -1.0, 1.0), 0
            for o, r, c in parts:
                A[o:o + r * c] = Q[row:row + r].ravel()
                row += r
        out.append(A)
    return out


def _vector(table, site, seed):
    x = np.random.default_rng(seed + 7).standard_normal(table.site_size(site))
    return x / np.linalg.norm(x)


def _mlp_data(case, seed):
    p = W.mlp_init(case["hidden"], seed)
    rng = np.random.default_rng(seed)
    n = case["rows"]
    F = np.empty((n, 5), np.float32)  # the features' own ranges: |r|/rms, three asinh, the diagonal correction
    F[:, 0] = np.abs(rng.standard_normal(n))
    F[:, 1] = np.arcsinh(-8.0 * rng.random(n))
    F[:, 2] = np.arcsinh(rng.random(n))
    F[:, 3] = np.arcsinh(F[:, 0] / 8.0)
    F[:, 4] = rng.standard_normal(n)
    return p, F, rng.standard_normal(n).astype(np.float32)


def _dev(a):
    return torch.tensor(a, device="cuda")


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "mlp":
        p, F, Y = _mlp_data(case, seed)
        s.update(model=sp.MLP(p), F=_dev(F), Y=_dev(Y))
        return s
    table, mpo = _table(case), _mpo(case)

    def handle(seed):
        return sp.SPMPS(table, _blocks(case, table, seed), mpo, case["twoS"], case["G"],
                        precision=case.get("precision", "fp64"))

    kind, L = case["kind"], case["L"]
    s["states"] = [handle(seed + 1000 * i) for i in range(case.get("states", 1))]
    st = s["states"][0]
    if kind in ("sweep", "batch"):
        s["guess"] = [[st.get_site(k) for k in range(1, L + 1)] for st in s["states"]]
    elif kind == "expect":
        s["op"] = _operator(case)
    else:
        k = case["site"]
        for j, A in enumerate(_left_sites(case, table, seed), 1):
            st.set_site(j, A)
            if j < k:
                st.env_update(j, +1)
        for name, site in (("a", k),) if kind == "product" else (("b", k + 1), ("a", k)):
            x = _dev(_vector(table, site, seed))
            out = torch.empty((2 if kind == "product" else 4, x.numel()), dtype=torch.float64, device="cuda")
            s[name] = (site, x, out)
        if case["precision"] != "fp64":  # the products carry FP32 accuracy at most and are kept as that
            s["kept"] = torch.empty(s["a"][2].shape, dtype=torch.float32, device="cuda")
    return s


# ---- one pass ----------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mlp":
        loss = s["model"].train_step(s["F"], s["Y"], 1e-3)
        p = s["model"].params()
        return loss, p["W1"], p["b1"], p["w2"], p["b2"], s["model"].forward(s["F"])
    st = s["states"][0]
    if kind == "product":
        k, x, out = s["a"]
        st.heff_apply(k, x, out[0], out[1])
        if "kept" in s:
            return s["kept"].copy_(out)
        return out[0], out[1]
    if kind == "step":
        got = []
        for name, site, way in (("b", case["site"], +1), ("a", case["site"] + 1, -1)):
            k, x, out = s[name]
            st.env_update(site, way)
            st.heff_diag(k, out[2], out[3])
            st.heff_apply(k, x, out[0], out[1])
            got += [out[0], out[1], out[2], out[3]]
        return got
    if kind == "expect":
        return st.expect(s["op"])
    for st, sites in zip(s["states"], s["guess"]):  # a new guess: tensors, then R of every bond
        for k, A in enumerate(sites):
            st.set_site(k + 1, A)
        for k in range(case["L"], 1, -1):
            st.env_update(k, -1)
    opts = dict(tol=1e-9, max_iter=case["iters"], max_sub=case["sub"], keep=3)
    if kind == "sweep":
        reports = [st.sweep(1, **opts)[1]]
    else:
        reports = sp.sweep_batch(s["states"], 1, **opts)[1]
    return [dict(energy=np.array([r["theta"] for r in rep]), norm=np.array([r["pnorm"] for r in rep]),
                 tensors=np.concatenate([st.get_site(k) for k in range(1, case["L"] + 1)]))
            for st, rep in zip(s["states"], reports)]


# ---- bytes and operations ------------------------------------------------------

def _channel_dn(mpo, L):
    """Particle change of every channel of every bond (0..L), from the MPO."""
    w, data = mpo
    n_of = np.array([0, 1, 1, 2])
    dn, nnz, off = [np.zeros(1, int)], [], 0
    for k in range(L):
        a, b = int(w[k]), int(w[k + 1])
        O = data[off:off + a * b * 16].reshape(a, b, 4, 4)
        off += a * b * 16
        ia, ib, si, ti = np.nonzero(O)
        d = np.zeros(b, int)
        d[ib] = dn[k][ia] + n_of[si] - n_of[ti]
        dn.append(d)
        nnz.append((len(ia), len(set(zip(ib.tolist(), si.tolist())))))
    return dn, nnz


def _nblocks(bond):
    out = {}
    for n, _, d in bond:
        out[n] = out.get(n, 0) + d
    return out


def _env_values(bond, dn):
    """Values of one environment of one quadrature point: a dense block per
    channel and bra particle number."""
    nb = _nblocks(bond)
    return sum(d * nb.get(n - c, 0) for c in dn.tolist() for n, d in nb.items())


def _counts(case, table, mpo, k):
    """(environment values left, right; operations of L x, of V R, of N_eff) at
    site k and one quadrature point, non-zero blocks only."""
    dn, nnz = _channel_dn(mpo, case["L"])
    bl, br = table.bonds[k - 1], table.bonds[k]
    nl, nr = _nblocks(bl), _nblocks(br)
    left = right = metric = 0.0
    for ia, sg, ib, rows, cols in table.site_blocks(k):
        n_in, n_out = bl[ia][0], br[ib][0]
        for c in dn[k - 1].tolist():  # L(c, i) of every bra number i on this block of x
            left += 2.0 * nl.get(n_in + c, 0) * rows * cols
        for c in dn[k].tolist():  # this output block from V(c', ket number) and R(c')
            right += 2.0 * rows * nr.get(n_out - c, 0) * cols
        metric += 2.0 * rows * nr[n_out] * cols
    return _env_values(bl, dn[k - 1]), _env_values(br, dn[k]), left, right, metric


def work(case):
    if case["kind"] == "mlp":
        n, H = case["rows"], case["hidden"]
        return dict(bytes=4.0 * n * 13 + 12.0 * (7 * H + 1), flops=float(n) * H * (12 + 16 + 12))
    table, L, G = _table(case), case["L"], case["G"]
    mpo = _operator(case) if case["kind"] == "expect" else _mpo(case)
    size = [table.site_size(k) for k in range(1, L + 1)]
    env = 4.0 if case.get("precision") == "fp32" else 8.0

    def product(k):
        l, r, a, b, c = _counts(case, table, mpo, k)
        return G * env * (l + r) + 24.0 * size[k - 1], G * (a + b + c)

    def update(k, sides):
        l, r, a, b, _ = _counts(case, table, mpo, k)
        return G * 8.0 * (l + r) * sides + 8.0 * size[k - 1], G * (a + b)

    by = fl = 0.0
    if case["kind"] == "product":
        by, fl = product(case["site"])
    elif case["kind"] == "step":
        k = case["site"]
        for got in (update(k, 1.0), product(k + 1), update(k + 1, 1.0), product(k)):
            by, fl = by + got[0], fl + got[1]
        by += 16.0 * (size[k - 1] + size[k])
    elif case["kind"] == "expect":
        by = 8.0 * sum(size)
        fl = sum(update(k, 0.0)[1] for k in range(1, L + 1))
    else:
        for k in range(1, L + 1):
            (ub, uf), (pb, pf) = update(k, 1.0), product(k)
            visits = 1.0 if k in (1, L) else 2.0
            by += ub * (1.0 + visits) + pb * visits * (case["iters"])
            fl += uf * (1.0 + visits) + pf * visits * (case["iters"])
        by, fl = by * case.get("states", 1), fl * case.get("states", 1)
    return dict(bytes=by, flops=fl)


# ---- the outputs in plain FP64 -------------------------------------------------

class _Dense:
    """The state of a case in dense FP64 tensors: site tensors (4, D, D') with
    zeros outside the blocks, environments (D, w, D) per quadrature point."""

    def __init__(self, case, seed, mpo):
        self.case, self.table, self.L = case, _table(case), case["L"]
        t = self.table
        self.start = [np.concatenate([[0], np.cumsum([d for _, _, d in b])]) for b in t.bonds]
        w, data = mpo
        self.W, off = [], 0
        for k in range(self.L):
            n = int(w[k]) * int(w[k + 1]) * 16
            self.W.append(_dev(data[off:off + n].reshape(int(w[k]), int(w[k + 1]), 4, 4).copy()))
            off += n
        flat, self.A, off = _blocks(case, t, seed), [], 0
        for k in range(1, self.L + 1):
            self.A.append(self.dense(k, flat[off:off + t.site_size(k)]))
            off += t.site_size(k)
        x, wt = np.polynomial.legendre.leggauss(case["G"])
        c, s = np.sqrt((1.0 + x) / 2.0), np.sqrt((1.0 - x) / 2.0)
        S, M = case["twoS"], case["twoM"]
        p, q = (S + M) // 2, (S - M) // 2
        f = math.factorial
        d = sum((-1) ** k * f(p) * f(q) / (f(p - k) * f(k) * f(k) * f(q - k)) * c ** (S - 2 * k) * s ** (2 * k)
                for k in range(min(p, q) + 1))
        self.coef = (S + 1) / 2.0 * wt * d
        self.rot = []
        for g in range(case["G"]):
            r = np.eye(4)
            r[1, 1] = r[2, 2] = c[g]
            r[1, 2], r[2, 1] = s[g], -s[g]
            self.rot.append(_dev(r))
        for k in range(self.L, 1, -1):
            self.right_orthonormal(k)

    def blocks(self, k):
        off = 0
        for ia, sg, ib, r, c in self.table.site_blocks(k):
            yield sg, slice(self.start[k - 1][ia], self.start[k - 1][ia] + r), slice(self.start[k][ib], self.start[k][ib] + c), off, r, c
            off += r * c

    def dense(self, k, packed):
        A = np.zeros((4, self.start[k - 1][-1], self.start[k][-1]))
        for sg, a, b, off, r, c in self.blocks(k):
            A[sg, a, b] = packed[off:off + r * c].reshape(r, c)
        return A

    def packed(self, k, A):
        A = A.cpu().numpy()
        return np.concatenate([A[sg, a, b].ravel() for sg, a, b, _, _, _ in self.blocks(k)])

    def right_orthonormal(self, k):
        """Positive-diagonal LQ per left sector, L into site k - 1."""
        A, D = self.A[k - 1], self.start[k - 1][-1]
        L = np.zeros((D, D))
        of = {}
        for sg, a, b, _, _, _ in self.blocks(k):
            of.setdefault((a.start, a.stop), []).append((sg, b))
        for (a0, a1), parts in of.items():
            Q, R = np.linalg.qr(np.concatenate([A[sg, a0:a1, b] for sg, b in parts], axis=1).T)
            sign = np.where(np.diag(R) < 0, -1.0, 1.0)
            Q, R, at = Q * sign, R * sign[:, None], 0
            for sg, b in parts:
                A[sg, a0:a1, b] = Q[at:at + b.stop - b.start].T
                at += b.stop - b.start
            L[a0:a1, a0:a1] = R.T
        self.A[k - 2] = self.A[k - 2] @ L

    def left_product(self, env, k, g, x, W):
        """V[v, s, a, d] = sum env[a, w, c] x[t', c, d] r[t, t'] W[w, v, s, t]."""
        x = torch.einsum("tu,ucd->tcd", self.rot[g], x)
        a, w, c = env.shape
        T = torch.stack([(env.reshape(a * w, c) @ x[t]).reshape(a, w, -1) for t in range(4)], 2)  # a w t d
        d = T.shape[-1]
        v = W.shape[1]
        V = W.permute(1, 2, 0, 3).reshape(v * 4, w * 4) @ T.reshape(a, w * 4, d).permute(1, 0, 2).reshape(w * 4, a * d)
        return V.reshape(v, 4, a, d)

    def env_left(self, env, k, g, W, A):
        V = self.left_product(env, k, g, A, W)
        v, _, a, d = V.shape
        out = sum(A[s].T @ V[:, s].permute(1, 0, 2).reshape(a, v * d) for s in range(4))
        return out.reshape(-1, v, d)

    def env_right(self, env, k, g, W, A):
        """The mirror image: R[a, w, c] from R[b, v, d]."""
        return self.env_left(env, k, g, W.permute(1, 0, 2, 3), A.permute(0, 2, 1).contiguous())

    def local(self, left, right, k, g, x, W):
        V = self.left_product(left, k, g, x, W)
        v, _, a, d = V.shape
        R = right.permute(1, 2, 0).reshape(v * d, -1)
        return torch.stack([V[:, s].permute(1, 0, 2).reshape(a, v * d) @ R for s in range(4)])

    def diagonal(self, left, right, k, g, W):
        Wd = torch.einsum("wvst,ts->wvs", W, self.rot[g])
        l, r = torch.einsum("awa->aw", left), torch.einsum("bvb->bv", right)
        return torch.stack([l @ Wd[:, :, s] @ r.T for s in range(4)])


def exact(case, seed):
    if case["kind"] in ("sweep", "batch"):  # no closed form: each site's solve stops at an iteration count
        return None
    if case["kind"] == "mlp":
        return _exact_mlp(case, seed)
    L, G = case["L"], case["G"]
    S = _Dense(case, seed, _operator(case) if case["kind"] == "expect" else _mpo(case))
    if case["kind"] != "expect":
        for j, v in enumerate(_left_sites(case, S.table, seed), 1):
            S.A[j - 1] = S.dense(j, v)
    A = [_dev(a) for a in S.A]
    one = torch.ones((1, 1, 1), dtype=torch.float64, device="cuda")
    unit = torch.eye(4, dtype=torch.float64, device="cuda").reshape(1, 1, 4, 4)
    k = case.get("site", 1)
    got = {}

    def add(name, v):
        got[name] = got[name] + v if name in got else v

    def at(name, site, g, lh, rh, li, ri, x):
        c = S.coef[g]
        add(name + "y", c * S.local(lh, rh, site, g, x, S.W[site - 1]))
        add(name + "n", c * S.local(li, ri, site, g, x, unit))
        if case["kind"] == "step":
            add(name + "dy", c * S.diagonal(lh, rh, site, g, S.W[site - 1]))
            add(name + "dn", c * S.diagonal(li, ri, site, g, unit))

    last = 1 if case["kind"] == "expect" else k
    x = {j: A[0] if case["kind"] == "expect" else _dev(S.dense(j, _vector(S.table, j, seed)))
         for j in ((k, k + 1) if case["kind"] == "step" else (k,))}
    for g in range(G):
        lh, li, rh, ri = one, one, one, one
        for j in range(1, last):
            lh, li = S.env_left(lh, j, g, S.W[j - 1], A[j - 1]), S.env_left(li, j, g, unit, A[j - 1])
        for j in range(L, last + 1, -1):
            rh, ri = S.env_right(rh, j, g, S.W[j - 1], A[j - 1]), S.env_right(ri, j, g, unit, A[j - 1])
        if case["kind"] == "step":
            at("b", k + 1, g, S.env_left(lh, k, g, S.W[k - 1], A[k - 1]), rh, S.env_left(li, k, g, unit, A[k - 1]), ri, x[k + 1])
        if last < L:
            rh, ri = S.env_right(rh, last + 1, g, S.W[last], A[last]), S.env_right(ri, last + 1, g, unit, A[last])
        at("a", last, g, lh, rh, li, ri, x[k])
    if case["kind"] == "expect":
        num, den = float((A[0] * got["ay"]).sum()), float((A[0] * got["an"]).sum())
        return num / den, den / float((A[0] * A[0]).sum())
    out = {n: S.packed(k + 1 if n[0] == "b" else k, v) for n, v in got.items()}
    if case["kind"] == "step":
        return [out[n + q] for n in "ba" for q in ("y", "n", "dy", "dn")]
    if case["precision"] != "fp64":
        return np.stack([out["ay"], out["an"]])
    return out["ay"], out["an"]


def _exact_mlp(case, seed):
    p, F, Y = _mlp_data(case, seed)
    H, n = case["hidden"], case["rows"]
    F, Y = _dev(F).double(), _dev(Y).double()
    w = {q: _dev(np.asarray(p[q], np.float64)) for q in ("W1", "b1", "w2", "b2")}
    z = F @ w["W1"].T + w["b1"]
    h = z.clamp_min(0.0)
    e = h @ w["w2"] + w["b2"] - Y
    dz = (e / n)[:, None] * w["w2"] * (z > 0)
    grad = dict(W1=dz.T @ F, b1=dz.sum(0), w2=h.T @ (e / n), b2=e.sum() / n)
    for q, v in grad.items():  # Adam's first step: m / (1 - 0.9) and v / (1 - 0.999) are g and g^2
        w[q] = (w[q] - 1e-3 * v / (v.abs() + 1e-8)).float().double()
    y = (F @ w["W1"].T + w["b1"]).clamp_min(0.0) @ w["w2"] + w["b2"]
    loss = 0.5 * float((e * e).mean())
    return (loss, *(w[q].cpu().numpy() for q in ("W1", "b1", "w2")), float(w["b2"]), y.cpu().numpy())
