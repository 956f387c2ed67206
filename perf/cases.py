"""Performance cases of the QAOA library: what a user's program calls, over the
sizes it calls it with.

A case names one public entry point and its sizes:

* ``gradient``    one E + adjoint gradient (``QaoaHandle.gradient``), the call an
                  optimiser repeats;
* ``autograd``    one forward and backward of ``QaoaExpectationModule``;
* ``statevector`` the state copied into the caller's device tensor;
* ``sample``      shots from the current state, with their objective values;
* ``instance``    a new problem: handle, one expectation, a few samples, close;
* ``batch``       one run of the batched engine (Adam on many small graphs);
* ``network``     loss and parameter gradient of the warm-start network.

Depths, families, weights and angles are those of ``qaoa_inputs``; complex64
handles hand their results on in float32, the precision that they have.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import qaoa_inputs as qi
from paper_2407_13012_amd import QaoaBatch, QaoaHandle, QaoaMpnn
from paper_2407_13012_amd.autograd import QaoaExpectationModule

_DEV = "cuda" if torch.cuda.is_available() else "cpu"
# registers and LDS of the card: vectors that fit there need not pass through memory
_ON_CHIP = 256 * (512 + 160) * 1024


def listed():
    return [
        # The smallest call: the unweighted 12-vertex graph at p = 2, where launches and
        # the wait for the result are the whole time.
        dict(name="maxcut12_grad", kind="gradient", family="er", n=12, p=2, precision="c128"),
        # The middle of the evaluated graphs (6 to 29 vertices, depth 6): an odd size, complete
        # graph, a few sweeps of a state that stays in the caches.
        dict(name="complete17_grad", kind="gradient", family="complete", n=17, p=6, precision="c128"),
        # A torch training loop in single precision: forward and backward as two calls.
        dict(name="autograd21_c64", kind="autograd", family="er_weighted", n=21, p=4, precision="c64"),
        # One L-BFGS evaluation of the warm-start evaluation's graphs, ER(24, 0.5), p = 8.
        dict(name="er24_grad", kind="gradient", family="er_weighted", n=24, p=8, precision="c128"),
        # The weighted 3-regular graph on 26 vertices at p = 6.
        dict(name="regular26_grad", kind="gradient", family="regular3", n=26, p=6, precision="c128"),
        # The large QUBO at a size that leaves room on the card: HBM-bound sweeps.
        dict(name="qubo30_grad", kind="gradient", family="qubo", n=30, p=3, precision="c128"),
        # The state of a 25-variable polynomial cost exported to a device tensor.
        dict(name="state25_c64", kind="statevector", family="poly", n=25, p=3, precision="c64"),
        # 10^6 shots kept on the device, after an optimisation has left its state.
        dict(name="sample26", kind="sample", family="qubo", n=26, p=3, shots=1_000_000, precision="c128"),
        # A new graph from edges to its expectation and 1024 samples on the host.
        dict(name="instance22", kind="instance", family="er", n=22, p=6, shots=1024, precision="c128"),
        # A few dozen graphs optimised together with the engine's default options.
        dict(name="batch48", kind="batch", count=48, nmin=10, nmax=20, p=4, steps=8, workgroups=0,
             waves_per_simd=1),
        # A training set's worth of graphs with the tuned options: every workgroup has a queue.
        dict(name="batch1024", kind="batch", count=1024, nmin=10, nmax=20, p=4, steps=3, workgroups=512,
             waves_per_simd=2),
        # One minibatch of the warm-start network's training: 256 graphs, p = 8.
        dict(name="network256", kind="network", count=256, nmin=10, nmax=20, p=8),
    ]


_FAMILIES = ("er", "er_weighted", "complete", "regular3", "qubo", "poly")


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gradient", "gradient", "gradient", "autograd", "statevector", "sample", "instance",
                       "batch", "batch", "network"])
    prec = rng.choice(["c128", "c64"])
    fam = rng.choice(_FAMILIES)
    if kind == "batch":
        nmax = rng.randint(11, 20)
        count = _logint(rng, 4, 1024 if nmax < 19 else 512)
        return dict(kind=kind, count=count, nmin=max(4, nmax - rng.randint(0, 10)), nmax=nmax, p=rng.randint(1, 6),
                    steps=rng.randint(1, 6), workgroups=rng.choice([0, 512]), waves_per_simd=rng.choice([1, 2]))
    if kind == "network":
        nmax = rng.randint(10, 32)
        return dict(kind=kind, count=_logint(rng, 8, 512), nmin=max(2, nmax - rng.randint(0, 12)), nmax=nmax,
                    p=rng.randint(1, 8))
    if kind == "gradient":
        # complex64 gradients are drawn through autograd, which hands them on in float32
        n, prec = rng.randint(6, 29), "c128"
        p = rng.randint(1, 5 if n == 29 else 8)
        return dict(kind=kind, family=_fit(fam, n), n=n, p=p, precision=prec)
    if kind == "autograd":
        n = rng.randint(8, 26)
        return dict(kind=kind, family=_fit(fam, n), n=n, p=rng.randint(1, 8), precision=prec)
    if kind == "statevector":
        n = rng.randint(10, 27)
        return dict(kind=kind, family=_fit(fam, n), n=n, p=rng.randint(1, 8), precision=prec)
    if kind == "sample":
        n = rng.randint(12, 27)
        return dict(kind=kind, family=_fit(fam, n), n=n, p=rng.randint(1, 4), shots=_logint(rng, 1000, 1_000_000),
                    precision="c128")
    n = rng.randint(8, 25)
    return dict(kind=kind, family=_fit(fam, n), n=n, p=rng.randint(1, 8), shots=_logint(rng, 100, 10_000),
                precision="c128")


def _fit(fam, n):
    return "er_weighted" if fam == "regular3" and n % 2 else fam


# ---------------------------------------------------------------- inputs

def _instance(case, seed):
    n, fam = case["n"], case["family"]
    s = [int(seed), n, 1]
    if fam == "er":
        return qi.erdos_renyi(n, 0.5, seed=s)
    if fam == "er_weighted":
        return qi.erdos_renyi(n, 0.5, seed=s, weights="uniform", wlow=-1.0, whigh=1.0)
    if fam == "complete":
        return qi.complete_graph(n, seed=s, weights="uniform", wlow=0.0, whigh=1.0)
    if fam == "regular3":
        return qi.random_regular(n, 3, seed=s, weights="uniform", wlow=0.0, whigh=1.0)
    if fam == "qubo":
        return qi.qubo_erdos_renyi(n, 0.1, seed=s)
    return qi.poly_random(n, 3 * n, 4, seed=s)


def _angles(case, seed):
    return qi.ramp_with_noise(case["p"], seed=[int(seed), case["p"], 2])


def _graphs(case, seed):
    """`count` graphs with n uniform in nmin..nmax, edge probability U[0.2, 0.8], weights U[-1, 1]."""
    rng = np.random.default_rng([int(seed), case["count"], 3])
    out = []
    for _ in range(case["count"]):
        n = int(rng.integers(case["nmin"], case["nmax"] + 1))
        iu, ju = np.triu_indices(n, 1)
        keep = rng.random(iu.size) < rng.uniform(0.2, 0.8)
        keep[0] = True  # never without an edge
        edges = np.stack([iu[keep], ju[keep]], axis=1).astype(np.int32)
        out.append(qi.MaxCut(n=n, edges=edges, weights=rng.uniform(-1.0, 1.0, edges.shape[0])))
    return out


def _starts(case, seed):
    """Start angles per graph: the ramp plus a little noise."""
    g, b = qi.linear_ramp(case["p"])
    rng = np.random.default_rng([int(seed), case["p"], 4])
    return (g + rng.normal(0.0, 0.05, (case["count"], case["p"])),
            b + rng.normal(0.0, 0.05, (case["count"], case["p"])))


def _theta(case, seed):
    return qi.mpnn_init_params(case["p"], [int(seed), 5]).astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, kind=kind)
    if kind == "batch":
        graphs = _graphs(case, seed)
        st["gamma"], st["beta"] = _starts(case, seed)
        st["batch"] = QaoaBatch(graphs, case["p"], steps=case["steps"], workgroups=case["workgroups"],
                                waves_per_simd=case["waves_per_simd"])
        return st
    if kind == "network":
        st["graphs"] = _graphs(case, seed)
        st["gamma"], st["beta"] = _starts(case, seed)
        st["net"] = QaoaMpnn(case["p"], _theta(case, seed))
        return st
    inst = _instance(case, seed)
    st["gamma"], st["beta"] = _angles(case, seed)
    if kind == "autograd":
        m = QaoaExpectationModule(inst, st["gamma"], st["beta"], case["precision"])
        st["module"] = m.float() if case["precision"] == "c64" else m
        return st
    if kind == "instance":
        st["instance"], st["seed"] = inst, int(seed)
        return st
    st["handle"] = QaoaHandle.from_instance(inst, case["precision"])
    if kind == "statevector":
        dt = torch.complex64 if case["precision"] == "c64" else torch.complex128
        st["out"] = torch.empty(1 << case["n"], dtype=dt, device="cuda")
    if kind == "sample":
        st["seed"] = int(seed)
        st["handle"].statevector(st["gamma"], st["beta"], copy=False)
        st["z"] = torch.empty(case["shots"], dtype=torch.int64, device="cuda")
        st["cost"] = torch.empty(case["shots"], dtype=torch.float64, device="cuda")
    return st


# ---------------------------------------------------------------- one pass

def run(state):
    kind, case = state["kind"], state["case"]
    g, b = state["gamma"], state["beta"]
    if kind == "gradient":
        E, dg, db = state["handle"].gradient(g, b)
        return {"E": E, "dgamma": dg, "dbeta": db}
    if kind == "autograd":
        m = state["module"]
        m.zero_grad(set_to_none=True)
        E = m().to(m.gamma.dtype)
        E.backward()
        return {"E": E.detach(), "dgamma": m.gamma.grad, "dbeta": m.beta.grad}
    if kind == "statevector":
        return {"psi": state["handle"].statevector(g, b, out=state["out"])}
    if kind == "sample":
        z, c = state["handle"].sample(case["shots"], state["seed"], z_out=state["z"], cost_out=state["cost"])
        return {"z": z, "cost": c}
    if kind == "instance":
        with QaoaHandle.from_instance(state["instance"], case["precision"]) as q:
            E = q.evaluate(g, b)
            z, c = q.sample(case["shots"], state["seed"])
        return {"E": E, "z": z.view(np.int64), "cost": c}
    if kind == "batch":
        gam, bet, e0, e1 = state["batch"].run(g, b)
        return {"gamma": gam, "beta": bet, "e_first": e0, "e_last": e1}
    loss, grad = state["net"].loss_grad(state["graphs"], g, b)
    return {"loss": loss, "grad": grad}


# ---------------------------------------------------------------- necessary work

def _evolve_work(n, p, precision, backward):
    """Bytes and operations of p layers (and of the adjoint sweep): a state that does not fit on the
    chip is read and written once per layer, state and adjoint vector once per layer backward, with
    the cost diagonal once each; one that fits needs the cost diagonal only."""
    s, c = (16, 8) if precision == "c128" else (8, 4)
    N = 2.0 ** n
    vectors = 2 if backward else 1
    if vectors * N * s <= _ON_CHIP:
        by = N * c
    else:
        by = N * (p * (2 * s + c) - s + (p * (4 * s + c) - 2 * s if backward else 0))
    # per amplitude: 4 flops a qubit and vector for the rotations, 4 a qubit for the <lam|X|phi>
    # terms, about 50 for a phase
    fl = N * p * (4 * n + 50 + (12 * n + 60 if backward else 0))
    return by, fl


def work(case):
    kind = case["kind"]
    if kind in ("batch", "network"):
        ns = range(case["nmin"], case["nmax"] + 1)
        share = case["count"] / len(ns)
    if kind == "batch":
        by = fl = 0.0
        for n in ns:
            b1, f1 = _evolve_work(n, case["p"], "c128", True)
            if 2 * 2.0 ** n * 16 <= _ON_CHIP:
                b1 = n * n * 12.0  # the graph; the cost diagonal follows from it
            by += share * case["steps"] * b1
            fl += share * case["steps"] * f1
        return {"bytes": by, "flops": fl}
    if kind == "network":
        nodes = share * sum(ns)
        edges = share * sum(0.25 * n * (n - 1) for n in ns)
        weights = 128 * 64 + 2 * 128 * 256 + 128 * 128 + 128 * 2 * case["p"]
        fl = 6.0 * nodes * (128 * 64 + 2 * 128 * 256) + 4.0 * 2 * edges * (32 + 2 * 128) * 2
        return {"bytes": edges * 16 + weights * 10.0 + case["count"] * case["p"] * 32.0, "flops": fl}
    n, p = case["n"], case["p"]
    N = 2.0 ** n
    s, c = (16, 8) if case["precision"] == "c128" else (8, 4)
    if kind == "sample":
        return {"bytes": N * s + case["shots"] * 16.0, "flops": 4.0 * N}
    by, fl = _evolve_work(n, p, case["precision"], kind in ("gradient", "autograd"))
    if kind == "statevector":
        by += N * s
    if kind == "instance":
        by += N * c + case["shots"] * 16.0
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------- 64-bit results

def _exact_cost(inst):
    n = inst.n
    z = torch.arange(1 << n, device=_DEV, dtype=torch.int64)
    if hasattr(inst, "edges"):
        C = torch.zeros(1 << n, device=_DEV, dtype=torch.float64)
        for (i, j), w in zip(inst.edges.tolist(), inst.weight_array().tolist()):
            C.add_(((z >> i) ^ (z >> j)).bitwise_and_(1), alpha=w)
        return C
    C = torch.full((1 << n,), float(inst.offset), device=_DEV, dtype=torch.float64)
    if hasattr(inst, "masks"):
        for m, w in zip(inst.masks.tolist(), inst.weights.tolist()):
            C.add_((z & m) == m, alpha=w)
        return C
    for (i, j), w in zip(inst.pairs.tolist(), inst.J.tolist()):
        C.add_(((z >> i) & (z >> j)).bitwise_and_(1), alpha=w)
    for i, w in enumerate(inst.h.tolist()):
        C.add_((z >> i).bitwise_and_(1), alpha=w)
    return C


def _phase_(psi, C, angle):
    """psi <- exp(-i angle C) psi, a slice at a time; angle: a number, or [G, 1] for psi [G, N]."""
    step = 1 << 26
    if not torch.is_tensor(angle):
        for k in range(0, psi.numel(), step):
            a = C[k:k + step] * -angle
            psi[k:k + step] *= torch.complex(a.cos(), a.sin())
    else:
        a = -angle * C
        psi *= torch.complex(a.cos(), a.sin())


def _mix_(psi, n, c, s):
    """psi <- prod_j (c - i s X_j) psi on the last axis; c, s: numbers, or [G, 1, 1] for psi [G, N]."""
    lead = psi.shape[:-1]
    for j in range(n):
        v = psi.view(*lead, -1, 2, 1 << j)
        a, b = v[..., 0, :], v[..., 1, :]
        t = a * c - 1j * (b * s)
        b.mul_(c).sub_(1j * (a * s))
        a.copy_(t)


def _xsum(lam, phi, n):
    """sum_j Im <lam|X_j|phi> over the last axis."""
    lead = phi.shape[:-1]
    tot = 0.0
    for j in range(n):
        p = phi.view(*lead, -1, 2, 1 << j)
        q = lam.view(*lead, -1, 2, 1 << j)
        for x, y in ((0, 1), (1, 0)):
            u, v = q[..., x, :], p[..., y, :]
            t = u.real * v.imag - u.imag * v.real
            tot = tot + t.sum(dim=(-1, -2))
    return tot


def _exact_gradient(C, n, gamma, beta):
    """(E, dgamma, dbeta); C [N] with numbers, or [G, N] with gamma, beta [G, p] tensors."""
    many = C.dim() == 2
    p = gamma.shape[-1]

    def ang(l):
        if not many:
            return float(gamma[l]), math.cos(float(beta[l])), math.sin(float(beta[l]))
        return gamma[:, l:l + 1], beta[:, l].cos().view(-1, 1, 1), beta[:, l].sin().view(-1, 1, 1)

    phi = torch.full(C.shape, 2.0 ** (-n / 2), dtype=torch.complex128, device=C.device)
    for l in range(p):
        g, c, s = ang(l)
        _phase_(phi, C, g)
        _mix_(phi, n, c, s)
    E = (C * phi.real ** 2).sum(-1) + (C * phi.imag ** 2).sum(-1)
    lam = phi * C
    dg, db = [None] * p, [None] * p
    for l in range(p - 1, -1, -1):
        g, c, s = ang(l)
        db[l] = 2 * _xsum(lam, phi, n)
        _mix_(phi, n, c, -s)
        _mix_(lam, n, c, -s)
        dg[l] = 2 * ((C * lam.real * phi.imag).sum(-1) - (C * lam.imag * phi.real).sum(-1))
        if l:
            _phase_(phi, C, -g)
            _phase_(lam, C, -g)
    return E, torch.stack(dg, -1), torch.stack(db, -1)


def _exact_state(C, n, gamma, beta):
    phi = torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device=C.device)
    for g, b in zip(gamma, beta):
        _phase_(phi, C, float(g))
        _mix_(phi, n, math.cos(float(b)), math.sin(float(b)))
    return phi


def _exact_batch(case, seed):
    """The batch's Adam runs in 64 bits, the graphs of one size together."""
    graphs = _graphs(case, seed)
    g0, b0 = _starts(case, seed)
    p, count = case["p"], case["count"]
    out = dict(gamma=np.empty((count, p)), beta=np.empty((count, p)), e_first=np.empty(count), e_last=np.empty(count))
    by_n = {}
    for i, gr in enumerate(graphs):
        by_n.setdefault(gr.n, []).append(i)
    for n, idx in by_n.items():
        most = max(1, (1 << 27) >> n)
        for k in range(0, len(idx), most):
            sel = idx[k:k + most]
            C = torch.stack([_exact_cost(graphs[i]) for i in sel])
            scale = torch.tensor([1.0 / np.abs(graphs[i].weights).sum() for i in sel], device=_DEV).view(-1, 1).double()
            th = torch.tensor(np.concatenate([g0[sel], b0[sel]], axis=1), device=_DEV)
            m, v = torch.zeros_like(th), torch.zeros_like(th)
            for t in range(1, case["steps"] + 2):
                E, dg, db = _exact_gradient(C, n, th[:, :p], th[:, p:])
                if t == 1:
                    out["e_first"][sel] = E.cpu().numpy()
                if t > case["steps"]:
                    out["e_last"][sel] = E.cpu().numpy()
                    break
                g = torch.cat([dg, db], 1) * scale
                m = 0.9 * m + 0.1 * g
                v = 0.999 * v + 0.001 * g * g
                th = th + 0.05 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
            out["gamma"][sel] = th[:, :p].cpu().numpy()
            out["beta"][sel] = th[:, p:].cpu().numpy()
    return out


def _exact_network(case, seed):
    """Loss and flat gradient of the network in 64 bits."""
    p, graphs = case["p"], _graphs(case, seed)
    gt, bt = _starts(case, seed)
    theta = torch.tensor(_theta(case, seed), dtype=torch.float64, requires_grad=True)
    par, o = {}, 0
    for name, shape in qi.mpnn_param_shapes(p):
        k = int(np.prod(shape))
        par[name] = theta[o:o + k].view(shape)
        o += k
    pooled = []
    for gr in graphs:
        A = torch.zeros(gr.n, gr.n, dtype=torch.float64)
        w = torch.tensor(gr.weights)
        i, j = torch.tensor(gr.edges[:, 0]).long(), torch.tensor(gr.edges[:, 1]).long()
        A[i, j] = w
        A[j, i] = w
        H = torch.zeros(gr.n, 32, dtype=torch.float64)
        H[:, 0] = (A != 0).sum(1) / 8.0
        H[:, 1] = A.sum(1) / 8.0
        H[:, 2] = 1.0
        H[:, 3] = (A * A).sum(1) / 8.0
        for l in range(3):
            H = torch.relu(torch.cat([H, A @ H], 1) @ par[f"W{l}"].T + par[f"b{l}"])
        pooled.append(H.mean(0))
    Y = torch.relu(torch.stack(pooled) @ par["Wh1"].T + par["bh1"]) @ par["Wh2"].T + par["bh2"]
    r = torch.arange(1, p + 1, dtype=torch.float64) / p
    ang = Y + torch.cat([r, 1.0 - r])
    loss = ((ang - torch.tensor(np.concatenate([gt, bt], axis=1))) ** 2).mean()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": theta.grad.numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None  # basis states: whole numbers
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "network":
        return _exact_network(case, seed)
    inst = _instance(case, seed)
    gamma, beta = _angles(case, seed)
    if kind == "autograd" and case["precision"] == "c64":
        gamma, beta = np.float32(gamma).astype(np.float64), np.float32(beta).astype(np.float64)
    C = _exact_cost(inst)
    if kind == "statevector":
        return {"psi": _exact_state(C, case["n"], gamma, beta)}
    if kind == "instance":
        psi = _exact_state(C, case["n"], gamma, beta)
        return {"E": float((C * (psi.real ** 2 + psi.imag ** 2)).sum()), "z": None, "cost": None}
    E, dg, db = _exact_gradient(C, case["n"], gamma, beta)
    return {"E": float(E), "dgamma": dg.cpu(), "dbeta": db.cpu()}
