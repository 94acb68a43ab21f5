"""The work this library is used for, as cases that can be timed and checked.

Every case goes through the public entry points of ``paper_2511_19291_amd``
with what a user's program keeps between calls (the state, the fusion plan,
the batch plan) prepared beforehand:

  run     a circuit gate by gate (``State.reset().run``) and every <Z_i>:
          12 qubits (a single small circuit, where launches and host time
          count), 20 qubits (the state fits the caches) and 27 qubits (it
          does not)
  fused   the same brickwork as planned blocks on the matrix cores
          (``apply_fused``), FP32 and split BF16
  step    a training step of the RX/RY ring, one state: loss <sum Z_i> and
          the gradient of every angle (``QuantumExpval``)
  ladder  a training step of the encoded RY ladder, a batch of input rows:
          every <Z_i> of every row, the gradients of inputs and angles
          (``MeasureAllZ``), from launch-bound to batch 16 at 18 qubits
  batch   many uneven circuits in one launch (``BatchPlan``)
  shots   exact draws and the estimates from them (``sample_exact``,
          ``sample_z_estimate``)
  gauss   the differentiable shot estimate, forward and backward
          (``gaussian_expval_z``, ``gaussian_expval_z_backward``)
  energy  the terms of a chain Hamiltonian (``State.expval``)

Angles, features and states are drawn from the seed. States that a case
starts from have normally distributed amplitudes, which is how the output
amplitudes of deep random circuits are distributed.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_19291_amd import circuits as C
from paper_2511_19291_amd import sv
from paper_2511_19291_amd.autograd import MeasureAllZ, QuantumExpval

MODES = {"fp32": sv.FUSED_FP32_MFMA, "bf16x3": sv.FUSED_BF16X3}


def listed():
    return [
        # one small circuit and its measurement: launch and host bound
        {"name": "hea12", "kind": "run", "circuit": "hea", "n": 12, "layers": 4},
        # a cache-resident state
        {"name": "brickwork20", "kind": "run", "circuit": "brickwork", "n": 20, "layers": 20},
        # a state far beyond the caches (1 GiB), 800 gates
        {"name": "brickwork27", "kind": "run", "circuit": "brickwork", "n": 27, "layers": 20},
        # planned blocks of five qubits in the default arithmetic
        {"name": "fused27_fp32", "kind": "fused", "mode": "fp32", "max_k": 5, "n": 27, "layers": 20},
        # and in split BF16, the fastest of the fused arithmetics
        {"name": "fused26_bf16x3", "kind": "fused", "mode": "bf16x3", "max_k": 5, "n": 26, "layers": 20},
        # a training step on one large state (odd width): 500 angles
        {"name": "ring25_step", "kind": "step", "n": 25, "layers": 10},
        # a training step of a small model on a small batch: launch and host bound
        {"name": "ladder10_b8", "kind": "ladder", "n": 10, "blocks": 3, "batch": 8},
        # the profiling workload's smallest measured width, batch 16
        {"name": "ladder18_b16", "kind": "ladder", "n": 18, "blocks": 3, "batch": 16},
        # 256 uneven circuits of 10..20 qubits in one launch
        {"name": "batch256", "kind": "batch", "circuits": 256, "nmin": 10, "nmax": 20, "layers": 6},
        # a million exact draws from a 27-qubit state
        {"name": "shots27", "kind": "shots", "n": 27, "shots": 1 << 20},
        # the differentiable estimate over every bin of a 26-qubit state
        {"name": "gauss26", "kind": "gauss", "n": 26, "shots": 1e9},
        # <X X>, <Y Y>, <Z Z> of every bond of a 24-qubit chain
        {"name": "energy24", "kind": "energy", "n": 24},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "fused", "fused", "step", "ladder", "ladder", "batch", "shots", "gauss",
                       "energy"])
    if kind == "run":
        circuit = rng.choice(["hea", "brickwork", "ring"])
        n = rng.randint(5, 26)
        return {"kind": kind, "circuit": circuit, "n": n, "layers": rng.randint(2, 20 if n <= 24 else 12)}
    if kind == "fused":
        mode = rng.choice(["fp32", "bf16x3"])
        return {"kind": kind, "mode": mode, "max_k": rng.choice([4, 5, 6] if mode == "bf16x3" else [3, 4, 5]),
                "n": rng.randint(14, 26), "layers": rng.randint(3, 20)}
    if kind == "step":
        return {"kind": kind, "n": rng.randint(9, 24), "layers": rng.randint(2, 10)}
    if kind == "ladder":
        n = rng.randint(6, 20)
        return {"kind": kind, "n": n, "blocks": rng.randint(1, 4), "batch": _log_int(rng, 2, 16)}
    if kind == "batch":
        nmin = rng.randint(8, 12)
        return {"kind": kind, "circuits": _log_int(rng, 24, 256), "nmin": nmin, "nmax": rng.randint(nmin + 2, 19),
                "layers": rng.randint(2, 6)}
    if kind == "shots":
        return {"kind": kind, "n": rng.randint(15, 27), "shots": _log_int(rng, 1000, 1 << 20)}
    if kind == "gauss":
        return {"kind": kind, "n": rng.randint(14, 26), "shots": float(10 ** rng.randint(5, 9))}
    return {"kind": kind, "n": rng.randint(12, 25)}


# ------------------------------------------------------------ inputs

def _circuit(case, seed):
    n, kind = case["n"], case["kind"]
    if kind == "step":
        # small initial angles, as circuits of this width are trained from:
        # with angles over the whole circle the loss is all cancellation
        c = C.rxry_ring(n, case["layers"], seed, small_angle=True)
    elif case.get("circuit") == "ring":
        c = C.rxry_ring(n, case["layers"], seed)
    elif case.get("circuit") == "hea":
        c = C.hea_ladder(n, case["layers"], seed)
    else:
        c = C.brickwork_u3_cz(n, case["layers"], seed)
    return c


def _amplitudes(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    t = torch.randn((1 << n, 2), device="cuda", generator=g)
    t *= 1.0 / math.sqrt(float(t.double().square().sum()) if n <= 24 else 2.0 * (1 << n))
    return torch.view_as_complex(t).reshape(1, 1 << n)


def _uniforms(count, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    return torch.rand(count, dtype=torch.float64, device="cuda", generator=g)


def _normals(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    return torch.randn(1 << n, dtype=torch.float64, device="cuda", generator=g)


def _upstream(n, seed):
    return np.random.default_rng(seed + 2).normal(size=n)


def _batch_circuits(case, seed):
    return C.batch_workload(case["circuits"], case["nmin"], case["nmax"], case["layers"], seed)


def _chain(n):
    terms = []
    for q in range(n - 1):
        terms += [C.pauli_term(0.5, f"X{q} X{q + 1}"), C.pauli_term(0.5, f"Y{q} Y{q + 1}"),
                  C.pauli_term(1.0, f"Z{q} Z{q + 1}")]
    return terms


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "fused"):
        circ = _circuit(case, seed)
        s = {"case": case, "circ": circ, "state": sv.State(case["n"])}
        if kind == "fused":
            s["blocks"] = sv.fuse_plan(circ, case["max_k"])
        return s
    if kind == "step":
        circ = _circuit(case, seed)
        theta = torch.tensor(circ.params, dtype=torch.float32, requires_grad=True)
        return {"case": case, "theta": theta, "model": QuantumExpval(circ, C.z_sum_terms(case["n"]))}
    if kind == "ladder":
        n = case["n"]
        circ, rows = C.profiling_ladder(n, case["blocks"], case["batch"], seed)
        x = torch.tensor(rows[:, :n], dtype=torch.float32, requires_grad=True)
        theta = torch.tensor(rows[0, n:], dtype=torch.float32, requires_grad=True)
        return {"case": case, "x": x, "theta": theta, "model": MeasureAllZ(circ, case["batch"])}
    if kind == "batch":
        plan = sv.BatchPlan(_batch_circuits(case, seed))
        return {"case": case, "plan": plan, "params": plan.pack(), "out": plan.out_buffer()}
    state = sv.State(case["n"], tensor=_amplitudes(case["n"], seed))
    s = {"case": case, "state": state}
    if kind == "shots":
        s["u"] = _uniforms(case["shots"], seed)
    elif kind == "gauss":
        s["z"] = _normals(case["n"], seed)
        s["g"] = _upstream(case["n"], seed)
    else:
        s["terms"] = _chain(case["n"])
    return s


# ------------------------------------------------------------ one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "run":
        st = s["state"]
        st.reset().run(s["circ"])
        # measured values in the precision the state is held in
        return {"state": st.tensor, "z": torch.as_tensor(st.expval_z_all(), dtype=torch.float32)}
    if kind == "fused":
        st = s["state"]
        st.reset().apply_fused(s["blocks"], MODES[case["mode"]])
        return {"state": st.tensor}
    if kind == "step":
        loss = s["model"](s["theta"])
        (grad,) = torch.autograd.grad(loss, s["theta"])
        return {"loss": loss.detach(), "grad": grad}
    if kind == "ladder":
        x, theta = s["x"], s["theta"]
        z = s["model"](torch.cat([x, theta.expand(x.shape[0], -1)], dim=1))
        gx, gt = torch.autograd.grad((z ** 2).sum(), (x, theta))
        return {"z": z.detach(), "grad_x": gx, "grad_theta": gt}
    if kind == "batch":
        s["plan"].launch(s["params"], s["out"])
        # features for a float32 model behind the circuits
        return {"z": s["out"].to(torch.float32)}
    st = s["state"]
    if kind == "shots":
        idx = st.sample_exact(s["u"])
        return {"indices": idx, "est": st.sample_z_estimate(idx)}
    if kind == "gauss":
        est = st.gaussian_expval_z(s["z"], case["shots"])
        return {"est": est, "weights": st.gaussian_expval_z_backward(s["z"], case["shots"], s["g"])}
    return {"terms": st.expval(s["terms"])}


# ------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: each input read once, each output written once. Operations per
    amplitude: 14 for a general gate (two complex products and their sum), 6
    for a rotation (its matrix has two real or imaginary numbers, or one
    phase), none for an exchange or a sign, 4 for a derivative (the real part
    of a product)."""
    kind = case["kind"]
    if kind == "batch":
        rng_mid = 0.5 * (case["nmin"] + case["nmax"])
        flops = sum(6.0 * (1 << n) * n * (1 + 2 * case["layers"]) for n in range(case["nmin"], case["nmax"] + 1))
        flops *= case["circuits"] / (case["nmax"] - case["nmin"] + 1)
        return {"bytes": case["circuits"] * 8.0 * (rng_mid * (2 + 2 * case["layers"])), "flops": flops}
    n = case["n"]
    amps = float(1 << n)
    if kind in ("run", "fused"):
        per_wire = {"ring": 12.0, "hea": 12.0}.get(case.get("circuit"), 14.0)
        return {"bytes": 8.0 * amps, "flops": per_wire * amps * n * case["layers"]}
    if kind == "step":
        p = 2 * n * case["layers"]
        return {"bytes": 8.0 * p, "flops": amps * p * (6.0 + 2 * 6.0 + 4.0)}
    if kind == "ladder":
        p = n * (1 + case["blocks"])
        return {"bytes": 8.0 * p * case["batch"], "flops": case["batch"] * amps * p * (6.0 + 2 * 6.0 + 4.0)}
    if kind == "shots":
        return {"bytes": 8.0 * amps + 24.0 * case["shots"], "flops": 4.0 * amps}
    if kind == "gauss":
        return {"bytes": (8.0 + 8.0 + 8.0) * amps, "flops": 40.0 * amps}
    return {"bytes": 8.0 * amps, "flops": 3.0 * (n - 1) * 8.0 * amps}


# ------------------------------------------------------------ the same in 64 bits

def _cols(p, op):
    return [p[:, j].reshape(-1, 1, 1) for j in op.params]


def _one_qubit(kind, v):
    """(m00, m01, m10, m11) per row."""
    if kind == "rz":
        return torch.exp(-0.5j * v[0]), None, None, torch.exp(0.5j * v[0])
    c, s = torch.cos(v[0] / 2), torch.sin(v[0] / 2)
    if kind == "ry":
        return c, -s, s, c
    if kind == "rx":
        return c, -1j * s, -1j * s, c
    if kind == "u3":
        return c, -torch.exp(1j * v[2]) * s, torch.exp(1j * v[1]) * s, torch.exp(1j * (v[1] + v[2])) * c
    raise ValueError(kind)


def _apply(psi, op, p, inverse=False):
    """psi [rows, 2^n] complex128, changed in place."""
    rows = psi.shape[0]
    if op.controls:
        c, t = op.controls[0], op.targets[0]
        hi, lo = max(c, t), min(c, t)
        v = psi.view(rows, -1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
        if op.kind == "z":
            v[:, :, 1, :, 1, :] *= -1.0
        else:
            a = v[:, :, 1, :, 0, :] if c == hi else v[:, :, 0, :, 1, :]
            b = v[:, :, 1, :, 1, :]
            keep = a.clone()
            a.copy_(b)
            b.copy_(keep)
        return
    m = _one_qubit(op.kind, _cols(p, op))
    if inverse:
        m = [None if x is None else x.conj() if x.is_complex() else x for x in (m[0], m[2], m[1], m[3])]
    v = psi.view(rows, -1, 2, 1 << op.targets[0])
    a, b = v[:, :, 0, :], v[:, :, 1, :]
    if m[1] is None:
        a *= m[0]
        b *= m[3]
        return
    new = m[0] * a
    new += m[1] * b
    b *= m[3]
    b += m[2] * a
    a.copy_(new)


def _zero_state(rows, n):
    psi = torch.zeros((rows, 1 << n), dtype=torch.complex128, device="cuda")
    psi[:, 0] = 1.0
    return psi


def _z_all(psi, n):
    q = psi.real.square() + psi.imag.square()
    return torch.stack([(q.view(q.shape[0], -1, 2, 1 << i).sum(dim=(1, 3)) @ q.new_tensor([1.0, -1.0]))
                        for i in range(n)] + [q.sum(dim=1)], dim=1)


def _forward(circ, p, rows=1):
    psi = _zero_state(rows, circ.n)
    for op in circ.ops:
        _apply(psi, op, p)
    return psi


def _gradient(circ, p, psi, coeff):
    """d sum_i coeff[r, i] <Z_i>_r / d p[r, :] for rotation gates."""
    rows, n = psi.shape[0], circ.n
    idx = torch.arange(1 << n, device="cuda")
    d = torch.zeros((rows, 1 << n), dtype=torch.float64, device="cuda")
    for i in range(n):
        d += coeff[:, i:i + 1] * (1.0 - 2.0 * ((idx >> i) & 1))
    lam = psi * d
    del d, idx
    grad = torch.zeros_like(p)
    for op in reversed(circ.ops):
        if op.params:
            a, b = (psi.view(rows, -1, 2, 1 << op.targets[0])[:, :, k, :] for k in (0, 1))
            la, lb = (lam.view(rows, -1, 2, 1 << op.targets[0])[:, :, k, :] for k in (0, 1))
            u = (la.conj() * b).sum(dim=(1, 2))
            w = (lb.conj() * a).sum(dim=(1, 2))
            # Im <lam|X|psi> or Im <lam|Y|psi>
            grad[:, op.params[0]] += (u + w).imag if op.kind == "rx" else (w - u).real
        _apply(psi, op, p, inverse=True)
        _apply(lam, op, p, inverse=True)
    return grad


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "fused"):
        circ = _circuit(case, seed)
        psi = _forward(circ, torch.tensor(circ.params, device="cuda").reshape(1, -1))
        if kind == "fused":
            return {"state": psi}
        return {"state": psi, "z": _z_all(psi, case["n"])}
    if kind == "step":
        circ = _circuit(case, seed)
        p = torch.tensor(circ.params, dtype=torch.float32).double().cuda().reshape(1, -1)
        psi = _forward(circ, p)
        loss = _z_all(psi, case["n"])[0, :-1].sum()
        grad = _gradient(circ, p, psi, torch.ones((1, case["n"]), dtype=torch.float64, device="cuda"))
        return {"loss": loss, "grad": grad[0]}
    if kind == "ladder":
        n = case["n"]
        circ, rows = C.profiling_ladder(n, case["blocks"], case["batch"], seed)
        p = torch.tensor(rows, dtype=torch.float32).double().cuda()
        psi = _forward(circ, p, case["batch"])
        z = _z_all(psi, n)[:, :-1]
        grad = _gradient(circ, p, psi, 2.0 * z)
        return {"z": z, "grad_x": grad[:, :n], "grad_theta": grad[:, n:].sum(dim=0)}
    if kind == "batch":
        circs = _batch_circuits(case, seed)
        if sum(len(c.ops) for c in circs) > 80000:
            return None
        out = torch.zeros((len(circs), sv.BATCH_OUT_STRIDE), dtype=torch.float64, device="cuda")
        for i, c in enumerate(circs):
            psi = _forward(c, torch.tensor(c.params, device="cuda").reshape(1, -1))
            out[i, : c.n] = _z_all(psi, c.n)[0, : c.n]
        return {"z": out}
    n = case["n"]
    psi = _amplitudes(n, seed).to(torch.complex128)
    if kind == "shots":
        q = (psi.real.square() + psi.imag.square()).reshape(-1)
        cum = torch.cumsum(q, dim=0)
        idx = torch.searchsorted(cum, _uniforms(case["shots"], seed) * cum[-1], right=True).clamp(max=(1 << n) - 1)
        est = torch.stack([1.0 - 2.0 * ((idx >> i) & 1).double().mean() for i in range(n)])
        return {"indices": None, "est": est}
    if kind == "gauss":
        return _gauss(case, seed, psi.reshape(-1))
    v = psi.reshape(-1)
    out = []
    for c, xm, zm in _chain(n):
        q = (xm or zm).bit_length() - 2
        w = v.view(-1, 2, 2, 1 << q)            # bits q + 1, q
        if not xm:
            s = (w.real.square() + w.imag.square()).sum(dim=(0, 3))
            out.append(c * (s[0, 0] + s[1, 1] - s[0, 1] - s[1, 0]))
        else:
            d = (w[:, 0, 0].conj() * w[:, 1, 1]).real.sum() * 2.0      # |11> <-> |00>
            o = (w[:, 0, 1].conj() * w[:, 1, 0]).real.sum() * 2.0      # |01> <-> |10>
            out.append(c * ((o - d) if zm else (o + d)))
    return {"terms": torch.stack(out).reshape(1, -1)}


def _gauss(case, seed, psi):
    """The reparameterised estimate y = n p + sqrt(n) D S z and its
    derivative by |psi|^2 with the normals held fixed, with autograd left to
    torch's arithmetic in closed form (u = sqrt p, d = e - u)."""
    n, shots = case["n"], case["shots"]
    q = psi.real.square() + psi.imag.square()
    del psi
    total = q.sum()
    u = (q / total).sqrt()
    z = _normals(n, seed).clone()
    z[-1] = 0.0
    d = -u
    d[-1] += 1.0
    r, k = (d * d).sum(), (d * z).sum()
    sz = z - 2.0 * d * (k / r)
    y = u * u + u * sz / math.sqrt(shots)
    est = torch.stack([(y.view(-1, 2, 1 << i).sum(dim=(0, 2)) * y.new_tensor([1.0, -1.0])).sum() for i in range(n)])
    del y
    idx = torch.arange(1 << n, device="cuda")
    c = torch.zeros_like(u)
    for i, g in enumerate(_upstream(n, seed)):
        c += float(g) * (1.0 - 2.0 * ((idx >> i) & 1))
    del idx
    sq = math.sqrt(shots)
    big_q = (c * u * d).sum()
    w = c + c * (k / (r * sq)) + (c * sz + z * (2.0 * big_q / r) - d * (4.0 * k * big_q / (r * r))) / (2.0 * sq * u)
    mean = (u * u * w).sum()
    return {"est": est, "weights": (w - mean) / total}
