"""Workloads timed on the GPU: the calls a user of this package makes, at the
sizes of the repository's own workloads and test shapes.

``listed()`` holds the named cases, ``draw(rng)`` gives another case of the
same ranges, ``prepare`` makes what a program has in hand before the call,
``run`` is one pass through the public entry points, ``work`` the bytes and
operations the pass cannot do without, and ``exact`` the same outputs in
64 bits from plain torch and numpy.
"""
import math

import numpy as np
import torch

import paper_2512_07311_amd as rcs

PATTERN = "ABCDCDAB"


def listed():
    return [
        # Whole call on the smallest workload: the exact 12-qubit circuit, its
        # shots, their XEB and every amplitude (checking a circuit by hand).
        dict(name="state_12q_exact", kind="state", rows=3, cols=4, cycles=8, chi=64, eps=0.0,
             network="snake", shots=10000, amps=4096),
        # Whole call with truncation at the bond cap: splits of up to
        # 1024 x 1024, centre moves and contractions of a real schedule.
        dict(name="state_20q_chi512", kind="state", rows=4, cols=5, cycles=8, chi=512, eps=1e-8,
             network="interleaved", shots=20000, amps=1000),
        # SVD of a saturated cut of the chi 1024 build: where the build of the
        # 53-qubit state spends its time.
        dict(name="svd_2048", kind="svd", len=2048, cnt=2048, low=0.05),
        # SVD of an edge cut or a small circuit: odd sizes, bound by latency.
        dict(name="svd_203x131", kind="svd", len=203, cnt=131, low=0.05),
        # Single-precision SVD of a cap-limited cut (learned/FP32 build): the
        # singular values and the rank-k truncation it is used for.
        dict(name="svd_f32_1024", kind="svd_f32", len=1024, cnt=1024, low=0.3),
        # Move of the orthogonality centre across a saturated site.
        dict(name="qr_2048x1024", kind="qr", len=2048, cnt=1024, low=0.03),
        # Two-site contraction at the cap, complex128 (plain build).
        dict(name="two_site_1024", kind="two_site", dl=1024, dm=1024, dr=1024, precision="c128"),
        # Two-site contraction in split bf16 (learned/FP32 build), ragged bonds.
        dict(name="two_site_bf16_ragged", kind="two_site", dl=700, dm=1001, dr=517, precision="split_bf16"),
        # Shots with their log-probabilities from a state at bond cap 1024.
        dict(name="sample_chi1024", kind="sample", n=24, chi=1024, shots=65536),
        # Shots from a heterogeneous batch of states (20 to 40 qubits).
        dict(name="sample_batch6", kind="sample_batch", states=6, n_lo=20, n_hi=40, chi=256, shots=4000),
        # Exact state vector, the probabilities of a shot list and its XEB.
        dict(name="dense_28q", kind="dense", rows=4, cols=7, cycles=8, shots=1000000),
        # One training step of the rank network at the driver's batch size.
        dict(name="train_256", kind="train", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["state", "svd", "svd", "svd_f32", "qr", "two_site", "two_site", "sample", "sample_batch",
                       "dense", "train"])
    if kind == "state":
        rows, cols, chi = rng.choice([(2, 5, 64), (3, 3, 64), (3, 4, 32), (3, 4, 64), (3, 5, 64), (4, 4, 64),
                                      (4, 4, 100), (4, 5, 96), (4, 5, 200), (4, 5, 256)])
        return dict(kind=kind, rows=rows, cols=cols, cycles=rng.randint(4, 8), chi=chi,
                    eps=rng.choice([0.0, 1e-8]), network=rng.choice(["snake", "interleaved"]),
                    shots=_log_int(rng, 500, 20000), amps=rng.randint(1, 1000))
    if kind == "svd":
        cnt = _log_int(rng, 24, 1500)
        return dict(kind=kind, len=rng.randint(cnt, 2 * cnt), cnt=cnt, low=round(rng.uniform(0.03, 0.3), 3))
    if kind == "svd_f32":
        cnt = _log_int(rng, 64, 1200)
        return dict(kind=kind, len=rng.randint(cnt, 2 * cnt), cnt=cnt, low=round(rng.uniform(0.2, 0.5), 3))
    if kind == "qr":
        cnt = _log_int(rng, 64, 1400)
        return dict(kind=kind, len=rng.randint(cnt, 2 * cnt), cnt=cnt, low=round(rng.uniform(0.02, 0.3), 3))
    if kind == "two_site":
        return dict(kind=kind, dl=_log_int(rng, 3, 1200), dm=_log_int(rng, 3, 1200), dr=_log_int(rng, 3, 1200),
                    precision=rng.choice(["c128", "c128", "c64", "split_bf16"]))
    if kind == "sample":
        chi = _log_int(rng, 40, 900)
        return dict(kind=kind, n=rng.randint(18, 26), chi=chi, shots=_log_int(rng, 700, 40000))
    if kind == "sample_batch":
        return dict(kind=kind, states=rng.randint(2, 6), n_lo=rng.randint(10, 20), n_hi=rng.randint(21, 40),
                    chi=_log_int(rng, 64, 256), shots=_log_int(rng, 300, 4000))
    if kind == "dense":
        rows, cols = rng.choice([(3, 4), (4, 4), (3, 7), (4, 5), (4, 6), (5, 5), (3, 9)])
        return dict(kind=kind, rows=rows, cols=cols, cycles=rng.randint(4, 10), shots=_log_int(rng, 1000, 1000000))
    return dict(kind=kind, batch=_log_int(rng, 16, 1024))


# ------------------------------------------------------------------ inputs
def _dev(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def _normal(g, *shape):
    re = torch.randn(*shape, dtype=torch.float64, device="cuda", generator=g)
    return torch.complex(re, torch.randn(*shape, dtype=torch.float64, device="cuda", generator=g))


def _phases(g, n):
    t = torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * (2 * math.pi)
    return torch.complex(torch.cos(t), torch.sin(t))


def _dft(n):
    i = torch.arange(n, dtype=torch.int64, device="cuda")
    t = (i[:, None] * i[None, :] % n).double() * (-2 * math.pi / n)
    return torch.complex(torch.cos(t), torch.sin(t)) / math.sqrt(n)


def _unitary(g, n):
    """A dense random unitary matrix: transform, random phases, transform."""
    f = _dft(n)
    return torch.matmul(f * _phases(g, n), f * _phases(g, n))


def _spectrum(case):
    """Singular values of a saturated cut: flat, falling to `low` of the
    largest; the fp32 case has the gap at the kept rank that makes its
    truncation well defined."""
    n = case["cnt"]
    if case["kind"] == "svd_f32":
        k = n // 2
        s = torch.cat([torch.logspace(0.0, math.log10(case["low"]), k, dtype=torch.float64),
                       torch.logspace(math.log10(case["low"] * 0.3), math.log10(case["low"] * 0.1), n - k,
                                      dtype=torch.float64)])
    else:
        s = torch.logspace(0.0, math.log10(case["low"]), n, dtype=torch.float64)
    return s.cuda()


def _planted(case, seed):
    """(u, s, v): the matrix is u diag(s) v^H, u len x cnt."""
    g = _dev(seed)
    u = _unitary(g, case["len"])[:, :case["cnt"]]
    return u, _spectrum(case), _unitary(g, case["cnt"])


def _planted_columns(case, seed):
    u, s, v = _planted(case, seed)
    return torch.matmul(u * s, v.conj().T).T.contiguous()     # (cnt, len): columns contiguous


def _bits(g, n_qubits, m):
    return torch.randint(0, 1 << min(n_qubits, 62), (m,), dtype=torch.int64, device="cuda", generator=g)


def _bond_dims(n, chi):
    return [min(1 << min(b, n - b, 30), chi) for b in range(n + 1)]


def _right_canonical(g, n, chi):
    """Site tensors (dl, 2, dr) with orthonormal rows: a random state of
    unit norm at the full bond profile of the cap."""
    d = _bond_dims(n, chi)
    return d, [_unitary(g, 2 * d[k + 1])[:d[k]].reshape(d[k], 2, d[k + 1]) for k in range(n)]


def _batch_states(case):
    m = case["states"]
    out = []
    for i in range(m):
        n = case["n_lo"] + (case["n_hi"] - case["n_lo"]) * i // max(m - 1, 1)
        out.append((n, max(2, case["chi"] >> (i % 3))))
    return out


def _snake(n, seed):
    return np.random.RandomState(seed & 0x7FFFFFFF).permutation(n).astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    g = _dev(seed)
    st = dict(case=case, kind=kind, seed=int(seed))
    if kind == "state":
        n = case["rows"] * case["cols"]
        st["circuit"] = rcs.Circuit(case["rows"], case["cols"], case["cycles"], seed=seed, network=case["network"])
        st["bits"] = torch.zeros(case["shots"], dtype=torch.int64, device="cuda")
        st["log2p"] = torch.zeros(case["shots"], dtype=torch.float64, device="cuda")
        st["query"] = _query(case, seed)
        st["amps"] = torch.zeros(case["amps"], dtype=torch.complex128, device="cuda")
        st["n"] = n
    elif kind in ("svd", "svd_f32", "qr"):
        st["m"] = _planted_columns(case, seed)
        st["x"] = torch.empty_like(st["m"])
        st["s"] = torch.zeros(case["cnt"], dtype=torch.float64, device="cuda")
        st["u"] = torch.zeros_like(st["m"])
        st["r"] = torch.zeros(case["cnt"], case["cnt"], dtype=torch.complex128, device="cuda")
    elif kind == "two_site":
        dl, dm, dr = case["dl"], case["dm"], case["dr"]
        st["a"] = _normal(g, dl, 2, dm) / math.sqrt(4 * dm)
        st["b"] = _normal(g, dm, 2, dr) / math.sqrt(4 * dr)
        st["gate"] = _fsim()
        st["out"] = torch.zeros(2 * dr, 2 * dl, dtype=torch.complex128, device="cuda")
    elif kind == "sample":
        d, a = _right_canonical(g, case["n"], case["chi"])
        st["state"] = rcs.State.from_host(d, _snake(case["n"], seed), [t.cpu().numpy() for t in a])
        st["bits"] = torch.zeros(case["shots"], dtype=torch.int64, device="cuda")
        st["log2p"] = torch.zeros(case["shots"], dtype=torch.float64, device="cuda")
    elif kind == "sample_batch":
        st["states"] = []
        for i, (n, chi) in enumerate(_batch_states(case)):
            d, a = _right_canonical(g, n, chi)
            st["states"].append(rcs.State.from_host(d, _snake(n, seed + i), [t.cpu().numpy() for t in a]))
        st["bits"] = torch.zeros(case["states"], case["shots"], dtype=torch.int64, device="cuda")
        st["log2p"] = torch.zeros(case["states"], case["shots"], dtype=torch.float64, device="cuda")
    elif kind == "dense":
        n = case["rows"] * case["cols"]
        st["n"] = n
        st["circuit"] = rcs.Circuit(case["rows"], case["cols"], case["cycles"], seed=seed)
        st["psi"] = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
        st["bits"] = _bits(g, n, case["shots"])
        st["p"] = torch.zeros(case["shots"], dtype=torch.float64, device="cuda")
    else:
        for k, t in zip(("w", "x", "y", "mom", "var"), _training(case, seed)):
            st[k] = t.float()
        st["grad"] = torch.zeros_like(st["w"])
        st["loss"] = torch.zeros(1, dtype=torch.float32, device="cuda")
        st["step"] = 100
    return st


def _query(case, seed):
    n = case["rows"] * case["cols"]
    if case["amps"] == 1 << n:
        return torch.arange(1 << n, dtype=torch.int64, device="cuda")
    return _bits(_dev(seed + 1), n, case["amps"])


def _fsim():
    c, s = math.cos(math.pi / 2), math.sin(math.pi / 2)
    return np.array([[1, 0, 0, 0], [0, c, -1j * s, 0], [0, -1j * s, c, 0],
                     [0, 0, 0, np.exp(-1j * math.pi / 6)]], dtype=np.complex128)


def _training(case, seed):
    """Weights, spectrum features, targets and Adam moments in mid-training
    (float32 values held in float64)."""
    g = _dev(seed)
    b = case["batch"]
    shapes = [(128, 66), (128, 128), (32, 128)]
    parts = []
    for o, i in shapes:
        parts.append(torch.randn(o * i, dtype=torch.float64, device="cuda", generator=g) * math.sqrt(2.0 / i))
        parts.append(torch.randn(o, dtype=torch.float64, device="cuda", generator=g) * 0.05)
    w = torch.cat(parts)
    x = torch.rand(b, 66, dtype=torch.float64, device="cuda", generator=g)
    x[:, :64] = x[:, :64] ** 8
    x[:, :64] /= x[:, :64].sum(dim=1, keepdim=True)
    y = -12.0 * torch.rand(b, 32, dtype=torch.float64, device="cuda", generator=g).cumsum(dim=1) / 20.0
    var = 1e-3 * torch.rand(w.numel(), dtype=torch.float64, device="cuda", generator=g) + 1e-4
    mom = 0.3 * torch.randn(w.numel(), dtype=torch.float64, device="cuda", generator=g) * var.sqrt()
    return [t.float().double() for t in (w, x, y, mom, var)]


# -------------------------------------------------------------------- pass
def _fixed_phase(u):
    """Singular vectors are defined up to a phase: the first entry of each
    (rows of u) is made real and positive."""
    p = u[:, :1]
    return u * (p.conj() / p.abs())


def run(state):
    kind = state["kind"]
    case = state["case"]
    if kind == "state":
        s = rcs.State.build(state["circuit"], case["chi"], case["eps"])
        s.sample(state["bits"], state["log2p"], seed=state["seed"])
        s.amplitudes(state["query"], state["amps"])
        xeb, err = rcs.xeb_log2(state["n"], state["log2p"])
        return dict(amps=state["amps"], bits=state["bits"], log2p=state["log2p"], xeb=xeb, xeb_err=err,
                    log_fidelity=s.info().log_fidelity_est)
    if kind == "svd":
        state["x"].copy_(state["m"])
        rcs.svd_jacobi(state["x"], state["s"], state["u"])
        return dict(s=state["s"], u=_fixed_phase(state["u"]))
    if kind == "svd_f32":
        rcs.svd_jacobi_f32(state["m"], state["s"], state["u"])
        k = case["cnt"] // 2
        uk = state["u"][:k]                                            # kept columns, rows of uk
        cut = torch.matmul(torch.matmul(state["m"], uk.conj().T), uk)  # M^T -> (U_k U_k^H M)^T
        return dict(s=state["s"].float(), cut=cut.to(torch.complex64))
    if kind == "qr":
        rcs.cholqr(state["m"], state["u"], state["r"])
        return dict(q=state["u"], r=state["r"])
    if kind == "two_site":
        rcs.two_site(state["a"], state["b"], state["gate"], state["out"], precision=case["precision"])
        return state["out"]
    if kind == "sample":
        state["state"].sample(state["bits"], state["log2p"], seed=state["seed"])
        return dict(bits=state["bits"], log2p=state["log2p"])
    if kind == "sample_batch":
        rcs.sample_batch(state["states"], case["shots"], state["seed"], state["bits"], state["log2p"])
        return dict(bits=state["bits"], log2p=state["log2p"])
    if kind == "dense":
        rcs.dense_simulate(state["circuit"], state["psi"])
        rcs.dense_gather(state["psi"], state["n"], state["bits"], state["p"])
        xeb, err = rcs.xeb(state["n"], state["p"])
        return dict(psi=state["psi"], p=state["p"], xeb=xeb, xeb_err=err)
    rcs.mlp_backward(state["w"], state["x"], state["y"], state["grad"], state["loss"])
    rcs.mlp_adam(state["w"], state["grad"], state["mom"], state["var"], state["step"])
    state["step"] += 1
    return dict(w=state["w"], grad=state["grad"], loss=state["loss"], mom=state["mom"], var=state["var"])


# -------------------------------------------------------------------- work
def _svd_flops(a, b):
    m, n = max(a, b), min(a, b)
    return 4.0 * (14.0 * m * n * n + 8.0 * n ** 3)     # thin SVD, Golub & Van Loan, complex = 4 real


def _sample_work(dims, shots):
    fl = by = 0.0
    for k in range(len(dims) - 1):
        fl += 8.0 * 1.5 * shots * dims[k] * dims[k + 1]
        by += 32.0 * dims[k] * dims[k + 1]
    return fl, by + 16.0 * shots


def work(case):
    kind = case["kind"]
    if kind == "state":
        n = case["rows"] * case["cols"]
        c = rcs.Circuit(case["rows"], case["cols"], case["cycles"], seed=1, network=case["network"])
        _, ops = c.schedule()
        d, cap = [1] * (n + 1), _bond_dims(n, case["chi"])
        fl = by = 0.0
        for o, i, _gate, _cycle in ops:
            if o == 0:
                by += sum(64.0 * d[k] * d[k + 1] for k in range(n))
                continue
            dl, dm, dr = d[i], d[i + 1], d[i + 2]
            fl += 32.0 * dl * dm * dr + _svd_flops(2 * dl, 2 * dr)
            k = min(2 * dl, 2 * dr, 4 * dm, cap[i + 1])
            by += 32.0 * (dl * dm + dm * dr + dl * k + k * dr)
            d[i + 1] = k
        f2, b2 = _sample_work(d, case["shots"])
        fl += f2 + 8.0 * case["amps"] * sum(d[k] * d[k + 1] for k in range(n))
        return dict(bytes=by + b2 + 24.0 * case["amps"], flops=fl)
    if kind in ("svd", "svd_f32"):
        ln, n = case["len"], case["cnt"]
        return dict(bytes=32.0 * ln * n + 8.0 * n, flops=_svd_flops(ln, n))
    if kind == "qr":
        ln, n = case["len"], case["cnt"]
        return dict(bytes=32.0 * ln * n + 16.0 * n * n, flops=2 * 4.0 * (2.0 * ln * n * n - 2.0 * n ** 3 / 3.0))
    if kind == "two_site":
        dl, dm, dr = case["dl"], case["dm"], case["dr"]
        return dict(bytes=32.0 * (dl * dm + dm * dr) + 64.0 * dl * dr, flops=32.0 * dl * dm * dr)
    if kind == "sample":
        fl, by = _sample_work(_bond_dims(case["n"], case["chi"]), case["shots"])
        return dict(bytes=by, flops=fl)
    if kind == "sample_batch":
        fl = by = 0.0
        for n, chi in _batch_states(case):
            f, b = _sample_work(_bond_dims(n, chi), case["shots"])
            fl, by = fl + f, by + b
        return dict(bytes=by, flops=fl)
    if kind == "dense":
        n = case["rows"] * case["cols"]
        size = 16.0 * (1 << n)
        gates = (case["cycles"] + 1) * n * 14.0 + case["cycles"] * n / 2 * 30.0
        # a vector larger than the caches is read and written once per cycle
        return dict(bytes=2 * size * case["cycles"] + 32.0 * case["shots"], flops=gates * (1 << n))
    b, p = case["batch"], 66 * 128 + 128 * 128 + 128 * 32
    return dict(bytes=4.0 * (8 * rcs.MLP_PARAMS + b * 98), flops=6.0 * b * p)


# ------------------------------------------------------------------- exact
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on uint64 arrays of 32-bit words."""
    mask = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) for v in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _gates(n, cycles, seed):
    q = np.arange(n, dtype=np.uint64)
    layers, prev = [], None
    for t in range(cycles + 1):
        x = _philox(q, np.uint64(t), np.uint64(0), np.uint64(0), seed)[0]
        if prev is None:
            prev = ((3 * x) >> np.uint64(32)).astype(int)
        else:
            others = np.array([[1, 2], [0, 2], [0, 1]])
            prev = others[prev, (x >> np.uint64(31)).astype(int)]
        layers.append(prev)
    return layers


def _couplers(rows, cols, letter):
    w, h = min(rows, cols), max(rows, cols)
    if letter in "AB":
        return [(r * w + c, r * w + c + 1) for r in range(h) for c in range("AB".index(letter), w - 1, 2)]
    return [(r * w + c, (r + 1) * w + c) for r in range("CD".index(letter), h - 1, 2) for c in range(w)]


def _dense(case, seed):
    n = case["rows"] * case["cols"]
    r2 = math.sqrt(2.0)
    one = [0.5 * np.array(m, dtype=np.complex128) for m in (
        [[1 + 1j, 1 - 1j], [1 - 1j, 1 + 1j]], [[1 + 1j, -1 - 1j], [1 + 1j, 1 + 1j]],
        [[1 + 1j, -1j * r2], [r2, 1 + 1j]])]
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1.0

    def layer(gates):
        for q in range(n):
            v = psi.view(1 << (n - q - 1), 2, 1 << q)
            u = one[gates[q]]
            a, b = v[:, 0].clone(), v[:, 1].clone()
            v[:, 0] = complex(u[0, 0]) * a + complex(u[0, 1]) * b
            v[:, 1] = complex(u[1, 0]) * a + complex(u[1, 1]) * b

    f = _fsim()
    gates = _gates(n, case["cycles"], seed & 0xFFFFFFFFFFFFFFFF)
    for t in range(case["cycles"]):
        layer(gates[t])
        for lo, hi in _couplers(case["rows"], case["cols"], PATTERN[t % 8]):
            v = psi.view(1 << (n - hi - 1), 2, 1 << (hi - lo - 1), 2, 1 << lo)   # fSim is symmetric in its qubits
            a, b = v[:, 0, :, 1].clone(), v[:, 1, :, 0].clone()
            v[:, 0, :, 1] = complex(f[1, 1]) * a + complex(f[1, 2]) * b
            v[:, 1, :, 0] = complex(f[2, 1]) * a + complex(f[2, 2]) * b
            v[:, 1, :, 1] *= complex(f[3, 3])
    layer(gates[case["cycles"]])
    return psi


def _xeb(n, p):
    v = p * 2.0 ** n
    return float(v.mean() - 1.0), float(v.std() / math.sqrt(v.numel()))


def _chain(tensors, shots, seed):
    """log2 probabilities of the shots the chain rule draws in 64 bits."""
    v = torch.ones(shots, 1, dtype=torch.complex128, device="cuda")
    i = np.arange(shots, dtype=np.uint64)
    p = None
    for k, a in enumerate(tensors):
        w = _philox(i, np.uint64(0), np.uint64(k >> 1), np.uint64(2), seed & 0xFFFFFFFFFFFFFFFF)
        lo, hi = (w[2], w[3]) if k & 1 else (w[0], w[1])
        u = (((hi << np.uint64(32)) | lo) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
        u = torch.from_numpy(u).cuda()
        w0, w1 = torch.matmul(v, a[:, 0].contiguous()), torch.matmul(v, a[:, 1].contiguous())
        p0, p1 = (w0.abs() ** 2).sum(dim=1), (w1.abs() ** 2).sum(dim=1)
        one = u * (p0 + p1) >= p0
        v = torch.where(one[:, None], w1, w0)
        p = torch.where(one, p1, p0)
    return torch.log2(p)


def exact(case, seed):
    kind = case["kind"]
    if kind == "state":
        n = case["rows"] * case["cols"]
        dims = _bond_dims(n, case["chi"])
        if case["eps"] > 0.0 or max(dims) < 1 << (n // 2):
            return None                                  # truncated: the method's own state
        amps = _dense(case, seed)[_query(case, seed)]
        return dict(amps=amps, bits=None, log2p=None, xeb=None, xeb_err=None, log_fidelity=None)
    if kind == "svd":
        u, s, _ = _planted(case, seed)
        return dict(s=s, u=_fixed_phase(u.T.contiguous()))
    if kind == "svd_f32":
        u, s, v = _planted(case, seed)
        k = case["cnt"] // 2
        return dict(s=s, cut=torch.matmul(u[:, :k] * s[:k], v[:, :k].conj().T).T.contiguous())
    if kind == "qr":
        q, r = torch.linalg.qr(_planted_columns(case, seed).T.contiguous().cpu())
        p = torch.diagonal(r) / torch.diagonal(r).abs()
        return dict(q=(q * p).T.contiguous(), r=(r * p.conj()[:, None]).T.contiguous())
    if kind == "two_site":
        st = prepare(case, seed)
        g = torch.from_numpy(st["gate"]).cuda().reshape(4, 4)
        t = [torch.matmul(st["a"][:, s1].contiguous(), st["b"][:, s2].contiguous()) for s1 in (0, 1) for s2 in (0, 1)]
        m = [sum(g[o, q] * t[q] for q in range(4)) for o in range(4)]
        return torch.cat([torch.cat([m[0], m[1]], dim=1), torch.cat([m[2], m[3]], dim=1)], dim=0).T.contiguous()
    if kind == "sample":
        return dict(bits=None, log2p=_chain(_right_canonical(_dev(seed), case["n"], case["chi"])[1], case["shots"], seed))
    if kind == "sample_batch":
        g = _dev(seed)
        rows = [_chain(_right_canonical(g, n, chi)[1], case["shots"], seed) for n, chi in _batch_states(case)]
        return dict(bits=None, log2p=torch.stack(rows))
    if kind == "dense":
        n = case["rows"] * case["cols"]
        psi = _dense(case, seed)
        p = psi[_bits(_dev(seed), n, case["shots"])].abs() ** 2
        xeb, err = _xeb(n, p)
        return dict(psi=psi, p=p, xeb=xeb, xeb_err=err)
    w, x, y, mom, var = _training(case, seed)
    w.requires_grad_(True)
    o, h = 0, x
    for i, (fo, fi) in enumerate([(128, 66), (128, 128), (32, 128)]):
        h = torch.matmul(h, w[o:o + fo * fi].reshape(fo, fi).T) + w[o + fo * fi:o + fo * fi + fo]
        o += fo * fi + fo
        h = torch.relu(h) if i < 2 else h
    loss = ((h - y) ** 2).mean()
    grad, = torch.autograd.grad(loss, w)
    mom, var = 0.9 * mom + 0.1 * grad, 0.999 * var + 0.001 * grad ** 2
    upd = (mom / (1 - 0.9 ** 100)) / ((var / (1 - 0.999 ** 100)).sqrt() + 1e-8)
    return dict(w=w.detach() - 1e-3 * upd, grad=grad, loss=loss.detach().reshape(1), mom=mom, var=var)
