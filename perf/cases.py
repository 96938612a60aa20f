"""The work whose speed counts: what users of the library have it do, through its public Python
binding, over the sizes, precisions and options that the repository's workloads, tests and
benchmark use.

`listed()` gives the named cases, `draw()` more of the same ranges; `prepare()` makes what a
user's program holds before the call (host arrays, and the solver with its data, prior and step
sizes), `run()` is one pass, `work()` what a pass cannot do without, and `exact()` the same result
in 64 bits by plain torch and numpy (a dense wavelet transform, a gather / scatter NUFFT), which
shares no code with the library.

The library runs on the HIP runtime it was built for and refuses the one that torch bundles, so a
process that has loaded torch cannot call it.  This module therefore starts itself once as a
plain worker process without torch (`serve()`), keeps every solver there, and hands arrays over
in shared memory; a pass is one request to that worker, answered when its results are written.
"""
import contextlib
import math
import mmap
import os
import pickle
import subprocess
import sys

import numpy as np

if __name__ != "__main__":
    import torch


# ---------------------------------------------------------------------------------------------
# cases

def _solve(name, n, M, taps=8, levels=4, fp64=False, cover="mixed", isnr=20.0, stages="100,100,100",
           mode="constrained", mueller=False):
    """Algorithm 2 from a zero state: the initialisation stage, then the reweighted stages."""
    return {"name": name, "kind": "solve", "n": n, "M": M, "taps": taps, "levels": levels, "fp64": fp64,
            "cover": cover, "isnr": isnr, "stages": stages, "mode": mode, "mueller": mueller}


def listed():
    return [
        # the smallest whole reconstruction (the 32 x 32 three-blob problem, six-tap kernel, FP64)
        _solve("blobs32_fp64", 32, 600, taps=6, levels=3, fp64=True, cover="gauss", isnr=30.0),
        # a small request of the served mix, an odd number of rows
        _solve("small64", 64, 1511, isnr=25.0),
        # sparse VLBI coverage on Earth-rotation arcs, both precisions
        _solve("ring128", 128, 12000, cover="arcs"),
        _solve("ring128_fp64", 128, 12000, cover="arcs", fp64=True, stages="60,60,60"),
        # the benchmark's image size and row count on its full schedule
        _solve("ring256", 256, 200000),
        # the large request of the served mix (fewer iterations: the rate is what counts)
        _solve("large512", 512, 1000000, stages="20,20,20"),
        # calibrated data: known Mueller matrices per row, the problem without the polarization
        # constraint
        _solve("mueller128", 128, 20001, mode="unconstrained", mueller=True),
        # independent solves of uneven sizes advanced together
        {"name": "batch16", "kind": "batch", "count": 16, "n_lo": 64, "n_hi": 256, "m_lo": 1000, "m_hi": 100000,
         "stages": "24,24,24"},
        # Algorithm 3, the l1 + TV prior with the polarization constraint
        {"name": "tv256", "kind": "tv", "n": 256, "M": 200000, "taps": 8, "fp64": False, "cover": "mixed",
         "isnr": 20.0, "iters": 100, "l1": True, "mode": "constrained"},
        # a solve that ends by the stopping test on the device
        {"name": "adaptive64_fp64", "kind": "adaptive", "n": 64, "M": 4099, "taps": 8, "levels": 4, "fp64": True,
         "cover": "mixed", "isnr": 25.0, "iters": 240, "check": 20},
        # a request from its host arrays to its image, everything set up anew
        {"name": "request128", "kind": "request", "n": 128, "M": 20000, "taps": 8, "levels": 4, "fp64": False,
         "cover": "mixed", "isnr": 25.0, "stages": "50,50,50", "mode": "constrained", "mueller": False},
        # the operators on their own, from and to host arrays
        {"name": "operators256", "kind": "operators", "n": 256, "M": 100003, "taps": 8, "levels": 4, "fp64": False,
         "cover": "mixed", "isnr": 20.0},
    ]


def draw(rng):
    """One more case: kinds as in the list, sides over the powers of two, rows log-uniform."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["solve"] * 6 + ["batch", "tv", "adaptive", "request", "operators"])
    fp64 = rng.random() < 0.3
    cover = rng.choice(["mixed", "mixed", "gauss", "arcs"])
    isnr = round(rng.uniform(15.0, 35.0), 2)
    if kind == "batch":
        return {"kind": "batch", "count": rng.randrange(3, 17), "n_lo": rng.choice([32, 64]), "n_hi": rng.choice([64, 128, 256]),
                "m_lo": log_int(300, 3000), "m_hi": log_int(5000, 100000), "stages": "%d,%d" % (rng.randrange(8, 30), rng.randrange(8, 41))}
    n = rng.choice([32, 64, 128, 256] if fp64 or kind != "solve" else [32, 64, 128, 256, 256, 512])
    M = log_int(500, min(15 * n * n // 8, 900000))
    taps = rng.choice([8, 8, 8, 6, 4])
    levels = rng.randrange(2, min(5, int(math.log2(n)) - 2) + 1)
    case = {"kind": kind, "n": n, "M": M, "taps": taps, "levels": levels, "fp64": fp64, "cover": cover, "isnr": isnr}
    most = 20 if n == 512 else 40 if n == 256 else 100
    if kind in ("solve", "request"):
        cycles = rng.randrange(1, 3)
        case["stages"] = ",".join(str(rng.randrange(most // 2, most + 1)) for _ in range(cycles + 1))
        case["mode"] = rng.choice(["constrained", "constrained", "unconstrained"])
        case["mueller"] = kind == "solve" and M < 100000 and rng.random() < 0.2
    elif kind == "tv":
        case.update(iters=rng.randrange(most // 2, most + 1), l1=rng.random() < 0.5,
                    mode=rng.choice(["constrained", "unconstrained"]))
    elif kind == "adaptive":
        check = rng.randrange(5, 26)
        case.update(iters=check * rng.randrange(2, 5), check=check)
    return case


def _members(case):
    """The solves of a batch: sides over the powers of two and rows log-uniform, spread evenly."""
    sides = [s for s in (32, 64, 128, 256) if case["n_lo"] <= s <= max(case["n_lo"], case["n_hi"])]
    out = []
    for i in range(case["count"]):
        t = (i * 0.6180339887498949) % 1.0
        M = int(round(case["m_lo"] * (case["m_hi"] / case["m_lo"]) ** t))
        out.append({"kind": "solve", "n": sides[i % len(sides)], "M": M, "taps": 8, "levels": 4, "fp64": False,
                    "cover": "mixed", "isnr": 15.0 + 20.0 * ((i * 0.7548776662466927) % 1.0),
                    "stages": case["stages"], "mode": "constrained", "mueller": False})
    return out


def _stages(case):
    return [int(s) for s in case["stages"].split(",")]


def work(case):
    """Bytes and operations of one pass: per iteration the state read and written once (rows Y and
    B with their geometry, coefficients and thresholds, images) and the arithmetic of the taps,
    FFTs and filters; the FFT grid and other intermediates are not counted."""
    if case["kind"] == "batch":
        each = [work(m) for m in _members(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    n, M, T, R = case["n"], case["M"], case["taps"], 8 if case["fp64"] else 4
    N, K = n * n, 2 * n
    fft = 4 * 5.0 * K * K * math.log2(K * K)
    taps = 4 * 2 * 2.0 * M * T * T
    bases = 8 * (8.0 / 3.0) * sum(2 * p for p in range(1, 9)) * N / 8 * 4
    if case["kind"] == "operators":
        return {"bytes": (8 * M * 2 + 4 * N * 4 + 2 * 36 * N) * 8.0, "flops": 2 * (fft + taps + bases)}
    rows = M * (3 * 8 * R + 4 + 2 * R)
    if case["kind"] == "tv":
        blocks = (3 if case["l1"] else 2) * 2
        per = {"bytes": rows - 16 * R * M + N * R * (4 * blocks + 24), "flops": 2 * (fft + taps) + 60.0 * N}
        its = case["iters"]
    else:
        per = {"bytes": rows + N * R * (3 * 36 + 24), "flops": 2 * (fft + taps + bases)}
        its = case["iters"] if case["kind"] == "adaptive" else sum(_stages(case))
    if case.get("mueller"):
        per["bytes"] += M * 32 * R
    if case["kind"] == "request":
        its += 40          # the power iteration that fixes the step sizes
    return {"bytes": float(per["bytes"] * its), "flops": float(per["flops"] * its)}


# ---------------------------------------------------------------------------------------------
# inputs: uv coverage, visibilities with noise, and the l2 bound, made from the seed alone

def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _inputs(case, seed):
    """Host arrays of one problem: uv (M x 2), Y (M x 4 complex), eps, truth (N x 4), and the
    Mueller matrices or None."""
    from paper_1801_02417_amd import workloads as wk
    n, M = case["n"], case["M"]
    rng = np.random.default_rng([2417, seed, n, M])
    I = wk.blobs_image(rng, n) if n <= 32 else wk.ring_jet_image(rng, n)
    if n >= 256:
        I = wk.add_knots(rng, I, 20)
    truth = wk.add_polarisation(rng, I)
    if case["cover"] == "gauss":
        uv = wk.gaussian_uv(rng, M)
    elif case["cover"] == "arcs":
        uv = wk.arc_uv(rng, M)
    else:
        uv = np.concatenate([wk.gaussian_uv(rng, M // 2), wk.arc_uv(rng, M - M // 2)], axis=0)
    noise = wk.unit_noise(rng, M)
    mueller = wk.station_mueller(rng, M) if case.get("mueller") else None
    phi = _Phi(n, uv, case["taps"], mueller)
    y0 = phi.forward(torch.from_numpy(np.ascontiguousarray(truth.transpose(2, 0, 1))).to(_device())).cpu().numpy()
    sigma = float(np.linalg.norm(y0)) / math.sqrt(4 * M) * 10.0 ** (-case["isnr"] / 20.0)
    eps = math.sqrt((8 * M + 2 * math.sqrt(2 * 8 * M)) * sigma * sigma / 2.0)
    out = {"uv": uv, "Y": y0 + sigma * noise, "eps": eps, "truth": truth.reshape(n * n, 4), "mueller": mueller}
    if case["kind"] not in ("request", "operators"):
        # the constants that such a program keeps with its solver: ||phi||^2 with a 1 % margin (a
        # fixed number of Lanczos steps, so that the reference in 64 bits takes the same value),
        # and gamma
        out["norm"] = 1.01 * phi.norm_sq(20)
        if case["kind"] != "tv":
            peak = _Sara(n, case["levels"]).adjoint(phi.adjoint(torch.from_numpy(out["Y"]).to(_device()))).abs().max()
            out["gamma"] = 1e-3 * float(peak) / out["norm"]
    return out


def _tv_weights(case):
    return [4e-3, 2e-3, 2e-3, 1e-3], ([2e-3, 1e-3, 1e-3, 5e-4] if case["l1"] else None)


# ---------------------------------------------------------------------------------------------
# the cases in the worker

class State:
    """A prepared case: the worker's handle of it."""

    def __init__(self, client, key):
        self.client, self.key = client, key

    def __del__(self):
        with contextlib.suppress(Exception):
            self.client.ask(("drop", self.key), {})


def prepare(case, seed):
    client = _client()
    if case["kind"] == "batch":
        arrays = {}
        for i, m in enumerate(_members(case)):
            arrays.update({"%d.%s" % (i, k): v for k, v in _inputs(m, seed + 1000 * i).items() if v is not None})
    else:
        arrays = {k: v for k, v in _inputs(case, seed).items() if v is not None}
    return State(client, client.ask(("prepare", case), arrays)["key"])


def run(state):
    return state.client.ask(("run", state.key), {})


class _Case:
    """A case in the worker: its solvers, and what a pass does with them."""

    def __init__(self, P, case, arrays):
        self.P, self.case = P, case
        self.real = np.float64 if case.get("fp64") else np.float32
        self.arrays = arrays
        if case["kind"] == "batch":
            self.members = _members(case)
            self.solvers = [self.solver(m, {k.split(".", 1)[1]: v for k, v in arrays.items() if k.startswith("%d." % i)})
                            for i, m in enumerate(self.members)]
        elif case["kind"] == "operators":
            self.solvers = [self.open(case, arrays)]
            self.solvers[0].set_prior(case["levels"], 1.0)
            rows = np.ascontiguousarray(arrays["Y"])
            self.coef = np.random.default_rng(5).standard_normal((9 * case["n"] ** 2, 4)) * float(np.abs(rows).mean())
        elif case["kind"] == "request":
            self.solvers = []
        else:
            self.solvers = [self.solver(case, arrays)]

    def open(self, case, arrays):
        P = self.P
        return P.Solver(case["n"], arrays["uv"], taps=case["taps"],
                        precision=P.PSARA_FP64 if case["fp64"] else P.PSARA_FP32_MIXED)

    def solver(self, case, arrays):
        """A solver ready to iterate: data, prior, operator norm, step sizes and gamma."""
        P, s = self.P, self.open(case, arrays)
        if case.get("mueller"):
            P.psara_set_mueller(s.ctx, arrays["mueller"])
        s.set_data(arrays["Y"], float(arrays["eps"]))
        if case["kind"] == "tv":
            s.set_prior_tv(*_tv_weights(case))
        else:
            s.set_prior(case["levels"], float(arrays.get("gamma", 1.0)))
        s.opnorm()
        if "norm" in arrays:
            s.set_steps(*P.psara_step_sizes({"tv": 2 if case.get("l1") else 1}.get(case["kind"], 0), float(arrays["norm"])))
        else:
            s.set_steps()
            P.psara_set_gamma(s.ctx, P.psara_data_gamma(s.ctx, 1e-3))
        return s

    def mode(self, case):
        return self.P.PSARA_CONSTRAINED if case["mode"] == "constrained" else self.P.PSARA_UNCONSTRAINED

    def report(self, r):
        return np.array([r["residual"], r["zeta"], r["objective"]], dtype=self.real)

    def image(self, s):
        # the library holds an FP32 solve's image in 32 bits and widens it on the way out
        return s.image().astype(self.real, copy=False)

    def run(self):
        P, case = self.P, self.case
        if case["kind"] == "solve":
            s = self.solvers[0]
            s.reset()
            r = s.reweighted_solve(self.mode(case), _stages(case))
            return {"image": self.image(s), "report": self.report(r)}
        if case["kind"] == "batch":
            for s in self.solvers:
                s.reset()
            P.batch_reweighted_solve(self.solvers, P.PSARA_CONSTRAINED, _stages(case))
            return {"image%d" % i: self.image(s) for i, s in enumerate(self.solvers)}
        if case["kind"] == "tv":
            s = self.solvers[0]
            s.reset()
            r = s.solve(self.mode(case), case["iters"])
            return {"image": self.image(s), "report": self.report(r)}
        if case["kind"] == "adaptive":
            s = self.solvers[0]
            s.reset()
            its, r = s.solve_adaptive(P.PSARA_CONSTRAINED, case["iters"], case["check"], (0.5, 1e-2, 50.0))
            return {"image": self.image(s), "report": self.report(r), "iterations": np.array(its, dtype=np.int64)}
        if case["kind"] == "request":
            s = self.solver(case, self.arrays)
            r = s.reweighted_solve(self.mode(case), _stages(case))
            out = {"image": self.image(s), "report": self.report(r)}
            s.close()
            return out
        s, to = self.solvers[0], self.real
        cx = np.complex128 if case["fp64"] else np.complex64
        return {"phi": s.phi(self.arrays["truth"]).astype(cx, copy=False),
                "phi_adjoint": s.phi_adjoint(self.arrays["Y"]).astype(to, copy=False),
                "psi_adjoint": s.psi_adjoint(self.arrays["truth"]).astype(to, copy=False),
                "psi": s.psi(self.coef).astype(to, copy=False)}

    def close(self):
        for s in self.solvers:
            s.close()


# ---------------------------------------------------------------------------------------------
# the worker process: requests over pipes, arrays in one shared block

class _Block:
    """The shared memory of the two processes, grown as needed by whoever writes."""

    def __init__(self, fd):
        self.fd, self.map = fd, None

    def view(self, size):
        if self.map is None or len(self.map) < size:
            if os.fstat(self.fd).st_size < size:
                os.ftruncate(self.fd, 2 * size)
            self.map = mmap.mmap(self.fd, os.fstat(self.fd).st_size)
        return self.map

    def put(self, arrays):
        """Writes the arrays; returns {name: (dtype, shape, offset)}."""
        where, at = {}, 0
        arrays = {k: np.ascontiguousarray(v) for k, v in arrays.items()}
        for k, v in arrays.items():
            where[k] = (v.dtype.str, np.shape(v), at)
            at += (v.nbytes + 63) & ~63
        m = self.view(max(at, 4096))
        for k, v in arrays.items():
            if v.size:
                np.frombuffer(m, v.dtype, v.size, where[k][2])[:] = v.reshape(-1)
        return where

    def get(self, where):
        out = {}
        for k, (dtype, shape, at) in where.items():
            d, size = np.dtype(dtype), int(np.prod(shape, dtype=np.int64))
            out[k] = np.frombuffer(self.view(at + d.itemsize * size + 4096), d, size, at).reshape(shape).copy()
        return out


def _send(f, value):
    data = pickle.dumps(value)
    f.write(len(data).to_bytes(8, "little") + data)
    f.flush()


def _receive(f):
    head = f.read(8)
    return pickle.loads(f.read(int.from_bytes(head, "little"))) if len(head) == 8 else None


class _Client:
    def __init__(self):
        fd = os.memfd_create("perf_cases")
        root = os.getcwd()
        self.block = _Block(fd)
        self.process = subprocess.Popen([sys.executable, os.path.abspath(__file__), str(fd), root], cwd=root,
                                        stdin=subprocess.PIPE, stdout=subprocess.PIPE, pass_fds=(fd,))

    def ask(self, request, arrays):
        where = self.block.put(arrays) if arrays else {}
        try:
            _send(self.process.stdin, (request, where))
            answer = _receive(self.process.stdout)
        except BrokenPipeError:
            answer = None
        if answer is None:
            status = self.process.wait()
            print("the worker process ended (%d) at %r" % (status, request), file=sys.stderr, flush=True)
            if status < 0:      # ended by a signal, as after a GPU fault: nothing more is to run here
                os.abort()
            raise RuntimeError("the worker process ended (%d)" % status)
        error, value, where = answer
        if error:
            raise RuntimeError(error)
        return self.block.get(where) if where else value


_the_client = None


def _client():
    global _the_client
    if _the_client is None:
        _the_client = _Client()
    return _the_client


def serve(fd, root):
    """The worker: answers requests until its input ends."""
    sys.path[:0] = [root]
    from paper_1801_02417_amd import psara as P
    block, kept, next_key = _Block(fd), {}, 0
    source, sink = sys.stdin.buffer, sys.stdout.buffer
    while (asked := _receive(source)) is not None:
        (verb, what), where = asked
        try:
            if verb == "prepare":
                next_key += 1
                kept[next_key] = _Case(P, what, block.get(where))
                answer = (None, {"key": next_key}, {})
            elif verb == "run":
                answer = (None, None, block.put(kept[what].run()))
            else:
                kept.pop(what).close()
                answer = (None, None, {})
        except Exception as e:
            answer = ("%s: %s" % (type(e).__name__, e), None, {})
        _send(sink, answer)


# ---------------------------------------------------------------------------------------------
# the method in 64 bits: plain torch on dense transforms, images as 4 x n x n

class _Phi:
    """Kaiser-Bessel NUFFT on a twice oversampled grid with the Stokes-to-brightness mixing."""
    CHUNK = 1 << 17

    def __init__(self, n, uv, T, mueller=None):
        dev = _device()
        self.n, self.K, self.T = n, 2 * n, T
        K = self.K
        beta = math.pi * math.sqrt((T / 2) ** 2 * 2.25 - 0.8)
        i0b = float(torch.special.i0(torch.tensor(beta, dtype=torch.float64)))
        t = torch.from_numpy(np.ascontiguousarray(uv)).to(dev) * (K / (2.0 * math.pi))
        first = torch.ceil(t - T / 2.0)
        taps = torch.arange(T, device=dev)
        at = t[:, :, None] - (first[:, :, None] + taps)                     # M x 2 x T
        inside = (1.0 - (2.0 * at / T) ** 2).clamp(min=0.0)
        psi = torch.where((2.0 * at / T).abs() <= 1.0, torch.special.i0(beta * inside.sqrt()) / i0b, torch.zeros_like(at))
        self.w1, self.w2 = psi[:, 0], psi[:, 1]
        where = (first.long()[:, :, None] + taps) % K
        self.c1, self.c2 = where[:, 0], where[:, 1]
        nu = (torch.arange(n, device=dev, dtype=torch.float64) - n // 2) / K
        z2 = beta * beta - (math.pi * T * nu) ** 2
        z = torch.sqrt(z2.to(torch.complex128))
        hat = (T / i0b) * (torch.sinh(z) / z).real
        self.scale = 1.0 / (hat[:, None] * hat[None, :])
        self.pos = (torch.arange(n, device=dev) - n // 2) % K
        mix = torch.tensor([[1, 0, 0, 1], [1, 0, 0, -1], [0, 1, 1, 0], [0, 1j, -1j, 0]], dtype=torch.complex128, device=dev)
        if mueller is not None:
            d = torch.from_numpy(np.ascontiguousarray(mueller)).to(dev)
            mix = torch.matmul(mix, d.transpose(1, 2).contiguous())       # M x 4 x 4
        self.mix = mix

    def _parts(self):
        for a in range(0, self.w1.shape[0], self.CHUNK):
            b = slice(a, a + self.CHUNK)
            cells = (self.c1[b][:, :, None] * self.K + self.c2[b][:, None, :]).reshape(-1)
            yield b, cells, (self.w1[b][:, :, None] * self.w2[b][:, None, :]).reshape(-1, 1)

    def stokes(self, S):
        """Phi S per Stokes map: M x 4 complex."""
        K = self.K
        grid = torch.zeros(4, K, K, dtype=torch.complex128, device=S.device)
        grid[:, self.pos[:, None], self.pos[None, :]] = (S * self.scale).to(torch.complex128)
        f = torch.view_as_real(torch.fft.fft2(grid).permute(1, 2, 0).contiguous()).reshape(K * K, 8)
        out = [(f[cells] * w).reshape(-1, self.T * self.T, 8).sum(1) for _, cells, w in self._parts()]
        return torch.view_as_complex(torch.cat(out).reshape(-1, 4, 2))

    def stokes_adjoint(self, V):
        """Re Phi^dagger V: 4 x n x n."""
        K = self.K
        v = torch.view_as_real(V.contiguous()).reshape(-1, 8)
        acc = torch.zeros(K * K, 8, dtype=torch.float64, device=V.device)
        for b, cells, w in self._parts():
            acc.index_add_(0, cells, w * v[b].repeat_interleave(self.T * self.T, dim=0))
        grid = torch.view_as_complex(acc.reshape(K, K, 4, 2)).permute(2, 0, 1)
        x = torch.fft.ifft2(grid) * (K * K)
        return x[:, self.pos[:, None], self.pos[None, :]].real * self.scale

    def forward(self, S):
        v = self.stokes(S)
        return v @ self.mix if self.mix.dim() == 2 else (v[:, :, None] * self.mix).sum(1)

    def adjoint(self, B):
        m = self.mix.conj()
        return self.stokes_adjoint(B @ m.transpose(0, 1) if m.dim() == 2 else (B[:, None, :] * m).sum(2))

    def norm_sq(self, steps):
        """The largest eigenvalue of S -> Re phi^dagger phi S by Lanczos with full
        reorthogonalisation."""
        dim = 4 * self.n * self.n
        gen = torch.Generator().manual_seed(7)
        q = torch.randn(dim, generator=gen, dtype=torch.float64).to(self.w1.device)
        Q, a, b = [q / q.norm()], [], []
        for _ in range(min(steps, dim - 1)):
            w = self.adjoint(self.forward(Q[-1].reshape(4, self.n, self.n))).reshape(-1)
            a.append(float(w @ Q[-1]))
            basis = torch.stack(Q)
            for _ in range(2):
                w = w - (basis @ w) @ basis
            b.append(float(w.norm()))
            Q.append(w / w.norm())
        return float(np.linalg.eigvalsh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))[-1])


class _Sara:
    """(1/3) [Dirac, Db1 .. Db8], periodised 2-D transforms as dense matrices."""

    def __init__(self, n, levels):
        self.n, self.levels, self.W = n, levels, []
        filters = [self.lowpass(p) for p in range(1, 9)]
        for lev in range(levels):
            m = n >> lev
            W = np.zeros((8, m, m))
            k = np.arange(m // 2)
            for b, h in enumerate(filters):
                for j in range(len(h)):
                    np.add.at(W[b], (k, (2 * k + j) % m), h[j])
                    np.add.at(W[b], (m // 2 + k, (2 * k + j) % m), (-1) ** j * h[len(h) - 1 - j])
            self.W.append(torch.from_numpy(W).to(_device())[:, None])

    @staticmethod
    def lowpass(p):
        """Db_p by spectral factorisation, the zeros inside the unit circle."""
        zeros = []
        for y in np.roots([math.comb(p - 1 + k, k) for k in range(p)][::-1]) if p > 1 else []:
            pair = np.roots([1.0, 4.0 * y - 2.0, 1.0])
            zeros.append(pair[np.argmin(np.abs(pair))])
        h = np.real(np.polymul(np.poly(zeros) if zeros else [1.0], [math.comb(p, k) for k in range(p + 1)]))
        return h * (math.sqrt(2.0) / h.sum())

    def adjoint(self, S):
        """Psi^dagger S: 9 x 4 x n x n."""
        c = S.expand(8, 4, self.n, self.n).clone()
        for lev, W in enumerate(self.W):
            m = self.n >> lev
            c[..., :m, :m] = W @ c[..., :m, :m].contiguous() @ W.transpose(2, 3).contiguous()
        return torch.cat([S[None], c]) / 3.0

    def forward(self, A):
        c = A[1:].clone()
        for lev in reversed(range(self.levels)):
            m, W = self.n >> lev, self.W[lev]
            c[..., :m, :m] = W.transpose(2, 3).contiguous() @ c[..., :m, :m].contiguous() @ W
        return (A[0] + c.sum(0)) / 3.0


class _Tv:
    """[identity,] forward differences along both axes, zero at the last row and column."""

    def __init__(self, l1):
        self.l1 = l1

    def adjoint(self, S):
        d1, d2 = torch.zeros_like(S), torch.zeros_like(S)
        d1[:, :-1] = S[:, 1:] - S[:, :-1]
        d2[:, :, :-1] = S[:, :, 1:] - S[:, :, :-1]
        return torch.stack(([S] if self.l1 else []) + [d1, d2])

    def forward(self, A):
        d1, d2 = A[-2], A[-1]
        out = torch.zeros_like(d1)
        out[:, 1:] += d1[:, :-1]
        out[:, :-1] -= d1[:, :-1]
        out[:, :, 1:] += d2[:, :, :-1]
        out[:, :, :-1] -= d2[:, :, :-1]
        return out + A[0] if self.l1 else out


class _Reference:
    """Algorithms 1 to 3 of the paper in 64 bits."""

    def __init__(self, case, inputs):
        dev, n = _device(), case["n"]
        self.case = case
        self.phi = _Phi(n, inputs["uv"], case["taps"], inputs["mueller"])
        self.Y, self.eps = torch.from_numpy(inputs["Y"]).to(dev), inputs["eps"]
        self.norm = inputs["norm"] if "norm" in inputs else self.phi.norm_sq(64)
        zero = torch.zeros(4, n, n, dtype=torch.float64, device=dev)
        if case["kind"] == "tv":
            tw, lw = _tv_weights(case)
            self.psi = _Tv(case["l1"])
            self.tw = torch.tensor(tw, dtype=torch.float64, device=dev)[:, None, None]
            self.lw = torch.tensor(lw, dtype=torch.float64, device=dev)[:, None, None] if lw else None
            p2 = 9.0 if case["l1"] else 8.0
            self.rho = (1.0 / p2, 1.0, 1.0)
            self.tau = 0.99 / (self.norm / 4.0 + 2.0)
            y = self.Y      # Y L^{-1}
            self.Y = torch.stack([(y[:, 0] + y[:, 3]) / 2, (y[:, 0] - y[:, 3]) / 2, (y[:, 1] + y[:, 2]) / 2,
                                  (y[:, 1] - y[:, 2]) / 2j], dim=1)
        else:
            self.psi = _Sara(n, case["levels"])
            self.rho = (1.0, 1.0 / self.norm, 1.0)
            self.tau = 0.99 / 3.0
            self.gamma = inputs.get("gamma")
            if self.gamma is None:
                self.gamma = 1e-3 * float(self.psi.adjoint(self.phi.adjoint(self.Y)).abs().max()) / self.norm
        self.S, self.C, self.old = zero, zero, zero
        self.Z = self.D = zero[:2]
        self.A = torch.zeros_like(self.psi.adjoint(zero))
        self.B = torch.zeros_like(self.Y)
        self.W = torch.ones_like(self.A)

    def iterate(self, count, mode):
        r1, r2, r3 = self.rho
        tv, prior, cone = self.case["kind"] == "tv", mode != "init", mode == "constrained"
        for _ in range(count):
            S, tau = self.S, self.tau
            g = self.phi.stokes_adjoint(self.phi.stokes(S) - self.Y) if tv else self.phi.adjoint(self.B)
            if prior:
                g = g + self.psi.forward(self.A)
            if cone:
                g = g + self.C
            S1 = S - tau * g
            if not cone:
                S1[0].clamp_(min=0.0)
            X = 2.0 * S1 - S
            if prior and tv:
                a = self.A + r1 * self.psi.adjoint(X)
                pair = a[-2:].pow(2).sum(0).sqrt()
                a[-2:] *= torch.where(pair > self.tw, self.tw / pair.clamp(min=1e-300), torch.ones_like(pair))
                if self.lw is not None:
                    a[0] = torch.minimum(torch.maximum(a[0], -self.lw), self.lw)
                self.A = a
            elif prior:
                t = self.gamma * self.W
                self.A = torch.minimum(torch.maximum(self.A + r1 * self.psi.adjoint(X), -t), t)
            if not tv:
                v = self.B / r2 + self.phi.forward(X) - self.Y
                size = float(torch.linalg.vector_norm(v))
                self.B = v * (r2 * (1.0 - self.eps / size) if size > self.eps else 0.0)
            if cone:
                z = self.Z - tau * self.D
                over = (z.sum(0) > 0.0)[None]
                Z1 = torch.where(over, 0.5 * torch.stack([z[0] - z[1], z[1] - z[0]]), z)
                c, d = (self.C + r3 * X) / r3, (self.D + r3 * (2.0 * Z1 - self.Z)) / r3
                keep = c[0] + d[0] >= 0.0
                p0, e0 = torch.where(keep, c[0], 0.5 * (c[0] - d[0])), torch.where(keep, d[0], 0.5 * (d[0] - c[0]))
                size = c[1:].pow(2).sum(0).sqrt()
                inside, polar = size <= d[1], size <= -d[1]
                f = torch.where(inside, torch.ones_like(size),
                                torch.where(polar, torch.zeros_like(size), 0.5 * (1.0 + d[1] / size.clamp(min=1e-300))))
                e1 = torch.where(inside, d[1], torch.where(polar, torch.zeros_like(size), f * size))
                self.C = r3 * (c - torch.cat([p0[None], f[None] * c[1:]]))
                self.D = r3 * (d - torch.stack([e0, e1]))
                self.Z = Z1
            self.old, self.S = S, S1

    def reweight(self, delta):
        self.W = delta / (delta + self.psi.adjoint(self.S).abs())

    def algorithm2(self):
        stages = _stages(self.case)
        self.iterate(stages[0], "init")
        delta = float(self.psi.adjoint(self.S).std(correction=0))
        for its in stages[1:]:
            self.reweight(delta)
            self.iterate(its, self.case["mode"])
            delta /= 10.0

    def adaptive(self, most, check, theta, rel_var, np_max):
        done = 0
        while done < most:
            k = min(check, most - done)
            self.iterate(k, "constrained")
            done += k
            residual, zeta, _ = self.report()
            num, den = (self.S - self.old).flatten(1).norm(dim=1), self.old.flatten(1).norm(dim=1)
            moved = max(float(a / b) if b > 0 else (math.inf if a > 0 else 0.0) for a, b in zip(num, den))
            outside = 100.0 * float((self.S[1:].pow(2).sum(0).sqrt() - self.S[0] > zeta).double().mean())
            if residual <= (1.0 + theta) * self.eps and moved <= rel_var and outside <= np_max:
                break
        return done

    def report(self):
        if self.case["kind"] == "tv":      # the report takes the brightness products of the data
            V = self.phi.stokes(self.S) - self.Y
            B = V @ self.phi.mix
            grad = self.psi.adjoint(self.S)
            objective = float((self.tw * grad[-2:].pow(2).sum(0).sqrt()).sum())
            if self.lw is not None:
                objective += float((self.lw * self.S.abs()).sum())
        else:
            B = self.phi.forward(self.S) - self.Y
            objective = float((self.W * self.psi.adjoint(self.S).abs()).sum())
        zeta = 3.0 * float((self.phi.adjoint(B)[0] / (2.0 * self.Y.shape[0])).pow(2).mean().sqrt())
        return float(torch.linalg.vector_norm(B)), zeta, objective

    def outputs(self):
        n = self.case["n"]
        return {"image": self.S.permute(1, 2, 0).reshape(n * n, 4).cpu().numpy(),
                "report": np.array(self.report())}


def exact(case, seed):
    if case["kind"] == "batch":
        out = {}
        for i, m in enumerate(_members(case)):
            ref = _Reference(m, _inputs(m, seed + 1000 * i))
            ref.algorithm2()
            out["image%d" % i] = ref.outputs()["image"]
        return out
    inputs = _inputs(case, seed)
    n = case["n"]
    if case["kind"] == "operators":
        dev = _device()
        phi, psi = _Phi(n, inputs["uv"], case["taps"]), _Sara(n, case["levels"])
        S = torch.from_numpy(np.ascontiguousarray(inputs["truth"].reshape(n, n, 4).transpose(2, 0, 1))).to(dev)
        coef = np.random.default_rng(5).standard_normal((9 * n * n, 4)) * float(np.abs(inputs["Y"]).mean())
        A = torch.from_numpy(np.ascontiguousarray(coef.reshape(9, n, n, 4).transpose(0, 3, 1, 2))).to(dev)

        def flat(x):
            return x.movedim(-3, -1).reshape(-1, 4).cpu().numpy()
        return {"phi": phi.forward(S).cpu().numpy(), "phi_adjoint": flat(phi.adjoint(torch.from_numpy(inputs["Y"]).to(dev))),
                "psi_adjoint": flat(psi.adjoint(S)), "psi": flat(psi.forward(A))}
    ref = _Reference(case, inputs)
    if case["kind"] == "tv":
        ref.iterate(case["iters"], case["mode"])
    elif case["kind"] == "adaptive":
        its = ref.adaptive(case["iters"], case["check"], 0.5, 1e-2, 50.0)
        return {**ref.outputs(), "iterations": np.array(its, dtype=np.int64)}
    else:
        ref.algorithm2()
    return ref.outputs()


if __name__ == "__main__":
    serve(int(sys.argv[1]), sys.argv[2])
