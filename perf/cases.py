"""Workloads of the library as its users run them, through its public entry points.

The matrices are the repository's own: trilinear hexahedra on the unit cube,
-div(sigma grad u) + c u with sigma = exp(N(0, 1)) per element, c = 1e-3 and
every node kept (N = n^3, nnz = (3n - 2)^3), right-hand sides U[-1, 1].  n = 51
has the size that the library was written for (N = 132651, nnz = 3442951), 16
is the smallest and 128 the largest that the tests and the benchmark solve.

Here the matrix is assembled with plain torch operations, in ELL form (27
slots a row), for exact(), and handed to the library in CSR.

solve   one right-hand side to a relative residual of 1e-10: the call the
        library exists for, in its standard and single-reduction iterations
        and with FP32 matrix values.
batch   many independent systems of uneven size in one call.
multi   up to 64 right-hand sides together, one recurrence a column.
block   the same right-hand sides with one shared Krylov space.
spmv    the sparse product alone.
q1      the same operator applied from its element coefficients.
train   one epoch of the warm start's network: minibatch steps, then the
        parameters.

A solve's result is its solution.  The other fields of the info record are the
call's wall time and scalars of the stopping test, not results.
"""
import math

import numpy as np
import torch

TOL = 1e-10
MASS = 1e-3
KHAT = (1.0 / 3.0, 0.0, -1.0 / 12.0, -1.0 / 12.0)
LEARNED = {"inputs": 24, "modes": 64, "samples": 1500}  # the 8 source centres; POD modes; training set


def listed():
    return [
        # A small system: launches, waits and host trips are all there is.
        {"name": "solve_16", "kind": "solve", "n": 16, "form": "standard", "values": "fp64"},
        # The size the library is written for, in both iterations.
        {"name": "solve_51", "kind": "solve", "n": 51, "form": "standard", "values": "fp64"},
        {"name": "solve_51_single", "kind": "solve", "n": 51, "form": "single", "values": "fp64"},
        # The largest system of the benchmark: the matrix no longer fits a cache.
        {"name": "solve_128", "kind": "solve", "n": 128, "form": "standard", "values": "fp64"},
        # The same with the FP32 copy of the values streamed.
        {"name": "solve_128_fp32", "kind": "solve", "n": 128, "form": "standard", "values": "fp32"},
        # Many systems of uneven size at once (a parameter study).
        {"name": "batch_96", "kind": "batch", "count": 96, "lo": 12, "hi": 48},
        # 64 load cases on one matrix, per column and as a block.
        {"name": "multi_51x64", "kind": "multi", "n": 51, "s": 64},
        {"name": "block_51x64", "kind": "block", "n": 51, "s": 64},
        # The product alone, from a cache and from memory.
        {"name": "spmv_51", "kind": "spmv", "n": 51},
        {"name": "spmv_128", "kind": "spmv", "n": 128},
        # The operator without its matrix.
        {"name": "q1_128", "kind": "q1", "n": 128},
        # Training the warm start's network: many small launches.
        {"name": "train_256", "kind": "train", "batch": 256, "hidden": 256, "precision": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "multi", "block", "spmv", "q1", "train"])
    if kind == "solve":
        form, values = rng.choice([("standard", "fp64"), ("single", "fp64"), ("standard", "fp32")])
        return {"kind": kind, "n": _log_int(rng, 16, 120), "form": form, "values": values}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(16, 96), "lo": rng.randint(12, 24), "hi": rng.randint(30, 47)}
    if kind in ("multi", "block"):
        return {"kind": kind, "n": _log_int(rng, 16, 51), "s": rng.randint(2, 64)}
    if kind == "train":
        return {"kind": kind, "batch": rng.randint(32, 256), "hidden": rng.randint(48, 256),
                "precision": rng.choice(["bf16", "fp32"])}
    return {"kind": kind, "n": _log_int(rng, 16, 128)}


def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _generator(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _sigma(n, g, device):
    m = n - 1
    return torch.exp(torch.randn((m, m, m), generator=g, device=device, dtype=torch.float64))


def _ell(n, sigma):
    """(column, value, present) of the n^3 operator, each N x 27 in ascending column order."""
    device = sigma.device
    h = 1.0 / (n - 1)
    pad = torch.zeros((n + 1, n + 1, n + 1), dtype=torch.float64, device=device)
    pad[1:n, 1:n, 1:n] = sigma
    one = (pad != 0).double()
    lower, upper = slice(0, n), slice(1, n + 1)
    # Elements that two nodes share along an axis, by the offset between them.
    shared = {-1: (lower,), 0: (lower, upper), 1: (upper,)}
    t = torch.arange(n, device=device)
    inside = {d: (t + d >= 0) & (t + d < n) for d in (-1, 0, 1)}
    row = torch.arange(n ** 3, device=device)
    col = torch.empty((n ** 3, 27), dtype=torch.int64, device=device)
    val = torch.empty((n ** 3, 27), dtype=torch.float64, device=device)
    here = torch.empty((n ** 3, 27), dtype=torch.bool, device=device)
    o = 0
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                d = abs(dx) + abs(dy) + abs(dz)
                hk, cm = h * KHAT[d], MASS * h ** 3 * (1.0 / 3.0) ** (3 - d) * (1.0 / 6.0) ** d
                acc = torch.zeros((n, n, n), dtype=torch.float64, device=device)
                for sz in shared[dz]:
                    for sy in shared[dy]:
                        for sx in shared[dx]:
                            acc += pad[sz, sy, sx] * hk + one[sz, sy, sx] * cm
                ok = (inside[dz][:, None, None] & inside[dy][None, :, None] & inside[dx][None, None, :]).reshape(-1)
                here[:, o] = ok
                val[:, o] = torch.where(ok, acc.reshape(-1), torch.zeros_like(val[:, o]))
                col[:, o] = torch.where(ok, row + dx + n * dy + n * n * dz, row)
                o += 1
    return col, val, here


class _Csr:
    def __init__(self, n, rowptr, col, val):
        self.n, self.rowptr, self.col, self.val = n, rowptr, col, val


def _csr(ell):
    col, val, here = ell
    rowptr = torch.zeros(col.shape[0] + 1, dtype=torch.int64, device=col.device)
    torch.cumsum(here.sum(1), 0, out=rowptr[1:])
    return _Csr(col.shape[0], rowptr.int(), col[here].int(), val[here])


def _uniform(shape, g, device):
    return torch.rand(shape, generator=g, device=device, dtype=torch.float64) * 2.0 - 1.0


def _sizes(case):
    """Edges of a batch's systems: every size of the range as likely as another."""
    rng = np.random.default_rng(1000 + case["count"])
    return [int(v) for v in rng.integers(case["lo"], case["hi"] + 1, case["count"])]


def _inputs(case, seed):
    """The matrices (ELL) and the right-hand side or operand of a case, from its seed."""
    device = _device()
    g = _generator(seed, device)
    kind = case["kind"]
    if kind == "batch":
        ells = [_ell(n, _sigma(n, g, device)) for n in _sizes(case)]
        return ells, _uniform(sum(e[0].shape[0] for e in ells), g, device)
    n = case["n"]
    sigma = _sigma(n, g, device)
    shape = (n ** 3, case["s"]) if kind in ("multi", "block") else (n ** 3,)
    return ([sigma] if kind == "q1" else [_ell(n, sigma)]), _uniform(shape, g, device)


def _epoch(case, seed):
    """Start parameters, inputs in [-1, 1] and standardised targets of the network's training set."""
    rng = np.random.default_rng(int(seed))
    dims = [LEARNED["inputs"], case["hidden"], case["hidden"], LEARNED["modes"]]
    params = []
    for a, b in zip(dims[:-1], dims[1:]):
        bound = math.sqrt(6.0 / a) / 2.0
        params += [rng.uniform(-bound, bound, a * b), np.zeros(b)]
    x = rng.uniform(-1.0, 1.0, (LEARNED["samples"], dims[0])).astype(np.float32)
    y = rng.standard_normal((LEARNED["samples"], dims[-1])).astype(np.float32)
    return dims, np.concatenate(params).astype(np.float32), x, y


def prepare(case, seed):
    from paper_1107_0538_amd import Batch, Solver
    from paper_1107_0538_amd.learned import MLP

    kind = case["kind"]
    state = {"case": case}
    if kind == "train":
        dims, params, x, y = _epoch(case, seed)
        net = MLP(dims, case["precision"], max_batch=case["batch"])
        net.set_params(params)
        state.update(net=net, x=torch.as_tensor(x, device=_device()), y=torch.as_tensor(y, device=_device()))
        return state
    mats, rhs = _inputs(case, seed)
    state["rhs"] = rhs
    if kind == "q1":
        state["sigma"] = mats[0].reshape(-1)
    elif kind == "batch":
        systems = [_csr(e) for e in mats]
        for a in systems:
            a.rowptr, a.col, a.val = a.rowptr.cpu().numpy(), a.col.cpu().numpy(), a.val.cpu().numpy()
        state["batch"] = Batch(systems)
    else:
        a = _csr(mats[0])
        del mats
        state["solver"] = Solver(a, form=case.get("form", "standard"), fp32_copy=case.get("values") == "fp32")
    return state


def run(state):
    from paper_1107_0538_amd import solver as api

    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        solve = state["solver"].solve_mixed_matrix if case["values"] == "fp32" else state["solver"].solve
        return solve(state["rhs"], tol=TOL)[0]
    if kind == "batch":
        return state["batch"].solve(state["rhs"], tol=TOL)[0]
    if kind == "multi":
        return state["solver"].solve_multi(state["rhs"], tol=TOL)[0]
    if kind == "block":
        return state["solver"].solve_block(state["rhs"], tol=TOL)[0]
    if kind == "spmv":
        return state["solver"].spmv(state["rhs"])
    if kind == "q1":
        return api.q1_apply(case["n"], state["sigma"], state["rhs"], c=MASS)
    net, x, y, b = state["net"], state["x"], state["y"], case["batch"]
    steps = x.shape[0] // b
    for i in range(steps):
        loss = net.train_step(x[i * b:(i + 1) * b], y[i * b:(i + 1) * b], want_loss=i == steps - 1)
    return {"params": net.get_params(), "loss": loss}


def work(case):
    """Inputs read once, results written once; an iteration's products and vector updates as operations."""
    kind = case["kind"]
    if kind == "train":
        i, h, m = LEARNED["inputs"], case["hidden"], LEARNED["modes"]
        params, rows = i * h + h * h + h * m + 2 * h + m, LEARNED["samples"] // case["batch"] * case["batch"]
        return {"bytes": 4.0 * (rows * (i + m) + 8 * params), "flops": 6.0 * rows * (i * h + h * h + h * m)}
    if kind == "batch":
        edges = list(range(case["lo"], case["hi"] + 1))
        share = case["count"] / len(edges)
    else:
        edges, share = [case["n"]], 1.0
    total = {"bytes": 0.0, "flops": 0.0}
    for n in edges:
        rows, nnz, s = n ** 3, (3 * n - 2) ** 3, case.get("s", 1)
        if kind == "q1":
            total["bytes"] += 8.0 * (n - 1) ** 3 + 16.0 * rows
            total["flops"] += 54.0 * rows
            continue
        value = 4 if case.get("values") == "fp32" else 8
        matrix = (value + 4.0) * nnz + 4.0 * (rows + 1)
        if kind == "spmv":
            total["bytes"] += matrix + 16.0 * rows
            total["flops"] += 2.0 * nnz
            continue
        iterations = 8.0 * n  # measured: 135, 410 and 982 at 16, 51 and 128
        if kind == "block":
            iterations = 1.9 * n  # measured with 64 columns: 95 at 51
            flops = iterations * (2.0 * nnz * s + 2.0 * rows * s * s * 9)
        else:
            flops = iterations * (2.0 * nnz + 12.0 * rows) * s
        total["bytes"] += share * (matrix + 24.0 * rows * s)
        total["flops"] += share * flops
    return total


class _Exact:
    """The systems of a case as one block-diagonal ELL operator, in difference form.

    (A x)_i = sum_j a_ij (x_j - x_i) + s_i x_i with the row sums s_i added with
    their rounding errors: A 1 is the small mass term, and this keeps it.
    """

    def __init__(self, ells):
        device = ells[0][0].device
        sizes = [e[0].shape[0] for e in ells]
        starts = np.concatenate([[0], np.cumsum(sizes)])
        self.col = torch.cat([e[0] + int(o) for e, o in zip(ells, starts)])
        self.val = torch.cat([e[1] for e in ells])
        own = torch.arange(int(starts[-1]), device=device)[:, None]
        self.diag = (self.val * (self.col == own) * torch.cat([e[2] for e in ells])).sum(1)
        s, low = torch.zeros_like(self.diag), torch.zeros_like(self.diag)
        for j in range(self.val.shape[1]):
            v = self.val[:, j]
            t = s + v
            k = t - s
            low += (s - (t - k)) + (v - k)
            s = t
        self.sums = s + low
        self.starts = [int(v) for v in starts]
        self.system = torch.repeat_interleave(torch.arange(len(sizes), device=device), torch.tensor(sizes, device=device))

    def apply(self, x):
        y = self.sums[:, None] * x
        for j in range(self.val.shape[1]):
            y += self.val[:, j, None] * (x[self.col[:, j]] - x)
        return y

    def dot(self, a, b):
        ab = a * b
        if len(self.starts) == 2:
            return ab.sum(0, keepdim=True)
        return torch.zeros((len(self.starts) - 1, ab.shape[1]), dtype=ab.dtype, device=ab.device).index_add_(
            0, self.system, ab)

    def spread(self, v):
        return v if len(self.starts) == 2 else v[self.system]

    def solve(self, b):
        x = torch.zeros_like(b)
        for _ in range(3):  # each round solves for what the last one left
            r = b - self.apply(x)
            goal = self.dot(r, r) * 1e-18
            d, z = torch.zeros_like(b), r / self.diag[:, None]
            p, rho = z.clone(), self.dot(r, z)
            for k in range(4000):
                q = self.apply(p)
                alpha = self.spread(rho / self.dot(p, q).clamp_min(1e-300))
                d += alpha * p
                r -= alpha * q
                if k % 16 == 15 and bool((self.dot(r, r) <= goal).all()):
                    break
                z = r / self.diag[:, None]
                new = self.dot(r, z)
                p = z + self.spread(new / rho.clamp_min(1e-300)) * p
                rho = new
            x += d
        return x


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed) if case["precision"] == "fp32" else None
    mats, rhs = _inputs(case, seed)
    if case["kind"] == "q1":
        mats = [_ell(case["n"], mats[0])]
    op = _Exact(mats)
    del mats
    if case["kind"] in ("spmv", "q1"):
        return op.apply(rhs[:, None])[:, 0]
    if rhs.dim() == 2:
        return op.solve(rhs)
    return op.solve(rhs[:, None])[:, 0]


def _exact_train(case, seed):
    dims, params, x, y = _epoch(case, seed)
    flat = torch.tensor(params, dtype=torch.float64)
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    x, y, b = torch.tensor(x, dtype=torch.float64), torch.tensor(y, dtype=torch.float64), case["batch"]
    loss = None
    for i in range(x.shape[0] // b):
        w = flat.clone().requires_grad_(True)
        h, o = x[i * b:(i + 1) * b], 0
        for layer, (fan_in, fan_out) in enumerate(zip(dims[:-1], dims[1:])):
            weight = w[o:o + fan_in * fan_out].reshape(fan_out, fan_in)
            o += fan_in * fan_out
            h = h @ weight.T + w[o:o + fan_out]
            o += fan_out
            if layer < len(dims) - 2:
                h = h * torch.sigmoid(h)
        loss = ((h - y[i * b:(i + 1) * b]) ** 2).mean()
        grad, = torch.autograd.grad(loss, w)
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        flat = flat - 1e-3 * (m / (1 - 0.9 ** (i + 1))) / ((v / (1 - 0.999 ** (i + 1))).sqrt() + 1e-8)
    return {"params": flat.numpy(), "loss": float(loss)}
