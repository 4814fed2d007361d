"""Workloads of the homomorphic matrix library, for timing a build of it.

Each case is one thing a user's program has the library do, through the
public Python binding: a client encrypting a matrix and reading a result, a
server rotating, multiplying and transforming ciphertexts, single and batched
matrix products, the block covariance and a PowerMethod round.  The rings and
chains are those of ``paper_2305_17341_amd.inputs`` (N = 2^13 .. 2^16).

A server holds its parameter set and switching keys for its whole life, so a
context is built once per chain and kept while cases of that chain are
prepared; the operands come from the seed.  A server hands results on as
ciphertext words (``export``); where the result is a batch of large
ciphertexts, or is computed for the client, the client's decryption is what
comes back.
"""
from __future__ import annotations

import numpy as np
import torch  # noqa: F401  (before the library, so that both use one HIP runtime)

from paper_2305_17341_amd import he, inputs

BATCHED, LAZY, FUSED, MERGED = 1, 2, 4, 64

# the matrix sizes served on each ring: d^2 entries fit the N/2 slots
SIZES = {"n13_small": (16, 32, 64), "n14_mid": (16, 32, 64), "n15_serve": (16, 32, 64, 128),
         "n16_large": (16, 32, 64, 128)}
TAYLOR_X0 = 2.0 ** 15 + 1


def listed():
    return [
        # the smallest call of a server: one key-switched rotation, latency only
        dict(name="rotate_n13", op="rotate", chain="n13_small", level=3, step=1),
        # one product of two ciphertexts, relinearised and rescaled (drawn: several by one factor)
        dict(name="mult_n14", op="mult", chain="n14_mid", level=8, count=1),
        # the client: encrypt a 64 x 64 matrix and send it, read back a result that used up most levels
        dict(name="client_n14", op="client", chain="n14_mid", level=8, d=64, back=2),
        # sliding sums: hoisted rotations of a few ciphertexts by an odd number of steps, added up
        dict(name="window_n15", op="window", chain="n15_serve", level=14, count=3, steps=11),
        # smallest matrix product, the paper's order (every product relinearised), nothing chosen by the caller
        dict(name="matmul16_n13", op="matmul", chain="n13_small", level=3, d=16, n1=0, nprime=0, flags=0),
        # ordinary product with the options the serving layer uses, at a level left by an earlier product
        dict(name="matmul64_n14", op="matmul", chain="n14_mid", level=7, d=64, n1=0, nprime=0, flags=LAZY | FUSED),
        # the paper's own setting: 128 x 128 at N = 2^15, decomposed transforms (n' = 32), n1 = 16, paper's order
        dict(name="matmul128_n15_dcd", op="matmul", chain="n15_serve", level=14, d=128, n1=16, nprime=32, flags=0),
        # one large product on its own, default options
        dict(name="matmul128_n16", op="matmul", chain="n16_large", level=30, d=128, n1=0, nprime=0, flags=0),
        # what a serving tick runs: requests of mixed sizes merged, odd counts
        dict(name="mixed_n14", op="batch", chain="n14_mid", level=8, ds="64,16,32,16,64,32,16", n1=0,
             flags=BATCHED | LAZY | FUSED | MERGED),
        # the largest call: eight 128 x 128 products as one batch, baby steps 64
        dict(name="batch8_n16", op="batch", chain="n16_large", level=30, ds="128,128,128,128,128,128,128,128", n1=64,
             flags=BATCHED | LAZY | FUSED),
        # covariance of 200 samples x 256 features in 128 x 128 blocks (last row block ragged)
        dict(name="covariance_n15", op="covariance", chain="n15_serve", level=14, d=128, k=2, samples=200,
             flags=LAZY | FUSED),
        # one round of the PowerMethod on a 256-feature covariance, the client refreshing on demand
        dict(name="power_n15", op="power", chain="n15_serve", level=14, d=128, k=2, newton=7, goldschmidt=False),
    ]


def draw(rng):
    op = rng.choice(["rotate", "mult", "client", "window", "transform", "matmul", "matmul", "matmul", "batch", "batch",
                     "covariance", "power"])
    name = rng.choice(sorted(SIZES))
    if op == "covariance":
        name = rng.choice(["n14_mid", "n15_serve"])
    elif op == "power":
        name = rng.choice(["n14_mid", "n15_serve", "n16_large"])
    top = inputs.CHAINS[name].top_level
    case = dict(op=op, chain=name)
    if op == "rotate":
        step = rng.choice([rng.randint(2, 200), -rng.randint(1, 200)])
        return dict(case, level=rng.randint(0, top), step=step)
    if op == "mult":
        return dict(case, level=rng.randint(1, top), count=rng.randint(1, 6))
    if op == "client":
        return dict(case, level=rng.randint(1, top), d=rng.choice(SIZES[name]), back=rng.randint(0, 1))
    if op == "window":
        return dict(case, level=rng.randint(1, top), count=rng.randint(1, 4), steps=rng.randint(2, 20))
    d = rng.choice(SIZES[name])
    if op == "transform":
        n1 = rng.choice([0, 4, 8])
        kind = rng.choice(["sigma", "tau", "transpose"])
        form = rng.choice(["plain", "plain", "decomposed", "substituted"]) if kind != "transpose" else "plain"
        return dict(case, level=rng.randint(3, top), d=d, kind=kind, n1=n1, form=form)
    if op == "matmul":
        flags = rng.choice([0, 0, LAZY, LAZY | FUSED, LAZY | FUSED])
        n1 = rng.choice([0, 0, 8, d // 2])
        dcd = top >= 14 and rng.random() < 0.3
        low = 6 if dcd else 3
        level = rng.randint(low, top)
        return dict(case, level=level, d=d, n1=n1, nprime=d // 2 if dcd else 0, flags=flags)
    if op == "batch":
        large = name == "n16_large"
        sizes = [s for s in SIZES[name] if not large or s <= 64]
        ds = [rng.choice(sizes) for _ in range(rng.randint(2, 4 if large else 8))]
        merged = len(set(ds)) > 1 and rng.random() < 0.6
        flags = BATCHED | rng.choice([0, LAZY | FUSED, LAZY | FUSED]) | (MERGED if merged else 0)
        return dict(case, level=rng.randint(3, min(top, 20)), ds=",".join(map(str, ds)), n1=0, flags=flags)
    if op == "covariance":
        d = rng.choice([16, 32, 64])
        return dict(case, level=rng.randint(6, top), d=d, k=rng.randint(1, 3), samples=rng.randint(2 * d + 1, 5 * d),
                    flags=rng.choice([0, LAZY | FUSED]))
    return dict(case, level=rng.randint(6, top), d=d, k=rng.randint(1, 2), newton=rng.randint(3, 9),
                goldschmidt=rng.random() < 0.4)


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------
_CONTEXT = {}


def _context(name):
    """the chain's context, kept while its cases are prepared (one chain at a time)"""
    if name not in _CONTEXT:
        _CONTEXT.clear()
        _CONTEXT[name] = he.chain_context(inputs.CHAINS[name], seed=1)
    return _CONTEXT[name]


def _opts(case):
    opts = {"flags": case.get("flags", 0)}
    if case.get("n1"):
        opts.update(n1_z=case["n1"], n1_t=case["n1"])
    if case.get("nprime"):
        opts.update(nprime_z=case["nprime"], nprime_t=case["nprime"])
    return opts


def _default_n1(d):
    return 1 << ((d.bit_length()) // 2)


def _transform_params(case):
    """(n1, n' of the decomposition, prefix of the key substitution)"""
    d = case["d"]
    n1 = case["n1"] or _default_n1(d)
    return n1, d // 2 if case["form"] == "decomposed" else 0, 2 if case["form"] == "substituted" else 0


def _steps(ctx, case):
    op = case["op"]
    if op == "rotate":
        return [case["step"]]
    if op == "window":
        return list(range(1, case["steps"] + 1))
    if op == "transform":
        n1, nprime, prefix = _transform_params(case)
        kind = {"sigma": "Z", "tau": "T", "transpose": "G"}[case["kind"]]
        if prefix:
            return he.smpkeysub_rot_steps(kind, case["d"], n1, prefix)
        return he.lintrans_rot_steps(kind, case["d"], n1, nprime)
    if op == "matmul":
        return ctx.matmul_rot_steps(case["d"], _opts(case))
    if op == "batch":
        return sorted({s for d in _sizes(case) for s in ctx.matmul_rot_steps(d, _opts(case))})
    if op == "covariance":
        return sorted(set(ctx.matmul_rot_steps(case["d"], _opts(case))) | set(ctx.transpose_rot_steps(case["d"])))
    if op == "power":
        return he.power_rot_steps(case["d"])
    return []


def _sizes(case):
    return [int(d) for d in case["ds"].split(",")]


def _data(case, seed):
    """the plaintext operands"""
    g = np.random.Generator(np.random.PCG64(seed))
    op, chain = case["op"], inputs.CHAINS[case["chain"]]
    if op in ("rotate", "mult", "window"):
        return g.uniform(-1, 1, size=(case.get("count", 1) + (op == "mult"), chain.N // 2))
    if op in ("client", "transform", "matmul"):
        return g.uniform(-1, 1, size=(2, case["d"], case["d"]))
    if op == "batch":
        return [g.uniform(-1, 1, size=(2, d, d)) for d in _sizes(case)]
    t = case["k"] * case["d"]
    if op == "covariance":
        X = g.uniform(0, 1, size=(case["samples"], t))
        return X - X.mean(axis=0)
    # a covariance whose leading eigenvalues the normalisation schedule expects, and a unit start vector
    Q, _ = np.linalg.qr(g.standard_normal((t, t)))
    v = g.standard_normal(t)
    return (Q * (8.0 * 0.75 ** np.arange(t))) @ Q.T, v / np.linalg.norm(v)


def _replicate(v, k, d, axis):
    """block i holds segment i of v as every row (axis 0) or every column (axis 1)"""
    rows = [np.tile(v[i * d:(i + 1) * d], (d, 1)) for i in range(k)]
    return [r if axis == 0 else r.T for r in rows]


def prepare(case, seed):
    ctx = _context(case["chain"])
    ctx.keygen(_steps(ctx, case))
    data, level, nonce = _data(case, seed), case["level"], 1000 * (seed + 1)
    state = dict(case=case, ctx=ctx)
    op = case["op"]
    if op in ("rotate", "mult", "window"):
        state["x"] = [ctx.encrypt(z, level, nonce + i) for i, z in enumerate(data)]
    elif op == "client":
        result = ctx.encrypt_matrix(data[1], case["back"], nonce)
        state.update(matrix=data[0], nonce=nonce + 1, words=result.export(), scale=result.scale)
    elif op in ("transform", "matmul"):
        state["x"] = [ctx.encrypt_matrix(z, level, nonce + i) for i, z in enumerate(data)]
    elif op == "batch":
        state["x"] = [ctx.encrypt_matrix(ab[0], level, nonce + 2 * i) for i, ab in enumerate(data)]
        state["y"] = [ctx.encrypt_matrix(ab[1], level, nonce + 2 * i + 1) for i, ab in enumerate(data)]
    elif op == "covariance":
        d, k = case["d"], case["k"]
        rows = -(-case["samples"] // d)
        X = np.zeros((rows * d, k * d))
        X[:case["samples"]] = data
        state["rows"] = rows
        state["x"] = [ctx.encrypt_matrix(X[r * d:(r + 1) * d, j * d:(j + 1) * d], level, nonce + r * k + j)
                      for r in range(rows) for j in range(k)]
    else:
        d, k = case["d"], case["k"]
        cov, v = data
        state["x"] = [ctx.encrypt_matrix(cov[r * d:(r + 1) * d, c * d:(c + 1) * d], level, nonce + r * k + c)
                      for r in range(k) for c in range(k)]
        state["y"] = [ctx.encrypt_matrix(b, level, nonce + 100 + i)
                      for i, b in enumerate(_replicate(v, k, d, 1))]
    ctx.sync()
    return state


# ---------------------------------------------------------------------------
# the call
# ---------------------------------------------------------------------------
def run(state):
    case, ctx = state["case"], state["ctx"]
    op = case["op"]
    if op == "rotate":
        return ctx.rotate(state["x"][0], case["step"]).export()
    if op == "mult":
        x = state["x"]
        return [ctx.rescale(ctx.mult(a, x[0])).export() for a in x[1:]]
    if op == "client":
        sent = ctx.encrypt_matrix(state["matrix"], case["level"], state["nonce"]).export()
        back = ctx.ct_import(state["words"], case["back"], state["scale"])
        return {"sent": sent, "read": ctx.decrypt(back, case["d"] ** 2)}
    if op == "window":
        out = []
        for x, turned in zip(state["x"], ctx.rotate_many(state["x"], range(1, case["steps"] + 1))):
            for t in turned:
                x = ctx.add(x, t)
            out.append(x)
        return [x.export() for x in out]
    if op == "transform":
        n1, nprime, prefix = _transform_params(case)
        x, kind, d = state["x"][0], case["kind"], case["d"]
        if case["form"] == "decomposed":
            return ctx.lintrans_dcd(x, kind, d, n1, nprime).export()
        if case["form"] == "substituted":
            return ctx.lintrans_smpkeysub(x, kind, d, n1, prefix).export()
        return ctx.lintrans(x, kind, d, n1).export()
    if op == "matmul":
        return ctx.matmul(state["x"][0], state["x"][1], case["d"], _opts(case)).export()
    if op == "batch":
        ds = _sizes(case)
        return [ctx.decrypt(c, d * d) for c, d in zip(ctx.matmul_batch(state["x"], state["y"], ds, _opts(case)), ds)]
    d, k = case["d"], case["k"]
    if op == "covariance":
        out = ctx.covariance(state["x"], state["rows"], k, d, case["samples"], _opts(case))
    else:
        out, _ = ctx.power_step(state["x"], k, d, state["y"], 1, case["newton"], TAYLOR_X0, False,
                                he.Refresher(ctx), goldschmidt=case["goldschmidt"])
    return [ctx.decrypt(c, d * d) for c in out]


def exact(case, seed):
    """the decrypted results in FP64; ciphertext words are randomised and have no such value"""
    op, data = case["op"], _data(case, seed)
    if op == "client":
        return {"sent": None, "read": data[1].ravel()}
    if op == "batch":
        return [(a @ b).ravel() for a, b in data]
    if op not in ("covariance", "power"):
        return None
    d, k = case["d"], case["k"]
    if op == "covariance":
        C = data.T @ data / case["samples"]
        return [C[a * d:(a + 1) * d, b * d:(b + 1) * d].ravel() for a in range(k) for b in range(k)]
    cov, v = data
    y = cov @ v
    x = float(y @ y)
    s = 1.5 * TAYLOR_X0 ** -0.5 - 0.5 * TAYLOR_X0 ** -1.5 * x
    for _ in range(case["newton"]):
        s = s * (1.5 - 0.5 * x * s * s)
    return [b.ravel() for b in _replicate(y * s, k, d, 0)]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: ciphertexts in and out and each switching key used, once.
    Flops: two per modular product of the key switches (transforms, basis
    conversions, key inner products) and of the tensors."""
    chain = inputs.CHAINS[case["chain"]]
    N, alpha, l = chain.N, len(chain.p_bits), case["level"]
    nq, nqp, beta = l + 1, l + 1 + alpha, -(-(l + 1) // alpha)
    ct, key = 2 * nq * N * 8.0, 2 * beta * nqp * N * 8.0
    ntt = N / 2 * chain.log_n
    down = 2 * (alpha + nq) * ntt + 2 * nq * alpha * N
    split = (nq + beta * (nqp - alpha)) * ntt + beta * nqp * alpha * N
    inner = 2 * beta * nqp * N

    def transform(d, n1, two_sided):
        giant = (2 if two_sided else 1) * -(-d // n1) - 1
        return (n1 - 1 + giant) * inner + giant * (down + split) + split + down, n1 - 1 + giant

    def product(d, n1, lazy):
        n1 = n1 or _default_n1(d)
        blocks = -(-d // n1)
        z, kz = transform(d, n1, True)
        t, kt = transform(d, n1, False)
        bases = 3 * blocks * split + 3 * d * inner + 2 * d * down
        relins = (1 if lazy else d) * (split + inner + down)
        return z + t + bases + relins + 4 * d * nq * N, kz + kt + 3

    op = case["op"]
    if op == "rotate":
        b, f = 2 * ct + key, split + inner + down
    elif op == "mult":
        n = case["count"]
        b, f = (2 * n + 1) * ct + key, n * (split + inner + down + 4 * nq * N)
    elif op == "client":
        b, f = 2 * ct + 2 * case["d"] ** 2 * 8, (3 * nq + 1) * ntt + 2 * N * chain.log_n
    elif op == "window":
        b = 2 * case["count"] * ct + case["steps"] * key
        f = case["count"] * (split + case["steps"] * (inner + down))
    elif op == "transform":
        f, keys = transform(case["d"], _transform_params(case)[0], case["kind"] != "tau")
        b = 2 * ct + keys * key
    elif op == "matmul":
        f, keys = product(case["d"], case["n1"], case["flags"] & LAZY)
        b = 3 * ct + keys * key
    elif op == "batch":
        parts = [product(d, case["n1"], case["flags"] & LAZY) for d in _sizes(case)]
        f = sum(p[0] for p in parts)
        b = 2 * len(parts) * ct + max(p[1] for p in parts) * key
    elif op == "covariance":
        d, k = case["d"], case["k"]
        rows, n1 = -(-case["samples"] // d), _default_n1(d)
        p, keys = product(d, 0, case["flags"] & LAZY)
        g, kg = transform(d, n1, True)
        f = rows * k * (p + g) + k * (k + 1) / 2 * rows * 4 * d * nq * N
        b = (rows * k + k * k) * ct + (keys + kg) * key
    else:
        k, lg = case["k"], case["d"].bit_length() - 1
        switches = k * k + k + 3 * case["newton"] + k + (k + 1) * 2 * lg
        b, f = (k * k + 2 * k) * ct + (3 * lg + 1) * key, switches * (split + inner + down)
    return {"bytes": float(b), "flops": 2.0 * f}
