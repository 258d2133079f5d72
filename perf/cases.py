"""The workloads that this library is timed on, over the range it is used in.

A case is a dict of plain values.  ``listed()`` gives the fixed cases,
``draw(rng)`` one more of the same ranges, ``prepare(case, seed)`` what a
program holds before the call (generators, packed batches, a running server,
network parameters), ``run(state)`` one pass through the public entry points
with all of its outputs, ``work(case)`` the bytes and operations that a pass
cannot do without, and ``exact(case, seed)`` the outputs in 64 bits where plain
numpy can give them.

Kinds of case:
  plain     one ``min_distance`` call per code (``min_distance_noalloc`` when
            ``noalloc``); ``hist``: the whole weight spectrum, no early end
  batch     one batched call on many codes
  serve     a running server: a burst of requests, polled until all are back
  mlp       one training step of the work predictor
  sliced    symbols packed into bit planes, one vector operation, unpacked
"""
import ctypes
import math

import numpy as np
import torch

from paper_2603_29942_amd import autotune, bz, predictor

DEV = "cuda:0"
SLICED = {"add": bz.OP_ADD, "sub": bz.OP_SUB, "double": bz.OP_DOUBLE, "kat": bz.OP_KAT_ADD}


def _plain(name, p, n, k, codes=1, host=False, check="stage", hist=False, noalloc=False):
    return {"name": name, "kind": "plain", "p": p, "n": n, "k": k, "codes": codes, "host": host, "check": check,
            "hist": hist, "noalloc": noalloc}


def listed():
    return [
        # the smallest call in earnest: one small ternary code, the time is all latency
        _plain("plain_f3_40_10", 3, 40, 10),
        # a study of random ternary codes of rate 1/2, one call each (the plain sub-block of the benchmark)
        _plain("plain_f3_72_36", 3, 72, 36, codes=8),
        # the same over F_7
        _plain("plain_f7_48_24", 7, 48, 24, codes=8),
        # the largest single code over F_7 that a user waits for: the rate 1/2 cap of the mixed batch
        _plain("plain_f7_56_28", 7, 56, 28),
        # a long ternary code, the upper end of the mixed batch's lengths at rate 1/3
        _plain("plain_f3_89_29", 3, 89, 29, codes=2),
        # a generator in host memory, ragged sizes, rate 1/3 (four information sets), the bound tested per round
        _plain("plain_host_f7_45_13", 7, 45, 13, codes=4, host=True, check="round"),
        # callers that may not allocate (tight loops, captured code)
        _plain("noalloc_f3_60_30", 3, 60, 30, codes=4, noalloc=True),
        # a whole weight spectrum: every stage, with histograms
        _plain("spectrum_f7_26_9", 7, 26, 9, hist=True),
        # a handful of codes handed over as host arrays and packed for the call, default task sizes
        {"name": "batch_24_host", "kind": "batch", "count": 24, "n_lo": 30, "n_hi": 48, "f7_half": 40, "f7_third": 45,
         "device": False},
        # the benchmark's own batch: 512 codes, generators resident, the autotuner's task sizes
        {"name": "batch_512", "kind": "batch", "count": 512, "n_lo": 30, "n_hi": 90, "f7_half": 56, "f7_third": 63,
         "device": True},
        # a burst of requests to a server that orders them by predicted work
        {"name": "serve_128", "kind": "serve", "count": 128, "k_lo": 10, "k_hi": 40, "f7_kmax": 28,
         "policy": "predicted"},
        # a training step of the work predictor on its 8000 training runs
        {"name": "mlp_train_8000", "kind": "mlp", "samples": 8000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choices(["plain", "noalloc", "spectrum", "batch", "serve", "mlp", "sliced"],
                       [9, 2, 2, 3, 2, 2, 1])[0]
    if kind in ("plain", "noalloc"):
        p = rng.choice([3, 7])
        half = rng.random() < 0.5
        top = 90 if p == 3 else ((48 if half else 57) if kind == "noalloc" else (54 if half else 61))
        n = rng.randint(24, top)
        k = n // 2 if half else n // 3
        return _plain_drawn(p, n, max(2, k + rng.choice([0, 0, -1])), codes=rng.randint(1, 4),
                            host=kind == "plain" and rng.random() < 0.3,
                            check="round" if rng.random() < 0.2 else "stage", noalloc=kind == "noalloc")
    if kind == "spectrum":
        p = rng.choice([3, 7])
        k = rng.randint(6, 15) if p == 3 else rng.randint(4, 9)
        return _plain_drawn(p, rng.randint(k + 5, 3 * k + 8), k, hist=True)
    if kind == "batch":
        n_lo = rng.randint(24, 40)
        return {"kind": "batch", "count": _log_int(rng, 4, 300), "n_lo": n_lo, "n_hi": n_lo + rng.randint(8, 50),
                "f7_half": rng.randint(40, 52), "f7_third": rng.randint(42, 58), "device": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": "serve", "count": _log_int(rng, 8, 128), "k_lo": 8, "k_hi": rng.randint(16, 38),
                "f7_kmax": rng.randint(16, 26), "policy": rng.choice(["fifo", "predicted"])}
    if kind == "mlp":
        return {"kind": "mlp", "samples": _log_int(rng, 200, 10000)}
    p, op = rng.choice([(3, "add"), (3, "sub"), (3, "kat"), (7, "add"), (7, "sub"), (7, "double")])
    return {"kind": "sliced", "p": p, "op": op, "nvec": _log_int(rng, 100, 20000), "nsym": rng.randint(33, 1100)}


def _plain_drawn(*args, **kw):
    c = _plain("", *args, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs
def _rng(seed, *more):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, *more])


def _mixed_codes(case, seed):
    """Random codes of the mixed batch: half over each field, rate 1/2 or 1/3."""
    rng = _rng(seed, 4)
    ps = np.array([3] * (case["count"] // 2) + [7] * (case["count"] - case["count"] // 2))
    rng.shuffle(ps)
    out = []
    for p in ps:
        while True:
            n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
            half = bool(rng.integers(0, 2))
            if p == 3 or n <= (case["f7_half"] if half else case["f7_third"]):
                break
        k = n // 2 if half else n // 3
        out.append((int(p), rng.integers(0, int(p), size=(k, n), dtype=np.uint8)))
    return out


def _requests(case, seed):
    rng = _rng(seed, 5)
    out = []
    for _ in range(case["count"]):
        p = 3 if rng.integers(0, 2) == 0 else 7
        k = int(rng.integers(case["k_lo"], (case["k_hi"] if p == 3 else min(case["k_hi"], case["f7_kmax"])) + 1))
        out.append((p, rng.integers(0, p, size=(k, 2 * k), dtype=np.uint8)))
    return out


def _plain_codes(case, seed):
    rng = _rng(seed, 1)
    return [rng.integers(0, case["p"], size=(case["k"], case["n"]), dtype=np.uint8) for _ in range(case["codes"])]


def _mlp_inputs(case, seed):
    """Features and targets like those of served codes, the trained network a
    few hundred steps further on."""
    rng = _rng(seed, 6)
    s = case["samples"]
    p = rng.choice([3, 7], size=s)
    k = np.where(p == 3, rng.integers(10, 41, size=s), rng.integers(10, 29, size=s))
    x = np.stack([(p - 5.0) / 2.0, (2 * k - 60.0) / 30.0, (k - 25.0) / 15.0, rng.integers(0, 4, size=s) / 8.0],
                 axis=1).astype(np.float32)
    t = (np.where(p == 3, 0.19, 0.33) * k + 1.0 + rng.normal(0, 0.3, size=s)).astype(np.float32)
    theta = (predictor.load()[0] + rng.normal(0, 0.01, predictor.NPARAM)).astype(np.float32)
    m = rng.normal(0, 1e-2, predictor.NPARAM).astype(np.float32)
    v = (rng.random(predictor.NPARAM) * 1e-3 + 1e-4).astype(np.float32)
    return x, t, theta, m, v


def _sliced_inputs(case, seed):
    rng = _rng(seed, 7)
    return [rng.integers(0, case["p"], size=(case["nvec"], case["nsym"]), dtype=np.uint8) for _ in range(2)]


def _to(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


class _Served:
    """A server that a program keeps running between bursts."""

    def __init__(self, case):
        predicted = case["policy"] == "predicted"
        self.server = bz.Server(policy=case["policy"], mlp_params=predictor.load()[0] if predicted else None,
                                slots=case["count"], max_n=2 * case["k_hi"])

    def __del__(self):
        self.server.stop()


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "plain":
        codes = _plain_codes(case, seed)
        st["codes"] = codes if case["host"] else [_to(G) for G in codes]
        st["options"] = bz.bz_default_options()
        st["options"].check = bz.CHECK_ROUND if case["check"] == "round" else bz.CHECK_STAGE
    elif kind == "batch":
        codes = _mixed_codes(case, seed)
        st["options"] = bz.bz_default_batch_options()
        if case["device"]:
            st["buf"], st["descs"] = bz.pack_batch(codes, device=DEV)
            ops, st["options"].blocks_per_cu = autotune.load()
            for d in st["descs"]:
                d.sweep_ops = int(ops(d.p, autotune.words(d.p, d.n, d.k)))
        else:
            st["codes"] = codes
    elif kind == "serve":
        st["requests"] = _requests(case, seed)
        st["served"] = _Served(case)
    elif kind == "mlp":
        st["x"], st["t"], st["theta"], st["m"], st["v"] = (_to(a) for a in _mlp_inputs(case, seed))
        n = case["samples"]
        st["cache"] = torch.empty((n, 128), dtype=torch.float32, device=DEV)
        st["dz"] = torch.empty((n, 129), dtype=torch.float32, device=DEV)
        st["grad"] = torch.empty(predictor.NPARAM, dtype=torch.float32, device=DEV)
        st["loss"] = torch.empty(1, dtype=torch.float32, device=DEV)
        st["step"] = 300
    else:
        st["a"], st["b"] = (_to(a) for a in _sliced_inputs(case, seed))
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- one pass
# A bz_result up to the kernel times: the whole answer.  What follows (kernel
# times, info bits) tells how a run was carried out and is no part of it.
ANSWER_BYTES = bz.bz_result.decompose_ms.offset


def _bytes(r):
    return np.frombuffer(r, dtype=np.uint8, count=ANSWER_BYTES)


ROW = 6 + bz.MAX_M + 6 * bz.MAX_STAGES


def _row(r):
    """A result dict as one row of whole numbers (zeros behind the last stage)."""
    flat = [r["status"], r["d"], r["m"], r["terminated_by"], r["codewords_total"], len(r["stages"]), *r["ranks"]]
    for stage in r["stages"]:
        flat += stage
    row = np.zeros(ROW, dtype=np.int64)
    row[:len(flat)] = flat
    return row


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "plain":
        p = case["p"]
        if case["hist"]:
            out = []
            for G in state["codes"]:
                r = bz.min_distance(p, G, check=case["check"], no_termination=True, histograms=True)
                hist = np.zeros((bz.MAX_STAGES, r["hist"].shape[1]), dtype=np.uint64)
                hist[:len(r["hist"])] = r["hist"]
                out.append({"d": r["d"], "answer": _row(r), "hist": hist})
            return out
        fn = bz.bz_min_distance_noalloc if case["noalloc"] else bz.bz_min_distance_ex
        out = []
        for G in state["codes"]:
            st, r = fn(p, G, state["options"])
            out.append({"status": st, "d": r.d, "answer": _bytes(r)})
        return out
    if kind == "batch":
        if case["device"]:
            buf, descs = state["buf"], state["descs"]
        else:
            buf, descs = bz.pack_batch(state["codes"])
        st, res, _ = bz.bz_min_distance_batch(buf, descs, state["options"])
        if st != bz.OK:
            raise RuntimeError(bz.bz_status_str(st))
        return {"status": np.array([s for s, _ in res]), "d": np.array([r.d for _, r in res]),
                "answer": np.concatenate([_bytes(r) for _, r in res])}
    if kind == "serve":
        server = state["served"].server
        for tag, (p, G) in enumerate(state["requests"]):
            server.submit(p, G, tag)
        rows = [None] * len(state["requests"])
        left = len(rows)
        while left:
            for tag, r in server.poll():
                rows[tag] = _row(r)
                left -= 1
        return np.stack(rows)
    if kind == "mlp":
        s = state
        y = bz.bz_mlp_forward(s["theta"], s["x"], s["cache"])
        bz.bz_mlp_backward(s["theta"], s["x"], s["t"], y, s["cache"], s["dz"], s["grad"], s["loss"])
        s["step"] += 1
        bz.bz_mlp_adam(s["theta"], s["grad"], s["m"], s["v"], s["step"], 3e-3)
        return {"y": y, "loss": s["loss"], "grad": s["grad"], "theta": s["theta"], "m": s["m"], "v": s["v"]}
    enc = bz.ENC_KAT if case["op"] == "kat" else bz.ENC_NATURAL
    A = bz.bz_sliced_pack(case["p"], state["a"], encoding=enc)
    B = bz.bz_sliced_pack(case["p"], state["b"], encoding=enc)
    C = bz.bz_sliced_op(case["p"], SLICED[case["op"]], A, B, case["nsym"])
    return {"planes": C, "symbols": bz.bz_sliced_unpack(case["p"], C, case["nsym"], encoding=enc)}


# ---------------------------------------------------------------- what a pass cannot do without
def _combinations(p, n, k, check="stage", everything=False):
    """Combinations that Algorithm 6 evaluates on a random code: stages (g, j)
    until L >= d, d the Gilbert-Varshamov estimate of the minimum weight."""
    ranks = [k] * (n // k) + ([n % k] if n % k else [])
    m = len(ranks)
    if everything:
        return m * (p ** k - 1) // (p - 1)
    log_words = math.log((p - 1)) + (n - k) * math.log(p)
    d, acc = 0, 0
    while d < n and (acc == 0 or math.log(acc) < log_words):
        d += 1
        acc += math.comb(n, d) * (p - 1) ** d
    d = min(d, n - k + 1)
    c = lambda g, kj: max(0, g + 1 - (k - kj))
    total = 0
    for g in range(1, k + 1):
        for j in range(1, m + 1):
            total += math.comb(k, g) * (p - 1) ** (g - 1)
            L = sum(c(g if i < j else g - 1, r) for i, r in enumerate(ranks))
            if L >= d and (check == "stage" or j == m):
                return total
    return total


def _code_work(p, n, k, check="stage", hist=False):
    """Bytes: the generator read, the result written.  Operations: a weight of
    n - k symbols per combination from bit planes (two boolean operations over
    F_3, three over F_7, and a popcount per word; one minimum)."""
    W = max((n - k + 31) // 32, 1)
    ops = 3 * W + 1 if p == 3 else 4 * W + 1
    c = _combinations(p, n, k, check, everything=hist)
    return k * n + ctypes.sizeof(bz.bz_result), c * ops


def _expected_mixed(case):
    """Sum of _code_work over an average draw of the mixed batch."""
    nb = nf = 0.0
    for p in (3, 7):
        cells = [(n, n // 2 if half else n // 3) for n in range(case["n_lo"], case["n_hi"] + 1) for half in (1, 0)
                 if p == 3 or n <= (case["f7_half"] if half else case["f7_third"])]
        cnt = case["count"] // 2 if p == 3 else case["count"] - case["count"] // 2
        for n, k in cells:
            b, f = _code_work(p, n, k)
            nb += cnt * b / len(cells)
            nf += cnt * f / len(cells)
    return nb, nf


def work(case):
    kind = case["kind"]
    if kind == "plain":
        b, f = _code_work(case["p"], case["n"], case["k"], case["check"], case["hist"])
        return {"bytes": float(b * case["codes"]), "flops": float(f * case["codes"])}
    if kind == "batch":
        b, f = _expected_mixed(case)
        return {"bytes": b, "flops": f}
    if kind == "serve":
        nb = nf = 0.0
        for p in (3, 7):
            ks = range(case["k_lo"], (case["k_hi"] if p == 3 else min(case["k_hi"], case["f7_kmax"])) + 1)
            for k in ks:
                b, f = _code_work(p, 2 * k, k)
                nb += case["count"] * b / 2 / len(ks)
                nf += case["count"] * f / 2 / len(ks)
        return {"bytes": nb, "flops": nf}
    if kind == "mlp":
        n, q = case["samples"], predictor.NPARAM
        # x and t read, y written; parameters and both moments read and written, the gradient written
        return {"bytes": 4.0 * (6 * n + 7 * q), "flops": 6.0 * n * (4 * 64 + 64 * 64 + 64)}
    planes = 2 if case["p"] == 3 else 3
    words = case["nvec"] * ((case["nsym"] + 31) // 32)
    operands = 1 if case["op"] == "double" else 2
    # symbols read, the result's planes and symbols written
    return {"bytes": float((operands + 1) * case["nvec"] * case["nsym"] + 4 * planes * words),
            "flops": float((9 if case["p"] == 3 else 22) * words)}


# ---------------------------------------------------------------- the same outputs in plain numpy, 64 bits
def exact(case, seed):
    kind = case["kind"]
    if kind == "plain" and case["p"] ** case["k"] <= 200000:
        out = []
        for G in _plain_codes(case, seed):
            if _rank(G, case["p"]) < case["k"]:
                return None
            r = {"d": _brute_force(G, case["p"]), "answer": None}
            r.update({"hist": None} if case["hist"] else {"status": 0})
            out.append(r)
        return out
    if kind == "mlp":
        return _exact_mlp(*_mlp_inputs(case, seed))
    if kind == "sliced":
        a, b = (s.astype(np.int64) for s in _sliced_inputs(case, seed))
        p = case["p"]
        c = {"add": a + b, "kat": a + b, "sub": a - b, "double": 2 * a}[case["op"]] % p
        return {"planes": None, "symbols": c.astype(np.uint8)}
    return None


def _rank(G, p):
    M, r = G.astype(np.int64) % p, 0
    for c in range(M.shape[1]):
        piv = np.nonzero(M[r:, c])[0]
        if piv.size == 0:
            continue
        M[[r, r + piv[0]]] = M[[r + piv[0], r]]
        M[r] = M[r] * pow(int(M[r, c]), -1, p) % p
        for i in range(M.shape[0]):
            if i != r:
                M[i] = (M[i] - M[i, c] * M[r]) % p
        r += 1
        if r == M.shape[0]:
            break
    return r


def _brute_force(G, p):
    """The smallest weight of a nonzero combination of the rows."""
    words = np.zeros((1, G.shape[1]), dtype=np.int64)
    for row in G.astype(np.int64):
        words = np.concatenate([(words + h * row) % p for h in range(p)])
    return int((words[1:] != 0).sum(axis=1).min())


def _exact_mlp(x, t, theta, m, v, step=301, lr=3e-3, b1=0.9, b2=0.999, eps=1e-8):
    x, t, theta, m, v = (a.astype(np.float64) for a in (x, t, theta, m, v))
    # the step's scalars are handed over in 32 bits
    lr, b1, b2, eps = (float(np.float32(s)) for s in (lr, b1, b2, eps))
    W1, c1 = theta[:256].reshape(64, 4), theta[256:320]
    W2, c2 = theta[320:4416].reshape(64, 64), theta[4416:4480]
    w3, c3 = theta[4480:4544], theta[4544]
    h1 = np.maximum(x @ W1.T + c1, 0)
    h2 = np.maximum(h1 @ W2.T + c2, 0)
    y = h2 @ w3 + c3
    dy = 2 * (y - t) / len(t)
    d2 = np.where(h2 > 0, dy[:, None] * w3, 0)
    d1 = np.where(h1 > 0, d2 @ W2, 0)
    grad = np.concatenate([(d1.T @ x).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), h2.T @ dy, [dy.sum()]])
    m = b1 * m + (1 - b1) * grad
    v = b2 * v + (1 - b2) * grad ** 2
    theta = theta - lr * (m / (1 - b1 ** step)) / (np.sqrt(v / (1 - b2 ** step)) + eps)
    return {"y": y, "loss": np.array([np.mean((y - t) ** 2)]), "grad": grad, "theta": theta, "m": m, "v": v}
