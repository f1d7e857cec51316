"""The verifier's performance cases: what a program that uses it calls, over the sizes it meets.

Each case is one pass through the public entry points of ``paper_2609_19758_amd.fpsketch`` on
operands that are already on the GPU, with the product C made by the black-box GEMM.  Kinds:

  probe      ``calls`` products verified one after another, the verdicts ORed into a device flag
             each and the statistics of the last one read: the check after a GEMM.
  deferred   the same through the pipelined probe, then the flush.
  cached     the B side (a weight) formed once beforehand, the probe streams A and C only.
  localize   a dirty product: probe, then localization with the noise of that probe
             (``fresh``: localization alone, which measures its own noise).
  apply      the repair step: records written into C, then the re-probe with a fresh hash round.
  calibrate  the periodic recalibration of the bucket count after some clean probes.

``exact`` restates the method in 64-bit torch and numpy: the splitmix64 hash, bucket sums of
E = AB - C, and the decision.
"""
import math

import numpy as np
import torch

from paper_2609_19758_amd import fpsketch as fk

GAMMA = 0x9E3779B97F4A7C15
CTX_SEED = 0x5EED5EED             # the context seed of default_params
EPS = 2.0 ** -23


# ---------------------------------------------------------------------------------------------
# Cases.


def bucket_count(n1, n2, n3, fmt):
    """The probe's bucket count a calibrated program arrives at: Eq. 4-5 with the noise constant
    measured for this GPU's GEMM, between the combinatorial floor 48 and the kernels' 4096."""
    cf = 0.1050 if fmt == "bf16" else 0.1073
    v = max(n1, n3) / 0.3 * cf * 2.0 ** -24 * math.sqrt(float(n1) * n3 * n2)
    return min(max(48, math.ceil(v)), 4096)


def _case(kind, n1, n2, n3, fmt, **kw):
    c = {"kind": kind, "n1": n1, "n2": n2, "n3": n3, "fmt": fmt,
         "m": bucket_count(n1, n2, n3, fmt), "calls": 1, "b_layout": 0, "faults": 0,
         "huge": 0, "fresh": False, "uniform": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest product of the test workloads: launches and latency
        _case("probe", 256, 256, 256, "fp16", m=64, uniform=True, name="probe_256_fp16"),
        # the headline product, four layers' operands in turn as in a training step
        _case("probe", 4096, 4096, 4096, "bf16", calls=4, name="probe_4096_bf16"),
        # prefill of a ragged batch through a fused projection: more buckets than the block path
        _case("probe", 2048, 4096, 12288, "bf16", m=80, name="probe_2048x4096x12288_bf16"),
        # an output head: a token count and a vocabulary that are no multiple of anything
        _case("probe", 1531, 4096, 32003, "fp16", name="probe_1531x4096x32003_fp16"),
        # the largest product of the paper's evaluation
        _case("probe", 16384, 16384, 16384, "fp16", m=698, uniform=True,
              name="probe_16384_fp16"),
        # an MLP down projection, four calls through the pipelined probe and its flush
        _case("deferred", 4096, 11008, 4096, "bf16", calls=4,
              name="deferred_4096x11008x4096_bf16"),
        # decode: 64 tokens against a linear layer's weight whose side is cached
        _case("cached", 64, 8192, 8192, "fp16", b_layout=1, name="cached_64x8192x8192_fp16"),
        # fault recovery on the headline product: eight small additive errors
        _case("localize", 4096, 4096, 4096, "bf16", faults=8, name="localize_4096_bf16"),
        # recovery without a probe's noise at hand, on an odd shape, with out-of-range entries
        _case("localize", 641, 1023, 770, "fp16", faults=4, huge=2, fresh=True,
              name="localize_641x1023x770_fp16"),
        # recovery on the largest product: thousands of localization buckets
        _case("localize", 16384, 16384, 16384, "fp16", m=698, faults=16, uniform=True,
              name="localize_16384_fp16"),
        # the repair step of a transformer projection: recomputed entries written, C re-probed
        _case("apply", 2048, 5120, 5120, "fp16", huge=8, name="apply_2048x5120x5120_fp16"),
        # the periodic recalibration of a square projection's bucket count
        _case("calibrate", 2048, 8192, 8192, "bf16", m=64,
              name="calibrate_2048x8192x8192_bf16"),
    ]


def _size(rng, lo, hi):
    """A dimension spread over the logarithm of its range: as a model has it (a multiple of 128)
    half of the time, else any integer."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and v >= 128:
        v = v // 128 * 128
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["probe", "probe", "probe", "deferred", "cached", "localize", "localize",
                       "apply", "calibrate"])
    fmt = rng.choice(["bf16", "fp16"])
    hi = 9000 if kind in ("localize", "calibrate") else 13824
    n1 = _size(rng, 16 if kind in ("probe", "cached", "deferred") else 256, hi)
    n2 = _size(rng, 128, hi)
    n3 = _size(rng, 256, 32768 if kind == "probe" else hi)
    kw = {"b_layout": 1 if rng.random() < 0.3 else 0}
    if kind == "deferred":
        kw["calls"] = rng.randint(2, 4)
    if kind == "localize":
        kw["faults"] = rng.randint(1, 8)
        kw["huge"] = rng.randint(0, 2)
        kw["fresh"] = rng.random() < 0.5
    if kind == "apply":
        kw["huge"] = rng.randint(1, 16)
    return _case(kind, n1, n2, n3, fmt, **kw)


def work(case):
    n1, n2, n3, m = case["n1"], case["n2"], case["n3"], case["m"]
    a, b, c = 2.0 * n1 * n2, 2.0 * n2 * n3, 4.0 * n1 * n3
    product = 2.0 * m * m * n2
    sums = float(n1) * n2 + float(n2) * n3 + float(n1) * n3
    kind, k = case["kind"], case["calls"]
    if kind in ("probe", "deferred"):
        return {"bytes": k * (a + b + c), "flops": k * (product + sums)}
    if kind == "cached":       # A, C and the cached FP32 sketch of the weight
        return {"bytes": a + c + 4.0 * m * n2, "flops": product + sums - float(n2) * n3}
    if kind == "localize":     # three hash rounds of one C, A and B
        return {"bytes": a + b + c, "flops": 3.0 * (product + sums)}
    if kind == "apply":
        return {"bytes": a + b + c, "flops": product + sums}
    samples = min(n1 * n3, 65536)
    return {"bytes": 4.0 * samples, "flops": 4.0 * samples}     # calibrate: rms-hat's samples


def tolerance(case):
    """The probe's statistics are sums of rounding noise: FP32 group sums in another order move
    them by a little of that noise (largest seen against 64 bits: max|S| 0.9 %, sigma-hat
    0.3 %).  Records and repaired entries are FP64 recomputations, rounded once to FP32 in C."""
    if case["kind"] in ("apply", "localize"):
        return {"rel": 1e-6}
    return {"rel": 1e-2 if case["kind"] == "calibrate" else 4e-2}


# ---------------------------------------------------------------------------------------------
# Inputs.


def _half(fmt):
    return torch.bfloat16 if fmt == "bf16" else torch.float16


def _operands(case, seed):
    """(A, B as stored, C, rng) of each call: activations N(0, 1) against weights N(0, 0.02), or
    U[-1, 1] squares; C is the FP32 product of the black-box GEMM."""
    n1, n2, n3, h = case["n1"], case["n2"], case["n3"], _half(case["fmt"])
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)

    def mat(r, c, std):
        if case["uniform"]:
            return torch.rand(r, c, generator=g, device="cuda").mul_(2).sub_(1).to(h)
        return torch.randn(r, c, generator=g, device="cuda").mul_(std).to(h)

    sets = []
    for _ in range(case["calls"]):
        A = mat(n1, n2, 1.0)
        B = mat(n3, n2, 0.02) if case["b_layout"] else mat(n2, n3, 0.02)
        C = torch.mm(A, B.t() if case["b_layout"] else B, out_dtype=torch.float32)
        sets.append((A, B, C))
    return sets


def _column(B, j, layout):
    return B[j] if layout else B[:, j]


def _sites(case, seed):
    """Distinct coordinates of the faults, no two of them in one row or column."""
    rng = np.random.default_rng([seed, 0xF])
    n = case["faults"] + case["huge"]
    i = rng.choice(case["n1"], size=n, replace=False)
    j = rng.choice(case["n3"], size=n, replace=False)
    return [(int(a), int(b)) for a, b in zip(i, j)]


def _inject(case, C, seed):
    """Writes the faults of a dirty product into C: additive errors of 0.2 to 4 times mean |C|,
    and exponent-bit upsets that leave an entry infinite or far out of range."""
    rng = np.random.default_rng([seed, 0xD])
    sites = _sites(case, seed)
    unit = float(C.abs().mean())
    for t, (i, j) in enumerate(sites):
        if t < case["faults"]:
            mag = math.exp(rng.uniform(math.log(0.2), math.log(4.0))) * unit
            C[i, j] += mag if rng.random() < 0.5 else -mag
        else:
            C[i, j] = float("inf") if t % 2 else -3.0e38
    return sites


def _verifier(case):
    return fk.Verifier(case["n1"], case["n2"], case["n3"], case["fmt"], m=case["m"],
                       b_layout=case["b_layout"])


def prepare(case, seed):
    sets = _operands(case, seed)
    v = _verifier(case)
    st = {"case": case, "v": v, "sets": sets, "seed": 7919 * seed + 3,
          "flags": torch.zeros(case["calls"], dtype=torch.int32, device="cuda")}
    A, B, C = sets[0]
    kind = case["kind"]
    if kind == "cached":
        v.cache_b(B)
    elif kind == "localize":
        _inject(case, C, seed)
    elif kind == "apply":
        # records as localize returns them for out-of-range entries: recomputed values
        recs = []
        for i, j in _sites(case, seed):
            d = torch.dot(A[i].double(), _column(B, j, case["b_layout"]).double()).item()
            recs.append((i, j, d, True, 0))
        st["recs"] = recs
        for i, j, _, _, _ in recs:
            C[i, j] = float("inf")
    elif kind == "calibrate":
        for _ in range(3):
            v.probe(A, B, C)
    torch.cuda.synchronize()
    return st


def _stats(v):
    s = v.probe_stats()
    return {"sigma_hat": s["sigma_hat"], "thr": s["thr"], "tau": s["tau"],
            "max_abs": s["max_abs"], "finite": int(s["finite"]), "dirty": int(s["dirty"]),
            "max_a": s["max_a"], "max_b": s["max_b"]}


def _records(recs):
    """A fault log: the records in row-major order."""
    recs = sorted(recs)
    return {"coords": np.array([[r[0], r[1]] for r in recs], dtype=np.int64).reshape(-1, 2),
            "delta": np.array([r[2] for r in recs], dtype=np.float64),
            "absolute": np.array([int(r[3]) for r in recs], dtype=np.int64)}


def run(state):
    case, v, flags = state["case"], state["v"], state["flags"]
    kind = case["kind"]
    A, B, C = state["sets"][0]
    if kind == "probe":
        for t, (a, b, c) in enumerate(state["sets"]):
            v.probe(a, b, c, d_dirty=flags[t:t + 1])
        return {"flags": flags, **_stats(v)}
    if kind == "deferred":
        for t, (a, b, c) in enumerate(state["sets"]):
            v.probe_deferred(a, b, c, d_dirty=flags[t:t + 1])
        v.probe_flush()
        return {"flags": flags, **_stats(v)}
    if kind == "cached":
        v.probe_cached(A, C, d_dirty=flags)
        return {"flags": flags, **_stats(v)}
    if kind == "localize":
        out = {}
        if not case["fresh"]:
            v.probe(A, B, C, d_dirty=flags)
            out["flags"] = flags
        recs, _, _ = v.localize(A, B, C, seed=state["seed"], sigma_from_probe=not case["fresh"])
        out.update(_records(recs))
        plan = v.plan()
        out.update({k: plan[k] for k in ("m_loc", "r", "n_abs", "rms_hat", "tau")})
        return out
    if kind == "apply":
        dirty = v.apply(A, B, C, state["recs"], seed=state["seed"])
        return {"C": C, "still_dirty": int(dirty)}
    m, sigma_bar, rebuilt = v.calibrate_noise(C)
    return {"m": m, "sigma_bar": sigma_bar, "rebuilt": int(rebuilt)}


# ---------------------------------------------------------------------------------------------
# The same in 64 bits, from the definitions.


def _mix(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _hash(seed, rnd, side, n, m):
    """Bucket and sign of every index of one side of a hash round, on the GPU."""
    mask = (1 << 64) - 1
    with np.errstate(over="ignore"):
        key = _mix(np.array([(seed + (2 * rnd + side + 1) * GAMMA) & mask], dtype=np.uint64))[0]
        x = _mix(key + np.arange(1, n + 1, dtype=np.uint64) * np.uint64(GAMMA))
        bucket = ((x >> np.uint64(32)) * np.uint64(m)) >> np.uint64(32)
    sign = 1.0 - 2.0 * (x & np.uint64(1)).astype(np.float64)
    return (torch.from_numpy(bucket.astype(np.int64)).cuda(), torch.from_numpy(sign).cuda())


def _sketch64(case, A, B, C, seed):
    """S = H1 (AB - C) H2^T in 64 bits."""
    n1, n3, m = case["n1"], case["n3"], case["m"]
    h1, v1 = _hash(seed, 0, 0, n1, m)
    h2, v2 = _hash(seed, 0, 1, n3, m)
    b64 = B.double()
    E = torch.mm(A.double(), b64.t() if case["b_layout"] else b64)
    del b64
    E.sub_(C.double())
    X = torch.zeros(m, n3, dtype=torch.float64, device="cuda")
    X.index_add_(0, h1, E.mul_(v1[:, None]))
    del E
    S = torch.zeros(m, m, dtype=torch.float64, device="cuda")
    S.index_add_(1, h2, X.mul_(v2[None, :]))
    return S


def _decide64(case, A, B, S):
    m = case["m"]
    a = S.abs()
    finite = bool(torch.isfinite(S).all())
    clip = 5.0 * a.mean()
    sigma = 1.2533 * float(torch.minimum(a, clip).mean())
    max_a, max_b = float(A.abs().max().double()), float(B.abs().max().double())
    tau = 100.0 * case["n2"] * EPS * max_a * max_b
    thr = min(tau, 4.0 * math.sqrt(2.0 * math.log(float(m) * m)) * sigma)
    top = float(a.max())
    return {"sigma_hat": sigma, "thr": thr, "tau": tau, "max_abs": top, "finite": int(finite),
            "dirty": int(not (finite and top <= thr)), "max_a": max_a, "max_b": max_b}


def exact(case, seed):
    sets = _operands(case, seed)
    kind = case["kind"]
    if kind in ("probe", "deferred", "cached"):
        out = None
        flags = []
        for A, B, C in sets:
            out = _decide64(case, A, B, _sketch64(case, A, B, C, CTX_SEED))
            flags.append(out["dirty"])
        return {"flags": torch.tensor(flags, dtype=torch.int32, device="cuda"), **out}
    A, B, C = sets[0]
    layout = case["b_layout"]
    if kind == "localize":
        sites = _inject(case, C, seed)
        rows = []
        for t, (i, j) in enumerate(sites):
            ab = float(torch.dot(A[i].double(), _column(B, j, layout).double()))
            huge = t >= case["faults"]
            rows.append((i, j, ab if huge else ab - float(C[i, j]), huge, 0))
        out = {} if case["fresh"] else {"flags": torch.ones(1, dtype=torch.int32, device="cuda")}
        out.update(_records(rows))
        stride = max(1, C.numel() // 65536)
        s = C.reshape(-1)[::stride].double().abs()
        s = s[torch.isfinite(s)]
        half = s.numel() // 2
        o = torch.sort(s).values
        med = float(o[half]) if s.numel() % 2 else 0.5 * float(o[half - 1] + o[half])
        rms = math.sqrt(float(torch.clamp(s, max=64.0 * med).square().mean()))
        tau = 100.0 * case["n2"] * EPS * float(A.abs().max().double()) * float(B.abs().max().double())
        out.update({"m_loc": None, "r": None, "n_abs": case["huge"], "rms_hat": rms, "tau": tau})
        return out
    if kind == "apply":
        out = C.double()
        for i, j in _sites(case, seed):
            out[i, j] = torch.dot(A[i].double(), _column(B, j, layout).double())
        return {"C": out, "still_dirty": 0}
    sigma = _decide64(case, A, B, _sketch64(case, A, B, C, CTX_SEED))["sigma_hat"]
    return {"m": case["m"], "sigma_bar": sigma, "rebuilt": 0}
