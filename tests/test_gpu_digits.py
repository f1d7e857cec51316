"""The bucket-space product on 8-bit digits: small-integer operands are exact in it, so sketches
equal the oracle's bit for bit - at its smallest sizes, ragged tiles and k-steps, several and
single slices - also where rows of the factors do not fit the digits (an entry in a channel that is
empty elsewhere, infinities, NaN) and their tiles run on the FP64 matrix cores beside it.  Operands
with channels of different scale lose nothing against the FP64 product."""
import numpy as np
import pytest

from oracle import fpsketch_oracle as o
from gpu_util import gemm_f32, int_case, to_dev_f32, to_dev_half
from paper_2609_19758_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fk():
    from paper_2609_19758_amd import fpsketch
    fpsketch.load()
    return fpsketch


def _reference(E, hr, m):
    X = np.zeros((m, E.shape[1]))
    np.add.at(X, hr.h1, hr.v1[:, None] * E)
    S = np.zeros((m, m))
    np.add.at(S.T, hr.h2, (X * hr.v2).T)
    return S


def _sketch(fk, a_bits, b_bits, c, m, layout, fmt="fp16"):
    n1, n2 = a_bits.shape
    n3 = b_bits.shape[1]
    v = fk.Verifier(n1, n2, n3, fmt, m=8, b_layout=layout)
    W = np.ascontiguousarray(b_bits.T) if layout else b_bits
    S = v.sketch(to_dev_half(a_bits, fmt), to_dev_half(W, fmt), to_dev_f32(c), seed=4, rnd=1, m=m,
                 moments=False)[0]
    v.close()
    return S


# m around tile edges with m^2 n2 >= 2^28 (some stay on the FP64 cores: below 2.75 x 2^28 at
# n2 < 4096, and m <= 256); n2 off the 32-k steps, odd and even step counts, slices
SIZES = [(400, 1700, 300, 400), (300, 1030, 520, 512), (260, 1025, 260, 513), (200, 800, 90, 641),
         (500, 513, 333, 769), (90, 520, 700, 1100), (700, 4800, 300, 241), (64, 512, 64, 2050),
         (400, 1700, 300, 700), (300, 1030, 520, 896), (260, 1025, 260, 897), (200, 800, 90, 1025),
         (500, 513, 333, 1281), (90, 4100, 700, 257), (700, 4800, 300, 385), (120, 4099, 300, 300),
         (40, 17001, 50, 300)]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n1,n2,n3,m", SIZES)
def test_exact(fk, n1, n2, n3, m, layout):
    assert m * m * n2 >= 2 ** 28
    a_bits, b_bits, a64, b64, c = int_case(n1, n2, n3, "fp16", m)
    rng = np.random.default_rng(m)
    c += rng.integers(-3, 4, size=c.shape).astype(np.float32)
    S = _sketch(fk, a_bits, b_bits, c, m, layout)
    assert np.array_equal(S, _reference(a64 @ b64 - c, o.make_round(4, 1, n1, n3, m), m))


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("side", ["A", "B", "both", "all rows"])
@pytest.mark.parametrize("m", [520, 900])
def test_rows_without_digits(fk, side, layout, m):
    """Some rows of A (columns of B) hold one entry of 30000 beside integers of at most 4, or all of
    them do in one channel."""
    n1, n2, n3 = 300, 1040, 280
    a_bits, b_bits, a64, b64, _ = int_case(n1, n2, n3, "fp16", 9)
    a, b = a64.copy(), b64.copy()
    if side in ("A", "both"):
        a[[3, 150], [7, 900]] = 30000.0
    if side in ("B", "both"):
        b[[5, 1000], [0, 277]] = -30000.0
    if side == "all rows":
        a[:, 11] = 30000.0
    # C is A B rounded to a multiple of 1024, exact in FP32
    c = (np.round(a @ b / 1024.0) * 1024.0).astype(np.float32)
    bits = [wl.f32_to_f16_bits(x.astype(np.float32)) for x in (a, b)]
    S = _sketch(fk, bits[0], bits[1], c, m, layout)
    assert np.array_equal(S, _reference(a @ b - c.astype(np.float64), o.make_round(4, 1, n1, n3, m), m))


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("side", [0, 1])
def test_rows_in_a_channel_without_a_size(fk, side, layout):
    """Channels that hold zeros in every sampled bucket of one factor (i m / 64) and entries in a few
    others: those rows take no part, their tiles run on the FP64 cores beside the digits'."""
    n1, n2, n3, m = 300, 1040, 280, 900
    a_bits, b_bits, a64, b64, _ = int_case(n1, n2, n3, "fp16", 9)
    hr = o.make_round(4, 1, n1, n3, m)
    sampled = {i * m // 64 for i in range(64)}
    h = hr.h1 if side == 0 else hr.h2
    free = [int(i) for i in range(len(h)) if int(h[i]) not in sampled]
    x = a64.copy() if side == 0 else b64.T.copy()      # rows of the factor's side
    x[:, [17, 600, 601, 1039]] = 0.0
    for i, k, val in [(free[0], 17, 2048.0), (free[3], 600, -3.0), (free[-1], 1039, 1.0)]:
        x[i, k] = val
    a, b = (x, b64) if side == 0 else (a64, x.T)
    c = (a @ b).astype(np.float32)
    rng = np.random.default_rng(5)
    c += rng.integers(-3, 4, size=c.shape).astype(np.float32)
    bits = [wl.f32_to_f16_bits(np.ascontiguousarray(v, dtype=np.float32)) for v in (a, b)]
    S = _sketch(fk, bits[0], bits[1], c, m, layout)
    assert np.array_equal(S, _reference(a @ b - c.astype(np.float64), hr, m))


def _scaled_case(n1, n2, n3, fmt, inverse, channels, outlier, seed):
    """Normal operands; half of the channels scaled by `inverse` in A and the others in B, and
    `channels` of A scaled by `outlier`.  On the GPU, with the black-box product."""
    import torch
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 0.02), seed)
    dt = torch.bfloat16 if fmt == "bf16" else torch.float16
    A, B = to_dev_half(a_bits, fmt).float(), to_dev_half(b_bits, fmt).float()
    order = torch.from_numpy(np.random.default_rng(seed).permutation(n2)).to(A.device)
    A[:, order[:n2 // 2]] *= inverse
    B[order[n2 // 2:]] *= inverse
    A[:, order[:channels]] *= outlier
    A, B = A.to(dt), B.to(dt)
    return A, B, gemm_f32(A, B)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("side", [0, 1])
def test_huge_entry_in_a_rare_channel(fk, side, layout):
    """An entry of 2^40 in a channel that one row of the other factor holds (in a sampled bucket,
    i m / 64): the rest of its row, 2^-40 of it, is in no digit, so the row must take no part."""
    n1, n2, n3, m = 400, 4100, 380, 300
    a_bits, b_bits, a64, b64, _ = int_case(n1, n2, n3, "bf16", 9)
    hr = o.make_round(4, 1, n1, n3, m)
    sampled = {i * m // 64 for i in range(64)}
    x, y, h = (a64.copy(), b64.copy().T, hr.h2) if side == 0 else (b64.copy().T, a64.copy(), hr.h1)
    holder = next(j for j in range(len(h)) if int(h[j]) in sampled)
    y[:, 5] = 0.0
    y[holder, 5] = 1.0
    x[11, 5] = 2.0 ** 40
    a, b = (x, y.T) if side == 0 else (y, x.T)
    c = (a @ b).astype(np.float32)
    bits = [wl.f32_to_bf16_bits(np.ascontiguousarray(v, dtype=np.float32)) for v in (a, b)]
    S = _sketch(fk, bits[0], bits[1], c, m, layout, fmt="bf16")
    assert np.array_equal(S, _reference(a @ b - c.astype(np.float64), hr, m))


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("side", [0, 1])
def test_no_tile_of_digits(fk, side, layout):
    """One factor's every 64 rows hold one that takes no part (a single entry of 30000 in a channel of
    its own): no tile is on the digits, in a grid whose last 128 rows are less than half full."""
    n1, n2, n3, m = 400, 4800, 400, 280
    a_bits, b_bits, a64, b64, _ = int_case(n1, n2, n3, "fp16", 9)
    x = a64.copy() if side == 0 else b64.T.copy()
    x[np.arange(400), 11 * np.arange(400)] = 30000.0
    a, b = (x, b64) if side == 0 else (a64, x.T)
    c = (np.round(a @ b / 1024.0) * 1024.0).astype(np.float32)
    bits = [wl.f32_to_f16_bits(np.ascontiguousarray(v, dtype=np.float32)) for v in (a, b)]
    S = _sketch(fk, bits[0], bits[1], c, m, layout)
    ref = _reference(a @ b - c.astype(np.float64), o.make_round(4, 1, n1, n3, m), m)
    assert np.array_equal(S, ref)


def _signs(h, v, m):
    """H1 or H2 in 64 bits on the GPU."""
    import torch
    H = torch.zeros(m, len(h), dtype=torch.float64, device="cuda")
    H[torch.from_numpy(np.asarray(h, dtype=np.int64)).cuda(), torch.arange(len(h), device="cuda")] = \
        torch.from_numpy(np.asarray(v, dtype=np.float64)).cuda()
    return H


def _exact_sums(hr, m, A, B, C):
    """S in 64 bits."""
    H1, H2 = _signs(hr.h1, hr.v1, m), _signs(hr.h2, hr.v2, m).T.contiguous()
    return (H1 @ A.double()) @ (B.double() @ H2) - (H1 @ C.double()) @ H2


SCALES = [("bf16", 1.0, 0, 1.0), ("bf16", 1e-2, 0, 1.0), ("bf16", 1e-3, 0, 1.0), ("bf16", 1e-4, 0, 1.0),
          ("bf16", 1e-5, 0, 1.0), ("bf16", 1e-6, 0, 1.0), ("fp16", 1e-2, 0, 1.0), ("fp16", 1e-3, 0, 1.0),
          ("bf16", 1.0, 1, 30.0), ("bf16", 1.0, 6, 30.0), ("fp16", 1.0, 6, 1000.0), ("bf16", 1e-3, 6, 1e4)]


@pytest.mark.parametrize("m", [260, 1000])
@pytest.mark.parametrize("fmt,inverse,channels,outlier", SCALES)
def test_channel_scales(fk, fmt, inverse, channels, outlier, m):
    """Channels of different scale: a row at the edge of taking part adds 4/15 of the mean square
    that rounding the factors to FP32 costs (a relative 2^-25.35 of each product), the Gaussian rows
    here 200 times less, so the error of S against 64 bits is within 1.1 of that of the FP64 product,
    which the sketch with moments takes for its S (its FP32 sums of a few entries are others).  Where
    a few channels hold nearly all of the product their sums of a few half-precision values are exact
    in FP32: the FP64 product's error is then far below that rounding, and the digits' share of the
    rounding is the bound."""
    n1, n2, n3 = 2048, 4096, 2048
    A, B, C = _scaled_case(n1, n2, n3, fmt, inverse, channels, outlier, 8)
    hr = o.make_round(4, 1, n1, n3, m)
    ref = _exact_sums(hr, m, A, B, C).cpu().numpy()
    v = fk.Verifier(n1, n2, n3, fmt, m=8)
    err = [np.sqrt(np.mean((v.sketch(A, B, C, seed=4, rnd=1, m=m, moments=mom)[0] - ref) ** 2))
           for mom in (False, True)]
    v.close()
    share = 0.0
    if channels:
        P, Q = _signs(hr.h1, hr.v1, m) @ A.double(), B.double() @ _signs(hr.h2, hr.v2, m).T.contiguous()
        share = float((P.pow(2).mean(0) @ Q.pow(2).mean(1) * 4 / 15).sqrt()) * 2.0 ** -25.35
    assert err[0] <= 1.1 * err[1] + share
    assert err[1] <= 0.02 * np.std(ref)          # (it is a small share of the noise)


@pytest.mark.parametrize("inverse", [1.0, 1e-3, 1e-6])
def test_fault_in_scaled_channels(fk, inverse):
    """The probe's noise is that of S in 64 bits, and an error of 0.02 rms(C) is found, as it is
    there."""
    n1, n2, n3, fmt, m = 2048, 4096, 2048, "bf16", 260
    A, B, C = _scaled_case(n1, n2, n3, fmt, inverse, 0, 1.0, 8)
    v = fk.Verifier(n1, n2, n3, fmt, m=m)
    hr = o.make_round(v.params.seed, 0, n1, n3, m)
    S = _exact_sums(hr, m, A, B, C).abs().cpu().numpy()
    v.probe(A, B, C)
    clean = v.probe_stats()
    want = 1.2533 * np.mean(np.minimum(S, 5 * np.mean(S)))
    assert not clean["dirty"] and abs(clean["sigma_hat"] - want) <= 1e-3 * want
    C[700, 900] += 0.02 * float(C.double().pow(2).mean().sqrt())
    v.probe(A, B, C)
    stats = v.probe_stats()
    v.close()
    S = _exact_sums(hr, m, A, B, C).abs().cpu().numpy()
    assert S.max() > 1.5 * stats["thr"] and stats["dirty"]
    assert abs(stats["max_abs"] - S.max()) <= 1e-3 * S.max()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("m", [520, 900])
def test_non_finite_rows(fk, bad, m):
    n1, n2, n3 = 300, 1040, 280
    a_bits, b_bits, a64, b64, c = int_case(n1, n2, n3, "fp16", 9)
    a = a64.astype(np.float32)
    a[42, 77] = bad
    hr = o.make_round(4, 1, n1, n3, m)
    S = _sketch(fk, wl.f32_to_f16_bits(a), b_bits, c, m, 0)
    ref = _reference(a64 @ b64 - c, hr, m)
    row = hr.h1[42]
    others = np.arange(m) != row
    assert np.array_equal(S[others], ref[others])
    # 0 x inf is NaN, and so is every bucket of that row
    assert not np.isfinite(S[row]).any()


@pytest.mark.parametrize("n1,n2,n3,m,fmt", [(3000, 1600, 2900, 700, "bf16"), (2000, 4100, 2500, 300, "fp16")])
def test_float_operands(fk, n1, n2, n3, m, fmt):
    """Float operands against the definition: within the bound every float sketch has (FP32 storage
    of the factors, 2^-20 of the bucket's absolute contributions), and far below the noise."""
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 0.02), 8)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    C = gemm_f32(A, B)
    v = fk.Verifier(n1, n2, n3, fmt, m=8)
    S = v.sketch(A, B, C, seed=4, rnd=1, m=m, moments=False)[0]
    a64, b64 = o.decode(a_bits, fmt), o.decode(b_bits, fmt)
    ref = _reference(a64 @ b64 - C.cpu().numpy().astype(np.float64), o.make_round(4, 1, n1, n3, m), m)
    v.close()
    hr = o.make_round(4, 1, n1, n3, m)
    D = o.abs_contributions(a64, b64, C.cpu().numpy(), hr)[0]
    assert (np.abs(S - ref) <= 2.0 ** -20 * D + 1e-300).all()
    assert np.std(S - ref) <= 0.05 * np.std(ref)


@pytest.mark.parametrize("n1,n2,n3,m", [(600, 4100, 500, 300), (900, 1100, 700, 1100),
                                        (500, 300, 400, 1500)])
def test_capture(fk, n1, n2, n3, m):
    """Probes on the digit product and on the work-groups for more than 1024 buckets, captured in a
    graph and replayed between eager calls, give the eager statistics."""
    import torch
    fmt = "bf16"
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 0.02), 8)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    C = gemm_f32(A, B)
    D = C.clone()
    D[n1 // 2, n3 // 3] += 50.0
    v = fk.Verifier(n1, n2, n3, fmt, m=m)
    v.probe(A, B, C)
    clean = v.probe_stats()
    v.probe(A, B, D)
    dirty = v.probe_stats()
    # With m > n1 most buckets are empty (73% and 93% here), the mean-based noise estimate is low and
    # the clean product exceeds its threshold (2.4 and 29 times, 0.5 times at m = 300): the oracle's
    # decision is the one to meet.
    ref = o.probe(wl.half_bits_to_f32(a_bits, fmt).astype(np.float64),
                  wl.half_bits_to_f32(b_bits, fmt).astype(np.float64), C.cpu().numpy(),
                  o.make_round(v.params.seed, 0, n1, n3, m), o.Params())
    assert bool(clean["dirty"]) == ref.dirty == (m > n1) and dirty["dirty"]
    assert dirty["max_abs"] > 2 * clean["max_abs"]
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    g, cap = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    cap.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(cap):
        with torch.cuda.graph(g, stream=cap):
            v.probe(A, B, D, d_dirty=flag)
    torch.cuda.synchronize()
    for _ in range(3):
        flag.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert int(flag.item()) == 1 and v.probe_stats() == dirty
        v.probe(A, B, C)
        assert v.probe_stats() == clean
    v.close()
