"""The bucket-space product on 8-bit digits: small-integer operands are exact in it, so sketches
equal the oracle's bit for bit - at its smallest sizes, ragged tiles and k-steps, several and
single slices - also where rows of the factors do not fit the digits (one entry far above the
rest, infinities, NaN) and their tiles run on the FP64 matrix cores beside it."""
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


# m around tile edges with m^2 n2 >= 2^28; n2 off the 32-k steps, odd and even step counts, slices
SIZES = [(400, 1700, 300, 400), (300, 1030, 520, 512), (260, 1025, 260, 513), (200, 800, 90, 641),
         (500, 513, 333, 769), (90, 520, 700, 1100), (700, 4800, 300, 241), (64, 512, 64, 2050)]


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
def test_rows_without_digits(fk, side, layout):
    """Some rows of A (columns of B) hold one entry of 30000 beside integers of at most 4: their
    buckets' factor rows go to the FP64 tiles, the others stay."""
    n1, n2, n3, m = 300, 1040, 280, 520
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


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_non_finite_rows(fk, bad):
    n1, n2, n3, m = 300, 1040, 280, 520
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
