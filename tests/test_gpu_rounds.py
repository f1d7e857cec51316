"""Hash-round tables built on the device and the recheck of whole search windows, at their edges:
lists and column tables through exact integer sketches (several row groups a wave, the widest
chunks, more than one of them, one bucket, both layouts), windows at corners of C and over each
other, both layouts, a ragged n2."""
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


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n1,n2,n3,m", [
    (9001, 8, 40, 1), (4097, 8, 520, 3), (70, 8, 16390, 2100), (40, 8, 33000, 4096),
    (513, 8, 8193, 1025), (100, 8, 4097, 512), (100, 8, 4095, 513), (3, 8, 5, 4096)])
def test_tables_through_exact_sketches(fk, n1, n2, n3, m, layout):
    a_bits, b_bits, a64, b64, c = int_case(n1, n2, n3, "bf16", 3)
    rng = np.random.default_rng(n1 + m)
    c += rng.integers(-2, 3, size=c.shape).astype(np.float32)
    E = a64 @ b64 - c
    A = to_dev_half(a_bits, "bf16")
    B = to_dev_half(np.ascontiguousarray(b_bits.T) if layout else b_bits, "bf16")
    v = fk.Verifier(n1, n2, n3, "bf16", m=8, b_layout=layout)
    hr = o.make_round(77, 2, n1, n3, m)
    X = np.zeros((m, n3))
    np.add.at(X, hr.h1, hr.v1[:, None] * E)
    ref = np.zeros((m, m))
    np.add.at(ref.T, hr.h2, (X * hr.v2).T)
    for moments in (False, True):
        S = v.sketch(A, B, to_dev_f32(c), seed=77, rnd=2, m=m, moments=moments)[0]
        assert np.array_equal(S, ref)
    v.close()


@pytest.mark.parametrize("n1,n3,m", [
    (150000, 40, 1025), (80000, 40, 1025), (40000, 520, 1030), (30000, 1500, 1100), (6000, 2100, 1030), (3000, 4096, 1300),
    (3000, 4097, 1025), (900, 8200, 1025)])
def test_wide_rows_shared_by_waves(fk, n1, n3, m):
    """More than 1024 buckets over few columns: 1, 2, 4, 8 and 16 column tiles a chunk (rounded up), so
    that 16 to 1 waves share a bucket's rows, several groups of 64 rows a bucket, a short last chunk."""
    n2, fmt = 3, "bf16"
    a_bits, b_bits, a64, b64, c = int_case(n1, n2, n3, fmt, 5)
    rng = np.random.default_rng(n1 + n3)
    c += rng.integers(-2, 3, size=c.shape).astype(np.float32)
    E = a64 @ b64 - c
    v = fk.Verifier(n1, n2, n3, fmt, m=8)
    hr = o.make_round(77, 2, n1, n3, m)
    X = np.zeros((m, n3))
    np.add.at(X, hr.h1, hr.v1[:, None] * E)
    ref = np.zeros((m, m))
    np.add.at(ref.T, hr.h2, (X * hr.v2).T)
    args = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt), to_dev_f32(c)
    assert np.array_equal(v.sketch(*args, seed=77, rnd=2, m=m, moments=False)[0], ref)
    S, R, _, _, _ = v.sketch(*args, seed=77, rnd=2, m=m, moments=True)
    v.close()
    Y = np.zeros((m, n3))
    np.add.at(Y, hr.h1, (hr.v1 * ((np.arange(n1) + 1) / o.pow2_ceil(n1)))[:, None] * E)
    refr = np.zeros((m, m))
    np.add.at(refr.T, hr.h2, (Y * hr.v2).T)
    assert np.array_equal(S, ref) and np.array_equal(R, refr)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n2", [5, 511, 1536])
@pytest.mark.parametrize("sites", [
    [(0, 0)], [(306, 402)], [(0, 402), (306, 0)], [(150, 200), (151, 203)],
    [(20, 30), (20, 33), (200, 300)]])
def test_windows(fk, layout, n2, sites):
    n1, n3, fmt, r = 307, 403, "bf16", 2
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 0.02), n2)
    A = to_dev_half(a_bits, fmt)
    W = to_dev_half(np.ascontiguousarray(b_bits.T) if layout else b_bits, fmt)
    c = gemm_f32(A, to_dev_half(b_bits, fmt)).cpu().numpy()
    for i, j in sites:
        c[i, j] += 4.0
    v = fk.Verifier(n1, n2, n3, fmt, m=64, b_layout=layout, rounds=1, r_star=r, r_max=r,
                    rho_min=1e-5)
    recs, n, _ = v.localize(A, W, to_dev_f32(c), seed=9, sigma_from_probe=False)
    plan = v.plan()
    v.close()
    assert plan["r"] == r
    a64, b64 = o.decode(a_bits, fmt), o.decode(b_bits, fmt)
    hr = o.make_round(9, 1, n1, n3, plan["m_loc"])
    buckets = [(hr.h1[i], hr.h2[j]) for i, j in sites]
    alone = [s for s, b in zip(sites, buckets) if buckets.count(b) == 1]
    got = {(i, j): d for i, j, d, _, _ in recs}
    assert set(got) >= set(alone) and set(got) <= set(sites)
    for (i, j), d in got.items():
        want = float(a64[i] @ b64[:, j]) - float(c[i, j])
        assert abs(d - want) <= 1e-12 * (abs(want) + np.abs(a64[i]) @ np.abs(b64[:, j]))
    if len(alone) == len(sites) and n2 > 100:     # (a near-exact product has MAD 0 and cut 0)
        # every coordinate of the sites' windows counted once (tau_d = n sigma / r leaves no others)
        union = {(i + a, j + b) for i, j in sites for a in range(-r, r + 1)
                 for b in range(-r, r + 1) if 0 <= i + a < n1 and 0 <= j + b < n3}
        assert plan["n_rechecked"] == len(union)


def test_many_faults_peeled(fk):
    """600 faults, more than the 512 entries that a peel takes at a time, several to a bucket: later
    rounds peel them from S, R and T, and every one is recovered at its value."""
    n1, n2, n3, fmt = 1024, 512, 1024, "bf16"
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 0.02), 4)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    c = gemm_f32(A, B).cpu().numpy()
    rng = np.random.default_rng(8)
    sites = rng.choice(n1 * n3, size=600, replace=False)
    c.reshape(-1)[sites] += rng.uniform(50.0, 60.0, size=600).astype(np.float32)
    v = fk.Verifier(n1, n2, n3, fmt, m=200, s_budget=600, k_cap=1024)
    C = to_dev_f32(c)
    v.probe(A, B, C)
    recs, n, _ = v.localize(A, B, C, seed=3, sigma_from_probe=True, cap=2048)
    v.close()
    assert sorted(i * n3 + j for i, j, _, _, _ in recs) == sorted(sites.tolist())
    assert max(r[4] for r in recs) > 1            # (some in a round that peeled others)
    a64, b64 = o.decode(a_bits, fmt), o.decode(b_bits, fmt)
    for i, j, d, _, _ in recs:
        want = float(a64[i] @ b64[:, j]) - float(c[i, j])
        assert abs(d - want) <= 1e-12 * (abs(want) + np.abs(a64[i]) @ np.abs(b64[:, j]))
