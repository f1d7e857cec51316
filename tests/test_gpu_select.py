"""Device order statistics of a localization: the noise of a fresh sketch (1.4826 x MAD, exact
selection: equal to numpy's on the same S) and rms-hat(C) (against the library's host rule and the
oracle's), where the selection changes form: one work-group or the chip, ties and clusters beyond
the kept keys, odd and even counts, samples that are not finite."""
import math

import numpy as np
import pytest

from oracle import fpsketch_oracle as o
from gpu_util import gemm_f32, to_dev_f32, to_dev_half
from paper_2609_19758_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fk():
    from paper_2609_19758_amd import fpsketch
    fpsketch.load()
    return fpsketch


def _mad(S):
    return 1.4826 * float(np.median(np.abs(S - np.median(S))))


def _fresh_sigma(fk, A, B, C, n1, n2, n3, fmt, m):
    v = fk.Verifier(n1, n2, n3, fmt, m=m)
    S = v.sketch(A, B, C, seed=21, rnd=0, m=m, moments=False)[0]
    v.localize(A, B, C, seed=21, sigma_from_probe=False)
    plan = v.plan()
    v.close()
    return plan, S


# grids of one and a few values, around one work-group's limit (128^2), above the kept keys' 2^16
@pytest.mark.parametrize("m", [1, 2, 3, 17, 127, 128, 129, 256, 257, 401])
def test_fresh_noise_equals_mad_of_sketch(fk, m):
    n1, n2, n3, fmt = 514, 96, 602, "bf16"
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 1.0), 5)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    plan, S = _fresh_sigma(fk, A, B, gemm_f32(A, B), n1, n2, n3, fmt, m)
    assert plan["sigma_hat"] == _mad(S)


@pytest.mark.parametrize("kind", ["zeros", "cluster", "mixed"])
def test_ties_and_clusters(fk, kind):
    """S set bucket by bucket through C: all zeros (one value, more than the kept keys), a cluster
    of values that share the first two digits (ditto), and both with outliers on each side."""
    n, m, fmt, n2 = 900, 301, "fp16", 8
    hr = o.make_round(21, 0, n, n, m)
    rng = np.random.default_rng(3)
    want = np.zeros((m, m))
    if kind != "zeros":
        want = 2.0 ** 21 + rng.integers(0, 256, size=(m, m))
    if kind == "mixed":
        want[rng.random((m, m)) < 0.2] = 0.0
        want[rng.random((m, m)) < 0.01] = -3.0
    C = np.zeros((n, n), dtype=np.float32)
    rows = [np.flatnonzero(hr.h1 == a) for a in range(m)]
    cols = [np.flatnonzero(hr.h2 == b) for b in range(m)]
    ra = [a for a in range(m) if rows[a].size]
    cb = [b for b in range(m) if cols[b].size]
    for a in ra:
        i = rows[a][0]
        for b in cb:
            j = cols[b][0]
            C[i, j] = -hr.v1[i] * hr.v2[j] * want[a, b]
    z = np.zeros((n, n2), dtype=np.uint16)
    A, B = to_dev_half(z, fmt), to_dev_half(np.ascontiguousarray(z.T), fmt)
    plan, S = _fresh_sigma(fk, A, B, to_dev_f32(C), n, n2, n, fmt, m)
    assert np.array_equal(S[np.ix_(ra, cb)], want[np.ix_(ra, cb)])
    assert plan["sigma_hat"] == _mad(S)


@pytest.mark.parametrize("n1,n3,bad", [(1, 1, 0), (1, 2, 1), (3, 5, 0), (255, 257, 3), (256, 256, 0),
                                       (257, 257, 7), (500, 1000, 1000), (40, 40, 1600)])
def test_rms_hat(fk, n1, n3, bad):
    rng = np.random.default_rng(n1 + n3)
    n2, fmt = 4, "bf16"
    c = (rng.standard_normal((n1, n3)) * 3.0).astype(np.float32)
    f = c.reshape(-1)
    f[rng.choice(f.size, size=f.size // 100, replace=False)] *= 1e6       # clipped at 64 x median
    idx = rng.choice(f.size, size=bad, replace=False)
    f[idx] = rng.choice(np.array([np.inf, -np.inf, np.nan], dtype=np.float32), size=bad)
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 1.0), 1)
    v = fk.Verifier(n1, n2, n3, fmt, m=4)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    for _ in range(2):                     # the second call finds the state the first one left
        v.localize(A, B, to_dev_f32(c), seed=2, sigma_from_probe=False)
        got = v.plan()["rms_hat"]
        want = o.rms_hat(c)
        host = fk.rms_hat_samples(f[::max(1, f.size // 65536)])
        if not np.isfinite(want):
            assert not np.isfinite(got) and not np.isfinite(host)
        else:
            # sums of at most 131072 squares in FP64 in another order
            assert math.isclose(got, want, rel_tol=1e-11) and math.isclose(got, host, rel_tol=1e-11)
    v.close()


@pytest.mark.parametrize("n1,n3,count,k_cap", [(1, 7, 3, 0), (2500, 300, 40, 0), (2500, 300, 40, 17),
                                               (1024, 64, 1, 1), (1025, 64, 5000, 64),
                                               (40, 3000, 2999, 500)])
def test_scan_entries_in_row_major_order(fk, n1, n3, count, k_cap):
    """The exact scan's records: the first K out-of-range or non-finite entries in row-major order
    with their recomputed values, over several groups of 1024 rows, many in one row, more than K."""
    n2, fmt = 24, "bf16"
    rng = np.random.default_rng(n1 + count)
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("int", -4, 4), ("int", -4, 4), 6)
    a64, b64 = o.decode(a_bits, fmt), o.decode(b_bits, fmt)
    c = (a64 @ b64).astype(np.float32)
    f = c.reshape(-1)
    idx = np.sort(rng.choice(f.size, size=count, replace=False))
    f[idx] = rng.choice(np.array([np.inf, -np.inf, np.nan, 3e38, -2.2e37], dtype=np.float32), size=count)
    v = fk.Verifier(n1, n2, n3, fmt, m=8, k_cap=k_cap)
    K = k_cap if k_cap else 128
    want = idx[:K]
    for fresh in (True, False):
        recs, n, _ = v.localize(to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt), to_dev_f32(c),
                                seed=2, sigma_from_probe=not fresh, cap=8192)
        absolute = [r for r in recs if r[3]]
        assert recs[:len(absolute)] == absolute
        assert [r[0] * n3 + r[1] for r in absolute] == want.tolist()
        assert all(r[4] == 0 and r[2] == a64[r[0]] @ b64[:, r[1]] for r in absolute)
        assert v.plan()["n_abs"] == len(want)
    v.close()


@pytest.mark.parametrize("dirty", [False, True])
def test_calibration_with_nothing_recorded(fk, dirty):
    """No probe, or only dirty ones: nothing changes, and the selections that follow are as ever."""
    n1, n2, n3, fmt, m = 300, 64, 500, "bf16", 40
    a_bits, b_bits = wl.gen_operands(n1, n2, n3, fmt, ("normal", 1.0), ("normal", 1.0), 2)
    A, B = to_dev_half(a_bits, fmt), to_dev_half(b_bits, fmt)
    C = gemm_f32(A, B)
    D = C.clone()
    D[3, 4] += 100.0
    v = fk.Verifier(n1, n2, n3, fmt, m=m)
    if dirty:
        v.probe(A, B, D)
    for _ in range(2):
        m_now, sigma, rebuilt = v.calibrate_noise(C)
        assert (m_now, rebuilt) == (m, False) and math.isnan(sigma)
    v.localize(A, B, C, seed=2, sigma_from_probe=False)
    assert math.isclose(v.plan()["rms_hat"], o.rms_hat(C.cpu().numpy()), rel_tol=1e-11)
    v.probe(A, B, C)
    clean = v.probe_stats()
    assert not clean["dirty"]
    assert v.calibrate_noise(C)[1] == clean["sigma_hat"]
    v.close()
