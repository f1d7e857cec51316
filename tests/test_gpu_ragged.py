"""Rows that are no whole aligned 16-byte groups: the stream pass's 8-element loads at any element
alignment, at the edges where they can go wrong - the matrix's last rows, row lengths below 8,
matrices of fewer than 8 elements, bases off a 16-byte boundary.  Small-integer operands with
C = AB + integer errors: every sum is exact, so the sketches equal the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import fpsketch_oracle as o
from gpu_util import int_case, to_dev_f32, to_dev_half

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fk():
    from paper_2609_19758_amd import fpsketch
    fpsketch.load()
    return fpsketch


def _shifted(t, shift):
    """The tensor at a base `shift` elements past an aligned one."""
    import torch
    if shift == 0:
        return t
    buf = torch.full((t.numel() + shift,), 7, dtype=t.dtype, device=t.device)
    buf[shift:] = t.reshape(-1)
    return buf[shift:].view(t.shape)


# n1, n2, n3, m, fmt, base shift in elements: every stream instance's ragged form
CASES = [
    (1, 1, 1, 1, "bf16", 0), (1, 7, 1, 1, "fp16", 0), (2, 3, 2, 2, "bf16", 1),
    (7, 1, 3, 3, "fp16", 1), (9, 5, 11, 4, "bf16", 3), (64, 9, 7, 8, "fp16", 0),
    (40, 64, 512, 16, "bf16", 1),        # whole groups, bases off alignment
    (130, 511, 513, 48, "bf16", 0), (300, 519, 4099, 60, "fp16", 5),
    (700, 33, 2055, 100, "bf16", 7),     # C tiles one per wave, padded lists
    (600, 1027, 4101, 192, "fp16", 1),   # the same, two B chunks
    (900, 21, 1031, 300, "bf16", 2), (500, 13, 2051, 700, "fp16", 0),
    (300, 17, 1025, 1500, "bf16", 3), (200, 11, 1027, 2500, "fp16", 0),
]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n1,n2,n3,m,fmt,shift", CASES)
def test_sketch_exact(fk, n1, n2, n3, m, fmt, shift, layout):
    a_bits, b_bits, a64, b64, c = int_case(n1, n2, n3, fmt, 11 + n1 + n3)
    rng = np.random.default_rng(n1 * n3 + m)
    c = c + rng.integers(-3, 4, size=c.shape).astype(np.float32)
    A = _shifted(to_dev_half(a_bits, fmt), shift)
    B = _shifted(to_dev_half(np.ascontiguousarray(b_bits.T) if layout else b_bits, fmt), shift)
    C = _shifted(to_dev_f32(c), shift)
    hr = o.make_round(5, 1, n1, n3, m)
    E = a64 @ b64 - c.astype(np.float64)
    v = fk.Verifier(n1, n2, n3, fmt, m=m, b_layout=layout)
    for moments in (False, True):
        S, R, T, ma, mb = v.sketch(A, B, C, seed=5, rnd=1, m=m, moments=moments)
        X = np.zeros((m, n3))
        np.add.at(X, hr.h1, hr.v1[:, None] * E)
        ref = np.zeros((m, m))
        np.add.at(ref.T, hr.h2, (X * hr.v2).T)
        assert np.array_equal(S, ref)
        assert ma == np.abs(a64).max() and mb == np.abs(b64).max()
        if moments:
            w1 = (np.arange(n1) + 1) / o.pow2_ceil(n1)
            Y = np.zeros((m, n3))
            np.add.at(Y, hr.h1, (hr.v1 * w1)[:, None] * E)
            refr = np.zeros((m, m))
            np.add.at(refr.T, hr.h2, (Y * hr.v2).T)
            w2 = (np.arange(n3) + 1) / o.pow2_ceil(n3)
            reft = np.zeros((m, m))
            np.add.at(reft.T, hr.h2, (X * hr.v2 * w2).T)
            assert np.array_equal(R, refr) and np.array_equal(T, reft)
    v.close()


@pytest.mark.parametrize("n1,n2,n3,m,fmt,shift", [
    (700, 1027, 2055, 60, "bf16", 1), (333, 129, 515, 40, "fp16", 0), (1, 2, 3, 2, "bf16", 0)])
def test_deferred_and_cached_equal_ordinary(fk, n1, n2, n3, m, fmt, shift):
    a_bits, b_bits, _, _, c = int_case(n1, n2, n3, fmt, 3)
    c[n1 - 1, n3 - 1] += 5.0                     # the matrix's very last element
    A, B = _shifted(to_dev_half(a_bits, fmt), shift), _shifted(to_dev_half(b_bits, fmt), shift)
    C = _shifted(to_dev_f32(c), shift)
    v = fk.Verifier(n1, n2, n3, fmt, m=m)
    v.probe(A, B, C)
    ref = v.probe_stats()
    assert ref["max_abs"] == 5.0
    v.probe_deferred(A, B, C)
    v.probe_flush()
    assert v.probe_stats() == ref
    v.cache_b(B)
    v.probe_cached(A, C)
    assert v.probe_stats() == ref
    v.probe_noalloc(A, B, C)
    assert v.probe_stats() == ref
    v.close()
