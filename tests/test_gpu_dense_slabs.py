"""SDDMM in slabs of scores (64 rows by 256 columns, a row's entries in chunks of 64 that begin at multiples of 64), forced
(CSRK_MFMA=2) where it can go wrong: row blocks, slabs and chunks that are full, short by one or one over, rows that begin
anywhere in a chunk, rows that are left to the entry-by-entry path, in place and not."""
import numpy as np
import pytest

import oracle
from test_gpu_bf16 import dev_bf16
from test_gpu_parity import check, csrk, dev  # noqa: F401  (csrk is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rows_of_lengths(rng, K, lengths):
    rows = [np.sort(rng.choice(K, n, replace=False)) for n in lengths]
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), np.concatenate(rows + [np.zeros(0)]).astype(np.int32)


# lengths around whole chunks, so that the rows behind begin at every kind of place; empty rows in front, between and behind
LENGTHS = [0, 64, 1, 63, 65, 0, 128, 127, 129, 2, 62, 200, 0, 256, 255, 31, 0]


@pytest.mark.parametrize("M,K", [(1, 256), (63, 257), (64, 255), (65, 511), (129, 513), (200, 1100), (70, 300)])
@pytest.mark.parametrize("D", [4, 32, 33, 64, 100, 128])
@pytest.mark.parametrize("bf16", [False, True])
def test_blocks_slabs_chunks(csrk, monkeypatch, M, K, D, bf16):
    monkeypatch.setenv("CSRK_MFMA", "2")
    rng = np.random.default_rng(M * 7 + K + D)
    lengths = np.minimum([LENGTHS[i % len(LENGTHS)] + (i // len(LENGTHS)) % 3 for i in range(M)], K)
    rp, ci = rows_of_lengths(rng, K, lengths)
    v = rng.uniform(-1, 1, len(ci)).astype(np.float32)
    A, B = (rng.normal(size=s).astype(np.float32) for s in ((M, D), (K, D)))
    (dA, A), (dB, B) = map(dev_bf16 if bf16 else lambda x: (dev(x), x), (A, B))
    call = csrk.sddmm_csr_bf16 if bf16 else csrk.sddmm_csr
    want = oracle.sddmm(M, K, D, rp, ci, v, A, B)
    check(call(M, K, D, dev(rp), dev(ci), dev(v), dA, dB).cpu().numpy(), *want, "sddmm")
    check(call(M, K, D, dev(rp), dev(ci), None, dA, dB).cpu().numpy(), *oracle.sddmm(M, K, D, rp, ci, np.ones_like(v), A, B), "ones")
    P = dev(v)
    call(M, K, D, dev(rp), dev(ci), P, dA, dB, P)
    check(P.cpu().numpy(), *want, "in place")


@pytest.mark.parametrize("what", ["swap", "reversed", "shuffled", "repeated", "nan", "inf", "huge", "tiny"])
@pytest.mark.parametrize("D", [24, 64, 96])
@pytest.mark.parametrize("bf16", [False, True])
def test_rows_that_stay_behind(csrk, monkeypatch, what, D, bf16):
    # Rows out of order stop where they are noticed; a value that pieces cannot hold stops every row that needs it.  K is cut
    # into ranges (few rows), and the calls are made in place: nothing may be computed twice.
    M, K = 150, 2100
    rng = np.random.default_rng(D)
    rp, ci = rows_of_lengths(rng, K, rng.integers(0, 700, M))
    v = rng.uniform(0.5, 1, len(ci)).astype(np.float32)
    A, B = (rng.normal(size=s).astype(np.float32) for s in ((M, D), (K, D)))
    for r in range(0, M, 5):
        c = ci[rp[r]:rp[r + 1]]
        if len(c) < 4:
            continue
        if what == "swap":
            i = int(rng.integers(len(c) - 1))
            c[[i, i + 1]] = c[[i + 1, i]]
        elif what == "reversed":
            c[:] = c[::-1].copy()
        elif what == "shuffled":
            c[:] = rng.permutation(c)
        elif what == "repeated":
            c[:] = np.sort(rng.choice(c, len(c)))
    bad = {"nan": np.nan, "inf": np.inf, "huge": 3e38, "tiny": 1e-41}.get(what)
    if bad is not None:
        A[3, 1] = B[1000, D - 1] = bad
    (dA, A), (dB, B) = map(dev_bf16 if bf16 else lambda x: (dev(x), x), (A, B))
    call = csrk.sddmm_csr_bf16 if bf16 else csrk.sddmm_csr
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        P = dev(v)
        call(M, K, D, dev(rp), dev(ci), P, dA, dB, P)
        got.append(P.cpu().numpy())
    x, y = got
    fine = np.isfinite(y)
    np.testing.assert_array_equal(np.isnan(x), np.isnan(y))
    np.testing.assert_array_equal(x[~fine & ~np.isnan(y)], y[~fine & ~np.isnan(y)])
    with np.errstate(all="ignore"):
        want, terms = oracle.sddmm(M, K, D, rp, ci, v, np.nan_to_num(A, posinf=0, neginf=0), np.nan_to_num(B, posinf=0, neginf=0))
    rows = np.repeat(np.arange(M), np.diff(rp))
    clean = fine & np.isfinite(A).all(1)[rows] & np.isfinite(B).all(1)[ci]
    check(x[clean], want[clean], terms[clean], "sddmm " + what)


@pytest.mark.parametrize("D", [65, 72, 96, 97, 128])
@pytest.mark.parametrize("mode", ["2", "3"])
def test_values_beside_halves_of_opposite_signs(csrk, monkeypatch, D, mode):
    # FP32 dot products of more than 64 elements are the sum of two halves (elements up to 64, the others): a stored value that is infinite,
    # or so large that it takes one half out of the range of floats, multiplies the sum.  Some halves are zero.
    monkeypatch.setenv("CSRK_MFMA", mode)
    M, K = 150, 1100
    rng = np.random.default_rng(D)
    rp, ci = rows_of_lengths(rng, K, rng.integers(0, 500, M))
    A, B = rng.uniform(0.5, 1, (M, D)).astype(np.float32), rng.uniform(0.5, 1, (K, D)).astype(np.float32)
    B[:, 64:] *= -rng.uniform(0.7, 0.95, (K, 1)) * 64 / (D - 64)
    B[::2] *= -1
    B[::7, :64] = 0
    B[1::7, 64:] = 0
    v = rng.choice(np.array([1e37, -1e37, 1e38, -1e38, 3e38, np.inf, -np.inf, np.nan, 1, -0.25, 1e-3, 0.5], np.float32), len(ci))
    v[rp[20]:rp[90]] = rng.uniform(-1, 1, rp[90] - rp[20])
    P = dev(v)
    args = M, K, D, dev(rp), dev(ci)
    got = [csrk.sddmm_csr(*args, dev(v), dev(A), dev(B)).cpu().numpy(), csrk.sddmm_csr(*args, P, dev(A), dev(B), P).cpu().numpy()]
    score, terms = oracle.sddmm(M, K, D, rp, ci, np.ones_like(v), A, B)
    v = v.astype(np.float64)
    with np.errstate(all="ignore"):
        want = score * v
    largest = float(np.finfo(np.float32).max)
    # (near the largest float whether there is an infinity, and near a score of zero which, is a matter of rounding)
    sure = np.isnan(v) | np.isinf(v) | (np.abs(np.abs(want) - largest) > 1e-5 * terms * np.abs(v))
    sure &= np.abs(score) > 1e-3 * terms
    assert sure.mean() > 0.95
    want[np.abs(want) > largest] = np.copysign(np.inf, want[np.abs(want) > largest])
    for x in got:
        fine = sure & np.isfinite(want)
        np.testing.assert_array_equal(x[sure & ~fine], want[sure & ~fine])
        check(x[fine], want[fine], (terms * np.abs(v))[fine], "sddmm")
