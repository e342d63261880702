"""SPMM and FusedMM of wide outputs over long ranges of K in half-precision pieces, forced (CSRK_MFMA=2): its tile edges, rows of every kind,
and the values that two pieces or their range of exponents cannot hold."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import csrk, dev  # noqa: F401  (csrk is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# Relative to the sum of the terms' magnitudes: two pieces leave 2^-23 of each operand and 2^-22 of their product, 4.8e-7 in all;
# the rows checked have up to 9000 terms, whose sums of random rounding errors stay below 1e-6 of it.
TOL = 2e-6
OPS = {"spmm": 1, "fusedmm": 3}


def assert_halves(csrk, op, M, K, N, D=0):
    """That the shape is one for half-precision pieces; its ranges of K."""
    products, ranges = csrk.csrk_matrix_core_form(OPS[op], M, K, N, D)
    assert products == 3
    return ranges


def matrix(rng, M, K):
    """About 1 % of the cells; every 50th row has none, one, two, every one of the first half's or every cell."""
    rows = []
    for r in range(M):
        kind = r % 250
        if kind == 0: c = np.zeros(0, int)
        elif kind == 50: c = rng.integers(K, size=1)
        elif kind == 100: c = rng.choice(K, 2, replace=False)
        elif kind == 150 and r < 1000: c = np.arange(K // 2)
        elif kind == 200 and r < 1000: c = np.arange(K)
        else: c = np.unique(rng.integers(K, size=K // 100))
        rows.append(np.sort(c))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int32)
    return rp, np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("M,K,N", [(16300, 8200, 500), (16384, 8192, 512), (16320, 9000, 300), (32650, 8224, 180),
                                   (8192, 16384, 512), (16300, 16390, 250)])       # two ranges of K
@pytest.mark.parametrize("kind", ["plain", "ones", "unsorted", "not finite", "small", "large", "mixed", "zeros"])
def test_long_ranges(csrk, monkeypatch, M, K, N, kind):
    monkeypatch.setenv("CSRK_MFMA", "2")
    assert assert_halves(csrk, "spmm", M, K, N) == K // 8192
    rng = np.random.default_rng(M + K + N)
    rp, ci = matrix(rng, M, K)
    v = rng.uniform(-1, 1, len(ci)).astype(np.float32)
    C = rng.normal(size=(K, N)).astype(np.float32)
    row_of = np.repeat(np.arange(M), np.diff(rp))
    if kind == "ones":
        v[:] = 1
    elif kind == "unsorted":        # every third row, and one pair of neighbours in some others
        for r in range(0, M, 3):
            ci[rp[r]:rp[r + 1]] = rng.permutation(ci[rp[r]:rp[r + 1]])
        for r in range(1, M, 300):
            if rp[r + 1] - rp[r] > 40:
                i = rp[r] + int(rng.integers(40))
                ci[i], ci[i + 1] = ci[i + 1], ci[i]
    elif kind == "not finite":
        C[5, 3], C[K - 1, N - 1], v[len(v) // 2], v[len(v) // 3] = np.inf, np.nan, -np.inf, np.nan
        C[K // 2, N // 2], v[len(v) // 5] = 3e38, 3e38
    elif kind == "small":           # far below what half precision reaches: the operands are scaled
        v *= np.float32(1e-20)
        C *= np.float32(1e-15)
    elif kind == "large":
        v *= np.float32(1e15)
        C *= np.float32(1e12)
    elif kind == "mixed":           # rows of S and C that are far below, or above, the rest of theirs
        v[row_of % 5 == 1] *= np.float32(1e-9)
        v[row_of % 5 == 2] *= np.float32(1e-13)
        v[row_of % 25 == 3] *= np.float32(1e7)
        C[:, N // 3] *= np.float32(1e-10)
        C[:, N // 4] *= np.float32(1e6)
    elif kind == "zeros":           # columns of nothing but zeros, with a value that is lost in one of them, and rows of lost values
        C[:, N // 2:] = 0
        C[K // 3, N // 2 + 1] = 1e-25
        v[row_of % 7 == 0] = 1e-30
        v[row_of % 7 == 1] = 0
    O = csrk.spmm_csr(M, K, N, dev(rp), dev(ci), None if kind == "ones" else dev(v), dev(C)).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(0, 1000, 50), np.arange(0, M, 41), rng.integers(M, size=60), [M - 1],
                                     np.arange(1, M, 1500), row_of[[len(v) // 2, len(v) // 3, len(v) // 5]]]))
    want, terms = oracle.spmm(M, K, N, rp, ci, v, C, rows=rows)
    got = O[rows]
    fine = np.isfinite(want) & (terms < 3e38)
    np.testing.assert_array_equal(np.isnan(got)[~fine & np.isnan(want)], True)
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])
    # (results below the smallest normal float are rounded to a multiple of 2^-149)
    bad = np.abs(got[fine] - want[fine]) > TOL * terms[fine] + 2.0 ** -148
    assert not bad.any(), (kind, bad.mean(), np.abs(got[fine] - want[fine])[bad].max())
    if kind == "zeros":
        assert (np.abs(want[:, N // 2 + 1]) > 0).any()


@pytest.mark.parametrize("M,K,D,N", [(16300, 8200, 64, 500), (16384, 8192, 32, 512), (16320, 9000, 1, 300), (32650, 8224, 33, 180),
                                     (8192, 16384, 64, 512), (16300, 16390, 20, 250)])
@pytest.mark.parametrize("kind", ["plain", "ones", "unsorted", "not finite", "small", "large", "mixed", "zeros"])
def test_long_ranges_fused(csrk, monkeypatch, M, K, D, N, kind):
    monkeypatch.setenv("CSRK_MFMA", "2")
    assert assert_halves(csrk, "fusedmm", M, K, N, D) == K // 8192
    rng = np.random.default_rng(M + K + N + D)
    rp, ci = matrix(rng, M, K)
    v = rng.uniform(-1, 1, len(ci)).astype(np.float32)
    A, B, C = (rng.normal(size=n).astype(np.float32) for n in ((M, D), (K, D), (K, N)))
    row_of = np.repeat(np.arange(M), np.diff(rp))
    if kind == "ones":
        v[:] = 1
    elif kind == "unsorted":
        for r in range(0, M, 3):
            ci[rp[r]:rp[r + 1]] = rng.permutation(ci[rp[r]:rp[r + 1]])
    elif kind == "not finite":
        A[M // 3, 0], C[5, 3], v[len(v) // 2] = np.nan, np.inf, -np.inf
        B[K // 4, D - 1] = np.inf
    elif kind == "small":
        v *= np.float32(1e-8)
        A *= np.float32(1e-12)
        B *= np.float32(1e-9)
        C *= np.float32(1e-6)
    elif kind == "large":
        v *= np.float32(1e9)
        A *= np.float32(1e10)
        B *= np.float32(1e8)
        C *= np.float32(1e6)
    elif kind == "mixed":
        v[row_of % 5 == 1] *= np.float32(1e-9)
        A[np.arange(M) % 5 == 2] *= np.float32(1e-13)
        A[np.arange(M) % 25 == 3] *= np.float32(1e6)
        C[:, N // 3] *= np.float32(1e-10)
    elif kind == "zeros":
        C[:, N // 2:] = 0
        C[K // 3, N // 2 + 1] = 1e-25
        v[row_of % 7 == 0] = 1e-30
        A[np.arange(M) % 7 == 1] = 0
        A[np.arange(M) % 7 == 2] = 1e-25
    O = csrk.fusedmm_csr(M, K, D, N, dev(rp), dev(ci), None if kind == "ones" else dev(v), dev(A), dev(B), dev(C)).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(0, 1000, 50), np.arange(0, M, 57), [M // 3, M - 1], row_of[[len(v) // 2]]]))
    want, terms = oracle.fusedmm(M, K, D, N, rp, ci, v, A, B, C, rows=rows)
    got = O[rows]
    fine = np.isfinite(want) & (terms < 3e38)
    assert fine.mean() > (0.3 if kind == "not finite" else 0.9)
    np.testing.assert_array_equal(np.isnan(got)[np.isnan(want)], True)
    np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)])
    bad = np.abs(got[fine] - want[fine]) > TOL * terms[fine] + 2.0 ** -148
    assert not bad.any(), (kind, bad.mean(), (np.abs(got[fine] - want[fine]) / terms[fine])[bad].max())


def bernoulli(gen, M, K, p):
    parts = [(torch.rand((2048, K), device="cuda", generator=gen) < p).nonzero() + torch.tensor([[r, 0]], device="cuda") for r in range(0, M, 2048)]
    at = torch.cat(parts)
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(at[:, 0], minlength=M), 0).to(torch.int32)
    return at, rp, at[:, 1].to(torch.int32).contiguous()


@pytest.mark.parametrize("op,M,K,D,N", [("spmm", 4096, 32768, 0, 512), ("fusedmm", 4096, 32768, 40, 500)])
def test_rows_in_one_range(csrk, monkeypatch, op, M, K, D, N):
    # rows with entries in one, two or all of four ranges of K, small ones in the others; results of zero in some
    monkeypatch.setenv("CSRK_MFMA", "2")
    assert assert_halves(csrk, op, M, K, N, D) == 4
    rng = np.random.default_rng(9)
    kinds = np.arange(M) % 8
    v, rows = [], []
    for r in range(M):
        ranges = [[0], [3], [1, 2], [0, 1, 2, 3], [0, 3], [2], [], [1]][kinds[r]]
        c = np.unique(np.concatenate([rng.integers(8192, size=200) + 8192 * q for q in ranges] or [np.zeros(0, int)]))
        x = rng.uniform(-1, 1, len(c))
        if kinds[r] == 4: x[c >= 8192] *= 1e-12     # the last range's values are small, and these are all that some columns add up
        if kinds[r] == 5: x[:] = 0
        rows.append(c)
        v.append(x)
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int32)
    ci, v = np.concatenate(rows).astype(np.int32), np.concatenate(v).astype(np.float32)
    A, B, C = (rng.normal(size=n).astype(np.float32) for n in ((M, D), (K, D), (K, N)))
    C[:8192, ::7] = 0
    some = np.unique(np.concatenate([np.arange(0, M, 11), [M - 1]]))
    if op == "spmm":
        O = csrk.spmm_csr(M, K, N, dev(rp), dev(ci), dev(v), dev(C)).cpu().numpy()
        want, terms = oracle.spmm(M, K, N, rp, ci, v, C, rows=some)
    else:
        O = csrk.fusedmm_csr(M, K, D, N, dev(rp), dev(ci), dev(v), dev(A), dev(B), dev(C)).cpu().numpy()
        want, terms = oracle.fusedmm(M, K, D, N, rp, ci, v, A, B, C, rows=some)
    bad = np.abs(O[some] - want) > TOL * terms
    assert not bad.any(), (bad.mean(), np.unique(kinds[some[bad.any(1)]]))


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
@pytest.mark.parametrize("M,K", [(16384, 8192), (8192, 16384)])
def test_every_entry_point_and_replays(csrk, monkeypatch, op, M, K):
    # planned, on a workspace and captured: the same bits as the plain call, on every replay, also after operands were exchanged
    # for ones with rows to be done again, and for ones that bfloat16 pieces do again
    monkeypatch.setenv("CSRK_MFMA", "2")
    D, N = 32, 512
    ranges = assert_halves(csrk, op, M, K, N, D if op == "fusedmm" else 0)
    assert ranges == K // 8192
    gen = torch.Generator(device="cuda").manual_seed(K)
    at, rp, ci = bernoulli(gen, M, K, 0.06)
    v, C = torch.rand(len(ci), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    A, B = torch.randn((M, D), device="cuda", generator=gen), torch.randn((K, D), device="cuda", generator=gen)
    plan = csrk.csrk_plan_create(M, K, rp, ci)
    ws = torch.empty(csrk.csrk_workspace_bytes(OPS[op], M, K, N, D), dtype=torch.uint8, device="cuda")
    if op == "spmm":
        plain = lambda: csrk.spmm_csr(M, K, N, rp, ci, v, C)
        others = [lambda: csrk.spmm_csr_plan(plan, N, v, C), lambda: csrk.spmm_csr_ws(M, K, N, rp, ci, v, C, ws)]
    else:
        plain = lambda: csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
        others = [lambda: csrk.fusedmm_csr_plan(plan, D, N, v, A, B, C), lambda: csrk.fusedmm_csr_ws(M, K, D, N, rp, ci, v, A, B, C, ws)]
    ordinary = plain()
    for f in others:
        assert torch.equal(f(), ordinary)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        out = others[1]()
    kept = C.clone()
    for change in (None, "few", "all", None, "all", "few", None):
        C.copy_(kept)
        if change == "few":             # a value that is not finite
            C[5, 7] = float("inf")
        elif change == "all":           # a value in every column that leaves the others out of its pieces' range
            C[torch.arange(N), torch.arange(N)] = 1e12
        want = plain()
        out.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.nan_to_num(out), torch.nan_to_num(want)), change
        assert change is not None or torch.equal(want, ordinary)


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
def test_short_rows(csrk, monkeypatch, op):
    # Rows of up to 32 entries among longer ones: no further from FP64 than the vector kernels by more than the order of a sum's
    # terms makes out, at most for two terms: two products and their sum are rounded, or one product and the sum with the other,
    # sqrt(3 / 2) = 1.22 in the 2-norm.
    M, K, D, N = 16384, 8192, 32, 512
    assert assert_halves(csrk, op, M, K, N, D if op == "fusedmm" else 0) == 1
    gen = torch.Generator(device="cuda").manual_seed(2)
    lens = torch.tensor([1, 2, 3, 5, 8, 16, 31, 32, 100, 33])
    counts = lens.repeat(M // len(lens) + 1)[:M]
    rp = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(counts, 0)])
    step = (K // counts).repeat_interleave(counts)
    ci = ((torch.arange(int(rp[-1])) - rp[:-1].repeat_interleave(counts)) * step).to(torch.int32).cuda()
    rp = rp.to(torch.int32).cuda()
    v, C = torch.rand(len(ci), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    A, B = torch.randn((M, D), device="cuda", generator=gen), torch.randn((K, D), device="cuda", generator=gen)
    S = torch.zeros((M, K), dtype=torch.float64, device="cuda")
    S[torch.arange(M, device="cuda").repeat_interleave(counts.cuda()), ci.long()] = v.double()
    if op == "fusedmm":
        S *= A.double() @ B.double().T
    want = S @ C.double()
    errors = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        got = csrk.spmm_csr(M, K, N, rp, ci, v, C) if op == "spmm" else csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
        d = got.double() - want
        errors.append([(d[counts == n].norm() / want[counts == n].norm()).item() for n in lens[:8].tolist()])
    for n, ours, vector in zip(lens.tolist(), *errors):
        assert ours <= 1.3 * vector, (n, ours, vector)


@pytest.mark.parametrize("M,K,N,p", [(16384, 8192, 512, 0.06), (16384, 8192, 512, 0.1), (16384, 9000, 384, 0.35)])
@pytest.mark.parametrize("sign", ["both", "one"])
def test_error_is_the_vector_kernels(csrk, monkeypatch, M, K, N, p, sign):
    # the 2-norm of the error against FP64 on a sample of rows, no larger than the vector kernels' (measured: 0.2-0.5 times)
    gen = torch.Generator(device="cuda").manual_seed(K)
    parts = [(torch.rand((2048, K), device="cuda", generator=gen) < p).nonzero() + torch.tensor([[r, 0]], device="cuda") for r in range(0, M, 2048)]
    at = torch.cat(parts)
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(at[:, 0], minlength=M), 0).to(torch.int32)
    ci = at[:, 1].to(torch.int32).contiguous()
    v, C = torch.rand(len(ci), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    v, C = (v - 0.5, C) if sign == "both" else (v, C.abs())
    some = torch.zeros((M, 1), device="cuda", dtype=torch.bool)
    some[::17] = True
    picked = some[at[:, 0], 0]
    S = torch.zeros((M // 17 + 1, K), dtype=torch.float64, device="cuda")
    S[at[picked, 0] // 17, at[picked, 1]] = v[picked].double()
    want = S @ C.double()
    err = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        err.append(((csrk.spmm_csr(M, K, N, rp, ci, v, C)[::17].double() - want).norm() / want.norm()).item())
    assert err[0] <= 1.02 * err[1], err


@pytest.mark.parametrize("M,K,D,N,p", [(16384, 8192, 64, 512, 0.06), (16384, 8192, 32, 512, 0.1), (8192, 16384, 64, 512, 0.06), (16384, 9000, 16, 384, 0.3)])
def test_error_is_the_vector_kernels_fused(csrk, monkeypatch, M, K, D, N, p):
    # the same for FusedMM (measured: 0.3-0.45 times)
    assert_halves(csrk, "fusedmm", M, K, N, D)
    gen = torch.Generator(device="cuda").manual_seed(K)
    at, rp, ci = bernoulli(gen, M, K, p)
    v, C = torch.rand(len(ci), device="cuda", generator=gen) - 0.5, torch.randn((K, N), device="cuda", generator=gen)
    A, B = torch.randn((M, D), device="cuda", generator=gen), torch.randn((K, D), device="cuda", generator=gen)
    picked = at[:, 0] % 17 == 0
    S = torch.zeros((M // 17 + 1, K), dtype=torch.float64, device="cuda")
    S[at[picked, 0] // 17, at[picked, 1]] = v[picked].double()
    want = (S * (A[::17].double() @ B.double().T)) @ C.double()
    err = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        err.append(((csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)[::17].double() - want).norm() / want.norm()).item())
    assert err[0] <= 1.02 * err[1], err
