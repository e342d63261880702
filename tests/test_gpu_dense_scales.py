"""Wide SPMM and FusedMM in half-precision pieces (forced, CSRK_MFMA=2) on operands whose rows and columns differ in size: sums of
one sign of values far below the rest of their operand, and what calls cost whose first columns say nothing about the others."""
import numpy as np
import pytest

from test_gpu_parity import csrk  # noqa: F401  (a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M, K, D = 16384, 16384, 64
# rows that are checked, and the entries in them (the others have 160)
LONG = {7: 3277, 300: 5734, 1001: 16384, 5000: 16384, 9000: 3277, 16383: 16384}
# Relative to the sum of the terms' magnitudes, which is the result here.  Pieces and products leave 3 x 6e-8 at most; sums of 512
# tiles of one sign drift by half a unit in the last place, 3e-8, for each of 128 tiles between two interruptions at most: 3.8e-6.
TOL = 4e-6
# Results that are computed again are sums of FP32, a term of 1 and thousands of 1e-8 among them: the library's tolerance.
TOL_AGAIN = 1e-5


def operands(seed, ones=False):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    counts = torch.full((M,), 160, dtype=torch.int64)
    for r, n in LONG.items():
        counts[r] = n
    step = (K // counts).repeat_interleave(counts)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(counts, 0)])
    ci = ((torch.arange(int(rp[-1])) - rp[:-1].repeat_interleave(counts)) * step).to(torch.int32).cuda()
    v = None if ones else torch.rand(len(ci), device="cuda", generator=gen)
    return gen, rp.to(torch.int32).cuda(), ci, v


def rows_of(rp, ci, v):
    """The checked rows as a dense FP64 matrix."""
    S = torch.zeros((len(LONG), K), dtype=torch.float64, device="cuda")
    for i, r in enumerate(LONG):
        at = slice(int(rp[r]), int(rp[r + 1]))
        S[i, ci[at].long()] = 1.0 if v is None else v[at].double()
    return S


def check(got, want, terms, what, tol):
    err = ((got[list(LONG)].double() - want).abs() / terms).max(0).values
    assert err.max().item() < tol, (what, err.argmax().item(), err.max().item())


SMALL = [0.6e-9, 1.9e-9, 5.5e-9, 9.3e-9, 3e-10, 1e-10, 1e-8, 1e-7, 1e-6]


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
@pytest.mark.parametrize("ones", [False, True])
@pytest.mark.parametrize("kind", ["columns", "rows", "large rows", "parts of columns", "parts of rows"])
def test_sums_of_small_values(csrk, monkeypatch, op, ones, kind):
    monkeypatch.setenv("CSRK_MFMA", "2")
    gen, rp, ci, v = operands(3, ones)
    N = 512 if op == "spmm" else 250
    C = torch.randn((K, N), device="cuda", generator=gen)
    if ones and "rows" in kind:
        v = torch.ones(len(ci), device="cuda")
    row = lambda r: slice(int(rp[r]), int(rp[r + 1]))
    if kind == "columns":
        for i, s in enumerate(SMALL):
            C[:, 11 * i + 9] = s
            C[:, 11 * i + 10] = s * torch.rand(K, device="cuda", generator=gen)
    elif kind == "rows":                # C of one sign
        C = C.abs()
        for r, s in zip(LONG, SMALL):
            v[row(r)] = s
    elif kind == "large rows":          # one row above the rest, below what half precision overflows at
        for r in LONG:
            v[row(r)] *= 60
        for i, s in enumerate(SMALL):
            C[:, 11 * i + 9] = s
    elif kind == "parts of columns":    # a column's largest value far above the others that a row adds up
        for i, s in enumerate(SMALL):
            C[:, 11 * i + 9] = s
            C[K - 3, 11 * i + 9] = 1
    else:                               # ... a row's
        C = C.abs()
        for r, s in zip(LONG, SMALL):
            v[row(r)] = s
            v[int(rp[r]) + 1] = 1
            C[ci[int(rp[r]) + 1].long()] = 0
    S = rows_of(rp, ci, v)
    if op == "spmm":
        got = csrk.spmm_csr(M, K, N, rp, ci, v, C)
    else:
        A, B = torch.rand((M, D), device="cuda", generator=gen), torch.rand((K, D), device="cuda", generator=gen)
        if kind == "rows":
            A[::3] *= 1e-7
        S = S * (A[list(LONG)].double() @ B.double().T)
        got = csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
    check(got, S @ C.double(), S.abs() @ C.double().abs(), (op, kind, ones), TOL_AGAIN if kind == "parts of columns" else TOL)


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
def test_small_values_behind_a_large_one(csrk, monkeypatch, op):
    # a value of 1 at the beginning of the checked rows and 2^-27 behind it: the other rows have results that only bfloat16 pieces
    # hold, and these do the whole call; the small values must not be lost one after the other in an accumulator that holds the large one
    monkeypatch.setenv("CSRK_MFMA", "2")
    _, rp, ci, v = operands(5, ones=True)
    N = 512
    C = torch.full((K, N), 2.0 ** -27, device="cuda")
    C[5] = 1        # (a column of S in which only rows of 3277 and of all entries have one)
    S = rows_of(rp, ci, v)
    if op == "spmm":
        got = csrk.spmm_csr(M, K, N, rp, ci, v, C)
    else:
        A, B = torch.full((M, D), 0.5, device="cuda"), torch.full((K, D), 0.5, device="cuda")
        S *= D / 4
        got = csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
    want = S @ C.double()
    check(got, want, want, op, TOL)


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
@pytest.mark.parametrize("kind", ["row", "column", "row of B"])
def test_values_that_scales_lose(csrk, monkeypatch, op, kind):
    # a value so far above the rest of its row or column that the others underflow where they are scaled, in results without it
    monkeypatch.setenv("CSRK_MFMA", "2")
    gen, rp, ci, v = operands(4)
    N = 250
    C = torch.randn((K, N), device="cuda", generator=gen)
    A, B = torch.rand((M, D), device="cuda", generator=gen) + 0.1, torch.rand((K, D), device="cuda", generator=gen) + 0.1
    if kind == "row":               # half of all rows: where a row's samples and its largest value meet is up to chance
        large = rp[:-1].long()[torch.arange(M, device="cuda") % 2 == 1]
        v *= 1e-28
        v[large] = 1e18
        C[ci[large].unique().long()] = 0
    elif kind == "column":
        C[:, ::5] *= 1e-30
        C[8, ::5] = 1e18            # a column of S that no checked row has an entry in
    else:
        B[8], A[:] = 1e17, A * 1e-6
        C[:, ::3] *= 1e-12
    used = (ci == 8).nonzero()
    if kind != "row":
        v[used[:, 0]] = 0
    S = rows_of(rp, ci, v)
    if op == "spmm":
        got = csrk.spmm_csr(M, K, N, rp, ci, v, C)
    else:
        S = S * (A[list(LONG)].double() @ B.double().T)
        got = csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
    want, terms = S @ C.double(), S.abs() @ C.double().abs()
    assert (terms > 0).any()
    bad = (got[list(LONG)].double() - want).abs() > TOL_AGAIN * terms + 2.0 ** -148
    assert not bad.any(), bad.float().mean()


@pytest.mark.parametrize("op", ["spmm", "fusedmm"])
@pytest.mark.parametrize("kind", ["first columns zero", "first columns small", "first columns large", "heavy tails", "one large", "rows", "equal rows"])
def test_cost_of_uneven_operands(csrk, monkeypatch, op, kind):
    # a call whose results are nearly all computed again, entry by entry, takes five to ten times as long
    monkeypatch.setenv("CSRK_MFMA", "2")
    gen = torch.Generator(device="cuda").manual_seed(11)
    N = 512
    keep = torch.rand((M, K), device="cuda", generator=gen) < 0.1
    if kind == "equal rows":            # rows of the same length that begin alike
        keep = torch.zeros((M, K), dtype=torch.bool, device="cuda")
        keep[:, ::10] = True
        keep[:, :16] = True
    at = keep.nonzero()
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(keep.sum(1), 0).to(torch.int32)
    ci = at[:, 1].to(torch.int32).contiguous()
    v, C = torch.rand(len(ci), device="cuda", generator=gen), torch.randn((K, N), device="cuda", generator=gen)
    A, B = torch.randn((M, D), device="cuda", generator=gen), torch.randn((K, D), device="cuda", generator=gen)
    f = {"spmm": lambda: csrk.spmm_csr(M, K, N, rp, ci, v, C), "fusedmm": lambda: csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)}[op]

    def ms():
        out = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            b.synchronize()
            out.append(a.elapsed_time(b))
        return min(out[1:])

    plain = ms()
    first = {"first columns zero": 0.0, "first columns small": 1e-3, "first columns large": 1e6}.get(kind)
    if first is not None:
        C[:, :8] *= first
        A[:, :8] *= first
        B[:, :8] *= first
    elif kind == "heavy tails":         # (Student's t with two degrees of freedom: some values of each column hundreds of times the median)
        C /= torch.rand((K, N), device="cuda", generator=gen).log().neg().sqrt()
        B /= torch.rand((K, 1), device="cuda", generator=gen).log().neg().sqrt()
        v /= torch.rand(len(ci), device="cuda", generator=gen).log().neg().sqrt()
    elif kind == "one large":
        C[K // 3, N // 2] = 1e4
        v[len(v) // 2] = 1e9
    elif kind == "rows":
        r = torch.arange(M, device="cuda") % 7
        v *= (10.0 ** (-4.0 * r))[at[:, 0]].float()
        A *= (10.0 ** (-3.0 * r))[:, None].float()
    elif kind == "equal rows":          # every row's first entries say nothing about the others
        v.view(M, -1)[:, :16] *= 1e-7
    uneven = ms()
    # (heavy tails of S, C and B at once leave FusedMM some results to do again; the whole call again in bfloat16 pieces is 2.4)
    assert uneven < (2.5 if kind == "heavy tails" else 1.6) * plain, (op, kind, plain, uneven)
