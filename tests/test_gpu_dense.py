"""The matrix-core kernels, forced (CSRK_MFMA=2) at the sizes where they can go wrong: edges of their tiles (128 rows, 32 and
64 columns of S, 16 columns of the output, 32 elements of a dot product), K cut into ranges, rows with up to every cell
stored, and what they hand to the entry-by-entry path: columns out of order, repeated entries, values that three
bfloat16 pieces cannot hold."""
import numpy as np
import pytest

import oracle
from paper_2311_00368_amd import inputs
from test_gpu_bf16 import dev_bf16
from test_gpu_parity import check, csrk, dev  # noqa: F401  (csrk is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def pattern(rng, M, K, p, kind):
    rp, ci = inputs.bernoulli_csr(int(rng.integers(1 << 30)), M, K, p)
    if kind == "rows":      # no entries, every cell, a few
        take = rng.choice(3, M)
        rows = [np.arange(K) if t == 0 else np.zeros(0) if t == 1 else np.sort(rng.choice(K, 3, replace=False)) for t in take]
        rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        ci = np.concatenate(rows).astype(np.int32)
    elif kind == "unsorted":
        for r in range(0, M, 3):
            ci[rp[r]:rp[r + 1]] = rng.permutation(ci[rp[r]:rp[r + 1]])
    elif kind == "repeated":
        for r in range(0, M, 2):
            n = rp[r + 1] - rp[r]
            ci[rp[r]:rp[r + 1]] = np.sort(rng.choice(ci[rp[r]:rp[r + 1]], n)) if n else ci[rp[r]:rp[r + 1]]
    return rp, ci


def results(csrk, M, K, D, N, rp, ci, v, A, B, C, bf16):
    f = (csrk.spmm_csr_bf16, csrk.sddmm_csr_bf16, csrk.fusedmm_csr_bf16) if bf16 else (csrk.spmm_csr, csrk.sddmm_csr, csrk.fusedmm_csr)
    s = (dev(rp), dev(ci), dev(v))
    O, P, F = f[0](M, K, N, *s, C), f[1](M, K, D, *s, A, B), f[2](M, K, D, N, *s, A, B, C)
    torch.cuda.synchronize()
    return O.cpu().numpy(), P.cpu().numpy(), F.cpu().numpy()


@pytest.mark.parametrize("M,K,D,N,p,kind", [
    (1, 32, 1, 1, 0.5, "even"), (127, 33, 31, 17, 0.3, "even"), (128, 64, 32, 32, 0.2, "even"), (129, 65, 33, 77, 0.35, "even"),
    (300, 1000, 64, 128, 0.1, "even"), (257, 97, 65, 129, 0.25, "even"), (200, 4099, 96, 200, 0.06, "even"),
    (130, 130, 128, 512, 0.4, "even"), (260, 700, 100, 300, 0.9, "even"), (300, 500, 48, 40, 0.2, "rows"),
    (270, 450, 64, 66, 0.2, "unsorted"), (140, 600, 20, 90, 0.15, "repeated"),
    (130, 257, 32, 1, 0.95, "even"), (150, 1025, 16, 1, 0.3, "rows"),     # SDDMM's tiles of 128 columns, rows that fill them
    # enough rows for the widest column blocks (192 and 256): the ones that work a tile further ahead, on 1 to 5 tiles
    (8300, 65, 1, 512, 0.3, "even"), (16500, 32, 3, 256, 0.5, "rows"), (16500, 130, 1, 250, 0.2, "even"),
    (24700, 70, 1, 190, 0.4, "unsorted")])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("ones", [False, True])
def test_tile_edges(csrk, monkeypatch, M, K, D, N, p, kind, bf16, ones):
    monkeypatch.setenv("CSRK_MFMA", "2")
    rng = np.random.default_rng(M + K + D + N)
    rp, ci = pattern(rng, M, K, p, kind)
    v = None if ones else rng.uniform(-1, 1, len(ci)).astype(np.float32)
    A, B, C = (rng.normal(size=s).astype(np.float32) for s in ((M, D), (K, D), (K, N)))
    (dA, A), (dB, B), (dC, C) = map(dev_bf16 if bf16 else lambda x: (dev(x), x), (A, B, C))
    O, P, F = results(csrk, M, K, D, N, rp, ci, v, dA, dB, dC, bf16)
    if ones:
        v = np.ones(len(ci), np.float32)
    what = f"M={M} K={K} D={D} N={N} {kind} bf16={bf16} ones={ones}"
    check(O, *oracle.spmm(M, K, N, rp, ci, v, C), "spmm " + what)
    check(P, *oracle.sddmm(M, K, D, rp, ci, v, A, B), "sddmm " + what)
    check(F, *oracle.fusedmm(M, K, D, N, rp, ci, v, A, B, C), "fusedmm " + what)


@pytest.mark.parametrize("M,K,D,N", [(1920, 1000, 40, 77), (4096, 1024, 24, 512), (5632, 700, 20, 200)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("first,step", [(-1, 1), (-2, 1), (0, 1), (-1, 17), (-18, 17)])
def test_one_swap_at_each_cut(csrk, monkeypatch, M, K, D, N, bf16, first, step):
    # Sorted rows but for one in every 128, whose entries number `first` and `first + step` from a multiple of 64 columns are
    # exchanged: across, before and behind every place where a range of K may begin.  Nothing else sends the rows of those
    # workgroups to the entry-by-entry path.  K is cut in all three shapes, and the second one (the third in bfloat16) has
    # the wide blocks that work a tile further ahead.
    monkeypatch.setenv("CSRK_MFMA", "2")
    rng = np.random.default_rng(M + step - first)
    rp, ci = pattern(rng, M, K, 0.2, "even")
    for block in range(M // 128):
        r = block * 128 + int(rng.integers(128))
        at = rp[r] + np.searchsorted(ci[rp[r]:rp[r + 1]], 64 * (1 + block % ((K - 1) // 64))) + first
        i, j = np.clip([at, at + step], rp[r], rp[r + 1] - 1)
        ci[i], ci[j] = ci[j], ci[i]
    v = rng.uniform(-1, 1, len(ci)).astype(np.float32)
    A, B, C = (rng.normal(size=s).astype(np.float32) for s in ((M, D), (K, D), (K, N)))
    (dA, A), (dB, B), (dC, C) = map(dev_bf16 if bf16 else lambda x: (dev(x), x), (A, B, C))
    O, P, F = results(csrk, M, K, D, N, rp, ci, v, dA, dB, dC, bf16)
    check(O, *oracle.spmm(M, K, N, rp, ci, v, C), "spmm")
    check(P, *oracle.sddmm(M, K, D, rp, ci, v, A, B), "sddmm")
    check(F, *oracle.fusedmm(M, K, D, N, rp, ci, v, A, B, C), "fusedmm")


@pytest.mark.parametrize("bad", [np.inf, np.nan, 3.4e38, 1e-41])
@pytest.mark.parametrize("where", ["v", "A", "B", "C"])
@pytest.mark.parametrize("M,K,D,N", [(150, 300, 40, 50), (150, 300, 40, 52), (700, 90, 128, 256), (300, 2100, 96, 33), (9000, 64, 64, 200)])
def test_values_without_pieces(csrk, monkeypatch, bad, where, M, K, D, N):
    # infinities, NaNs, magnitudes that round to infinity and those whose last bits lie below the smallest bfloat16: same
    # places of infinities and NaNs as in the vector kernels, other values to rounding
    rng = np.random.default_rng(3)
    rp, ci = pattern(rng, M, K, 0.2, "even")
    x = {"v": rng.uniform(-1, 1, len(ci)), "A": rng.normal(size=(M, D)), "B": rng.normal(size=(K, D)), "C": rng.normal(size=(K, N))}
    x = {k: a.astype(np.float32) for k, a in x.items()}
    x[where].flat[x[where].size // 2] = bad
    if bad == np.float64(1e-41):
        x[where][...] = rng.integers(1, 1 << 20, x[where].shape).astype(np.int32).view(np.float32)
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        got.append(results(csrk, M, K, D, N, rp, ci, x["v"], dev(x["A"]), dev(x["B"]), dev(x["C"]), False))
    terms = [oracle.spmm(M, K, N, rp, ci, x["v"], x["C"])[1], oracle.sddmm(M, K, D, rp, ci, x["v"], x["A"], x["B"])[1],
             oracle.fusedmm(M, K, D, N, rp, ci, x["v"], x["A"], x["B"], x["C"])[1]]
    for a, b, t in zip(*got, terms):
        # (finite terms of more than the largest float in all: whether a sum of some of them overflows is a matter of order)
        same = t < np.finfo(np.float32).max if np.isfinite(bad) else np.ones(a.shape, bool)
        assert same.mean() > 0.5
        a, b = a[same], b[same]
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b))
        np.testing.assert_array_equal(np.isposinf(a), np.isposinf(b))
        fine = np.isfinite(a) & np.isfinite(b)
        scale = np.abs(b[fine]).max() if fine.any() else 0.0
        np.testing.assert_allclose(a[fine], b[fine], rtol=1e-4, atol=1e-5 * scale)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("where", ["A", "B", "C"])
@pytest.mark.parametrize("M,K,D,N", [(150, 300, 40, 50), (700, 90, 128, 256), (300, 2100, 96, 32)])
def test_bf16_values_out_of_range(csrk, monkeypatch, bad, where, M, K, D, N):
    # (three of them: a row of B's and a column of C's are done again together)
    rng = np.random.default_rng(4)
    rp, ci = pattern(rng, M, K, 0.2, "even")
    v = rng.uniform(-1, 1, len(ci)).astype(np.float32)
    x = {k: dev_bf16(rng.normal(size=n).astype(np.float32))[0] for k, n in (("A", (M, D)), ("B", (K, D)), ("C", (K, N)))}
    x[where].view(-1)[x[where].numel() // 2] = bad
    x["C"][K // 3, N // 3] = bad
    x["B"][K - 1, D - 1] = bad
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        got.append(results(csrk, M, K, D, N, rp, ci, v, x["A"], x["B"], x["C"], True))
    for a, b in zip(*got):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b))
        np.testing.assert_array_equal(np.isposinf(a), np.isposinf(b))
        fine = np.isfinite(a) & np.isfinite(b)
        assert fine.any() and not fine.all()
        np.testing.assert_allclose(a[fine], b[fine], rtol=1e-4, atol=1e-5 * np.abs(b[fine]).max())


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("D", [24, 100])
def test_scores_out_of_range(csrk, monkeypatch, D, in_place):
    # finite operands whose dot products leave the range of floats: infinities of their sign, as in the vector kernels (the
    # products of the smaller pieces overflow to either sign), beside products that stay inside
    M, K = 200, 300
    rng = np.random.default_rng(D)
    rp, ci = pattern(rng, M, K, 0.3, "even")
    v = rng.uniform(0.5, 1, len(ci)).astype(np.float32)
    A, B = rng.uniform(1, 2, (M, D)).astype(np.float32), rng.uniform(1, 2, (K, D)).astype(np.float32)
    A[::5] *= np.float32(1e20)
    B[::3] *= np.float32(-1e20)
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        d_v = dev(v)
        got.append(csrk.sddmm_csr(M, K, D, dev(rp), dev(ci), d_v, dev(A), dev(B), P=d_v if in_place and mode == "2" else None).cpu().numpy())
    assert np.isneginf(got[1]).any() and np.isfinite(got[1]).any()
    np.testing.assert_allclose(got[0], got[1], rtol=1e-5)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("where", ["A", "B"])
@pytest.mark.parametrize("in_place", [False, True])
def test_bf16_scores_out_of_range(csrk, monkeypatch, bad, where, in_place):
    M, K, D = 200, 300, 40
    rng = np.random.default_rng(5)
    rp, ci = pattern(rng, M, K, 0.3, "even")
    v = rng.uniform(0.5, 1, len(ci)).astype(np.float32)
    A, B = rng.normal(size=(M, D)).astype(np.float32), rng.normal(size=(K, D)).astype(np.float32)
    (dA, A), (dB, B) = dev_bf16(A), dev_bf16(B)
    (A if where == "A" else B)[7, 3] = bad
    (dA if where == "A" else dB)[7, 3] = bad
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        d_v = dev(v)
        got.append(csrk.sddmm_csr_bf16(M, K, D, dev(rp), dev(ci), d_v, dA, dB, P=d_v if in_place and mode == "2" else None).cpu().numpy())
    fine = np.isfinite(got[1])
    assert fine.any() and not fine.all()
    np.testing.assert_array_equal(got[0][~fine], got[1][~fine])
    _, terms = oracle.sddmm(M, K, D, rp, ci, v, np.nan_to_num(A, posinf=0), np.nan_to_num(B, posinf=0))
    assert (np.abs(got[0][fine] - got[1][fine]) <= 2e-5 * terms[fine]).all()


def best_time(call):
    call()
    torch.cuda.synchronize()
    times = []
    for _ in range(5):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(4):
            call()
        e[1].record()
        torch.cuda.synchronize()
        times.append(e[0].elapsed_time(e[1]) / 4 * 1e3)
    return min(times)


def altered(rng, kind, rp, ci, v, x):
    """The pattern, values and dense operands with what the matrix cores cannot do."""
    ci, v, x = ci.copy(), v.copy(), {k: a.copy() for k, a in x.items()}
    operand, _, what = kind.partition(" ")
    if kind == "unsorted":
        for r in range(len(rp) - 1):
            ci[rp[r]:rp[r + 1]] = rng.permutation(ci[rp[r]:rp[r + 1]])
    elif kind == "one pair":
        r = len(rp) // 2
        ci[rp[r] + 3], ci[rp[r] + 4] = ci[rp[r] + 4], ci[rp[r] + 3]
    elif operand == "v":
        v[len(v) // 2] = float(what)
    else:
        x[operand].flat[x[operand].size // 2] = float(what)
    return ci, v, x


@pytest.mark.parametrize("op,kind", [(op, kind) for op, operands in (("spmm", "vC"), ("sddmm", "vAB"), ("fusedmm", "vABC"))
                                     for kind in ("unsorted", "one pair", "v nan", "A inf", "B nan", "C nan")
                                     if kind[0] in operands + "uo"])
@pytest.mark.parametrize("M,K,D,N", [(4096, 4096, 128, 128), (3001, 2999, 77, 77)])
def test_time_of_what_is_left(csrk, monkeypatch, M, K, D, N, op, kind):
    # What the matrix cores cannot do costs no multiple of the vector kernels' time: it was 3 to 16 times as much, and 0.3
    # to 1.9 times as much is measured now.
    rng = np.random.default_rng(M)
    rp, ci = pattern(rng, M, K, 0.3, "even")
    ci, v, x = altered(rng, kind, rp, ci, rng.uniform(-1, 1, len(ci)).astype(np.float32),
                       {k: rng.normal(size=n).astype(np.float32) for k, n in (("A", (M, D)), ("B", (K, D)), ("C", (K, N)))})
    s, (A, B, C) = (dev(rp), dev(ci), dev(v)), (dev(x[k]) for k in "ABC")
    call = {"spmm": lambda: csrk.spmm_csr(M, K, N, *s, C), "sddmm": lambda: csrk.sddmm_csr(M, K, D, *s, A, B),
            "fusedmm": lambda: csrk.fusedmm_csr(M, K, D, N, *s, A, B, C)}[op]
    us = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        us.append(best_time(call))
    assert us[0] < 2.5 * us[1] + 30, us


@pytest.mark.parametrize("op,where", [("spmm", "v"), ("spmm", "C"), ("sddmm", "v"), ("sddmm", "A"), ("sddmm", "B"),
                                      ("fusedmm", "v"), ("fusedmm", "A"), ("fusedmm", "B"), ("fusedmm", "C")])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("factor", [1e-35, 1e15])
def test_small_and_large_values(csrk, monkeypatch, op, where, bf16, factor):
    # normal floats far from 1, underflowed probabilities and the like, stay on the matrix cores: results as good as any, and no
    # slower than the vector kernels (all entries one by one it was 1.5 to 3 times)
    M, K, D, N = 4096, 2048, 100, 128
    rng = np.random.default_rng(M)
    rp, ci = pattern(rng, M, K, 0.3, "even")
    x = {"v": rng.uniform(0.5, 1, len(ci)), "A": rng.normal(size=(M, D)), "B": rng.normal(size=(K, D)), "C": rng.normal(size=(K, N))}
    x = {k: a.astype(np.float32) for k, a in x.items()}
    x[where] *= np.float32(factor)
    d = {k: (dev_bf16 if bf16 and k != "v" else lambda a: (dev(a), a))(a) for k, a in x.items()}
    s, (A, B, C), w = (dev(rp), dev(ci), d["v"][0]), (d[k][0] for k in "ABC"), {k: d[k][1] for k in d}
    suffix = "_bf16" if bf16 else ""
    call, want = {
        "spmm": (lambda: getattr(csrk, "spmm_csr" + suffix)(M, K, N, *s, C), lambda r: oracle.spmm(M, K, N, rp, ci, w["v"], w["C"], rows=r)),
        "sddmm": (lambda: getattr(csrk, "sddmm_csr" + suffix)(M, K, D, *s, A, B), lambda r: oracle.sddmm(M, K, D, rp, ci, w["v"], w["A"], w["B"], rows=r)),
        "fusedmm": (lambda: getattr(csrk, "fusedmm_csr" + suffix)(M, K, D, N, *s, A, B, C),
                    lambda r: oracle.fusedmm(M, K, D, N, rp, ci, w["v"], w["A"], w["B"], w["C"], rows=r))}[op]
    us = []
    for mode in ("3", "2"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        got = call()
        us.append(best_time(call))
    rows = np.arange(0, M, 13)
    want, terms = want(rows)
    got = got.cpu().numpy().astype(np.float64)
    got = got[rows] if op != "sddmm" else got[~np.isnan(want)]
    if op == "sddmm":
        want, terms = want[~np.isnan(want)], terms[~np.isnan(terms)]
    assert (np.abs(got - want) <= 2e-6 * terms).all()
    assert us[1] < 1.2 * us[0] + 10, us


@pytest.mark.parametrize("op,M,K,D,N", [("spmm", 16114, 3635, 0, 64), ("spmm", 5003, 2999, 0, 77), ("spmm", 8192, 4096, 0, 256),
                                        ("sddmm", 4096, 2048, 128, 0), ("sddmm", 3001, 1999, 64, 0), ("sddmm", 2048, 2048, 24, 0),
                                        ("fusedmm", 15872, 3072, 32, 48), ("fusedmm", 6000, 2048, 128, 128), ("fusedmm", 2048, 4096, 64, 512)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("sign", ["both", "one"])
def test_error_is_the_vector_kernels(csrk, monkeypatch, op, M, K, D, N, bf16, sign):
    # The 2-norm of the error against FP64, compared with the vector kernels'.  Data of one sign shows what is always rounded
    # one way (up to 2.05 times the vector kernels' error with one truncating accumulator).  Random draws of these ranges had
    # ratios of up to 1.00 for data of both signs, and of up to 1.13 with one, where both are close to the error of
    # rounding the result once.
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    rand = lambda *n: torch.rand(n, device="cuda", generator=gen) * (1 if sign == "one" else 2) - (0 if sign == "one" else 1)
    keep = torch.rand((M, K), device="cuda", generator=gen) < 0.2
    at = keep.nonzero()
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(keep.sum(1), 0).to(torch.int32)
    ci, v = at[:, 1].to(torch.int32).contiguous(), rand(len(at))
    A, B, C = rand(M, max(D, 1)), rand(K, max(D, 1)), rand(K, max(N, 1))
    if bf16:
        A, B, C = A.bfloat16(), B.bfloat16(), C.bfloat16()
    f = getattr(csrk, {"spmm": "spmm_csr", "sddmm": "sddmm_csr", "fusedmm": "fusedmm_csr"}[op] + ("_bf16" if bf16 else ""))
    args = {"spmm": (M, K, N, rp, ci, v, C), "sddmm": (M, K, D, rp, ci, v, A, B), "fusedmm": (M, K, D, N, rp, ci, v, A, B, C)}[op]
    got = []
    for mode in ("2", "3"):
        monkeypatch.setenv("CSRK_MFMA", mode)
        got.append(f(*args).double())
    s = v.double()
    if D:
        s = s * (A.double() @ B.double().t().contiguous())[at[:, 0], at[:, 1]]
    if N:
        dense = torch.zeros((M, K), dtype=torch.float64, device="cuda")
        dense[at[:, 0], at[:, 1]] = s
        s = dense @ C.double()
    matrix, vector = ((g - s).norm().item() / s.norm().item() for g in got)
    assert matrix <= (1.02 if sign == "both" else 1.2) * vector, (matrix, vector)


@pytest.mark.parametrize("op,M,K,D,N", [("sddmm", 2048, 2048, 64, 0), ("spmm", 3072, 2048, 0, 64), ("fusedmm", 2048, 2048, 32, 64)])
def test_choice_with_unaligned_operands(csrk, monkeypatch, op, M, K, D, N):
    # without 128-bit accesses the vector kernels are slow: such calls go to the matrix cores (which of the two kernels it was
    # shows in the last bits)
    rng = np.random.default_rng(M)
    rp, ci = pattern(rng, M, K, 0.3, "even")
    s = dev(rp), dev(ci), dev(rng.uniform(-1, 1, len(ci)).astype(np.float32))
    A, B, C = (dev(np.append(np.float32(0), rng.normal(size=n).astype(np.float32)))[1:].view(*n) for n in ((M, D), (K, D), (K, N)))
    call = {"spmm": lambda: csrk.spmm_csr(M, K, N, *s, C), "sddmm": lambda: csrk.sddmm_csr(M, K, D, *s, A, B),
            "fusedmm": lambda: csrk.fusedmm_csr(M, K, D, N, *s, A, B, C)}[op]
    got = {}
    for mode in "123":
        monkeypatch.setenv("CSRK_MFMA", mode)
        got[mode] = call()
    assert torch.equal(got["1"], got["2"]) and not torch.equal(got["1"], got["3"])


@pytest.mark.parametrize("M,K,D,N", [(400, 900, 64, 48), (33000, 200, 40, 33)])
def test_graph_replays_with_other_values(csrk, monkeypatch, M, K, D, N):
    # one captured call of each operation, replayed on operands that have nothing special in them, then something to be done
    # again, then nothing again: what a call leaves in its workspace says nothing to the next one
    monkeypatch.setenv("CSRK_MFMA", "2")
    rng = np.random.default_rng(M)
    rp, ci = pattern(rng, M, K, 0.3, "unsorted" if M < 1000 else "even")
    s = dev(rp), dev(ci), dev(rng.uniform(-1, 1, len(ci)).astype(np.float32))
    A, B, C = (dev(rng.normal(size=n).astype(np.float32)) for n in ((M, D), (K, D), (K, N)))
    ws = [torch.empty(csrk.csrk_workspace_bytes(op, M, K, N, D), dtype=torch.uint8, device="cuda") for op in (1, 2, 3)]
    out = [torch.empty(n, dtype=torch.float32, device="cuda") for n in ((M, N), (len(ci),), (M, N))]

    def calls(O, P, F):
        csrk.spmm_csr_ws(M, K, N, *s, C, ws[0], O)
        csrk.sddmm_csr_ws(M, K, D, *s, A, B, ws[1], P)
        csrk.fusedmm_csr_ws(M, K, D, N, *s, A, B, C, ws[2], F)

    calls(*out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(*out)
    for special in (None, (B, 3), None, (C, 5), (A, 7), None):
        if special:
            x, at = special
            kept = x.view(-1)[at * x.shape[1]].clone()
            x.view(-1)[at * x.shape[1]] = float("nan")
        graph.replay()
        torch.cuda.synchronize()
        replayed = [x.clone() for x in out]
        eager = [torch.empty_like(x) for x in out]
        calls(*eager)
        torch.cuda.synchronize()
        for a, b in zip(replayed, eager):
            assert torch.equal(a.nan_to_num(nan=1e30), b.nan_to_num(nan=1e30))
        if special:
            assert torch.isnan(replayed[2]).any()
            x.view(-1)[at * x.shape[1]] = kept
        else:
            assert not any(torch.isnan(a).any() for a in replayed)
