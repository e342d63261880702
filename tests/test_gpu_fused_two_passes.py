"""FusedMM that is done as SDDMM and SPMM on its result: taken where the scratch for the products can be had, with the results of the two
calls, and by FusedMM's own kernel where it cannot."""
import numpy as np
import pytest

from test_gpu_parity import csrk, dev  # noqa: F401  (csrk is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(15360, 8200, 36, 260), (16383, 8193, 63, 301)]       # M, K, D, N


def operands(M, K, D, N, seed, density=0.06):
    g = torch.Generator(device="cuda").manual_seed(seed)
    keep = torch.rand((M, K), device="cuda", generator=g) < density
    keep[::500] = False
    keep[7, :] = True
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = keep.sum(1).cumsum(0)
    ci = keep.nonzero()[:, 1].to(torch.int32)
    v, A, B, C = (torch.rand(s, device="cuda", generator=g) * 2 - 1 for s in (len(ci), (M, D), (K, D), (K, N)))
    return rp, ci, v, A, B, C


def two_calls(csrk, M, K, D, N, rp, ci, v, A, B, C):
    return csrk.spmm_csr(M, K, N, rp, ci, csrk.sddmm_csr(M, K, D, rp, ci, v, A, B), C)


def scratch_of(csrk, call):
    csrk.csrk_release_workspace()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("M,K,D,N", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "ones", "unsorted", "not finite", "plan"])
def test_results(csrk, M, K, D, N, kind):
    rp, ci, v, A, B, C = operands(M, K, D, N, M + D)
    r, c = rp.cpu().numpy(), ci.cpu().numpy()
    if kind == "ones":
        v = None
    elif kind == "unsorted":        # pairs of neighbours, and a row in descending order
        for row in range(1, M, 97):
            c[r[row]], c[r[row] + 1] = c[r[row] + 1], c[r[row]]
        c[r[9]:r[10]] = c[r[9]:r[10]][::-1].copy()
        ci = dev(c)
    elif kind == "not finite":
        A[4, 1], B[50, D - 1], C[K - 1, N - 1], v[len(v) // 2] = np.inf, np.nan, -np.inf, np.nan
        A[5, 0] = 3e38
    s = rp, ci, v, A, B, C
    if kind == "plan":
        plan = csrk.csrk_plan_create(M, K, rp, ci)
        got = csrk.fusedmm_csr_plan(plan, D, N, v, A, B, C)
        products = csrk.sddmm_csr_plan(plan, D, v, A, B)
        want = csrk.spmm_csr_plan(plan, N, products, C)
    else:
        got, want = csrk.fusedmm_csr(M, K, D, N, *s), two_calls(csrk, M, K, D, N, *s)
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy(), equal_nan=True)
    rows = [0, 1, 4, 5, 7, 9, 98, 500, 501, M // 2, M - 1]
    out = got.cpu().numpy()
    h = [x.cpu().numpy().astype(np.float64) if x is not None else np.ones(len(c)) for x in (v, A, B, C)]
    with np.errstate(all="ignore"):
        for row in rows:
            k = c[r[row]:r[row + 1]]
            p = h[0][r[row]:r[row + 1]] * (h[2][k] @ h[1][row])
            exact, size = p @ h[3][k], np.abs(p) @ np.abs(h[3][k])
            fine = np.isfinite(exact) & (size < 1e38)
            # FP32 scores and pieces, sums of up to 8200 terms: see test_gpu_dense_halves.py; the scores' own rounding errors are
            # relative to their terms' magnitudes, some sqrt(D) times theirs
            terms = (np.abs(h[0][r[row]:r[row + 1]]) * (np.abs(h[2][k]) @ np.abs(h[1][row]))) @ np.abs(h[3][k])
            assert np.all(np.abs(out[row][fine] - exact[fine]) <= 2e-6 * size[fine] + 2e-7 * terms[fine]), row
            assert not np.isfinite(out[row][~np.isfinite(exact)]).any(), row


def test_scratch(csrk, monkeypatch):
    M, K, D, N = SHAPES[0]
    s = operands(M, K, D, N, 1)
    products = 4 * len(s[1])
    one = csrk.csrk_workspace_bytes(csrk.CSRK_OP_FUSEDMM, M, K, N, D)
    assert scratch_of(csrk, lambda: csrk.fusedmm_csr(M, K, D, N, *s)) > products + one // 2
    monkeypatch.setenv("CSRK_MFMA", "2")
    kernel = csrk.fusedmm_csr(M, K, D, N, *s)
    monkeypatch.setenv("CSRK_MFMA", "1")
    both = csrk.fusedmm_csr(M, K, D, N, *s)
    # a workspace of the size that is asked for, and one with room for the products
    for room, want in ((0, kernel), (products + (1 << 20), both)):
        ws = torch.empty(one + room, dtype=torch.uint8, device="cuda")
        assert torch.equal(csrk.fusedmm_csr_ws(M, K, D, N, *s, ws), want)


@pytest.mark.parametrize("has", ["vector kernels", "one kernel", "two passes"])
def test_capture(csrk, monkeypatch, has):
    # a call whose scratch would have to grow during a capture takes the kernels that there is scratch for
    M, K, D, N = SHAPES[0]
    s = operands(M, K, D, N, 2)
    csrk.csrk_release_workspace()
    monkeypatch.setenv("CSRK_MFMA", {"vector kernels": "3", "one kernel": "2", "two passes": "1"}[has])
    want = csrk.fusedmm_csr(M, K, D, N, *s)
    monkeypatch.setenv("CSRK_MFMA", "1")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = csrk.fusedmm_csr(M, K, D, N, *s)
    for _ in range(3):
        out.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("M,K,D,N", SHAPES)
def test_a_count_that_is_too_small(csrk, monkeypatch, M, K, D, N):
    # csrk_call's count is an expectation: nothing may be sized by it.  The call does without products in memory, also where its
    # scratch has room for them; csrk_call_bounded vouches for the count.
    s = operands(M, K, D, N, 3)
    rp, ci, v, A, B, C = s
    lib, nnz = csrk.load(), len(ci)
    monkeypatch.setenv("CSRK_MFMA", "2")
    kernel = csrk.fusedmm_csr(M, K, D, N, *s)
    monkeypatch.setenv("CSRK_MFMA", "1")
    out = torch.empty((M, N), device="cuda")
    # (what the header says is enough for the products)
    ws = torch.empty(csrk.csrk_workspace_bytes(csrk.CSRK_OP_FUSEDMM, M, K, N, D) + (4 * (nnz + nnz // 50) + 255) // 256 * 256,
                     dtype=torch.uint8, device="cuda")

    def call(fn, count, workspace=None):
        out.fill_(7)
        status = fn(csrk.CSRK_OP_FUSEDMM, 0, count, M, K, D, N, *(t.data_ptr() for t in s), out.data_ptr(),
                    workspace.data_ptr() if workspace is not None else None, workspace.numel() if workspace is not None else 0,
                    torch.cuda.current_stream().cuda_stream)
        assert status == 0, csrk.csrk_last_error()
        return out.clone()

    for workspace in (None, ws):
        for count in (nnz, nnz - 1, nnz - nnz // 50, nnz + nnz // 50):
            assert torch.equal(call(lib.csrk_call, count, workspace), kernel), count
        for count in (nnz, nnz + nnz // 50):
            assert torch.equal(call(lib.csrk_call_bounded, count, workspace), two_calls(csrk, M, K, D, N, *s)), count
    # a count that is far off: another kernel, the same results to rounding
    for count in (0, nnz // 3, -1):
        assert (call(lib.csrk_call, count) - kernel).norm() <= 1e-6 * kernel.norm(), count
    # (the scratch of the one kernel)
    one = csrk.csrk_workspace_bytes(csrk.CSRK_OP_FUSEDMM, M, K, N, D)
    assert scratch_of(csrk, lambda: call(lib.csrk_call, nnz)) < one + 2 * nnz


def test_scratch_that_cannot_be_had(csrk, monkeypatch):
    # A call that cannot have room for its products keeps the area there is, and with it the graphs captured on it, and does not ask
    # again before the area is released.  (CSRK_SCRATCH_MB stands in for a device without memory.)
    M, K, D, N = SHAPES[0]
    s = operands(M, K, D, N, 4)
    one = csrk.csrk_workspace_bytes(csrk.CSRK_OP_FUSEDMM, M, K, N, D)
    csrk.csrk_release_workspace()
    monkeypatch.setenv("CSRK_MFMA", "2")
    kernel = csrk.fusedmm_csr(M, K, D, N, *s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = csrk.fusedmm_csr(M, K, D, N, *s)
    monkeypatch.setenv("CSRK_MFMA", "1")
    monkeypatch.setenv("CSRK_SCRATCH_MB", "1")
    before = torch.cuda.mem_get_info()[0]
    for _ in range(2):
        out = csrk.fusedmm_csr(M, K, D, N, *s)
        captured.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, kernel) and torch.equal(captured, kernel)
    monkeypatch.delenv("CSRK_SCRATCH_MB")
    assert torch.equal(csrk.fusedmm_csr(M, K, D, N, *s), kernel)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] > before - one // 2
    csrk.csrk_release_workspace()
    assert torch.equal(csrk.fusedmm_csr(M, K, D, N, *s), two_calls(csrk, M, K, D, N, *s))
    # nothing at all to be had for the matrix cores
    csrk.csrk_release_workspace()
    monkeypatch.setenv("CSRK_SCRATCH_MB", "1")
    out = csrk.fusedmm_csr(M, K, D, N, *s)
    monkeypatch.setenv("CSRK_MFMA", "3")
    assert torch.equal(out, csrk.fusedmm_csr(M, K, D, N, *s))


@pytest.mark.parametrize("M,K,D,N", SHAPES)
@pytest.mark.parametrize("wider", [0, 3])
def test_reserved_plan(csrk, M, K, D, N, wider):
    # a plan's own scratch has room for the products: the same kernels, and so the same bits, as without it, and in a capture
    # (so many entries that their products do not fit into the room for the other kernels by chance)
    s = operands(M, K, D, N, 5, density=0.13)
    rp, ci, v, A, B, C = s
    want = two_calls(csrk, M, K, D, N, *s)
    csrk.csrk_release_workspace()
    plan = csrk.csrk_plan_create(M, K, rp, ci)
    csrk.csrk_plan_reserve(plan, N + wider)
    assert torch.equal(csrk.fusedmm_csr_plan(plan, D, N, v, A, B, C), want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = csrk.fusedmm_csr_plan(plan, D, N, v, A, B, C)
    for _ in range(3):
        out.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("M,K,D,N", SHAPES)
def test_cost_of_rows_of_b_that_are_not_numbers(csrk, M, K, D, N):
    # a NaN in B is one in every product of its column: the rows that store it are NaNs, and are not to be added up entry by entry.
    # (csrk_call keeps the one kernel.  The two passes take 1.4 and 1.5 times as long, with every row added up 3.9 and 4.0 times)
    rows = 30
    rp, ci, v, A, B, C = s = operands(M, K, D, N, 6, density=0.13)
    B[torch.arange(rows, device="cuda") * (K // rows), 1] = float("nan")
    lib, out = csrk.load(), torch.empty((M, N), device="cuda")
    times, results = [], []
    for fn in (lib.csrk_call, lib.csrk_call_bounded):
        def call():
            assert fn(csrk.CSRK_OP_FUSEDMM, 0, len(ci), M, K, D, N, *(t.data_ptr() for t in s), out.data_ptr(), None, 0,
                      torch.cuda.current_stream().cuda_stream) == 0, csrk.csrk_last_error()
        best = []
        for _ in range(5):
            call()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                call()
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b))
        times.append(min(best))
        results.append(out.clone())
    one, two = results
    assert torch.equal(one.isnan(), two.isnan()) and one.isnan().any(1).float().mean() > 0.15
    fine = ~one.isnan()
    assert (one - two)[fine].norm() <= 1e-6 * one[fine].norm()
    assert not torch.equal(one[fine], two[fine])        # (two passes)
    assert times[1] < 2.2 * times[0], times
