"""Calls that the fitted ratio of the two times gives to the matrix-core kernels: they are taken there, agree
with the vector kernels, and stay with these where the scratch they need would have to be allocated during a capture."""
import numpy as np
import pytest

from test_gpu_dense import pattern
from test_gpu_parity import csrk, dev  # noqa: F401  (csrk is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [("spmm", "f32", 3000, 3000, 0, 96, 0.3), ("spmm", "f32", 3000, 3000, 0, 256, 0.2), ("spmm", "f32", 2048, 2048, 0, 512, 0.25),
          ("sddmm", "f32", 2048, 2048, 128, 0, 0.3), ("sddmm", "f32", 2999, 3001, 96, 0, 0.12), ("sddmm", "bf16", 2048, 2048, 128, 0, 0.3),
          ("fusedmm", "f32", 2048, 2048, 64, 256, 0.15), ("fusedmm", "f32", 2048, 2048, 128, 256, 0.15),
          # by the vector kernels' estimate for their family: equal shares, whole rows, whole-row kernels, tiled
          ("spmm", "f32", 512, 2560, 0, 480, 0.316), ("spmm", "f32", 1536, 4608, 0, 480, 0.135),
          ("fusedmm", "f32", 768, 2304, 32, 488, 0.226), ("fusedmm", "f32", 3164, 3228, 48, 96, 0.169), ("fusedmm", "f32", 753, 2207, 88, 512, 0.262),
          ("fusedmm", "f32", 4005, 2992, 96, 96, 0.109), ("fusedmm", "f32", 2086, 1056, 128, 392, 0.282), ("fusedmm", "f32", 1024, 8448, 128, 472, 0.126),
          # outside of the sizes that the ratio was fitted to
          ("spmm", "f32", 3200, 896, 0, 632, 0.294), ("sddmm", "f32", 11264, 384, 120, 0, 0.587), ("fusedmm", "f32", 1595, 706, 16, 656, 0.682)]


def call_of(csrk, op, dtype, M, K, D, N, density):
    rng = np.random.default_rng(M + K + N + D)
    rp, ci = pattern(rng, M, K, density, "even")
    s = dev(rp), dev(ci), dev(rng.uniform(-1, 1, len(ci)).astype(np.float32))
    A, B, C = (dev(rng.normal(size=n).astype(np.float32)) for n in ((M, D), (K, D), (K, N)))
    bf = "_bf16" if dtype == "bf16" else ""
    if bf:
        A, B, C = A.bfloat16(), B.bfloat16(), C.bfloat16()
    f = getattr(csrk, f"{op}_csr{bf}")
    return {"spmm": lambda: f(M, K, N, *s, C), "sddmm": lambda: f(M, K, D, *s, A, B), "fusedmm": lambda: f(M, K, D, N, *s, A, B, C)}[op]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_taken_and_equal(csrk, monkeypatch, shape):
    call = call_of(csrk, *shape)
    got = {}
    for mode in "123":
        monkeypatch.setenv("CSRK_MFMA", mode)
        got[mode] = call()
    assert torch.equal(got["1"], got["2"]) and not torch.equal(got["1"], got["3"])
    # both sides round sums of up to 3000 terms at random: 1e-6 of the result's norm at most
    a, b = got["1"].double(), got["3"].double()
    assert ((a - b).norm() / b.norm()).item() < 1e-6


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3], SHAPES[7]], ids=lambda s: "-".join(map(str, s)))
def test_capture_without_the_scratch(csrk, monkeypatch, shape):
    call = call_of(csrk, *shape)
    csrk.csrk_release_workspace()
    monkeypatch.setenv("CSRK_MFMA", "3")
    vector = call()                             # leaves the scratch of the vector kernels
    monkeypatch.setenv("CSRK_MFMA", "1")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for _ in range(3):
        out.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, vector)
    dense = call()
    assert not torch.equal(dense, vector)
    csrk.csrk_release_workspace()
    assert torch.equal(call(), dense)


# op, M, K, D, N, density, rows, planned
NO_LESS_EXACT = [("fusedmm", 29184, 3840, 84, 32, 0.07, "even", False), ("spmm", 30424, 574, 0, 32, 0.21, "even", False),
                 ("spmm", 16384, 512, 0, 64, 0.157, "lognormal", False), ("fusedmm", 16760, 578, 64, 36, 0.214, "lognormal", False),
                 ("fusedmm", 12764, 3172, 104, 456, 0.1129, "even", False), ("spmm", 6656, 5120, 0, 336, 0.0792, "lognormal", False),
                 ("spmm", 7258, 2725, 0, 352, 0.0729, "lognormal", False),
                 ("spmm", 12288, 768, 0, 480, 0.1008, "lognormal", False),
                 ("spmm", 16384, 1024, 0, 32, 0.208, "lognormal", False), ("fusedmm", 12032, 512, 88, 32, 0.187, "lognormal", False),
                 ("fusedmm", 15532, 558, 48, 64, 0.153, "lognormal", False), ("spmm", 5632, 1792, 0, 328, 0.102, "lognormal", False),
                 # (these are taken)
                 ("fusedmm", 2917, 3143, 72, 20, 0.138, "even", False), ("spmm", 2406, 3083, 0, 64, 0.25, "even", False),
                 ("fusedmm", 9370, 1605, 104, 44, 0.1, "lognormal", False),
                 ("spmm", 512, 2560, 0, 480, 0.316, "even", False), ("spmm", 1536, 4608, 0, 480, 0.135, "lognormal", False),
                 ("fusedmm", 1024, 8448, 128, 472, 0.126, "even", False), ("fusedmm", 753, 2207, 88, 512, 0.262, "lognormal", False),
                 ("spmm", 512, 2560, 0, 480, 0.316, "even", True)]


@pytest.mark.parametrize("shape", NO_LESS_EXACT, ids=lambda s: "-".join(map(str, s)))
def test_no_less_exact_on_data_of_one_sign(csrk, monkeypatch, shape):
    # whatever is chosen by the family that would do the call: no further from FP64 than the vector kernels, in the 2-norm.  (Sums of one
    # sign, where the matrix cores' truncation shows most; the same inputs every time, on which the ratio lies below 0.95 or is 1)
    op, M, K, D, N, density, rows, planned = shape
    g = torch.Generator(device="cuda").manual_seed(M + K)
    p = torch.full((M,), density, device="cuda")
    if rows == "lognormal":
        p = (density * torch.exp(torch.randn(M, device="cuda", generator=g) - 0.5)).clamp(1 / K, 1)
    keep = torch.rand((M, K), device="cuda", generator=g) < p[:, None]
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = keep.sum(1).cumsum(0)
    ci = keep.nonzero()[:, 1].to(torch.int32)
    v, A, B, C = (torch.rand(s, device="cuda", generator=g) for s in (len(ci), (M, D), (K, D), (K, N)))
    S = torch.zeros((M, K), dtype=torch.float64, device="cuda")
    S[keep] = v.double()
    if op == "fusedmm":
        S *= A.double() @ B.double().T
    want = S @ C.double()
    plan = csrk.csrk_plan_create(M, K, rp, ci) if planned else None
    error = {}
    for mode in "13":
        monkeypatch.setenv("CSRK_MFMA", mode)
        if op == "spmm":
            out = csrk.spmm_csr_plan(plan, N, v, C) if planned else csrk.spmm_csr(M, K, N, rp, ci, v, C)
        else:
            out = csrk.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C)
        error[mode] = ((out.double() - want).norm() / want.norm()).item()
    assert error["1"] <= error["3"], error


@pytest.mark.parametrize("even", [False, True])
@pytest.mark.parametrize("M,K,D,density", [(8170, 10048, 32, 0.0618), (3966, 10910, 32, 0.0946)])
def test_planned_sddmm_of_uneven_rows(csrk, monkeypatch, even, M, K, D, density):
    # near the line, where slabs of scores lose what uneven rows cost them: only a plan can tell
    g = torch.Generator(device="cuda").manual_seed(K)
    z = torch.zeros(M, device="cuda") if even else torch.randn(M, device="cuda", generator=g) - 0.5
    p = (density * torch.exp(z)).clamp(1 / K, 1)
    keep = torch.rand((M, K), device="cuda", generator=g) < p[:, None]
    rp = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rp[1:] = keep.sum(1).cumsum(0)
    ci = keep.nonzero()[:, 1].to(torch.int32)
    v, A, B = (torch.rand(s, device="cuda", generator=g) for s in (len(ci), (M, D), (K, D)))
    plan = csrk.csrk_plan_create(M, K, rp, ci)
    assert csrk.csrk_plan_info(plan)[2] == even
    planned, plain = {}, {}
    for mode in "123":
        monkeypatch.setenv("CSRK_MFMA", mode)
        planned[mode] = csrk.sddmm_csr_plan(plan, D, v, A, B)
        plain[mode] = csrk.sddmm_csr(M, K, D, rp, ci, v, A, B)
    assert torch.equal(planned["1"], planned["2" if even else "3"])
    assert torch.equal(plain["1"], plain["2"]) and not torch.equal(plain["1"], plain["3"])
