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
