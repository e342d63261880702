"""The binding where the extension module is missing or belongs to another torch: every call through ctypes."""
import subprocess
import sys

import numpy as np
import pytest

from paper_2311_00368_amd import binding, inputs

torch = pytest.importorskip("torch")


def test_loads_without_the_extension():
    code = """
import sys, warnings
sys.modules["paper_2311_00368_amd._torch_calls"] = None     # an import of it raises ImportError
from paper_2311_00368_amd import binding
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    assert binding.csrk_version().startswith("csrk")
assert any("ctypes" in str(x.message) for x in w)
assert binding._call(1, 2) is None and binding._call_plan(1) is None
"""
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


@pytest.mark.gpu
def test_same_results_without_the_extension(monkeypatch):
    M, K, D, N = 300, 260, 20, 36
    rp, ci = inputs.bernoulli_csr(5, M, K, 0.2)
    gen = torch.Generator().manual_seed(1)
    rand = lambda *n: torch.randn(n, generator=gen).cuda()
    rp, ci, v, A, B, C = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), rand(len(ci)), rand(M, D), rand(K, D), rand(K, N)
    plan = binding.csrk_plan_create(M, K, rp, ci)
    ws = torch.empty(binding.csrk_workspace_bytes(binding.CSRK_OP_FUSEDMM, M, K, N, D), dtype=torch.uint8, device="cuda")

    def results():
        out = [binding.spmm_csr(M, K, N, rp, ci, v, C), binding.sddmm_csr(M, K, D, rp, ci, v, A, B),
               binding.fusedmm_csr(M, K, D, N, rp, ci, v, A, B, C), binding.fusedmm_csr_ws(M, K, D, N, rp, ci, v, A, B, C, ws),
               binding.spmm_csr_plan(plan, N, v, C), binding.sddmm_csr_plan(plan, D, v, A, B),
               binding.fusedmm_csr_plan(plan, D, N, v, A, B, C), binding.spmm_csr_bf16(M, K, N, rp, ci, v, C.bfloat16())]
        return [x.cpu().numpy() for x in out]

    want = results()
    monkeypatch.setattr(binding, "_call", binding._turned_down)
    monkeypatch.setattr(binding, "_call_plan", binding._turned_down)
    for got, w in zip(results(), want):
        np.testing.assert_array_equal(got, w)
