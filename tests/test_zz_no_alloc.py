"""sdv2_gemm_bf16_noalloc (the entry point that allocates nothing) against sdv2_gemm_bf16 with a caller workspace.

Two calls in a row share the library's built-in scratch array; the second is smaller and lays its partial sums out
differently, so stale contents of the first would show.  Bar: the two entry points run the same kernels on the same
plan, so their outputs are equal bit for bit; both are also held to the per-kernel bar against the oracle.
"""

import numpy as np
import pytest
import torch

from oracle.dit_block import linear as oracle_linear
from paper_2511_07399_amd import binding
from parity_util import max_rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def draw(shape, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(torch.bfloat16)


def one_case(M, N, K, epi, seed):
    a, w = draw((M, K), seed).to(DEV), draw((N, K), seed + 1, 0.05).to(DEV)
    bias = draw((N,), seed + 2, 0.5).float().to(DEV)
    gate_a = draw((N,), seed + 3, 0.3).float().to(DEV)
    gate_b = draw((1, N), seed + 4, 0.3).float().to(DEV)
    x0 = draw((M, N), seed + 5).float().to(DEV)
    ws_bytes = binding.gemm_workspace_bytes(M, N, K, epi)
    assert 0 < ws_bytes <= binding.gemm_noalloc_max_scratch_bytes(), "the case must split k and fit the scratch"
    ws = torch.full((ws_bytes // 4,), float("nan"), dtype=torch.float32, device=DEV)
    want_out = x0.clone() if epi >= 2 else torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    binding.gemm_bf16(a, w, bias, want_out, epi, gate_a, gate_b, N, M, workspace=ws)
    got_out = x0.clone() if epi >= 2 else torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    binding.gemm_bf16_noalloc(a, w, bias, got_out, epi, gate_a, gate_b, N, M)
    torch.cuda.synchronize()
    assert torch.equal(got_out, want_out), "no-alloc entry point differs from the workspace entry point"
    acc = oracle_linear(a.cpu().double().numpy(), w.cpu().double().numpy(), bias.cpu().double().numpy())
    if epi == 2:
        gate = (gate_a + gate_b[0]).cpu().double().numpy()
        ref = x0.cpu().double().numpy() + gate[None, :] * acc
    else:
        ref = acc
    assert max_rel_err(got_out.cpu().double().numpy(), ref) < (1e-4 if epi >= 2 else 1e-2)


def test_noalloc_gemm_two_calls_in_a_row_second_smaller():
    # FFN-2 of the 1.3B block with two streams (two k parts of 2048 rows), then with one (four parts of 1024 rows)
    one_case(2048, 1536, 8960, 2, 100)
    one_case(1024, 1536, 8960, 2, 200)
    # a forced split on a small ragged shape, bf16 output
    binding.tuning_set("gemm_tile", "1,4,2,2")
    try:
        one_case(300, 512, 1024, 0, 300)
    finally:
        binding.tuning_set("gemm_tile", None)


@pytest.mark.parametrize("M,N,K,epi", [
    (1024, 5120, 13824, 2),         # FFN-2 of the 14B block
    (1024, 5120, 20480, 3),
    (1560, 3072, 12288, 2),         # two parts of 18 MiB
    (3072, 1536, 8960, 2),          # FFN-2 of the 1.3B block on three streams
])
def test_noalloc_gemm_runs_whole_what_its_scratch_does_not_hold(M, N, K, epi):
    assert 2 * 4 * M * N > binding.gemm_noalloc_max_scratch_bytes()
    assert binding.gemm_workspace_bytes(M, N, K, epi) > binding.gemm_noalloc_max_scratch_bytes()
    a, w = draw((M, K), 500).to(DEV), draw((N, K), 501, 0.05).to(DEV)
    x0 = draw((M, N), 502).float().to(DEV)
    gate_a, gate_b = draw((N,), 503, 0.3).float().to(DEV), draw((1, N), 504, 0.3).float().to(DEV)
    out = x0.clone()
    binding.gemm_bf16_noalloc(a, w, None, out, epi, gate_a, gate_b, N, M)
    acc = a.double() @ w.double().t()
    ref = x0.double() + (acc * (gate_a + gate_b[0]).double() if epi == 2 else acc)
    assert max_rel_err(out.cpu().double().numpy(), ref.cpu().numpy()) < 1e-4


def test_noalloc_gemm_takes_as_many_parts_as_the_scratch_holds():
    # the plan is four k parts of 512 x 5120 floats (40 MiB), of which the scratch holds three
    M, N, K = 512, 5120, 13824
    assert binding.gemm_workspace_bytes(M, N, K, 3) > binding.gemm_noalloc_max_scratch_bytes() > 2 * 4 * M * N
    a, w = draw((M, K), 400), draw((N, K), 401, 0.05)
    x0 = draw((M, N), 402).float()
    out = x0.to(DEV)
    binding.gemm_bf16_noalloc(a.to(DEV), w.to(DEV), None, out, 3)
    ref = x0.double() + (a.float() @ w.float().t()).double()
    assert max_rel_err(out.cpu().double().numpy(), ref.numpy()) < 1e-4
