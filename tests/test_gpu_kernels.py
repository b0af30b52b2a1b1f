"""GPU parity of the individual kernels, through the C ABI, against the CPU oracle.

Tolerances: the dense kernels multiply bf16 operands exactly and accumulate in fp32, so against the
float64 oracle on the same bf16 inputs the only errors are fp32 summation order (relative 1e-6 per
term) and the final rounding of the output to bf16 (relative 2^-9).  Attention also rounds the
probabilities to bf16 before the second product.  Bars: 1e-2 of the largest output for bf16 outputs,
1e-4 for fp32 outputs; cache bookkeeping and copied cache contents are bit-exact.
"""


import math
import numpy as np
import pytest
import torch

import oracle
from oracle.dit_block import linear as oracle_linear
from paper_2511_07399_amd import binding
from parity_util import max_rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bf16_randn(shape, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(torch.bfloat16)


def f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


# ------------------------------------------------------------------------------------------ GEMM
GEMM_CASES = [
    # M, N, K, epilogue, tile override ("tm,tn[,pf[,parts of k]]" register-staged kernel, "d<id>[,parts of k]" a tile of the
    # direct-load kernel) or None
    (128, 128, 64, 0, None),
    (1, 128, 64, 0, None),                 # a single row
    (200, 384, 192, 0, "1,3"),             # ragged M, N tile of 96
    (333, 640, 512, 1, "2,5"),             # GELU epilogue, 256 x 160 tiles, ragged M
    (1024, 1536, 512, 0, "1,7"),           # N not a multiple of the 224-wide tile
    (300, 512, 1024, 2, "1,4"),            # gated residual, ragged M
    (300, 512, 1024, 2, None),
    (260, 256, 2048, 3, "2,8"),            # residual, biggest tile
    (300, 384, 768, 0, "1,3,3"),           # three register sets (loads three k tiles ahead), 12 k tiles
    (520, 640, 704, 2, "2,5,3"),           # three sets, 11 k tiles (tail of the unrolled-by-6 loop)
    (256, 256, 64, 3, "2,2,3"),            # three sets, a single k tile
    (256, 384, 448, 1, "1,6,3"),           # three sets, 7 k tiles
    (1024, 2048, 512, 1, None),            # tiny workload FFN-1
    (1024, 4608, 1536, 0, None),           # 1.3B QKV
    (1024, 1536, 8960, 2, None),           # 1.3B FFN-2
    (1024, 15360, 5120, 0, None),          # 14B QKV: 240 tiles of 256 x 256
    (1000, 1536, 512, 0, "d1"),            # 256 x 256, ragged M
    (5, 384, 320, 2, "d1"),                # a single row group of fewer than eight rows, half a tile past the columns
    (259, 512, 256, 0, "d1"),              # the second tile row holds three rows
    (1023, 15360, 320, 0, "d1"),           # several tiles per workgroup up to a short last row group
    (300, 640, 192, 3, "d2"),              # 192 x 256, N not a multiple of the tile, 3 k tiles
    (256, 256, 64, 2, "d2"),               # a single k tile
    (520, 2048, 1024, 1, "d3"),            # 256 x 192, one wave per SIMD, GELU
    (128, 512, 512, 2, "d4"),              # 256 x 160, a single ragged M tile
    (260, 384, 128, 0, "d3"),              # two k tiles in rings of two and three stages
    (1000, 1536, 512, 1, "d5"),            # 256 x 128, GELU, ragged M
    (300, 640, 192, 2, "d6"),              # 192 x 192, N not a multiple of the tile, 3 k tiles
    (256, 256, 64, 3, "d6"),               # one k tile: fewer than the rings hold
    (130, 256, 32 * 2, 0, "d5"),           # the same, a single ragged M tile
    (520, 768, 1024, 2, "d6,3"),           # three k parts (fp32 partial sums + reduce), gated residual
    (1000, 512, 640, 1, "d5,2"),           # two k parts, GELU in the reduce pass, ragged M
    (1000, 1536, 512, 1, "d17"),           # 64 x 32, rings of six stages; GELU, ragged M
    (300, 640, 192, 2, "d18"),             # 32 x 32, rings of eight stages, 3 k tiles
    (256, 256, 64, 3, "d18"),              # one k tile
    (130, 256, 128, 0, "d17"),             # two k tiles
    (520, 768, 1024, 2, "d18,3"),          # three k parts
    (2048, 2048, 2048, 0, "d18"),          # 4096 tiles on 512 workgroups, 32 k tiles
    (1024, 1024, 320, 0, "d17"),           # five k tiles: one fewer than the rings hold
    (1024, 1024, 384, 0, "d18"),           # six k tiles of eight stages
    (300, 512, 1024, 2, "1,4,2,2"),        # k split in two parts + reduce kernel, gated residual, ragged M
    (260, 256, 2048, 3, "2,8,2,4"),        # four parts, residual
    (1024, 1536, 1536, 1, "1,5,2,3"),      # three parts, GELU in the reduce kernel, ragged N tile
    (130, 384, 192, 0, "1,3,2,8"),         # more parts asked than k allows: clamped to one part per two k tiles
    (300, 384, 320, 0, "d7"),              # 128 x 192, 5 k tiles
    (1024, 1536, 1536, 2, "d8"),           # 128 x 160: the C x C projections of the 1.3B block
    (200, 640, 192, 1, "d9"),              # 128 x 128, 3 k tiles in rings of four and five stages
    (260, 512, 448, 3, "d10"),             # 128 x 96
    (520, 768, 1024, 2, "d11,2"),          # 192 x 128, two k parts
    (333, 640, 512, 1, "d12"),             # 128 x 192 on four waves, two workgroups per unit; ragged M and N
    (1024, 8960, 1536, 1, "d13"),          # 128 x 64: FFN-1 of the 1.3B block, 1120 tiles
    (300, 1280, 256, 0, "d14"),            # 64 x 128
    (130, 768, 640, 2, "d15,3"),           # 64 x 96, three k parts
    (1000, 1536, 512, 1, "d16"),           # 64 x 64
    (1024, 1536, 8960, 2, "d15,4"),        # FFN-2 of the 1.3B block, four k parts
]


@pytest.mark.parametrize("M,N,K,epi,tile", GEMM_CASES)
def test_gemm_matches_oracle(M, N, K, epi, tile):
    a = bf16_randn((M, K), 1)
    w = bf16_randn((N, K), 2, 0.05)
    bias = bf16_randn((N,), 3, 0.5).float()
    rows_per_gate = max(M // 3, 1)
    n_gate = (M + rows_per_gate - 1) // rows_per_gate
    gate_a = bf16_randn((N,), 4, 0.3).float()
    gate_b = bf16_randn((n_gate, 2 * N), 5, 0.3).float()        # stride 2N: a strided table
    x0 = bf16_randn((M, N), 6).float()
    acc = oracle_linear(f64(a), f64(w), f64(bias))
    if epi == 0:
        want = acc
    elif epi == 1:
        want = oracle.gelu_tanh(acc)
    elif epi == 2:
        gate = f64(gate_a)[None, :] + f64(gate_b)[np.arange(M) // rows_per_gate, :N]
        want = f64(x0) + gate * acc
    else:
        want = f64(x0) + acc
    binding.tuning_set("gemm_tile", tile)
    try:
        # with the scratch the plan asks for (NaN-filled: every partial sum that is read was written), then without
        ws_bytes = binding.gemm_workspace_bytes(M, N, K, epi)
        ws = torch.full((ws_bytes // 4,), float("nan"), dtype=torch.float32, device=DEV) if ws_bytes else None
        for workspace in ([ws, None] if ws is not None else [None]):
            out = (torch.empty(M, N, dtype=torch.bfloat16) if epi < 2 else x0.clone()).to(DEV)
            binding.gemm_bf16(a.to(DEV), w.to(DEV), bias.to(DEV), out, epi, gate_a.to(DEV), gate_b.to(DEV), 2 * N,
                              rows_per_gate, workspace=workspace)
            torch.cuda.synchronize()
            err = max_rel_err(f64(out), want)
            assert err < (1e-2 if epi < 2 else 1e-4), err
    finally:
        binding.tuning_set("gemm_tile", None)


@pytest.mark.parametrize("tile", range(1, 19))
@pytest.mark.parametrize("M,N,K,epi", [
    (1, 128, 64, 0),            # one row, one k tile: fewer than any ring of stages holds
    (257, 384, 128, 1),         # one row past the largest tile
    (515, 640, 704, 2),         # ragged in both directions, eleven k tiles
    (5200, 3328, 640, 3),       # more tiles than workgroups for the small tiles: the next tile's loads under the epilogue
])
def test_gemm_every_tile_at_its_edges(M, N, K, epi, tile):
    test_gemm_matches_oracle(M, N, K, epi, "d%d" % tile)


@pytest.mark.parametrize("tile", range(1, 19))
@pytest.mark.parametrize("epi,biased", [(0, True), (0, False), (1, False), (2, True), (2, False), (3, False)])
def test_gemm_several_tiles_per_workgroup(epi, biased, tile):
    """More output tiles than workgroups for every tile size, ten k tiles (more than any ring holds): the next tile's loads
    run under the stores.  Without a bias no load marks that they have landed, and the stores are waited for with them; bf16
    and fp32 stores; gates of 100 rows, so that the gate changes inside a wave's tile."""
    M, N, K, rows_per_gate = 5200, 3328, 640, 100
    g = torch.Generator(device=DEV).manual_seed(40 + epi)
    rand = lambda *shape: torch.randn(*shape, generator=g, device=DEV)
    a, w = rand(M, K).to(torch.bfloat16), (rand(N, K) * 0.05).to(torch.bfloat16)
    bias = rand(N) if biased else None
    gate_a, gate_b, x0 = rand(N), rand(M // rows_per_gate, N), rand(M, N)
    acc = a.double() @ w.double().t()
    if biased:
        acc += bias.double()
    if epi == 1:
        acc = torch.nn.functional.gelu(acc, approximate="tanh")
    elif epi == 2:
        acc = x0 + acc * (gate_a + gate_b.repeat_interleave(rows_per_gate, 0)).double()
    elif epi == 3:
        acc = x0 + acc
    binding.tuning_set("gemm_tile", "d%d" % tile)
    try:
        for _ in range(2):
            out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV) if epi < 2 else x0.clone()
            binding.gemm_bf16(a, w, bias, out, epi, gate_a, gate_b, N, rows_per_gate)
            torch.cuda.synchronize()
            err = ((out.double() - acc).abs().max() / acc.abs().max()).item()
            assert err < (1e-2 if epi < 2 else 1e-4), err
    finally:
        binding.tuning_set("gemm_tile", None)


@pytest.mark.parametrize("heads,tokens", [(26, 77), (40, 128), (40, 77), (12, 512), (4, 16)])
def test_text_keys_and_values_in_one_launch(heads, tokens):
    """The two products of a prompt in one launch: the first three shapes would be split in k with scratch.  Keys (after their
    RMSNorm) and values against 64 bits."""
    C = 128 * heads
    g = torch.Generator(device=DEV).manual_seed(heads)
    rand = lambda *shape: torch.randn(*shape, generator=g, device=DEV)
    t = {"W_ck": (rand(C, C) * 0.02).to(torch.bfloat16), "W_cv": (rand(C, C) * 0.02).to(torch.bfloat16), "b_ck": rand(C) * 0.02,
         "b_cv": rand(C) * 0.02, "g_ck": 1.0 + 0.1 * rand(C)}
    ctx = rand(tokens, C).to(torch.bfloat16)
    cfg = binding.model_cfg(C, heads, 4 * C, 2, 2, tokens, 1)
    cap = (tokens + 63) // 64 * 64
    kt, vtt = (torch.zeros(binding.text_kv_bytes(cfg), dtype=torch.uint8, device=DEV) for _ in range(2))
    binding.text_kv_prepare(cfg, binding.block_weights(t), ctx, kt, vtt,
                            torch.empty(binding.text_kv_workspace_bytes(cfg), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    K = kt.view(torch.bfloat16).view(heads, cap, 128)[:, :tokens].permute(1, 0, 2).reshape(tokens, C)
    V = vtt.view(torch.bfloat16).view(heads, 128, cap)[:, :, binding.vt_columns(cap).to(DEV)][:, :, :tokens].permute(2, 0, 1).reshape(tokens, C)
    k, v = (ctx.double() @ t["W_" + n].double().t() + t["b_" + n].double() for n in ("ck", "cv"))
    k = k / (k.pow(2).mean(1, keepdim=True) + 1e-6).sqrt() * t["g_ck"].double()
    assert max_rel_err(f64(K), f64(k)) < 1e-2 and max_rel_err(f64(V), f64(v)) < 1e-2


# heads in every step of the append kernel's widths, beyond 40 with gains that come a few steps ahead of their use
@pytest.mark.parametrize("heads", [7, 16, 21, 29, 41, 44, 53, 63, 64])
def test_text_keys_of_every_width(heads):
    test_text_keys_and_values_in_one_launch(heads, 35)


@pytest.mark.parametrize("tile", [None, "1,4"] + ["d%d" % i for i in range(1, 19)])
def test_gemm_adds_the_bias_to_the_finished_sum(tile):
    """A bias 25 times the product's size must not coarsen the sum of the products: fp32 output against 64 bits.  One
    rounding of the result (2^-24 relative, at most) and the sum's own error (1e-6 of the product, above the 6e-7 that a
    chain of 4096 terms shows): 1.0e-7 of the result.  Accumulators that start from the bias show 5e-7."""
    M, N, K = 300, 640, 4096
    a, w = bf16_randn((M, K), 21).to(DEV), bf16_randn((N, K), 22, 0.02).to(DEV)
    g = torch.Generator().manual_seed(23)
    bias = (torch.randn(N, generator=g) * 32.0).to(DEV)
    acc = a.double() @ w.double().t()
    want = acc + bias.double()
    out = torch.zeros(M, N, device=DEV)
    binding.tuning_set("gemm_tile", tile)
    try:
        binding.gemm_bf16(a, w, bias, out, 3)
        torch.cuda.synchronize()
    finally:
        binding.tuning_set("gemm_tile", None)
    err = (out.double() - want).norm().item()
    assert err <= 2.0 ** -24 * want.norm().item() + 1e-6 * acc.norm().item(), err / want.norm().item()


def test_gemm_of_a_long_sum_is_split_in_three():
    """FFN-2 of the 14B-shaped block (1024 x 5120 x 13824), fp32 output, against 64 bits.  The rounding error of a sum grows
    with the root of its longest chain: 4.2e-7 relative for chains of 4608 products, 5.2e-7 for 6912, 7.5e-7 for all of
    them.  The bar lies between the first two."""
    M, N, K = 1024, 5120, 13824
    g = torch.Generator(device=DEV).manual_seed(1)
    a = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    ws = torch.empty(binding.gemm_workspace_bytes(M, N, K, 3), dtype=torch.uint8, device=DEV)
    out = torch.zeros(M, N, device=DEV)
    binding.gemm_bf16(a, w, None, out, 3, workspace=ws)
    want = a.double() @ w.double().t()
    err = ((out.double() - want).norm() / want.norm()).item()
    assert err <= 4.7e-7, err


def test_gemm_of_rows_so_wide_that_a_tile_spans_4_gib():
    """64 rows of 16 908 288 fp32 columns: a row index times the row's bytes exceeds 32 bits in the last rows.  Residual
    epilogue; every row at columns from both ends and the middle."""
    M, N, K = 64, 16908288, 64
    g = torch.Generator(device=DEV).manual_seed(12)
    a = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
    w = torch.randn(N, K, generator=g, device=DEV, dtype=torch.bfloat16)
    out = torch.empty(M, N, device=DEV)
    out.copy_(torch.arange(M, device=DEV, dtype=torch.float32)[:, None])
    binding.gemm_bf16(a, w, None, out, 3)
    for c0 in (0, N // 2 - 4096, N - 8192):
        want = torch.arange(M, device=DEV)[:, None] + a.double() @ w[c0:c0 + 8192].double().t()
        assert max_rel_err(f64(out[:, c0:c0 + 8192]), f64(want)) < 1e-4, c0


@pytest.mark.parametrize("a0,w0", [(0, 2), (1, 0), (2, 1), (4, 4)])
@pytest.mark.parametrize("M,N,K,epi", [(257, 384, 128, 0), (1024, 1536, 1536, 3)])
def test_gemm_of_operands_at_any_address(M, N, K, epi, a0, w0):
    """Operands that start 2 to 8 bytes past a multiple of 16: loads straight into LDS need the multiple, so such a call goes
    to the kernel that loads into registers; a forced tile of the other kernel is refused."""
    g = torch.Generator(device=DEV).manual_seed(50)
    rand = lambda n, scale: (torch.randn(n, generator=g, device=DEV) * scale).to(torch.bfloat16)
    a, w = rand(M * K + 8, 1.0)[a0:a0 + M * K].view(M, K), rand(N * K + 8, 0.05)[w0:w0 + N * K].view(N, K)
    assert (a.data_ptr() | w.data_ptr()) % 16 != 0
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV) if epi == 0 else torch.zeros(M, N, device=DEV)
    binding.tuning_set("gemm_tile", "d5")
    try:
        with pytest.raises(binding.Sdv2Error):
            binding.gemm_bf16(a, w, None, out, epi)
    finally:
        binding.tuning_set("gemm_tile", None)
    binding.gemm_bf16(a, w, None, out, epi)
    torch.cuda.synchronize()
    assert max_rel_err(f64(out), f64(a.double() @ w.double().t())) < (1e-2 if epi < 2 else 1e-4)


@pytest.mark.parametrize("offset", [2, 4, 6])
def test_append_of_rows_at_any_address(offset):
    P, H = 6, 5
    ccfg = binding.cache_cfg(1, 1, H, P, P, 2 * P)
    storage = torch.full((binding.kv_cache_bytes(ccfg),), 0xFF, dtype=torch.uint8, device=DEV)
    h = binding.kv_cache_init(ccfg, storage)
    n = P * H * 128
    k, v = (bf16_randn((n + 8,), s).to(DEV)[offset:offset + n].view(P, H * 128) for s in (1, 2))
    binding.kv_cache_append_evict(h, 0, 0, k, v)
    torch.cuda.synchronize()
    _, _, _, cap = binding.kv_cache_device_ptrs(h, 0, 0)
    K = storage[:H * cap * 256].view(torch.bfloat16).view(H, cap, 128)[:, :P].permute(1, 0, 2).reshape(P, H * 128)
    V = storage[H * cap * 256:2 * H * cap * 256].view(torch.bfloat16).view(H, 128, cap)
    V = V[:, :, binding.vt_columns(cap).to(DEV)][:, :, :P].permute(2, 0, 1).reshape(P, H * 128)
    assert torch.equal(K, k) and torch.equal(V, v)
    binding.kv_cache_destroy(h)


def test_gemm_full_size_batched_480p_shape_sampled_rows():
    """FFN-1 of the 14B-shaped block on 4 streams x 4680 tokens (M 18720, N 13824, K 5120: the direct-load kernel,
    74 x 54 tiles, ragged last M tile): whole output finite, 48 sampled rows against the oracle."""
    M, N, K = 18720, 13824, 5120
    g = torch.Generator(device=DEV).manual_seed(7)
    a = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    bias = (torch.randn(N, generator=g, device=DEV) * 0.5).to(torch.bfloat16).float()
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    binding.gemm_bf16(a, w, bias, out, 1)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    rows = sorted(set(np.random.default_rng(0).integers(0, M, 44).tolist()) | {0, 255, 256, M - 1})
    want = oracle.gelu_tanh(oracle_linear(f64(a[rows]), f64(w), f64(bias)))
    assert max_rel_err(f64(out[rows]), want) < 1e-2


def test_gemm_rejects_bad_shapes():
    a = torch.zeros(8, 100, dtype=torch.bfloat16, device=DEV)
    w = torch.zeros(128, 100, dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(8, 128, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(binding.Sdv2Error) as e:
        binding.gemm_bf16(a, w, None, out)
    assert e.value.code == binding.INVALID_ARG


# ------------------------------------------------------------------------------------------ attention
def pack_kv(k_rows, v_rows, H, cap):
    """Token rows [n, C] -> the cache layouts K [H][cap][128], V^T [H][128][cap] (slot s in column vt_columns[s]);
    padding slots are NaN."""
    n, Cw = k_rows.shape
    D = Cw // H
    K = torch.full((H, cap, D), float("nan"), dtype=torch.bfloat16)
    VT = torch.full((H, D, cap), float("nan"), dtype=torch.bfloat16)
    K[:, :n, :] = k_rows.reshape(n, H, D).permute(1, 0, 2)
    VT[:, :, binding.vt_columns(cap)[:n]] = v_rows.reshape(n, H, D).permute(1, 2, 0)
    return K.contiguous(), VT.contiguous()


ATTN_CASES = [
    # B, L, H, kv_lens, forced splits
    (1, 128, 1, [64], 0),
    (1, 32, 2, [1], 0),                    # a single key
    (1, 100, 2, [63], 0),                  # ragged queries and keys inside one tile
    (1, 130, 2, [65], 0),                  # one key into the second tile
    (2, 300, 3, [384, 129], 0),            # two streams with different lengths
    (1, 128, 4, [384], 3),                 # split-KV, merged
    (2, 200, 2, [1000, 70], 4),            # a stream with fewer tiles than splits
    (1, 1024, 12, [3072], 0),              # 1.3B steady state (planner's split)
    (1, 1024, 12, [512], 0),               # text cross-attention shape
    (1, 70, 2, [200], 0),                  # a 128-key tile and a tail of 72: slices 2 and 3 of the tail hold 8 and 0 keys
    (2, 64, 1, [40, 129], 0),              # fewer keys than one slice; one key into the second 128-key tile
]


# waves 0: the planner's choice; 4 / 8: 128 / 256 queries per workgroup, one key stream; 2: the key-split form
# (2 query blocks x 4 key slices per workgroup, 128-key tiles, capacity a multiple of 128)
@pytest.mark.parametrize("waves", [0, 4, 8, 2])
@pytest.mark.parametrize("B,L,H,kv_lens,splits", ATTN_CASES)
def test_attention_matches_oracle(B, L, H, kv_lens, splits, waves):
    D = 128
    Cw = H * D
    q = bf16_randn((B, L, Cw), 10)
    ks, vts, caps, want = [], [], [], []
    for b, n in enumerate(kv_lens):
        k_rows = bf16_randn((n, Cw), 20 + b)
        v_rows = bf16_randn((n, Cw), 30 + b)
        cap = (n + 127) // 128 * 128 + 128 * (b % 2) if waves == 2 else (n + 63) // 64 * 64 + 64 * (b % 2)
        K, VT = pack_kv(k_rows, v_rows, H, cap)
        ks.append(K.to(DEV))
        vts.append(VT.to(DEV))
        caps.append(cap)
        want.append(oracle.attention_dense(f64(q[b]).reshape(L, H, D), f64(k_rows).reshape(n, H, D),
                                           f64(v_rows).reshape(n, H, D)).reshape(L, Cw))
    o = torch.full((B, L, Cw), float("nan"), dtype=torch.bfloat16, device=DEV)
    binding.tuning_set("attn_splits", splits or None)
    binding.tuning_set("attn_waves", waves or None)
    try:
        ws = torch.empty(max(binding.attention_workspace_bytes(B, L, Cw, max(kv_lens)), 256), dtype=torch.uint8, device=DEV)
        binding.attention_bf16(q.to(DEV), ks, vts, kv_lens, caps, o, H, ws)
        torch.cuda.synchronize()
    finally:
        binding.tuning_set("attn_splits", None)
        binding.tuning_set("attn_waves", None)
    got = f64(o)
    assert np.isfinite(got).all()
    for b in range(B):
        err = max_rel_err(got[b], want[b])
        assert err < 1e-2, (b, err)


def test_attention_workspace_of_the_longest_range_serves_the_shorter_ones():
    L, H, D, longest = 748, 9, 128, 8648
    q, k_rows, v_rows = (bf16_randn((n, H * D), 40 + i) for i, n in enumerate((L, longest, longest)))
    ws = torch.empty(binding.attention_workspace_bytes(1, L, H * D, longest), dtype=torch.uint8, device=DEV)
    for n in (longest, 7003, 700, 64):
        cap = (n + 63) // 64 * 64
        K, VT = pack_kv(k_rows[:n], v_rows[:n], H, cap)
        o = torch.full((1, L, H * D), float("nan"), dtype=torch.bfloat16, device=DEV)
        binding.attention_bf16(q[None].to(DEV), [K.to(DEV)], [VT.to(DEV)], [n], [cap], o, H, ws)
        heads = lambda x: x.to(DEV).float().reshape(-1, H, D).transpose(0, 1)
        p = torch.softmax(heads(q) @ heads(k_rows[:n]).transpose(1, 2) / math.sqrt(D), dim=-1)
        want = (p @ heads(v_rows[:n])).transpose(0, 1).reshape(1, L, H * D)
        assert max_rel_err(f64(o), f64(want)) < 1e-2, n


# Query tiles, heads, streams and parts that are one, odd, or no divisors of the eight XCDs over which the workgroups are
# numbered; a chunk that ends one query into a tile, whose other rows are copies of its last.
@pytest.mark.parametrize("waves", [4, 8, 2])
@pytest.mark.parametrize("B,L,H,kv_lens,splits", [
    (1, 1, 1, [1], 0),
    (3, 257, 5, [70, 200, 65], 1),
    (2, 129, 3, [330, 260], 2),
    (8, 33, 1, [64, 1, 65, 127, 128, 129, 63, 200], 1),
])
def test_attention_workgroup_numbering(B, L, H, kv_lens, splits, waves):
    test_attention_matches_oracle(B, L, H, kv_lens, splits, waves)


# Streams with fewer key tiles than the launch has parts, beside one that has more: of the parts without tiles the first is
# first in the range.  A stream's tiles may all be full (64, 192, 256, 320 keys) or not.
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("B,L,H,kv_lens,splits", [
    (2, 70, 2, [256, 64], 2),
    (4, 130, 3, [64, 192, 1024, 70], 5),
    (3, 300, 1, [320, 2048, 256], 12),
    (8, 33, 2, [64, 2112, 128, 960, 1, 1023, 576, 65], 16),
])
def test_attention_of_streams_with_fewer_tiles_than_parts(B, L, H, kv_lens, splits, waves):
    assert min(kv_lens) <= 64 * (splits - 1) and max(kv_lens) >= 128 * splits         # so many parts are made
    test_attention_matches_oracle(B, L, H, kv_lens, splits, waves)


@pytest.mark.parametrize("waves,splits", [(4, 1), (4, 2), (8, 1), (8, 3), (2, 1)])
@pytest.mark.parametrize("q0,o0", [(1, 0), (2, 1), (4, 4), (0, 2)])
def test_attention_of_queries_at_any_address(q0, o0, waves, splits):
    """Queries and outputs that start 2 to 8 bytes past a multiple of 16: loads straight into LDS need the multiple, so such
    queries are fetched into registers.  Chunks that end inside a tile and inside a wave, tails of keys."""
    B, L, H, kv_lens = 2, 157, 3, [450, 384]
    Cw, n = H * 128, B * L * H * 128
    q = bf16_randn((n + 8,), 10).to(DEV)[q0:q0 + n].view(B, L, Cw)
    o = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device=DEV)[o0:o0 + n].view(B, L, Cw)
    assert (q.data_ptr() | o.data_ptr()) % 16 != 0
    rows = [(bf16_randn((m, Cw), 20 + b), bf16_randn((m, Cw), 30 + b)) for b, m in enumerate(kv_lens)]
    caps = [512, 384]
    packed = [pack_kv(k, v, H, cap) for (k, v), cap in zip(rows, caps)]
    ks, vts = [p[0].to(DEV) for p in packed], [p[1].to(DEV) for p in packed]
    binding.tuning_set("attn_splits", splits)
    binding.tuning_set("attn_waves", waves)
    try:
        ws = torch.empty(max(binding.attention_workspace_bytes(B, L, Cw, max(kv_lens)), 256), dtype=torch.uint8, device=DEV)
        binding.attention_bf16(q, ks, vts, kv_lens, caps, o, H, ws)
        torch.cuda.synchronize()
    finally:
        binding.tuning_set("attn_splits", None)
        binding.tuning_set("attn_waves", None)
    for b, m in enumerate(kv_lens):
        want = oracle.attention_dense(f64(q[b]).reshape(L, H, 128), f64(rows[b][0]).reshape(m, H, 128),
                                      f64(rows[b][1]).reshape(m, H, 128)).reshape(L, Cw)
        assert max_rel_err(f64(o[b]), want) < 1e-2


# Score profiles along the key index, in log2 units of the exponent (what the kernel's running reference point is
# measured in).  The kernels keep that reference only loosely behind the row maximum and form no maximum in the
# steady state, so these walk through every way the reference has to move: maxima that keep growing across tiles,
# one key far above everything seen, scores far above and far below zero from the first key on, maxima that only fall.
SCORE_PROFILES = {
    "growing": lambda j, n: 100.0 * j / n,
    "falling": lambda j, n: 100.0 * (1.0 - j / n),
    "spike": lambda j, n: np.where(j == n // 2 + 3, 200.0, 0.0),
    "huge": lambda j, n: 300.0 + 5.0 * np.sin(j),
    "far below zero": lambda j, n: -300.0 + 5.0 * np.sin(j),
    "steps": lambda j, n: 20.0 * (j // 90),
}


@pytest.mark.parametrize("waves,splits", [(0, 0), (4, 0), (8, 0), (2, 0), (4, 3)])
@pytest.mark.parametrize("profile", sorted(SCORE_PROFILES))
def test_attention_score_ranges(profile, waves, splits):
    """q_i = a_i u + noise, k_j = b_j u + noise with u in {-1, +1}^128, so that the scaled score of (i, j) in log2 units is
    about a_i T(j): a_i runs from 0.5 to 1.5 over the queries and is negated for every third query (its profile is
    mirrored), so the lanes of a wave need their reference moved at different tiles, and some never."""
    L, H, D, n = 96, 2, 128, 700
    Cw = H * D
    g = torch.Generator().manual_seed(77)
    u = (torch.randint(0, 2, (H, D), generator=g) * 2 - 1).to(torch.float32)
    per_unit = math.sqrt(D) * math.log2(math.e)          # log2-domain score of a = b = 1
    j = np.arange(n)
    b_j = torch.tensor(np.asarray(SCORE_PROFILES[profile](j, n), dtype=np.float64) / per_unit, dtype=torch.float32)
    a_i = 0.5 + torch.arange(L, dtype=torch.float32) / L
    a_i[::3] *= -1.0
    q = (a_i[:, None, None] * u[None] + 0.1 * torch.randn(L, H, D, generator=g)).to(torch.bfloat16).reshape(1, L, Cw)
    k_rows = (b_j[:, None, None] * u[None] + 0.1 * torch.randn(n, H, D, generator=g)).to(torch.bfloat16).reshape(n, Cw)
    v_rows = bf16_randn((n, Cw), 78)
    cap = (n + 127) // 128 * 128
    K, VT = pack_kv(k_rows, v_rows, H, cap)
    want = oracle.attention_dense(f64(q[0]).reshape(L, H, D), f64(k_rows).reshape(n, H, D),
                                  f64(v_rows).reshape(n, H, D)).reshape(L, Cw)
    o = torch.full((1, L, Cw), float("nan"), dtype=torch.bfloat16, device=DEV)
    binding.tuning_set("attn_splits", splits or None)
    binding.tuning_set("attn_waves", waves or None)
    try:
        ws = torch.empty(max(binding.attention_workspace_bytes(1, L, Cw, n), 256), dtype=torch.uint8, device=DEV)
        binding.attention_bf16(q.to(DEV), [K.to(DEV)], [VT.to(DEV)], [n], [cap], o, H, ws)
        torch.cuda.synchronize()
    finally:
        binding.tuning_set("attn_splits", None)
        binding.tuning_set("attn_waves", None)
    got = f64(o)
    assert np.isfinite(got).all()
    err = max_rel_err(got[0], want)
    assert err < 1e-2, err


def test_attention_full_size_480p_shape_sampled_queries():
    """Self-attention of the 14B 480p workload at steady state for one stream (4680 queries, 40 heads, 10 920 resident
    slots = 170 tiles and a tail of 40): whole output finite, 24 sampled queries x all heads against the oracle."""
    L, H, D, n = 4680, 40, 128, 10920
    Cw = H * D
    cap = (n + 63) // 64 * 64
    g = torch.Generator(device=DEV).manual_seed(11)
    q = torch.randn(1, L, Cw, generator=g, device=DEV).to(torch.bfloat16)
    k_rows = torch.randn(n, Cw, generator=g, device=DEV).to(torch.bfloat16)
    v_rows = torch.randn(n, Cw, generator=g, device=DEV).to(torch.bfloat16)
    K = torch.full((H, cap, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    VT = torch.full((H, D, cap), float("nan"), dtype=torch.bfloat16, device=DEV)
    K[:, :n, :] = k_rows.reshape(n, H, D).permute(1, 0, 2)
    VT[:, :, binding.vt_columns(cap)[:n].to(DEV)] = v_rows.reshape(n, H, D).permute(1, 2, 0)
    o = torch.full((1, L, Cw), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(max(binding.attention_workspace_bytes(1, L, Cw, n), 256), dtype=torch.uint8, device=DEV)
    binding.attention_bf16(q, [K], [VT], [n], [cap], o, H, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    rows = sorted(set(np.random.default_rng(1).integers(0, L, 20).tolist()) | {0, 127, 128, L - 1})
    want = oracle.attention_dense(f64(q[0, rows]).reshape(len(rows), H, D), f64(k_rows).reshape(n, H, D),
                                  f64(v_rows).reshape(n, H, D)).reshape(len(rows), Cw)
    assert max_rel_err(f64(o[0, rows]), want) < 1e-2


# ------------------------------------------------------------------------------------------ standalone cache
CACHE_CASES = [
    # P, S_frames, W_frames, heads, chunk sizes in frames (advance flag per chunk: True unless negative)
    (6, 1, 2, 1, [1, 1, 1, 1, 1, 1]),
    (15, 1, 6, 2, [3, 3, 3, 3, 3]),        # first chunk straddles sink and ring; third wraps mid-append
    (70, 0, 3, 1, [1, 2, 3, 1, 2]),        # no sink, tiles of 64 tokens with ragged tails
    (8, 2, 4, 3, [1, 1, 2, -2, 4, -4, 1]), # negative: same size again with advance = 0
]


@pytest.mark.parametrize("P,Sf,Wf,H,sizes", CACHE_CASES)
def test_append_evict_is_bit_exact(P, Sf, Wf, H, sizes):
    D = 128
    Cw = H * D
    S, W = Sf * P, Wf * P
    ccfg = binding.cache_cfg(2, 2, H, P, S, W)
    storage = torch.full((binding.kv_cache_bytes(ccfg),), 0xFF, dtype=torch.uint8, device=DEV)
    h = binding.kv_cache_init(ccfg, storage)
    layer, stream = 1, 1
    oc = oracle.RollingKVCache(S, W, P, Cw)
    for i, frames in enumerate(sizes):
        n = abs(frames) * P
        k = bf16_randn((n, Cw), 100 + i)
        v = bf16_randn((n, Cw), 200 + i)
        binding.kv_cache_append_evict(h, layer, stream, k.to(DEV), v.to(DEV), advance=frames > 0)
        oc.append_evict(f64(k), f64(v), advance=frames > 0)
        torch.cuda.synchronize()
        assert binding.kv_cache_state(h, layer, stream) == oc.state()
        want_map = oc.slot_map()
        assert binding.kv_cache_slot_map(h, layer, stream, S + W) == want_map.tolist()
        kp, vp, ip, cap = binding.kv_cache_device_ptrs(h, layer, stream)
        base = storage.data_ptr()
        nb = H * cap * D * 2
        K = storage[kp - base:kp - base + nb].view(torch.bfloat16).view(H, cap, D).permute(1, 0, 2).reshape(cap, Cw)
        V = storage[vp - base:vp - base + nb].view(torch.bfloat16).view(H, D, cap)
        V = V[:, :, binding.vt_columns(cap).to(DEV)].permute(2, 0, 1).reshape(cap, Cw)       # column order -> slot order
        ids = storage[ip - base:ip - base + cap * 8].view(torch.int64).cpu().numpy()
        live = want_map >= 0
        assert np.array_equal(ids[:S + W][live], want_map[live])
        ko, vo = oc.slot_contents()
        assert np.array_equal(f64(K)[:S + W][live], ko[live])          # copies: exact
        assert np.array_equal(f64(V)[:S + W][live], vo[live])
        # slots never written keep the poison
        assert torch.isnan(K[:S + W][torch.from_numpy(~live)].float()).all()
    # the other (layer, stream) pairs were not touched
    assert binding.kv_cache_state(h, 0, 0)["total"] == 0 and binding.kv_cache_state(h, 1, 0)["total"] == 0
    binding.kv_cache_reset(h, stream)
    assert binding.kv_cache_state(h, layer, stream)["total"] == 0
    binding.kv_cache_destroy(h)


@pytest.mark.parametrize("H", [4, 5, 12, 40, 63, 64, 65, 70])
def test_append_of_every_head_count(H):
    """Keys of all heads arrive (a row is copied in steps of four heads, compiled for up to 64): copies, so exact."""
    P, D = 6, 128
    ccfg = binding.cache_cfg(1, 1, H, P, P, 2 * P)
    storage = torch.full((binding.kv_cache_bytes(ccfg),), 0xFF, dtype=torch.uint8, device=DEV)
    h = binding.kv_cache_init(ccfg, storage)
    k, v = bf16_randn((P, H * D), H), bf16_randn((P, H * D), H + 1)
    binding.kv_cache_append_evict(h, 0, 0, k.to(DEV), v.to(DEV))
    torch.cuda.synchronize()
    kp, vp, _, cap = binding.kv_cache_device_ptrs(h, 0, 0)
    base, nb = storage.data_ptr(), H * cap * D * 2
    K = storage[kp - base:kp - base + nb].view(torch.bfloat16).view(H, cap, D)[:, :P].permute(1, 0, 2).reshape(P, H * D)
    V = storage[vp - base:vp - base + nb].view(torch.bfloat16).view(H, D, cap)
    V = V[:, :, binding.vt_columns(cap).to(DEV)][:, :, :P].permute(2, 0, 1).reshape(P, H * D)
    assert torch.equal(K.cpu(), k) and torch.equal(V.cpu(), v)
    binding.kv_cache_destroy(h)


def test_append_evict_errors_leave_state_untouched():
    P, H = 4, 1
    ccfg = binding.cache_cfg(1, 1, H, P, 4, 8)
    storage = torch.zeros(binding.kv_cache_bytes(ccfg), dtype=torch.uint8, device=DEV)
    h = binding.kv_cache_init(ccfg, storage)
    k = torch.zeros(4, 128, dtype=torch.bfloat16, device=DEV)
    binding.kv_cache_append_evict(h, 0, 0, k, k)
    before = binding.kv_cache_state(h, 0, 0)
    for bad_n, adv, code in ((12, True, binding.INVALID_ARG), (6, True, binding.INVALID_ARG), (8, False, binding.BAD_STATE)):
        kk = torch.zeros(bad_n, 128, dtype=torch.bfloat16, device=DEV)
        with pytest.raises(binding.Sdv2Error) as e:
            binding.kv_cache_append_evict(h, 0, 0, kk, kk, advance=adv)
        assert e.value.code == code
        assert binding.kv_cache_state(h, 0, 0) == before
    with pytest.raises(binding.Sdv2Error):
        binding.kv_cache_append_evict(h, 1, 0, k, k)
    binding.kv_cache_destroy(h)
