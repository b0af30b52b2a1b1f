"""Host-side checks that need no GPU: the built library loads, exports every symbol the header
declares, sizes its buffers as documented and rejects bad arguments before touching anything."""

import ctypes as C
import os
import random
import re
import struct
import subprocess

import pytest

from paper_2511_07399_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.load_library()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "sdv2.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(sdv2_[a-z0-9_]+)\s*\(", header))
    assert len(declared) >= 20
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    assert lib.sdv2_version() >= 1


def test_struct_sizes_match_the_header_layout():
    assert C.sizeof(binding.ModelCfg) == 44
    assert C.sizeof(binding.CacheCfg) == 28
    assert C.sizeof(binding.ChunkDesc) == 16
    assert C.sizeof(binding.CacheState) == 32
    assert C.sizeof(binding.BlockWeights) == 8 + 23 * 8
    assert C.sizeof(binding.ModelWeights) == 8 + 7 * 8


def test_cache_bytes_formula(lib):
    # per (layer, stream): K and V^T of n_heads * cap * 128 bf16 each, plus cap int64 ids; cap = 64-aligned S+W
    cfg = binding.cache_cfg(30, 1, 12, 1024, 1024, 2048)
    cap = 3072
    assert binding.kv_cache_bytes(cfg) == 30 * (2 * 12 * cap * 128 * 2 + cap * 8)
    cfg = binding.cache_cfg(2, 4, 40, 1560, 1560, 9360)
    cap = 10944                                   # 10920 rounded up to 64
    assert binding.kv_cache_bytes(cfg) == 8 * (2 * 40 * cap * 128 * 2 + cap * 8)


@pytest.mark.parametrize("args", [
    (1, 1, 1, 4, -4, 8),      # negative sink
    (1, 1, 1, 4, 4, 0),       # empty window
    (1, 1, 1, 4, 6, 8),       # sink not whole frames
    (1, 1, 1, 4, 4, 10),      # window not whole frames
    (0, 1, 1, 4, 4, 8),       # no layers
])
def test_cache_cfg_errors(lib, args):
    with pytest.raises(binding.Sdv2Error) as e:
        binding.kv_cache_bytes(binding.cache_cfg(*args))
    assert e.value.code == binding.INVALID_ARG


def test_empty_cache_state_and_init_errors(lib):
    cfg = binding.cache_cfg(2, 3, 1, 4, 4, 8)
    need = lib.sdv2_kv_cache_bytes(C.byref(cfg))
    h = C.c_void_p()
    fake = C.c_void_p(0x10000)                    # never dereferenced: init launches nothing
    assert lib.sdv2_kv_cache_init(C.byref(cfg), fake, need - 1, C.byref(h)) == binding.INVALID_ARG
    assert lib.sdv2_kv_cache_init(C.byref(cfg), None, need, C.byref(h)) == binding.INVALID_ARG
    assert lib.sdv2_kv_cache_init(C.byref(cfg), C.c_void_p(0x10010), need, C.byref(h)) == binding.INVALID_ARG
    assert lib.sdv2_kv_cache_init(C.byref(cfg), fake, need, C.byref(h)) == binding.OK
    st = binding.kv_cache_state(h, 1, 2)
    assert st == {"total": 0, "sink_fill": 0, "win_fill": 0, "oldest_slot": -1, "next_slot": 0, "evicted": 0}
    assert binding.kv_cache_slot_map(h, 1, 2, 12) == [-1] * 12
    with pytest.raises(binding.Sdv2Error):
        binding.kv_cache_state(h, 2, 0)
    with pytest.raises(binding.Sdv2Error):
        binding.kv_cache_state(h, 0, 3)
    binding.kv_cache_destroy(h)


def test_workspace_sizes_and_model_cfg_errors(lib):
    cfg = binding.model_cfg(1536, 12, 8960, 32, 32, 512, 30)
    rows, Cw, F = 1024, 1536, 8960
    # h, qkv, q, o, u in bf16 at least
    assert binding.block_workspace_bytes(cfg, 1, 1024) >= rows * (6 * Cw + F) * 2
    assert binding.denoise_workspace_bytes(cfg, 1, 1024) > binding.block_workspace_bytes(cfg, 1, 1024)
    assert binding.text_kv_bytes(cfg) == 512 * 1536 * 2
    bad = binding.model_cfg(1500, 12, 8960, 32, 32, 512, 30)
    assert binding.block_workspace_bytes(bad, 1, 1024) == 0
    assert binding.block_workspace_bytes(cfg, 9, 1024) == 0          # more streams than SDV2_MAX_BATCH


def test_slo_pick_batch_matches_the_oracle_on_random_tables():
    """Host-only entry point: the library's choice of B* against the oracle's on 500 random latency tables."""
    import numpy as np
    import oracle
    binding.load_library()
    g = np.random.default_rng(1)
    for trial in range(500):
        sizes = g.permutation(g.choice(np.arange(1, 20), size=int(g.integers(1, 7)), replace=False)).tolist()
        lat = {int(B): float(g.uniform(0.5, 3.0)) * (0.3 + B) * 1e-3 for B in sizes}
        T = int(g.integers(1, 5))
        f_slo = float(g.uniform(100, 3000))
        frames = int(g.integers(0, 60))
        tol = float(g.choice([0.0, 0.05, 0.2]))
        got = binding.slo_pick_batch(lat, T, f_slo, frames, tol)
        want = oracle.pick_batch(lat, T, f_slo, frames, tol)
        if want is None:
            assert got is None
        else:
            assert got[0] == want[0] and got[2] == want[2] and abs(got[1] - want[1]) <= 1e-9 * want[1]
    for bad in (lambda: binding.slo_pick_batch({0: 1.0}, 1, 1.0, 10), lambda: binding.slo_pick_batch({1: 0.0}, 1, 1.0, 10),
                lambda: binding.slo_pick_batch({1: 1.0}, 0, 1.0, 10), lambda: binding.slo_pick_batch({1: 1.0}, 1, 1.0, 10, 1.0)):
        try:
            bad()
            assert False, "accepted a bad argument"
        except binding.Sdv2Error as e:
            assert e.code == binding.INVALID_ARG


def test_bench_refuses_more_than_one_gpu():
    """This build runs on one GPU only: bench.py --gpus N with N > 1 says so and exits without touching a GPU."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2 and "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_stream_batch_handle_and_planner_hooks_on_the_host(lib):
    """Host-only parts of the newer entry points: stream-batch handle validation (nothing is launched), the planner's
    kernel names, and the tuning hook's parsing."""
    cfg = binding.model_cfg(512, 4, 2048, 8, 16, 64, 1)
    need = binding.stream_batch_rows_bytes(cfg, 4, 1)
    assert need >= 4 * 128 * 512 * 4
    assert binding.stream_batch_rows_bytes(cfg, 9, 1) == 0            # more depths than SDV2_MAX_BATCH
    fake = C.c_void_p(0x100000)                                       # never dereferenced by create
    h = C.c_void_p()
    ids = (C.c_int32 * 4)(0, 1, 2, 3)
    same = (C.c_int32 * 4)(0, 1, 1, 3)
    f = lib.sdv2_stream_batch_create
    assert f(C.byref(cfg), 4, same, 1, fake, need, C.byref(h)) == binding.INVALID_ARG
    assert f(C.byref(cfg), 4, ids, 1, fake, need - 256, C.byref(h)) == binding.WORKSPACE_TOO_SMALL
    assert f(C.byref(cfg), 4, ids, 1, C.c_void_p(0x100010), need, C.byref(h)) == binding.INVALID_ARG     # alignment
    assert f(C.byref(cfg), 0, ids, 1, fake, need, C.byref(h)) == binding.INVALID_ARG
    assert f(C.byref(cfg), 4, ids, 1, fake, need, C.byref(h)) == binding.OK
    assert lib.sdv2_stream_batch_reset(h) == binding.OK
    assert lib.sdv2_stream_batch_destroy(h) == binding.OK
    assert lib.sdv2_denoise_graph_state_bytes() >= 8 * (8 + 4 + 4 + 4)
    # the planner's kernel names: every shape within 32-bit offsets takes the direct-load kernel, the single-chunk attention
    # of the 1.3B block the key-split form, a capacity that is no multiple of 128 the one-key-stream form
    assert binding.prof_kernel_name("gemm", 4, 4680, 13824, 5120, 1).startswith("gemm_alt64_kernel<")
    # an activation matrix of 4 GiB or more is beyond the 32-bit lane offsets of the direct-load kernels
    assert binding.prof_kernel_name("gemm", 8, 40000, 8192, 8192, 0).startswith("gemm_kernel<")
    assert binding.prof_kernel_name("gemm", 8, 30000, 8192, 8192, 0).startswith("gemm_alt64_kernel<")
    # so are 64 rows of 20 million fp32 columns, which a wave's tile of that kernel could span; 32 rows are not
    assert binding.prof_kernel_name("gemm", 1, 64, 20971520, 64, 3).startswith("gemm_kernel<")
    assert binding.prof_kernel_name("gemm", 1, 32, 20971520, 64, 3).startswith("gemm_alt64_kernel<")
    assert binding.prof_kernel_name("attention", 1, 1024, 12, 3072, 3072) == "attention_ks_kernel<2, 4>"
    assert binding.prof_kernel_name("attention", 1, 1024, 12, 3072, 3136).startswith("attention_kernel<")
    assert binding.prof_kernel_name("attention", 4, 4680, 40, 10920, 10944) == "attention_kernel<8>"
    # the kernel of a sample that no profiled run has
    assert lib.sdv2_prof_sample_kernel(1 << 29, C.create_string_buffer(64), 64) == binding.INVALID_ARG
    assert lib.sdv2_prof_sample_kernel(0, None, 64) == binding.INVALID_ARG
    binding.tuning_set("gemm_tile", "1,3")
    try:
        assert binding.prof_kernel_name("gemm", 4, 4680, 13824, 5120, 1) == "gemm_kernel<1, 3, 64, 2>"
    finally:
        binding.tuning_set("gemm_tile", None)
    for name, value in (("gemm_tile", "9,9"), ("attn_waves", "3"), ("fetch_ahead", "2"), ("no_such_knob", "1")):
        with pytest.raises(binding.Sdv2Error) as e:
            binding.tuning_set(name, value)
        assert e.value.code == binding.INVALID_ARG
    assert binding.gemm_noalloc_max_scratch_bytes() == 32 << 20


def test_latent_io_sizes_and_refusals_on_the_host(lib):
    """Host-only parts of the latents-in / latents-out entry points: workspace sizes and the argument checks that
    come before any launch (nothing here touches a GPU)."""
    cfg = binding.model_cfg(512, 4, 2048, 8, 16, 64, 2)
    L = 8 * 16
    io_ws = binding.latent_io_workspace_bytes(cfg, 3, L)
    assert io_ws >= 3 * L * 512 * 2 + 3 * L * 64 * 4 and io_ws % 256 == 0
    assert binding.latent_io_workspace_bytes(cfg, 0, L) == 0 and binding.latent_io_workspace_bytes(cfg, 9, L) == 0
    total = binding.denoise_latents_workspace_bytes(cfg, 3, L)
    assert total >= binding.denoise_workspace_bytes(cfg, 3, L) + io_ws + 3 * L * 512 * 4
    fake = C.c_void_p(0x100000)                                       # never dereferenced: every call below is refused
    one = (C.c_float * 1)(0.5)
    big = (C.c_float * 1)(1.5)
    less = (C.c_float * 1)(0.25)
    assert lib.sdv2_noise_latents(None, fake, fake, 1, 1024, one, None) == binding.INVALID_ARG
    assert lib.sdv2_noise_latents(fake, fake, fake, 1, 1024, big, None) == binding.INVALID_ARG          # rate above 1
    assert lib.sdv2_noise_latents(fake, fake, fake, 9, 1024, one, None) == binding.INVALID_ARG          # too many streams
    assert lib.sdv2_sampler_update(fake, fake, fake, fake, None, 1, 1024, less, one, None) == binding.INVALID_ARG   # sigma grows
    assert lib.sdv2_sampler_update(fake, fake, None, fake, None, 1, 1024, one, less, None) == binding.INVALID_ARG   # noise missing
    assert lib.sdv2_sampler_update(fake, fake, fake, fake, None, 1, 0, one, less, None) == binding.INVALID_ARG
    io = binding.IoWeights()                                          # struct_size 0, null pointers
    assert lib.sdv2_patch_embed(C.byref(cfg), C.byref(io), fake, 1, 1, fake, fake, io_ws, None) == binding.INVALID_ARG
    assert lib.sdv2_output_head(C.byref(cfg), C.byref(io), fake, fake, 1, 1, fake, fake, io_ws, None) == binding.INVALID_ARG
    assert b"io weights" in lib.sdv2_last_error()
    assert lib.sdv2_prof_lds_rates(100, None, 40960, None) == binding.INVALID_ARG
    assert lib.sdv2_prof_lds_rates(100, fake, 1024, None) == binding.INVALID_ARG


def test_stream_batch_of_latents_sizes_on_the_host(lib):
    cfg = binding.model_cfg(512, 4, 2048, 8, 16, 64, 2)
    L = 8 * 16
    for n in (1, 2, 4):
        need = binding.stream_batch_latents_workspace_bytes(cfg, n, 1)
        assert need >= binding.denoise_latents_workspace_bytes(cfg, n, L) + n * 64 * L * 4
        # the rows buffer of the handle (hidden states) also holds the latent rows
        assert binding.stream_batch_rows_bytes(cfg, n, 1) >= n * 64 * L * 4
    assert binding.stream_batch_latents_workspace_bytes(cfg, 9, 1) == 0


@pytest.mark.parametrize("C_,heads,F", [(1536, 12, 8960), (3072, 24, 12288), (5120, 40, 13824)])
def test_a_workspace_for_a_batch_serves_smaller_ones(lib, C_, heads, F):
    """Fewer rows can split k where more rows do not: the size must grow with the rows all the same, because a workspace
    is made for the largest call (the stream batch fills up over calls of 1, 2, ... rows)."""
    for P in (32, 32), (30, 52):
        cfg = binding.model_cfg(C_, heads, F, P[0], P[1], 512, 30)
        sizes = [binding.block_workspace_bytes(cfg, B, P[0] * P[1]) for B in range(1, 9)]
        assert sizes[0] > 0 and sizes == sorted(sizes)


@pytest.mark.parametrize("C_,heads,F", [(512, 4, 2048), (1024, 8, 4096), (1536, 12, 8960), (5120, 40, 13824), (8192, 64, 24576)])
@pytest.mark.parametrize("grid", [(1, 4), (8, 16), (16, 16), (22, 39), (30, 52)])
def test_every_workspace_serves_fewer_streams_and_shorter_chunks(lib, C_, heads, F, grid):
    """The parts of a split key range take room too, and small frames split it in many parts: every size function grows with
    the streams and with the frames of a chunk, so that the call's own check never refuses a part of what was planned for."""
    cfg = binding.model_cfg(C_, heads, F, grid[0], grid[1], 512, 30)
    P = grid[0] * grid[1]
    for size in (lambda B, f: binding.block_workspace_bytes(cfg, B, f * P), lambda B, f: binding.denoise_workspace_bytes(cfg, B, f * P),
                 lambda B, f: binding.denoise_latents_workspace_bytes(cfg, B, f * P),
                 lambda B, f: binding.stream_batch_latents_workspace_bytes(cfg, B, f)):
        table = [[size(B, f) for f in range(1, 5)] for B in range(1, 9)]
        assert table[0][0] > 0
        assert all(row == sorted(row) for row in table), table
        assert all(list(col) == sorted(col) for col in zip(*table)), table


@pytest.mark.parametrize("M,N,K,epilogue,products", [
    (77, 3328, 3328, 0, 2), (128, 5120, 5120, 0, 2), (77, 5120, 5120, 0, 2), (512, 1536, 1536, 0, 2),      # text keys and values
    (1024, 64, 5120, 4, 1), (4680, 64, 5120, 4, 1),                                                        # output head
    (1024, 5120, 13824, 2, 1), (1560, 3072, 12288, 3, 1), (128, 5120, 5120, 2, 1), (300, 2560, 7680, 1, 1),
])
def test_a_plan_is_the_best_that_the_call_can_run(lib, M, N, K, epilogue, products):
    """Without scratch: no k split and, by the planner's own estimate, no better tile.  With scratch: as many parts as it
    holds, and never worse than a split in fewer parts or none; sums of more than 12 288 in at least three parts where they
    fit."""
    part = 4 * M * N
    cap = (64 if K > 12288 else 48) << 20
    for scratch in (0, part, 2 * part - 1, 2 * part, 3 * part + 5, 48 << 20, 1 << 40):
        least = 3 if K > 12288 and products == 1 and 3 * part <= min(scratch, cap) else 1
        tile, parts, us = binding.prof_gemm_plan(M, N, K, epilogue, products, scratch)
        assert 1 <= tile <= 18 and (parts == 1 or (products == 1 and parts * part <= scratch))
        others = []
        try:
            for want in (1, 2, 3, 4, 6):
                if want < least or (want > 1 and (products > 1 or want * part > min(scratch, cap) or K < 512 * want)):
                    continue
                for t in range(1, 19):
                    binding.tuning_set("gemm_tile", "d%d,%d" % (t, want))
                    assert binding.prof_gemm_plan(M, N, K, epilogue, products, scratch)[:2] == (t, want)
                    others.append(binding.prof_gemm_plan(M, N, K, epilogue, products, scratch)[2])
        finally:
            binding.tuning_set("gemm_tile", None)
        assert us == min(others)


def test_refresh_launches_cover_caches_beyond_32_bits(tmp_path):
    """The ranges that a sink copy and a key rotation are launched in: they cover every (head, token) once, and none holds
    more 16-byte pieces or heads than a launch can index.  One range at the sizes of a model."""
    source = tmp_path / "ranges.cpp"
    source.write_text('''
#include "refresh_ranges.h"
extern "C" int ranges(int H, int T, int pieces, int max_heads, int* out, int capacity) {
    int n = 0;
    sdv2::for_refresh_ranges(H, T, pieces, max_heads, [&](int h0, int hn, int t0, int tn) {
        if (n < capacity) { out[4 * n] = h0; out[4 * n + 1] = hn; out[4 * n + 2] = t0; out[4 * n + 3] = tn; }
        ++n;
    });
    return n;
}''')
    so = tmp_path / "ranges.so"
    csrc = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(source), "-o", str(so)], check=True)
    f = C.CDLL(str(so)).ranges
    for H, T, pieces, max_heads in ((12, 1560, 16, 12), (40, 10920, 6, 65535), (64, 1 << 20, 16, 64),      # models
                                    (1, 1 << 28, 16, 1), (1, 1 << 30, 6, 65535), (4, 1 << 26, 16, 4), (1024, 1 << 18, 16, 1024),
                                    (3, (1 << 28) + 5, 16, 3), (70000, 64, 6, 65535), (200000, 3, 6, 65535), (65535, 1, 1, 65535)):
        buf = (C.c_int * 4096)()
        n = f(H, T, pieces, max_heads, buf, 1024)
        assert 1 <= n <= 1024
        got = [tuple(buf[4 * i:4 * i + 4]) for i in range(n)]
        assert all(0 < hn <= max_heads and 0 < tn and hn * tn * pieces <= 1 << 31 for _, hn, _, tn in got)
        heads = sorted({(h0, hn) for h0, hn, _, _ in got})
        assert heads[0][0] == 0 and all(a + b == c for (a, b), (c, _) in zip(heads, heads[1:])) and sum(heads[-1]) == H
        for h in heads:
            tokens = [(t0, tn) for h0, hn, t0, tn in got if (h0, hn) == h]
            assert tokens[0][0] == 0 and all(a + b == c for (a, b), (c, _) in zip(tokens, tokens[1:])) and sum(tokens[-1]) == T
        assert (n == 1) == (H * T * pieces <= 1 << 31 and H <= max_heads)


def test_parts_of_a_key_range_cover_its_tiles_once(tmp_path):
    """The tiles that the parts of an attention's key range walk: every tile of the range once, the one with slots past the
    range as such, and none in a part without tiles (a range of fewer tiles than parts, its length a multiple of the tile or not)."""
    source = tmp_path / "tiles.cpp"
    source.write_text('''
#include "attention_ranges.h"
extern "C" void tiles(int kv_len, int tile, int part, int parts, int* out) {
    const sdv2::KeyTiles t = sdv2::key_tiles(kv_len, tile, part, parts);
    out[0] = t.first; out[1] = t.full; out[2] = t.end;
}''')
    so = tmp_path / "tiles.so"
    csrc = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(source), "-o", str(so)], check=True)
    f = C.CDLL(str(so)).tiles
    buf = (C.c_int * 3)()
    for kv_len in [*range(1, 1200), 3072, 4680, 10920, 1 << 30, (1 << 30) + 1]:
        n, whole = (kv_len + 63) // 64, kv_len // 64
        for parts in range(1, 17):
            at = 0
            for part in range(parts):
                f(kv_len, 64, part, parts, buf)
                first, full, end = buf
                assert first == at and first <= full <= end <= n, (kv_len, part, parts)
                assert full == max(first, min(end, whole)), (kv_len, part, parts)
                at = end
            assert at == n


# ------------------------------------------------------------------------------------------ what the compiler made of the kernels
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernel_metadata():
    """The metadata (registers, scratch) that the compiler left in the library's gfx950 code objects, by kernel name."""
    msgpack = pytest.importorskip("msgpack")
    data = open(binding.LIB_PATH, "rb").read()
    kernels, at = {}, data.find(BUNDLE)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + len(BUNDLE))[0], at + len(BUNDLE) + 8
        for _ in range(n):
            offset, size, chars = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + chars]:
                elf = data[at + offset:at + offset + size]
                sections, = struct.unpack_from("<Q", elf, 40)
                entry, count = struct.unpack_from("<HH", elf, 58)
                for s in range(count):
                    kind, _, _, start = struct.unpack_from("<IQQQ", elf, sections + s * entry + 4)
                    if kind == 7:                          # a note: the name's and the description's length, type, "AMDGPU", msgpack
                        name, desc, _ = struct.unpack_from("<III", elf, start)
                        first = start + 12 + (name + 3) // 4 * 4
                        for k in msgpack.unpackb(elf[first:first + desc])["amdhsa.kernels"]:
                            kernels[k[".name"]] = k
            p += 24 + chars
        at = data.find(BUNDLE, at + len(BUNDLE))
    return kernels


def test_matrix_kernels_spill_nothing(lib):
    """A spilled register is reloaded from memory, and the wait for it is a wait for every tile load in flight.  Of the ordinary
    kernels and of those that also read memory for other launches."""
    kernels = kernel_metadata()
    found = [(n, k) for n, k in kernels.items() if "gemm_alt64_kernel" in n or "attention_kernel" in n or "attention_ks_kernel" in n]
    fetching = [(n, k) for n, k in kernels.items() if "fetching_kernel" in n]
    assert len(found) == len(fetching) == 18 + 3
    found += fetching
    for name, k in found:
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, (name, k[".vgpr_spill_count"])


def test_row_kernels_leave_room_for_a_second_workgroup(lib):
    """Passes over rows hide their latencies behind each other: 512 registers hold two workgroups of four waves of up to 256."""
    found = [(n, k) for n, k in kernel_metadata().items() if "splitk_reduce_ln_kernel" in n or "plain_append_kernel" in n]
    assert found
    for name, k in found:
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_count"])


def test_attention_plan_keeps_to_its_scratch_and_counts_rounds(lib):
    """A planned number of parts stays within what the workspaces of a call are sized for (at most 16 parts of at least six
    64-key tiles, parts * B * L * heads up to 65 536), and the form of a launch follows its rounds, not workgroups alone."""
    rng = random.Random(11)
    for _ in range(3000):
        B, L, H, kv = rng.randint(1, 8), rng.randint(1, 3000), rng.randint(1, 40), rng.randint(1, 13000)
        per_part = B * L * H * (128 + 2) * 4
        n = binding.attention_workspace_bytes(B, L, 128 * H, kv)
        assert n % per_part < 256                     # rounded up
        parts = n // per_part
        if parts > 0:
            assert 2 <= parts <= 16 and (kv + 63) // 64 // parts >= 6 and parts * B * L * H <= 65536, (B, L, H, kv, parts)
    # a workspace for the longest key range of a program serves its shorter ones
    for B, L, H, lengths in [(1, 748, 9, (7003, 8648))] + [
            (rng.randint(1, 8), rng.randint(1, 2500), rng.randint(1, 40), sorted(rng.randint(1, 13000) for _ in range(8))) for _ in range(1500)]:
        sizes = [binding.attention_workspace_bytes(B, L, 128 * H, kv) for kv in lengths]
        assert sizes == sorted(sizes), (B, L, H, lengths, sizes)
    for (B, L, H, kv, cap), form in (((1, 1560, 12, 512, 512), "attention_kernel<4>"), ((8, 1024, 12, 3072, 3072), "attention_kernel<4>"),
                                     ((1, 1024, 12, 3072, 3072), "attention_ks_kernel<2, 4>"), ((1, 1024, 40, 3072, 3072), "attention_kernel<8>"),
                                     ((4, 4680, 40, 10920, 10944), "attention_kernel<8>")):
        assert binding.prof_kernel_name("attention", B, L, H, kv, cap) == form
