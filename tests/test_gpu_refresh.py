"""GPU parity of the adaptive sink refresh and the RoPE refresh (Section 4.1) against the CPU oracle.

Standalone cases feed the same bf16 K/V rows to the library's cache (sdv2_kv_cache_append_evict) and to the
oracle's, so that similarity is compared at fp32-vs-fp64 summation accuracy and the sink copy bit for bit; the
stream cases run the block on both sides around a refresh.  Bars: alpha within 2e-5 on identical inputs (fp32 partial
sums over up to 8 M products) and 5e-3 after the block (bf16 values against the oracle's fp64 ones); copies, ids,
slot maps and counters exact; rotated keys within one bf16 rounding of the oracle's (1e-2 of the largest key);
block outputs 2e-2.
"""

import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2511_07399_amd import binding, workloads as wk
from parity_util import GpuRunner, OracleRunner, max_rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class CachePair:
    """One (layer, stream) cache on the GPU and in the oracle, fed with the same rows."""

    def __init__(self, H, P, sink_frames, window_frames, seed=0):
        binding.load_library()
        self.H, self.P, self.C = H, P, H * 128
        self.S, self.W = sink_frames * P, window_frames * P
        self.ccfg = binding.cache_cfg(1, 1, H, P, self.S, self.W)
        self.storage = torch.full((binding.kv_cache_bytes(self.ccfg),), 0xFF, dtype=torch.uint8, device=DEV)
        self.handle = binding.kv_cache_init(self.ccfg, self.storage)
        self.ora = oracle.RollingKVCache(self.S, self.W, P, self.C)
        self.gen = torch.Generator().manual_seed(seed)
        self.ws = torch.empty(binding.sink_similarity_workspace_bytes(self.handle), dtype=torch.uint8, device=DEV)
        self.alpha = torch.empty(max(sink_frames, 1), dtype=torch.float32, device=DEV)

    def rows(self, n, scale=1.0):
        return (torch.randn(n, self.C, generator=self.gen) * scale).to(torch.bfloat16)

    def append(self, k, v, advance=True):
        binding.kv_cache_append_evict(self.handle, 0, 0, k.to(DEV), v.to(DEV), advance)
        self.ora.append_evict(k.double().numpy(), v.double().numpy(), advance=advance)

    def similarity(self, frame_back=0):
        binding.sink_similarity(self.handle, 0, 0, self.alpha, self.ws, frame_back)
        torch.cuda.synchronize()
        return self.alpha.cpu().numpy().astype(np.float64), oracle.sink_similarity(self.ora, frame_back)

    def logical(self):
        kp, vp, ip, cap = binding.kv_cache_device_ptrs(self.handle, 0, 0)
        base = self.storage.data_ptr()
        n = self.H * cap * 128 * 2
        kraw = self.storage[kp - base:kp - base + n].view(torch.bfloat16).view(self.H, cap, 128)
        vraw = self.storage[vp - base:vp - base + n].view(torch.bfloat16).view(self.H, 128, cap)
        ids = self.storage[ip - base:ip - base + cap * 8].view(torch.int64)
        ns = self.S + self.W
        K = kraw.permute(1, 0, 2).reshape(cap, self.C)[:ns].float().cpu().numpy()
        vraw = vraw[:, :, binding.vt_columns(cap).to(vraw.device)]
        V = vraw.permute(2, 0, 1).reshape(cap, self.C)[:ns].float().cpu().numpy()
        return K, V, ids[:ns].cpu().numpy()

    def check_exact(self):
        """Cache contents, device ids, host slot map and counters against the oracle, bit for bit."""
        torch.cuda.synchronize()
        K, V, ids = self.logical()
        want = self.ora.slot_map()
        live = want >= 0
        ko, vo = self.ora.slot_contents()
        assert np.array_equal(ids[live], want[live])
        assert np.array_equal(np.asarray(binding.kv_cache_slot_map(self.handle, 0, 0, self.S + self.W)), want)
        assert np.array_equal(K[live], ko[live]) and np.array_equal(V[live], vo[live])
        assert binding.kv_cache_state(self.handle, 0, 0) == self.ora.state()

    def close(self):
        binding.kv_cache_destroy(self.handle)


def mixed(pair, base, weight):
    """Rows that are `weight` parts of `base` and the rest fresh noise: cosine to `base` near `weight`-dependent."""
    noise = pair.rows(base.shape[0]).float()
    return (weight * base.float() + (1.0 - weight) * noise).to(torch.bfloat16)


@pytest.mark.parametrize("H,P,sink_frames,window_frames,fpc", [
    (2, 15, 2, 4, 2),          # frame starts at every residue mod 16 of the V^T column permutation, two sinks
    (3, 64, 1, 3, 1),          # aligned frames
    (1, 40, 3, 5, 3),          # three sinks, three-frame chunks (frame_back 0 .. 2)
])
def test_similarity_refresh_and_eviction_small(H, P, sink_frames, window_frames, fpc):
    pair = CachePair(H, P, sink_frames, window_frames, seed=H * 100 + P)
    sink_v = pair.rows(sink_frames * P)
    # fill the sink in chunk-sized appends
    n_fill = 0
    while n_fill < sink_frames * P:
        n = min(fpc * P, sink_frames * P - n_fill)
        pair.append(pair.rows(n), sink_v[n_fill:n_fill + n])
        n_fill += n
    seen = []
    for chunk in range(2 * window_frames):
        # each frame of the chunk resembles one of the sink frames to a different degree
        vs = []
        for f in range(fpc):
            i = (chunk + f) % sink_frames
            vs.append(mixed(pair, sink_v[i * P:(i + 1) * P], weight=[0.9, 0.5, 0.1][(chunk + f) % 3]))
        pair.append(pair.rows(fpc * P, scale=3.0), torch.cat(vs))
        for back in range(fpc):
            got, want = pair.similarity(back)
            assert np.abs(got - want).max() <= 2e-5, (chunk, back, got, want)
            seen.extend(want.tolist())
        if chunk % 2 == 1:
            # the rule of Section 4.1 with tau = 0.6, decided from the library's alpha
            got, want = pair.similarity(0)
            assert [a >= 0.6 for a in got] == [a >= 0.6 for a in want]
            for i, a in enumerate(got):
                if not a >= 0.6:
                    binding.kv_cache_refresh_sink(pair.handle, 0, 0, i, 0)
                    oracle.refresh_sink(pair.ora, i, 0)
                    sink_v[i * P:(i + 1) * P] = vs[-1]
        pair.check_exact()
    assert pair.ora.state()["evicted"] > 0
    assert max(seen) > 0.9 and min(seen) < 0.3 and any(0.4 < a < 0.8 for a in seen)     # the cases span the range
    pair.close()


def test_refresh_closes_the_chunk_and_rejects_bad_calls():
    pair = CachePair(2, 16, 1, 3)
    k, v = pair.rows(16), pair.rows(16)
    with pytest.raises(binding.Sdv2Error) as e:                      # nothing appended, sink empty
        binding.sink_similarity(pair.handle, 0, 0, pair.alpha, pair.ws)
    assert e.value.code == binding.BAD_STATE
    pair.append(k, v)                                                # this frame IS the sink
    for call in (lambda: binding.sink_similarity(pair.handle, 0, 0, pair.alpha, pair.ws),
                 lambda: binding.kv_cache_refresh_sink(pair.handle, 0, 0, 0, 0)):
        with pytest.raises(binding.Sdv2Error) as e:
            call()
        assert e.value.code == binding.BAD_STATE
    pair.append(pair.rows(32), pair.rows(32))
    for bad in (lambda: binding.sink_similarity(pair.handle, 0, 0, pair.alpha, pair.ws, 2),      # frame_back
                lambda: binding.sink_similarity(pair.handle, 0, 0, pair.alpha, pair.ws, -1),
                lambda: binding.kv_cache_refresh_sink(pair.handle, 0, 0, 1, 0),                  # sink_frame
                lambda: binding.kv_cache_refresh_sink(pair.handle, 1, 0, 0, 0)):                 # layer
        with pytest.raises(binding.Sdv2Error) as e:
            bad()
        assert e.value.code == binding.INVALID_ARG
    with pytest.raises(binding.Sdv2Error) as e:
        binding.sink_similarity(pair.handle, 0, 0, pair.alpha, pair.ws[:16])
    assert e.value.code == binding.WORKSPACE_TOO_SMALL
    pair.check_exact()                                               # none of the refused calls changed anything
    k2, v2 = pair.rows(32), pair.rows(32)
    pair.append(k2, v2, advance=False)                               # a second denoising step: fine
    binding.kv_cache_refresh_sink(pair.handle, 0, 0, 0, 1)
    oracle.refresh_sink(pair.ora, 0, 1)
    pair.check_exact()
    with pytest.raises(binding.Sdv2Error) as e:                      # the chunk is closed now
        binding.kv_cache_append_evict(pair.handle, 0, 0, k2.to(DEV), v2.to(DEV), False)
    assert e.value.code == binding.BAD_STATE
    with pytest.raises(RuntimeError):
        pair.ora.append_evict(k2.double().numpy(), v2.double().numpy(), advance=False)
    pair.append(k2, v2)
    pair.append(k2, v2, advance=False)
    pair.check_exact()
    pair.close()


def test_rotate_keys_small_against_oracle_and_unfilled_slots_untouched():
    pair = CachePair(2, 24, 1, 4, seed=7)
    pair.append(pair.rows(24), pair.rows(24))
    pair.append(pair.rows(48), pair.rows(48))                       # window half full
    before = pair.storage.clone()
    for delta in (5, -12, 1000):
        binding.kv_cache_rotate_keys(pair.handle, 0, 0, delta)
        oracle.rotate_keys(pair.ora, delta, pair.H)
        torch.cuda.synchronize()
        K, V, ids = pair.logical()
        want = pair.ora.slot_map()
        live = want >= 0
        ko, vo = pair.ora.slot_contents()
        assert max_rel_err(K[live], ko[live]) <= 1e-2          # three moves, one bf16 rounding each
        assert np.array_equal(V[live], vo[live]) and np.array_equal(ids[live], want[live])
    # slots that hold nothing still carry the 0xFF bytes they were created with
    kp, vp, ip, cap = binding.kv_cache_device_ptrs(pair.handle, 0, 0)
    base = pair.storage.data_ptr()
    kraw = pair.storage[kp - base:kp - base + pair.H * cap * 256].view(pair.H, cap, 256)
    kraw0 = before[kp - base:kp - base + pair.H * cap * 256].view(pair.H, cap, 256)
    empty = torch.from_numpy(np.nonzero(pair.ora.slot_map() < 0)[0]).to(DEV)
    assert torch.equal(kraw[:, empty], kraw0[:, empty]) and bool((kraw[:, empty] == 0xFF).all())
    assert torch.equal(kraw[:, pair.S + pair.W:], kraw0[:, pair.S + pair.W:])
    pair.close()


def test_stream_with_sink_refresh_and_rope_reset_through_the_block():
    """Block on both sides: chunks until eviction, then an adaptive sink update decided from the library's alpha,
    then a RoPE reset (cached keys moved by T_reset frames, the next chunk at the lowered frame index)."""
    wl = wk.Workload("refresh", C=256, H=2, F=384, grid_h=3, grid_w=5, frames_per_chunk=2, sink_frames=2,
                     window_frames=4, L_t=20, B=1, N=2, steps=(1,), chunks=8)
    gpu = GpuRunner(wl)
    ora = OracleRunner(wl)
    ws = torch.empty(binding.sink_similarity_workspace_bytes(gpu.cache), dtype=torch.uint8, device=gpu.device)
    alpha = torch.empty(2, dtype=torch.float32, device=gpu.device)
    shift = 0
    t_reset = 7
    for chunk in range(8):
        frame0 = chunk * wl.frames_per_chunk
        if frame0 - shift > t_reset:                                 # theta_t = theta_{t - T_reset}
            shift += t_reset
            for layer in range(wl.N):
                binding.kv_cache_rotate_keys(gpu.cache, layer, 0, t_reset)
                oracle.rotate_keys(ora.caches[layer][0], t_reset, wl.H)
        desc = (0, frame0 - shift, wl.frames_per_chunk, 1)
        x = wk.chunk_input(wl, chunk, 0)
        t = wk.timestep(wl, chunk, 0, 0)
        xg = x.to(gpu.device).reshape(1, wl.L, wl.C).contiguous()
        gpu.denoise(xg, [desc], timesteps=[t])
        xo = ora.denoise(x.double().numpy(), desc, timestep=t)
        torch.cuda.synchronize()
        assert max_rel_err(xg[0].cpu().numpy(), xo) <= 2e-2, chunk
        if chunk >= 1:
            for layer in range(wl.N):
                binding.sink_similarity(gpu.cache, layer, 0, alpha, ws, 0)
                torch.cuda.synchronize()
                got = alpha.cpu().numpy().astype(np.float64)
                want = oracle.sink_similarity(ora.caches[layer][0], 0)
                assert np.abs(got - want).max() <= 5e-3, (chunk, layer, got, want)
                if chunk in (3, 6):                                  # tau above every alpha: refresh the least similar
                    i = int(np.argmin(want))
                    binding.kv_cache_refresh_sink(gpu.cache, layer, 0, i, 0)
                    oracle.refresh_sink(ora.caches[layer][0], i, 0)
        for layer in range(wl.N):
            oc = ora.caches[layer][0]
            assert gpu.state(layer, 0) == oc.state()
            assert np.array_equal(gpu.slot_map(layer, 0), oc.slot_map())
            K, V, ids = gpu.cache_logical(layer, 0)
            live = oc.slot_map() >= 0
            ko, vo = oc.slot_contents()
            assert np.array_equal(ids[live], oc.slot_map()[live])
            assert max_rel_err(K[live], ko[live]) <= 1e-2 and max_rel_err(V[live], vo[live]) <= 1e-2
    assert shift == t_reset
    gpu.close()


@pytest.mark.parametrize("name", ["wan1.3b-block", "wan14b-480p-b4"])
def test_refresh_kernels_at_full_cache_sizes(name):
    """One (layer, stream) cache of the 1.3B block (1024-token frames) and of the batched 480p workload (1560-token
    frames, 40 heads, 10920 slots): similarity, copy and key move on a full, wrapped cache."""
    wl = wk.WORKLOADS[name]
    pair = CachePair(wl.H, wl.P, wl.S // wl.P, wl.W // wl.P, seed=11)
    n = wl.frames_per_chunk * wl.P
    sink_v = pair.rows(wl.S)
    pair.append(pair.rows(wl.S), sink_v)
    n_chunks = wl.W // n + 2                                          # fill the window and wrap
    for chunk in range(n_chunks):
        v = torch.cat([mixed(pair, sink_v[:wl.P], 0.3 + 0.2 * f) for f in range(wl.frames_per_chunk)])
        pair.append(pair.rows(n), v)
    assert pair.ora.state()["evicted"] > 0
    for back in range(wl.frames_per_chunk):
        got, want = pair.similarity(back)
        assert np.abs(got - want).max() <= 2e-5 and want.max() > 0.2, (back, got, want)
    binding.kv_cache_refresh_sink(pair.handle, 0, 0, 0, 0)
    oracle.refresh_sink(pair.ora, 0, 0)
    pair.check_exact()
    binding.kv_cache_rotate_keys(pair.handle, 0, 0, 37)
    torch.cuda.synchronize()
    K, V, ids = pair.logical()
    ko0, vo0 = pair.ora.slot_contents()
    # the oracle's rotation, on sampled slots (it turns one row at a time)
    sample = np.unique(np.concatenate([np.arange(0, 8), np.arange(wl.S - 4, wl.S + 4),
                                       np.random.default_rng(0).integers(0, wl.S + wl.W, 64),
                                       np.arange(wl.S + wl.W - 8, wl.S + wl.W)]))
    pos = np.array([[-37, 0, 0]], dtype=np.float64)
    for slot in sample:
        want = oracle.rope_3d(ko0[slot].reshape(1, wl.H, 128), pos).reshape(-1)
        assert np.abs(K[slot] - want).max() <= 1e-2 * np.abs(want).max(), slot
    assert np.array_equal(V, vo0)
    pair.close()


@pytest.mark.parametrize("H,P", [(40, 2048), (40, 777), (12, 1560)])
def test_similarity_of_many_heads_is_a_single_precision_number(H, P):
    """alpha against 64 bits on the same bf16 rows: its own rounding to single precision (2^-25 for values in [1/2, 1)) and
    2e-8 for the partial sums.  Sums of a whole row per lane are 6e-8 off at 40 heads of 2048 tokens."""
    binding.load_library()
    cf = binding.cache_cfg(1, 1, H, P, P, 2 * P)
    storage = torch.zeros(binding.kv_cache_bytes(cf), dtype=torch.uint8, device=DEV)
    g = torch.Generator(device=DEV)
    for seed in range(8):
        g.manual_seed(seed)
        h = binding.kv_cache_init(cf, storage)
        sink = torch.randn((P, 128 * H), generator=g, device=DEV).to(torch.bfloat16)
        new = (0.6 * sink.float() + 0.4 * torch.randn((P, 128 * H), generator=g, device=DEV)).to(torch.bfloat16)
        for rows in (sink, new):
            binding.kv_cache_append_evict(h, 0, 0, rows, rows)
        alpha = torch.empty(1, device=DEV)
        ws = torch.empty(binding.sink_similarity_workspace_bytes(h), dtype=torch.uint8, device=DEV)
        binding.sink_similarity(h, 0, 0, alpha, ws)
        x, y = new.double().flatten(), sink.double().flatten()
        want = ((x @ y) / (x.norm() * y.norm())).item()
        assert 0.5 < want < 1.0
        assert abs(alpha.item() - want) <= 2.0 ** -25 + 2e-8, (seed, alpha.item() - want)
        binding.kv_cache_destroy(h)


def test_refresh_of_more_heads_than_a_grid_has_rows():
    """70 000 heads of two tokens per frame: the rotation is launched in two ranges of heads, the copy in one."""
    H, P = 70000, 2
    binding.load_library()
    cf = binding.cache_cfg(1, 1, H, P, P, 2 * P)
    storage = torch.zeros(binding.kv_cache_bytes(cf), dtype=torch.uint8, device=DEV)
    h = binding.kv_cache_init(cf, storage)
    g = torch.Generator(device=DEV).manual_seed(3)
    rows = [torch.randn((P, 128 * H), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2)]
    for r in rows:
        binding.kv_cache_append_evict(h, 0, 0, r, r)
    _, _, _, cap = binding.kv_cache_device_ptrs(h, 0, 0)
    K = storage[:H * cap * 256].view(torch.bfloat16).view(H, cap, 128)
    new = rows[1].view(P, H, 128).permute(1, 0, 2)
    binding.kv_cache_refresh_sink(h, 0, 0, 0)
    assert torch.equal(K[:, :P], new) and torch.equal(K[:, P:2 * P], new)
    binding.kv_cache_rotate_keys(h, 0, 0, 5)
    torch.cuda.synchronize()
    n = oracle.dit_block.rope_pair_split(128)[0]
    angle = -5.0 * oracle.dit_block.ROPE_BASE ** (-torch.arange(n, device=DEV, dtype=torch.float64) / n)
    x = new.double().reshape(H, P, 64, 2)
    want = x.clone()
    want[:, :, :n, 0] = x[:, :, :n, 0] * angle.cos() - x[:, :, :n, 1] * angle.sin()
    want[:, :, :n, 1] = x[:, :, :n, 0] * angle.sin() + x[:, :, :n, 1] * angle.cos()
    for s0 in (0, P):
        got = K[:, s0:s0 + P].double().reshape(H, P, 64, 2)
        assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-6).all()       # one rounding to bf16 (the sums' fp32 below it)
    binding.kv_cache_destroy(h)
