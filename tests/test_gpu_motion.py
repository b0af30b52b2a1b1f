"""GPU parity of the motion-aware noise scheduler (Section 4.1) against the CPU oracle.

The same fp32 latent frames go to both sides.  The library adds the squared differences in fp32 (partial sums,
then double) where the oracle uses float64 throughout: bar 1e-5 relative on d_t, 1e-5 absolute on dhat_t and s_t
(a value of d_t that lands within rounding of the clip point or of the window maximum moves dhat_t by no more than
that)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2511_07399_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_stream(shape, chunks, k, sigma, lam, s_min, s_max, s_init, frame_fn, offset_elems=0):
    """Feeds `chunks` (list of frames-per-call) to the library and every frame to the oracle; returns both traces."""
    binding.load_library()
    n = int(np.prod(shape))
    cfg = binding.motion_cfg(k, sigma, lam, s_min, s_max, s_init)
    state = torch.empty(binding.motion_state_bytes(cfg), dtype=torch.uint8, device=DEV)
    binding.motion_init(cfg, state)
    sch = oracle.MotionNoiseScheduler(k, sigma, lam, s_min, s_max, s_init)
    got, want = [], []
    prev = None
    t = 0
    for T in chunks:
        frames = torch.stack([frame_fn(t + i) for i in range(T)]).reshape(T, n).float()
        buf = torch.empty(T * n + offset_elems, dtype=torch.float32, device=DEV)
        fd = buf[offset_elems:].view(T, n)
        fd.copy_(frames)
        outs = [torch.empty(T, dtype=torch.float32, device=DEV) for _ in range(3)]
        binding.motion_update(cfg, state, fd, prev, *outs)
        torch.cuda.synchronize()
        for i in range(T):
            got.append(tuple(float(o[i]) for o in outs))
            want.append(sch.step(frames[i].double().numpy()))
        prev = fd[T - 1].clone()
        t += T
    return np.array(got), np.array(want)


def check(got, want):
    assert np.abs(got[:, 0] - want[:, 0]).max() <= 1e-5 * max(want[:, 0].max(), 1e-30), (got[:, 0], want[:, 0])
    assert np.abs(got[:, 1] - want[:, 1]).max() <= 1e-5
    assert np.abs(got[:, 2] - want[:, 2]).max() <= 1e-5


@pytest.mark.parametrize("shape,chunks", [
    ((16, 64, 64), [1, 1, 4, 4, 3, 1, 4, 2]),          # 512 x 512 latents, chunks of up to four frames
    ((16, 60, 104), [4, 4, 4, 4, 4]),                  # 480 x 832
    ((3, 5, 7), [2, 16, 5]),                           # a size that is not a multiple of four: scalar loads
    ((16, 64, 64), [3] * 6),
])
def test_random_motion_stream(shape, chunks):
    gen = torch.Generator().manual_seed(sum(shape))
    base = torch.randn(shape, generator=gen)
    # a slowly moving scene with bursts: amplitude of the change varies from frame to frame
    amps = [0.02, 0.5, 0.05, 1.5, 0.01, 0.3, 0.0, 0.8]
    frames = {}

    def frame_fn(t):
        if t not in frames:
            prev = base if t == 0 else frames[t - 1]
            frames[t] = prev + amps[t % len(amps)] * torch.randn(shape, generator=gen)
        return frames[t]

    off = 1 if shape == (16, 64, 64) and chunks[0] == 3 else 0     # a buffer that is not 16-byte aligned
    got, want = run_stream(shape, chunks, k=3, sigma=1.2, lam=0.3, s_min=0.1, s_max=0.9, s_init=0.5, frame_fn=frame_fn,
                           offset_elems=off)
    check(got, want)
    # the stream reaches the clip and also sits strictly inside (0, 1)
    assert want[:, 1].max() == 1.0 and np.any((want[:, 1] > 0.05) & (want[:, 1] < 0.95))


def test_static_stream_and_spike():
    shape = (16, 32, 32)
    base = torch.randn(shape, generator=torch.Generator().manual_seed(1))
    got, want = run_stream(shape, [4, 4, 4], k=2, sigma=2.0, lam=0.2, s_min=0.1, s_max=0.8, s_init=0.3,
                           frame_fn=lambda t: base)
    check(got, want)
    assert np.all(got[:, 0] == 0.0) and np.all(got[:, 1] == 0.0)
    closed = 0.8 - (0.8 - 0.3) * (1 - 0.2) ** np.arange(1, 13)
    assert np.abs(got[:, 2] - closed).max() <= 1e-6
    # one jump by 1.0 at frame 5: d = 1, held in the window for k + 1 = 3 frames, then gone
    got, want = run_stream(shape, [4, 4, 4], k=2, sigma=2.0, lam=0.5, s_min=0.0, s_max=1.0, s_init=1.0,
                           frame_fn=lambda t: base + (1.0 if t >= 5 else 0.0))
    check(got, want)
    assert list(np.round(got[:, 1], 6)) == [0, 0, 0, 0, 0, 0.5, 0.5, 0.5, 0, 0, 0, 0]


@pytest.mark.parametrize("k,chunks", [(0, [16, 16]), (8, [16, 5, 16]), (63, [16] * 5), (64, [16] * 5), (100, [16] * 8), (1023, [7, 16])])
def test_sixteen_frames_a_call_and_long_windows(k, chunks):
    """The most frames a call takes, windows below, at and above a wavefront's width, rings that wrap inside a call; one jump
    early in the stream that a long window holds on to and a short one forgets."""
    shape = (3, 5, 7)
    gen = torch.Generator().manual_seed(k)
    frames = [torch.randn(shape, generator=gen)]
    for t in range(1, sum(chunks)):
        frames.append(frames[-1] + (1.5 if t == 4 else 0.1 + 0.3 * (t % 7 == 0)) * torch.randn(shape, generator=gen))
    got, want = run_stream(shape, chunks, k=k, sigma=2.0, lam=0.3, s_min=0.1, s_max=0.9, s_init=0.5, frame_fn=lambda t: frames[t])
    check(got, want)


def test_motion_call_validation():
    binding.load_library()
    good = binding.motion_cfg(3, 1.0, 0.5, 0.1, 0.9, 0.5)
    for bad in (binding.motion_cfg(-1, 1.0, 0.5, 0.1, 0.9, 0.5), binding.motion_cfg(3, 0.0, 0.5, 0.1, 0.9, 0.5),
                binding.motion_cfg(3, 1.0, 1.0, 0.1, 0.9, 0.5), binding.motion_cfg(3, 1.0, 0.5, 0.9, 0.1, 0.5)):
        assert binding.motion_state_bytes(bad) == 0
    state = torch.empty(binding.motion_state_bytes(good), dtype=torch.uint8, device=DEV)
    binding.motion_init(good, state)
    frames = torch.zeros(17, 64, device=DEV)
    outs = [torch.empty(17, dtype=torch.float32, device=DEV) for _ in range(3)]
    with pytest.raises(binding.Sdv2Error) as e:
        binding.motion_update(good, state, frames, None, *outs)            # more than 16 frames in one call
    assert e.value.code == binding.INVALID_ARG
    with pytest.raises(binding.Sdv2Error) as e:
        binding.motion_update(good, state[:64], frames[:4], None, *outs)
    assert e.value.code == binding.WORKSPACE_TOO_SMALL
    with pytest.raises(binding.Sdv2Error) as e:
        binding.motion_init(binding.motion_cfg(3, -1.0, 0.5, 0.1, 0.9, 0.5), state)
    assert e.value.code == binding.INVALID_ARG


def test_wave_sums_add_the_halves_first():
    """The order of a sum over a wavefront: lanes 32 apart, then 16, 8, 4, 2, 1.  Seen in the partial sums that the state
    keeps behind its header (16 floats) and ring (k + 1 floats, rounded up to 16): 64 per frame, one per workgroup.  Every
    lane holds one squared difference that is exact in single precision."""
    binding.load_library()
    k, n = 3, 64 * 256 * 4
    cfg = binding.motion_cfg(k, 1.0, 0.5, 0.1, 0.9, 0.5)
    state = torch.empty(binding.motion_state_bytes(cfg), dtype=torch.uint8, device=DEV)
    binding.motion_init(cfg, state)
    d = torch.zeros(n // 4, 4)
    d[:, 0] = torch.randint(1, 4096, (n // 4,), generator=torch.Generator().manual_seed(9)).float() / 64.0
    outs = [torch.empty(1, dtype=torch.float32, device=DEV) for _ in range(3)]
    binding.motion_update(cfg, state, d.reshape(1, n).to(DEV), torch.zeros(n, device=DEV), *outs)
    torch.cuda.synchronize()
    got = state.view(torch.float32)[32:32 + 64].cpu().numpy()
    v = (d[:, 0].numpy() ** 2).reshape(64, 4, 64)
    for off in (32, 16, 8, 4, 2, 1):
        v = v + v[:, :, np.arange(64) ^ off]
    want = (v[:, 0, 0] + v[:, 1, 0]) + (v[:, 2, 0] + v[:, 3, 0])
    assert v.dtype == np.float32 and np.array_equal(got, want)
