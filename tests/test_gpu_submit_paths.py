"""Every way to submit a frame gives the same records: host images pushed
(linear uploads at the level's pitch, whatever the width), device images pushed
on the handle's and on a caller's stream, staged and stepped, staged and stepped
asynchronously, and pushes among frames in flight or staged host images."""
import numpy as np
import pytest

import synthgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("w,h,cams", [(320, 240, 1), (360, 255, 1), (641, 479, 2), (752, 480, 2), (1030, 700, 2)])
@pytest.mark.parametrize("extra", [{}, {"plain": True}, {"eager": True}, {"pyramid_stream": 1}, {"pyramid_stream": 2},
                                   {"stereo_mode": 1}])
def test_submit_paths_agree(w, h, cams, extra):
    import torch
    import paper_2609_30459_amd as vf
    seq = synthgen.render(seed=w * 7 + h, width=w, height=h, n_frames=5, stereo=cams == 2, density=4.0, max_scale=0.01)
    dev = torch.from_numpy(seq.frames).cuda()
    side = torch.cuda.Stream()

    def padded(im):  # rows further apart than the width
        wide = np.full((h, w + 13), 255, np.uint8)
        wide[:, :w] = im
        return wide[:, :w]

    def host(fe, t):
        fe.push_stereo_frame(0, t + 1, list(seq.frames[t]))

    def device(fe, t):
        fe.push_stereo_frame_device(0, t + 1, list(dev[t]))

    def caller_stream(fe, t):
        fe.push_stereo_frame_device(0, t + 1, list(dev[t]), hip_stream=side)

    def step_host(fe, t):
        fe.stage_frame(0, t + 1, [padded(im) for im in seq.frames[t]])
        fe.step()

    def step_device(fe, t):
        fe.stage_frame_device(0, t + 1, list(dev[t]))
        fe.step()

    def asynchronous(fe, t):
        fe.stage_frame_device(0, t + 1, list(dev[t]))
        fe.step_async()
        fe.wait()

    def mixed(fe, t):
        [host, asynchronous, caller_stream, step_host, device][t](fe, t)

    want = None
    for how in (host, device, caller_stream, step_host, step_device, asynchronous, mixed):
        with vf.Frontend([(cams, w, h)], vf.make_params(max_keypoints=200, cell_size=32, **extra)) as fe:
            got = []
            for t in range(5):
                how(fe, t)
                got.append(fe.get_tracks(0).tobytes())
        want = want or got
        assert got == want, how.__name__
    assert len(want[-1]) > 40 * 40


def test_push_among_frames_in_flight_and_staged_host_images():
    """Two streams: a push on one with the other's frame in flight, or with its
    host images staged for a later step (queued on the other stream)."""
    import paper_2609_30459_amd as vf
    seq = synthgen.render(seed=5, width=400, height=301, n_frames=5, stereo=True, density=4.0, max_scale=0.01)
    streams = [(2, 400, 301)] * 2
    p = vf.make_params(max_keypoints=200, cell_size=32)
    with vf.Frontend(streams, p) as a, vf.Frontend(streams, p) as b:
        for t in range(5):
            fr = list(seq.frames[t])
            for s in (0, 1):
                b.push_stereo_frame(s, t + 1, fr)
            a.stage_frame(0, t + 1, fr)
            if t % 2:
                a.step_async()
                a.push_stereo_frame(1, t + 1, fr)
            else:
                a.push_stereo_frame(1, t + 1, fr)
                a.step()
            for s in (0, 1):
                assert a.get_tracks(s).tobytes() == b.get_tracks(s).tobytes(), (t, s)


@pytest.mark.parametrize("learned", [False, True])
def test_sixty_four_cameras_partly_staged(learned):
    """The most cameras a handle can have, of two sizes, with every third stream
    left out of each step: the records are those of pushing each stream alone."""
    import paper_2609_30459_amd as vf
    seqs = [synthgen.render(seed=s, width=64 + 16 * s, height=48 + 9 * s, n_frames=4, density=4.0) for s in (0, 1, 2)]
    streams = [(1,) + seqs[s % 3].size + (20 + s % 7, 16) for s in range(64)]
    kw = dict(init_mode=1, learned_levels=2, learned_iters=3, learned_rho=0.05) if learned else {}
    p = vf.make_params(levels=3, **kw)
    with vf.Frontend(streams, p) as a, vf.Frontend(streams, p) as b:
        if learned:
            rng = np.random.default_rng(3)
            params = rng.normal(0, 0.02, vf.MLP_NPARAM).astype(np.float32)
            a.set_mlp(params)
            b.set_mlp(params)
        at = [0] * 64
        for t in range(4):
            now = [s for s in range(64) if (s + t) % 3]
            for s in now:
                im = [seqs[s % 3].frames[at[s], 0]]
                at[s] += 1
                a.stage_frame(s, t + 1, im)
                b.push_stereo_frame(s, t + 1, im)
            a.step()
            for s in now:
                assert a.get_tracks(s).tobytes() == b.get_tracks(s).tobytes(), (t, s)
