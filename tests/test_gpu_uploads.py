"""Host images go up in one launch for a stream's cameras or in one each, from
256 KiB a camera on, or from 1.5 MiB a frame where several streams are staged: frames
on both sides of the lines, just at and below them, give the records and pyramids of
device images."""
import pytest

import synthgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,cams", [(512, 511, 2), (512, 512, 2), (449, 512, 4), (449, 511, 4), (320, 240, 2),
                                      (250, 190, 4), (16, 16, 2)])
def test_host_equals_device_images(w, h, cams):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    seqs = [synthgen.render(seed=w + h + i, width=w, height=h, n_frames=3, stereo=True, density=6.0, max_scale=0.01)
            for i in range(cams // 2)]
    levels = 4 if w > 32 else 2
    frames = [[im for s in seqs for im in s.frames[t]] for t in range(3)]
    got = []
    for host in (True, False):
        out = []
        with vf.Frontend([(cams, w, h, 200, 32)], vf.make_params(levels=levels)) as fe:
            for t in range(3):
                if host:
                    fe.push_stereo_frame(0, t + 1, frames[t])
                else:
                    fe.push_stereo_frame_device(0, t + 1, [torch.from_numpy(im).cuda() for im in frames[t]])
                out.append(fe.get_tracks(0).tobytes())
                out += [fe.get_pyramid(0, c, l).tobytes() for c in range(cams) for l in range(levels)]
        got.append(out)
    assert got[0] == got[1]


@pytest.mark.parametrize("sizes", [[(2, 512, 512), (2, 1024, 767)], [(2, 1024, 768), (1, 320, 240)],
                                   [(4, 768, 512), (4, 768, 511)]])
def test_staged_among_streams(sizes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_30459_amd as vf
    frames = []
    for n, (c, w, h) in enumerate(sizes):
        s = synthgen.render(seed=n + w, width=w, height=h, n_frames=3, stereo=True, density=3.0, max_scale=0.01)
        frames.append([[s.frames[t][k % 2] for k in range(c)] for t in range(3)])
    got = []
    for host in (True, False):
        out = []
        with vf.Frontend([(c, w, h, 200, 32) for c, w, h in sizes], vf.make_params()) as fe:
            for t in range(3):
                for i, f in enumerate(frames):
                    if host:
                        fe.stage_frame(i, t + 1, f[t])
                dev = [torch.from_numpy(im).cuda() for f in frames for im in f[t]]
                if not host:
                    fe.stage_frames_device(list(range(len(sizes))), [t + 1] * len(sizes), dev)
                fe.step()
                out += [fe.get_tracks(i).tobytes() for i in range(len(sizes))]
                out += [fe.get_pyramid(i, c, 0).tobytes() for i, z in enumerate(sizes) for c in range(z[0])]
        got.append(out)
    assert got[0] == got[1]
