"""Host images go up in one launch for a stream's cameras or in one each, from
256 KiB a camera on: streams on both sides of the line, just at and below it, give
the records and pyramids of device images."""
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
